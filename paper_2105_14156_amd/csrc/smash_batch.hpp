// smash_batch.hpp -- kernels of the batched launch: many independent
// products C_p = A_p * B_p run as one pipeline over the concatenated row
// space of all problems.
//
// Global row g of the batch is row g - row0[p] of problem p.  Every kernel
// has a fixed grid (sized from the batch's row count or the machine), reads
// the bin sizes it needs from device memory and loops over its work items,
// so the whole sequence can be captured once in a graph and replayed with no
// host synchronisation: analysis, binning, symbolic per bin, one row-pointer
// scan over the batch (each C_p lands at a device-computed offset of one
// output pool), numeric per bin.  Rows whose bound exceeds the LDS hash
// limit are counted in an LDS bitmap over B's columns and merged at the ranks
// of such a bitmap (up to kRankMaxCols columns) or accumulated in LDS windows
// of columns (wide_rank_row); per-row global tables only for problems wider
// than kWideMaxCols columns.
#pragma once

#include <hip/hip_runtime.h>

#include "smash_kernels.hpp"

namespace smash {

struct BatchDesc {
    const int *Arp, *Acol;
    const void *Aval;
    const int *Brp, *Bcol;
    const void *Bval;
    int rows, cols;
    long long row0;             // first global row of the problem
};

struct BatchHdr {
    BinHdr sym, num;
    unsigned long long products;
    long long nnz_c;            // total entries of all C_p
    long long gneed;            // global table slots of the heavy rows
    int error;
    int windows;                // a heavy row may take the windowed numeric kernel (k_bwindows)
    int rank_queue;             // next heavy row of the bitmap numeric kernel
    int wide_queue;             // next heavy row of the windowed numeric kernel
};

// Heavy rows of problems with at most kWideMaxCols columns are counted with
// an LDS bitmap over all columns and merged by bitmap ranks or, where that
// would take too many passes over their products and beyond kRankMaxCols
// columns, in LDS windows of kWideWin columns; wider problems use per-row
// global tables.
constexpr int kWideMaxCols = 1 << 20;
constexpr int kWideWin = 8192;
constexpr int kWideThreads = 512;

// Whether a heavy row of nc entries, with `entries` A entries and `products`
// products in a problem of `cols` columns, is merged by the column bitmap,
// kWideCap entries at a time (k_bnum_wide_rank), or in windows (k_bnum_wide).
// The bitmap's prefix counts are 16 bits wide, so a row of 65536 entries takes
// the windows.  So does a row whose products the bitmap form would go through
// too often: it does so once per kWideCap entries (the first time costs little
// more than in the windows), where the windows take each product once, but
// clear and scan 8192 slots per window, some 7000 products' time, and, with
// more than kWideThreads A entries, search every selected B row twice, 10
// products' time.  Those have to gain a third besides, since a few of them do
// not fill a launch of their own.  Replay of 1000 rows in us, bitmap and
// windows: 22500 products in 3000 columns 282 and 288, in 8192 columns 343 and
// 294, in 131072 columns 517 and 449; 10000 products there 255 and 323; 8000
// rows of 14000 products from 700 A entries, in 16384 columns 1477 and 1140, in
// 32768 columns 1480 and 1760.  RMAT scale 16, edge factor 16, A * A: 6.7 ms
// all by bitmap, 4.5 all in windows, 3.05 so.
constexpr int kWideCap = 3072;
constexpr int kWideRankThreads = 512;
constexpr int kWideWaves = kWideRankThreads / kWave;
constexpr int kWideRankMaxEntries = 65535;

__device__ __forceinline__ bool wide_rank_row(int cols, int nc, int entries, long long products)
{
    const long long passes = ((unsigned)nc + kWideCap - 1) / kWideCap, windows = ((unsigned)cols + kWideWin - 1) / kWideWin;
    const long long window = entries > kWideThreads ? 8192 + 16LL * entries : 7168;
    return cols <= kRankMaxCols && nc <= kWideRankMaxEntries && (5 * passes - 4) * products <= 5 * windows * window;
}

// What an LDS-bin kernel needs of one row, gathered in permutation order by
// k_browdesc so that the bin kernels read one contiguous record per row
// instead of a chain of dependent loads (row id, problem, row pointers,
// C offset).
struct RowDesc {
    int grow;                   // global row
    int prob;                   // problem
    int e0, e1;                 // the row's entries in A_p
    long long rb;               // C offset (numeric only)
    int nc;                     // C entries (numeric only)
    int pad;
};

// Table size class of a row bound: 2^LOGT >= bound << shift slots.
__device__ __forceinline__ int lds_bin_shift(long long bound, int shift)
{
    int lt = ceil_log2(bound << shift);
    return (lt < kMinLogT ? kMinLogT : lt) - kMinLogT;
}

// Problem of global row g: the last whose first row is not behind it
// (row0s[0] = 0, row0s[count] = M; problems without rows share a first row).
__device__ __forceinline__ int problem_of(const long long *__restrict__ row0s, int count, long long g)
{
    int lo = 0, hi = count;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (row0s[mid] <= g) lo = mid;
        else hi = mid;
    }
    return lo;
}

constexpr int kBatchShortRow = 128;   // entries of a row that eight lanes sum (k_banalyze)

// Blocks of k_banalyze that look for long rows, and all of them.
__host__ __device__ __forceinline__ int banalyze_long_blocks(long long M) { return (int)((M + 255) / 256) + 1; }
inline int banalyze_blocks(long long M) { return banalyze_long_blocks(M) + (int)((M + 255) / 256); }

// Per global row: its problem, products ub, bound cap = min(ub, cols), bin
// (empty, LDS by cap << shift, or heavy above lds_row_max) and, for heavy
// rows of problems wider than kWideMaxCols, its global table size.
//
// Bound by the latency of two dependent gathers per entry; the split is that
// of for_rows.  Rows of at most kBatchShortRow entries: a wave takes 64 consecutive
// rows, reads their bounds one per lane and sums them eight at a time, eight
// lanes each: in turn, hence a lower limit than there (four products of RMAT
// scale 16, edge factor 8, with a B of 8 entries per row: 41 us, with 256
// entries 65).  Longer rows: by a whole wave, eight entries per lane in flight,
// the rows a wave looks at an odd stride apart.  Batch of 512 RMAT pairs:
// 0.40 ms; with 64 consecutive rows per wave, the long ones (they come in
// clusters) in turn and one entry per lane in flight, 0.71.
__global__ __launch_bounds__(256) void k_banalyze(long long M, int count, const long long *__restrict__ row0s,
                                                  const BatchDesc *__restrict__ desc, int lds_row_max, int shift,
                                                  int *__restrict__ prob, long long *__restrict__ ub_out,
                                                  int *__restrict__ cap_out, int *__restrict__ nnzc,
                                                  unsigned char *__restrict__ bin_out, long long *__restrict__ gsz)
{
    const int lane = lane_id(), nl = banalyze_long_blocks(M);
    auto finish = [&](long long g, int pr, long long ub) {
        const int cols = desc[pr].cols;
        const int cap = (int)(ub < cols ? ub : cols);
        int b = kBinEmpty;
        if (ub > 0) {
            b = cap > lds_row_max ? kBinHeavy : lds_bin_shift(cap, shift);
            if (b >= kLdsBins) b = kBinHeavy;
        }
        prob[g] = pr;
        ub_out[g] = ub;
        cap_out[g] = cap;
        nnzc[g] = 0;
        bin_out[g] = (unsigned char)b;
        gsz[g] = b == kBinHeavy && cols > kWideMaxCols ? 1LL << gtable_log2(cap) : 0;
    };
    if ((int)blockIdx.x < nl) {
        const long long waves = (long long)nl * 4 - 1, w = (long long)blockIdx.x * 4 + threadIdx.x / kWave;
        if (w == waves) return;
        const long long g = (long long)lane * waves + w;
        int pr = 0, e0 = 0, e1 = 0;
        if (g < M) {
            pr = problem_of(row0s, count, g);
            const BatchDesc &d = desc[pr];
            e0 = d.Arp[g - d.row0];
            e1 = d.Arp[g - d.row0 + 1];
        }
        for (unsigned long long todo = __ballot(e1 - e0 > kBatchShortRow); todo; todo &= todo - 1) {
            const int src = __ffsll((long long)todo) - 1;
            const int f0 = __builtin_amdgcn_readlane(e0, src), f1 = __builtin_amdgcn_readlane(e1, src);
            const int lp = __builtin_amdgcn_readlane(pr, src);
            RowPart r;
            row_part<false, 8>(desc[lp].Acol, desc[lp].Brp, f0 + lane, f1, kWave, r);
            row_reduce<false>(r, kWave);
            if (lane == 0) finish((long long)src * waves + w, lp, r.ub);
        }
        return;
    }
    const long long base = ((long long)((int)blockIdx.x - nl) * 4 + threadIdx.x / kWave) * kWave;
    if (base >= M) return;
    const long long g = base + lane;
    int pr = problem_of(row0s, count, base), e0 = 0, e1 = 0;
    if (g < M) {
        while (row0s[pr + 1] <= g) ++pr;
        const BatchDesc &d = desc[pr];
        e0 = d.Arp[g - d.row0];
        e1 = d.Arp[g - d.row0 + 1];
    }
    const bool here = g < M && e1 - e0 <= kBatchShortRow;
    const int sl = lane & (kRowLanes - 1);
    long long ub = 0;
    for (int t = 0; t < kWave / kRowLanes; ++t) {
        const int src = t * kRowLanes + lane / kRowLanes;       // this group's row
        const int f0 = __shfl(e0, src, kWave), f1 = __shfl(e1, src, kWave), lp = __shfl(pr, src, kWave);
        RowPart r;
        if (f1 - f0 <= kBatchShortRow) row_part<false>(desc[lp].Acol, desc[lp].Brp, f0 + sl, f1, kRowLanes, r);
        row_reduce<false>(r, kRowLanes);
        const long long mine = __shfl(r.ub, sl * kRowLanes, kWave);
        if (lane / kRowLanes == t) ub = mine;
    }
    if (here) finish(g, pr, ub);
}

constexpr int kWideLong = 262144;

// Numeric bin of a heavy row: windows, or none of its own.
__device__ __forceinline__ int heavy_bin(const BatchDesc &d, long long g, int nc, long long products)
{
    const int *rp = d.Arp + (g - d.row0);
    if (d.cols > kWideMaxCols || wide_rank_row(d.cols, nc, rp[1] - rp[0], products)) return kBinHeavy;
    return products > kWideLong ? kBinWinLong : kBinWin;
}

// Whether a heavy row may take the windows, from the rows' bounds (when a plan
// is made or configured).
__global__ __launch_bounds__(256) void k_bwindows(long long M, const BatchDesc *__restrict__ desc,
                                                  const int *__restrict__ prob, const long long *__restrict__ ub,
                                                  const int *__restrict__ cap,
                                                  const unsigned char *__restrict__ sym_bin, int *windows)
{
    for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < M;
         g += (long long)gridDim.x * blockDim.x)
        if (sym_bin[g] == kBinHeavy && heavy_bin(desc[prob[g]], g, cap[g], ub[g]) != kBinHeavy) *windows = 1;
}

// Numeric bins from the exact counts: heavy rows stay heavy, rows without
// entries drop out, LDS rows take the class of their count.  Heavy rows that
// take the windows have bins of their own (windows: whether there may be any,
// as k_bwindows found, or rows of more entries than the bitmap form holds): those of more
// than kWideLong products come first, as each of them keeps a block busy for
// half a millisecond (RMAT scale 16, edge factor 16, A * A: 3.05 ms, 3.46 with
// all of them in row order; with rows numbered from another vertex 3.14, 3.65).
__global__ __launch_bounds__(256) void k_bnum_bins(long long M, int shift, const BatchDesc *__restrict__ desc,
                                                   const int *__restrict__ prob, const long long *__restrict__ ub,
                                                   const int *__restrict__ nnzc,
                                                   const unsigned char *__restrict__ sym_bin,
                                                   unsigned char *__restrict__ num_bin, bool windows)
{
    for (long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x; g < M;
         g += (long long)gridDim.x * blockDim.x) {
        const int nc = nnzc[g];
        int b = sym_bin[g];
        if (b < kLdsBins) b = nc ? lds_bin_shift(nc, shift) : kBinEmpty;
        if (windows && b == kBinHeavy) b = heavy_bin(desc[prob[g]], g, nc, ub[g]);
        num_bin[g] = (unsigned char)b;
    }
}

// Row records of the rows in the LDS bins of one binning (positions
// [0, offset[kLdsBins]) of perm), for k_bsym_rows / k_bnum_rows; with Crp
// non-NULL also their C offsets and counts.
__global__ __launch_bounds__(256) void k_browdesc(const BatchDesc *__restrict__ desc, const int *__restrict__ prob,
                                                  const BinHdr *h, const int *__restrict__ perm,
                                                  const long long *__restrict__ Crp, RowDesc *__restrict__ rd)
{
    const int n = h->offset[kLdsBins];
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x) {
        RowDesc o;
        o.grow = perm[r];
        o.prob = prob[o.grow];
        const BatchDesc &d = desc[o.prob];
        const int arow = (int)(o.grow - d.row0);
        o.e0 = d.Arp[arow];
        o.e1 = d.Arp[arow + 1];
        o.rb = Crp ? Crp[o.grow] : 0;
        o.nc = Crp ? (int)(Crp[o.grow + 1] - o.rb) : 0;
        o.pad = 0;
        rd[r] = o;
    }
}

// Symbolic, LDS bin `bin`: RPW rows of WPR waves per work item; the next
// item's row record is loaded while this one is processed.
template <int LOGT, int WPR, int RPW, bool SMALL = true>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_bsym_rows(const BatchDesc *__restrict__ desc,
                                                               const RowDesc *__restrict__ rd, const BinHdr *h,
                                                               int bin, int *__restrict__ nnzc, int *err)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    constexpr int G = WPR * kWave;
    __shared__ int s_keys[RPW][1 << LOGT];
    __shared__ EnumScratch<float, G> s_en[RPW];
    __shared__ int s_cnt[RPW];
    const int cnt = h->count[bin];
    const RowDesc *rows = rd + h->offset[bin];
    const int g = threadIdx.x / kWave / WPR;
    const int gt = threadIdx.x - g * G;
    const int stride = gridDim.x * RPW;
    int base = blockIdx.x * RPW;
    RowDesc cur{};
    if (base + g < cnt) cur = rows[base + g];
    for (; base < cnt; base += stride) {
        const bool active = base + g < cnt;
        RowDesc nxt{};
        if (base + stride + g < cnt) nxt = rows[base + stride + g];
        const BatchDesc &d = desc[active ? cur.prob : 0];
        sym_row<LOGT, WPR, SMALL>(cur.e0, cur.e1, d.Acol, d.Brp, d.Bcol, d.cols, active, gt, s_keys[g], s_en[g],
                                  &s_cnt[g], &nnzc[active ? cur.grow : 0], err);
        group_sync<WPR>();
        cur = nxt;
    }
}

// Numeric, LDS bin `bin` (row records with C offsets).  Does nothing when
// the output pool is too small (the capacity check has then flagged the
// batch).  HASH as in num_row (0 multiplicative, 1 order-preserving).
template <typename V, int LOGT, int WPR, int RPW, int HASH, bool SMALL = true>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_bnum_rows(const BatchDesc *__restrict__ desc,
                                                               const RowDesc *__restrict__ rd, const BatchHdr *bh,
                                                               int bin, long long ccap, int *__restrict__ Ccol,
                                                               V *__restrict__ Cval, int *err)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    constexpr int T = 1 << LOGT;
    constexpr int G = WPR * kWave;
    __shared__ int s_keys[RPW][T];
    __shared__ double s_vals[RPW][T];
    __shared__ EnumScratch<V, G> s_en[RPW];
    __shared__ int s_scan[RPW][WPR + 1];
    __shared__ int s_maxd[RPW];
    if (bh->nnz_c > ccap) return;
    const int cnt = bh->num.count[bin];
    const RowDesc *rows = rd + bh->num.offset[bin];
    const int g = threadIdx.x / kWave / WPR;
    const int gt = threadIdx.x - g * G;
    const int stride = gridDim.x * RPW;
    int base = blockIdx.x * RPW;
    RowDesc cur{};
    if (base + g < cnt) cur = rows[base + g];
    for (; base < cnt; base += stride) {
        const bool active = base + g < cnt;
        RowDesc nxt{};
        if (base + stride + g < cnt) nxt = rows[base + stride + g];
        const BatchDesc &d = desc[active ? cur.prob : 0];
        num_row<V, LOGT, WPR, HASH, SMALL>(cur.e0, cur.e1, d.Acol, (const V *)d.Aval, d.Brp, d.Bcol, (const V *)d.Bval,
                                           cur.rb, cur.nc, active, gt, s_keys[g], s_vals[g], s_en[g], s_scan[g], Ccol,
                                           Cval, d.cols, err, &s_maxd[g]);
        group_sync<WPR>();
        cur = nxt;
    }
}

// The LDS bins from 256 slots on by a column bitmap (rank_sym_row and
// rank_num_row), in batches whose problems are at most kBatchRankCols columns
// per slot wide; lds_cols: the widest.  Dynamic LDS: RPW times the group's.  The
// limit is twice the single product's: a wave still clears and counts at most
// four words a slot, and most rows of a mixed batch belong to its widest
// problems.  Batch of 512: these rows take 1.84 ms numeric and 0.94 symbolic,
// hashed 3.08 and 1.17; with a limit of 64 (the 256-slot rows hashed) 2.11 and
// 0.94.
constexpr int kBatchRankCols = 128;

template <int WPR, int RPW, bool READ>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_bsym_rank_rows(const BatchDesc *__restrict__ desc,
                                                                    const RowDesc *__restrict__ rd, const BinHdr *h,
                                                                    int bin, int lds_cols, int *__restrict__ nnzc)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int g = threadIdx.x / kWave / WPR, gt = threadIdx.x - g * WPR * kWave;
    unsigned char *raw = s_raw + g * rank_sym_lds<WPR>(lds_cols);
    const int cnt = h->count[bin], stride = gridDim.x * RPW;
    const RowDesc *rows = rd + h->offset[bin];
    RowDesc nxt{};
    int r = blockIdx.x * RPW + g;
    if (r < cnt) nxt = rows[r];
    for (; r < cnt; r += stride) {
        const RowDesc cur = nxt;
        if (r + stride < cnt) nxt = rows[r + stride];
        const BatchDesc &d = desc[cur.prob];
        rank_sym_row<WPR, READ>(cur.e0, cur.e1, d.Acol, d.Brp, d.Bcol, d.cols, gt, raw, &nnzc[cur.grow]);
        group_sync<WPR>();
    }
}

template <typename V, int WPR, int RPW, bool READ>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_bnum_rank_rows(const BatchDesc *__restrict__ desc,
                                                                    const RowDesc *__restrict__ rd,
                                                                    const BatchHdr *bh, int bin, int lds_cols, int cap,
                                                                    long long ccap, int *__restrict__ Ccol,
                                                                    V *__restrict__ Cval, int *err)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    extern __shared__ __align__(16) unsigned char s_raw[];
    if (bh->nnz_c > ccap) return;
    const int g = threadIdx.x / kWave / WPR, gt = threadIdx.x - g * WPR * kWave;
    unsigned char *raw = s_raw + g * rank_row_lds<V, WPR>(lds_cols, cap);
    const int cnt = bh->num.count[bin], stride = gridDim.x * RPW;
    const RowDesc *rows = rd + bh->num.offset[bin];
    RowDesc nxt{};
    int r = blockIdx.x * RPW + g;
    if (r < cnt) nxt = rows[r];
    for (; r < cnt; r += stride) {
        const RowDesc cur = nxt;
        if (r + stride < cnt) nxt = rows[r + stride];
        const BatchDesc &d = desc[cur.prob];
        rank_num_row<V, WPR, READ>(cur.e0, cur.e1, d.Acol, (const V *)d.Aval, d.Brp, d.Bcol, (const V *)d.Bval, cur.rb,
                                   cur.nc, d.cols, lds_cols, cap, gt, raw, Ccol, Cval, err);
        group_sync<WPR>();
    }
}

// Symbolic, heavy rows: one block per row, key table at goff[row] in the
// global pool (cleared here; gcap slots in all).
__global__ __launch_bounds__(kGlobalThreads) void k_bsym_global(const BatchDesc *__restrict__ desc,
                                                                const int *__restrict__ prob, const BinHdr *h,
                                                                const int *__restrict__ perm,
                                                                const int *__restrict__ cap,
                                                                const long long *__restrict__ goff, long long gcap,
                                                                GSlot *pool, int *__restrict__ nnzc, int *err)
{
    __shared__ PieceScratch<float, kGlobalThreads> S;
    __shared__ int s_front[1 << kFrontLog];
    __shared__ int s_cnt;
    const int cnt = h->count[kBinHeavy];
    const int *rows = perm + h->offset[kBinHeavy];
    for (int r = blockIdx.x; r < cnt; r += gridDim.x) {
        const int grow = rows[r];
        const BatchDesc &d = desc[prob[grow]];
        if (d.cols <= kWideMaxCols) continue;
        const long long off = goff[grow];
        const int T = 1 << gtable_log2(cap[grow]);
        if (off + T > gcap) {
            if (threadIdx.x == 0) atomicOr(err, kErrCapacity);
            continue;
        }
        int *keys = (int *)(pool + off);             // its first 4 T bytes
        for (int t = threadIdx.x; t < T; t += kGlobalThreads) keys[t] = kEmpty;
        __syncthreads();
        sym_global_row(d.Arp, d.Acol, d.Brp, d.Bcol, (int)(grow - d.row0), cap[grow], keys, S, s_front, &s_cnt, &nnzc[grow],
                       err);
        __syncthreads();
    }
}

// Numeric, heavy rows: one block per row (dynamic LDS: the rank bitmap).
template <typename V>
__global__ __launch_bounds__(kGlobalThreads) void k_bnum_global(const BatchDesc *__restrict__ desc,
                                                                const int *__restrict__ prob, const BatchHdr *bh,
                                                                const int *__restrict__ perm,
                                                                const long long *__restrict__ goff, long long gcap,
                                                                GSlot *pool, long long ccap,
                                                                const long long *__restrict__ Crp,
                                                                int *__restrict__ Ccol, V *__restrict__ Cval, int *err)
{
    extern __shared__ unsigned s_bm[];
    __shared__ GlobalNumLds<V> L;
    if (bh->nnz_c > ccap) return;
    const int cnt = bh->num.count[kBinHeavy];
    const int *rows = perm + bh->num.offset[kBinHeavy];
    for (int r = blockIdx.x; r < cnt; r += gridDim.x) {
        const int grow = rows[r];
        const BatchDesc &d = desc[prob[grow]];
        if (d.cols <= kWideMaxCols) continue;
        const long long off = goff[grow];
        const int nc = (int)(Crp[grow + 1] - Crp[grow]);
        if (off + (1LL << gtable_log2(nc)) > gcap) {
            if (threadIdx.x == 0) atomicOr(err, kErrCapacity);
            continue;
        }
        num_global_row<V>(d.Arp, d.Acol, (const V *)d.Aval, d.Brp, d.Bcol, (const V *)d.Bval, (int)(grow - d.row0),
                          grow, d.cols, pool + off, L, s_bm, Crp, Ccol, Cval, err);
        __syncthreads();
    }
}

// Symbolic, heavy rows of problems with at most kWideMaxCols columns: one
// block per row sets one bit per column of the row in an LDS bitmap over all
// of B's columns (dynamic LDS, ceil(cols / 32) words) and counts the bits.
// READ as in rank_sym_row.
template <bool READ>
__global__ __launch_bounds__(kWideThreads) void k_bsym_wide(const BatchDesc *__restrict__ desc,
                                                            const int *__restrict__ prob, const BinHdr *h,
                                                            const int *__restrict__ perm, int *__restrict__ nnzc)
{
    extern __shared__ unsigned s_bmw[];
    __shared__ PieceScratch<float, kWideThreads> S;
    __shared__ int s_cnt;
    const int cnt = h->count[kBinHeavy];
    const int *rows = perm + h->offset[kBinHeavy];
    const int gt = threadIdx.x;
    for (int r = blockIdx.x; r < cnt; r += gridDim.x) {
        const int grow = rows[r];
        const BatchDesc &d = desc[prob[grow]];
        if (d.cols > kWideMaxCols) continue;
        const int nw = (d.cols + 31) >> 5;
        const int arow = (int)(grow - d.row0);
        for (int t = gt; t < nw; t += kWideThreads) s_bmw[t] = 0u;
        if (gt == 0) s_cnt = 0;                            // the products' first barrier follows
        auto mark = [&](const auto &j, const auto &ok) {
            mark_columns<READ>(s_bmw, j, ok);
        };
        piece_products<float, false, kWideThreads, kWideThreads, 4, true, kRankPiece>(
            d.Arp[arow], d.Arp[arow + 1], gt, S, d.Acol, (const float *)nullptr, d.Brp, 1, 1, d.Bcol,
            (const float *)nullptr, mark);
        int c = 0;
        for (int t = gt; t < nw; t += kWideThreads) c += __popc(s_bmw[t]);
        c = wave_sum(c);
        if (lane_id() == 0 && c) atomicAdd(&s_cnt, c);
        __syncthreads();
        if (gt == 0) nnzc[grow] = s_cnt;
    }
}

// Numeric, heavy rows (but those that take the windows): one block per row
// (from a queue: long and short rows balance across the persistent blocks; no
// more blocks than rows use it, as thousands on one counter take 25 us) merges
// it by a column bitmap, kWideCap entries at a time.
// Windows of 8192 columns (below) scan every slot of every window, thousands
// for the few hundred entries a row has there: 2.50 ms in a batch of 512
// problems of up to 32768 columns, against 1.39 (four waves per row instead of
// eight: 1.67; 5120 entries at a time, two blocks per CU: 1.47).
template <typename V>
__global__ __launch_bounds__(kWideRankThreads) void k_bnum_wide_rank(const BatchDesc *__restrict__ desc,
                                                                 const int *__restrict__ prob, BatchHdr *bh,
                                                                 const int *__restrict__ perm, long long ccap,
                                                                 const long long *__restrict__ Crp, int lds_cols,
                                                                 int *__restrict__ Ccol, V *__restrict__ Cval)
{
    extern __shared__ __align__(16) unsigned char s_raw[];
    __shared__ int s_r;
    if (bh->nnz_c > ccap) return;
    const int cnt = bh->num.count[kBinHeavy];
    const int *rows = perm + bh->num.offset[kBinHeavy];
    if ((int)blockIdx.x >= cnt) return;
    for (;;) {
        __syncthreads();                                // the previous row is done with s_r and the LDS
        if (threadIdx.x == 0) s_r = atomicAdd(&bh->rank_queue, 1);
        __syncthreads();
        const int r = s_r;
        if (r >= cnt) break;
        const int grow = rows[r];
        const BatchDesc &d = desc[prob[grow]];
        if (d.cols > kWideMaxCols) continue;
        const int arow = (int)(grow - d.row0);
        const long long rb = Crp[grow];
        rank_num_row<V, kWideWaves>(d.Arp[arow], d.Arp[arow + 1], d.Acol, (const V *)d.Aval, d.Brp, d.Bcol,
                                    (const V *)d.Bval, rb, (int)(Crp[grow + 1] - rb), d.cols, lds_cols, kWideCap,
                                    threadIdx.x, s_raw, Ccol, Cval, &bh->error);
    }
}

// Numeric, the heavy rows in the windows' bins: one block per row takes B's
// columns in windows of kWideWin; in each window the row's products with
// columns inside it are added into an LDS array of doubles indexed by column
// (occupancy marked by the -0.0 start value, as in the dense chunks of single
// products), and each wave ranks its share of the window with ballots and
// stores its entries in column order through its own slots (dynamic LDS: the
// kWideWin doubles).  Each window enumerates only the B entries inside it: a
// row with at most kWideThreads A entries keeps, per thread, a cursor into its
// B row that the windows advance (one search per window); longer rows search
// both window bounds in every B row they visit.
template <typename V>
__global__ __launch_bounds__(kWideThreads) void k_bnum_wide(const BatchDesc *__restrict__ desc,
                                                            const int *__restrict__ prob, BatchHdr *bh,
                                                            const int *__restrict__ perm, long long ccap,
                                                            const long long *__restrict__ Crp, int *__restrict__ Ccol,
                                                            V *__restrict__ Cval)
{
    constexpr int NW = kWideThreads / kWave;
    constexpr int CPW = kWideWin / NW;                  // columns ranked by each wave
    constexpr int ROUNDS = CPW / kWave;
    extern __shared__ __align__(16) unsigned char s_raw[];
    double *acc = (double *)s_raw;                      // [kWideWin]
    __shared__ EnumScratch<V, kWideThreads> S;
    __shared__ int s_wt[NW];
    __shared__ int s_r;
    if (bh->nnz_c > ccap) return;
    const int cnt = bh->num.count[kBinWinLong] + bh->num.count[kBinWin];
    const int *rows = perm + bh->num.offset[kBinWinLong];
    const int gt = threadIdx.x, lane = lane_id(), wg = gt / kWave;
    // heavy rows from a queue, as above
    if ((int)blockIdx.x >= cnt) return;
    for (;;) {
        __syncthreads();                                // the previous row is done with s_r and the window
        if (gt == 0) s_r = atomicAdd(&bh->wide_queue, 1);
        __syncthreads();
        const int r = s_r;
        if (r >= cnt) break;
        const int grow = rows[r];
        const BatchDesc &d = desc[prob[grow]];
        const int *Acol = d.Acol, *Brp = d.Brp;
        const V *Aval = (const V *)d.Aval;
        const int arow = (int)(grow - d.row0);
        const long long rb = Crp[grow];
        const int nc = (int)(Crp[grow + 1] - rb);
        const int e0 = d.Arp[arow], e1 = d.Arp[arow + 1];
        const bool single = e1 - e0 <= kWideThreads;       // one A entry per thread at most
        int cur = 0, bend = 0;                             // this thread's B row: next entry, end
        if (single && gt < e1 - e0) {
            const int k = Acol[e0 + gt];
            cur = Brp[k];
            bend = Brp[k + 1];
        }
        int done = 0;
        for (int lo = 0; lo < d.cols; lo += kWideWin) {
            const int hi = lo + kWideWin;
            const int nxt = single && gt < e1 - e0 ? lower_bound_col(d.Bcol, cur, bend, hi) : 0;
            for (int t = gt; t < kWideWin; t += kWideThreads) acc[t] = -0.0;
            __syncthreads();
            group_products<V, true, kWideThreads, 2>(
                e0, e1, gt, S, d.Bcol, (const V *)d.Bval,
                [&](int e, int &bs, int &bl, V &a) {
                    if (single) {                          // e is this thread's entry
                        bs = cur;
                        bl = nxt - cur;
                    } else {
                        const int k = Acol[e];
                        const int b1 = Brp[k + 1];
                        bs = lower_bound_col(d.Bcol, Brp[k], b1, lo);
                        bl = lower_bound_col(d.Bcol, bs, b1, hi) - bs;
                    }
                    a = Aval[e];
                },
                [&](int j, double p) {
                    const unsigned jl = (unsigned)(j - lo);
                    if (jl < (unsigned)kWideWin) atomicAdd(&acc[jl], p + 0.0);
                });
            cur = nxt;
            __syncthreads();
            double vr[ROUNDS];
            unsigned long long msk[ROUNDS];
            int wcount = 0;
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q) {
                const int jl = wg * CPW + q * kWave + lane;
                vr[q] = acc[jl];
                msk[q] = wave_ballot(reached(vr[q]));
                wcount += __popcll(msk[q]);
            }
            if (lane == 0) s_wt[wg] = wcount;
            __syncthreads();
            int run = done, tot = 0;
            for (int w = 0; w < NW; ++w) {
                const int t = s_wt[w];
                if (w < wg) run += t;
                tot += t;
            }
            const int n = wcount < nc - run ? wcount : (nc - run > 0 ? nc - run : 0);
            wave_store_ranked<V, ROUNDS>(vr, msk, acc + wg * CPW, lo + wg * CPW, rb + run, n, Ccol, Cval);
            done += tot;
            __syncthreads();
        }
        if (gt == 0 && done != nc) atomicOr(&bh->error, kErrCount);
    }
}

// Flags a batch whose entries exceed the output pool.
__global__ void k_bcheck(BatchHdr *bh, long long ccap)
{
    if (threadIdx.x == 0 && bh->nnz_c > ccap) atomicOr(&bh->error, kErrCapacity);
}

// Entries of each problem: nnz[p] = Crp[row0[p + 1]] - Crp[row0[p]].
__global__ __launch_bounds__(256) void k_bproblem_nnz(int count, const long long *__restrict__ row0s,
                                                      const long long *__restrict__ Crp, long long *__restrict__ nnz)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < count) nnz[p] = Crp[row0s[p + 1]] - Crp[row0s[p]];
}

}  // namespace smash
