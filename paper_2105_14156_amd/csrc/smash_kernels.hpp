// smash_kernels.hpp -- gfx950 kernels of the row-wise hash SpGEMM C = A * B.
//
// Method (SMASH thesis, arXiv 2105.14156): the row-wise product of the
// Background chapter (eq. "row_wise"), where each output row's partial
// products are merged in an on-chip hash table as they are generated, with an
// atomic compare-and-swap claiming empty slots and an atomic fetch-and-add
// merging values (SMASH Kernels chapter, "Hashing Phase").  The output is
// sized from per-row product counts (Window Distribution Phase) refined by an
// exact symbolic pass, and written back as sorted CSR (Write-back Phase).
//
// MI355X mapping (not the PIUMA design of the paper):
//   * a group of 64-lane wavefronts owns one output row (or one column
//     segment of a heavy row) and its LDS table; rows are binned by table
//     size so each bin launches a workgroup shape that fits its rows (the
//     paper's windows sized to the scratchpad);
//   * the group loads a chunk of A's row and prefix-sums the lengths of the B
//     rows it selects; their products are enumerated in pieces of 8 or 16
//     consecutive entries, each piece located once for its lanes, or, where
//     the ranges are too short to fill pieces (short_ranges), "flat", every
//     thread taking products q = t, t + G, ... of the concatenation (the paper
//     gives each row two threads for the same reason, "SMASH Version 2:
//     Tokenization"); several products per thread are loaded before any is
//     merged, to keep loads in flight;
//   * slots come from a multiplicative (Fibonacci) hash of the column, which
//     spreads clustered columns like the paper's low-order-bit hash of
//     version 2, with +1 linear probing;
//   * heavy rows (output bound above the LDS row limit) are cut into column
//     segments of at most kSegCap entries using per-8192-column counts from
//     the symbolic phase.  Small segments, and those of rows with many A
//     entries, are hashed in LDS, the others merged at the ranks of a column
//     bitmap (seg_bin); chunks with more than kDenseMin entries are
//     accumulated directly by column (the paper's per-row dense/sparse
//     decision of the Window Distribution Phase).  Optionally a
//     heavy row instead uses one hash table in global memory (version 3,
//     "Fragmenting Memory").
//   * output is written in column order: ranks from an occupancy bitmap of
//     the row's (or segment's) column range, built in the table's own LDS
//     once its entries are in registers, where that range is at most 64
//     times the table size, else a bitonic sort; dense chunks rank by
//     ballots over the accumulator; entries are staged in LDS so the global
//     stores are coalesced.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace smash {

constexpr int kWave = 64;
constexpr int kEmpty = -1;              // empty-slot tag (Algorithm "SMASH SETUP": EMPTY = -1)
constexpr int kMinLogT = 6;             // smallest LDS row table: 64 slots
constexpr int kMaxLogT = 11;            // largest LDS row table: 2048 slots
constexpr int kLdsBins = kMaxLogT - kMinLogT + 1;
constexpr int kBinHeavy = kLdsBins;
constexpr int kBinEmpty = kLdsBins + 1;
constexpr int kNumBins = kLdsBins + 2;
constexpr int kBinWinLong = kNumBins;     // a batch's heavy rows that take column windows: long ones
constexpr int kBinWin = kNumBins + 1;     // and the others
constexpr int kBatchBins = kNumBins + 2;
constexpr int kChunkCols = 8192;        // column granularity of heavy-row counts
constexpr int kChunkWords = kChunkCols / 32;
constexpr int kSymWinChunks = 16;       // symbolic heavy window: 16 chunks, 16 KiB bitmap
// Chunks with more entries are accumulated by column.  RMAT A * A in ms a call
// with 512, 1024 and 2048: scale 16, edge factor 16: 2.10, 1.82, 1.76; 17, 4: 1.18,
// 1.05, 1.08; 18, 8: 6.04, 5.25, 5.32; scale 16 times 16 per row of 200000 columns
// 0.82, 0.82, 0.86.
constexpr int kDenseMin = 1024;
constexpr int kSegCap = 2048;           // entries of one segment
constexpr int kSegMaxSpan = 16;         // chunks spanned by one segment
constexpr int kSegHash = 128;           // segments of at most this many entries are hashed by a wave
constexpr int kSegBins = 4;             // segments hashed by a wave, ranked, hashed by a block; dense chunks
constexpr int kSegDense = 3;
constexpr int kRankEntries = 256;       // A entries up to which a row's segments are ranked (k_num_rank)
constexpr int kBinBlockRows = 1024;     // rows per block of the binning kernels

enum : int {
    kErrProbe = 1,      // a hash table ran out of slots (inconsistent sizes)
    kErrCsrA = 2,       // A violates the CSR preconditions
    kErrCsrB = 4,       // B violates the CSR preconditions
    kErrCount = 8,      // numeric found a row count different from C_row_ptr
    kErrCapacity = 16,  // the workspace (or an output pool) is too small
};
// Conditions under which the rest of a pipeline must not run: its kernels
// test them on entry (the flags were set by earlier kernels of the same
// stream), so that no kernel indexes through an invalid matrix or beyond the
// workspace, and the host learns of it at its one synchronisation.
constexpr int kErrStop = kErrCsrA | kErrCsrB | kErrCapacity;

__device__ __forceinline__ bool stopped(const int *err)
{
    return err && (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrStop) != 0;
}

struct BinHdr {
    long long wsum[kBatchBins]; // sum of the per-row weights (output entries) per bin
    int count[kBatchBins];      // rows per bin
    int offset[kBatchBins + 1]; // exclusive offsets of the bins in the row permutation
};

struct SegHdr {
    long long nnz[kSegBins];  // output entries per segment bin
    int count[kSegBins];
    int offset[kSegBins + 1];
};

struct DevHdr {
    unsigned long long products;       // sum over rows of products
    unsigned long long gneed[2];       // global-hash slots: [0] symbolic, [1] numeric
    long long nnz_c;
    long long stage_total;             // staging entries of the fused pass
    BinHdr sym, num, fz;
    SegHdr seg;
    int error;                         // flags of the symbolic pipeline
    int num_error;                     // flags of numeric calls, kept until read
    int fused_ok;                      // rows completed by the fused pass
    unsigned long long fused_entries;  // their entries
    // workspace query (smash_workspace_size): heavy rows, and the global
    // tables of the symbolic pass (total and largest, in slots)
    int q_heavy;
    unsigned long long q_gsum;
    unsigned long long q_gmax;
};

// A column segment of a heavy row: the row, its A entries, the chunk range,
// the number of output entries and their offset in C.
struct Seg {
    int row, e0, e1, c0, c1, count;
    long long out;
};

// ------------------------------------------------------------------ helpers

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Orders LDS accesses of one wavefront (lanes execute in lockstep; the fence
// keeps the compiler from moving LDS accesses across it).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

template <int WAVES>
__device__ __forceinline__ void group_sync()
{
    if constexpr (WAVES == 1) wave_sync();
    else __syncthreads();
}

// DPP controls of GFX9 (CDNA) used by the int scans below: shifts within
// rows of 16 lanes, broadcasts of lanes 15 and 31 to the following rows,
// and a whole-wave shift by one lane.
constexpr int kDppRowShr = 0x110;
constexpr int kDppBcast15 = 0x142;
constexpr int kDppBcast31 = 0x143;
constexpr int kDppWaveShr1 = 0x138;

// Inclusive scan over the 64 lanes of a wave with operator `op` and its
// identity `id`, in DPP moves (no LDS crossbar round trips): Hillis-Steele
// within each row of 16 lanes, then row 0's total into row 1 and row 2's
// into row 3, then rows 0-1's total into rows 2-3.
template <typename Op>
__device__ __forceinline__ int wave_scan_dpp(int v, int id, Op op)
{
    v = op(v, __builtin_amdgcn_update_dpp(id, v, kDppRowShr | 1, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(id, v, kDppRowShr | 2, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(id, v, kDppRowShr | 4, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(id, v, kDppRowShr | 8, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(id, v, kDppBcast15, 0xa, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(id, v, kDppBcast31, 0xc, 0xf, false));
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v)
{
    if constexpr (sizeof(T) == 4) {
        return (T)wave_scan_dpp((int)v, 0, [](int a, int b) { return a + b; });
    } else {
        const int lane = lane_id();
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            T t = __shfl_up(v, d, kWave);
            if (lane >= d) v += t;
        }
        return v;
    }
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

__device__ __forceinline__ int ceil_log2(long long x)
{
    return x <= 1 ? 0 : 64 - __clzll((unsigned long long)(x - 1));
}

// Output stores of C bypass cache retention: C is written once and never
// read back by the product, and keeping it out of L2 and the MALL leaves
// room for B and the split table, which every row re-reads.
template <typename T>
__device__ __forceinline__ void store_c(T *p, T v)
{
    __builtin_nontemporal_store(v, p);
}

// Fibonacci hashing of a column index onto 2^logT slots.
__device__ __forceinline__ unsigned slot_of(int key, int logT)
{
    return ((unsigned)key * 2654435769u) >> (32 - logT);
}

// log2 of the global hash table size of a heavy row with at most n keys
// (load factor at most one half).
__host__ __device__ __forceinline__ int gtable_log2(long long n)
{
    long long x = 2 * (n > 1 ? n : 1);
    int l = 0;
    while ((1LL << l) < x) ++l;
    return l;
}

// Bin of a light row from its table bound (cap for symbolic, exact count for
// numeric): table of next_pow2(2 * bound) slots, at least 64.
__device__ __forceinline__ int lds_bin(long long bound)
{
    int lt = ceil_log2(2LL * bound);
    return (lt < kMinLogT ? kMinLogT : lt) - kMinLogT;
}

// Block-wide exclusive scan of one value per thread (all threads call it).
template <typename T, int THREADS>
__device__ __forceinline__ T block_excl_scan(T v, T *s_tmp /* THREADS/64 + 1 */, T &total)
{
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    T incl = wave_incl_scan(v);
    if (lane == kWave - 1) s_tmp[wave] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        T run = 0;
        for (int w = 0; w < THREADS / kWave; ++w) { T t = s_tmp[w]; s_tmp[w] = run; run += t; }
        s_tmp[THREADS / kWave] = run;
    }
    __syncthreads();
    T res = s_tmp[wave] + incl - v;
    total = s_tmp[THREADS / kWave];
    __syncthreads();
    return res;
}

// ----------------------------------------------------- product enumeration
//
// Shared LDS scratch of one group of G threads.
template <typename V, int G>
struct EnumScratch {
    int pincl[G];       // inclusive prefix of the piece counts of the long B ranges
    int sincl[G];       // inclusive prefix of the lengths of the short B ranges
    int bs[G];          // B range start of each A entry of the chunk
    int be[G];          // B range end of each A entry of the chunk
    V a[G];             // value of each A entry of the chunk
    int wsum[2 * (G / kWave)];
};

// Loads the U products of one thread (column, and value in double) with no
// branch between the loads, so all of them are in flight before the first is
// used.  A product with pos < 0 is absent; it loads entry 0 of B, which
// exists whenever the caller enumerates any product.
template <typename V, bool WITH_VAL, int U>
__device__ __forceinline__ void load_products(const int *__restrict__ Bcol, const V *__restrict__ Bval,
                                              const int (&pos)[U], int (&j)[U], double (&bv)[U])
{
    V raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int q = pos[u] >= 0 ? pos[u] : 0;
        j[u] = Bcol[q];
        if constexpr (WITH_VAL) raw[u] = Bval[q];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (WITH_VAL) bv[u] = (double)raw[u];
        else bv[u] = 0.0;
    }
}

// Hands U loaded products of one thread to the sink: one call per product
// (sink(j, a * b), or sink(j) without values), or with ARRAY_SINK one call
// with all U (sink(j[U], p[U], ok[U]), or sink(j[U], ok[U])), so that the
// sink can overlap their LDS round trips.
template <bool WITH_VAL, int U, bool ARRAY_SINK, typename Sink>
__device__ __forceinline__ void emit_products(Sink &sink, const int (&pos)[U], const int (&j)[U],
                                              const double (&av)[U], const double (&bv)[U])
{
    if constexpr (ARRAY_SINK) {
        bool ok[U];
        double p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ok[u] = pos[u] >= 0;
            p[u] = av[u] * bv[u];
        }
        if constexpr (WITH_VAL) sink(j, p, ok);
        else sink(j, ok);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (pos[u] >= 0) {
                if constexpr (WITH_VAL) sink(j[u], av[u] * bv[u]);
                else sink(j[u]);
            }
        }
    }
}

// Calls sink(j, a * b) -- the product formed in double -- (or sink(j)
// without values) for every product of the A entries [e0, e1) of one row,
// each restricted to the B range returned by get(e, &bstart, &blen, &a).  The
// G threads of the group (thread index gt) take the row in chunks of G A
// entries.  B ranges of at least 64 entries are cut into pieces of 64
// products: each wave takes U consecutive pieces at a time, finds their A
// entry with one search that all its lanes share, and every lane loads one
// product per piece (coalesced, no per-lane search).  Shorter ranges, which
// carry few of the products, are enumerated flat: thread gt takes products
// q = gt, gt + G, ... and finds its A entry by binary search (consecutive
// lanes then read consecutive B entries where a range continues).  U products
// per thread are located and loaded before any is merged.
template <typename V, bool WITH_VAL, int G, int U, typename Get, typename Sink, bool ARRAY_SINK = false>
__device__ __forceinline__ void group_products(int e0, int e1, int gt, EnumScratch<V, G> &S,
                                               const int *__restrict__ Bcol, const V *__restrict__ Bval,
                                               Get get, Sink sink)
{
    constexpr int WG = G / kWave;
    const int lane = lane_id(), wg = gt / kWave;
    for (int base = e0; base < e1; base += G) {
        const int e = base + gt;
        int bs = 0, bl = 0;
        V a = V(0);
        if (e < e1) get(e, bs, bl, a);
        const bool lng = bl >= kWave;
        int ip = wave_incl_scan(lng ? (bl + kWave - 1) / kWave : 0);
        int is = wave_incl_scan(lng ? 0 : bl);
        if constexpr (WG > 1) {
            if (lane == kWave - 1) {
                S.wsum[wg] = ip;
                S.wsum[WG + wg] = is;
            }
            group_sync<WG>();
            int ap = 0, as = 0;
            for (int w = 0; w < wg; ++w) {
                ap += S.wsum[w];
                as += S.wsum[WG + w];
            }
            ip += ap;
            is += as;
        }
        S.pincl[gt] = ip;
        S.sincl[gt] = is;
        S.bs[gt] = bs;
        S.be[gt] = bs + bl;
        if constexpr (WITH_VAL) S.a[gt] = a;
        group_sync<WG>();
        const int ptot = S.pincl[G - 1], stot = S.sincl[G - 1];
        // long ranges, piece by piece: wave wg takes U consecutive pieces per
        // round.  A wave's pieces only move forward, so it keeps a cursor `cur` (no piece of
        // it lies in an A entry before cur) and finds the A entry of piece
        // pc from one wave-wide read: lane l holds the boundary
        // pincl[cur + l - 1] (lane 0 the one before cur, never above pc),
        // and the first lane whose boundary exceeds pc names the entry.  One
        // read serves all U pieces of a round unless they run past it.
        int cur = 0;
        auto window = [&]() {
            const int t = cur + lane - 1;
            return t < 0 ? 0 : S.pincl[t < G ? t : G - 1];
        };
        auto locate_pieces = [&](int pc0, int (&pos)[U], double (&av)[U]) {
            int v = window();
            int last = cur;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int pc = pc0 + u;
                pos[u] = -1;
                av[u] = 0.0;
                if (pc < ptot) {                                   // wave-uniform
                    unsigned long long hit;
                    while (!(hit = __ballot(v > pc))) {
                        cur += kWave - 1;
                        v = window();
                    }
                    const int k = __ffsll((long long)hit) - 1;     // >= 1
                    const int src = cur + k - 1;
                    const int pex = __builtin_amdgcn_readlane(v, k - 1);
                    const int p = S.bs[src] + (pc - pex) * kWave + lane;
                    if (p < S.be[src]) {
                        pos[u] = p;
                        if constexpr (WITH_VAL) av[u] = (double)S.a[src];
                    }
                    last = src;
                }
            }
            cur = last;
        };
        {
            int pos[U], j[U];
            double av[U], bv[U];
            for (int pc0 = wg * U; pc0 < ptot; pc0 += WG * U) {
                locate_pieces(pc0, pos, av);
                load_products<V, WITH_VAL, U>(Bcol, Bval, pos, j, bv);
                emit_products<WITH_VAL, U, ARRAY_SINK>(sink, pos, j, av, bv);
            }
        }
        // short ranges, flat: thread gt takes products q = q0 + u * G + gt
        // and finds its A entry by binary search (consecutive lanes then read
        // consecutive B entries where a range continues)
        auto locate_flat = [&](int q0, int (&pos)[U], double (&av)[U]) {
            // the U searches advance step by step together, so that their
            // LDS reads are in flight at once
            int src[U];
#pragma unroll
            for (int u = 0; u < U; ++u) src[u] = 0;
#pragma unroll
            for (int step = G / 2; step > 0; step >>= 1) {
                int t[U];
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] = S.sincl[src[u] + step - 1];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (t[u] <= q0 + u * G + gt) src[u] += step;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = q0 + u * G + gt;
                pos[u] = -1;
                av[u] = 0.0;
                if (q < stot) {
                    const int excl = src[u] ? S.sincl[src[u] - 1] : 0;
                    pos[u] = S.bs[src[u]] + (q - excl);
                    if constexpr (WITH_VAL) av[u] = (double)S.a[src[u]];
                }
            }
        };
        {
            int pos[U], j[U];
            double av[U], bv[U];
            for (int q0 = 0; q0 < stot; q0 += G * U) {
                locate_flat(q0, pos, av);
                load_products<V, WITH_VAL, U>(Bcol, Bval, pos, j, bv);
                emit_products<WITH_VAL, U, ARRAY_SINK>(sink, pos, j, av, bv);
            }
        }
        group_sync<WG>();
    }
}

// ---------------------------------------------- product enumeration by pieces
//
// piece_products enumerates the same products in pieces of at most PL = 16 (or
// 8, for rows of short B ranges) of one B range: 64 / PL pieces per wave step,
// each loaded by PL lanes.  A piece is located once, by one lane (a binary
// search over the prefix of the entries' piece counts), and its start, end and
// A value reach the lanes that load it by DPP row broadcasts: no LDS access
// and no search per product, and a short range wastes at most PL - 1 lanes.
constexpr int kPiece = 16;
constexpr int kDppRowNewBcast = 0x150;   // lane t of each row of 16 to the whole row (gfx90a and later)

template <typename V, int GE>
struct PieceScratch {
    int incl[GE];   // inclusive prefix of the entries' piece counts, 64 entries at a time
    int bs[GE];     // B range of each entry
    int be[GE];
    V a[GE];        // A value
    int wsum[GE / kWave];   // pieces of each 64 entries
};

template <int T>
__device__ __forceinline__ int row_bcast(int v)
{
    return __builtin_amdgcn_mov_dpp(v, kDppRowNewBcast + T, 0xf, 0xf, true);   // every lane has a source
}

template <int T>
__device__ __forceinline__ float row_bcast(float v)
{
    return __int_as_float(row_bcast<T>(__float_as_int(v)));
}

template <int T>
__device__ __forceinline__ double row_bcast(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = row_bcast<T>((int)(b & 0xffffffff)), hi = row_bcast<T>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The value of x in the lane of this lane's group of PL that located step T's
// piece.
template <int PL, int T, typename X>
__device__ __forceinline__ X piece_bcast(X x)
{
    if constexpr (PL == 16) {
        return row_bcast<T>(x);
    } else {
        static_assert(PL == 8, "half a row");
        const X lo = row_bcast<T>(x), hi = row_bcast<T + 8>(x);
        return lane_id() & 8 ? hi : lo;
    }
}

// Lists one A entry per thread gt < GE (its B range [bs, bs + bl), empty beyond
// the n entries of the step) in S: the prefix of the piece counts runs within
// each 64 entries, so no barrier is needed inside.  Every thread of the group
// calls it; readers of S come after a barrier.
template <typename V, bool WITH_VAL, int GE, int PL = kPiece>
__device__ __forceinline__ void piece_list(int n, int gt, int bs, int bl, V a, PieceScratch<V, GE> &S)
{
    static_assert(GE % kWave == 0, "entry step");
    if (gt >= GE) return;                                          // whole waves
    int ip = 0;
    if (gt - lane_id() < n) {
        ip = wave_incl_scan((bl + PL - 1) / PL);
        S.incl[gt] = ip;
        S.bs[gt] = bs;
        S.be[gt] = bs + bl;
        if constexpr (WITH_VAL) S.a[gt] = a;
    }
    if (lane_id() == kWave - 1) S.wsum[gt / kWave] = ip;
}

// Number of pieces listed in S.
template <typename V, int GE>
__device__ __forceinline__ int piece_count(const PieceScratch<V, GE> &S)
{
    int P = 0;
#pragma unroll
    for (int w = 0; w < GE / kWave; ++w) P += S.wsum[w];
    return P;
}

// U wave steps of the located pieces (st, en, al) from step T on, loaded.
template <typename V, bool WITH_VAL, int U, int PL>
struct PieceGroup {
    int pos[U], j[U];
    bool ok[U];
    V a[U], raw[U];

    template <int T>
    __device__ __forceinline__ void load(int st, int en, V al, const int *__restrict__ Bcol,
                                         const V *__restrict__ Bval)
    {
        take<T, 0>(st, en, al);
#pragma unroll
        for (int u = 0; u < U; ++u) {                              // an absent product loads entry 0
            j[u] = Bcol[pos[u]];
            if constexpr (WITH_VAL) raw[u] = Bval[pos[u]];
        }
    }

    template <int T, int N>
    __device__ __forceinline__ void take(int st, int en, V al)
    {
        if constexpr (N < U) {
            const int q = piece_bcast<PL, T + N>(st) + (lane_id() & (PL - 1));
            ok[N] = q < piece_bcast<PL, T + N>(en);
            pos[N] = ok[N] ? q : 0;
            if constexpr (WITH_VAL) a[N] = piece_bcast<PL, T + N>(al);
            take<T, N + 1>(st, en, al);
        }
    }

    template <typename Sink>
    __device__ __forceinline__ void emit(Sink &sink)
    {
        if constexpr (WITH_VAL) {
            double p[U];
#pragma unroll
            for (int u = 0; u < U; ++u) p[u] = (double)a[u] * (double)raw[u];
            sink(j, p, ok);
        } else {
            sink(j, ok);
        }
    }
};

// Steps T, T + 1, ... of the located pieces to the sink, U at a time; the
// loads of the next U are in flight while this U are handed over (`cur` holds
// step T's).
template <typename V, bool WITH_VAL, int U, int PL, int T, typename Sink>
__device__ __forceinline__ void piece_steps(int left, int st, int en, V al, const int *__restrict__ Bcol,
                                            const V *__restrict__ Bval, PieceGroup<V, WITH_VAL, U, PL> &cur, Sink &sink)
{
    if constexpr (T + U < PL) {
        if ((T + U) * (kWave / PL) < left) {             // wave-uniform
            PieceGroup<V, WITH_VAL, U, PL> nxt;
            nxt.template load<T + U>(st, en, al, Bcol, Bval);
            cur.emit(sink);
            piece_steps<V, WITH_VAL, U, PL, T + U>(left, st, en, al, Bcol, Bval, nxt, sink);
            return;
        }
    }
    cur.emit(sink);
}

// Locates 64 of the listed pieces (of n entries), [p0, p1) at most: lane l
// finds piece p0 + (l % PL) * (64 / PL) + l / PL, so that step t takes lane t of
// every PL lanes.  Absent pieces are empty (st = en = 0).
template <typename V, bool WITH_VAL, int GE, int PL = kPiece>
__device__ __forceinline__ void piece_locate(int p0, int p1, int n, const PieceScratch<V, GE> &S, int &st, int &en,
                                             V &al)
{
    const int lane = lane_id();
    int pc = p0 + (lane & (PL - 1)) * (kWave / PL) + lane / PL;
    st = en = 0;
    al = V(0);
    if (pc < p1) {
        int g = 0;                                                 // the 64 entries that hold piece pc
        if (n > kWave) {
#pragma unroll
            for (int w = 0; w < GE / kWave - 1; ++w) {
                const int t = S.wsum[w];
                if (g == w * kWave && pc >= t) {
                    pc -= t;
                    g += kWave;
                }
            }
        }
        const int *incl = S.incl + g;
        const int m = n - g < kWave ? n - g : kWave;
        int src = 0;                                               // their entries whose prefix is <= pc
        for (int s = n > kWave ? kWave / 2 : n > 1 ? 1 << (31 - __clz(n - 1)) : 0; s > 0; s >>= 1) {
            const int t = src + s;
            if (t < m && incl[t - 1] <= pc) src = t;
        }
        const int ex = src ? incl[src - 1] : 0;
        src += g;
        st = S.bs[src] + (pc - ex) * PL;
        en = S.be[src];
        if constexpr (WITH_VAL) al = S.a[src];
    }
}

// Pieces of each wave when the waves of a group share P pieces in equal
// contiguous parts (whole steps).
template <int WG, int PL = kPiece>
__device__ __forceinline__ int piece_share(int P)
{
    constexpr int STEP = kWave / PL;
    return ((P + WG - 1) / WG + STEP - 1) & ~(STEP - 1);
}

// Hands every product of the P pieces listed in S (of n entries) to the sink
// (sink(j[U], p[U], ok[U]) or, without values, sink(j[U], ok[U])).
template <typename V, bool WITH_VAL, int GE, int G, int U, int PL, typename Sink>
__device__ __forceinline__ void piece_run(int P, int n, int gt, const PieceScratch<V, GE> &S,
                                          const int *__restrict__ Bcol, const V *__restrict__ Bval, Sink &sink)
{
    const int wg = __builtin_amdgcn_readfirstlane(gt / kWave), per = piece_share<G / kWave, PL>(P);
    const int p1 = (wg + 1) * per < P ? (wg + 1) * per : P;
    for (int p0 = wg * per; p0 < p1; p0 += kWave) {
        int st, en;
        V al;
        piece_locate<V, WITH_VAL, GE, PL>(p0, p1, n, S, st, en, al);
        PieceGroup<V, WITH_VAL, U, PL> first;
        first.template load<0>(st, en, al, Bcol, Bval);
        piece_steps<V, WITH_VAL, U, PL, 0>(p1 - p0, st, en, al, Bcol, Bval, first, sink);
    }
}

// Hands every product of the A entries [e0, e1) of one row to the sink, GE
// entries at a time: entry e takes row Acol[e] of B between its split points
// split[k * per] and split[k * per + d].  The split points of the next GE
// entries and the columns of those after them are on their way while one list
// is run, so that a hub row's steps do not each wait for two dependent
// gathers.  Every thread of the group of G calls it; S is free again when it
// returns.  AHEAD = false leaves that out, where registers are short.
template <typename V, bool WITH_VAL, int GE, int G, int U, bool AHEAD = true, int PL = kPiece, typename Sink>
__device__ __forceinline__ void piece_products(int e0, int e1, int gt, PieceScratch<V, GE> &S,
                                               const int *__restrict__ Acol, const V *__restrict__ Aval,
                                               const int *__restrict__ split, long long per, int d,
                                               const int *__restrict__ Bcol, const V *__restrict__ Bval, Sink &sink)
{
    constexpr int WG = G / kWave;
    const unsigned len = (unsigned)(e1 - e0);
    long long k = -1;
    V a = V(0), a1 = V(0);
    int bs = 0, be = 0;
    auto column = [&](unsigned r, V &val) {              // entry e0 + r
        k = -1;
        if (gt < GE && r < len) {
            k = Acol[e0 + (int)r] * per;
            if constexpr (WITH_VAL) val = Aval[e0 + (int)r];
        }
    };
    auto range = [&]() {
        bs = be = 0;
        if (k >= 0) {
            bs = split[k];
            be = split[k + d];
        }
    };
    column(gt, a);
    range();
    if constexpr (AHEAD) column(GE + gt, a1);
    for (unsigned base = 0; base < len; base += GE) {
        const int n = len - base < GE ? (int)(len - base) : GE;
        piece_list<V, WITH_VAL, GE, PL>(n, gt, bs, be - bs, a, S);
        group_sync<WG>();
        if constexpr (AHEAD) {
            if (base + GE < len) {
                range();
                a = a1;
                column(base + 2 * GE + gt, a1);
            }
        }
        piece_run<V, WITH_VAL, GE, G, U, PL>(piece_count(S), n, gt, S, Bcol, Bval, sink);
        if constexpr (!AHEAD) {
            if (base + GE < len) {
                column(base + GE + gt, a);
                range();
            }
        }
        group_sync<WG>();
    }
}

// f(integral_constant<int, T>) for T = 0 .. N - 1 while pieces are left
// (wave-uniform): the steps of a wave with `left` located pieces.
template <int N, int PL = kPiece, typename F, int T = 0>
__device__ __forceinline__ void piece_each(int left, F &f)
{
    if constexpr (T < N) {
        if (T * (kWave / PL) >= left) return;
        f(std::integral_constant<int, T>());
        piece_each<N, PL, F, T + 1>(left, f);
    }
}

// ------------------------------------------------------------ LDS hashing

// Claims the slot of `key` in an LDS key table, probing from slot h; returns
// 1 if the key was new.
__device__ __forceinline__ int lds_insert_key_at(int *keys, int logT, int key, unsigned h, int *err)
{
    const unsigned mask = (1u << logT) - 1;
    for (unsigned probe = 0; probe <= mask; ++probe) {
        int cur = __hip_atomic_load(&keys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == key) return 0;
        if (cur == kEmpty) {
            int old = atomicCAS(&keys[h], kEmpty, key);
            if (old == kEmpty) return 1;
            if (old == key) return 0;
        }
        h = (h + 1) & mask;
    }
    atomicOr(err, kErrProbe);
    return 0;
}

// Claims or finds the slot of `key`, probing from slot h, and adds `p` to its
// value (values are accumulated in double: the LDS FP64 atomic add is the
// fast one on gfx950).
__device__ __forceinline__ void lds_insert_add_at(int *keys, double *vals, int logT, int key, double p, unsigned h,
                                                  int *err)
{
    const unsigned mask = (1u << logT) - 1;
    for (unsigned probe = 0; probe <= mask; ++probe) {
        int cur = __hip_atomic_load(&keys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == kEmpty) {
            int old = atomicCAS(&keys[h], kEmpty, key);
            cur = old == kEmpty ? key : old;
        }
        if (cur == key) {
            atomicAdd(&vals[h], p);
            return;
        }
        h = (h + 1) & mask;
    }
    atomicOr(err, kErrProbe);
}

// U products of one thread at once, each starting with a compare-and-swap
// of its home slot (empty -> column), all U issued before any result is
// used: the CAS returns the slot's previous key, so one LDS round trip tells
// whether the column was claimed (empty), is already there (its key), or
// met another column (probing continues one product at a time from the next
// slot).  Two products of the same column in one thread are safe: the
// second CAS returns the first one's key.
template <int U>
__device__ __forceinline__ void lds_insert_add_u(int *keys, double *vals, int logT, const int (&j)[U],
                                                 const double (&p)[U], const bool (&ok)[U], int *err)
{
    const unsigned mask = (1u << logT) - 1;
    unsigned h[U];
    int old[U];
#pragma unroll
    for (int u = 0; u < U; ++u) h[u] = slot_of(j[u], logT);
#pragma unroll
    for (int u = 0; u < U; ++u) old[u] = ok[u] ? atomicCAS(&keys[h[u]], kEmpty, j[u]) : j[u];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!ok[u]) continue;
        if (old[u] == kEmpty || old[u] == j[u]) atomicAdd(&vals[h[u]], p[u]);
        else lds_insert_add_at(keys, vals, logT, j[u], p[u], (h[u] + 1) & mask, err);
    }
}

// Key-only variant: returns how many of the U columns were new.
template <int U>
__device__ __forceinline__ int lds_insert_key_u(int *keys, int logT, const int (&j)[U], const bool (&ok)[U], int *err)
{
    const unsigned mask = (1u << logT) - 1;
    unsigned h[U];
    int old[U];
    int added = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) h[u] = slot_of(j[u], logT);
#pragma unroll
    for (int u = 0; u < U; ++u) old[u] = ok[u] ? atomicCAS(&keys[h[u]], kEmpty, j[u]) : j[u];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!ok[u]) continue;
        if (old[u] == kEmpty) ++added;
        else if (old[u] != j[u]) added += lds_insert_key_at(keys, logT, j[u], (h[u] + 1) & mask, err);
    }
    return added;
}

// Order-preserving variant (the paper's first version, High-Bit Hashing):
// the home slot of column j is j >> shift, so slots rise with the column;
// CAS-first like lds_insert_add_u, then +1 linear probing (modulo T).  The
// longest probe distance of the row is kept in *maxd: the table is then
// sorted except within that distance (see order_row_entries_ord).
template <int U>
__device__ __forceinline__ void lds_insert_add_ord_u(int *keys, double *vals, int logT, int shift, const int (&j)[U],
                                                     const double (&p)[U], const bool (&ok)[U], int *maxd, int *err)
{
    const unsigned mask = (1u << logT) - 1;
    unsigned h[U];
    int old[U];
#pragma unroll
    for (int u = 0; u < U; ++u) h[u] = ((unsigned)j[u] >> shift) & mask;
#pragma unroll
    for (int u = 0; u < U; ++u) old[u] = ok[u] ? atomicCAS(&keys[h[u]], kEmpty, j[u]) : j[u];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!ok[u]) continue;
        if (old[u] == kEmpty || old[u] == j[u]) {
            atomicAdd(&vals[h[u]], p[u]);
            continue;
        }
        unsigned hh = h[u];
        bool placed = false;
        for (unsigned d = 1; d <= mask; ++d) {
            hh = (hh + 1) & mask;
            int cur = __hip_atomic_load(&keys[hh], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (cur == kEmpty) {
                const int o = atomicCAS(&keys[hh], kEmpty, j[u]);
                cur = o == kEmpty ? j[u] : o;
            }
            if (cur == j[u]) {
                atomicAdd(&vals[hh], p[u]);
                if ((int)d > __hip_atomic_load(maxd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
                    atomicMax(maxd, (int)d);
                placed = true;
                break;
            }
        }
        if (!placed) atomicOr(err, kErrProbe);
    }
}

// --------------------------------------------------------------- small rows
//
// A row of at most 64 products is merged in one wave's registers, a product
// per lane: a bitonic network over the lanes sorts the columns, equal
// neighbours are one entry, their values are added by a segmented scan.  No
// table is cleared, probed, compacted or ranked: half the instructions of the
// hashed form (which spends some 200 on ordering 64 entries alone), and
// instructions are what bounds these rows.  A million rows of 8 x 8 products,
// FP32: numeric 1.09 -> 0.50 ms, symbolic 0.58 -> 0.31.
constexpr int kSmallCols = 1 << 25;      // a column and a lane in 32 bits

// The value of lane (l ^ MASK): DPP within a row of 16, else the LDS crossbar.
template <int MASK>
__device__ __forceinline__ unsigned lane_xor(unsigned v)
{
    if constexpr (MASK == 1) return __builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true);         // quad_perm 1 0 3 2
    else if constexpr (MASK == 2) return __builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true);    // quad_perm 2 3 0 1
    else if constexpr (MASK == 3) return __builtin_amdgcn_update_dpp(0, (int)v, 0x1b, 0xf, 0xf, true);    // quad_perm 3 2 1 0
    else if constexpr (MASK == 7) return __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);   // row_half_mirror
    else if constexpr (MASK == 8) return __builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true);   // row_ror:8
    else if constexpr (MASK == 15) return __builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true);  // row_mirror
    else if constexpr (MASK < 32) return __builtin_amdgcn_ds_swizzle((int)v, (MASK << 10) | 0x1f);
    else return __shfl_xor((int)v, MASK, kWave);
}

// Compare-exchange of every lane with lane (l ^ MASK): the one whose bit BIT is
// clear keeps the smaller value.
template <int MASK, int BIT>
__device__ __forceinline__ void sort_step(unsigned &v)
{
    const unsigned o = lane_xor<MASK>(v);
    const unsigned lo = v < o ? v : o, hi = v < o ? o : v;
    v = lane_id() & BIT ? hi : lo;
}

// Ascending sort of one value per lane of the wave.
__device__ __forceinline__ void wave_sort(unsigned &v)
{
    sort_step<1, 1>(v);
    sort_step<3, 2>(v);
    sort_step<1, 1>(v);
    sort_step<7, 4>(v);
    sort_step<2, 2>(v);
    sort_step<1, 1>(v);
    sort_step<15, 8>(v);
    sort_step<4, 4>(v);
    sort_step<2, 2>(v);
    sort_step<1, 1>(v);
    sort_step<31, 16>(v);
    sort_step<8, 8>(v);
    sort_step<4, 4>(v);
    sort_step<2, 2>(v);
    sort_step<1, 1>(v);
    sort_step<63, 32>(v);
    sort_step<16, 16>(v);
    sort_step<8, 8>(v);
    sort_step<4, 4>(v);
    sort_step<2, 2>(v);
    sort_step<1, 1>(v);
}

// One lane's share of a merged small row: with `tail` set, entry `pos` of the
// row is (col, val); count is the row's number of entries.
struct SmallRow {
    bool tail;
    int pos, col, count;
    double val;
};

// Merges the products of the A entries [e0, e1) if they are at most 64 (else,
// and for more than 64 entries, returns false).  own: 64 ints of the wave's
// LDS.  Every lane of the wave calls it.
template <typename V, bool WITH_VAL>
__device__ __forceinline__ bool small_row(int e0, int e1, const int *__restrict__ Acol, const V *__restrict__ Aval,
                                          const int *__restrict__ Brp, const int *__restrict__ Bcol,
                                          const V *__restrict__ Bval, int ncols, int *own, SmallRow &out)
{
    const int lane = lane_id();
    if (e1 - e0 > kWave || ncols > kSmallCols) return false;      // wave-uniform
    int bs = 0, bl = 0;
    V a = V(0);
    if (e0 + lane < e1) {
        const int k = Acol[e0 + lane];
        bs = Brp[k];
        bl = Brp[k + 1] - bs;
        if constexpr (WITH_VAL) a = Aval[e0 + lane];
    }
    const int incl = wave_incl_scan(bl);
    const int n = __builtin_amdgcn_readlane(incl, kWave - 1);
    // a prefix that wraps is not small either: every length is at most n then
    if (n > kWave || __ballot(bl > kWave)) return false;
    // the entry of lane q's product: each entry marks its first product, and
    // the marks' running maximum names the entry
    const int first = incl - bl;
    own[lane] = 0;
    wave_sync();
    if (bl > 0) own[first] = lane;
    wave_sync();
    const int src = wave_scan_dpp(own[lane], 0, [](int x, int y) { return x > y ? x : y; });
    const bool live = lane < n;
    const int q = __shfl(bs - first, src, kWave) + lane;
    const int at = live ? q : 0;
    const int j = Bcol[at];
    double p = 0.0;
    if constexpr (WITH_VAL) {
        const V b = Bval[at];
        p = (double)__shfl(a, src, kWave) * (double)b + 0.0;      // a sum that starts at 0.0
    }
    unsigned c = live ? ((unsigned)j << 6) | (unsigned)lane : 0xffffffffu;
    wave_sort(c);
    const int col = (int)(c >> 6);                                 // absent products come last
    const int before = __builtin_amdgcn_update_dpp(-1, col, kDppWaveShr1, 0xf, 0xf, false);
    const unsigned long long heads = __ballot(live && col != before);
    out.count = __popcll(heads);
    if constexpr (WITH_VAL) {
        p = __shfl(p, (int)(c & 63u), kWave);
        const unsigned long long upto = heads & (~0ull >> (63 - lane));
        if (out.count < n) {
            // runs of equal columns: an inclusive scan within each run
            const int start = 63 - __clzll((long long)upto);
            for (int d = 1; d < kWave; d <<= 1) {
                const bool take = live && lane - d >= start;
                if (!__ballot(take)) break;
                const double o = __shfl_up(p, d, kWave);
                if (take) p += o;
            }
        }
        out.tail = live && (lane == n - 1 || (heads >> (lane + 1) & 1));
        out.pos = __popcll(upto) - 1;
        out.col = col;
        out.val = p;
    }
    return true;
}

// --------------------------------------------------------------- validation

// CSR preconditions of one matrix in two passes (a violation sets `flag` in
// *err).  Rows, one thread per row: row_ptr starts at 0, ends at nnz and
// never decreases; the first entry of every non-empty row is marked in a
// bitmap over the entries (cleared beforehand).  Entries, one thread per
// entry (coalesced): the column is in range and above the previous entry's
// unless the entry starts a row.  Without a bitmap (starts = NULL) only what
// memory safety needs is checked: row pointers and column ranges.
__global__ __launch_bounds__(256) void k_validate_rows(int rows, long long nnz, const int *__restrict__ rp,
                                                       unsigned *__restrict__ starts, int flag, int *err)
{
    const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    if (r == 0 && (rp[0] != 0 || (long long)rp[rows] != nnz)) bad = true;
    if (r < rows) {
        const int a = rp[r], b = rp[r + 1];
        if (b < a || a < 0 || (long long)b > nnz) bad = true;
        else if (a < b && starts) atomicOr(&starts[a >> 5], 1u << (a & 31));
    }
    if (__syncthreads_or(bad) && threadIdx.x == 0) atomicOr(err, flag);
}

__global__ __launch_bounds__(256) void k_validate_cols(int cols, long long nnz, const int *__restrict__ ci,
                                                       const unsigned *__restrict__ starts, int flag, int *err)
{
    const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    if (p < nnz) {
        const int c = ci[p];
        if (c < 0 || c >= cols) bad = true;
        else if (starts && p > 0 && c <= ci[p - 1] && !((starts[p >> 5] >> (p & 31)) & 1u)) bad = true;
    }
    if (__syncthreads_or(bad) && threadIdx.x == 0) atomicOr(err, flag);
}

// The same for a matrix of at most kFewRows rows in one launch and without the
// bitmap: an entry not above its predecessor looks for itself among the row
// pointers (a search of 13 steps, made about once per row).  Without `strict`
// only what memory safety needs is checked.
//
// Up to kFewRows rows every step of a product is one launch.  The line lies
// where that stops to pay: products of 8192 rows in us a call, so and with a
// launch per bin: 16 products a row 126 and 143, 100 in 1M columns 208 and 218,
// 400 there 354 and 329, 900 in 4096 columns 240 and 185; RMAT scale 13, edge
// factor 4 175 and 203, 16 270 and 290.
constexpr int kFewRows = 8192;

__global__ __launch_bounds__(256) void k_validate_few(int rows, int cols, long long nnz, const int *__restrict__ rp,
                                                      const int *__restrict__ ci, int strict, int flag, int *err)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = t == 0 && (rp[0] != 0 || (long long)rp[rows] != nnz);
    if (t < rows) {
        const int a = rp[t], b = rp[t + 1];
        if (b < a || a < 0 || (long long)b > nnz) bad = true;
    }
    if (t < nnz) {
        const int c = ci[t];
        if (c < 0 || c >= cols) {
            bad = true;
        } else if (strict && t > 0 && c <= ci[t - 1]) {
            int lo = 0, hi = rows;                       // first row pointer >= t
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (rp[mid] < t) lo = mid + 1;
                else hi = mid;
            }
            if (rp[lo] != t) bad = true;
        }
    }
    if (__syncthreads_or(bad) && threadIdx.x == 0) atomicOr(err, flag);
}

// Start of a symbolic call: the header cleared, and the `words` words of the
// validation bitmap.
__global__ __launch_bounds__(256) void k_begin(DevHdr *h, long long words, unsigned *__restrict__ starts)
{
    static_assert(sizeof(DevHdr) % sizeof(int) == 0, "cleared as ints");
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x, step = (long long)gridDim.x * blockDim.x;
    for (long long i = t; i < (long long)(sizeof(DevHdr) / sizeof(int)); i += step) ((int *)h)[i] = 0;
    for (long long i = t; i < words; i += step) starts[i] = 0u;
}

// --------------------------------------------------------- analysis & bins

// Feature t (0..5) of the learned predictor for a row with na A entries:
// log2(1 + x) of na, the products ub, max_k nnz(B_k), min_k nnz(B_k),
// min(ub, cols) and sum_k nnz(B_k)^2 / ub, in double, rounded to float; 0 for
// a row without entries.  The selection is branch-free so that six lanes
// evaluate their features together.
__device__ __forceinline__ float row_feature(int t, int na, long long ub, double sq, int mx, int mn, int ncols)
{
    if (na == 0) return 0.f;
    const double cap = ub < ncols ? (double)ub : (double)ncols;
    const double x = t == 0 ? (double)na
                   : t == 1 ? (double)ub
                   : t == 2 ? (double)mx
                   : t == 3 ? (double)mn
                   : t == 4 ? cap
                            : (ub > 0 ? sq / (double)ub : 0.0);
    return (float)log2(1.0 + x);
}

// Row analysis (step a1): products ub_i = sum_k nnz(B_k) over row i of A, the
// output bound cap_i = min(ub_i, cols) and the row's symbolic bin.  With feats
// non-NULL it also writes the learned predictor's six features and
// max_k nnz(B_k) (maxb_out) of the rows whose bound exceeds the LDS row limit,
// the only rows the predictor is asked about.
//
// Bound by the latency of two dependent gathers per entry, so the work is
// spread for it (for_rows): rows of at most short_row entries are summed by
// groups of eight lanes, consecutive rows in consecutive groups; longer rows by
// a whole wave, eight entries per lane in flight, and the rows a wave looks
// at lie an odd stride apart, since hub rows come in clusters (consecutive
// rows in RMAT matrices).  RMAT scale 21, edge factor 8 (rows of up to 40K
// entries): 0.23 ms; with eight consecutive rows per wave, long ones summed by
// the wave in turn, 0.58.  The limit: a wave has at most a few entries per lane
// of rows just above it and waits for each row's gathers in turn (features of a
// million rows of 150 entries with a limit of 128: 0.77 ms, 256: 0.66), eight
// lanes take longer with longer rows (RMAT scale 20, edge factor 8: 0.150 ms,
// 512: 0.176).  From a million and a half rows on, whose clusters of such rows
// are longer, the lower limit (RMAT scale 21, edge factor 8: 0.246 and 0.277 ms).
constexpr int kRowLanes = 8;
constexpr int kShortRow = 256;          // 128 in tall matrices: short_row
constexpr int kRowThreads = 256;
constexpr int kBlockRows = kRowThreads / kRowLanes;

// Partial sums of one lane over entries e0 + first, e0 + first + step, ...
struct RowPart {
    long long ub = 0;
    double sq = 0.0;
    int mx = 0, mn = 0x7fffffff;
};

template <bool FEATS, int U = 4>
__device__ __forceinline__ void row_part(const int *__restrict__ Acol, const int *__restrict__ Brp, int e, int e1,
                                         int step, RowPart &r)
{
    for (; e < e1 - (U - 1) * step; e += U * step) {
        int k[U], len[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = Acol[e + u * step];
#pragma unroll
        for (int u = 0; u < U; ++u) len[u] = Brp[k[u] + 1] - Brp[k[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            r.ub += len[u];
            if constexpr (FEATS) {
                r.sq += (double)len[u] * (double)len[u];
                r.mx = len[u] > r.mx ? len[u] : r.mx;
                r.mn = len[u] < r.mn ? len[u] : r.mn;
            }
        }
    }
    if constexpr (U > 1) row_part<FEATS, U / 2>(Acol, Brp, e, e1, step, r);
}

// Reduction of RowPart over lanes that differ in the bits of `width - 1`.
template <bool FEATS>
__device__ __forceinline__ void row_reduce(RowPart &r, int width)
{
    for (int d = width / 2; d > 0; d >>= 1) {
        r.ub += __shfl_xor(r.ub, d, kWave);
        if constexpr (FEATS) {
            r.sq += __shfl_xor(r.sq, d, kWave);
            const int a = __shfl_xor(r.mx, d, kWave), b = __shfl_xor(r.mn, d, kWave);
            r.mx = a > r.mx ? a : r.mx;
            r.mn = b < r.mn ? b : r.mn;
        }
    }
}

// Sums of the entries [e0, e1) of the wave's eight rows, one row per group of
// eight lanes, into the lanes of each group (every lane of the wave calls it).
template <bool FEATS>
__device__ __forceinline__ RowPart wave_rows(int e0, int e1, const int *__restrict__ Acol,
                                             const int *__restrict__ Brp)
{
    const int lane = lane_id(), sl = lane & (kRowLanes - 1);
    const bool lng = e1 - e0 > kShortRow;
    RowPart r;
    if (!lng) row_part<FEATS>(Acol, Brp, e0 + sl, e1, kRowLanes, r);
    row_reduce<FEATS>(r, kRowLanes);
    unsigned long long todo = __ballot(lng && sl == 0);
    while (todo) {
        const int src = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        RowPart w;
        row_part<FEATS>(Acol, Brp, __builtin_amdgcn_readlane(e0, src) + lane, __builtin_amdgcn_readlane(e1, src),
                        kWave, w);
        row_reduce<FEATS>(w, kWave);
        if (lane / kRowLanes == src / kRowLanes) r = w;
    }
    return r;
}

// Blocks for the long rows and for all rows of an analysis of m rows; the long
// ones come first in the grid.  All but one of the long blocks' waves look at
// rows (an odd number of waves is the stride): 64 each from a million rows on,
// and fewer where that is too few waves for rows that may all be long.
// Features of 8192 rows of 1000 entries: 51 us, with 64 rows a wave 303; of 400
// rows of 30000 entries 58 and 2040.
__host__ __device__ __forceinline__ int long_row_blocks(int m)
{
    const int k = 31 - __builtin_clz(m | 1);
    const int per = k >= 20 ? 6 : k >= 16 ? k - 14 : k >= 14 ? 2 : k >= 12 ? k - 12 : 0;      // log2 rows per wave
    return (int)((((long long)m + (1 << per) - 1) >> per) / (kRowThreads / kWave)) + 1;
}
// Entries up to which for_rows sums a row of m by eight lanes.
__device__ __forceinline__ int short_row(int m) { return m > 3 << 19 ? kShortRow / 2 : kShortRow; }
__host__ __device__ __forceinline__ int row_blocks(int m)
{
    return long_row_blocks(m) + (m + kBlockRows - 1) / kBlockRows;
}

// finish(row, sl, e0, e1, sums) for every row of A, by eight lanes sl = 0 .. 7 at
// least.  A grid of row_blocks(m) blocks of kRowThreads threads.
template <bool FEATS, typename F>
__device__ __forceinline__ void for_rows(int m, const int *__restrict__ Arp, const int *__restrict__ Acol,
                                         const int *__restrict__ Brp, F finish)
{
    const int lane = lane_id(), nl = long_row_blocks(m);
    if ((int)blockIdx.x < nl) {
        const int waves = nl * (kRowThreads / kWave) - 1, w = blockIdx.x * (kRowThreads / kWave) + threadIdx.x / kWave;
        if (w == waves) return;
        const long long row = (long long)lane * waves + w;
        const int e0 = row < m ? Arp[row] : 0, e1 = row < m ? Arp[row + 1] : 0;
        for (unsigned long long todo = __ballot(e1 - e0 > short_row(m)); todo; todo &= todo - 1) {
            const int src = __ffsll((long long)todo) - 1;
            const int f0 = __builtin_amdgcn_readlane(e0, src), f1 = __builtin_amdgcn_readlane(e1, src);
            RowPart r;
            row_part<FEATS, 8>(Acol, Brp, f0 + lane, f1, kWave, r);
            row_reduce<FEATS>(r, kWave);
            finish(src * waves + w, lane, f0, f1, r);
        }
        return;
    }
    const int row = ((int)blockIdx.x - nl) * kBlockRows + (int)threadIdx.x / kRowLanes, sl = lane & (kRowLanes - 1);
    const int e0 = row < m ? Arp[row] : 0, e1 = row < m ? Arp[row + 1] : 0;
    const bool here = row < m && e1 - e0 <= short_row(m);
    RowPart r;
    if (here) row_part<FEATS>(Acol, Brp, e0 + sl, e1, kRowLanes, r);
    row_reduce<FEATS>(r, kRowLanes);
    if (here) finish(row, sl, e0, e1, r);
}

__global__ __launch_bounds__(kRowThreads) void k_analyze(int m, int ncols, int lds_row_max,
                                                 const int *__restrict__ Arp, const int *__restrict__ Acol,
                                                 const int *__restrict__ Brp, long long *__restrict__ ub_out,
                                                 int *__restrict__ cap_out, int *__restrict__ nnzc,
                                                 unsigned char *__restrict__ bin_out, float *__restrict__ feats,
                                                 int *__restrict__ maxb_out, const int *err)
{
    if (stopped(err)) return;
    auto finish = [&](int row, int sl, int e0, int e1, const RowPart &r) {
        const long long ub = r.ub;
        if (feats && sl < 6 && (ub < ncols ? ub : ncols) > lds_row_max) {
            // the predictor's six features (the same arithmetic as k_features):
            // lanes 0..5 write one each
            feats[(long long)row * 6 + sl] = row_feature(sl, e1 - e0, ub, r.sq, r.mx, r.mn, ncols);
            if (sl == 0) maxb_out[row] = e1 > e0 ? r.mx : 0;
        }
        if (sl == 0) {
            const int cap = (int)(ub < ncols ? ub : ncols);
            int b;
            if (ub == 0) b = kBinEmpty;
            else if (cap > lds_row_max) b = kBinHeavy;
            else b = lds_bin(cap);
            ub_out[row] = ub;
            cap_out[row] = cap;
            nnzc[row] = 0;
            bin_out[row] = (unsigned char)b;
        }
    };
    if (feats) for_rows<true>(m, Arp, Acol, Brp, finish);
    else for_rows<false>(m, Arp, Acol, Brp, finish);
}

// Workspace query (smash_workspace_size): the number of heavy rows and the
// slots their global tables would take (total and largest), from the same
// bounds as k_analyze (eight rows per wave, grid-stride over whole waves);
// the counts of a block's rows are summed in LDS and added with one atomic
// per block and counter.
__global__ __launch_bounds__(256) void k_ws_query(int m, int ncols, int lds_row_max, const int *__restrict__ Arp,
                                                  const int *__restrict__ Acol, const int *__restrict__ Brp,
                                                  DevHdr *h)
{
    constexpr int RPB = 256 / kWave * kRowLanes;        // rows per block and step
    __shared__ unsigned long long s_sum[256 / kWave], s_max[256 / kWave];
    __shared__ int s_cnt[256 / kWave];
    const int lane = lane_id(), w = threadIdx.x / kWave, sl = lane & (kRowLanes - 1);
    int cnt = 0;
    unsigned long long gsum = 0, gmax = 0;
    if (!stopped(&h->error)) {
        for (int r0 = blockIdx.x * RPB + w * kRowLanes; r0 < m; r0 += gridDim.x * RPB) {
            const int row = r0 + lane / kRowLanes;
            const int e0 = row < m ? Arp[row] : 0, e1 = row < m ? Arp[row + 1] : 0;
            const RowPart r = wave_rows<false>(e0, e1, Acol, Brp);
            const long long cap = r.ub < ncols ? r.ub : ncols;
            if (row < m && sl == 0 && cap > lds_row_max) {
                const unsigned long long t = 1ull << gtable_log2(cap);
                ++cnt;
                gsum += t;
                gmax = t > gmax ? t : gmax;
            }
        }
    }
    // wave totals, then the block's
    for (int d = kWave / 2; d > 0; d >>= 1) {
        cnt += __shfl_xor(cnt, d, kWave);
        gsum += __shfl_xor(gsum, d, kWave);
        const unsigned long long o = __shfl_xor(gmax, d, kWave);
        gmax = o > gmax ? o : gmax;
    }
    if (lane == 0) {
        s_cnt[w] = cnt;
        s_sum[w] = gsum;
        s_max[w] = gmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < 256 / kWave; ++v) {
            cnt += s_cnt[v];
            gsum += s_sum[v];
            gmax = s_max[v] > gmax ? s_max[v] : gmax;
        }
        if (cnt) {
            atomicAdd(&h->q_heavy, cnt);
            atomicAdd(&h->q_gsum, gsum);
            atomicMax(&h->q_gmax, gmax);
        }
    }
}

// Numeric bin of a row from its symbolic bin and exact count: heavy rows stay
// heavy, rows outside the plan (no products, or completed by the fused pass)
// stay out.
__device__ __forceinline__ int num_bin(int sym_bin, int nc)
{
    return sym_bin == kBinHeavy ? kBinHeavy : (sym_bin == kBinEmpty || nc == 0 ? kBinEmpty : lds_bin(nc));
}

// Numeric bin of every row.
__global__ __launch_bounds__(256) void k_num_bins(int m, const int *__restrict__ nnzc,
                                                  const unsigned char *__restrict__ sym_bin_of,
                                                  unsigned char *__restrict__ bin_out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    bin_out[i] = (unsigned char)num_bin(sym_bin_of[i], nnzc[i]);
}

// Per-block bin histograms (kBinBlockRows rows per block, no global atomics):
// bcount[blk * NB + b], the block's per-bin sum of the row weights wt
// (bw, when wt is given) and the block's sum of products (bprod, when ub is
// given).
template <int NB>
__global__ __launch_bounds__(256) void k_bin_count(int m, const unsigned char *__restrict__ bin_of,
                                                   const long long *__restrict__ ub, const int *__restrict__ wt,
                                                   int *__restrict__ bcount, unsigned long long *__restrict__ bprod,
                                                   long long *__restrict__ bw, const int *err)
{
    if (stopped(err)) return;
    __shared__ int s_hist[NB];
    __shared__ unsigned long long s_w[NB];
    __shared__ unsigned long long s_prod;
    if (threadIdx.x < NB) {
        s_hist[threadIdx.x] = 0;
        s_w[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) s_prod = 0;
    __syncthreads();
    unsigned long long prod = 0;
    for (int r = threadIdx.x; r < kBinBlockRows; r += 256) {
        const long long i = (long long)blockIdx.x * kBinBlockRows + r;
        if (i < m) {
            const int b = bin_of[i];
            atomicAdd(&s_hist[b], 1);
            if (wt) atomicAdd(&s_w[b], (unsigned long long)wt[i]);
            if (ub) prod += (unsigned long long)ub[i];
        }
    }
    prod = wave_sum(prod);
    if (lane_id() == 0 && prod) atomicAdd(&s_prod, prod);
    __syncthreads();
    if (threadIdx.x < NB) {
        bcount[blockIdx.x * NB + threadIdx.x] = s_hist[threadIdx.x];
        if (bw) bw[blockIdx.x * NB + threadIdx.x] = (long long)s_w[threadIdx.x];
    }
    if (threadIdx.x == 0 && bprod) bprod[blockIdx.x] = s_prod;
}

// Bin totals and offsets, and every block's base inside each bin (one block of
// a wave per bin).
template <int NB>
__global__ __launch_bounds__(NB *kWave) void k_bin_scan(int nblk, int *__restrict__ bcount,
                                                  const unsigned long long *__restrict__ bprod,
                                                  const long long *__restrict__ bw, BinHdr *h,
                                                  unsigned long long *products, int *err, long long heavy_cap)
{
    // err: with heavy_cap >= 0, more heavy rows than the workspace holds
    // raise kErrCapacity (every later kernel of the pipeline then stops)
    if (stopped(err)) return;
    __shared__ int s_tot[NB];
    __shared__ long long s_wt[NB];
    // one wave per bin scans the block counts in place (exclusive)
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    {
        const int b = wave;
        int run = 0;
        for (int c0 = 0; c0 < nblk; c0 += kWave) {
            const int c = c0 + lane;
            const int v = c < nblk ? bcount[c * NB + b] : 0;
            const int incl = wave_incl_scan(v);
            if (c < nblk) bcount[c * NB + b] = run + incl - v;
            run += __shfl(incl, kWave - 1, kWave);
        }
        long long ws = 0;
        if (bw)
            for (int c = lane; c < nblk; c += kWave) ws += bw[c * NB + b];
        ws = wave_sum(ws);
        if (lane == 0) {
            s_tot[b] = run;
            s_wt[b] = ws;
        }
    }
    unsigned long long p = 0;
    if (bprod)
        for (int c = threadIdx.x; c < nblk; c += NB * kWave) p += bprod[c];
    p = wave_sum(p);
    __shared__ unsigned long long s_p[NB];
    if (lane == 0) s_p[wave] = p;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int b = 0; b < NB; ++b) {
            h->count[b] = s_tot[b];
            h->wsum[b] = s_wt[b];
            h->offset[b] = run;
            run += s_tot[b];
        }
        h->offset[NB] = run;
        if (bprod && products) {
            unsigned long long sum = 0;
            for (int w = 0; w < NB; ++w) sum += s_p[w];
            *products = sum;
        }
        if (err && heavy_cap >= 0 && s_tot[kBinHeavy] > heavy_cap) atomicOr(err, kErrCapacity);
    }
}

// Groups row ids by bin (empty rows are left out): perm[offset[b] + block base
// + rank in block].  For the heavy bin, also records the row's global-hash
// table size (gsz, by heavy index) when gsize_of is given.
template <int NB>
__global__ __launch_bounds__(256) void k_scatter(int m, const unsigned char *__restrict__ bin_of,
                                                 const int *__restrict__ bbase, const BinHdr *h,
                                                 int *__restrict__ perm, const int *__restrict__ gsize_of,
                                                 long long *__restrict__ gsz, const int *err)
{
    if (stopped(err)) return;
    __shared__ int s_cnt[NB];
    if (threadIdx.x < NB) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    for (int r = threadIdx.x; r < kBinBlockRows; r += 256) {
        const long long i = (long long)blockIdx.x * kBinBlockRows + r;
        if (i >= m) break;
        const int b = bin_of[i];
        const int local = atomicAdd(&s_cnt[b], 1);
        if (b == kBinEmpty) continue;
        const int pos = h->offset[b] + bbase[blockIdx.x * NB + b] + local;
        perm[pos] = (int)i;
        if (b == kBinHeavy && gsize_of) gsz[pos - h->offset[kBinHeavy]] = 1LL << gtable_log2(gsize_of[i]);
    }
}

// Binning of at most kFewRows rows in one block (k_bin_count, k_bin_scan and
// k_scatter in one launch): a product with so few rows is bound by the number
// of launches, 3 to 5 us each.  A wave ranks its rows within each bin by
// ballots.  wsum is filled for heavy rows only (the one that is read).
constexpr int kFewThreads = 1024;

template <typename B>
__device__ __forceinline__ void bin_few(int m, B bin_at, const long long *__restrict__ ub, const int *__restrict__ wt,
                                        BinHdr *h, unsigned long long *products, int *__restrict__ perm,
                                        const int *__restrict__ gsize_of, long long *__restrict__ gsz, int *err,
                                        long long heavy_cap)
{
    constexpr int PER = kFewRows / kFewThreads;
    __shared__ int s_cnt[kNumBins], s_off[kNumBins + 1];
    __shared__ unsigned long long s_w, s_prod;
    if (threadIdx.x < kNumBins) s_cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) s_w = s_prod = 0;
    __syncthreads();
    int bin[PER], at[PER];
    unsigned long long prod = 0, w = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = q * kFewThreads + threadIdx.x;
        bin[q] = i < m ? bin_at(i) : -1;
        at[q] = 0;
        if (__ballot(bin[q] >= 0) == 0) continue;
        if (i < m && ub) prod += (unsigned long long)ub[i];
        if (bin[q] == kBinHeavy && wt) w += (unsigned long long)wt[i];
#pragma unroll
        for (int b = 0; b < kNumBins; ++b) {
            const unsigned long long mask = __ballot(bin[q] == b);
            if (!mask) continue;
            int base = 0;
            if (lane_id() == 0) base = atomicAdd(&s_cnt[b], __popcll(mask));
            base = __builtin_amdgcn_readfirstlane(base);
            if (bin[q] == b) at[q] = base + __popcll(mask & ((1ull << lane_id()) - 1));
        }
    }
    prod = wave_sum(prod);
    w = wave_sum(w);
    if (lane_id() == 0 && prod) atomicAdd(&s_prod, prod);
    if (lane_id() == 0 && w) atomicAdd(&s_w, w);
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int b = 0; b < kNumBins; ++b) {
            h->count[b] = s_cnt[b];
            h->wsum[b] = b == kBinHeavy ? (long long)s_w : 0;
            h->offset[b] = s_off[b] = run;
            run += s_cnt[b];
        }
        h->offset[kNumBins] = run;
        if (ub && products) *products = s_prod;
        if (err && heavy_cap >= 0 && s_cnt[kBinHeavy] > heavy_cap) atomicOr(err, kErrCapacity);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = q * kFewThreads + threadIdx.x, b = bin[q];
        if (b < 0 || b == kBinEmpty) continue;
        perm[s_off[b] + at[q]] = i;
        if (b == kBinHeavy && gsize_of) gsz[at[q]] = 1LL << gtable_log2(gsize_of[i]);
    }
}

__global__ __launch_bounds__(kFewThreads) void k_bin_few(int m, const unsigned char *__restrict__ bin_of,
                                                         const long long *__restrict__ ub, const int *__restrict__ wt,
                                                         BinHdr *h, unsigned long long *products,
                                                         int *__restrict__ perm, const int *__restrict__ gsize_of,
                                                         long long *__restrict__ gsz, int *err, long long heavy_cap)
{
    if (stopped(err)) return;
    bin_few(m, [&](int i) { return (int)bin_of[i]; }, ub, wt, h, products, perm, gsize_of, gsz, err, heavy_cap);
}

// ------------------------------------------ light rows by a column bitmap
//
// Where B is at most kRankColsPerSlot times as wide as the row's hash table
// would be long, a light row needs no table: its columns are marked in an LDS
// bitmap over all of B's columns, the bitmap's prefix counts rank every product,
// and the products are added at their ranks (as in the ranked segments of
// heavy rows).  The hashed form clears and reads back a table of twice the
// entries, probes it, and orders what it holds by the same bitmap; and its LDS
// is 12 bytes a slot whatever B's width.  Bound by instruction issue and the
// latency of the gathers.  RMAT scale 21 times a 4096-column matrix, FP32, rows
// of 65 to 1024 entries: numeric 867 -> 554 us, symbolic 470 -> 225 (pieces of
// 16 products instead of 8: 689 and 225).  A wider B costs a longer bitmap per
// row; at the limit it is two words a slot, as the hashed form's ordering.
constexpr int kRankColsPerSlot = 64;
constexpr int kRankPiece = 8;
constexpr int kRankMaxCols = kRankColsPerSlot << kMaxLogT;      // 2^17: 16-bit columns and one bit more

// Whether a product's A entries select so few products each (products per
// entry below halves / 2, on average) that most lanes of a piece are idle, and
// the hashed forms, which take a product per lane, are faster.  Single product,
// numeric pass of light rows of B rows of one length, hashed and by bitmap:
// length 1, 4096 columns, rows of 220: 0.75 and 1.03 ms a call; length 3: 0.48 and
// 0.55; length 4: 0.43 and 0.36 (rows of 100, whose table is ranked by as few
// words: 0.50 and 0.51; 60 entries of length 4 in 128 columns: 0.52 and 0.57).
// The symbolic pass is ahead by bitmap from length 2 on.  In batches wider
// than kRankColsPerSlot columns a slot the hashed form has to sort: rows of 450,
// 131072 columns, length 1: 1.61 and 1.78, length 2: 1.27 and 1.02; rows of
// 220, 65536 columns, whose blocks hold 64 KB by bitmap, length 2: 0.86 and 0.98,
// length 3: 0.87 both.
inline bool short_ranges(int halves, long long products, long long entries) { return 2 * products < halves * entries; }

__host__ __device__ __forceinline__ int rank_words(int ncols) { return ((ncols + 31) / 32 + 7) & ~7; }

// LDS of one group of WPR waves (a multiple of 16): bitmap, prefix counts,
// sums and columns of cap entries, entry list, scan scratch.
template <typename V, int WPR>
__host__ __device__ __forceinline__ size_t rank_row_lds(int ncols, int cap)
{
    return (((size_t)rank_words(ncols) * 6 + (size_t)cap * 10 + sizeof(PieceScratch<V, WPR * kWave>) +
             WPR * sizeof(int)) + 15) & ~(size_t)15;
}

template <int WPR>
__host__ __device__ __forceinline__ size_t rank_sym_lds(int ncols)
{
    return (((size_t)rank_words(ncols) * 4 + sizeof(PieceScratch<float, WPR * kWave>) + sizeof(int)) + 15) & ~(size_t)15;
}

// Marks the columns j (where ok) in a bitmap over B's columns.  READ: those
// marked already skip the atomic, whose lanes wait for each other where they
// meet in one word; the reads overlap, and an OR after a stale read is merely
// redundant.
template <bool READ, typename J, typename K>
__device__ __forceinline__ void mark_columns(unsigned *bm, const J &j, const K &ok)
{
    constexpr int N = sizeof(j) / sizeof(j[0]);
    if constexpr (READ) {
        unsigned w[N];
#pragma unroll
        for (int u = 0; u < N; ++u) w[u] = ok[u] ? bm[j[u] >> 5] : ~0u;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const unsigned bit = 1u << (j[u] & 31);
            if (!(w[u] & bit)) atomicOr(&bm[j[u] >> 5], bit);
        }
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (ok[u]) atomicOr(&bm[j[u] >> 5], 1u << (j[u] & 31));
    }
}

// Marks are read first where the average row has more than kRepeatRead products
// per column (most marks are set already) of at most 4096 columns (many lanes
// meet in a word): 8000 rows of 300 x 300 products 2.55 ms a replay without and
// 2.34 with in 1500 columns (60 per column), 2.97 and 2.12 in 600, 5.37 and 2.96
// in 300.  Elsewhere the reads cost: rows of 600 x 300 products in 6000 columns
// (30 per column) 4.34 and 4.44, the batch of 512 RMAT pairs 5.93 and 5.97.
constexpr int kRepeatRead = 24;

inline bool read_marks(double products, long long rows, long long cols)
{
    return cols <= 4096 && products > (double)kRepeatRead * rows * cols;
}

// Symbolic count of one light row by a group of WPR waves, stored to *out.
// raw: rank_sym_lds bytes.  B is at most ncols wide.  READ: marks are read
// before they are set (kRepeatRead).
template <int WPR, bool READ>
__device__ __forceinline__ void rank_sym_row(int e0, int e1, const int *__restrict__ Acol,
                                             const int *__restrict__ Brp, const int *__restrict__ Bcol, int ncols,
                                             int gt, unsigned char *raw, int *out)
{
    constexpr int G = WPR * kWave;
    const int W = rank_words(ncols);
    unsigned *bm = reinterpret_cast<unsigned *>(raw);
    auto &S = *reinterpret_cast<PieceScratch<float, G> *>(bm + W);
    int *cnt = reinterpret_cast<int *>(&S + 1);
    for (int t = gt * 4; t < W; t += 4 * G) *(uint4 *)&bm[t] = make_uint4(0, 0, 0, 0);
    if (gt == 0) *cnt = 0;                                  // the products' first barrier follows
    auto mark = [&](const auto &j, const auto &ok) {
        mark_columns<READ>(bm, j, ok);
    };
    piece_products<float, false, G, G, 4, true, kRankPiece>(e0, e1, gt, S, Acol, (const float *)nullptr, Brp, 1, 1,
                                                            Bcol, (const float *)nullptr, mark);
    int pc = 0;
    for (int t = gt * 4; t < W; t += 4 * G) {
        const uint4 v = *(const uint4 *)&bm[t];
        pc += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
    pc = wave_sum(pc);
    if constexpr (WPR > 1) {
        if (lane_id() == 0 && pc) atomicAdd(cnt, pc);
        __syncthreads();
        pc = *cnt;
        __syncthreads();
    }
    if (gt == 0) *out = pc;
}

// Numeric pass of one row by a group of WPR waves: its products merged and
// written in column order at C's offset rb (nc entries expected, at most 65535:
// the bitmap's prefix counts are 16 bits wide), cap entries
// at a time (rows of more entries repeat the second pass).  raw: rank_row_lds
// bytes for lds_cols >= ncols columns.  Products stay in registers between the
// passes where the row's A entries fit one list and its pieces one locating.
// READ as in rank_sym_row.
template <typename V, int WPR, bool READ = false>
__device__ __forceinline__ void rank_num_row(int e0, int e1, const int *__restrict__ Acol, const V *__restrict__ Aval,
                                             const int *__restrict__ Brp, const int *__restrict__ Bcol,
                                             const V *__restrict__ Bval, long long rb, int nc, int ncols, int lds_cols,
                                             int cap, int gt, unsigned char *raw, int *__restrict__ Ccol,
                                             V *__restrict__ Cval, int *err)
{
    constexpr int G = WPR * kWave, PL = kRankPiece;
    const int lane = lane_id(), wg = __builtin_amdgcn_readfirstlane(gt / kWave);
    const int W = rank_words(ncols), WL = rank_words(lds_cols);
    double *vals = reinterpret_cast<double *>(raw);
    unsigned *bm = reinterpret_cast<unsigned *>(vals + cap);
    unsigned short *pref = reinterpret_cast<unsigned short *>(bm + WL);
    unsigned short *cols = pref + WL;
    auto &S = *reinterpret_cast<PieceScratch<V, G> *>(cols + cap);     // cap: a multiple of 32
    int *scan = reinterpret_cast<int *>(&S + 1);
    for (int t = gt * 4; t < W; t += 4 * G) *(uint4 *)&bm[t] = make_uint4(0, 0, 0, 0);
    for (int t = gt; t < (nc < cap ? nc : cap); t += G) vals[t] = 0.0;
    int hc[PL], left = 0;
    V hv[PL], al = V(0);
    bool hok[PL], held = false;
    // every product of the row, 64 pieces of a wave at a time, through use(step);
    // the last ones stay in hc, hv, hok and al
    auto pass = [&](auto &use) {
        for (unsigned base = 0, len = (unsigned)(e1 - e0); base < len; base += G) {
            const int n = len - base < G ? (int)(len - base) : G;
            int bs = 0, bl = 0;
            V a = V(0);
            if (gt < n) {
                const int k = Acol[e0 + (int)base + gt];
                a = Aval[e0 + (int)base + gt];
                bs = Brp[k];
                bl = Brp[k + 1] - bs;
            }
            piece_list<V, true, G, PL>(n, gt, bs, bl, a, S);
            group_sync<WPR>();
            const int P = piece_count(S), share = piece_share<WPR, PL>(P);
            const int p1 = (wg + 1) * share < P ? (wg + 1) * share : P;
            held = len <= G && share <= kWave;
            for (int p0 = wg * share; p0 < p1; p0 += kWave) {
                int st, en;
                piece_locate<V, true, G, PL>(p0, p1, n, S, st, en, al);
                left = p1 - p0;
                auto load = [&](auto t) {
                    constexpr int T = decltype(t)::value;
                    const int q = piece_bcast<PL, T>(st) + (lane & (PL - 1));
                    hok[T] = q < piece_bcast<PL, T>(en);
                    const int at = hok[T] ? q : 0;
                    hc[T] = Bcol[at];
                    hv[T] = Bval[at];
                };
                piece_each<PL, PL>(left, load);
                piece_each<PL, PL>(left, use);
            }
            group_sync<WPR>();
        }
    };
    auto mark = [&](auto t) {
        constexpr int T = decltype(t)::value;
        if constexpr (READ) {
            const unsigned bit = 1u << (hc[T] & 31);
            if (hok[T] && !(bm[hc[T] >> 5] & bit)) atomicOr(&bm[hc[T] >> 5], bit);
        } else {
            if (hok[T]) atomicOr(&bm[hc[T] >> 5], 1u << (hc[T] & 31));
        }
    };
    pass(mark);
    // prefix counts: every thread the same number of consecutive 4-word groups
    const int q4 = (W / 4 + G - 1) / G;
    const int w0 = gt * q4 * 4, w1 = w0 + q4 * 4 < W ? w0 + q4 * 4 : W;
    int pc = 0;
    for (int w = w0; w < w1; w += 4) {
        const uint4 v = *(const uint4 *)&bm[w];
        pc += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
    const int inc = wave_incl_scan(pc);
    int run = 0, total = 0;
    if constexpr (WPR > 1) {
        if (lane == kWave - 1) scan[wg] = inc;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WPR; ++w) {
            const int t = scan[w];
            if (w < wg) run += t;
            total += t;
        }
    } else {
        total = __builtin_amdgcn_readlane(inc, kWave - 1);
    }
    unsigned at = (unsigned)(run + inc - pc);
    for (int w = w0; w < w1; w += 4) {
        const uint4 v = *(const uint4 *)&bm[w];
        const unsigned a1 = at + __popc(v.x), a2 = a1 + __popc(v.y), a3 = a2 + __popc(v.z);
        *(uint2 *)&pref[w] = make_uint2(at | a1 << 16, a2 | a3 << 16);
        at = a3 + __popc(v.w);
    }
    group_sync<WPR>();
    if (gt == 0 && total != nc) atomicOr(err, kErrCount);
    const int cnt = total < nc ? total : nc;
    // entries from `half` on lie in columns of 65536 and more
    const int half = W > 2048 ? pref[2048] : cnt;
    for (int r0 = 0; r0 < cnt; r0 += cap) {
        const int n = cnt - r0 < cap ? cnt - r0 : cap;
        if (r0 > 0) {
            for (int t = gt; t < n; t += G) vals[t] = 0.0;
            group_sync<WPR>();
        }
        auto put = [&](auto t) {
            constexpr int T = decltype(t)::value;
            const double p = (double)piece_bcast<PL, T>(al) * (double)hv[T];
            if (!hok[T]) return;
            const int j = hc[T];
            const unsigned r = pref[j >> 5] + __popc(bm[j >> 5] & ((1u << (j & 31)) - 1u)) - r0;
            if (r < (unsigned)n) {
                atomicAdd(&vals[r], p);
                cols[r] = (unsigned short)j;
            }
        };
        if (held) piece_each<PL, PL>(left, put);
        else pass(put);
        group_sync<WPR>();
        for (int t = gt; t < n; t += G) {
            store_c(&Ccol[rb + r0 + t], (int)cols[t] + (r0 + t >= half ? 65536 : 0));
            store_c(&Cval[rb + r0 + t], (V)vals[t]);
        }
        if (r0 + cap < cnt) group_sync<WPR>();
    }
}

// Light rows of one bin (see k_sym_rows and k_num_rows) by a column bitmap;
// dynamic LDS: RPW times the group's.
template <int WPR, int RPW, bool READ>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_sym_rank_rows(
    const int *__restrict__ Arp, const int *__restrict__ Acol, const int *__restrict__ Brp,
    const int *__restrict__ Bcol, const int *__restrict__ perm, const BinHdr *h, int bin, int ncols,
    int *__restrict__ nnzc, const int *err)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    extern __shared__ __align__(16) unsigned char s_raw[];
    if (stopped(err)) return;
    const int g = threadIdx.x / kWave / WPR, gt = threadIdx.x - g * WPR * kWave;
    unsigned char *raw = s_raw + g * rank_sym_lds<WPR>(ncols);
    const int nrows = h->count[bin];
    const int *rows = perm + h->offset[bin];
    for (int r = blockIdx.x * RPW + g; r < nrows; r += gridDim.x * RPW) {
        const int row = rows[r];
        rank_sym_row<WPR, READ>(Arp[row], Arp[row + 1], Acol, Brp, Bcol, ncols, gt, raw, &nnzc[row]);
        group_sync<WPR>();
    }
}

template <typename V, int WPR, int RPW>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_num_rank_rows(
    const int *__restrict__ Arp, const int *__restrict__ Acol, const V *__restrict__ Aval,
    const int *__restrict__ Brp, const int *__restrict__ Bcol, const V *__restrict__ Bval,
    const int *__restrict__ rows, int nrows, const long long *__restrict__ Crp, int *__restrict__ Ccol,
    V *__restrict__ Cval, int ncols, int cap, int *err)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int g = threadIdx.x / kWave / WPR, gt = threadIdx.x - g * WPR * kWave;
    const int r = blockIdx.x * RPW + g;
    if (r >= nrows) return;                                 // whole groups
    const int row = rows[r];
    const long long rb = Crp[row];
    rank_num_row<V, WPR>(Arp[row], Arp[row + 1], Acol, Aval, Brp, Bcol, Bval, rb, (int)(Crp[row + 1] - rb), ncols,
                         ncols, cap, gt, s_raw + g * rank_row_lds<V, WPR>(ncols, cap), Ccol, Cval, err);
}

// ------------------------------------------------------- symbolic, LDS hash

// Tables up to this size hold rows of at most 64 entries, nearly all of which
// have at most 64 products.
constexpr int kSmallLogT = 7;

// Symbolic count of one light row by a group of WPR waves (gt: thread index
// in the group; every thread of the group calls it): the distinct columns of
// the row's A entries [e0, e1) times B, counted in an LDS key table of
// 2^LOGT slots (step a3), are stored to *out by the group's first thread.
// SMALL: try small_row on rows of the smallest tables (a template parameter:
// a branch on a flag takes registers from both forms, 12% of a call).
template <int LOGT, int WPR, bool SMALL = true>
__device__ __forceinline__ void sym_row(int e0, int e1, const int *__restrict__ Acol, const int *__restrict__ Brp,
                                        const int *__restrict__ Bcol, int ncols, bool active, int gt, int *keys,
                                        EnumScratch<float, WPR * kWave> &en, int *s_cnt, int *out, int *err)
{
    constexpr int T = 1 << LOGT;
    constexpr int G = WPR * kWave;
    if constexpr (WPR == 1 && LOGT <= kSmallLogT && SMALL) {
        SmallRow r;
        if (!active) return;
        if (small_row<float, false>(e0, e1, Acol, nullptr, Brp, Bcol, nullptr, ncols, en.pincl, r)) {
            if (gt == 0) *out = r.count;
            return;
        }
    }
    for (int t = gt; t < T; t += G) keys[t] = kEmpty;
    if (gt == 0) *s_cnt = 0;
    group_sync<WPR>();
    int mine = 0;
    if (active) {
        auto get = [&](int e, int &bs, int &bl, float &) {
            const int k = Acol[e];
            bs = Brp[k];
            bl = Brp[k + 1] - bs;
        };
        auto sink = [&](const int (&j)[2], const bool (&ok)[2]) { mine += lds_insert_key_u<2>(keys, LOGT, j, ok, err); };
        group_products<float, false, G, 2, decltype(get), decltype(sink), true>(e0, e1, gt, en, Bcol,
                                                                                (const float *)nullptr, get, sink);
    }
    mine = wave_sum(mine);
    if (lane_id() == 0 && mine) atomicAdd(s_cnt, mine);
    group_sync<WPR>();
    if (active && gt == 0) *out = *s_cnt;
}

// Light rows of bin `bin`: one row per group of WPR waves (RPW groups per
// block; RPW > 1 only with WPR = 1).  The grid is persistent: the bin's rows
// and their number come from the device (perm + h->offset[bin],
// h->count[bin]) and the groups stride over them, so the launch needs no
// host-side count.  With RPW > 1 each group is one wave and loops on its
// own; with WPR > 1 the block is one group and loops as a whole.
template <int LOGT, int WPR, int RPW, bool SMALL = true>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_sym_rows(const int *__restrict__ Arp, const int *__restrict__ Acol,
                                                              const int *__restrict__ Brp, const int *__restrict__ Bcol,
                                                              const int *__restrict__ perm, const BinHdr *h, int bin,
                                                              int ncols, int *__restrict__ nnzc, int *err)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    constexpr int G = WPR * kWave;
    if (stopped(err)) return;
    __shared__ int s_keys[RPW][1 << LOGT];
    __shared__ EnumScratch<float, G> s_en[RPW];
    __shared__ int s_cnt[RPW];
    const int g = threadIdx.x / kWave / WPR;
    const int gt = threadIdx.x - g * G;
    const int nrows = h->count[bin];
    const int *rows = perm + h->offset[bin];
    for (int r0 = blockIdx.x * RPW; r0 < nrows; r0 += gridDim.x * RPW) {
        const int r = r0 + g;
        const bool active = r < nrows;
        const int row = active ? rows[r] : 0;
        const int e0 = active ? Arp[row] : 0, e1 = active ? Arp[row + 1] : 0;
        sym_row<LOGT, WPR, SMALL>(e0, e1, Acol, Brp, Bcol, ncols, active, gt, s_keys[g], s_en[g], &s_cnt[g], &nnzc[row],
                                  err);
        group_sync<WPR>();
    }
}

// Rows of all bins in one launch, for products of at most kFewRows rows (six
// launches, one per bin, cost more than the rows): work item `it` of a grid of
// 256-thread blocks is a row of the largest tables (one per item, all four
// waves), or four rows of up to 512 slots (a wave each).  body(bin constant,
// waves per row constant, first row, rows of the bin, its rows).
template <typename F>
__device__ __forceinline__ void few_items(const BinHdr &h, const int *__restrict__ perm, int it, F body)
{
    auto bin = [&](auto logt, auto wpr) {
        constexpr int B = decltype(logt)::value - kMinLogT, RPW = 4 / decltype(wpr)::value;
        const int items = (h.count[B] + RPW - 1) / RPW;
        if (it >= 0 && it < items) body(logt, wpr, it * RPW, h.count[B], perm + h.offset[B]);
        it -= items;
    };
    using std::integral_constant;
    bin(integral_constant<int, 11>(), integral_constant<int, 4>());
    bin(integral_constant<int, 10>(), integral_constant<int, 4>());
    bin(integral_constant<int, 9>(), integral_constant<int, 1>());
    bin(integral_constant<int, 8>(), integral_constant<int, 1>());
    bin(integral_constant<int, 7>(), integral_constant<int, 1>());
    bin(integral_constant<int, 6>(), integral_constant<int, 1>());
}

// Number of its work items.
__host__ __device__ __forceinline__ int few_count(const BinHdr &h)
{
    int n = 0;
    for (int b = 0; b < kLdsBins; ++b) n += b + kMinLogT >= 10 ? h.count[b] : (h.count[b] + 3) / 4;
    return n;
}

template <int LOGT, int WPR>
struct FewSymLds {
    int keys[4 / WPR][1 << LOGT];
    EnumScratch<float, WPR * kWave> en[4 / WPR];
    int cnt[4 / WPR];
};

__global__ __launch_bounds__(256) void k_sym_few(const int *__restrict__ Arp, const int *__restrict__ Acol,
                                                 const int *__restrict__ Brp, const int *__restrict__ Bcol,
                                                 const int *__restrict__ perm, const BinHdr *h, int ncols,
                                                 int *__restrict__ nnzc, int *err)
{
    if (stopped(err)) return;
    constexpr size_t BYTES = sizeof(FewSymLds<9, 1>) > sizeof(FewSymLds<11, 4>) ? sizeof(FewSymLds<9, 1>)
                                                                                : sizeof(FewSymLds<11, 4>);
    __shared__ __align__(16) unsigned char raw[BYTES];
    const int total = few_count(*h);
    for (int it = blockIdx.x; it < total; it += gridDim.x) {
        few_items(*h, perm, it, [&](auto logt, auto wpr, int r0, int cnt, const int *rows) {
            constexpr int LOGT = decltype(logt)::value, WPR = decltype(wpr)::value;
            auto &L = *reinterpret_cast<FewSymLds<LOGT, WPR> *>(raw);
            const int g = threadIdx.x / kWave / WPR, r = r0 + g;
            const bool active = r < cnt;
            const int row = active ? rows[r] : 0;
            sym_row<LOGT, WPR>(active ? Arp[row] : 0, active ? Arp[row + 1] : 0, Acol, Brp, Bcol, ncols, active,
                               threadIdx.x - g * WPR * kWave, L.keys[g], L.en[g], &L.cnt[g], &nnzc[row], err);
        });
        __syncthreads();
    }
}

// -------------------------------------------------------- numeric, LDS hash

// Key-value bitonic sort of n2 (a power of two) LDS entries by a group of G
// threads whose index in the group is gt.
template <typename V, int WPR>
__device__ __forceinline__ void group_bitonic(int *keys, V *vals, int n2, int gt)
{
    constexpr int G = WPR * kWave;
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int p = gt; p < (n2 >> 1); p += G) {
                const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1));
                const int l = i + j;
                const bool up = (i & k) == 0;
                const int ki = keys[i], kl = keys[l];
                if ((ki > kl) == up) {
                    keys[i] = kl;
                    keys[l] = ki;
                    const V vi = vals[i];
                    vals[i] = vals[l];
                    vals[l] = vi;
                }
            }
            group_sync<WPR>();
        }
    }
}

// Puts the entries of a row's table in column order at the front of the
// table (keys[0 .. total), vals[0 .. total)).  kr/vr hold each thread's SPT
// slots of the table (kEmpty where free), cnt/incl/wbase their count, its
// inclusive wave prefix and the wave's offset in the group; every thread of
// the group calls it.  The columns lie in [lo, lo + ncols).  With ncols at
// most 64 T the order comes from ranks in an occupancy bitmap over that
// range built in the table's own LDS; otherwise the entries are compacted
// and sorted (bitonic), or, for one wave and at most 64 entries, ranked by
// counting the smaller columns across the wave's lanes.  Only that second
// form reads total, cnt, incl and wbase.  Returns the number of entries:
// the bitmap's count, or total.
template <int T, int WPR, int SPT>
__device__ __forceinline__ int order_row_entries(const int (&kr)[SPT], const double (&vr)[SPT], int *keys,
                                                 double *vals, int *s_scan, int total, int wbase, int incl, int cnt,
                                                 int ncols, int gt, int lo = 0)
{
    constexpr int G = WPR * kWave;
    const int lane = lane_id(), wg = gt / kWave;
    group_sync<WPR>();
    if (ncols <= 64 * T) {
        // bitmap over B's columns in the value area (2T words), the prefix
        // of its popcounts per word (16-bit) in the key area; then every
        // entry's rank from two reads, and the entries staged in rank order
        // for coalesced stores.  Each thread takes 16 words per step.
        unsigned *bm = reinterpret_cast<unsigned *>(vals);
        unsigned *pw = reinterpret_cast<unsigned *>(keys);
        const unsigned short *pref = reinterpret_cast<const unsigned short *>(keys);
        const int W16 = (((ncols + 31) >> 5) + 15) & ~15;     // at most 2T
        for (int t = gt; t < W16; t += G) bm[t] = 0u;
        group_sync<WPR>();
#pragma unroll
        for (int s = 0; s < SPT; ++s)
            if (kr[s] != kEmpty) atomicOr(&bm[(kr[s] - lo) >> 5], 1u << ((kr[s] - lo) & 31));
        group_sync<WPR>();
        int run = 0;
        for (int g0 = 0; g0 < W16; g0 += 16 * G) {
            const int w0 = g0 + gt * 16;
            int c[16];
            int pc = 0;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                c[q] = w0 < W16 ? __popc(bm[w0 + q]) : 0;
                pc += c[q];
            }
            const int inc = wave_incl_scan(pc);
            if (lane == kWave - 1) s_scan[wg] = inc;
            group_sync<WPR>();
            int wb = 0, tot = 0;
            for (int w = 0; w < WPR; ++w) {
                const int t = s_scan[w];
                if (w < wg) wb += t;
                tot += t;
            }
            if (w0 < W16) {
                unsigned p = (unsigned)(run + wb + inc - pc);
#pragma unroll
                for (int q = 0; q < 16; q += 2) {
                    const unsigned p1 = p + c[q];
                    pw[(w0 >> 1) + (q >> 1)] = p | (p1 << 16);
                    p = p1 + c[q + 1];
                }
            }
            run += tot;
            group_sync<WPR>();
        }
        int rk[SPT];
#pragma unroll
        for (int s = 0; s < SPT; ++s) {
            rk[s] = -1;
            if (kr[s] != kEmpty) {
                const int j = kr[s] - lo, w = j >> 5;
                rk[s] = (int)pref[w] + __popc(bm[w] & ((1u << (j & 31)) - 1u));
            }
        }
        group_sync<WPR>();
#pragma unroll
        for (int s = 0; s < SPT; ++s)
            if (rk[s] >= 0 && rk[s] < T) {
                keys[rk[s]] = kr[s];
                vals[rk[s]] = vr[s];
            }
        total = run;
    } else {
        int pos = wbase + incl - cnt;
#pragma unroll
        for (int s = 0; s < SPT; ++s) {
            if (kr[s] != kEmpty) {
                keys[pos] = kr[s];
                vals[pos] = vr[s];
                ++pos;
            }
        }
        if constexpr (WPR == 1) {
            if (total <= kWave) {
                // one wave, at most 64 entries: lane l takes entry l, and its
                // rank is the number of smaller columns, counted over the
                // wave's lanes (no sorting network, no LDS round trips)
                wave_sync();
                const int lane = lane_id();
                const int k = lane < total ? keys[lane] : 0x7fffffff;
                const double v = lane < total ? vals[lane] : 0.0;
                int r = 0;
                for (int q = 0; q < total; ++q) r += __builtin_amdgcn_readlane(k, q) < k;
                wave_sync();
                if (lane < total) {
                    keys[r] = k;
                    vals[r] = v;
                }
                wave_sync();
                return total;
            }
        }
        const int n2 = total <= 1 ? 1 : (1 << ceil_log2(total));
        for (int t = total + gt; t < n2; t += G) keys[t] = 0x7fffffff;
        group_sync<WPR>();
        group_bitonic<double, WPR>(keys, vals, n2, gt);
    }
    group_sync<WPR>();
    return total;
}

// Write-back of an order-preserving table (the paper's Write-back Phase,
// whose insertion sort finishes the order of a semi-sorted table).  kr/vr
// hold each thread's SPT slots; home(j) = j >> shift; D is the longest probe
// distance.  The occupied slots are compacted in "unwrapped" slot order:
// entries at or after their home slot by slot, then those that wrapped past
// the table's end.  In that order an entry lies at most D places from its
// place in column order (two entries can be out of order only if both lie
// within D slots of the lower one's home), so its rank is its position
// corrected by the entries within D places on either side that belong on
// its other side: the bounded form of insertion sort, one entry per thread.
// Leaves the entries in column order at the front of keys/vals; returns
// their number.  s_scan holds WPR + 1 ints.
template <int T, int WPR, int SPT>
__device__ __forceinline__ int order_row_entries_ord(const int (&kr)[SPT], const double (&vr)[SPT], int *keys,
                                                     double *vals, int *s_scan, int gt, int shift, int D)
{
    constexpr int G = WPR * kWave;
    const int lane = lane_id(), wg = gt / kWave;
    int packed = 0;                                   // non-wrapped | wrapped << 16
#pragma unroll
    for (int s = 0; s < SPT; ++s)
        if (kr[s] != kEmpty) packed += (gt * SPT + s) >= (int)((unsigned)kr[s] >> shift) ? 1 : (1 << 16);
    const int incl = wave_incl_scan(packed);
    group_sync<WPR>();
    if (lane == kWave - 1) s_scan[wg] = incl;
    group_sync<WPR>();
    int base = 0, tot = 0;
    for (int w = 0; w < WPR; ++w) {
        const int t = s_scan[w];
        if (w < wg) base += t;
        tot += t;
    }
    const int n0 = tot & 0xffff, total = n0 + (tot >> 16);
    const int ex = base + incl - packed;
    int p0 = ex & 0xffff, p1 = n0 + (ex >> 16);
#pragma unroll
    for (int s = 0; s < SPT; ++s) {
        if (kr[s] == kEmpty) continue;
        const int at = (gt * SPT + s) >= (int)((unsigned)kr[s] >> shift) ? p0++ : p1++;
        keys[at] = kr[s];
        vals[at] = vr[s];
    }
    group_sync<WPR>();
    int xk[SPT], rk[SPT];
    double xv[SPT];
#pragma unroll
    for (int q = 0; q < SPT; ++q) {
        const int i = gt + q * G;
        rk[q] = -1;
        if (i < total) {
            const int x = keys[i];
            int r = i;
            for (int d = 1; d <= D; ++d) {
                if (i - d >= 0 && keys[i - d] > x) --r;
                if (i + d < total && keys[i + d] < x) ++r;
            }
            xk[q] = x;
            xv[q] = vals[i];
            rk[q] = r;
        }
    }
    group_sync<WPR>();
#pragma unroll
    for (int q = 0; q < SPT; ++q)
        if (rk[q] >= 0 && rk[q] < T) {
            keys[rk[q]] = xk[q];
            vals[rk[q]] = xv[q];
        }
    group_sync<WPR>();
    return total;
}

// Numeric pass of one light row by a group of WPR waves (steps a5 and a7):
// the products of the row's A entries [e0, e1) times B merged in an LDS
// tag/value table of 2^LOGT slots, then written in column order at C's
// offset rb (nc entries expected).  When B has
// at most 64 * 2^LOGT columns the order comes from ranks in an occupancy
// bitmap over all of B's columns, built in the table's own LDS once its
// entries are in registers (no sort); otherwise the occupied slots are
// compacted and sorted (bitonic).
// HASH selects the table's hash: 0 = multiplicative, 1 = order-preserving
// (home slot j >> shift, shift = ceil(log2 ncols) - LOGT, at least 0, with
// the bounded insertion write-back of order_row_entries_ord; s_maxd is the
// group's LDS word for the longest probe).
template <typename V, int LOGT, int WPR, int HASH = 0, bool SMALL = true>
__device__ __forceinline__ void num_row(int e0, int e1, const int *__restrict__ Acol, const V *__restrict__ Aval,
                                        const int *__restrict__ Brp, const int *__restrict__ Bcol,
                                        const V *__restrict__ Bval, long long rb, int nc, bool active, int gt,
                                        int *keys, double *vals, EnumScratch<V, WPR * kWave> &en, int *s_scan,
                                        int *__restrict__ Ccol, V *__restrict__ Cval, int ncols, int *err,
                                        int *s_maxd = nullptr)
{
    constexpr int T = 1 << LOGT;
    constexpr int G = WPR * kWave;
    constexpr int SPT = T / G;          // slots per thread in the compaction
    static_assert(SPT >= 1, "table smaller than its group");
    const int lane = lane_id(), wg = gt / kWave;
    if constexpr (WPR == 1 && LOGT <= kSmallLogT && HASH == 0 && SMALL) {
        SmallRow r;
        if (!active) return;
        if (small_row<V, true>(e0, e1, Acol, Aval, Brp, Bcol, Bval, ncols, en.pincl, r)) {
            if (gt == 0 && nc != r.count) atomicOr(err, kErrCount);
            if (r.tail && r.pos < nc) {
                store_c(&Ccol[rb + r.pos], r.col);
                store_c(&Cval[rb + r.pos], (V)r.val);
            }
            return;
        }
    }
    const int lc = ceil_log2(ncols);
    const int shift = lc > LOGT ? lc - LOGT : 0;
    for (int t = gt; t < T; t += G) {
        keys[t] = kEmpty;
        vals[t] = 0.0;
    }
    if constexpr (HASH == 1)
        if (gt == 0) *s_maxd = 0;
    group_sync<WPR>();
    if (active) {
        auto get = [&](int e, int &bs, int &bl, V &a) {
            const int k = Acol[e];
            bs = Brp[k];
            bl = Brp[k + 1] - bs;
            a = Aval[e];
        };
        auto sink = [&](const int (&j)[2], const double (&p)[2], const bool (&ok)[2]) {
            if constexpr (HASH == 1) lds_insert_add_ord_u<2>(keys, vals, LOGT, shift, j, p, ok, s_maxd, err);
            else lds_insert_add_u<2>(keys, vals, LOGT, j, p, ok, err);
        };
        group_products<V, true, G, 2, decltype(get), decltype(sink), true>(e0, e1, gt, en, Bcol, Bval, get, sink);
    }
    group_sync<WPR>();
    if constexpr (HASH == 1) {
        int kr[SPT];
        double vr[SPT];
#pragma unroll
        for (int s = 0; s < SPT; ++s) {
            kr[s] = keys[gt * SPT + s];
            vr[s] = vals[gt * SPT + s];
        }
        const int D = *s_maxd;
        const int total = order_row_entries_ord<T, WPR, SPT>(kr, vr, keys, vals, s_scan, gt, shift, D);
        if (active) {
            if (gt == 0 && nc != total) atomicOr(err, kErrCount);
            const int nw = total < nc ? total : nc;
            for (int t = gt; t < nw; t += G) {
                store_c(&Ccol[rb + t], keys[t]);
                store_c(&Cval[rb + t], (V)vals[t]);
            }
        }
        return;
    }
    // compaction of the occupied slots to the front of the table
    int kr[SPT];
    double vr[SPT];
    int cnt = 0;
#pragma unroll
    for (int s = 0; s < SPT; ++s) {
        kr[s] = keys[gt * SPT + s];
        vr[s] = vals[gt * SPT + s];
        cnt += kr[s] != kEmpty;
    }
    const int incl = wave_incl_scan(cnt);
    if (lane == kWave - 1) s_scan[wg] = incl;
    group_sync<WPR>();
    int wbase = 0, total = 0;
    for (int w = 0; w < WPR; ++w) {
        const int t = s_scan[w];
        if (w < wg) wbase += t;
        total += t;
    }
    order_row_entries<T, WPR, SPT>(kr, vr, keys, vals, s_scan, total, wbase, incl, cnt, ncols, gt);
    if (active) {
        if (gt == 0 && nc != total) atomicOr(err, kErrCount);
        const int nw = total < nc ? total : nc;
        for (int t = gt; t < nw; t += G) {
            store_c(&Ccol[rb + t], keys[t]);
            store_c(&Cval[rb + t], (V)vals[t]);
        }
    }
}

// Light rows: one row per group of WPR waves (RPW groups per block).
template <typename V, int LOGT, int WPR, int RPW, int HASH = 0, bool SMALL = true>
__global__ __launch_bounds__(kWave *WPR *RPW) void k_num_rows(
    const int *__restrict__ Arp, const int *__restrict__ Acol, const V *__restrict__ Aval,
    const int *__restrict__ Brp, const int *__restrict__ Bcol, const V *__restrict__ Bval,
    const int *__restrict__ rows, int nrows, const long long *__restrict__ Crp, int *__restrict__ Ccol,
    V *__restrict__ Cval, int ncols, int *err)
{
    static_assert(RPW == 1 || WPR == 1, "multi-row blocks use one wave per row");
    constexpr int T = 1 << LOGT;
    constexpr int G = WPR * kWave;
    __shared__ int s_keys[RPW][T];
    __shared__ double s_vals[RPW][T];
    __shared__ EnumScratch<V, G> s_en[RPW];
    __shared__ int s_scan[RPW][WPR + 1];
    __shared__ int s_maxd[RPW];
    const int g = threadIdx.x / kWave / WPR;
    const int gt = threadIdx.x - g * G;
    const int r = blockIdx.x * RPW + g;
    const bool active = r < nrows;
    const int row = active ? rows[r] : 0;
    const int e0 = active ? Arp[row] : 0, e1 = active ? Arp[row + 1] : 0;
    const long long rb = active ? Crp[row] : 0;
    const int nc = active ? (int)(Crp[row + 1] - rb) : 0;
    num_row<V, LOGT, WPR, HASH, SMALL>(e0, e1, Acol, Aval, Brp, Bcol, Bval, rb, nc, active, gt, s_keys[g], s_vals[g],
                                s_en[g], s_scan[g], Ccol, Cval, ncols, err, &s_maxd[g]);
}

template <typename V, int LOGT, int WPR>
struct FewNumLds {
    double vals[4 / WPR][1 << LOGT];
    int keys[4 / WPR][1 << LOGT];
    EnumScratch<V, WPR * kWave> en[4 / WPR];
    int scan[4 / WPR][WPR + 1];
    int maxd[4 / WPR];
};

// Light rows of all bins of a product of few rows (see few_items): block b is
// work item b.
template <typename V, int HASH>
__global__ __launch_bounds__(256) void k_num_few(const int *__restrict__ Arp, const int *__restrict__ Acol,
                                                 const V *__restrict__ Aval, const int *__restrict__ Brp,
                                                 const int *__restrict__ Bcol, const V *__restrict__ Bval,
                                                 const int *__restrict__ perm, BinHdr h,
                                                 const long long *__restrict__ Crp, int *__restrict__ Ccol,
                                                 V *__restrict__ Cval, int ncols, int *err)
{
    constexpr size_t BYTES = sizeof(FewNumLds<V, 9, 1>) > sizeof(FewNumLds<V, 11, 4>) ? sizeof(FewNumLds<V, 9, 1>)
                                                                                      : sizeof(FewNumLds<V, 11, 4>);
    __shared__ __align__(16) unsigned char raw[BYTES];
    few_items(h, perm, blockIdx.x, [&](auto logt, auto wpr, int r0, int cnt, const int *rows) {
        constexpr int LOGT = decltype(logt)::value, WPR = decltype(wpr)::value;
        auto &L = *reinterpret_cast<FewNumLds<V, LOGT, WPR> *>(raw);
        const int g = threadIdx.x / kWave / WPR, r = r0 + g;
        const bool active = r < cnt;
        const int row = active ? rows[r] : 0;
        const long long rb = active ? Crp[row] : 0;
        num_row<V, LOGT, WPR, HASH>(active ? Arp[row] : 0, active ? Arp[row + 1] : 0, Acol, Aval, Brp, Bcol, Bval, rb,
                                    active ? (int)(Crp[row + 1] - rb) : 0, active,
                                    threadIdx.x - g * WPR * kWave,
                                    L.keys[g], L.vals[g], L.en[g], L.scan[g], Ccol, Cval, ncols, err, &L.maxd[g]);
    });
}

// ---------------------------------------------------------------- row scan

// out = exclusive prefix of cnt (int or int64 counts) in three passes over
// blocks of kScanItems entries; out[n] and *total receive the sum.
constexpr int kScanThreads = 256;
constexpr int kScanPer = 16;
constexpr int kScanItems = kScanThreads * kScanPer;

template <typename TIn>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(long long n, const TIn *__restrict__ cnt,
                                                              long long *__restrict__ bsum)
{
    __shared__ long long s_tmp[kScanThreads / kWave + 1];
    const long long base = (long long)blockIdx.x * kScanItems + threadIdx.x * kScanPer;
    long long s = 0;
#pragma unroll
    for (int t = 0; t < kScanPer; ++t)
        if (base + t < n) s += cnt[base + t];
    long long total;
    block_excl_scan<long long, kScanThreads>(s, s_tmp, total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_top(int nb, long long *__restrict__ bsum,
                                                           long long *__restrict__ total_out)
{
    __shared__ long long s_tmp[kScanThreads / kWave + 1];
    __shared__ long long s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int b0 = 0; b0 < nb; b0 += kScanThreads) {
        const int b = b0 + threadIdx.x;
        const long long v = b < nb ? bsum[b] : 0;
        long long tot;
        const long long ex = block_excl_scan<long long, kScanThreads>(v, s_tmp, tot);
        const long long carry = s_carry;
        if (b < nb) bsum[b] = carry + ex;
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total_out = s_carry;
}

template <typename TIn>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(long long n, const TIn *__restrict__ cnt,
                                                             const long long *__restrict__ boff,
                                                             const long long *__restrict__ total,
                                                             long long *__restrict__ out)
{
    __shared__ long long s_tmp[kScanThreads / kWave + 1];
    const long long base = (long long)blockIdx.x * kScanItems + threadIdx.x * kScanPer;
    long long v[kScanPer];
    long long s = 0;
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) {
        v[t] = base + t < n ? (long long)cnt[base + t] : 0;
        s += v[t];
    }
    long long tot;
    long long run = block_excl_scan<long long, kScanThreads>(s, s_tmp, tot) + boff[blockIdx.x];
#pragma unroll
    for (int t = 0; t < kScanPer; ++t) {
        if (base + t < n) out[base + t] = run;
        run += v[t];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = *total;
}

// The same for at most kFewRows counts, in one block.
template <typename TIn>
__device__ __forceinline__ void scan_few(int n, const TIn *__restrict__ cnt, long long *__restrict__ total,
                                         long long *__restrict__ out)
{
    constexpr int PER = kFewRows / kFewThreads;
    __shared__ long long s_tmp[kFewThreads / kWave + 1];
    const int base = threadIdx.x * PER;
    long long v[PER], sum = 0, tot;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        v[t] = base + t < n ? (long long)cnt[base + t] : 0;
        sum += v[t];
    }
    long long run = block_excl_scan<long long, kFewThreads>(sum, s_tmp, tot);
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        if (base + t < n) out[base + t] = run;
        run += v[t];
    }
    if (threadIdx.x == 0) out[n] = *total = tot;
}

template <typename TIn>
__global__ __launch_bounds__(kFewThreads) void k_scan_few(int n, const TIn *__restrict__ cnt,
                                                          long long *__restrict__ total, long long *__restrict__ out)
{
    scan_few<TIn>(n, cnt, total, out);
}

// Row pointers, numeric bins (see k_num_bins) and their binning of at most
// kFewRows rows in one launch.  With `host` (pinned memory) it is the symbolic
// pass's last kernel and copies the header's `words` ints there, also when the
// pass has stopped.
__global__ __launch_bounds__(kFewThreads) void k_plan_few(int m, const int *__restrict__ nnzc,
                                                          const unsigned char *__restrict__ sym_bin, DevHdr *h,
                                                          int *__restrict__ perm, long long *__restrict__ Crp,
                                                          int *__restrict__ host, int words)
{
    if (!stopped(&h->error)) {
        scan_few<int>(m, nnzc, &h->nnz_c, Crp);
        bin_few(m, [&](int i) { return num_bin(sym_bin[i], nnzc[i]); }, nullptr, nnzc, &h->num, nullptr, perm, nullptr,
                nullptr, nullptr, -1);
    }
    if (!host) return;
    __syncthreads();
    for (int t = threadIdx.x; t < words; t += kFewThreads)
        host[t] = __hip_atomic_load((const int *)h + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ------------------------------------------------------ heavy rows: chunks

// lower_bound of `x` in the ascending columns Bcol[lo, hi).
__device__ __forceinline__ int lower_bound_col(const int *__restrict__ Bcol, int lo, int hi, int x)
{
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (Bcol[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Split points of every B row at the chunk boundaries:
// Bsplit[k * (nchunks + 1) + c] = first position of row k with column >= c * kChunkCols.
__global__ __launch_bounds__(256) void k_bsplit(int brows, int nchunks, const int *__restrict__ Brp,
                                                const int *__restrict__ Bcol, int *__restrict__ Bsplit, const int *err)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long per = nchunks + 1;
    if (t >= (long long)brows * per || stopped(err)) return;
    const int k = (int)(t / per), c = (int)(t % per);
    const int b0 = Brp[k], b1 = Brp[k + 1];
    int pos;
    if (c == 0) pos = b0;
    else if (c == nchunks) pos = b1;
    else pos = lower_bound_col(Bcol, b0, b1, c * kChunkCols);
    Bsplit[t] = pos;
}

// Symbolic phase of heavy rows: block (w, h) marks the columns of heavy row h
// that fall in symbolic window w (kSymWinChunks chunks) in an LDS bitmap, then
// stores the number of columns of every chunk (wcnt) and adds them to the
// row's count.  The grid covers hcap heavy rows (the workspace's capacity, a
// host-side bound); the number present, sh->count[kBinHeavy], comes from the
// device, and blocks beyond it return at once.  Bound by instruction issue
// (three quarters of the cycles at RMAT scale 19) and, where B is narrow, by
// the hub rows, which one block works through alone.  With products located per
// piece of 16 and the next lists' gathers in flight: scale 19 8.0 -> 6.7 ms, the
// rectangular product (scale 21 times 4096 columns) 0.79 -> 0.44 ms; two
// products in flight instead of four: 6.8 and 0.52.
constexpr int kSymHeavyThreads = 256;
constexpr int kSymU = 4;                // products in flight per thread and step

__global__ __launch_bounds__(kSymHeavyThreads) void k_sym_heavy(
    const int *__restrict__ Arp, const int *__restrict__ Acol, const int *__restrict__ Bcol,
    const int *__restrict__ Bsplit, long long per, const int *__restrict__ perm, const BinHdr *sh, int hcap,
    int nchunks, int *__restrict__ wcnt, int *__restrict__ nnzc, const int *err)
{
    constexpr int G = kSymHeavyThreads;
    constexpr int WG = G / kWave;
    constexpr int WORDS = kSymWinChunks * kChunkWords;
    __shared__ unsigned bm[WORDS];
    __shared__ PieceScratch<float, G> S;
    // window-major: blocks launched together share one column window of B
    const int w = blockIdx.x / hcap, h = blockIdx.x % hcap;
    if (h >= sh->count[kBinHeavy] || stopped(err)) return;
    const int row = perm[sh->offset[kBinHeavy] + h];
    const int gt = threadIdx.x, lane = lane_id(), wg = gt / kWave;
    const int c0 = w * kSymWinChunks;
    const int c1 = c0 + kSymWinChunks < nchunks ? c0 + kSymWinChunks : nchunks;
    const int lo = c0 * kChunkCols;
    for (int t = gt; t < WORDS; t += G) bm[t] = 0u;         // the products' first barrier follows
    // all words of the thread's products are read before any is tested, so
    // the reads overlap; most repeated columns then skip the atomic (an OR
    // after a stale read is merely redundant)
    auto sink = [&](const auto &j, const auto &ok) {
        constexpr int N = sizeof(j) / sizeof(j[0]);
        unsigned w[N];
#pragma unroll
        for (int u = 0; u < N; ++u) w[u] = ok[u] ? bm[(j[u] - lo) >> 5] : ~0u;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const unsigned bit = 1u << ((j[u] - lo) & 31);
            if (!(w[u] & bit)) atomicOr(&bm[(j[u] - lo) >> 5], bit);
        }
    };
    piece_products<float, false, G, G, kSymU>(Arp[row], Arp[row + 1], gt, S, Acol, (const float *)nullptr, Bsplit + c0,
                                              per, c1 - c0, Bcol, (const float *)nullptr, sink);
    // per-chunk counts: one wave per chunk
    int local = 0;
    for (int c = wg; c < c1 - c0; c += WG) {
        int pc = 0;
        for (int t = lane; t < kChunkWords; t += kWave) pc += __popc(bm[c * kChunkWords + t]);
        pc = wave_sum(pc);
        if (lane == 0) wcnt[(long long)h * nchunks + c0 + c] = pc;
        local += pc;
    }
    if (lane == 0 && local) atomicAdd(&nnzc[row], local);
}

// Exclusive prefix of the chunk counts of every heavy row (row-relative output
// offsets of the chunks); one wave per heavy row, 64 chunks per step
// (coalesced).
__global__ __launch_bounds__(256) void k_chunk_prefix(const BinHdr *sh, int nchunks, const int *__restrict__ wcnt,
                                                      int *__restrict__ woff, const int *err)
{
    const int h = blockIdx.x * 4 + threadIdx.x / kWave;
    if (h >= sh->count[kBinHeavy] || stopped(err)) return;
    const int lane = lane_id();
    const long long base = (long long)h * nchunks;
    int run = 0;
    for (int c0 = 0; c0 < nchunks; c0 += kWave) {
        const int c = c0 + lane;
        const int v = c < nchunks ? wcnt[base + c] : 0;
        const int incl = wave_incl_scan(v);
        if (c < nchunks) woff[base + c] = run + incl - v;
        run += __shfl(incl, kWave - 1, kWave);
    }
}

// Cuts every heavy row into segments (one thread per heavy row): a chunk
// with more than kDenseMin columns is a dense segment of its own; otherwise
// consecutive chunks are merged while the count stays <= kSegCap and the
// span <= kSegMaxSpan chunks.  Pass 0 counts segments per block and bin;
// pass 1 writes them at offset[bin] + block base + rank in block.
//
// Segments of more than kSegHash entries are ranked where the row's A entries
// fit one list, and hashed by a block where they do not: a ranked segment then
// lists them and loads its products twice, and as it has at most 2048 entries,
// most of their ranges hold few products or none, which leaves most lanes of a
// piece idle.  Rows of 300 entries times B rows of 20, 60 and 150 in 1M columns:
// hashed 2.40, 3.66 and 7.23 ms a call, ranked 3.51, 4.64 and 9.65 (400 entries
// the same; 3000 times 32: 20.9 and 35.8).  Rows of 100 entries times 100 in
// 300000 columns: hashed 1.77, ranked 0.99; of 200 times 200 in 1M: 2.29 and
// 1.67.  RMAT scale 16, edge factor 16, times B rows of 16 in 200000 columns,
// rows of all lengths: 0.83, all hashed 0.87, all ranked 0.88.  See k_seg_scan
// for products that have few of them.
__device__ __forceinline__ int seg_bin(int count, int entries, bool dense)
{
    return dense ? kSegDense : count <= kSegHash ? 0 : entries <= kRankEntries ? 1 : 2;
}

template <typename F>
__device__ __forceinline__ void plan_row_segments(const int *__restrict__ wc, int nchunks, F emit)
{
    int c = 0;
    while (c < nchunks) {
        const int n0 = wc[c];
        if (n0 == 0) { ++c; continue; }
        if (n0 > kDenseMin) { emit(c, c + 1, n0, true); ++c; continue; }
        const int start = c;
        int sum = 0, last = c;
        while (c < nchunks && c - start < kSegMaxSpan) {
            const int n = wc[c];
            if (n > kDenseMin || sum + n > kSegCap) break;
            sum += n;
            if (n) last = c;
            ++c;
        }
        emit(start, last + 1, sum, false);
        c = last + 1;
    }
}

// Segments are laid out bin by bin and, within a bin, chunk by chunk (by
// their first chunk): blocks launched together then work on the same column
// slice of B, which stays in L2.  Pass 0 counts segments per (bin, chunk) in
// hist; k_seg_scan turns the counts into offsets (and cursors); pass 1 writes
// every segment at its (bin, chunk) cursor.  Blocks aggregate their counts
// in LDS (one global atomic per block and group) when the kSegBins x nchunks
// histogram fits kSegPlanLds entries.
constexpr int kSegPlanLds = 5464;       // 1366 chunks

__global__ __launch_bounds__(256) void k_seg_plan(int pass, const BinHdr *bh, const int *__restrict__ perm,
                                                  int nchunks, const int *__restrict__ wcnt,
                                                  const int *__restrict__ woff, const int *__restrict__ Arp,
                                                  const long long *__restrict__ Crp, int *__restrict__ hist,
                                                  SegHdr *sh, Seg *__restrict__ segs, const int *err)
{
    if (stopped(err)) return;
    const int nheavy = bh->count[kBinHeavy];
    const int *__restrict__ heavy_rows = perm + bh->offset[kBinHeavy];
    __shared__ unsigned long long s_nnz[kSegBins];
    __shared__ int s_cnt[kSegPlanLds];
    const int cells = kSegBins * nchunks;
    const bool local = cells <= kSegPlanLds;
    if (threadIdx.x < kSegBins) s_nnz[threadIdx.x] = 0;
    if (local)
        for (int t = threadIdx.x; t < cells; t += 256) s_cnt[t] = 0;
    __syncthreads();
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    const int *wc = wcnt + (long long)h * nchunks;
    int row = 0, e0 = 0, e1 = 0;
    if (h < nheavy) {
        row = heavy_rows[h];
        e0 = Arp[row];
        e1 = Arp[row + 1];
    }
    // count this block's segments per (bin, chunk)
    if (h < nheavy) {
        long long lnnz[kSegBins] = {};
        plan_row_segments(wc, nchunks, [&](int a, int, int n, bool dense) {
            const int b = seg_bin(n, e1 - e0, dense);
            if (pass == 0) {
                if (local) atomicAdd(&s_cnt[b * nchunks + a], 1);
                else atomicAdd(&hist[(long long)b * nchunks + a], 1);
                lnnz[b] += n;
            } else if (local) {
                atomicAdd(&s_cnt[b * nchunks + a], 1);
            }
        });
        if (pass == 0)
            for (int b = 0; b < kSegBins; ++b)
                if (lnnz[b]) atomicAdd(&s_nnz[b], (unsigned long long)lnnz[b]);
    }
    __syncthreads();
    if (pass == 0) {
        if (local)
            for (int t = threadIdx.x; t < cells; t += 256)
                if (s_cnt[t]) atomicAdd(&hist[t], s_cnt[t]);
        if (threadIdx.x < kSegBins && s_nnz[threadIdx.x])
            atomicAdd((unsigned long long *)&sh->nnz[threadIdx.x], s_nnz[threadIdx.x]);
        return;
    }
    // pass 1: reserve this block's range of every group, then place
    if (local)
        for (int t = threadIdx.x; t < cells; t += 256)
            s_cnt[t] = s_cnt[t] ? atomicAdd(&hist[t], s_cnt[t]) : 0;
    __syncthreads();
    if (h < nheavy) {
        const long long rb = Crp[row];
        const int *wo = woff + (long long)h * nchunks;
        plan_row_segments(wc, nchunks, [&](int a, int b, int n, bool dense) {
            const int bin = seg_bin(n, e1 - e0, dense);
            const int cell = bin * nchunks + a;
            const int pos = local ? atomicAdd(&s_cnt[cell], 1) : atomicAdd(&hist[cell], 1);
            segs[pos] = Seg{row, e0, e1, a, b, n, rb + wo[a]};
        });
    }
}

// Offsets of the segment bins and of every (bin, chunk) group; hist becomes
// the write cursor of each group (one wave).  Block-hashed segments that are few
// beside the ranked ones are ranked, chunk by chunk with these: a launch of their
// own has a long tail (RMAT 40009, edge factor 16, FP64: 696 us a call, 712 with
// it), and ranked after the others they read the columns' slices of B again
// (RMAT scale 21, edge factor 4: 22.2 ms in k_num_rank, 23.5 so).
__global__ __launch_bounds__(kWave) void k_seg_scan(int nchunks, int *__restrict__ hist, SegHdr *sh, const int *err)
{
    if (stopped(err)) return;
    const int lane = lane_id();
    int ranked = 0, hashed = 0;
    for (int c = lane; c < nchunks; c += kWave) {
        ranked += hist[nchunks + c];
        hashed += hist[2LL * nchunks + c];
    }
    const bool join = 4LL * wave_sum(hashed) <= wave_sum(ranked);
    int run = 0;
    for (int b = 0; b < kSegBins; ++b) {
        if (lane == 0) sh->offset[b] = run;
        const int start = run;
        if (!(join && b == 2))
            for (int c0 = 0; c0 < nchunks; c0 += kWave) {
                const int c = c0 + lane;
                const long long at = (long long)b * nchunks + c;
                const int own = c < nchunks ? hist[at] : 0;
                const int v = own + (join && b == 1 && c < nchunks ? hist[at + nchunks] : 0);
                const int incl = wave_incl_scan(v);
                if (c < nchunks) {
                    hist[at] = run + incl - v;
                    if (join && b == 1) hist[at + nchunks] = run + incl - v + own;
                }
                run += __shfl(incl, kWave - 1, kWave);
            }
        if (lane == 0) sh->count[b] = run - start;
    }
    if (lane == 0) sh->offset[kSegBins] = run;
}

// Hashed segment of a heavy row: products of the row whose columns lie in
// chunks [c0, c1) merged in an LDS table of 2^LOGT slots; entries ranked by
// an occupancy bitmap of the segment's columns (built in the table's own
// storage once the entries are in registers, so the block needs no other
// LDS and more blocks fit a CU), staged in column order and copied out with
// coalesced stores.
template <typename V, int LOGT, int THREADS>
__global__ __launch_bounds__(THREADS) void k_num_seg(
    const int *__restrict__ Acol, const V *__restrict__ Aval, const int *__restrict__ Bcol,
    const V *__restrict__ Bval, const int *__restrict__ Bsplit, long long per, const Seg *__restrict__ segs,
    int *__restrict__ Ccol, V *__restrict__ Cval, int *err)
{
    constexpr int T = 1 << LOGT;
    constexpr int SPT = T / THREADS;
    static_assert(SPT >= 1, "table smaller than the block");
    constexpr int WPR = THREADS / kWave;
    __shared__ int keys[T];
    __shared__ double vals[T];
    __shared__ EnumScratch<V, THREADS> S;
    __shared__ int s_scan[WPR + 1];
    const Seg sg = segs[blockIdx.x];
    const int gt = threadIdx.x;
    const int lo = sg.c0 * kChunkCols;
    const int *__restrict__ split0 = Bsplit + sg.c0;
    const int *__restrict__ split1 = Bsplit + sg.c1;
    for (int t = gt; t < T; t += THREADS) {
        keys[t] = kEmpty;
        vals[t] = 0.0;
    }
    __syncthreads();
    auto get = [&](int e, int &bs, int &bl, V &a) {
        const int k = Acol[e];
        bs = split0[k * per];
        bl = split1[k * per] - bs;
        a = Aval[e];
    };
    // one product per thread in flight: the segment kernels are bound by how
    // many blocks fit a CU, and fewer registers per thread let more in
    auto sink = [&](const int (&j)[1], const double (&p)[1], const bool (&ok)[1]) {
        lds_insert_add_u<1>(keys, vals, LOGT, j, p, ok, err);
    };
    group_products<V, true, THREADS, 1, decltype(get), decltype(sink), true>(sg.e0, sg.e1, gt, S, Bcol, Bval, get,
                                                                            sink);
    __syncthreads();
    int kr[SPT];
    double vr[SPT];
    int cnt = 0;
#pragma unroll
    for (int s = 0; s < SPT; ++s) {
        kr[s] = keys[gt * SPT + s];
        vr[s] = vals[gt * SPT + s];
        cnt += kr[s] != kEmpty;
    }
    int incl = 0, wbase = 0, total = 0;
    if constexpr (64 * T < kSegMaxSpan * kChunkCols) {
        // a segment can be too wide for the bitmap ranks, and the sort that
        // takes it then needs each thread's place among the entries
        const int lane = lane_id(), wg = gt / kWave;
        incl = wave_incl_scan(cnt);
        if (lane == kWave - 1) s_scan[wg] = incl;
        __syncthreads();
        for (int w = 0; w < WPR; ++w) {
            const int t = s_scan[w];
            if (w < wg) wbase += t;
            total += t;
        }
    }
    total = order_row_entries<T, WPR, SPT>(kr, vr, keys, vals, s_scan, total, wbase, incl, cnt,
                                           (sg.c1 - sg.c0) * kChunkCols, gt, lo);
    if (gt == 0 && total != sg.count) atomicOr(err, kErrCount);
    const long long out0 = sg.out;
    const int n = total < sg.count ? total : sg.count;
    for (int t = gt; t < n; t += THREADS) {
        store_c(&Ccol[out0 + t], keys[t]);
        store_c(&Cval[out0 + t], (V)vals[t]);
    }
}

// Ranked segments of heavy rows: at most kSegCap entries in at most
// kSegMaxSpan chunks.  A first pass over a segment's products marks their
// columns in an LDS bitmap; with the bitmap's prefix counts every column's
// rank is two LDS reads, so a second pass adds each product straight into its
// entry's sum and notes its column: no table, no probing, and the entries are
// in column order when the pass ends.  Products are loaded once, into
// registers (HOLD steps per wave; more than that takes them from memory
// twice).
//
// A segment has some 1900 products, four per thread, so a block that starts
// from nothing spends its time in a chain of six memory latencies.  The grid
// is persistent (the LDS, 48 KB FP32 and 49 KB FP64, lets three blocks of
// eight waves share a CU) and the chain is spread over three segments: while
// one is marked and added, the next one's A entries and split points are on
// their way, and its products are loaded before this one is written out.
// RMAT scale 19 A * A FP32 (1.5M segments): 10.9 ms, 11.6 without the
// persistent grid, 13.9 loading the products twice, 12.9 with four waves;
// hashed segments of up to 1024 entries in 8 chunks (3.4M of them) took 21.3.
constexpr int kRankThreads = 512;
constexpr int kRankWords = kSegMaxSpan * kChunkWords;

template <typename V>
__global__ __launch_bounds__(kRankThreads, 6) void k_num_rank(
    const int *__restrict__ Acol, const V *__restrict__ Aval, const int *__restrict__ Bcol,
    const V *__restrict__ Bval, const int *__restrict__ Bsplit, long long per, const Seg *__restrict__ segs, int nseg,
    int *__restrict__ Ccol, V *__restrict__ Cval, int *err)
{
    constexpr int G = kRankThreads, NW = G / kWave, WPT = kRankWords / G, GE = kRankEntries;
    constexpr int HOLD = 4096 / G;      // steps of products held in registers
    static_assert(WPT == 8, "one 16-byte store of prefix counts per thread");
    __shared__ __align__(16) unsigned bm[kRankWords];
    __shared__ __align__(16) unsigned short pref[kRankWords];   // entries below each word
    __shared__ double vals[kSegCap];
    __shared__ unsigned short cols[kSegCap];                    // low 16 bits of each entry's column
    __shared__ PieceScratch<V, GE> S;
    __shared__ int s_scan[NW];
    const int gt = threadIdx.x, lane = lane_id(), wg = __builtin_amdgcn_readfirstlane(gt / kWave);
    const int w0 = gt * WPT;
    const int last = nseg - 1, step = gridDim.x;
    auto at = [&](int i) { return segs[i < last ? i : last]; };
    // the products of the segment at hand, its located pieces and its list
    int hc[HOLD], st = 0, en = 0, left = 0;
    V hv[HOLD], al = V(0);
    bool hok[HOLD], held = false;
    auto entries = [](const Seg &g) { return g.e1 - g.e0 < GE ? g.e1 - g.e0 : GE; };
    auto locate_and_load = [&](const Seg &g) {
        const int P = piece_count(S);
        held = g.e1 - g.e0 <= GE && P <= NW * HOLD * 4;
        if (!held) return;
        const int share = piece_share<NW>(P), p0 = wg * share;
        left = (p0 + share < P ? p0 + share : P) - p0;
        piece_locate<V, true, GE>(p0, p0 + left, g.e1 - g.e0, S, st, en, al);
        auto load = [&](auto t) {
            constexpr int T = decltype(t)::value;
            const int q = row_bcast<T>(st) + (lane & (kPiece - 1));
            hok[T] = q < row_bcast<T>(en);
            const int pos = hok[T] ? q : 0;
            hc[T] = Bcol[pos];
            hv[T] = Bval[pos];
        };
        piece_each<HOLD>(left, load);
    };
    auto clear = [&]() {
        *(uint4 *)&bm[w0] = make_uint4(0, 0, 0, 0);
        *(uint4 *)&bm[w0 + 4] = make_uint4(0, 0, 0, 0);
    };
    Seg sg = at(blockIdx.x), nx = at(blockIdx.x + step);
    {
        int bs = 0, bl = 0;
        V a = V(0);
        if (gt < entries(sg)) {
            const long long k = Acol[sg.e0 + gt] * per;
            a = Aval[sg.e0 + gt];
            bs = Bsplit[k + sg.c0];
            bl = Bsplit[k + sg.c1] - bs;
        }
        piece_list<V, true, GE>(entries(sg), gt, bs, bl, a, S);
        clear();
        __syncthreads();
        locate_and_load(sg);
    }
    for (int i = blockIdx.x; i < nseg; i += step) {
        const Seg nn = at(i + 2 * step);
        const int lo = sg.c0 * kChunkCols, W = (sg.c1 - sg.c0) * kChunkWords;
        // the next segment's A entries
        const int ne = entries(nx);
        int nbs = 0, nbl = 0;
        long long nk = 0;
        V na = V(0);
        if (gt < ne) {
            nk = Acol[nx.e0 + gt] * per;
            na = Aval[nx.e0 + gt];
        }
        for (int t = gt; t < sg.count; t += G) vals[t] = 0.0;
        // the general form of a pass: the row's entries, a list at a time
        auto pass = [&](auto with_val, auto &sink) {
            piece_products<V, decltype(with_val)::value, GE, G, 1, false>(sg.e0, sg.e1, gt, S, Acol, Aval, Bsplit + sg.c0,
                                                                          per, sg.c1 - sg.c0, Bcol, Bval, sink);
        };
        if (held) {
            auto mark = [&](auto t) {
                constexpr int T = decltype(t)::value;
                hc[T] -= lo;
                if (hok[T]) atomicOr(&bm[hc[T] >> 5], 1u << (hc[T] & 31));
            };
            piece_each<HOLD>(left, mark);
        } else {
            auto mark = [&](const auto &j, const auto &ok) {
                constexpr int N = sizeof(j) / sizeof(j[0]);
                unsigned w[N];
#pragma unroll
                for (int u = 0; u < N; ++u) w[u] = ok[u] ? bm[(j[u] - lo) >> 5] : ~0u;
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const unsigned bit = 1u << ((j[u] - lo) & 31);
                    if (!(w[u] & bit)) atomicOr(&bm[(j[u] - lo) >> 5], bit);
                }
            };
            pass(std::false_type(), mark);
        }
        // the next segment's split points
        if (gt < ne) {
            nbs = Bsplit[nk + nx.c0];
            nbl = Bsplit[nk + nx.c1];
        }
        __syncthreads();
        // prefix counts: eight words per thread
        int pc = 0;
        unsigned pw[WPT / 2];
        if (w0 < W) {
#pragma unroll
            for (int q = 0; q < WPT; q += 4) {
                const uint4 v = *(const uint4 *)&bm[w0 + q];
                pw[q / 2] = (unsigned)pc | (unsigned)(pc + __popc(v.x)) << 16;
                pc += __popc(v.x) + __popc(v.y);
                pw[q / 2 + 1] = (unsigned)pc | (unsigned)(pc + __popc(v.z)) << 16;
                pc += __popc(v.z) + __popc(v.w);
            }
        }
        const int inc = wave_incl_scan(pc);
        if (lane == kWave - 1) s_scan[wg] = inc;
        __syncthreads();
        int run = 0, total = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int t = s_scan[w];
            if (w < wg) run += t;
            total += t;
        }
        if (w0 < W) {
            const unsigned add = (unsigned)(run + inc - pc) * 0x10001u;
            *(uint4 *)&pref[w0] = make_uint4(pw[0] + add, pw[1] + add, pw[2] + add, pw[3] + add);
        }
        __syncthreads();
        if (gt == 0 && total != sg.count) atomicOr(err, kErrCount);
        const int cnt = total < sg.count ? total : sg.count;
        auto rank = [&](int c) { return pref[c >> 5] + __popc(bm[c >> 5] & ((1u << (c & 31)) - 1u)); };
        if (held) {
            auto put = [&](auto t) {
                constexpr int T = decltype(t)::value;
                const double p = (double)row_bcast<T>(al) * (double)hv[T];
                if (hok[T]) {
                    const int r = rank(hc[T]);
                    if (r < cnt) {
                        atomicAdd(&vals[r], p);
                        cols[r] = (unsigned short)hc[T];
                    }
                }
            };
            piece_each<HOLD>(left, put);
        } else {
            auto put = [&](const auto &j, const auto &p, const auto &ok) {
                constexpr int N = sizeof(j) / sizeof(j[0]);
                int r[N];
#pragma unroll
                for (int u = 0; u < N; ++u) r[u] = ok[u] ? rank(j[u] - lo) : kSegCap;
#pragma unroll
                for (int u = 0; u < N; ++u)
                    if (r[u] < cnt) {
                        atomicAdd(&vals[r[u]], p[u]);
                        cols[r[u]] = (unsigned short)(j[u] - lo);
                    }
            };
            pass(std::true_type(), put);
        }
        // entries from `half` on lie 65536 or more columns above lo
        const int half = W > 2048 ? pref[2048] : cnt;
        const long long out = sg.out;
        piece_list<V, true, GE>(ne, gt, nbs, nbl - nbs, na, S);
        __syncthreads();
        clear();
        sg = nx;
        nx = nn;
        if (i + step < nseg) locate_and_load(sg);
        for (int t = gt; t < cnt; t += G) {
            store_c(&Ccol[out + t], lo + cols[t] + (t >= half ? 65536 : 0));
            store_c(&Cval[out + t], (V)vals[t]);
        }
        __syncthreads();
    }
}

constexpr long long kNegZeroBits = (long long)0x8000000000000000ULL;

// A slot of a dense window was reached by a product when its sum is no
// longer the bit pattern of -0.0 (the window starts at -0.0 and every
// product is added as p + 0.0).
__device__ __forceinline__ bool reached(double v) { return __double_as_longlong(v) != kNegZeroBits; }

// Mask of the lanes of the wave for which p holds (a compare straight into
// a scalar register pair, with no 0/1 select in between).
__device__ __forceinline__ unsigned long long wave_ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Number of lanes below this one whose bit is set in m.
__device__ __forceinline__ int lanes_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Stores the entries a wave has ranked in its ROUNDS x 64 slots of a dense
// window: slot r * 64 + lane holds column col0 + r * 64 + lane and value
// vr[r], occupied where reached(vr[r]); msk[r] = wave_ballot(reached(vr[r])).  The first n of them,
// in column order, go to C[out, out + n): staged in the wave's own LDS slots
// (whose values are already in registers) and copied with consecutive lanes
// on consecutive addresses, so stores cover whole cache lines.  FP32 stages
// (column, value) pairs in one pass, FP64 columns and then values.  Every
// lane of the wave calls it; the slots are left dirty.
template <typename V, int ROUNDS>
__device__ __forceinline__ void wave_store_ranked(const double (&vr)[ROUNDS], const unsigned long long (&msk)[ROUNDS],
                                                  double *slots, int col0, long long out, int n,
                                                  int *__restrict__ Ccol, V *__restrict__ Cval)
{
    const int lane = lane_id();
    int lr = 0;
    if constexpr (sizeof(V) == 4) {
        int2 *st = reinterpret_cast<int2 *>(slots);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (reached(vr[r]))
                st[lr + lanes_below(msk[r])] = make_int2(col0 + r * kWave + lane, __float_as_int((float)vr[r]));
            lr += __popcll(msk[r]);
        }
        wave_sync();
        for (int k = lane; k < n; k += kWave) {
            const int2 e = st[k];
            store_c(&Ccol[out + k], e.x);
            store_c(&Cval[out + k], (V)__int_as_float(e.y));
        }
    } else {
        int *st_col = reinterpret_cast<int *>(slots);
        V *st_val = reinterpret_cast<V *>(slots);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (reached(vr[r])) st_col[lr + lanes_below(msk[r])] = col0 + r * kWave + lane;
            lr += __popcll(msk[r]);
        }
        wave_sync();
        for (int k = lane; k < n; k += kWave) store_c(&Ccol[out + k], st_col[k]);
        wave_sync();
        lr = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (reached(vr[r])) st_val[lr + lanes_below(msk[r])] = (V)vr[r];
            lr += __popcll(msk[r]);
        }
        wave_sync();
        for (int k = lane; k < n; k += kWave) store_c(&Cval[out + k], st_val[k]);
    }
    wave_sync();
}

// Dense chunk of a heavy row: products whose columns lie in chunk c0 added
// directly into an LDS array of doubles indexed by column; each wave then
// ranks its own 1024 columns with ballots, stages its entries in column
// order in those same LDS slots and copies them to C with whole-line stores.
// Occupancy needs no bitmap: the array starts at -0.0 and every product is
// added as p + 0.0, which is never -0.0, so a column was reached exactly when
// its sum is no longer the bit pattern of -0.0 (a sum of terms that are not
// -0.0 is never -0.0 under round-to-nearest, even when they cancel).
//
// The kernel is persistent: a grid that fills the GPU once (two blocks of
// eight waves per CU, by LDS) takes the dense chunks from a global queue (one
// atomic per `claim` chunks), so that long and short chunks balance across
// CUs, and each wave puts -0.0 back in its slots once its entries are out, so
// the array is ready for the next chunk without a separate clearing pass.
// Bound by traffic, with instruction issue close behind: RMAT scale 19 A * A
// FP32 (844K chunks, 4.9e9 products) moves 63 GB to and from the L2s in 14.7
// ms, 4.3 TB/s where a copy reaches 5.1 (one B entry per product, C once).
// With a search per product instead of per piece of 16 it was 17.9 ms, with
// four instead of up to eight products per thread in flight 16.9.  Chunks
// dealt ahead, their A entries and split points fetched while the one before
// is ranked, were no faster (15.1).
//
// SHORT: a product per lane instead of a piece, for chunks in which the average
// A entry selects fewer than two products, so that most lanes of a piece have
// none.  8192 rows of 5000 entries, B rows of one, 4096 columns: 1.81 ms a call,
// by pieces 2.09; 20000 entries, B rows of 4, 20000 columns: 0.85 and 1.10,
// 200000 columns 3.63 and 5.02 (4.56 and 5.02 with two and four products per
// thread in flight); 3000 entries, B rows of 16, 4096 columns: 0.77 and 0.75.
// In wide products, whose dense chunks are few and not average, the other way
// round (RMAT scale 20, edge factor 4, 256 chunks, three products: 18.8 and
// 18.1; scale 21, 3: 40.8 and 40.1), hence not beyond kDenseShortChunks.
constexpr int kDenseThreads = 512;
constexpr int kDenseShortChunks = 64;
// dense chunks a block claims with one atomic on the queue when every block
// has many to do (one atomic per chunk from every resident block serialises
// on the counter); one at a time otherwise, for the balance of the tail
constexpr int kDenseClaim = 4;
constexpr int kDenseClaimMinPerBlock = 256;

template <typename V, bool SHORT>
__global__ __launch_bounds__(kDenseThreads) void k_num_dense(
    const int *__restrict__ Acol, const V *__restrict__ Aval, const int *__restrict__ Bcol,
    const V *__restrict__ Bval, const int *__restrict__ Bsplit, long long per, const Seg *__restrict__ segs, int nseg,
    int claim, int *__restrict__ Ccol, V *__restrict__ Cval, int *err, int *queue)
{
    constexpr int G = kDenseThreads, NW = G / kWave;
    constexpr int CPW = kChunkCols / NW;              // columns ranked by each wave
    constexpr int ROUNDS = CPW / kWave;
    extern __shared__ __align__(16) unsigned char s_raw[];
    double *acc = (double *)s_raw;                      // [kChunkCols]
    __shared__ std::conditional_t<SHORT, EnumScratch<V, G>, PieceScratch<V, G>> S;
    __shared__ int s_wt[NW];
    __shared__ int s_next;
    const int gt = threadIdx.x, lane = lane_id(), wg = gt / kWave;
    for (int t = gt; t < kChunkCols; t += G) acc[t] = -0.0;
    for (int t = 0, last = 0;; ++t) {
        if (t >= last) {
            if (gt == 0) s_next = atomicAdd(queue, claim);
            __syncthreads();
            t = s_next;
            if (t >= nseg) break;
            last = t + claim < nseg ? t + claim : nseg;
        }
        const Seg sg = segs[t];
        const int lo = sg.c0 * kChunkCols;
        const int *__restrict__ split0 = Bsplit + sg.c0;
        auto sink = [&](const auto &j, const auto &p, const auto &ok) {
            constexpr int N = sizeof(j) / sizeof(j[0]);
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (ok[u]) atomicAdd(&acc[j[u] - lo], p[u] + 0.0);
        };
        // its first barrier also says that the previous chunk is fully written
        if constexpr (SHORT) {
            auto get = [&](int e, int &bs, int &bl, V &a) {
                const int k = Acol[e];
                bs = split0[k * per];
                bl = split0[k * per + 1] - bs;
                a = Aval[e];
            };
            group_products<V, true, G, 1, decltype(get), decltype(sink), true>(sg.e0, sg.e1, gt, S, Bcol, Bval, get,
                                                                               sink);
            __syncthreads();
        } else {
            piece_products<V, true, G, G, 4>(sg.e0, sg.e1, gt, S, Acol, Aval, split0, per, 1, Bcol, Bval, sink);
        }
        double vr[ROUNDS];
        unsigned long long msk[ROUNDS];
        int wcount = 0;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            vr[r] = acc[wg * CPW + r * kWave + lane];
            msk[r] = wave_ballot(reached(vr[r]));
            wcount += __popcll(msk[r]);
        }
        if (lane == 0) s_wt[wg] = wcount;
        __syncthreads();
        int run = 0, tot = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int c = s_wt[w];
            if (w < wg) run += c;
            tot += c;
        }
        if (gt == 0 && tot != sg.count) atomicOr(err, kErrCount);
        const int n = wcount < sg.count - run ? wcount : (sg.count - run > 0 ? sg.count - run : 0);
        wave_store_ranked<V, ROUNDS>(vr, msk, acc + wg * CPW, lo + wg * CPW, sg.out + run, n, Ccol, Cval);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) acc[wg * CPW + r * kWave + lane] = -0.0;   // cleared for the next chunk
        __syncthreads();                                // s_wt and s_next are reused
    }
}

// ---------------------------------------------- heavy rows: global hash path
//
// A row's table lies in global memory but belongs to one block, so everything
// about it has workgroup scope: atomics then run in the XCD's L2, where agent
// scope sends them to memory, and a barrier orders them, where a fence of
// agent scope writes the L2 back.

__device__ __forceinline__ int gload(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <typename V>
__device__ __forceinline__ V gload_v(const V *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Compare-and-swap kEmpty -> key; returns the previous key.
__device__ __forceinline__ int gclaim(int *p, int key)
{
    int old = kEmpty;
    __hip_atomic_compare_exchange_strong(p, &old, key, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
    return old;
}

// A slot of a numeric table: key and value side by side, so that a probe and
// the add that follows it touch one cache line.  `list` is not of this slot: in
// slot i < nc (the row's entries) it is the number of the i-th slot that was
// claimed, in slot nc + i that slot's key (a table has at least 2 nc slots).
struct alignas(16) GSlot {
    double val;
    int key;
    int list;
};

// Slots of the U columns j in a table of 2^logT keys, key_at(h) the address of
// slot h's (claimed where new; -1 for an absent product or a full table, which
// sets kErrProbe): the first reads of all U are in flight together, and a
// column that is there already costs no compare-and-swap.  claimed(slot, key)
// is called for every new key.
template <int U, typename K, typename F>
__device__ __forceinline__ void gfind(int logT, const int (&j)[U], const bool (&ok)[U], int (&slot)[U], int *err,
                                      K key_at, F claimed)
{
    const unsigned mask = (1u << logT) - 1;
    int cur[U];
    unsigned open = 0;                                   // products still looking for their slot
#pragma unroll
    for (int u = 0; u < U; ++u) {
        slot[u] = ok[u] ? (int)slot_of(j[u], logT) : -1;
        cur[u] = ok[u] ? gload(key_at(slot[u])) : 0;
        open |= ok[u] ? 1u << u : 0u;
    }
    for (unsigned probe = 0; open; ++probe) {
        // claims of free slots, all in flight, then the next reads
#pragma unroll
        for (int u = 0; u < U; ++u)
            if ((open >> u & 1) && cur[u] == kEmpty) {
                cur[u] = gclaim(key_at(slot[u]), j[u]);
                if (cur[u] == kEmpty) {
                    claimed(slot[u], j[u]);
                    open &= ~(1u << u);
                }
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (open >> u & 1) {
                if (cur[u] == j[u]) {
                    open &= ~(1u << u);
                } else if (probe >= mask) {
                    atomicOr(err, kErrProbe);
                    slot[u] = -1;
                    open &= ~(1u << u);
                } else {
                    slot[u] = (int)((unsigned)(slot[u] + 1) & mask);
                    cur[u] = gload(key_at(slot[u]));
                }
            }
    }
}

// Fills `n` ints with `v` (table initialisation).
__global__ __launch_bounds__(256) void k_fill_i32(long long n, int *__restrict__ p, int v)
{
    for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x)
        p[t] = v;
}

constexpr int kGlobalThreads = 512;

// In front of a row's global table lies an LDS table of 2^kFrontLog slots: a
// column takes one of its kFrontProbes home slots there if one is free when it
// first comes, else it lives in the global table, for the whole row either
// way.  The tables of the rows in flight are several times the L2 (16 B a slot,
// 8K slots a row, 256 CUs), so every access to them is a line from memory; the
// columns that come first, and a skewed row's frequent ones among them, stay
// on chip.
constexpr int kFrontLog = 12;
constexpr int kFrontProbes = 2;

// LDS slot of column j in the front table, -1 if both its places are taken;
// fresh: it was claimed now.
__device__ __forceinline__ int front_find(int *keys, int j, bool &fresh)
{
    unsigned h = slot_of(j, kFrontLog);
    fresh = false;
#pragma unroll
    for (int p = 0; p < kFrontProbes; ++p) {
        const int old = atomicCAS(&keys[h], kEmpty, j);
        fresh = old == kEmpty;
        if (fresh || old == j) return (int)h;
        h = (h + 1) & ((1u << kFrontLog) - 1);
    }
    return -1;
}

// Symbolic count of one heavy row in global mode by a whole block: the row's
// columns are inserted in its global key table of next_pow2(2 cap) slots
// (the table must hold kEmpty) and counted into *out.
__device__ __forceinline__ void sym_global_row(const int *__restrict__ Arp, const int *__restrict__ Acol,
                                               const int *__restrict__ Brp, const int *__restrict__ Bcol, int arow,
                                               int cap, int *keys, PieceScratch<float, kGlobalThreads> &S, int *front,
                                               int *s_cnt, int *out, int *err)
{
    const int logT = gtable_log2(cap);
    for (int t = threadIdx.x; t < 1 << kFrontLog; t += kGlobalThreads) front[t] = kEmpty;
    if (threadIdx.x == 0) *s_cnt = 0;                      // the products' first barrier follows
    int mine = 0;
    auto sink = [&](const auto &j, const auto &ok) {
        constexpr int N = sizeof(j) / sizeof(j[0]);
        int slot[N];
        bool far[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            bool fresh = false;
            far[u] = ok[u] && front_find(front, j[u], fresh) < 0;
            mine += fresh;
        }
        gfind<N>(logT, j, far, slot, err, [&](int h) { return &keys[h]; }, [&](int, int) { ++mine; });
    };
    piece_products<float, false, kGlobalThreads, kGlobalThreads, 4>(Arp[arow], Arp[arow + 1], threadIdx.x, S, Acol,
                                                                    (const float *)nullptr, Brp, 1, 1, Bcol,
                                                                    (const float *)nullptr, sink);
    __syncthreads();
    mine = wave_sum(mine);
    if (lane_id() == 0 && mine) atomicAdd(s_cnt, mine);
    __syncthreads();
    if (threadIdx.x == 0) *out = *s_cnt;
}

// Symbolic phase of heavy rows in global mode: one block per row.
__global__ __launch_bounds__(kGlobalThreads) void k_sym_global(
    const int *__restrict__ Arp, const int *__restrict__ Acol, const int *__restrict__ Brp,
    const int *__restrict__ Bcol, const int *__restrict__ rows, const int *__restrict__ cap,
    const long long *__restrict__ goff, long long gbase, int *gkeys, int *__restrict__ nnzc, int *err)
{
    __shared__ PieceScratch<float, kGlobalThreads> S;
    __shared__ int s_front[1 << kFrontLog];
    __shared__ int s_cnt;
    const int row = rows[blockIdx.x];
    sym_global_row(Arp, Acol, Brp, Bcol, row, cap[row], gkeys + (goff[blockIdx.x] - gbase), S, s_front, &s_cnt,
                   &nnzc[row], err);
}

// Numeric pass of one heavy row in global mode by a whole block: clears the
// row's global table, merges the row's products into it with compare-and-swap
// on the key and atomic add on the FP64 value (the sum is rounded to the output
// type once, at write-out), then writes the entries in column order at C's row
// `crow`.  Every slot the row claims is appended, with its column, to the row's
// touched-slot list (nc entries: the paper's third version keeps its tags in
// dense arrays with an offset array for the same purpose), so the write-out
// reads the row's nc entries instead of scanning all T >= 2 nc slots of its
// table: per window of kGlobalRankBits columns, the listed columns of the window
// are marked in an LDS bitmap and ranked by its prefix counts (a count per owner
// thread, and 16-bit counts of the words inside the owner's range).  The bitmap
// and those counts are the block's dynamic LDS (global_rank_lds bytes, no more
// than B's columns need, so that several rows share a CU where B is narrow).
//
// Bound by memory traffic: the tables' lines and their clearing.  RMAT 12289
// A * A (edge factor 12, 20M products in heavy rows), FP32: 0.77 ms; without the
// front table 1.53, with keys and values in separate arrays and a
// compare-and-swap per product 1.80, with agent scope and a 2^19-column
// bitmap per row 5.64 (symbolic pass 0.17, 0.57, 0.81 and 0.47 ms).  Every
// window looks at the whole list twice, hence the columns in it: 500 rows of
// 2000 x 100 products in eight windows 32 ms, 59 where each look reads the
// listed slot's key; 50 rows of 300 x 300 in 191 windows 33 and 61.
constexpr int kGlobalRankBits = 1 << 19;

__host__ __device__ __forceinline__ size_t global_rank_lds(long long ncols)
{
    const long long bits = ncols < kGlobalRankBits ? ncols : kGlobalRankBits;
    return (size_t)((bits + 31) / 32 + 1) / 2 * 2 * (sizeof(unsigned) + sizeof(unsigned short));
}

template <typename V>
struct GlobalNumLds {
    double fval[1 << kFrontLog];           // front table
    int fkey[1 << kFrontLog];
    PieceScratch<V, kGlobalThreads> S;
    int tmp[kGlobalThreads / kWave + 1];
    int base[kGlobalThreads];
    int nfront, ntouched;                  // columns in the front table and in the row's table
};

template <typename V>
__device__ __forceinline__ void num_global_row(const int *__restrict__ Arp, const int *__restrict__ Acol,
                                               const V *__restrict__ Aval, const int *__restrict__ Brp,
                                               const int *__restrict__ Bcol, const V *__restrict__ Bval, int arow,
                                               long long crow, int ncols, GSlot *tab, GlobalNumLds<V> &L,
                                               unsigned *s_bm, const long long *__restrict__ Crp,
                                               int *__restrict__ Ccol, V *__restrict__ Cval, int *err)
{
    constexpr int G = kGlobalThreads;
    const long long rb = Crp[crow];
    const int nc = (int)(Crp[crow + 1] - rb);
    const int logT = gtable_log2(nc);
    const int T = 1 << logT;
    for (int t = threadIdx.x; t < T; t += G) tab[t] = GSlot{0.0, kEmpty, 0};
    for (int t = threadIdx.x; t < 1 << kFrontLog; t += G) {
        L.fkey[t] = kEmpty;
        L.fval[t] = 0.0;
    }
    if (threadIdx.x == 0) L.nfront = L.ntouched = 0;
    __syncthreads();
    int mine = 0;
    auto sink = [&](const auto &j, const auto &p, const auto &ok) {
        constexpr int N = sizeof(j) / sizeof(j[0]);
        int slot[N];
        bool far[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            bool fresh = false;
            const int f = ok[u] ? front_find(L.fkey, j[u], fresh) : 0;
            far[u] = f < 0;
            mine += fresh;
            if (ok[u] && f >= 0) atomicAdd(&L.fval[f], p[u]);
        }
        gfind<N>(logT, j, far, slot, err, [&](int h) { return &tab[h].key; }, [&](int h, int key) {
            const int at = atomicAdd(&L.ntouched, 1);
            if (at < nc) {
                tab[at].list = h;
                tab[nc + at].list = key;
            }
        });
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (slot[u] >= 0)
                __hip_atomic_fetch_add(&tab[slot[u]].val, p[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    piece_products<V, true, G, G, 4>(Arp[arow], Arp[arow + 1], threadIdx.x, L.S, Acol, Aval, Brp, 1, 1, Bcol, Bval,
                                     sink);
    mine = wave_sum(mine);
    if (lane_id() == 0 && mine) atomicAdd(&L.nfront, mine);
    __syncthreads();
    // the row's entries: the front table's slots, then the list
    const int nt = L.ntouched < nc ? L.ntouched : nc, listed = L.nfront + nt;
    const int nf = 1 << kFrontLog;
    auto key_of = [&](int t) { return t < nf ? L.fkey[t] : tab[nc + t - nf].list; };
    const int top = ncols < kGlobalRankBits ? ncols : kGlobalRankBits;
    const int words = (top + 31) >> 5;
    unsigned short *s_pref = reinterpret_cast<unsigned short *>(s_bm + ((words + 1) & ~1));
    const int sh = words <= G ? 0 : ceil_log2((words + G - 1) / G);      // 2^sh words per owner thread, at most 32
    long long done = 0;
    for (int lo = 0; lo < ncols; lo += kGlobalRankBits) {
        const int hi = lo < ncols - kGlobalRankBits ? lo + kGlobalRankBits : ncols;
        for (int t = threadIdx.x; t < words; t += G) s_bm[t] = 0u;
        __syncthreads();
        for (int t = threadIdx.x; t < nf + nt; t += G) {
            const int j = key_of(t);                       // kEmpty lies below every window
            if (j >= lo && j < hi) atomicOr(&s_bm[(j - lo) >> 5], 1u << ((j - lo) & 31));
        }
        __syncthreads();
        int pc = 0;
        for (int q = (int)threadIdx.x << sh, e = q + (1 << sh) < words ? q + (1 << sh) : words; q < e; ++q) {
            s_pref[q] = (unsigned short)pc;
            pc += __popc(s_bm[q]);
        }
        int tot;
        const int ex = block_excl_scan<int, G>(pc, L.tmp, tot);
        L.base[threadIdx.x] = ex;
        __syncthreads();
        for (int t = threadIdx.x; t < nf + nt; t += G) {
            const int j = key_of(t);
            if (j < lo || j >= hi) continue;
            const int jl = j - lo, wd = jl >> 5;
            const long long pos = done + L.base[wd >> sh] + s_pref[wd] + __popc(s_bm[wd] & ((1u << (jl & 31)) - 1u));
            if (pos < nc) {
                store_c(&Ccol[rb + pos], j);
                store_c(&Cval[rb + pos], (V)(t < nf ? L.fval[t] : gload_v(&tab[tab[t - nf].list].val)));
            }
        }
        done += tot;
        __syncthreads();
        if (done >= listed || hi == ncols) break;     // every entry is out
    }
    if (threadIdx.x == 0 && (done != nc || L.nfront + L.ntouched != nc)) atomicOr(err, kErrCount);
}

// Numeric phase of heavy rows in global mode: one block per row.
template <typename V>
__global__ __launch_bounds__(kGlobalThreads) void k_num_global(
    const int *__restrict__ Arp, const int *__restrict__ Acol, const V *__restrict__ Aval,
    const int *__restrict__ Brp, const int *__restrict__ Bcol, const V *__restrict__ Bval,
    const int *__restrict__ rows, int ncols, const long long *__restrict__ goff, long long gbase, GSlot *pool,
    const long long *__restrict__ Crp, int *__restrict__ Ccol, V *__restrict__ Cval, int *err)
{
    extern __shared__ unsigned s_bm[];                     // global_rank_lds(ncols) bytes
    __shared__ GlobalNumLds<V> L;
    const int row = rows[blockIdx.x];
    num_global_row<V>(Arp, Acol, Aval, Brp, Bcol, Bval, row, row, ncols,
                      pool + (goff[blockIdx.x] - gbase), L, s_bm, Crp, Ccol, Cval, err);
}

}  // namespace smash
