"""GPU parity of the batched launch (smash_batch_plan_*) against the oracle.

Each problem's C_p, read from the shared output pool, must match the oracle
like any single product (structure bit-exact, values within tolerance), in
eager runs and in replays of the captured graph (several replays, with other
GPU work and synchronisations in between, each checked), under every
autotuner candidate shape class, and for degenerate batches.  The full
512-problem workload is checked exactly on every problem's row counts and
entry by entry on sampled problems.
"""
import os
import tempfile

import numpy as np
import pytest

import synthetic as syn
from tests._parity import check_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2105_14156_amd import smash
    assert torch.cuda.is_available()
    ctx = smash.Context(0)
    yield torch, smash, ctx
    ctx.close()


def _problems(count, dtype=np.float32):
    return [(w.A.astype(dtype), w.B.astype(dtype)) for w in syn.workload_batch(count, dtype)]


def _check_plan(plan, probs, refs, oracle_mod, where, stream=None):
    tot, per = plan.result(stream)
    assert tot == int(sum(r["row_ptr"][-1] for r in refs)), f"{where}: total entries"
    for p, ((A, B), ref) in enumerate(zip(probs, refs)):
        C = plan.problem(p)
        assert per[p] == ref["row_ptr"][-1], f"{where}: problem {p} entries"
        check_rows(C.row_ptr.cpu().numpy(), C.col_idx.cpu().numpy(), C.val.cpu().numpy(), ref, A.val.dtype,
                   f"{where} problem {p}")


def _make_plan(smash, ctx, probs, config=None):
    dA = [smash.to_device(A) for A, _ in probs]
    dB = [smash.to_device(B) for _, B in probs]
    return smash.BatchPlan(ctx, dA, dB, config)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_batch_eager_and_graph(env, oracle_mod, dtype):
    torch, smash, ctx = env
    probs = _problems(40, dtype)
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs)
    plan.run()
    _check_plan(plan, probs, refs, oracle_mod, "eager")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plan.capture(stream)
    for rep in range(3):
        plan.C_col.fill_(-7)                       # other work between replays
        torch.cuda.synchronize()
        plan.launch(stream)
        _check_plan(plan, probs, refs, oracle_mod, f"replay {rep}", stream)
    plan.close()


@pytest.mark.parametrize("config", [
    dict(lds_row_max=256, table_shift=2, wide_groups=1, blocks_per_cu=1, row_hash=0),
    dict(lds_row_max=512, table_shift=2, wide_groups=0, blocks_per_cu=32, row_hash=1),
    dict(lds_row_max=32, table_shift=1, wide_groups=1, blocks_per_cu=4, row_hash=0),
    dict(lds_row_max=1024, table_shift=1, wide_groups=1, blocks_per_cu=16, row_hash=1),
    dict(lds_row_max=1024, table_shift=1, wide_groups=0, blocks_per_cu=8, row_hash=1),
])
def test_batch_configs(env, oracle_mod, config):
    torch, smash, ctx = env
    probs = _problems(24)
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs, config)
    assert plan.config() == config
    plan.run()
    _check_plan(plan, probs, refs, oracle_mod, str(config))
    plan.close()


def test_batch_degenerate(env, oracle_mod):
    """Problems without rows, without entries, rectangular shapes and
    rows heavy enough for the global tables, in one batch."""
    torch, smash, ctx = env
    f32 = np.float32
    probs = [
        (syn.empty(0, 10, f32), syn.random_sparse(10, 7, 0.3, 1, f32)),
        (syn.empty(50, 40, f32), syn.random_sparse(40, 30, 0.2, 2, f32)),
        (syn.random_sparse(60, 80, 0.05, 3, f32), syn.random_sparse(80, 3000, 0.01, 4, f32)),
        (syn.dense_rows(8, 3000, [1, 5], 5, f32), syn.random_sparse(3000, 5000, 0.004, 6, f32)),
        (syn.identity(100, f32), syn.random_sparse(100, 9, 0.5, 7, f32)),
        (syn.random_sparse(1, 1, 1.0, 8, f32), syn.random_sparse(1, 1, 1.0, 9, f32)),
        # wider than the LDS bitmap limit: heavy rows use global tables
        (syn.random_sparse(30, 200, 0.3, 10, f32), syn.uniform_k_per_row(200, (1 << 20) + 3000, 40, 11, f32)),
        # products that are all +-0.0, in the LDS windows of heavy rows
        _zero_case(),
    ]
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs, dict(lds_row_max=64, table_shift=1, wide_groups=0, blocks_per_cu=2))
    plan.run()
    _check_plan(plan, probs, refs, oracle_mod, "degenerate")
    plan.close()


def _zero_case():
    B = syn.uniform_k_per_row(8, 8192, 3000, 0x2E0, np.float32)
    A = syn.CSR(3, 8, np.array([0, 2, 4, 6], np.int32), np.arange(6, dtype=np.int32),
                np.array([0.0, -0.0, -0.0, -0.0, 0.5, -0.0], np.float32))
    return A, B


def test_batch_subnormal_wide_window(env, oracle_mod):
    """FP64 heavy rows in the LDS windows (occupancy by leaving -0.0): a
    negative subnormal sum and a cancelling sum keep their entries."""
    torch, smash, ctx = env
    n, width = 8192, 1500
    cols = np.arange(width, dtype=np.int32)
    b0, b1 = np.ones(width), np.ones(width)
    b0[7], b1[7] = -1e-320, 0.0
    b0[9], b1[9] = 1.0, -1.0
    B = syn.CSR(2, n, np.array([0, width, 2 * width], np.int32), np.concatenate([cols, cols]),
                np.concatenate([b0, b1]))
    A = syn.CSR(1, 2, np.array([0, 2], np.int32), np.array([0, 1], np.int32), np.array([1.0, 1.0]))
    probs = [(A, B), _problems(2, np.float64)[1]]
    refs = [oracle_mod.spgemm(a, b) for a, b in probs]
    plan = _make_plan(smash, ctx, probs, dict(lds_row_max=256, table_shift=1, wide_groups=0, blocks_per_cu=4))
    plan.run()
    _check_plan(plan, probs, refs, oracle_mod, "subnormal window")
    C = plan.problem(0)
    v = C.val.cpu().numpy()
    assert v[7] == -1e-320 and v[9] == 0.0
    plan.close()


def test_batch_without_rows(env):
    torch, smash, ctx = env
    probs = [(syn.empty(0, 5, np.float32), syn.random_sparse(5, 5, 0.5, 1, np.float32))] * 3
    plan = _make_plan(smash, ctx, probs)
    plan.run()
    stream = torch.cuda.Stream()
    plan.capture(stream)
    plan.launch(stream)
    tot, per = plan.result(stream)
    assert tot == 0 and list(per) == [0, 0, 0]
    assert plan.C_row_ptr.cpu().tolist() == [0]
    plan.close()


def test_batch_invalid_operand(env):
    """Creation validates every operand: one problem whose B has a repeated
    column in a row fails the whole batch with INVALID_CSR."""
    torch, smash, ctx = env
    probs = _problems(6)
    A, B = probs[4]
    ci = B.col_idx.copy()
    r = int(np.argmax(np.diff(B.row_ptr)))                 # a row with at least two entries
    ci[B.row_ptr[r] + 1] = ci[B.row_ptr[r]]
    probs[4] = (A, syn.CSR(B.rows, B.cols, B.row_ptr, ci, B.val))
    with pytest.raises(smash.SmashError) as e:
        _make_plan(smash, ctx, probs)
    assert e.value.status == 2


def test_batch_capacity_error(env):
    """A structure change after creation that needs more entries than the
    pool holds is reported as CAPACITY."""
    torch, smash, ctx = env
    n = 4096
    A = syn.strided_columns(n, n, 6, 2, 11, np.float32)          # even columns only
    B = syn.uniform_k_per_row(n, n, 8, 12, np.float32)
    dA, dB = smash.to_device(A), smash.to_device(B)
    plan = smash.BatchPlan(ctx, [dA], [dB])
    plan.run()
    plan.result()
    # same shape and nnz, but even rows hold 16 entries and odd rows none:
    # every row of A now reaches 96 products, twice the pool's 48 per row
    half = syn.uniform_k_per_row(n // 2, n, 16, 13, np.float32)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(np.where(np.arange(n) % 2 == 0, 16, 0))
    assert rp[-1] == B.nnz == half.nnz
    dB.row_ptr.copy_(torch.from_numpy(rp.astype(np.int32)))
    dB.col_idx.copy_(torch.from_numpy(half.col_idx.astype(np.int32)))
    plan.run()
    with pytest.raises(smash.SmashError) as ei:
        plan.result()
    assert ei.value.status == 4
    plan.close()


def test_batch_autotune_and_cache(env, oracle_mod):
    torch, smash, ctx = env
    probs = _problems(32)
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs)
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "tune.txt")
        cfg, ms = plan.autotune(reps=1, cache_path=path)
        assert ms > 0 and plan.config() == cfg
        plan.run()
        _check_plan(plan, probs, refs, oracle_mod, "autotuned")
        plan.configure(dict(lds_row_max=32, table_shift=1, wide_groups=0, blocks_per_cu=1))
        cfg2, ms2 = plan.autotune(reps=1, cache_path=path)      # cache hit
        assert ms2 == 0.0 and cfg2 == cfg and plan.config() == cfg
    plan.close()


@pytest.mark.timeout(600)
def test_batch_full_512(env, oracle_mod):
    """The 512-problem workload in its graph: exact row counts of every
    problem, entries of sampled problems (the largest ones and seeded picks)."""
    torch, smash, ctx = env
    probs = _problems(512)
    plan = _make_plan(smash, ctx, probs)
    stream = torch.cuda.Stream()
    plan.capture(stream)
    plan.launch(stream)
    plan.launch(stream)
    tot, per = plan.result(stream)
    crp = plan.C_row_ptr.cpu().numpy()
    for p, (A, B) in enumerate(probs):
        nz = oracle_mod.row_nnz(A, B)
        r0, r1 = plan.row0[p], plan.row0[p + 1]
        assert np.array_equal(np.diff(crp[r0:r1 + 1]), nz), f"problem {p} row counts"
    prods = np.array([int(np.diff(B.row_ptr)[A.col_idx].sum()) for A, B in probs])
    pick = set(np.argsort(-prods)[:4].tolist()) | set((syn.uniform01(0xBA7, 0, 8) * 512).astype(int).tolist())
    for p in sorted(pick):
        A, B = probs[p]
        C = plan.problem(p)
        check_rows(C.row_ptr.cpu().numpy(), C.col_idx.cpu().numpy(), C.val.cpu().numpy(), oracle_mod.spgemm(A, B),
                   np.float32, f"512 batch problem {p}")
    plan.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("widths", [(2000, 32768), (32769, 65537), (131072,), (131072, 131073, 1 << 20, (1 << 20) + 1)])
def test_batch_widths(env, oracle_mod, dtype, widths):
    """The heavy and LDS rows of a batch at every limit of B's width: bitmap rows
    (up to 128 columns per table slot, and 2^17), windows (2^20), global tables
    above.  Rows of 40 to 6000 entries: light rows of every table, heavy rows of
    one and of several passes, A rows longer than one list."""
    torch, smash, ctx = env
    probs = []
    for q, n in enumerate(widths):
        B = syn.uniform_k_per_row(900, n, 20, 300 + q, dtype)
        lens = [2, 5, 13, 26, 52, 55, 130, 310, 700]
        ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        col = np.concatenate([np.arange(k) + 11 * i for i, k in enumerate(lens)]).astype(np.int32)
        probs.append((syn.CSR(len(lens), 900, ptr, col, (2.0 * syn.uniform01(7, 0, len(col)) - 1.0).astype(dtype)), B))
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    for row_hash in (0, 1):
        plan = _make_plan(smash, ctx, probs, dict(lds_row_max=1024, table_shift=1, wide_groups=0, blocks_per_cu=8,
                                                  row_hash=row_hash))
        for rep in range(2):
            plan.run()
            _check_plan(plan, probs, refs, oracle_mod, f"widths {widths} hash {row_hash} run {rep}")
        plan.close()


@pytest.mark.parametrize("rows", [[1], [63, 0, 1, 64, 65], [255, 1, 300]])
def test_batch_row_bounds(env, oracle_mod, rows):
    """Rows around the limits of the bound's split: lanes of a group of eight
    (7..9 entries), the longest row of a group and the shortest of a wave
    (128, 129), one and two steps of a wave (512, 513), rows without entries,
    over problems that start inside a wave's 64 rows.  Sums of B-row lengths
    decide the bins and capacities, so a wrong one changes the result;
    structure and row counts exact."""
    torch, smash, ctx = env
    lens = np.array([129, 0, 1, 7, 8, 9, 128, 130, 513, 512, 31, 33, 1025, 64, 3])
    probs = []
    for p, m in enumerate(rows):
        k = lens[(np.arange(m) + p) % len(lens)]
        ptr = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
        col = np.concatenate([np.zeros(0, np.int32)] + [np.arange(n, dtype=np.int32) + i % 200 for i, n in enumerate(k)])
        A = syn.CSR(m, 2048, ptr, col, np.ones(len(col), np.float32))
        probs.append((A, syn.rmat_rect(2048, 2, 9 + p, np.float32)))
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs)
    plan.run()
    _check_plan(plan, probs, refs, oracle_mod, f"rows {rows}")
    plan.close()


def _long_rows(n, dtype):
    """B of n > 65536 columns with rows of 65535, 65536 (columns 0 to 65535),
    65537 and n entries and some of 3000, and an A whose rows are B's long
    rows alone and merged with shorter ones."""
    allc = np.arange(n, dtype=np.int32)
    rows = [np.delete(allc, 77)[n - 65536:], allc[:65536], np.delete(allc[:65538], 30000), allc]
    rows += [np.sort((syn.uniform01(17 + q, 0, 6000) * n).astype(np.int32)) for q in range(6)]
    rows = [np.unique(r)[:3000] if q > 3 else r for q, r in enumerate(rows)]
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    col = np.concatenate(rows)
    B = syn.CSR(len(rows), n, ptr, col, (2.0 * syn.uniform01(n, 0, len(col)) - 1.0).astype(dtype))
    sets = [[0], [1], [2], [3], [0, 4], [1, 5, 6], [2, 3], [4, 5, 6, 7, 8, 9], list(range(10))]
    aptr = np.concatenate([[0], np.cumsum([len(x) for x in sets])]).astype(np.int32)
    acol = np.concatenate(sets).astype(np.int32)
    A = syn.CSR(len(sets), len(rows), aptr, acol, (2.0 * syn.uniform01(5, 0, len(acol)) - 1.0).astype(dtype))
    assert [int(np.diff(ptr)[q]) for q in range(4)] == [65535, 65536, 65537, n]
    return A, B


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_batch_long_rows(env, oracle_mod, dtype):
    """Heavy rows of 65535 to 131072 entries: more than 16 bits count, in
    problems narrow enough for the bitmap form of heavy rows."""
    torch, smash, ctx = env
    probs = [_long_rows(n, dtype) for n in (65540, 100000, 131072)]
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs)
    for rep in range(2):
        plan.run()
        _check_plan(plan, probs, refs, oracle_mod, f"long rows run {rep}")
    plan.close()
    A = syn.rmat(17, 16, 3, dtype)                # its longest row of A * A has more than 65536 entries
    prods = np.diff(A.row_ptr)[A.col_idx]
    prods = np.add.reduceat(np.append(prods, 0), A.row_ptr[:-1]) * (np.diff(A.row_ptr) > 0)
    rows = np.sort(np.argsort(-prods)[:24]).astype(np.int64)
    plan = _make_plan(smash, ctx, [(A, A)])
    plan.run()
    plan.result()
    C = plan.problem(0)
    ptr = C.row_ptr.cpu().numpy()
    assert np.diff(ptr).max() > 65536
    sel = [slice(int(ptr[r]), int(ptr[r + 1])) for r in rows]
    check_rows(np.concatenate([[0], np.cumsum(np.diff(ptr)[rows])]),
               np.concatenate([C.col_idx[s].cpu().numpy() for s in sel]),
               np.concatenate([C.val[s].cpu().numpy() for s in sel]), oracle_mod.spgemm(A, A, rows=rows), dtype,
               "rmat 17 longest rows")
    plan.close()


@pytest.mark.parametrize("widths", [(3000,), (8193, 16384), (40000, 300, (1 << 20) + 5)])
def test_batch_windows_rule(env, oracle_mod, widths):
    """Heavy rows on both sides of the line between bitmap and windows (few and
    many products; at most 512 A entries and more; over 262144 products), next
    to light rows, problems without any, and rows in global tables; replayed."""
    torch, smash, ctx = env
    probs = []
    for q, n in enumerate(widths):
        B = syn.uniform_k_per_row(1200, n, 150, 40 + q, np.float32)
        lens = [8, 30, 100, 150, 512, 513, 1100, 2, 0] if n > 1000 else [1, 2]
        if n > 1 << 20:
            lens = [40, 3]
        if q == 0:
            B = syn.uniform_k_per_row(1200, n, 400, 50, np.float32)
        ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        col = np.concatenate([np.arange(k) + 7 * i for i, k in enumerate(lens)]).astype(np.int32)
        probs.append((syn.CSR(len(lens), 1200, ptr, col, (2.0 * syn.uniform01(9, 0, len(col)) - 1.0).astype(np.float32)), B))
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs)
    stream = torch.cuda.Stream()
    plan.capture(stream)
    for rep in range(3):
        plan.C_col.fill_(-7)
        torch.cuda.synchronize()
        plan.launch(stream)
        _check_plan(plan, probs, refs, oracle_mod, f"widths {widths} replay {rep}", stream)
    plan.close()


@pytest.mark.parametrize("n,per_row", [(4096, 1), (32768, 2), (65536, 2), (65536, 3), (131072, 1), (131072, 3)])
def test_batch_short_b_rows(env, oracle_mod, n, per_row):
    """B rows of one to three entries, on both sides of the lines between hash
    tables and bitmaps, in batches of one width."""
    torch, smash, ctx = env
    probs = []
    for q in range(3):
        B = syn.uniform_k_per_row(5000, n, per_row, 30 + q, np.float32)
        lens = np.array([2, 40, 70, 110, 230, 470, 950, 3000])[(np.arange(64) + q) % 8] // per_row
        ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        col = np.concatenate([np.arange(m) + 31 * i for i, m in enumerate(lens)]).astype(np.int32)
        probs.append((syn.CSR(64, 5000, ptr, col, (2.0 * syn.uniform01(q, 0, len(col)) - 1.0).astype(np.float32)), B))
    refs = [oracle_mod.spgemm(A, B) for A, B in probs]
    plan = _make_plan(smash, ctx, probs)
    for rep in range(2):
        plan.run()
        _check_plan(plan, probs, refs, oracle_mod, f"{n} columns, {per_row} per row, run {rep}")
    plan.close()


@pytest.mark.parametrize("n", [5, 64, 65, 128, 129, 256, 512, 1024, 1025])
def test_batch_narrow_b(env, oracle_mod, n):
    """B of few columns in batches, on both sides of the same lines."""
    torch, smash, ctx = env
    for mean in (7, 9, 51, 53, 103, 210):
        probs = []
        for q in range(3):
            B = syn.uniform_k_per_row(3000, n, min(8, n), 40 + q, np.float32)
            lens = np.arange(400) * 7 % (2 * mean + 1)
            ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
            col = ((np.arange(ptr[-1]) - np.repeat(ptr[:-1], lens)) * 7 + np.repeat(np.arange(400) % 17, lens)).astype(np.int32)
            probs.append((syn.CSR(400, 3000, ptr, col, (2.0 * syn.uniform01(q, 0, len(col)) - 1.0).astype(np.float32)), B))
        refs = [oracle_mod.spgemm(A, B) for A, B in probs]
        plan = _make_plan(smash, ctx, probs)
        for rep in range(2):
            plan.run()
            _check_plan(plan, probs, refs, oracle_mod, f"{n} columns, {mean} entries per A row, run {rep}")
        plan.close()


@pytest.mark.parametrize("n", [129, 300, 600, 1500, 3000])
def test_batch_repeated_columns(env, oracle_mod, n):
    """Rows with many products per column of B in batches, light and heavy, on
    both sides of the line from which marks are read before they are set."""
    torch, smash, ctx = env
    for mean in (18 * n // 128, 32 * n // 128):
        probs = []
        for q in range(2):
            B = syn.uniform_k_per_row(2000, n, 128, 50 + q, np.float32)
            lens = np.arange(100) * 7 % (2 * mean + 1)
            ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
            col = ((np.arange(ptr[-1]) - np.repeat(ptr[:-1], lens)) + np.repeat(np.arange(100) % 17, lens)).astype(np.int32)
            probs.append((syn.CSR(100, 2000, ptr, col, (2.0 * syn.uniform01(q, 0, len(col)) - 1.0).astype(np.float32)), B))
        refs = [oracle_mod.spgemm(A, B) for A, B in probs]
        plan = _make_plan(smash, ctx, probs)
        for rep in range(2):
            plan.run()
            _check_plan(plan, probs, refs, oracle_mod, f"{n} columns, {mean} entries per A row, run {rep}")
        plan.close()
