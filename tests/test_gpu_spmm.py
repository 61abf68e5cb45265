"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element
by element on the same seeded inputs.  Tolerance per element, as stated for
this build: |y_gpu - y_fp64| <= 1e-5 * sum_j |a_ij x_jk| + 1e-6 (fp32
accumulation against an fp64 reference)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from util import wgrad_rows_per_wavefront, wgrad_tolerance, assert_close_to_oracle, ensure_built, layer_tolerance, tolerance

pytestmark = pytest.mark.gpu

ensure_built()
import paper_2511_18297_amd as G  # noqa: E402


@pytest.fixture(autouse=True, params=[0, 1], ids=["ld_plain", "ld_pipelined"])
def ld_kernel_choice(request):
    """Every case runs with each of the two LD kernels (the pipelined one applies to F = 32, 64, 128;
    other widths take the plain kernel either way)."""
    G.groot_set_tuning("ld_pipeline", request.param)
    yield request.param
    G.groot_set_tuning("ld_pipeline", -1)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    assert torch.cuda.is_available(), "these tests need a GPU"
    torch.cuda.set_device(0)
    return torch


def _run(torch, g, T, X_np, guard_rows=3, phases=None):
    """execute with canary rows around Y; returns Y as numpy"""
    n = G.groot_graph_view(g)["n"]
    F = X_np.shape[1]
    plan = G.groot_spmm_plan(g, T)
    G.groot_plan_upload(plan, F)
    X = torch.from_numpy(X_np).cuda()
    buf = torch.full((n + 2 * guard_rows, F), float("nan"), dtype=torch.float32, device="cuda")
    buf[:guard_rows] = 12345.0
    buf[n + guard_rows:] = 12345.0
    Y = buf[guard_rows:n + guard_rows]
    G.groot_spmm_execute(plan, X, Y, F)
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    assert (out[:guard_rows] == 12345.0).all() and (out[n + guard_rows:] == 12345.0).all(), "wrote outside Y"
    return out[guard_rows:n + guard_rows], plan, X, Y


def _aig_case(n, batch, flags=G.GROOT_DEFAULT_FLAGS):
    aig = wl.csa_multiplier_aig(n)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, batch, flags)
    o = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, batch, flags)
    return aig, g, o


@pytest.mark.parametrize("n_bits,batch,F,T", [(64, 2, 32, 32), (32, 3, 64, 16), (96, 1, 128, 64)])
def test_booth_multiplier_degree_profile(torch_cuda, n_bits, batch, F, T):
    """Radix-4 Booth multipliers: about 3.5 n high-degree rows of n to 4n entries (recoding signals and
    primary inputs), many of them split into several pieces, next to the short rows."""
    aig = wl.booth_multiplier_aig(n_bits)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, batch)
    rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, batch)
    X = wl.uniform_features_numpy(40 + n_bits, 0, aig.num_nodes * batch, F)
    Y, plan, _, _ = _run(torch_cuda, g, T, X)
    assert G.groot_plan_view(plan)["n_hd"] >= 2 * n_bits * batch
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, f"booth {n_bits}x{batch} F={F} T={T}")


@pytest.mark.parametrize("n_bits,batch,F,T", [(48, 2, 32, 32), (32, 1, 64, 8), (24, 3, 128, 7)])
def test_lut4_mapped_multiplier_shape(torch_cuda, uniform_detect, n_bits, batch, F, T):
    """4-LUT-mapped carry-save array: interior rows of 7 entries (longer than the pipelined kernel's 6
    slots: there they go through its plain loop), 2n rows of 2n+1; T = 7 makes almost every row high-degree."""
    s = wl.lut4_csa_graph(n_bits, batch)
    g = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
    X = wl.uniform_features_numpy(60 + n_bits, 0, s.n, F)
    Y, plan, _, _ = _run(torch_cuda, g, T, X)
    Y64, S = oracle.spmm_f64(s.rowptr, s.col, s.val, X)
    assert_close_to_oracle(Y, Y64, S, f"lut4 {n_bits}x{batch} F={F} T={T}")


@pytest.mark.parametrize("n_bits,batch,F,T", [(48, 2, 32, 32), (40, 1, 64, 16), (24, 3, 128, 5)])
def test_cell_mapped_multiplier_shape(torch_cuda, uniform_detect, n_bits, batch, F, T):
    """Standard-cell-mapped carry-save array: AND2 rows of 4 entries, adder rows of 6 (all within the
    pipelined kernel's slots), 2n rows of n+1; T = 5 makes every adder row high-degree."""
    s = wl.cellmap_csa_graph(n_bits, batch)
    g = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
    X = wl.uniform_features_numpy(70 + n_bits, 0, s.n, F)
    Y, plan, _, _ = _run(torch_cuda, g, T, X)
    Y64, S = oracle.spmm_f64(s.rowptr, s.col, s.val, X)
    assert_close_to_oracle(Y, Y64, S, f"cells {n_bits}x{batch} F={F} T={T}")


def test_config1_32bit_structural_features(torch_cuda):
    """32-bit multiplier, F = 32, node-type / polarity columns + U(-1,1), T = 32."""
    aig, g, (rowptr, col, val, pol) = _aig_case(32, 1)
    X = wl.aig_node_features(aig, 0, 32)
    Y, plan, _, _ = _run(torch_cuda, g, 32, X)
    assert G.groot_plan_view(plan)["n_hd"] == 64
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, "config 1")


@pytest.fixture
def compact_always():
    """The compact matrix is read at every size of X."""
    G.groot_set_tuning("csr_compress", 2)
    yield
    G.groot_set_tuning("csr_compress", 1)


def test_config2_256bit(torch_cuda, compact_always):
    """256-bit multiplier (522,496 nodes), F = 64, seed 1, T = 32."""
    aig, g, (rowptr, col, val, pol) = _aig_case(256, 1)
    X = wl.uniform_features_numpy(1, 0, aig.num_nodes, 64)
    Y, plan, Xd, Yd = _run(torch_cuda, g, 32, X)
    assert G.groot_plan_view(plan)["n_hd"] == 512
    # the pipelined kernel runs with 5 slots per row (only 256 rows have 6 entries) on the compact matrix
    # (2-byte column codes; the 498 rows they cannot express -- primary outputs more than 16,384 rows behind their
    # drivers, and those drivers -- join the 256 long rows on the row list)
    if G.groot_plan_query(plan, "ld_pipelined"):
        assert G.groot_plan_query(plan, "pipe_depth") == 5 and G.groot_plan_query(plan, "csr_compressed") == 1
        assert G.groot_plan_query(plan, "uncoded_rows") == 498 and G.groot_plan_query(plan, "mid_rows") == 256 + 498
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, "config 2")
    # no atomics anywhere: a second run is bitwise identical
    Yd.fill_(float("nan"))
    G.groot_spmm_execute(plan, Xd, Yd, 64)
    torch_cuda.cuda.synchronize()
    assert np.array_equal(Yd.cpu().numpy(), Y)


@pytest.mark.parametrize("F", [4, 8, 12, 20, 36, 64, 100, 128, 132, 256, 260, 512])
def test_feature_widths(torch_cuda, F):
    aig, g, (rowptr, col, val, pol) = _aig_case(24, 2)
    X = wl.uniform_features_numpy(10 + F, 0, 2 * aig.num_nodes, F)
    Y, _, _, _ = _run(torch_cuda, g, 8, X)
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, f"F={F}")


@pytest.mark.parametrize("n,batch,T", [(2, 1, 32), (2, 1, 1), (3, 5, 4), (17, 1, 18), (17, 3, 5), (40, 1, 41), (40, 1, 42)])
def test_row_counts_and_thresholds(torch_cuda, n, batch, T):
    """ragged tails (N not a multiple of 64 or 256), every row high-degree (T = 1),
    no row high-degree (T above the largest row)."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n, batch)
    X = wl.uniform_features_numpy(n, 0, batch * aig.num_nodes, 32)
    Y, _, _, _ = _run(torch_cuda, g, T, X)
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, f"n={n} batch={batch} T={T}")


@pytest.mark.parametrize("flags", [0, 1, 3, 4, 5])
def test_flag_variants_with_empty_rows(torch_cuda, flags):
    """directed / no self-loops: primary inputs (and isolated nodes) have empty rows -> 0"""
    aig, g, (rowptr, col, val, pol) = _aig_case(16, 2, flags)
    X = wl.uniform_features_numpy(3, 0, 2 * aig.num_nodes, 16)
    Y, _, _, _ = _run(torch_cuda, g, 6, X)
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, f"flags={flags}")
    empty = np.diff(rowptr) == 0
    if flags & 3 == 0:      # directed, no self-loops: primary inputs aggregate nothing
        assert empty.any()
    assert (Y[empty] == 0).all()


def test_tiny_graphs(torch_cuda):
    # a single row; and a graph whose only non-empty row is the last one
    g = G.groot_graph_from_csr(np.array([0, 1]), np.array([0], dtype=np.int32), np.array([2.0], dtype=np.float32))
    X = np.arange(8, dtype=np.float32)[None, :]
    Y, _, _, _ = _run(torch_cuda, g, 32, X)
    assert np.array_equal(Y, 2 * X)
    n = 300
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[-1] = n
    col = np.arange(n, dtype=np.int32)
    val = np.full(n, 0.5, dtype=np.float32)
    X = wl.uniform_features_numpy(1, 0, n, 8)
    for T in (32, 400):
        g = G.groot_graph_from_csr(rowptr, col, val)
        Y, _, _, _ = _run(torch_cuda, g, T, X)
        Y64, S = oracle.spmm_f64(rowptr, col, val, X)
        assert_close_to_oracle(Y, Y64, S, "last-row graph")
        assert (Y[:-1] == 0).all()


@pytest.mark.parametrize("T", [16, 32, 64, 128])
def test_stress_graph_threshold_sweep(torch_cuda, uniform_detect, T):
    """Polarized degrees (scaled-down law of the 16M-row stress workload): rows
    of up to 16,385 non-zeros are split over several workgroups."""
    s = wl.stress_graph(4, 1 << 16, window=4096, dmin=64, dmax=16384)
    g = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
    X = wl.uniform_features_numpy(4, 0, s.n, 128)
    Y, plan, _, _ = _run(torch_cuda, g, T, X)
    deg = np.diff(s.rowptr)
    assert G.groot_plan_query(plan, "weight_mode") == (1 if uniform_detect else 2)
    assert G.groot_plan_view(plan)["n_hd"] == int((deg >= T).sum())
    Y64, S = oracle.spmm_f64(s.rowptr, s.col, s.val, X)
    assert_close_to_oracle(Y, Y64, S, f"stress T={T}")


@pytest.mark.parametrize("max_len,T,F,explicit", [(14, 32, 64, False), (14, 9, 32, False), (10, 4, 128, True),
                                                   (9, 32, 64, True), (40, 16, 64, False), (8, 32, 32, False)])
def test_mixed_row_lengths(torch_cuda, compact_always, max_len, T, F, explicit):
    """Row lengths drawn uniformly from 0..max_len (empty rows included), 20,011 rows (a ragged last tile at every
    width): in the pipelined kernel every tile mixes rows that fit its 5 to 8 slots, longer low-degree rows (masked
    there, computed from the row list) and high-degree rows (masked, computed by the HD kernel); with max_len = 40
    most low-degree rows are longer than any slot count (the knob still forces the pipelined kernel).  Weights
    1 / row length (recomputed in the kernels) or arbitrary (read)."""
    n = 20011
    rng = np.random.default_rng(1000 + max_len + T + F)
    deg = rng.integers(0, max_len + 1, size=n)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=rowptr[1:])
    start = rng.integers(0, n, size=n)
    col = np.concatenate([np.sort((start[i] + 37 * np.arange(deg[i])) % n) for i in range(n)]).astype(np.int32)
    if explicit:
        val = rng.uniform(-1.0, 1.0, col.shape[0]).astype(np.float32)
    else:
        val = np.repeat((np.float32(1.0) / np.maximum(deg, 1).astype(np.float32)), deg).astype(np.float32)
    g = G.groot_graph_from_csr(rowptr, col, val)
    X = wl.uniform_features_numpy(44, 0, n, F)
    Y, plan, _, _ = _run(torch_cuda, g, T, X)
    assert G.groot_plan_query(plan, "weight_mode") == (2 if explicit else 1)
    if G.groot_plan_query(plan, "ld_pipelined"):
        depth = G.groot_plan_query(plan, "pipe_depth")
        # rows near the end wrap around to columns near 0: farther than a 2-byte code reaches, and such a column
        # is a named high-degree row only by chance -> those rows are left to the row list
        rows = np.repeat(np.arange(n), deg)
        short = (deg <= depth) & (deg < T)
        delta = col.astype(np.int64) - rows
        hot_mask = np.zeros(n, dtype=bool)
        hot_mask[np.nonzero(deg >= T)[0][:32767]] = True
        uncoded = np.unique(rows[short[rows] & ~((delta >= -16384) & (delta < 16384)) & ~hot_mask[col]])
        if uncoded.shape[0] * 50 <= n:
            assert G.groot_plan_query(plan, "csr_compressed") == 1
            assert G.groot_plan_query(plan, "uncoded_rows") == uncoded.shape[0]
            assert G.groot_plan_query(plan, "mid_rows") == int(((deg > depth) & (deg < T)).sum()) + uncoded.shape[0]
        else:
            assert G.groot_plan_query(plan, "csr_compressed") == 0
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, f"mixed rows max_len={max_len} T={T} F={F}")
    G.groot_set_tuning("csr_compress", 1)                    # the plain arrays at this size
    Y, _, _, _ = _run(torch_cuda, g, T, X)
    assert_close_to_oracle(Y, Y64, S, f"plain arrays, mixed rows max_len={max_len} T={T} F={F}")


@pytest.mark.parametrize("max_len,T,F,explicit", [(5, 32, 20, False), (6, 9, 28, True), (8, 32, 36, False), (8, 32, 60, True),
                                                   (7, 32, 124, False), (5, 6, 132, True), (5, 32, 252, False),
                                                   (8, 4, 256, True), (40, 16, 100, False), (4, 4, 48, False)])
def test_mixed_row_lengths_at_other_widths(torch_cuda, compact_always, max_len, T, F, explicit):
    """The same at widths that fill no power of two of lanes (the lanes past a row's end double its last one), with 5 to 8
    slots per row, and with the high-degree rows in the low-degree launch (T = 9 with rows up to 6: none at all) or in
    one of their own (thousands of pieces)."""
    test_mixed_row_lengths(torch_cuda, compact_always, max_len, T, F, explicit)


@pytest.mark.parametrize("pieces", [512, 513, 1023, 1024, 1025, 2047, 2048, 2600])
def test_high_degree_rows_beside_the_low_degree_ones(torch_cuda, pieces):
    """Around the numbers of pieces up to which the high-degree rows ride in the low-degree rows' launch (1,024 at F = 64 and from
    128 on, 512 at other widths), and around the one
    from which the list is dealt to the XCDs in runs of 64 (2600: the last runs are short or empty): rows of two pieces
    and of one, the first row and the last among them, next to rows of 1 to 4 entries."""
    n, T = 9000, 32
    heavies = 300 if pieces < 600 else 600 if pieces < 1200 else 1500
    split = pieces - heavies
    rng = np.random.default_rng(pieces)
    deg = rng.integers(1, 5, size=n)
    heavy = np.unique(np.concatenate([[0, n - 1], rng.permutation(np.arange(1, n - 1))[:heavies - 2]]))
    deg[heavy] = 40
    deg[heavy[:split]] = 600                              # two pieces of 300
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=rowptr[1:])
    col = np.concatenate([np.sort((i + 13 * np.arange(d)) % n) for i, d in enumerate(deg)]).astype(np.int32)
    val = np.repeat(np.float32(1.0) / deg.astype(np.float32), deg).astype(np.float32)
    g = G.groot_graph_from_csr(rowptr, col, val)
    for F in (32, 64, 100, 136):
        X = wl.uniform_features_numpy(45, 0, n, F)
        Y, plan, _, _ = _run(torch_cuda, g, T, X)
        assert G.groot_plan_query(plan, "hd_pieces") == pieces
        Y64, S = oracle.spmm_f64(rowptr, col, val, X)
        assert_close_to_oracle(Y, Y64, S, f"{pieces} pieces F={F}")


def _long_row_list(n_long, base, seed):
    """A graph with n_long rows of 9 to 12 entries among rows of base - 1 and base: as many rows as the list of those may be"""
    rng = np.random.default_rng(seed)
    n = 52 * n_long + 17
    lens = rng.integers(base - 1, base + 1, n)
    lens[rng.permutation(n)[:n_long]] = 9 + np.arange(n_long) % 4
    return n, _graph_of_row_lengths(lens, seed + 1)


@pytest.mark.parametrize("F,base,n_long", [(100, 5, 4096), (100, 5, 4097), (64, 8, 8192), (64, 8, 8193), (36, 6, 8193),
                                           (32, 5, 16384), (32, 5, 16385), (24, 5, 16385)])
def test_long_rows_beside_the_sweep_and_in_a_launch_of_their_own(torch_cuda, F, base, n_long):
    """Around the lengths up to which the list of longer low-degree rows rides in the sweep's launch: 4,096 rows where X fits
    the last-level cache, 8,192 with 6 to 8 slots per row, 16,384 at F = 32; at F = 24 it always does."""
    n, (rowptr, col, val) = _long_row_list(n_long, base, 70)
    X = wl.uniform_features_numpy(46, 0, n, F)
    Y, plan, _, _ = _run(torch_cuda, G.groot_graph_from_csr(rowptr, col, val), 32, X)
    if G.groot_plan_query(plan, "ld_pipelined"):
        assert G.groot_plan_query(plan, "pipe_depth") == base
        assert G.groot_plan_query(plan, "mid_rows") - G.groot_plan_query(plan, "uncoded_rows") == n_long
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, f"{n_long} long rows F={F}")


@pytest.mark.parametrize("n", [65536, 65537, 524287, 524288])
def test_narrow_matrices_without_high_degree_rows(torch_cuda, n):
    """F = 20 and 28 around the sizes between which a graph without high-degree rows stays on the plain kernel."""
    lens = np.random.default_rng(n).integers(3, 6, n)
    lens[:: 1000] = 9
    rowptr, col, val = _graph_of_row_lengths(lens, 74)
    for F in (20, 28):
        X = wl.uniform_features_numpy(47, 0, n, F)
        Y, _, _, _ = _run(torch_cuda, G.groot_graph_from_csr(rowptr, col, val), 32, X)
        Y64, S = oracle.spmm_f64(rowptr, col, val, X)
        assert_close_to_oracle(Y, Y64, S, f"n={n} F={F}")


def test_masked_rows_do_not_slow_the_sweep_down(torch_cuda):
    """One row in 52 with 9 to 12 entries at a width that fills no power of two of lanes: the call takes what these rows' own
    entries take (measured 1.05 to 1.1 times the call without them), not 1.6 times as when the masked rows' sums all went
    to one place."""
    torch = torch_cuda
    n, long_rows = _long_row_list(20000, 5, 71)
    times = []
    for rowptr, col, val in (_graph_of_row_lengths(np.random.default_rng(72).integers(4, 6, n), 72), long_rows):
        plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
        G.groot_plan_upload(plan, 100)
        X, Y = torch.rand((n, 100), device="cuda"), torch.empty((n, 100), device="cuda")
        call = lambda: G.groot_spmm_execute(plan, X, Y)
        call()
        times.append(_best_time(torch, call))
    assert times[1] < 1.35 * times[0], f"{times[0]:.3f} ms without long rows, {times[1]:.3f} ms with"


@pytest.mark.parametrize("case", ["aig", "stress"])
def test_transposed_spmm(torch_cuda, case):
    """dX = A_hat^T dY through groot_graph_transpose + the ordinary plan/execute, against the oracle's
    scatter definition of the transposed product."""
    if case == "aig":
        aig, g, (rowptr, col, val, pol) = _aig_case(48, 2)
        n, T, F = 2 * aig.num_nodes, 32, 64
    else:
        s = wl.stress_graph(7, 1 << 15, window=1024, dmin=64, dmax=4096)
        g = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
        rowptr, col, val, n, T, F = s.rowptr, s.col, s.val, s.n, 32, 32
    dY = wl.uniform_features_numpy(13, 0, n, F)
    gt = G.groot_graph_transpose(g)
    dX, _, _, _ = _run(torch_cuda, gt, T, dY)
    want, S = oracle.spmm_t_f64(rowptr, col, val, dY)
    assert_close_to_oracle(dX, want, S, f"transposed {case}")


@pytest.fixture(params=[1, 0], ids=["detect-uniform", "as-given"])
def uniform_detect(request):
    """Graphs given as CSR with weights 1/row length run as row-uniform weights (the weight array is not read)
    when groot_plan_upload detects that, and entry by entry when it is told not to look: both must be right."""
    G.groot_set_tuning("uniform_detect", request.param)
    yield request.param
    G.groot_set_tuning("uniform_detect", 1)


SAGE_VARIANTS = {"wavefronts": dict(sage_kernel=1), "roles-bf16": dict(sage_kernel=0, sage_split=1),
                 "roles-fp32": dict(sage_kernel=0, sage_split=0)}


@pytest.fixture(params=sorted(SAGE_VARIANTS))
def sage_variant(request):
    """Every fused-layer test runs with each kernel: the self-contained wavefronts (bf16 piece products), and
    the 12-wavefront kernel with bf16 piece products and with fp32 matrix instructions."""
    for k, v in SAGE_VARIANTS[request.param].items():
        G.groot_set_tuning(k, v)
    yield request.param
    G.groot_set_tuning("sage_kernel", 1)
    G.groot_set_tuning("sage_split", 1)


def _sage_check(torch, g, rowptr, col, val, T, n, seed, relu, with_bias, what, row_scale=None, F=64, F_out=None,
                pieces=3):
    """F_out None: the square call (F -> F); else the call with separate input and output widths.  pieces: what
    the library's sage_pieces knob is set to (the caller sets it), for the tolerance."""
    rng = np.random.default_rng(seed)
    X = wl.uniform_features_numpy(seed, 0, n, F)
    if row_scale is not None:
        X = (X * row_scale[:, None]).astype(np.float32)
    FO = F if F_out is None else F_out
    Wn, Ws = (rng.uniform(-0.125, 0.125, (F, FO)).astype(np.float32) for _ in range(2))
    b = rng.uniform(-0.125, 0.125, FO).astype(np.float32) if with_bias else None
    plan = G.groot_spmm_plan(g, T)
    G.groot_plan_upload(plan, F)
    dev = lambda a: torch.from_numpy(a).cuda()
    guard = 2
    buf = torch.full((n + 2 * guard, FO), float("nan"), dtype=torch.float32, device="cuda")
    buf[:guard] = 777.0
    buf[n + guard:] = 777.0
    H = buf[guard:n + guard]
    if F_out is None:
        G.groot_sage_layer_forward(plan, dev(X), dev(Wn), dev(Ws), None if b is None else dev(b), relu, H, F)
    else:
        G.groot_sage_layer_forward_io(plan, dev(X), dev(Wn), dev(Ws), None if b is None else dev(b), relu, H, F, FO)
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    assert (out[:guard] == 777.0).all() and (out[n + guard:] == 777.0).all(), "wrote outside H"
    want, A, S = oracle.sage_layer_f64(rowptr, col, val, X, Wn, Ws, b, relu)
    a64 = lambda a: np.abs(a.astype(np.float64))
    scale = np.abs(A) @ a64(Wn) + a64(X) @ a64(Ws) + (a64(b) if b is not None else 0.0)
    tol = layer_tolerance(S, scale, a64(Wn), pieces=pieces)
    err = np.abs(out[guard:n + guard].astype(np.float64) - want)
    assert np.isfinite(err).all(), f"{what}: non-finite output"
    assert (err <= tol).all(), f"{what}: max err/tol {np.max(err / tol)}"
    return out[guard:n + guard], scale, err, S @ a64(Wn)


@pytest.mark.parametrize("n_bits,batch,T,relu,with_bias", [(48, 2, 32, True, True), (48, 1, 32, False, False),
                                                            (3, 1, 32, True, True), (17, 3, 5, True, False),
                                                            (40, 1, 1, False, True)])
def test_fused_sage_layer_on_multipliers(torch_cuda, sage_variant, n_bits, batch, T, relu, with_bias):
    """H = act((A_hat X) Wn + X Ws + b) with the aggregation kept on chip; rows counts that are not
    multiples of the 64-row tile, high-degree rows (picked up from the HD kernel), every row high-degree."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
    _sage_check(torch_cuda, g, rowptr, col, val, T, batch * aig.num_nodes, 100 + n_bits, relu, with_bias,
                f"sage {n_bits}x{batch} T={T}")


@pytest.mark.parametrize("n_bits,batch,T,relu,with_bias", [(48, 2, 32, True, True), (3, 1, 32, False, False),
                                                            (17, 3, 5, True, False), (40, 1, 1, False, True)])
def test_fused_sage_layer_width_32(torch_cuda, n_bits, batch, T, relu, with_bias):
    """The layer at the embedding width of the paper's kernel evaluation (F = 32): 8 lanes per row, two sweeps
    per 16-row tile, a 64 x 32 weight matrix."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
    _sage_check(torch_cuda, g, rowptr, col, val, T, batch * aig.num_nodes, 300 + n_bits, relu, with_bias,
                f"sage F=32 {n_bits}x{batch} T={T}", F=32)


@pytest.mark.parametrize("F_in,F_out", [(32, 16), (32, 64), (64, 32), (64, 16), (32, 32), (64, 64)])
@pytest.mark.parametrize("n_bits,batch,T,relu,with_bias", [(48, 2, 32, True, True), (17, 3, 5, False, False),
                                                            (40, 1, 1, True, False)])
def test_fused_sage_layer_input_and_output_widths(torch_cuda, F_in, F_out, n_bits, batch, T, relu, with_bias):
    """A layer that narrows or widens (X [N, F_in] -> H [N, F_out]): every supported pair of widths, with
    high-degree rows (their sums pass through the plan's side buffer), low thresholds, and every row
    high-degree."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
    _sage_check(torch_cuda, g, rowptr, col, val, T, batch * aig.num_nodes, 500 + n_bits + F_in + F_out, relu, with_bias,
                f"sage {F_in}->{F_out} {n_bits}x{batch} T={T}", F=F_in, F_out=F_out)


def test_fused_sage_layer_widths_on_booth_and_stress_shapes(torch_cuda):
    """High-degree rows scattered through the graph (Booth recoding signals; heavy rows of a polarized graph,
    some of them split into pieces): every tile that holds one takes the path that looks its sum up."""
    aig = wl.booth_multiplier_aig(32)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 2)
    rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, 2)
    _sage_check(torch_cuda, g, rowptr, col, val, 16, 2 * aig.num_nodes, 61, True, True, "sage booth 64->32", F=64, F_out=32)
    s = wl.stress_graph(12, 1 << 14, window=512, dmin=64, dmax=2048)
    gs = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
    _sage_check(torch_cuda, gs, s.rowptr, s.col, s.val, 32, s.n, 62, False, True, "sage stress 32->16", F=32, F_out=16)
    plan = G.groot_spmm_plan(g, 16)
    G.groot_plan_upload(plan, 64)
    z = lambda *shape: torch_cuda.zeros(shape, device="cuda")
    n = 2 * aig.num_nodes
    with pytest.raises(G.GrootError):                       # output width 48 is not built
        G.groot_sage_layer_forward_io(plan, z(n, 64), z(64, 48), z(64, 48), None, True, z(n, 48), 64, 48)
    with pytest.raises(G.GrootError):                       # input width 16 is not built
        G.groot_sage_layer_forward_io(plan, z(n, 16), z(16, 32), z(16, 32), None, True, z(n, 32), 16, 32)
    with pytest.raises(ValueError):                         # the binding: weights too small for 64 -> 32
        G.groot_sage_layer_forward_io(plan, z(n, 64), z(32, 32), z(64, 32), None, True, z(n, 32), 64, 32)


def test_fused_sage_layer_bf16_pieces_keep_fp32_accuracy(torch_cuda):
    """The six-piece products must be as accurate as fp32 products, not merely within the layer's tolerance:
    against the fp64 layer every kernel stays within 4e-6 of the sum of absolute terms of the dense part plus
    the rounding of the aggregation itself (rows of at most 6 entries summed in order: 7 * 2^-24 of their
    absolute terms; the 81 high-degree rows of 41 entries as trees: below 2^-20), pushed through |Wn|.  Plain
    16-bit operands (the low pieces dropped) would leave about 1.5e-5 of the scale."""
    aig, g, (rowptr, col, val, pol) = _aig_case(40, 2)
    n = 2 * aig.num_nodes
    try:
        for name, knobs in SAGE_VARIANTS.items():
            for k, v in knobs.items():
                G.groot_set_tuning(k, v)
            _, scale, err, SW = _sage_check(torch_cuda, g, rowptr, col, val, 32, n, 77, False, True, f"sage {name}")
            bound = 4e-6 * scale + 2.0 ** -20 * SW + 1e-7
            assert (err <= bound).all(), f"{name}: {np.max(err / bound)}"
    finally:
        G.groot_set_tuning("sage_kernel", 1)
        G.groot_set_tuning("sage_split", 1)


@pytest.mark.parametrize("F_in,F_out", [(64, 64), (32, 32), (64, 16), (32, 64)])
@pytest.mark.parametrize("n_bits,batch,T,relu,with_bias", [(48, 2, 32, True, True), (17, 3, 5, False, False)])
def test_fused_sage_layer_with_two_pieces_per_operand(torch_cuda, F_in, F_out, n_bits, batch, T, relu, with_bias):
    """The knob sage_pieces = 2: three piece products instead of six.  Within the wider bar that two pieces allow
    (3 * 2^-18 of the dense part's absolute terms more), and not the same numbers as with three pieces (the knob
    does reach the kernel)."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
    n = batch * aig.num_nodes
    args = (torch_cuda, g, rowptr, col, val, T, n, 900 + n_bits + F_in + F_out, relu, with_bias)
    three = _sage_check(*args, f"sage {F_in}->{F_out}, three pieces", F=F_in, F_out=F_out)[0]
    G.groot_set_tuning("sage_pieces", 2)
    try:
        two, scale, err, _ = _sage_check(*args, f"sage {F_in}->{F_out}, two pieces", F=F_in, F_out=F_out, pieces=2)
    finally:
        G.groot_set_tuning("sage_pieces", 3)
    assert not np.array_equal(two, three)
    with pytest.raises(G.GrootError):
        G.groot_set_tuning("sage_pieces", 4)


@pytest.mark.parametrize("F_out,F_in", [(64, 64), (32, 32), (64, 16), (32, 64), (64, 32), (32, 16)])
@pytest.mark.parametrize("n_bits,batch,T", [(48, 2, 32), (17, 3, 5), (40, 1, 1), (3, 1, 32)])
def test_fused_sage_layer_backward_data(torch_cuda, F_out, F_in, n_bits, batch, T):
    """dX = A_hat^T (dZ Wn^T) + dZ Ws^T through the layer kernel's gradient form (unit-weight sums of the rows of
    dZ / deg, own row scaled back by its length) against the fp64 definition: every pair of widths, high-degree
    rows (summed by the HD kernel with unit weights), every row high-degree, a ragged last tile.  About half of
    dZ is zero, as behind a ReLU.  groot_rows_over_degree is the division it claims to be, bit for bit."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
    _backward_data_check(torch_cuda, g, rowptr, col, val, T, batch * aig.num_nodes, 700 + n_bits + F_out + F_in, F_out, F_in)


def _backward_data_check(torch, g, rowptr, col, val, T, n, seed, F_out, F_in):
    rng = np.random.default_rng(seed)
    dZ = (wl.uniform_features_numpy(seed, 0, n, F_out) * (rng.random((n, F_out)) < 0.55)).astype(np.float32)
    Wn, Ws = (rng.uniform(-0.125, 0.125, (F_in, F_out)).astype(np.float32) for _ in range(2))
    plan = G.groot_spmm_plan(g, T)
    G.groot_plan_upload(plan, F_out)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dZ_dev = dev(dZ)
    scaled = torch.empty_like(dZ_dev)
    G.groot_rows_over_degree(plan, dZ_dev, scaled)
    deg = np.diff(rowptr).astype(np.float32)
    assert np.array_equal(scaled.cpu().numpy(), dZ / deg[:, None])
    G.groot_rows_over_degree(plan, dZ_dev, dZ_dev)            # in place
    assert torch.equal(dZ_dev, scaled)
    guard = 2
    buf = torch.full((n + 2 * guard, F_in), float("nan"), dtype=torch.float32, device="cuda")
    buf[:guard] = 777.0
    buf[n + guard:] = 777.0
    G.groot_sage_layer_backward_data(plan, scaled, dev(Wn.T), dev(Ws.T), buf[guard:n + guard])
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    assert (out[:guard] == 777.0).all() and (out[n + guard:] == 777.0).all(), "wrote outside dX"
    want, Tm, S = oracle.sage_layer_backward_data_f64(rowptr, col, val, dZ, Wn, Ws)
    a64 = lambda a: np.abs(a.astype(np.float64))
    scale = np.abs(Tm) @ a64(Wn.T) + a64(dZ) @ a64(Ws.T)
    tol = layer_tolerance(S, scale, a64(Wn.T))
    err = np.abs(out[guard:n + guard].astype(np.float64) - want)
    assert np.isfinite(err).all()
    assert (err <= tol).all(), f"max err/tol {np.max(err / tol)}"


def test_fused_sage_layer_gradients_on_the_booth_shape(torch_cuda):
    """High-degree rows scattered through the graph and rows of up to 8 entries (the Booth recoding signals): the
    gradient kernels' plain path for the tiles that hold them, input gradient and weight gradients."""
    aig = wl.booth_multiplier_aig(32)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 2)
    rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, 2)
    n = 2 * aig.num_nodes
    _backward_data_check(torch_cuda, g, rowptr, col, val, 16, n, 71, 64, 32)
    _backward_data_check(torch_cuda, g, rowptr, col, val, 16, n, 72, 32, 32)
    _wgrad_check(torch_cuda, g, rowptr, col, val, 16, n, 73, 64)
    _wgrad_check(torch_cuda, g, rowptr, col, val, 16, n, 74, 32, F_out=16)


def test_fused_sage_layer_backward_data_errors(torch_cuda):
    """The gradient form needs a symmetric graph with mean weights (it uses A_hat^T = A D^-1): a graph given as
    CSR, the transposed graph and a graph built without normalisation are refused, and so are unsupported widths
    and overlapping buffers."""
    torch = torch_cuda
    z = lambda *shape: torch.zeros(shape, device="cuda")
    aig, g, (rowptr, col, val, pol) = _aig_case(17, 1)
    n = aig.num_nodes
    for bad in (G.groot_graph_from_csr(rowptr, col, val), G.groot_graph_transpose(g),
                G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 1, flags=G.GROOT_SYMMETRIC | G.GROOT_SELF_LOOPS)):
        plan = G.groot_spmm_plan(bad, 32)
        G.groot_plan_upload(plan, 64)
        with pytest.raises(G.GrootError):
            G.groot_sage_layer_backward_data(plan, z(n, 64), z(64, 64), z(64, 64), z(n, 64))
    plan = G.groot_spmm_plan(g, 32)
    with pytest.raises(G.GrootError):                       # not uploaded
        G.groot_sage_layer_backward_data(plan, z(n, 64), z(64, 64), z(64, 64), z(n, 64))
    G.groot_plan_upload(plan, 64)
    with pytest.raises(G.GrootError):                       # dZ of width 16 is not built
        G.groot_sage_layer_backward_data(plan, z(n, 16), z(16, 32), z(16, 32), z(n, 32))
    with pytest.raises(G.GrootError):                       # dX of width 48 is not built
        G.groot_sage_layer_backward_data(plan, z(n, 64), z(64, 48), z(64, 48), z(n, 48))
    x = z(n, 64)
    with pytest.raises(G.GrootError):                       # in place
        G.groot_sage_layer_backward_data(plan, x, z(64, 64), z(64, 64), x)
    with pytest.raises(ValueError):                         # the binding: weights of the wrong shape
        G.groot_sage_layer_backward_data(plan, z(n, 64), z(32, 32), z(64, 32), z(n, 32))


def _wgrad_check(torch, g, rowptr, col, val, T, n, seed, F, F_out=None):
    """X of width F, dZ of width F_out (default F)."""
    FO = F if F_out is None else F_out
    rng = np.random.default_rng(seed)
    X = wl.uniform_features_numpy(seed, 0, n, F)
    dZ = (wl.uniform_features_numpy(seed + 1, 0, n, FO) * (rng.random((n, FO)) < 0.55)).astype(np.float32)
    plan = G.groot_spmm_plan(g, T)
    G.groot_plan_upload(plan, F)
    need = G.groot_sage_layer_backward_weights_workspace(plan, F, FO)
    ws = torch.full((need // 4 + 64,), float("nan"), dtype=torch.float32, device="cuda")
    ws[need // 4:] = 777.0
    out = torch.full((2, F, FO), float("nan"), dtype=torch.float32, device="cuda")
    dev = lambda a: torch.from_numpy(a).cuda()
    Xd, Zd = dev(X), dev(dZ)
    G.groot_sage_layer_backward_weights(plan, Xd, Zd, out[0], out[1], ws, F)
    torch.cuda.synchronize()
    assert bool((ws[need // 4:] == 777.0).all()), "wrote past the workspace it asked for"
    got = out.cpu().numpy().astype(np.float64)
    again = torch.full_like(out, float("nan"))
    G.groot_sage_layer_backward_weights(plan, Xd, Zd, again[0], again[1], ws, F)
    torch.cuda.synchronize()
    assert torch.equal(out, again), "no atomics: the same bits on every run"
    dWn, dWs, Sn, Ss = oracle.sage_layer_backward_weights_f64(rowptr, col, val, X, dZ)
    rows = wgrad_rows_per_wavefront(n, torch.cuda.get_device_properties(0).multi_processor_count)
    tol_n, tol_s = wgrad_tolerance(Sn, Ss, np.abs(dZ.astype(np.float64)).sum(axis=0), rows, F, FO)
    assert np.isfinite(got).all()
    en, es = np.abs(got[0] - dWn), np.abs(got[1] - dWs)
    assert (en <= tol_n).all(), f"dWn: max err/tol {np.max(en / tol_n)}"
    assert (es <= tol_s).all(), f"dWs: max err/tol {np.max(es / tol_s)}"
    return got


@pytest.mark.parametrize("F", [64, 32])
@pytest.mark.parametrize("n_bits,batch,T", [(48, 2, 32), (17, 3, 5), (40, 1, 1), (3, 1, 32), (64, 1, 32)])
def test_fused_sage_layer_backward_weights(torch_cuda, F, n_bits, batch, T):
    """dWn = (A_hat X)^T dZ and dWs = X^T dZ in one pass against the fp64 definition: both widths, high-degree rows
    (their sums come from the HD kernel), every row high-degree, fewer rows than one tile, a ragged last tile;
    twice, bit for bit the same; nothing written past the workspace."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
    _wgrad_check(torch_cuda, g, rowptr, col, val, T, batch * aig.num_nodes, 800 + n_bits + F, F)


@pytest.mark.parametrize("F_in,F_out", [(64, 32), (64, 16), (32, 64), (32, 16)])
@pytest.mark.parametrize("n_bits,batch,T", [(48, 2, 32), (17, 3, 5), (3, 1, 32)])
def test_fused_sage_layer_backward_weights_of_a_layer_that_narrows_or_widens(torch_cuda, F_in, F_out, n_bits, batch, T):
    """X [N, F_in] and dZ [N, F_out] of different widths: the rows of dZ ride with the lane groups of X."""
    aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
    _wgrad_check(torch_cuda, g, rowptr, col, val, T, batch * aig.num_nodes, 850 + n_bits + F_in + F_out, F_in, F_out=F_out)


def test_fused_sage_layer_backward_weights_other_graphs_and_errors(torch_cuda):
    """Unit weights (a graph built without normalisation), a graph given as CSR whose weights are 1 / row length
    (heavy rows split into pieces), the knob sage_pieces, which does not reach this call (the same bits); explicit weights, a short workspace, F = 16 and a plan
    that is not uploaded are refused."""
    torch = torch_cuda
    aig = wl.csa_multiplier_aig(24)
    flags = G.GROOT_SYMMETRIC | G.GROOT_SELF_LOOPS
    g1 = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 2, flags=flags)
    rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, 2, flags=flags)
    _wgrad_check(torch, g1, rowptr, col, val, 32, 2 * aig.num_nodes, 31, 64)
    s = wl.stress_graph(12, 1 << 14, window=512, dmin=64, dmax=2048)
    gs = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
    _wgrad_check(torch, gs, s.rowptr, s.col, s.val, 32, s.n, 32, 32)
    aig2, g2, (rowptr2, col2, val2, _) = _aig_case(48, 2)
    three = _wgrad_check(torch, g2, rowptr2, col2, val2, 32, 2 * aig2.num_nodes, 33, 64)
    G.groot_set_tuning("sage_pieces", 2)
    try:
        assert np.array_equal(_wgrad_check(torch, g2, rowptr2, col2, val2, 32, 2 * aig2.num_nodes, 33, 64), three)
    finally:
        G.groot_set_tuning("sage_pieces", 3)
    z = lambda *shape: torch.zeros(shape, device="cuda")
    n = 2 * aig2.num_nodes
    plan = G.groot_spmm_plan(g2, 32)
    with pytest.raises(G.GrootError):                       # not uploaded
        G.groot_sage_layer_backward_weights(plan, z(n, 64), z(n, 64), z(64, 64), z(64, 64), z(1 << 24), 64)
    G.groot_plan_upload(plan, 64)
    need = G.groot_sage_layer_backward_weights_workspace(plan, 64)
    with pytest.raises(G.GrootError):                       # workspace one float short
        G.groot_sage_layer_backward_weights(plan, z(n, 64), z(n, 64), z(64, 64), z(64, 64), z(need // 4 - 1), 64)
    with pytest.raises(G.GrootError):                       # width 16 is not built
        G.groot_sage_layer_backward_weights(plan, z(n, 16), z(n, 16), z(16, 16), z(16, 16), z(need // 4), 16)
    with pytest.raises(G.GrootError):
        G.groot_sage_layer_backward_weights_workspace(plan, 48)
    plan_t = G.groot_spmm_plan(G.groot_graph_transpose(g2), 32)     # explicit weights
    G.groot_plan_upload(plan_t, 64)
    with pytest.raises(G.GrootError):
        G.groot_sage_layer_backward_weights(plan_t, z(n, 64), z(n, 64), z(64, 64), z(64, 64), z(need // 4), 64)


@pytest.mark.parametrize("F_in,F_out,graph", [(32, 16, "all_noted"), (64, 64, "csa"), (32, 32, "csa"), (64, 32, "one")])
def test_weight_gradients_at_the_edges_of_the_pipeline(torch_cuda, F_in, F_out, graph):
    """Edges of the weight-gradient kernel's bookkeeping.  "all_noted": with T = 4 nearly every row is high-degree, so that
    every tile is noted, and 1,277,200 rows are 39 tiles for some wavefronts: more than the 32 that one notes before it
    must complete them.  "csa": 62,808 rows, 3,926 tiles: the last one ragged, wavefronts with two tiles, one or none;
    rows past the end of X and of dZ must not be read as numbers (NaN behind both).  "one": a single row."""
    torch = torch_cuda
    T = 32
    if graph == "all_noted":
        aig, g, (rowptr, col, val, _) = _aig_case(400, 1)
        n, T = aig.num_nodes, 4
        noted = np.add.reduceat(np.diff(rowptr) >= T, np.arange(0, n, 16)) > 0
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        tile = np.arange(noted.size)
        part = tile // -(-noted.size // 8)
        wavefront = part * (cus // 8 * 8) + (tile - part * -(-noted.size // 8)) % (cus // 8 * 8)
        assert np.bincount(wavefront, weights=noted).max() > 32
    elif graph == "csa":
        aig, g, (rowptr, col, val, _) = _aig_case(89, 1)
        n = aig.num_nodes
    else:
        rowptr, col, val = np.array([0, 1], np.int64), np.array([0], np.int32), np.array([1.0], np.float32)
        g, n = G.groot_graph_from_csr(rowptr, col, val), 1
    _wgrad_check(torch, g, rowptr, col, val, T, n, 95, F_in, F_out=F_out)
    if graph == "csa":
        assert n % 16 != 0
        plan = G.groot_spmm_plan(g, 32)
        G.groot_plan_upload(plan, F_in)
        X = torch.full((n + 64, F_in), float("nan"), device="cuda")
        dZ = torch.full((n + 64, F_out), float("nan"), device="cuda")
        X[:n].uniform_(-1, 1)
        dZ[:n].uniform_(-1, 1)
        ws = torch.empty(G.groot_sage_layer_backward_weights_workspace(plan, F_in, F_out) // 4, device="cuda")
        dW = torch.empty((2, F_in, F_out), device="cuda")
        G.groot_sage_layer_backward_weights(plan, X, dZ, dW[0], dW[1], ws)
        assert bool(torch.isfinite(dW).all())


@pytest.mark.parametrize("case", ["all_noted", "lut4", "cells", "ragged"])
def test_fused_layer_at_the_edges_of_the_pipeline(torch_cuda, case):
    """Edges of the layer kernel's pipeline.  "all_noted": T = 4 makes nearly every row high-degree, so every tile of every
    wavefront (717,900 rows, 44,869 tiles over 2,048 wavefronts) has rows that its slots do not serve.  "lut4": rows of 7 entries, 8 slots per row and half a tile in flight; "cells":
    rows of 6.  "ragged": a last tile of 1 row, and of 15; forward layer, input gradient and weight gradients."""
    torch = torch_cuda
    if case == "all_noted":
        aig, g, (rowptr, col, val, pol) = _aig_case(300, 1)
        _sage_check(torch, g, rowptr, col, val, 4, aig.num_nodes, 41, True, True, case, F=32, F_out=16)
    elif case in ("lut4", "cells"):
        c = (wl.lut4_csa_graph if case == "lut4" else wl.cellmap_csa_graph)(40, 2)
        g = G.groot_graph_from_csr(c.rowptr, c.col, c.val)
        for F, FO in ((64, 64), (64, 16), (32, 32), (32, 64)):
            _sage_check(torch, g, c.rowptr, c.col, c.val, 32, c.n, 42 + F, FO != 32, True, case, F=F, F_out=FO)
            _wgrad_check(torch, g, c.rowptr, c.col, c.val, 32, c.n, 43 + F, F, F_out=FO)
    else:
        for n_bits, batch, left in ((15, 1, 15), (17, 1, 1)):
            aig, g, (rowptr, col, val, pol) = _aig_case(n_bits, batch)
            n = batch * aig.num_nodes
            assert n % 16 == left
            for F, FO in ((64, 64), (32, 16), (32, 32)):
                _sage_check(torch, g, rowptr, col, val, 32, n, 44 + F, False, True, case, F=F, F_out=FO)
                _backward_data_check(torch, g, rowptr, col, val, 32, n, 45 + F, F, FO)
                _wgrad_check(torch, g, rowptr, col, val, 32, n, 46 + F, F, F_out=FO)


def _graph_of_row_lengths(lens, seed):
    """CSR arrays with these row lengths: consecutive columns from a random one within 1,000 of the row, mean weights"""
    rng = np.random.default_rng(seed)
    n = lens.shape[0]
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    first = np.clip(np.arange(n) + rng.integers(-1000, 1000, n), 0, n - lens)
    row = np.repeat(np.arange(n), lens)
    col = (first[row] + np.arange(rowptr[-1]) - rowptr[row]).astype(np.int32)
    val = np.repeat(np.float32(1) / np.maximum(lens, 1).astype(np.float32), lens).astype(np.float32)
    return rowptr, col, val


@pytest.mark.parametrize("n_hd", [0, 1, 64, 65, 4096, 4097])
def test_fused_layer_rows_that_the_slots_do_not_serve(torch_cuda, n_hd):
    """Rows of every length from 0 to 31 among short ones, and n_hd high-degree rows: the sums that are parked over a tile's
    own (eight entries at a time: 8, 9, 16, 17, 24, 25), the search for a row's place in the list of high-degree rows (64
    samples a step: one step up to 64 rows, two up to 4,096), first and last row of the graph among them, a ragged last
    tile with long rows."""
    rng = np.random.default_rng(60 + n_hd)
    n = 16 * 640 + 11
    lens = rng.integers(3, 6, n)
    odd = rng.permutation(n)[:3200]
    lens[odd] = np.arange(3200) % 32
    heavy = np.concatenate([[0, n - 1], 1 + rng.permutation(n - 2)])[:n_hd]
    lens[heavy] = rng.integers(32, 40, n_hd)
    rowptr, col, val = _graph_of_row_lengths(lens, 61)
    g = G.groot_graph_from_csr(rowptr, col, val)
    assert G.groot_plan_view(G.groot_spmm_plan(g, 32))["n_hd"] == n_hd
    for F, FO in ((64, 64), (32, 16)):
        _sage_check(torch_cuda, g, rowptr, col, val, 32, n, 62 + F, False, True, f"{n_hd} heavy", F=F, F_out=FO)
        _wgrad_check(torch_cuda, g, rowptr, col, val, 32, n, 63 + F, F, F_out=FO)


def test_weight_gradients_noted_tiles_count_towards_a_fold(torch_cuda):
    """A wavefront's accumulators take at most 512 rows between two additions to its second set of sums, the tiles that it
    notes and completes later among them.  The first wavefront's first 32 tiles have a row of 8 entries each, so they are
    noted, and the first of these rows adds 2^27 to every sum; its next 32 tiles add 512 rows of ones, every four of which
    would be lost beside 2^27 (spacing 16) but not as 512."""
    torch = torch_cuda
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    stride = cus // 8 * 8                                    # wavefronts that share an eighth of the tiles
    n = 16 * 8 * 64 * stride
    tile_row = 16 * stride * np.arange(64)                   # first rows of the first wavefront's tiles
    lens = np.ones(n, np.int64)
    lens[tile_row[:32]] = 8
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.repeat(np.arange(n), lens).astype(np.int32)
    col += (np.arange(rowptr[-1]) - rowptr[col]).astype(np.int32)
    val = np.repeat(np.float32(1) / lens.astype(np.float32), lens).astype(np.float32)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, 32)
    X, dZ = torch.ones((n, 32), device="cuda"), torch.zeros((n, 16), device="cuda")
    dZ[0] = 2.0 ** 27
    dZ[torch.from_numpy((tile_row[32:, None] + np.arange(16)).ravel()).cuda()] = 1.0
    ws = torch.empty(G.groot_sage_layer_backward_weights_workspace(plan, 32, 16) // 4, device="cuda")
    dW = torch.empty((2, 32, 16), device="cuda")
    G.groot_sage_layer_backward_weights(plan, X, dZ, dW[0], dW[1], ws)
    assert bool((dW == 2.0 ** 27 + 512).all()), (dW - 2.0 ** 27).unique()


@pytest.mark.parametrize("F_in,F_out", [(64, 64), (64, 16), (32, 32)])
def test_weight_gradients_of_the_wavefronts_meet_in_fp64(torch_cuda, F_in, F_out):
    """2,048 rows, one tile per wavefront: two wavefronts of a workgroup add 2^24 and 1, one of another workgroup -2^24.  No
    fp32 rounding on the way between them: the sum is 1."""
    torch = torch_cuda
    n = 2048
    rowptr, col, val = np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.ones(n, np.float32)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F_in)
    X, dZ = torch.ones((n, F_in), device="cuda"), torch.zeros((n, F_out), device="cuda")
    dZ[0], dZ[16], dZ[8 * 16] = 2.0 ** 24, 1.0, -2.0 ** 24
    ws = torch.empty(G.groot_sage_layer_backward_weights_workspace(plan, F_in, F_out) // 4, device="cuda")
    dW = torch.empty((2, F_in, F_out), device="cuda")
    G.groot_sage_layer_backward_weights(plan, X, dZ, dW[0], dW[1], ws)
    assert bool((dW == 1.0).all()), dW.unique()


def _best_time(torch, fn, reps=8, inner=4):
    """milliseconds of a call among others, the best of some"""
    best = float("inf")
    for _ in range(reps):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(inner):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / inner)
    return best


def test_a_few_long_rows_do_not_slow_the_layer_down(torch_cuda):
    """One row in 50 with 9 to 12 entries, so that one tile in four has one: the layer takes what these rows' own entries
    take (1.15 times the layer without them, measured), not the time of computing such tiles twice (2.0 times)."""
    torch = torch_cuda
    n, times = 1 << 20, []
    for frac in (0.0, 0.02):
        rng = np.random.default_rng(8)
        lens = rng.integers(4, 6, n)
        long = rng.random(n) < frac
        lens[long] = rng.integers(9, 13, int(long.sum()))
        g = G.groot_graph_from_csr(*_graph_of_row_lengths(lens, 9))
        plan = G.groot_spmm_plan(g, 32)
        G.groot_plan_upload(plan, 64)
        X, H = torch.rand((n, 64), device="cuda"), torch.empty((n, 64), device="cuda")
        W = torch.rand((2, 64, 64), device="cuda")
        call = lambda: G.groot_sage_layer_forward(plan, X, W[0], W[1], None, False, H, 64)
        call()
        times.append(_best_time(torch, call))
    assert times[1] < 1.4 * times[0], f"{times[0]:.3f} ms without long rows, {times[1]:.3f} ms with"


def test_calls_that_only_enqueue_run_under_graph_capture(torch_cuda):
    """groot_spmm_execute, the fused layer, its input gradient (with groot_rows_over_degree) and its weight
    gradients only enqueue kernels and allocate nothing, so a caller may capture them into a graph: the captured
    sequence is replayed three times on fresh inputs, with eager work and synchronisation between the replays, and
    every replay gives bit for bit what the same calls give eagerly."""
    torch = torch_cuda
    aig, g, _ = _aig_case(48, 2)
    n, F = 2 * aig.num_nodes, 64
    plan = G.groot_spmm_plan(g, 32)
    G.groot_plan_upload(plan, F)
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *shape: torch.rand(shape, generator=gen, device="cuda") - 0.5
    Wn, Ws, b = rnd(F, F) * 0.25, rnd(F, F) * 0.25, rnd(F) * 0.25
    WnT, WsT = Wn.t().contiguous(), Ws.t().contiguous()
    workspace = torch.empty((G.groot_sage_layer_backward_weights_workspace(plan, F) // 4,), device="cuda")
    X, dZ = rnd(n, F), rnd(n, F)

    def calls(out):
        G.groot_spmm_execute(plan, X, out["Y"], F)
        G.groot_sage_layer_forward(plan, X, Wn, Ws, b, True, out["H"], F)
        G.groot_rows_over_degree(plan, dZ, out["scaled"])
        G.groot_sage_layer_backward_data(plan, out["scaled"], WnT, WsT, out["dX"])
        G.groot_sage_layer_backward_weights(plan, X, dZ, out["dW"][0], out["dW"][1], workspace)

    buffers = lambda: dict(Y=torch.empty((n, F), device="cuda"), H=torch.empty((n, F), device="cuda"),
                           scaled=torch.empty((n, F), device="cuda"), dX=torch.empty((n, F), device="cuda"),
                           dW=torch.empty((2, F, F), device="cuda"))
    eager, captured = buffers(), buffers()
    calls(eager)                                             # warm-up outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls(captured)
    for replay in range(3):
        X.copy_(rnd(n, F))                                   # eager work between the replays
        dZ.copy_(rnd(n, F) * (rnd(n, F) > 0))
        for t in captured.values():
            t.fill_(float("nan"))
        calls(eager)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name in eager:
            assert torch.equal(eager[name], captured[name]), f"replay {replay}: {name}"


def test_fused_sage_layer_wide_dynamic_range(torch_cuda, sage_variant):
    """Feature rows scaled by powers of two from 2^-60 to 2^60 (each copy of the multiplier its own scale, so
    that neighbours share it): the bf16 pieces have the exponent range of fp32, so the error stays relative
    to the terms of each output element at every magnitude."""
    aig, g, (rowptr, col, val, pol) = _aig_case(24, 5)
    n = 5 * aig.num_nodes
    row_scale = np.repeat(np.ldexp(1.0, [-60, -20, 0, 20, 60]), aig.num_nodes).astype(np.float32)
    F = 64
    rng = np.random.default_rng(9)
    X = (wl.uniform_features_numpy(9, 0, n, F) * row_scale[:, None]).astype(np.float32)
    Wn, Ws = (rng.uniform(-0.125, 0.125, (F, F)).astype(np.float32) for _ in range(2))
    plan = G.groot_spmm_plan(g, 32)
    G.groot_plan_upload(plan, F)
    dev = lambda a: torch_cuda.from_numpy(a).cuda()
    H = torch_cuda.full((n, F), float("nan"), device="cuda")
    G.groot_sage_layer_forward(plan, dev(X), dev(Wn), dev(Ws), None, False, H, F)
    torch_cuda.cuda.synchronize()
    want, A, S = oracle.sage_layer_f64(rowptr, col, val, X, Wn, Ws, None, False)
    a64 = lambda a: np.abs(a.astype(np.float64))
    scale = np.abs(A) @ a64(Wn) + a64(X) @ a64(Ws)
    tol = layer_tolerance(S, scale, a64(Wn), floor=0.0)          # purely relative: no absolute floor
    err = np.abs(H.cpu().numpy().astype(np.float64) - want)
    assert np.isfinite(err).all() and (err <= tol).all(), f"max err/tol {np.max(err / np.maximum(tol, 1e-300))}"


def test_fused_sage_layer_on_csr_graph_with_mean_weights(torch_cuda, uniform_detect):
    """A graph given as CSR whose weights are 1/row length: with the detection the layer runs as self-contained
    wavefronts (rows of up to 2,048 entries take its plain path), without it as the kernel for explicit weights."""
    s = wl.stress_graph(12, 1 << 14, window=512, dmin=64, dmax=2048)
    g = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
    _sage_check(torch_cuda, g, s.rowptr, s.col, s.val, 32, s.n, 6, True, True, "sage csr mean")
    if uniform_detect:
        _sage_check(torch_cuda, g, s.rowptr, s.col, s.val, 32, s.n, 7, False, False, "sage csr mean F=32", F=32)


def test_fused_sage_layer_explicit_weights_and_errors(torch_cuda, sage_variant):
    torch = torch_cuda
    s = wl.stress_graph(11, 1 << 14, window=512, dmin=64, dmax=2048)
    s.val[:] = np.random.default_rng(3).uniform(0.01, 0.5, s.val.shape[0]).astype(np.float32)   # not 1 / row length
    g = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
    _sage_check(torch, g, s.rowptr, s.col, s.val, 32, s.n, 5, True, True, "sage stress")
    plan = G.groot_spmm_plan(g, 32)
    z = lambda *shape: torch.zeros(*shape, device="cuda")
    with pytest.raises(G.GrootError):                       # not uploaded
        G.groot_sage_layer_forward(plan, z(s.n, 64), z(64, 64), z(64, 64), None, True, z(s.n, 64), 64)
    G.groot_plan_upload(plan, 64)
    with pytest.raises(G.GrootError):                       # explicit weights: only F = 64
        G.groot_sage_layer_forward(plan, z(s.n, 32), z(32, 32), z(32, 32), None, True, z(s.n, 32), 32)
    with pytest.raises(G.GrootError):                       # never F = 16
        G.groot_sage_layer_forward(plan, z(s.n, 16), z(16, 16), z(16, 16), None, True, z(s.n, 16), 16)
    x = z(s.n, 64)
    with pytest.raises(G.GrootError):                       # in place
        G.groot_sage_layer_forward(plan, x, z(64, 64), z(64, 64), None, True, x, 64)


def test_tuning_knobs_do_not_change_results(torch_cuda):
    aig, g, (rowptr, col, val, pol) = _aig_case(64, 2)
    X = wl.uniform_features_numpy(8, 0, 2 * aig.num_nodes, 64)
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    try:
        for remap in (0, 1):
            for chunk in (64, 4096):
                G.groot_set_tuning("xcd_remap", remap)
                G.groot_set_tuning("hd_chunk", chunk)
                Y, _, _, _ = _run(torch_cuda, g, 12, X)
                assert_close_to_oracle(Y, Y64, S, f"remap={remap} chunk={chunk}")
        G.groot_set_tuning("xcd_remap", 1)
        G.groot_set_tuning("hd_chunk", 512)
        for compress in (0, 2):
            for depth in (0, 5, 6, 7, 8):
                G.groot_set_tuning("csr_compress", compress)
                G.groot_set_tuning("pipe_depth", depth)
                Y, plan, _, _ = _run(torch_cuda, g, 12, X)
                if G.groot_plan_query(plan, "ld_pipelined"):
                    assert G.groot_plan_query(plan, "csr_compressed") == (compress == 2)
                    assert G.groot_plan_query(plan, "pipe_depth") == (depth or 5)
                assert_close_to_oracle(Y, Y64, S, f"compress={compress} depth={depth}")
    finally:
        G.groot_set_tuning("xcd_remap", 1)
        G.groot_set_tuning("hd_chunk", 512)
        G.groot_set_tuning("csr_compress", 1)
        G.groot_set_tuning("pipe_depth", 0)


def test_phases_cover_disjoint_rows(torch_cuda):
    torch = torch_cuda
    aig, g, (rowptr, col, val, pol) = _aig_case(32, 1)
    n, F = aig.num_nodes, 32
    plan = G.groot_spmm_plan(g, 16)
    G.groot_plan_upload(plan, F)
    pv = G.groot_plan_view(plan)
    X = wl.uniform_features(2, 0, n, F, device="cuda")
    Y = torch.full((n, F), float("nan"), device="cuda")
    G.groot_spmm_execute_phases(plan, X, Y, F, G.GROOT_PHASE_LD)
    torch.cuda.synchronize()
    written = ~torch.isnan(Y).any(dim=1).cpu().numpy()
    assert np.array_equal(written, pv["row_class"] == 0)
    G.groot_spmm_execute_phases(plan, X, Y, F, G.GROOT_PHASE_HD | G.GROOT_PHASE_FINISH)
    torch.cuda.synchronize()
    Y64, S = oracle.spmm_f64(rowptr, col, val, X.cpu().numpy())
    assert_close_to_oracle(Y.cpu().numpy(), Y64, S, "phases")
    # F larger than the uploaded maximum is refused
    with pytest.raises(G.GrootError):
        G.groot_spmm_execute(plan, torch.zeros(n, 64, device="cuda"), torch.zeros(n, 64, device="cuda"), 64)
    with pytest.raises(G.GrootError):      # overlap
        G.groot_spmm_execute(plan, X, X, F)


def test_execute_on_side_stream(torch_cuda):
    torch = torch_cuda
    aig, g, (rowptr, col, val, pol) = _aig_case(48, 1)
    F = 64
    plan = G.groot_spmm_plan(g, 32)
    G.groot_plan_upload(plan, F)
    X = wl.uniform_features(5, 0, aig.num_nodes, F, device="cuda")
    Y = torch.empty_like(X)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        G.groot_spmm_execute(plan, X, Y, F)          # picks up the current (side) stream
    side.synchronize()
    Y64, S = oracle.spmm_f64(rowptr, col, val, X.cpu().numpy())
    assert_close_to_oracle(Y.cpu().numpy(), Y64, S, "side stream")


@pytest.mark.parametrize("n,batch,P,T,F", [(32, 2, 4, 32, 64), (48, 1, 5, 8, 32), (24, 3, 2, 200, 20)])
def test_partitioned_mode_owned_rows_written_in_place(torch_cuda, n, batch, P, T, F):
    """groot_spmm_execute_rows on every re-grown part (first n_owned local rows, written at their global
    ids) fills the full result without computing boundary rows or copying: every element against the
    oracle on the full graph (every row is owned by exactly one part), and nothing else is written."""
    torch = torch_cuda
    aig, g, (rowptr, col, val, pol) = _aig_case(n, batch)
    N = batch * aig.num_nodes
    X_np = wl.uniform_features_numpy(16, 0, N, F)
    X = torch.from_numpy(X_np).cuda()
    guard = 2
    buf = torch.full((N + 2 * guard, F), float("nan"), device="cuda")
    buf[:guard] = 555.0
    buf[N + guard:] = 555.0
    Y = buf[guard:N + guard]
    parts = G.groot_partition_regrow(g, P)
    for p in range(P):
        pv = G.groot_parts_view(parts, p)
        ids = torch.from_numpy(pv["global_id"].copy()).cuda()
        Xp = torch.empty((ids.shape[0], F), device="cuda")
        G.groot_rows_gather(ids, X, Xp, F)
        plan = G.groot_spmm_plan(pv["sub"], T)
        G.groot_plan_upload(plan, F)
        G.groot_spmm_execute_rows(plan, Xp, Y, F, pv["n_owned"], ids)
        torch.cuda.synchronize()
    out = buf.cpu().numpy()
    assert (out[:guard] == 555.0).all() and (out[N + guard:] == 555.0).all(), "wrote outside Y"
    Y64, S = oracle.spmm_f64(rowptr, col, val, X_np)
    assert_close_to_oracle(out[guard:N + guard], Y64, S, f"owned rows in place, P={P} T={T} F={F}")


def test_execute_rows_prefix_without_map_and_errors(torch_cuda):
    torch = torch_cuda
    aig, g, (rowptr, col, val, pol) = _aig_case(40, 1)
    N, F = aig.num_nodes, 64
    X_np = wl.uniform_features_numpy(17, 0, N, F)
    X = torch.from_numpy(X_np).cuda()
    plan = G.groot_spmm_plan(g, 16)
    G.groot_plan_upload(plan, F)
    Y64, S = oracle.spmm_f64(rowptr, col, val, X_np)
    for n_rows in (0, 1, 37, 300, N - 1, N):            # 37 < 2n: cuts through the high-degree input rows
        Y = torch.full((N, F), -3.0, device="cuda")
        G.groot_spmm_execute_rows(plan, X, Y, F, n_rows)
        torch.cuda.synchronize()
        out = Y.cpu().numpy()
        assert (out[n_rows:] == -3.0).all(), f"n_rows={n_rows}: wrote past the requested rows"
        if n_rows:
            assert_close_to_oracle(out[:n_rows], Y64[:n_rows], S[:n_rows], f"prefix of {n_rows} rows")
    with pytest.raises(ValueError):            # the binding: Y would be too short
        G.groot_spmm_execute_rows(plan, X, torch.empty_like(X), F, N + 1)
    with pytest.raises(G.GrootError):          # the library: more rows than the graph has
        G.groot_spmm_execute_rows(plan, X, torch.empty((N + 1, F), device="cuda"), F, N + 1)
    with pytest.raises(ValueError):            # a feature matrix with fewer rows than the graph
        G.groot_spmm_execute(plan, X[:N - 1], torch.empty_like(X), F)
    with pytest.raises(TypeError):
        G.groot_spmm_execute(plan, X.double(), torch.empty_like(X), F)
    with pytest.raises(G.GrootError):
        G.groot_spmm_execute_rows(plan, X, torch.empty_like(X), F, -1)


def test_execute_and_fused_layer_replay_from_a_hip_graph(torch_cuda):
    """The execute calls only enqueue kernels (no allocation, no synchronisation, no memset), so a
    two-layer forward pass can be captured into a HIP graph once and replayed: every replay, with new
    inputs written into the captured buffers and eager work in between, must equal the eager result."""
    torch = torch_cuda
    aig, g, (rowptr, col, val, pol) = _aig_case(40, 2)
    n, F = 2 * aig.num_nodes, 64
    plan = G.groot_spmm_plan(g, 16)
    G.groot_plan_upload(plan, F)
    rng = np.random.default_rng(9)
    Wn, Ws = (torch.from_numpy(rng.uniform(-0.125, 0.125, (F, F)).astype(np.float32)).cuda() for _ in range(2))
    X = torch.zeros((n, F), device="cuda")
    A, H, Y = torch.empty_like(X), torch.empty_like(X), torch.empty_like(X)

    def forward():
        G.groot_spmm_execute(plan, X, A, F)                              # plain aggregation
        G.groot_sage_layer_forward(plan, A, Wn, Ws, None, True, H, F)    # fused layer on top of it
        G.groot_spmm_execute(plan, H, Y, F)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        X.copy_(wl.uniform_features(70, 0, n, F, device="cuda"))
        forward()                                                        # warm-up outside the capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        forward()
    for seed in (71, 72, 73):
        X.copy_(wl.uniform_features(seed, 0, n, F, device="cuda"))
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        replayed = Y.clone()
        Y.fill_(float("nan"))
        forward()                                                        # eager, same buffers
        torch.cuda.synchronize()
        assert torch.equal(replayed, Y), f"replay with seed {seed} differs from the eager run"
        Y64, S = oracle.spmm_f64(rowptr, col, val, H.cpu().numpy())
        assert_close_to_oracle(replayed.cpu().numpy(), Y64, S, f"graph replay, seed {seed}")


@pytest.mark.parametrize("n,batch,P,regrow", [(32, 2, 4, 1), (64, 1, 16, 1), (32, 1, 3, 0)])
def test_partitioned_mode_scatters_back_to_full_result(torch_cuda, n, batch, P, regrow):
    """rows_gather -> per-part SpMM -> rows_scatter reproduces the full-graph
    oracle on every owned row (with re-growth); without re-growth it equals the
    oracle evaluated on the induced sub-graphs."""
    torch = torch_cuda
    aig, g, (rowptr, col, val, pol) = _aig_case(n, batch)
    N, F = batch * aig.num_nodes, 64
    X_np = wl.uniform_features_numpy(6, 0, N, F)
    X = torch.from_numpy(X_np).cuda()
    Y = torch.full((N, F), float("nan"), device="cuda")
    parts = G.groot_partition_regrow(g, P, None, G.GROOT_REGROW if regrow else 0)
    part_of = oracle.part_of_default(N, aig.num_nodes, P)
    Y64 = np.empty((N, F))
    S = np.empty((N, F))
    for p in range(P):
        pv = G.groot_parts_view(parts, p)
        ids = torch.from_numpy(pv["global_id"].copy()).cuda()
        n_loc = ids.shape[0]
        Xp = torch.empty((n_loc, F), device="cuda")
        Yp = torch.empty((n_loc, F), device="cuda")
        G.groot_rows_gather(ids, X, Xp, F)
        plan = G.groot_spmm_plan(pv["sub"], 32)
        G.groot_plan_upload(plan, F)
        G.groot_spmm_execute(plan, Xp, Yp, F)
        G.groot_rows_scatter(ids[:pv["n_owned"]], Yp, Y, F)
        torch.cuda.synchronize()
        assert np.array_equal(Xp.cpu().numpy(), X_np[pv["global_id"]])
        if not regrow:
            want = oracle.regrow_part(rowptr, col, val, part_of, p, 0, 1)
            yp, sp = oracle.spmm_f64(want["rowptr"], want["col"], want["val"], X_np[want["global_id"]])
            Y64[want["global_id"]] = yp
            S[want["global_id"]] = sp
    if regrow:
        Y64, S = oracle.spmm_f64(rowptr, col, val, X_np)
    assert_close_to_oracle(Y.cpu().numpy(), Y64, S, "partitioned")


@pytest.mark.parametrize("matrices,F", [(5.0, 64), (2.25, 32), (3.5, 20)])
def test_feature_placement_returns_a_usable_pair(torch_cuda, matrices, F):
    """groot_feature_placement measures; whatever pair of offsets it returns must be inside the arena, aligned, not
    overlapping, and the aggregation computed there must match the oracle (the arena's contents are not kept)."""
    torch = torch_cuda
    aig, g, (rowptr, col, val, pol) = _aig_case(48, 2)
    n = 2 * aig.num_nodes
    plan = G.groot_spmm_plan(g, 32)
    G.groot_plan_upload(plan, 64)
    size = n * F * 4
    quarter = max(4096, size // 4 // 4096 * 4096)
    arena_floats = int(matrices * n * F) + 4 * quarter // 4
    arena = torch.full((arena_floats,), float("nan"), dtype=torch.float32, device="cuda")
    place = G.groot_feature_placement(plan, arena, F)
    ox, oy = place["x_offset"], place["y_offset"]
    assert ox % quarter == 0 and oy % quarter == 0 and abs(ox - oy) >= size
    assert max(ox, oy) + size <= arena.numel() * 4
    assert place["best_ms"] > 0 and place["first_ms"] >= place["best_ms"]
    X_np = wl.uniform_features_numpy(33, 0, n, F)
    X = arena[ox // 4:ox // 4 + n * F].view(n, F)
    Y = arena[oy // 4:oy // 4 + n * F].view(n, F)
    X.copy_(torch.from_numpy(X_np))
    G.groot_spmm_execute(plan, X, Y, F)
    torch.cuda.synchronize()
    Y64, S = oracle.spmm_f64(rowptr, col, val, X_np)
    assert_close_to_oracle(Y.cpu().numpy(), Y64, S, f"placed at {ox}, {oy}")
    # errors: an arena that does not hold two matrices, a plan that is not uploaded
    with pytest.raises(G.GrootError):
        G.groot_feature_placement(plan, arena[: n * F + n * F // 2], F)
    with pytest.raises(G.GrootError):
        G.groot_feature_placement(G.groot_spmm_plan(g, 32), arena, F)


@pytest.mark.parametrize("F", [4, 12, 32, 60, 128, 260, 512])
@pytest.mark.parametrize("explicit,chunk", [(False, 512), (True, 512), (False, 1300)])
def test_lengths_of_high_degree_pieces(torch_cuda, F, explicit, chunk):
    """Pieces whose quarters, rounds of eight gathers and runs of 128 entries end in every way: rows of a few entries to
    several pieces, and pieces longer than what is staged at a time (the hd_chunk knob)."""
    lengths = [1, 2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257, 509, 511, 512, 513, 516, 1024, 1025, 1300, 1301]
    n, rng = 1400, np.random.default_rng(F)
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in lengths] + [np.array([i]) for i in range(len(lengths), n)]
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    col = np.concatenate(cols).astype(np.int32)
    length = np.diff(rowptr)
    val = rng.uniform(-1, 1, col.size).astype(np.float32) if explicit else np.repeat(np.float32(1) / length.astype(np.float32), length)
    G.groot_set_tuning("hd_chunk", chunk)
    try:
        X = wl.uniform_features_numpy(90 + F, 0, n, F)
        Y, plan, _, _ = _run(torch_cuda, G.groot_graph_from_csr(rowptr, col, val), 2, X)
    finally:
        G.groot_set_tuning("hd_chunk", 512)
    assert G.groot_plan_view(plan)["n_hd"] == len(lengths) - 1
    Y64, S = oracle.spmm_f64(rowptr, col, val, X)
    assert_close_to_oracle(Y, Y64, S, f"piece lengths F={F} explicit={explicit} chunk={chunk}")


@pytest.mark.parametrize("F,depth,explicit", [(32, 5, False), (64, 5, True), (100, 5, False), (128, 7, False), (200, 5, True),
                                              (252, 8, False), (36, 5, False), (72, 5, True), (136, 5, False), (136, 6, False)])
def test_compact_matrix_where_it_is_read(torch_cuda, F, depth, explicit):
    """The compact matrix against the plain arrays on either side of the size of X from which it is read: the same sums in the
    same order, so the same bits.  Rows of 1 to depth entries near the row or among the high-degree rows, a few longer ones,
    a few with an entry that no code expresses, a high-degree row count that is no multiple of four, a ragged last tile."""
    line = (192 << 20) if depth == 5 else (1 << 30)
    rng = np.random.default_rng(F)
    for n in ((line - 1) // (4 * F), -(-line // (4 * F)) + 1):
        length = rng.integers(max(1, depth - 1), depth + 1, n)
        hot = np.sort(16000 + rng.choice(n - 32000, 1021, replace=False))
        length[rng.choice(n, n // 400, replace=False)] = depth + 2
        length[hot] = 60
        row = np.repeat(np.arange(n), length)
        col = np.clip(row + rng.integers(-16000, 16001, row.size), 0, n - 1)
        pick = rng.random(row.size)
        col = np.where(pick < 0.2, hot[rng.integers(0, hot.size, row.size)], col)
        col = np.where(pick > 0.9999, rng.integers(0, n, row.size), col)
        row, col = np.divmod(np.unique(row * n + col), n)        # ascending, no column twice in a row
        length = np.bincount(row, minlength=n)
        rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
        col = col.astype(np.int32)
        val = rng.uniform(-1, 1, col.size).astype(np.float32) if explicit else np.repeat(
            np.float32(1) / np.maximum(length, 1).astype(np.float32), length)
        g = G.groot_graph_from_csr(rowptr, col, val)
        X = torch_cuda.empty((n, F), device="cuda").uniform_(-1, 1)
        out = []
        for compress in (1, 0):
            G.groot_set_tuning("csr_compress", compress)
            G.groot_set_tuning("pipe_depth", depth)
            try:
                plan = G.groot_spmm_plan(g, 32)
                G.groot_plan_upload(plan, F)
            finally:
                G.groot_set_tuning("csr_compress", 1)
                G.groot_set_tuning("pipe_depth", 0)
            if G.groot_plan_query(plan, "ld_pipelined"):
                assert G.groot_plan_query(plan, "csr_compressed") == (compress and 4 * F * n >= line)   # not built for no reader
                if compress:
                    entries = int(rowptr[-1]) - G.groot_plan_query(plan, "nnz_hd")
                    weights = 4 if explicit else 0
                    read = 4 * (n + 1) + (2 + weights) * entries if 4 * F * n >= line else 8 * (n + 1) + (4 + weights) * entries
                    assert G.groot_plan_query(plan, "csr_bytes_ld") == read
            Y = torch_cuda.full((n, F), float("nan"), device="cuda")
            G.groot_spmm_execute(plan, X, Y, F)
            out.append(Y)
        assert torch_cuda.equal(out[0], out[1]), f"F={F} n={n}"


def _dense_rows_graph(n, n_dense, share, rng):
    """n_dense rows with a share of all columns each, a few of 40 entries, the others short; columns ascending, weights
    1 / row length"""
    length = rng.integers(1, 5, n)
    dense = rng.choice(n, n_dense, replace=False)
    length[rng.choice(n, 20, replace=False)] = 40
    length[dense] = int(share * n)
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in length]
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    return rowptr, np.concatenate(cols).astype(np.int32), np.repeat(np.float32(1) / length.astype(np.float32), length), dense


@pytest.mark.parametrize("n,n_dense,want,widths", [(3001, 10, 0, [64]), (20011, 130, 128, [64, 100, 132]), (30016, 33, 33, [140, 260]),
                                                   (40001, 16, 16, [212, 512]), (50020, 300, 300, [12, 64]),
                                                   (90049, 200, 192, [8, 12, 32, 36])])
@pytest.mark.parametrize("ones", [False, True])
def test_high_degree_rows_as_a_dense_product(torch_cuda, n, n_dense, want, widths, ones):
    """Rows that hold a quarter of all columns: 16, 32 or 64 at a time, a last tile that is not full, columns that are no
    multiple of 32 or 128, every kind of feature tile, from 2^25 entries times features on."""
    rng = np.random.default_rng(n + n_dense)
    rowptr, col, val, dense = _dense_rows_graph(n, n_dense, 0.25, rng)
    if ones:
        val = np.ones_like(val)
    g = G.groot_graph_from_csr(rowptr, col, val)
    for F in widths:
        X = wl.uniform_features_numpy(n + F, 0, n, F)
        Y, plan, _, _ = _run(torch_cuda, g, 32, X)
        assert G.groot_plan_query(plan, "dense_rows") == want
        assert not want or want * (n // 4) * F >= 2 ** 25
        assert G.groot_plan_query(plan, "weight_mode") == (0 if ones else 1)
        Y64, S = oracle.spmm_f64(rowptr, col, val, X)
        assert_close_to_oracle(Y, Y64, S, f"dense rows n={n} {n_dense} F={F}")


def test_dense_product_phase_by_phase_and_from_a_hip_graph(torch_cuda):
    """The phases one by one, and replays of a captured call on new inputs with eager work between them, give the bits of the
    whole eager call; each phase writes the rows that it is said to."""
    torch = torch_cuda
    n, F = 50020, 64
    rowptr, col, val, dense = _dense_rows_graph(n, 230, 0.25, np.random.default_rng(4))
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == 230 and 230 * (n // 4) * F >= 2 ** 25
    X = wl.uniform_features(21, 0, n, F, device="cuda")
    whole, steps = torch.full((n, F), float("nan"), device="cuda"), torch.full((n, F), float("nan"), device="cuda")
    G.groot_spmm_execute(plan, X, whole, F)
    low = torch.from_numpy(np.diff(rowptr) < 32).cuda()
    G.groot_spmm_execute_phases(plan, X, steps, F, G.GROOT_PHASE_LD)
    assert torch.equal(~torch.isnan(steps).any(dim=1), low)
    for phase in (G.GROOT_PHASE_HD, G.GROOT_PHASE_FINISH):
        G.groot_spmm_execute_phases(plan, X, steps, F, phase)
        assert torch.equal(steps[low], whole[low])
    assert torch.equal(steps, whole)
    Y = torch.empty_like(X)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        G.groot_spmm_execute(plan, X, Y, F)
    for seed in (22, 23, 24):
        X.copy_(wl.uniform_features(seed, 0, n, F, device="cuda"))
        if seed == 23:
            X[n // 2, 3] = float("inf")                      # the other sweeps of the dense product, too
        Y.fill_(float("nan"))
        G.groot_spmm_execute(plan, X, whole, F)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, whole), f"replay with seed {seed}"
    Y64, S = oracle.spmm_f64(rowptr, col, val, X.cpu().numpy())
    assert_close_to_oracle(Y.cpu().numpy(), Y64, S, "replay")


@pytest.mark.parametrize("n_dense,max_F,said,served", [(500, 12, 500, True), (500, 4, 0, False), (16, 64, 16, False)])
def test_bytes_that_are_said_to_be_read_with_dense_rows(torch_cuda, n_dense, max_F, said, served):
    """"csr_bytes_hd" of a plan whose widest call computes the dense rows from one bit per column, and of one whose calls
    gather them."""
    n = 50020
    rowptr, col, val, dense = _dense_rows_graph(n, n_dense, 0.25, np.random.default_rng(3))
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, max_F)
    assert G.groot_plan_query(plan, "dense_rows") == said
    length = np.diff(rowptr)
    others = np.count_nonzero(length == 40)                  # one piece each
    pieces, nnz_hd = G.groot_plan_query(plan, "hd_pieces"), G.groot_plan_query(plan, "nnz_hd")
    assert pieces == others + n_dense * -(-int(0.25 * n) // 512) and nnz_hd == length[length >= 32].sum()
    mask = -(-(-(-n // 32)) // 4) * 512 * 4 * 4              # 128 columns of a row in 16 bytes, rows in tiles of 64
    read = 4 * 40 * others + 24 * (others + n_dense) + mask if served else 4 * nnz_hd + 24 * pieces
    assert G.groot_plan_query(plan, "csr_bytes_hd") == read
    assert G.groot_plan_query(plan, "csr_bytes") == read + G.groot_plan_query(plan, "csr_bytes_ld")


def test_dense_product_with_numbers_that_are_not_finite(torch_cuda):
    """An infinity or a NaN in X reaches the rows that have its column and no others."""
    n, F = 30020, 100
    rng = np.random.default_rng(5)
    rowptr, col, val, dense = _dense_rows_graph(n, 64, 0.2, rng)
    g = G.groot_graph_from_csr(rowptr, col, val)
    X = wl.uniform_features_numpy(6, 0, n, F)
    X[17, 3], X[n - 1, 35], X[2000, 8] = np.inf, -np.inf, np.nan
    X[31, 20], X[32, 20] = 3e38, 3e38                    # finite, their sum is not
    plan = G.groot_spmm_plan(g, 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == 64
    Xd = torch_cuda.from_numpy(X).cuda()
    Y = torch_cuda.empty_like(Xd)
    G.groot_spmm_execute(plan, Xd, Y, F)
    Y = Y.cpu().numpy()
    row = np.repeat(np.arange(n), np.diff(rowptr))
    for c, f, bad in ((17, 3, lambda y: np.isposinf(y)), (n - 1, 35, lambda y: np.isneginf(y)), (2000, 8, np.isnan)):
        has = np.zeros(n, bool)
        has[row[col == c]] = True
        assert has[dense].any() and not has[dense].all()
        assert bad(Y[has, f]).all() and np.isfinite(Y[~has, f]).all(), (c, f)
    keep = np.array([k for k in range(F) if k not in (3, 8, 20, 35)])
    Y64, S = oracle.spmm_f64(rowptr, col, val, X[:, keep])
    assert_close_to_oracle(Y[:, keep], Y64, S, "the other features")


@pytest.mark.parametrize("F,depth,explicit", [(36, 5, False), (40, 5, True), (48, 5, False), (72, 5, True), (80, 5, False), (132, 5, False),
                                              (164, 5, True), (176, 5, False), (36, 6, True), (44, 7, False), (72, 8, False),
                                              (96, 6, False), (136, 7, True), (148, 8, False)])
def test_rows_that_share_their_lanes(torch_cuda, F, depth, explicit):
    """Widths at which a sweep deals a tile's float4 out to all lanes (half to three quarters of L lanes per row otherwise): a
    ragged last tile, empty rows, masked rows first and last in a tile, on either side of 64 MB of X.  Against the plain
    kernel, which adds a row's entries in the same order."""
    rng = np.random.default_rng(F + depth)
    line = (64 << 20) // (4 * F)
    for n in ((line - 1, line + 38) if depth == 5 else (1, 47, 9001)):
        length = rng.integers(max(0, depth - 5), depth + 1, n)
        length[rng.choice(n, n // 30, replace=False)] = depth + 3
        length[rng.choice(n, n // 300, replace=False)] = 40
        length = np.minimum(length, n)
        row = np.repeat(np.arange(n), length)
        col = (row + rng.integers(-300, 301, row.size)) % n
        row, col = np.divmod(np.unique(row * n + col), n)
        length = np.bincount(row, minlength=n)
        rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
        val = rng.uniform(-1, 1, col.size).astype(np.float32) if explicit else np.repeat(
            np.float32(1) / np.maximum(length, 1).astype(np.float32), length)
        g = G.groot_graph_from_csr(rowptr, col.astype(np.int32), val)
        X = torch_cuda.empty((n, F), device="cuda").uniform_(-1, 1)
        out = []
        for pipeline in (1, 0):
            G.groot_set_tuning("ld_pipeline", pipeline)
            G.groot_set_tuning("pipe_depth", depth)
            try:
                plan = G.groot_spmm_plan(g, 32)
                G.groot_plan_upload(plan, F)
            finally:
                G.groot_set_tuning("ld_pipeline", -1)
                G.groot_set_tuning("pipe_depth", 0)
            buf = torch_cuda.full((n + 6, F), float("nan"), device="cuda")
            G.groot_spmm_execute(plan, X, buf[3:n + 3], F)
            assert torch_cuda.isnan(buf[:3]).all() and torch_cuda.isnan(buf[n + 3:]).all(), "wrote outside Y"
            out.append(buf[3:n + 3])
        assert torch_cuda.equal(out[0], out[1]), f"F={F} depth={depth} n={n}"


@pytest.mark.parametrize("F,depth,T,weights", [(36, 5, 32, "mean"), (44, 5, 4, "explicit"), (72, 5, 32, "ones"), (80, 5, 32, "mean"),
                                               (136, 5, 32, "explicit"), (176, 5, 5, "ones"), (36, 6, 32, "explicit"), (48, 7, 5, "mean"),
                                               (40, 8, 32, "ones"), (72, 6, 32, "mean"), (96, 7, 32, "explicit"), (76, 8, 6, "ones"),
                                               (132, 6, 32, "ones"), (148, 7, 32, "mean"), (136, 8, 32, "explicit")])
def test_rows_that_share_their_lanes_on_the_compact_matrix(torch_cuda, F, depth, T, weights):
    """The same widths with the matrix as 2-byte codes: entries near the row, at either end of what a code reaches, among the
    high-degree rows and beyond any code (a row with such an entry is masked, wherever it lies in a tile), empty rows, rows longer
    than the slots, a threshold below them, a ragged last tile.  Against the plain kernel, which adds in the same order."""
    rng = np.random.default_rng(F * depth)
    n = (64 << 20) // (4 * F) + 38 if depth == 5 else 40013
    length = rng.integers(max(0, min(depth, T - 1) - 5), min(depth, T - 1) + 1, n)
    length[rng.choice(n, n // 200, replace=False)] = min(depth, T) + 3
    length[rng.choice(n, n // 900, replace=False)] = min(depth, T)
    hot = np.sort(rng.choice(n, n // 300, replace=False))
    length[hot] = 40
    row = np.repeat(np.arange(n), length)
    pick = rng.random(row.size)
    col = row + rng.integers(-300, 301, row.size)
    col = np.where(pick < 0.02, row - 16384, np.where(pick < 0.04, row + 16383, col))
    col = np.where((col < 0) | (col >= n), row, col)
    col = np.where(pick > 0.8, hot[rng.integers(0, hot.size, row.size)], col)
    col = np.where(pick > 0.9995, rng.integers(0, n, row.size), col)
    row, col = np.divmod(np.unique(row * n + col), n)
    length = np.bincount(row, minlength=n)
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    val = {"mean": np.repeat(np.float32(1) / np.maximum(length, 1).astype(np.float32), length), "ones": np.ones(col.size, np.float32),
           "explicit": rng.uniform(-1, 1, col.size).astype(np.float32)}[weights]
    g = G.groot_graph_from_csr(rowptr, col.astype(np.int32), val)
    X = torch_cuda.empty((n, F), device="cuda").uniform_(-1, 1)
    out = []
    for pipeline in (1, 0):
        for name, value in (("ld_pipeline", pipeline), ("pipe_depth", depth), ("csr_compress", 2)):
            G.groot_set_tuning(name, value)
        try:
            plan = G.groot_spmm_plan(g, T)
            G.groot_plan_upload(plan, F)
        finally:
            for name, value in (("ld_pipeline", -1), ("pipe_depth", 0), ("csr_compress", 1)):
                G.groot_set_tuning(name, value)
        if pipeline:
            assert G.groot_plan_query(plan, "csr_compressed") == 1 and 0 < G.groot_plan_query(plan, "uncoded_rows") < n // 50
            assert G.groot_plan_query(plan, "weight_mode") == {"ones": 0, "mean": 1, "explicit": 2}[weights]
        buf = torch_cuda.full((n + 6, F), float("nan"), device="cuda")
        G.groot_spmm_execute(plan, X, buf[3:n + 3], F)
        assert torch_cuda.isnan(buf[:3]).all() and torch_cuda.isnan(buf[n + 3:]).all(), "wrote outside Y"
        out.append(buf[3:n + 3])
    assert torch_cuda.equal(out[0], out[1])


def test_dense_rows_of_a_plan_whose_columns_are_renamed(torch_cuda):
    """Once a plan's columns name rows of a larger matrix, its dense rows are gathered like the others: the bits name the
    plan's own rows."""
    n, n_global, F = 20011, 23000, 64
    rng = np.random.default_rng(8)
    rowptr, col, val, dense = _dense_rows_graph(n, 128, 0.25, rng)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == 128
    ids = np.sort(rng.choice(n_global, n, replace=False)).astype(np.int64)
    ids_dev = torch_cuda.from_numpy(ids).cuda()
    G.groot_plan_use_global_columns(plan, ids_dev, n_global)
    assert G.groot_plan_query(plan, "dense_rows") == 0
    X = wl.uniform_features_numpy(9, 0, n_global, F)
    Xd = torch_cuda.from_numpy(X).cuda()
    Y64, S = oracle.spmm_f64(rowptr, col, val, X[ids])
    Y = torch_cuda.full((n, F), float("nan"), device="cuda")
    G.groot_spmm_execute(plan, Xd, Y, F)
    assert_close_to_oracle(Y.cpu().numpy(), Y64, S, "renamed columns")
    Y = torch_cuda.full((n, F), float("nan"), device="cuda")
    G.groot_spmm_execute_rows(plan, Xd, Y, F, n)
    assert_close_to_oracle(Y.cpu().numpy(), Y64, S, "renamed columns, rows")


def _dense_rows_of(rowptr, col, val, rows):
    """the rows as a matrix of their own"""
    length = np.diff(rowptr)[rows]
    pick = np.concatenate([np.arange(rowptr[r], rowptr[r + 1]) for r in rows])
    return np.concatenate([[0], np.cumsum(length)]).astype(np.int64), col[pick], val[pick]


@pytest.mark.parametrize("n,n_dense,share,F", [(20011, 512, 0.25, 128), (65536, 320, 0.25, 256), (65536, 64, 0.5, 512),
                                               (100003, 640, 0.08, 128), (131072, 320, 0.25, 64)])
def test_dense_product_is_no_less_precise_than_the_gathers(torch_cuda, n, n_dense, share, F):
    """The sums of dense rows against fp64, in the 2-norm over all of them, beside the sums that the same rows get by gathers
    (groot_spmm_execute_rows), for inputs that cancel: however many columns there are, no chain of additions grows with them."""
    rng = np.random.default_rng(n + F)
    rowptr, col, val, dense = _dense_rows_graph(n, n_dense, share, rng)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == n_dense and n_dense * int(share * n) * F >= 2 ** 25
    X = wl.uniform_features_numpy(n_dense, 0, n, F)
    Xd = torch_cuda.from_numpy(X).cuda()
    want, _ = oracle.spmm_f64(*_dense_rows_of(rowptr, col, val, dense), X)
    Y = torch_cuda.empty_like(Xd)
    off = []
    for call in (lambda: G.groot_spmm_execute(plan, Xd, Y, F), lambda: G.groot_spmm_execute_rows(plan, Xd, Y, F, n)):
        call()
        off.append(np.linalg.norm(Y.cpu().numpy()[dense].astype(np.float64) - want) / np.linalg.norm(want))
    assert off[0] <= off[1], off


@pytest.mark.parametrize("n,n_dense,share,F", [(20011, 512, 0.25, 128), (65536, 64, 0.5, 512), (100003, 448, 0.08, 128)])
@pytest.mark.parametrize("kind", ["exp(4 N)", "2^U(-20, 0)", "2^U(-40, 0)", "one in a thousand", "one in a stretch"])
def test_dense_product_of_positive_numbers_over_many_binades(torch_cuda, n, n_dense, share, F, kind):
    """Features of one sign and of very different size, small ones of which lose bits beside large ones in a truncating chain of matrix
    instructions, always to the same side: in the 2-norm no further off than the gathers, or than a unit in the last place where a workgroup
    sums 128 or 256 columns, so that there are no long chains."""
    torch = torch_cuda
    rng = np.random.default_rng(n + F)
    dense = np.sort(rng.choice(n, n_dense, replace=False))
    graph = _spread_dense_rows_graph(n, dense, int(share * n), rng)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(*graph), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == n_dense and n_dense * int(share * n) * F >= 2 ** 25
    X = torch.empty((n, F), device="cuda").uniform_(0, 1, generator=torch.Generator(device="cuda").manual_seed(n))
    if kind == "exp(4 N)":
        X = torch.exp(4 * torch.erfinv((2 * X.double() - 1).clamp(-1 + 1e-9, 1 - 1e-9)) * 2 ** 0.5).float()
    elif kind.startswith("2^"):
        X = torch.exp2(X * (-20 if "20" in kind else -40))
    elif kind == "one in a thousand":
        X = (X + 1) * 2.0 ** -15
        X[5::997] = 1
        X[3] = 4
    else:
        X = (X + 1) * 2.0 ** -17
        X[::2048] = 1
    want = torch.stack([X[torch.from_numpy(graph[1][graph[0][r]:graph[0][r + 1]].astype(np.int64)).cuda()].double().mean(0) for r in dense])
    rows, Y, off = torch.from_numpy(dense).cuda(), torch.empty_like(X), []
    for call in (lambda: G.groot_spmm_execute(plan, X, Y, F), lambda: G.groot_spmm_execute_rows(plan, X, Y, F, n)):
        call()
        off.append(((Y[rows].double() - want).norm() / want.norm()).item())
    assert off[0] <= max(off[1], 2.0 ** -23 if n < 2 ** 15 else 0), off


@pytest.mark.parametrize("F,scale", [(64, 8e36), (12, 3e37), (64, 1e-41)])
def test_dense_product_of_very_large_and_very_small_numbers(torch_cuda, F, scale):
    """Rows whose plain sums overflow and whose weighted sums, like the gathers', do not; and numbers below the least normal one,
    where every weighted sum of a few entries is rounded to 2^-149: no further off than the gathers."""
    n, n_dense = 50020, 300
    rowptr, col, val, dense = _dense_rows_graph(n, n_dense, 0.25, np.random.default_rng(6))
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == n_dense and n_dense * (n // 4) * F >= 2 ** 25
    X = (np.random.default_rng(7).uniform(0.5, 1, (n, F)) * scale).astype(np.float32)
    Xd = torch_cuda.from_numpy(X).cuda()
    want, _ = oracle.spmm_f64(*_dense_rows_of(rowptr, col, val, dense), X)
    off = []
    for call in (lambda Y: G.groot_spmm_execute(plan, Xd, Y, F), lambda Y: G.groot_spmm_execute_rows(plan, Xd, Y, F, n)):
        Y = torch_cuda.empty_like(Xd)
        call(Y)
        off.append(np.abs(Y.cpu().numpy()[dense].astype(np.float64) - want))
    if scale > 1:
        assert all((x <= 1e-5 * want).all() for x in off)
    else:
        assert off[0].max() <= off[1].max() and off[0].mean() <= off[1].mean()


def _spread_dense_rows_graph(n, dense, length, rng):
    """The rows `dense` with `length` columns each all over the matrix, one in every stretch of n / length columns; the others with
    their diagonal alone; weights 1 / row length"""
    lengths = np.ones(n, np.int64)
    lengths[dense] = length
    rowptr = np.concatenate([[0], np.cumsum(lengths)])
    col = np.repeat(np.arange(n, dtype=np.int32), lengths)
    first = np.arange(length, dtype=np.int64) * n // length
    room = np.diff(np.append(first, n))
    for r in dense:
        col[rowptr[r]:rowptr[r + 1]] = first + (rng.random(length) * room).astype(np.int64)
    return rowptr, col, np.repeat(np.float32(1) / lengths.astype(np.float32), lengths)


@pytest.mark.parametrize("n,share,F", [(262144, 0.5, 512), (1200000, 0.25, 512)])
def test_dense_product_of_very_large_numbers_over_long_stretches(torch_cuda, n, share, F):
    """8,192 and 37,504 columns that a workgroup sums (in one and in two partial sums): their mean is finite, and so is every partial sum of
    theirs: numbers up to 2 / 32 of the largest float pass in rows of half of the columns, up to 4 / 32 in rows of a quarter."""
    rng = np.random.default_rng(n)
    dense = np.sort(rng.choice(n, 64, replace=False))
    graph = _spread_dense_rows_graph(n, dense, int(share * n), rng)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(*graph), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == 64
    X = torch_cuda.empty((n, F), device="cuda").uniform_(1e37, 2e37)
    Y = torch_cuda.empty_like(X)
    G.groot_spmm_execute(plan, X, Y, F)
    for r in dense[::7]:
        of_row = torch_cuda.from_numpy(graph[1][graph[0][r]:graph[0][r + 1]].astype(np.int64)).cuda()
        want = X[of_row].double().mean(0)
        assert ((Y[r].double() - want).abs() <= 1e-6 * want).all(), r


@pytest.mark.parametrize("n,n_dense,F", [(30011, 96, 68), (300011, 16, 512)])
def test_dense_product_of_subnormal_numbers_with_unit_weights(torch_cuda, n, n_dense, F):
    """Sums of numbers of a few multiples of 2^-149 are exact, from single ones to numbers that are normal again, in workgroups of
    256 and of 9,472 columns."""
    rng = np.random.default_rng(n)
    dense = np.sort(rng.choice(n, n_dense, replace=False))
    rowptr, col, val = _spread_dense_rows_graph(n, dense, n // 4, rng)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, np.ones_like(val)), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == n_dense and G.groot_plan_query(plan, "weight_mode") == 0
    times = torch_cuda.from_numpy(rng.integers(-3, 4, (n, F))).cuda()
    for exp in (-149, -140, -133, -127, -110):
        X = (times.double() * 2.0 ** exp).float()
        Y = torch_cuda.empty_like(X)
        G.groot_spmm_execute(plan, X, Y, F)
        for r in dense[::5]:
            want = times[torch_cuda.from_numpy(col[rowptr[r]:rowptr[r + 1]].astype(np.int64)).cuda()].sum(0)
            assert torch_cuda.equal(Y[r].double() * 2.0 ** 149, want.double() * 2.0 ** (exp + 149)), (exp, r)


@pytest.mark.parametrize("exp", [-118, -110, -107, -104, -96, 102, 104, 106])
def test_dense_product_is_as_precise_at_the_ends_of_the_range(torch_cuda, exp):
    """Numbers whose third piece would be subnormal, and numbers that are partly too large for the scale of the cut: the same sums as of
    numbers around 1, as far as these are not rounded to multiples of 2^-149, or no further off than the gathers."""
    n, F = 20011, 128
    rowptr, col, val, dense = _dense_rows_graph(n, 128, 0.25, np.random.default_rng(15))
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == 128
    X = torch_cuda.from_numpy(wl.uniform_features_numpy(5, 0, n, F)).cuda()
    want = oracle.spmm_f64(*_dense_rows_of(rowptr, col, val, dense), X.cpu().numpy())[0]
    out = [torch_cuda.empty_like(X) for _ in range(3)]
    for Y, scale, call in zip(out, (0, exp, exp), (G.groot_spmm_execute, G.groot_spmm_execute, G.groot_spmm_execute_rows)):
        call(plan, X * 2.0 ** scale, Y, F, *([n] if call is G.groot_spmm_execute_rows else []))
    off = [np.linalg.norm(np.ldexp(Y.cpu().numpy()[dense].astype(np.float64), -s) - want) for Y, s in zip(out, (0, exp, exp))]
    assert off[1] <= (1.001 * off[0] if -112 < exp < 104 else off[2]), off


@pytest.mark.parametrize("how", ["one", "a hundredth", "a stretch", "all"])
@pytest.mark.parametrize("ones", [False, True])
def test_dense_product_gives_infinities_and_nan_like_the_gathers(torch_cuda, how, ones):
    """Any number of infinities and NaN in X, in any order: the same elements are infinite, of the same sign, and NaN as by
    gathers, and the others are as close to them as two orders of summation are."""
    n, F = 40013, 68
    rng = np.random.default_rng(11)
    rowptr, col, val, dense = _dense_rows_graph(n, 96, 0.2, rng)
    if ones:
        val = np.ones_like(val)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == 96
    X = wl.uniform_features_numpy(12, 0, n, F)
    kinds = np.array([np.inf, -np.inf, np.nan], np.float32)
    if how == "one":
        X[n // 2, 7] = -np.inf
    elif how == "a hundredth":                               # of the columns, in a few features
        rows = rng.choice(n, n // 100, replace=False)
        X[rows, rng.integers(0, 9, rows.size)] = kinds[rng.integers(0, 3, rows.size)]
        X[rng.choice(n, 3, replace=False), 20] = np.inf
        X[rng.choice(n, 2, replace=False), 21] = np.inf, -np.inf
    elif how == "a stretch":
        X[5000:5040, 10:30] = np.inf
        X[9000:9900, 40] = -np.inf
    else:
        X[:] = kinds[rng.integers(0, 2, X.shape)]
        X[:, 3], X[:, 4], X[:, 5] = np.inf, -np.inf, np.nan
    Xd = torch_cuda.from_numpy(X).cuda()
    out = []
    for call in (lambda Y: G.groot_spmm_execute(plan, Xd, Y, F), lambda Y: G.groot_spmm_execute_rows(plan, Xd, Y, F, n)):
        Y = torch_cuda.full((n, F), 7.0, device="cuda")
        call(Y)
        out.append(Y.cpu().numpy())
    a, b = out
    assert (np.isnan(a) == np.isnan(b)).all() and (np.isposinf(a) == np.isposinf(b)).all() and (np.isneginf(a) == np.isneginf(b)).all()
    assert how == "all" or np.isfinite(b[dense]).any()
    keep = np.isfinite(b)
    terms, bound = np.where(np.isfinite(X), np.abs(X), 0), np.zeros((n, F))
    bound[dense] = oracle.spmm_f64(*_dense_rows_of(rowptr, col, val, dense), terms.astype(np.float32))[0]
    assert (np.abs(np.where(keep, a, 0) - np.where(keep, b, 0)) <= 2 * tolerance(bound)).all()


def test_one_number_that_is_not_finite_does_not_slow_the_dense_product_down(torch_cuda):
    """Only the stretch of columns that holds it is summed again (a row that was gathered again by a single workgroup took 3.4
    times as long); the rest is allowance for the clock."""
    n, F = 131072, 128
    rng = np.random.default_rng(13)
    rowptr, col, val, _ = _dense_rows_graph(n, 320, 0.25, rng)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    X = torch_cuda.empty((n, F), device="cuda").uniform_(-1, 1)
    Y = torch_cuda.empty_like(X)
    run = lambda: G.groot_spmm_execute(plan, X, Y, F)
    finite = _best_time(torch_cuda, run)
    X[n // 3, 5] = float("nan")
    assert _best_time(torch_cuda, run) < 1.7 * finite


@pytest.mark.parametrize("n,rows,want", [(30016, [(95, 0.25)], 95), (30016, [(95, 0.1)], 95), (30016, [(159, 0.25)], 159),
                                         (30016, [(70, 0.5)], 70), (30016, [(70, 0.1)], 64), (70000, [(4, 0.5)], 4), (70000, [(7, 0.5)], 7),
                                         (70000, [(2, 0.9)], 2), (70000, [(16, 0.25), (60, 0.02)], 64),
                                         (30016, [(64, 0.25), (40, 0.02)], 64), (30016, [(64, 0.3), (8, 0.27)], 72),
                                         (30016, [(64, 0.25), (40, 0.04)], 104), (30016, [(64, 0.25), (33, 0.05)], 97),
                                         (40000, [(40, 0.04)], 40)])
def test_rows_that_are_computed_as_a_dense_product(torch_cuda, n, rows, want):
    """A last tile of rows is taken by the entries that it holds, however few its rows are; so are the only rows."""
    rng = np.random.default_rng(n)
    lengths = np.concatenate([np.full(k, int(share * n)) for k, share in rows])
    dense = np.sort(rng.choice(n, lengths.size, replace=False))
    length = np.ones(n, np.int64)
    length[dense] = lengths
    rowptr = np.concatenate([[0], np.cumsum(length)])
    col = np.repeat(np.arange(n, dtype=np.int32), length)
    for r in dense:
        col[rowptr[r]:rowptr[r + 1]] = np.arange(length[r])
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, np.repeat(np.float32(1) / length.astype(np.float32), length)), 32)
    G.groot_plan_upload(plan, 128)
    assert G.groot_plan_query(plan, "dense_rows") == want


@pytest.mark.parametrize("n,n_dense,F", [(8192, 17, 512), (8193, 17, 512), (8223, 30, 300), (262149, 12, 32), (300015, 40, 100)])
def test_last_columns_and_partial_sums_of_a_few_dense_rows(torch_cuda, n, n_dense, F):
    """A few rows, 128 to 1,024 partial sums each, whose last columns are in a unit of the matrix instruction that ends with or behind the last
    column; X is infinite in the columns before them, which such a unit loads, too, and the rows do not name."""
    dense = np.arange(1, n, n // n_dense)[:n_dense]
    first = n - (n % 32 or 7)
    cols = np.concatenate([np.arange(n // 2, dtype=np.int32), np.arange(first, n, dtype=np.int32)])
    length = np.ones(n, np.int64)
    length[dense] = cols.size
    rowptr = np.concatenate([[0], np.cumsum(length)])
    col = np.repeat(np.arange(n, dtype=np.int32), length)
    for r in dense:
        col[rowptr[r]:rowptr[r + 1]] = cols
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, np.repeat(np.float32(1) / length.astype(np.float32), length)), 32)
    G.groot_plan_upload(plan, F)
    assert G.groot_plan_query(plan, "dense_rows") == n_dense and n_dense * cols.size * F >= 2 ** 25
    X = torch_cuda.empty((n, F), device="cuda").uniform_(-1, 1)
    X[n - 50:first] = float("inf")
    Y = torch_cuda.empty_like(X)
    G.groot_spmm_execute(plan, X, Y, F)
    want = X[torch_cuda.from_numpy(cols.astype(np.int64)).cuda()].double()
    err = (Y[torch_cuda.from_numpy(dense).cuda()].double() - want.mean(0)).abs()
    assert (err <= 2.0 ** -21 * want.abs().mean(0)).all(), err.max()


def test_very_small_numbers_do_not_slow_the_dense_product_down(torch_cuda):
    """They are summed as all others (as exceptions, in a pass of their own, they took twice as long)."""
    n, F = 131072, 128
    rowptr, col, val, _ = _dense_rows_graph(n, 320, 0.25, np.random.default_rng(13))
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    X = torch_cuda.empty((n, F), device="cuda").uniform_(-1, 1)
    Y = torch_cuda.empty_like(X)
    run = lambda: G.groot_spmm_execute(plan, X, Y, F)
    usual = _best_time(torch_cuda, run)
    X *= 2.0 ** -120
    assert _best_time(torch_cuda, run) < 1.3 * usual


@pytest.mark.parametrize("n,n_dense,share,F", [(16384, 64, 0.3, 60), (16385, 100, 0.3, 68), (16511, 192, 0.2, 100), (16512, 256, 0.2, 32),
                                               (20000, 320, 0.2, 96), (20001, 384, 0.2, 64), (20033, 448, 0.1, 128), (9999, 512, 0.2, 160),
                                               (12345, 576, 0.2, 64), (30001, 1100, 0.05, 132), (200001, 32, 0.2, 300),
                                               (200001, 16, 0.2, 512), (540000, 1024, 0.021, 512)])
def test_dense_product_in_tiles_of_every_height(torch_cuda, n, n_dense, share, F):
    """16 to 448 rows to a workgroup and several workgroups' worth, columns that end anywhere in a step of 128, stretches of one step
    and of many, one and two partial sums per stretch, feature tiles of both kinds; features of very small and of subnormal numbers among
    the others.  Against fp64: the pieces are exact, and a chain of four matrix instructions truncates four times, by 2^-23 of its own sum
    each at most, so by 2^-21 of the absolute sum at most; the additions of chains round by 2^-24 of a running sum that cancels.  2^-148
    where the result itself is rounded to multiples of 2^-149."""
    torch = torch_cuda
    rng = np.random.default_rng(n)
    length = np.ones(n, np.int64)
    dense = np.sort(rng.choice(n, n_dense, replace=False))
    length[dense] = int(share * n)
    rowptr = np.concatenate([[0], np.cumsum(length)])
    col = np.repeat(np.arange(n, dtype=np.int32), length)
    for r in dense:
        first = np.sort(rng.choice(n - 1, min(64, length[r]), replace=False))   # a step of the columns apart, from a random place on
        step = max(1, (n - 1) // length[r])
        c = np.unique((first[0] + np.arange(length[r]) * step + rng.integers(0, step, length[r])) % n) if step > 1 else None
        if c is None or c.size != length[r]:
            c = np.sort(rng.permutation(n)[:length[r]])
        col[rowptr[r]:rowptr[r + 1]] = c
    val = np.repeat(np.float32(1) / length.astype(np.float32), length)
    plan = G.groot_spmm_plan(G.groot_graph_from_csr(rowptr, col, val), 32)
    G.groot_plan_upload(plan, F)
    served = G.groot_plan_query(plan, "dense_rows")
    assert served in (n_dense, n_dense // 64 * 64) and served * int(share * n) * F >= 2 ** 24
    X = torch.empty((n, F), device="cuda").uniform_(-1, 1, generator=torch.Generator(device="cuda").manual_seed(n))
    X[:, 1] *= 2.0 ** -112
    X[:, F - 3] *= 2.0 ** -135
    X[::97, F - 1] *= 2.0 ** -130
    Y = torch.full((n, F), float("nan"), device="cuda")
    G.groot_spmm_execute(plan, X, Y, F)
    assert torch.isfinite(Y).all()
    for r in rng.choice(dense, 40):
        x = X[torch.from_numpy(col[rowptr[r]:rowptr[r + 1]].astype(np.int64)).cuda()].double()
        w = float(val[rowptr[r]])
        err = (Y[r].double() - x.sum(0) * w).abs()
        assert (err <= 2.0 ** -21 * w * x.abs().sum(0) + 2.0 ** -148).all(), (r, err.max().item())
