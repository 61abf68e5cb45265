"""Host side of the library against the oracle, bit for bit (no GPU): CSR,
weights, polarity bytes, plan lists, partition outputs, error paths, and the
exported symbol table."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
import workloads as wl
from util import ensure_built

ensure_built()
import paper_2511_18297_amd as G  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "groot.h")).read()
    declared = set(re.findall(r"\b(groot_[a-z_]+)\s*\(", header))
    assert declared == set(G.EXPORTS)
    lib = ctypes.CDLL(G.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name


def test_upload_without_host_memory_is_an_error_and_no_exception(tmp_path):
    """The first allocation of host memory inside groot_plan_upload fails: GROOT_ENOMEM, no exception through the C entry."""
    source, driver = tmp_path / "driver.cpp", tmp_path / "driver"
    source.write_text("""
        #include <cstdio>
        #include <cstdlib>
        #include <new>
        #include "groot.h"
        static thread_local int fail_next = 0;
        void *operator new(std::size_t n)
        {
            if (fail_next) { fail_next = 0; throw std::bad_alloc(); }
            if (void *p = std::malloc(n ? n : 1)) return p;
            throw std::bad_alloc();
        }
        void operator delete(void *p) noexcept { std::free(p); }
        void operator delete(void *p, std::size_t) noexcept { std::free(p); }
        int main()
        {
            const int64_t rowptr[] = {0, 1, 2};
            const int32_t col[] = {0, 1};
            const float val[] = {1.f, 1.f};
            groot_graph *g = nullptr;
            groot_plan *plan = nullptr;
            if (groot_graph_from_csr(2, rowptr, col, val, &g) || groot_spmm_plan(g, 32, &plan)) return 1;
            fail_next = 1;
            const int st = groot_plan_upload(plan, 64);
            std::printf("%d %d %s", st, fail_next, groot_last_error());
            groot_plan_free(plan);
            groot_graph_free(g);
            return 0;
        }
    """)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-o", str(driver), str(source), G.LIB_PATH,
                    "-Wl,--allow-shlib-undefined", f"-Wl,-rpath,{os.path.dirname(G.LIB_PATH)}", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    run = subprocess.run([str(driver)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stderr[-500:]
    assert run.stdout == f"{G.GROOT_ENOMEM} 0 groot_plan_upload: out of host memory"


@pytest.mark.parametrize("n,batch,flags", [
    (2, 1, 7), (3, 2, 7), (8, 1, 7), (32, 1, 7), (32, 3, 7), (64, 2, 7),
    (8, 1, 0), (8, 2, 1), (8, 1, 2), (8, 1, 3), (8, 1, 5), (8, 1, 6),
])
def test_graph_build_bit_exact(n, batch, flags):
    aig = wl.csa_multiplier_aig(n)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, batch, flags)
    v = G.groot_graph_view(g)
    rowptr, col, val, pol = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, batch, flags)
    assert v["n"] == aig.num_nodes * batch and v["nnz"] == rowptr[-1]
    assert np.array_equal(v["rowptr"], rowptr)
    assert np.array_equal(v["col"], col)
    assert np.array_equal(v["val"].view(np.uint32), val.view(np.uint32))
    assert np.array_equal(v["pol"], pol)


@pytest.mark.parametrize("n,batch", [(8, 1), (16, 3), (48, 2)])
def test_graph_build_bit_exact_on_booth_multipliers(n, batch):
    aig = wl.booth_multiplier_aig(n)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, batch)
    v = G.groot_graph_view(g)
    rowptr, col, val, pol = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, batch)
    assert np.array_equal(v["rowptr"], rowptr) and np.array_equal(v["col"], col)
    assert np.array_equal(v["val"].view(np.uint32), val.view(np.uint32)) and np.array_equal(v["pol"], pol)
    for T in (8, 32):
        pv = G.groot_plan_view(G.groot_spmm_plan(g, T))
        want = oracle.plan(rowptr, T)
        for key in ("row_class", "hd_rows", "ld_rows", "ld_rows_by_degree", "ld_deg_offsets"):
            assert np.array_equal(pv[key], want[key]), key


def test_graph_build_hand_made_aig_with_repeated_fanin():
    # node 3 = AND(x, !x) on the same driver, node 4 = AND(!2, 3), PO on !4
    typ = np.array([0, 0, 1, 1, 1, 2], dtype=np.uint8)
    f0 = np.array([-1, -1, 0, 4, 5, 9], dtype=np.int32)
    f1 = np.array([-1, -1, 2, 5, 6, 9], dtype=np.int32)
    for flags in (7, 0, 3):
        g = G.groot_graph_build(typ, f0, f1, 2, flags)
        v = G.groot_graph_view(g)
        o = oracle.csr_build(typ, f0, f1, 2, flags)
        for a, b in zip((v["rowptr"], v["col"], v["val"], v["pol"]), o):
            assert np.array_equal(a, b)


def test_graph_build_rejects_bad_input():
    aig = wl.csa_multiplier_aig(4)
    t, a, b = aig.type.copy(), aig.fanin0.copy(), aig.fanin1.copy()

    def expect(status, **kw):
        args = dict(type_=t, fanin0=a, fanin1=b, batch=1, flags=7)
        args.update(kw)
        with pytest.raises(G.GrootError) as e:
            G.groot_graph_build(**args)
        assert e.value.status == status and len(str(e.value)) > 20

    expect(G.GROOT_EINVAL, batch=0)
    expect(G.GROOT_EINVAL, flags=8)
    bad = a.copy(); bad[10] = 2 * 10          # literal pointing at itself: not topological
    expect(G.GROOT_EINVAL, fanin0=bad)
    bad = a.copy(); bad[10] = -1
    expect(G.GROOT_EINVAL, fanin0=bad)
    bad = a.copy(); bad[0] = 2                # primary input with a fanin
    expect(G.GROOT_EINVAL, fanin0=bad)
    bad = a.copy(); bad[-1] ^= 1              # PO slots differ
    expect(G.GROOT_EINVAL, fanin0=bad)
    bad = t.copy(); bad[7] = 3
    expect(G.GROOT_EINVAL, type_=bad)
    expect(G.GROOT_ERANGE, batch=2 ** 31 // aig.num_nodes + 1)
    status = G.binding._lib.groot_graph_build(4, None, None, None, 1, 7, None)
    assert status == G.GROOT_EINVAL and "NULL" in G.groot_last_error()


def test_from_csr_roundtrip_and_checks():
    g0 = wl.stress_graph(3, 1 << 12, window=64, dmin=64, dmax=512)
    g = G.groot_graph_from_csr(g0.rowptr, g0.col, g0.val)
    v = G.groot_graph_view(g)
    assert np.array_equal(v["rowptr"], g0.rowptr) and np.array_equal(v["col"], g0.col)
    assert np.array_equal(v["val"], g0.val) and v["pol"] is None
    bad = g0.col.copy(); bad[1], bad[0] = bad[0], bad[1]
    with pytest.raises(G.GrootError):
        G.groot_graph_from_csr(g0.rowptr, bad, g0.val)
    bad = g0.col.copy(); bad[5] = g0.n
    with pytest.raises(G.GrootError):
        G.groot_graph_from_csr(g0.rowptr, bad, g0.val)
    rp = g0.rowptr.copy(); rp[3] = rp[4] + 1
    with pytest.raises(G.GrootError):
        G.groot_graph_from_csr(rp, g0.col, g0.val)


@pytest.mark.parametrize("case", ["aig", "aig_directed", "stress"])
def test_graph_transpose_bit_exact(case):
    if case == "stress":
        s = wl.stress_graph(2, 1 << 12, window=64, dmin=64, dmax=512)
        g = G.groot_graph_from_csr(s.rowptr, s.col, s.val)
        rowptr, col, val = s.rowptr, s.col, s.val
    else:
        aig = wl.csa_multiplier_aig(16)
        flags = 7 if case == "aig" else 4
        g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 2, flags)
        rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, 2, flags)
    t = G.groot_graph_view(G.groot_graph_transpose(g))
    want = oracle.csr_transpose(rowptr, col, val)
    assert np.array_equal(t["rowptr"], want[0]) and np.array_equal(t["col"], want[1])
    assert np.array_equal(t["val"].view(np.uint32), want[2].view(np.uint32)) and t["pol"] is None
    assert G.binding._lib.groot_graph_transpose(None, None) == G.GROOT_EINVAL


@pytest.mark.parametrize("n,batch,T", [(8, 1, 7), (8, 3, 9), (32, 1, 32), (32, 2, 33), (32, 1, 34), (32, 1, 1),
                                       (64, 1, 4), (64, 1, 6), (256, 1, 32)])
def test_plan_bit_exact(n, batch, T):
    aig = wl.csa_multiplier_aig(n)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, batch)
    pv = G.groot_plan_view(G.groot_spmm_plan(g, T))
    rowptr = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, batch)[0]
    want = oracle.plan(rowptr, T)
    for k, w in want.items():
        assert np.array_equal(pv[k], w), k
    assert pv["n_hd"] == len(want["hd_rows"]) and pv["n_ld"] == len(want["ld_rows"])


@pytest.mark.parametrize("T", [16, 32, 64, 128])
def test_plan_bit_exact_on_stress_graph(T):
    g0 = wl.stress_graph(4, 1 << 15, window=256, dmin=64, dmax=1024)
    g = G.groot_graph_from_csr(g0.rowptr, g0.col, g0.val)
    pv = G.groot_plan_view(G.groot_spmm_plan(g, T))
    want = oracle.plan(g0.rowptr, T)
    for k, w in want.items():
        assert np.array_equal(pv[k], w), k


@pytest.mark.parametrize("T,hd_chunk", [(16, 512), (32, 64), (128, 300)])
def test_schedule_of_the_high_degree_rows(T, hd_chunk):
    """The HD kernel's launch list of a host plan (Section "Kernel Design - GROOT-GPU": the non-zeros of a
    high-degree row are split statically): every stored entry of every high-degree row lies in exactly one piece,
    a row of d entries has ceil(d / hd_chunk) balanced pieces, the partial-sum slots of a split row are one run,
    and the pieces run in the order of their first column (ties in row order)."""
    g0 = wl.stress_graph(4, 1 << 15, window=256, dmin=64, dmax=4096)
    g = G.groot_graph_from_csr(g0.rowptr, g0.col, g0.val)
    G.groot_set_tuning("hd_chunk", hd_chunk)
    try:
        plan = G.groot_spmm_plan(g, T)
    finally:
        G.groot_set_tuning("hd_chunk", 512)
    pc = G.groot_plan_hd_pieces(plan)                    # before any upload: the host copy
    deg = np.diff(g0.rowptr)
    hd_rows = np.flatnonzero(deg >= T)
    pieces_of = np.maximum(1, -(-deg[hd_rows] // hd_chunk))
    assert len(pc["row"]) == int(pieces_of.sum()) == G.groot_plan_query(plan, "hd_pieces")
    assert G.groot_plan_query(plan, "hd_partials") == int(pieces_of[pieces_of > 1].sum())
    covered = np.zeros(len(g0.col), np.int32)
    for b, ln, r in zip(pc["begin"], pc["len"], pc["row"]):
        assert g0.rowptr[r] <= b and b + ln <= g0.rowptr[r + 1] and 0 < ln <= hd_chunk
        covered[b:b + ln] += 1
    assert np.array_equal(covered, np.repeat(deg >= T, deg).astype(np.int32))
    first_col = g0.col[pc["begin"]]
    assert (np.diff(first_col) >= 0).all()
    ties = np.flatnonzero(np.diff(first_col) == 0)
    assert ((pc["row"][ties] < pc["row"][ties + 1]) |
            ((pc["row"][ties] == pc["row"][ties + 1]) & (pc["begin"][ties] < pc["begin"][ties + 1]))).all()
    for r, count in zip(hd_rows, pieces_of):
        mine = np.flatnonzero(pc["row"] == r)
        assert len(mine) == count
        lens = pc["len"][mine]
        assert lens.max() - lens.min() <= -(-deg[r] // count) - deg[r] // count + (count - 1)   # balanced
        slots = np.sort(pc["slot"][mine])
        if count == 1:
            assert slots[0] == -1
        else:
            assert slots[0] >= 0 and np.array_equal(slots, slots[0] + np.arange(count))


def _compare_parts(g, rowptr, col, val, part_of, P, flags, weight_mode):
    parts = G.groot_partition_regrow(g, P, part_of, flags)
    assert G.groot_parts_count(parts) == P
    po = part_of
    for p in range(P):
        got = G.groot_parts_view(parts, p)
        want = oracle.regrow_part(rowptr, col, val, po, p, flags, weight_mode)
        sub = G.groot_graph_view(got["sub"])
        for k in ("n_owned", "n_halo", "n_crossing"):
            assert got[k] == want[k], (p, k)
        assert np.array_equal(got["global_id"], want["global_id"])
        assert np.array_equal(sub["rowptr"], want["rowptr"])
        assert np.array_equal(sub["col"], want["col"])
        assert np.array_equal(sub["val"].view(np.uint32), want["val"].view(np.uint32))


@pytest.mark.parametrize("n,batch,P", [(2, 1, 2), (4, 2, 3), (8, 1, 5), (16, 2, 16), (32, 1, 7)])
@pytest.mark.parametrize("flags", [G.GROOT_REGROW, 0])
def test_partition_bit_exact_default_rule(n, batch, P, flags):
    aig = wl.csa_multiplier_aig(n)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, batch)
    rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, batch)
    part_of = oracle.part_of_default(len(rowptr) - 1, aig.num_nodes, P)
    parts = G.groot_partition_regrow(g, P, None, flags)
    for p in range(P):
        got = G.groot_parts_view(parts, p)
        want = oracle.regrow_part(rowptr, col, val, part_of, p, flags, 1)
        sub = G.groot_graph_view(got["sub"])
        assert (got["n_owned"], got["n_halo"], got["n_crossing"]) == (want["n_owned"], want["n_halo"], want["n_crossing"])
        assert np.array_equal(got["global_id"], want["global_id"])
        assert np.array_equal(sub["rowptr"], want["rowptr"]) and np.array_equal(sub["col"], want["col"])
        assert np.array_equal(sub["val"].view(np.uint32), want["val"].view(np.uint32))


def test_partition_bit_exact_user_parts_and_weight_modes():
    rng = np.random.default_rng(5)
    aig = wl.csa_multiplier_aig(8)
    # random assignment on the mean-normalised graph
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 1)
    rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, 1)
    part_of = rng.integers(0, 4, size=aig.num_nodes).astype(np.int32)
    _compare_parts(g, rowptr, col, val, part_of, 4, G.GROOT_REGROW, 1)
    # unit weights
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 1, 3)
    rowptr, col, val, _ = oracle.csr_build(aig.type, aig.fanin0, aig.fanin1, 1, 3)
    _compare_parts(g, rowptr, col, val, part_of, 4, G.GROOT_REGROW, 0)
    # directed graph with explicit weights (one-way crossing edges)
    s = wl.stress_graph(9, 1 << 11, window=32, dmin=64, dmax=256)
    w = rng.random(len(s.col)).astype(np.float32)
    g = G.groot_graph_from_csr(s.rowptr, s.col, w)
    part_of = rng.integers(0, 3, size=s.n).astype(np.int32)
    _compare_parts(g, s.rowptr, s.col, w, part_of, 3, G.GROOT_REGROW, 2)
    _compare_parts(g, s.rowptr, s.col, w, part_of, 3, 0, 2)
    # an empty part is legal
    part_of[:] = 0
    _compare_parts(g, s.rowptr, s.col, w, part_of, 2, G.GROOT_REGROW, 2)


def test_partition_and_misc_error_paths():
    aig = wl.csa_multiplier_aig(4)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 1)
    for kw in (dict(num_parts=0), dict(num_parts=aig.num_nodes + 1), dict(num_parts=2, flags=2),
               dict(num_parts=2, part_of=np.full(aig.num_nodes, 2, dtype=np.int32))):
        with pytest.raises(G.GrootError) as e:
            G.groot_partition_regrow(g, **kw)
        assert e.value.status == G.GROOT_EINVAL
    parts = G.groot_partition_regrow(g, 2)
    with pytest.raises(G.GrootError):
        G.groot_parts_view(parts, 2)
    with pytest.raises(G.GrootError):
        G.groot_set_tuning("no_such_knob", 1)
    with pytest.raises(G.GrootError):
        G.groot_set_tuning("hd_chunk", 7)
    G.groot_set_tuning("hd_chunk", 512)
    for knob, bad, good in (("ld_pipeline", 2, -1), ("ld_pipeline", -2, -1), ("sage_gap", 5, 2), ("sage_gap", -1, 2),
                            ("sage_kernel", 2, 1), ("sage_split", -1, 1), ("uniform_detect", 2, 1)):
        with pytest.raises(G.GrootError):
            G.groot_set_tuning(knob, bad)
        G.groot_set_tuning(knob, good)
    plan = G.groot_spmm_plan(g, 32)
    # executing without device residency is refused on the host, before any HIP call
    lib = G.binding._lib
    assert lib.groot_spmm_execute(plan.handle, 16, 32, 64, None) == G.GROOT_EINVAL
    assert "groot_plan_upload" in G.groot_last_error()
    assert lib.groot_spmm_execute(plan.handle, None, 32, 64, None) == G.GROOT_EINVAL
    assert lib.groot_spmm_execute(plan.handle, 16, 36, 64, None) == G.GROOT_EINVAL      # misaligned
    assert lib.groot_spmm_execute(plan.handle, 16, 32, 6, None) == G.GROOT_EINVAL       # F % 4
    assert lib.groot_rows_gather(None, 5, 16, 32, 64, None) == G.GROOT_EINVAL
    assert lib.groot_rows_gather(None, 0, 16, 32, 64, None) == G.GROOT_OK               # empty: no-op
    assert lib.groot_plan_upload(plan.handle, 6) == G.GROOT_EINVAL
    G.binding._lib.groot_graph_free(None)
    G.binding._lib.groot_plan_free(None)
    G.binding._lib.groot_parts_free(None)


def test_device_plan_lists_host_checks():
    """Argument checks of the device-side plan that need no GPU: a plan that was never uploaded and
    NULL outputs are refused before any device work."""
    aig = wl.csa_multiplier_aig(4)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 1)
    plan = G.groot_spmm_plan(g, 4)
    lib = G.binding._lib
    dummy = ctypes.c_void_p(256)
    assert lib.groot_plan_lists_device(plan.handle, dummy, dummy, dummy, dummy, dummy, dummy, None) == G.GROOT_EINVAL
    assert "not on the device" in G.groot_last_error()
    assert lib.groot_plan_lists_device(plan.handle, None, dummy, dummy, dummy, dummy, dummy, None) == G.GROOT_EINVAL
    assert lib.groot_plan_lists_device(None, dummy, dummy, dummy, dummy, dummy, dummy, None) == G.GROOT_EINVAL
    with pytest.raises(G.GrootError):
        G.groot_plan_query(plan, "ld_pipelined")          # not uploaded


def test_device_regrow_host_checks():
    """Argument checks of the device-side re-growth that need no GPU."""
    aig = wl.csa_multiplier_aig(4)
    g = G.groot_graph_build(aig.type, aig.fanin0, aig.fanin1, 1)
    plan = G.groot_spmm_plan(g, 4)
    lib = G.binding._lib
    out = ctypes.c_void_p()
    assert lib.groot_partition_regrow_device(plan.handle, 2, None, 1, 0, None, ctypes.byref(out)) == G.GROOT_EINVAL
    assert "not on the device" in G.groot_last_error() and not out.value
    assert lib.groot_partition_regrow_device(None, 2, None, 1, 0, None, ctypes.byref(out)) == G.GROOT_EINVAL
    assert lib.groot_partition_regrow_device(plan.handle, 2, None, 1, 0, None, None) == G.GROOT_EINVAL
    assert lib.groot_dev_part_view(None, None, None, None, None, None, None, None, None) == G.GROOT_EINVAL
    assert lib.groot_dev_part_plan(None, 4, 64, None, ctypes.byref(out)) == G.GROOT_EINVAL
    assert lib.groot_dev_part_download(None, None, None, None, None, None) == G.GROOT_EINVAL
    lib.groot_dev_part_free(None)


def test_build_module_is_importable_without_loading_the_library():
    """A tree without libgroot.so must still be able to import the build step (which makes the library);
    only the use of the binding needs it."""
    import subprocess
    import sys

    code = ("import sys; import paper_2511_18297_amd.build as b; from paper_2511_18297_amd import build as b2; "
            "assert b is b2 and callable(b.build); "
            "assert 'paper_2511_18297_amd.binding' not in sys.modules; print('ok')")
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stderr


def test_traffic_stamp_of_the_bench_ignores_comments_only(tmp_path, monkeypatch):
    """bench.py ties its measured-traffic figure to a hash of the kernel code: rewording a comment must keep it,
    changing a statement must not."""
    import importlib.util
    import shutil

    spec = importlib.util.spec_from_file_location("bench_for_test", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    stamp = bench.kernel_sources_sha16()
    csrc = tmp_path / "paper_2511_18297_amd" / "csrc"
    csrc.mkdir(parents=True)
    for name in bench.KERNEL_SOURCES:
        shutil.copy(os.path.join(ROOT, "paper_2511_18297_amd", "csrc", name), csrc / name)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_sources_sha16() == stamp
    path = csrc / "groot_ld_pipe.hip"
    text = path.read_text()
    path.write_text("// another comment\n" + text.replace("// ----", "//   ----", 1) + "\n   /* and a block\n comment */\n")
    assert bench.kernel_sources_sha16() == stamp
    path.write_text(text.replace("constexpr int kPipeWaves = 4;", "constexpr int kPipeWaves = 8;", 1))
    assert bench.kernel_sources_sha16() != stamp
