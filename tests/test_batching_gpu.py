"""GPU tests of the batched paths: one launch over several plans (cells of
different velocity grids), hipGraph capture and replay, and the launch-shape
autotuner. The operator is cell-local, so every variant must reproduce the
single-plan results bitwise."""

import ctypes
import json
import os

import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2103_14890_amd import qcoll
    return qcoll


SLOTS = [(32, 8.0, "hard_sphere", 8, "fx16", False, 37), (16, 8.0, "maxwell", 16, "fx16", False, 9),
         (24, 8.0, "hard_sphere", 8, "fp32", False, 13), (32, 8.0, "maxwell", 8, "fx16", True, 5),
         (12, 5.0, "hard_sphere", 8, "fp32", True, 3), (48, 8.0, "hard_sphere", 8, "fx16", False, 4),
         (64, 8.0, "maxwell", 8, "fx16", True, 3)]


def _setup(qc, seed=0):
    plans, fs = [], []
    for i, (N, L, kern, M, prec, cons, cells) in enumerate(SLOTS):
        plans.append(qc.Plan(2, N, L, kern, M, precision=prec, conserve=cons))
        fs.append(torch.tensor(wl.mixture_cells(2, N, L, cells, 100 + i + seed), dtype=torch.float32, device="cuda"))
    return plans, fs


def test_eval_multi_bitwise_equals_single_launches(qc):
    plans, fs = _setup(qc)
    singles = [p.eval(f) for p, f in zip(plans, fs)]
    outs = [torch.full_like(s, float("nan")) for s in singles]
    qc.eval_multi(plans, fs, outs)
    torch.cuda.synchronize()
    for a, b in zip(singles, outs):
        assert torch.equal(a, b)
    for p in plans:
        p.close()


def test_concurrent_launches_stay_ordered_on_the_callers_stream(qc):
    """Two launches in one call (ten slots: a full slot table of eight, tile-64
    and N <= 32 plans mixed, and a second table) run on the caller's stream and
    a side stream; work queued on the caller's stream after the call (no host
    synchronisation in between) sees every result."""
    cfg = [(64, 8.0, "hard_sphere", 8, 3), (48, 8.0, "maxwell", 8, 2), (64, 10.0, "maxwell", 16, 2),
           (40, 8.0, "hard_sphere", 8, 1), (48, 6.0, "hard_sphere", 8, 3), (32, 8.0, "hard_sphere", 8, 70),
           (16, 8.0, "maxwell", 16, 5), (24, 8.0, "hard_sphere", 8, 4), (64, 8.0, "hard_sphere", 8, 2),
           (20, 8.0, "maxwell", 8, 6)]
    plans, fs = [], []
    for i, (N, L, kern, M, cells) in enumerate(cfg):
        plans.append(qc.Plan(2, N, L, kern, M, precision="fx16"))
        fs.append(torch.tensor(wl.mixture_cells(2, N, L, cells, 300 + i), dtype=torch.float32, device="cuda"))
    singles = [p.eval(f) for p, f in zip(plans, fs)]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        outs = [torch.full_like(x, float("nan")) for x in singles]
        qc.eval_multi(plans, fs, outs, stream=side)
        copies = [o.clone() for o in outs]          # queued behind the call on the same stream
    torch.cuda.synchronize()
    for a, b in zip(singles, copies):
        assert torch.equal(a, b)
    for p in plans:
        p.close()


@pytest.mark.parametrize("scheme", ["explicit", "imex"])
def test_step_multi_bitwise_equals_single_launches(qc, scheme):
    plans, fs = _setup(qc, seed=7)
    ref = [f.clone() for f in fs]
    for p, f in zip(plans, ref):
        p.step(f, 0.02, 0.5, scheme)
    st = [torch.full((f.shape[0],), -1, dtype=torch.int32, device="cuda") for f in fs]
    qc.step_multi(plans, fs, 0.02, 0.5, scheme, st)
    torch.cuda.synchronize()
    for a, b, s in zip(ref, fs, st):
        assert torch.equal(a, b)
        assert (s == 0).all()
    for p in plans:
        p.close()


def test_graph_capture_and_replay(qc):
    """Capture single and batched launches in one graph; every replay (with eager
    work and synchronisation in between) equals the eager result bitwise."""
    plans, fs = _setup(qc, seed=3)
    eager = [p.eval(f) for p, f in zip(plans, fs)]
    torch.cuda.synchronize()
    q_single = torch.empty_like(eager[0])
    q_multi = [torch.empty_like(e) for e in eager]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):   # warm-up on the side stream before capture
        plans[0].eval(fs[0], q_single)
        qc.eval_multi(plans, fs, q_multi)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plans[0].eval(fs[0], q_single)
        qc.eval_multi(plans, fs, q_multi)
    for r in range(3):
        q_single.fill_(float("nan"))
        for q in q_multi:
            q.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(q_single, eager[0])
        for a, b in zip(q_multi, eager):
            assert torch.equal(a, b)
        other = plans[1].eval(fs[1])          # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(other, eager[1])
    for p in plans:
        p.close()


def test_autotune_keeps_results_and_caches(qc, tmp_path):
    plan = qc.Plan(2, 32, 8.0, "hard_sphere", 8, precision="fx16")
    f = torch.tensor(wl.mixture_cells(2, 32, 8.0, 1024, 9), dtype=torch.float32, device="cuda")
    before = plan.eval(f)
    cache = str(tmp_path / "tune.json")
    best = plan.autotune(f, reps=2, cache=cache)
    assert best["tile"] == 32 and best["waves_per_block"] in (1, 2, 4, 8) and best["max_blocks"] >= 1
    after = plan.eval(f)
    torch.cuda.synchronize()
    assert torch.equal(before, after)
    data = json.load(open(cache))
    assert data[plan.key] == best
    other = qc.Plan(2, 32, 8.0, "hard_sphere", 8, precision="fx16")
    assert other.load_tuning(cache) and other.shape() == best
    for ws in (1, 2, 4, 8):
        other.set_launch(ws, 64)
        assert torch.equal(other.eval(f), before)
    with pytest.raises(qc.QcollError):
        other.set_tile(16)                  # 18..32-point grids have one tile family
    plan.close()
    other.close()


@pytest.mark.parametrize("precision", ["fx16", "fp32"])
def test_autotune_tile_family(qc, tmp_path, precision):
    """A 16x16 plan runs on either tile family (the 16x16 kernels, or the 32x32
    kernels on the zero-padded grid): both stay within the precision's bound of
    the oracle, the autotuner picks among tiles x cells per workgroup x grid
    caps, the cached choice reproduces its results bitwise, and the batched
    call follows the plan's selected tile."""
    from oracle import spectral as sp
    tol = {"fx16": 1e-5, "fp32": 2e-4}[precision]
    f64 = wl.mixture_cells(2, 16, 8.0, 600, 19)
    f = torch.tensor(f64, dtype=torch.float32, device="cuda")
    ref = sp.q_fast(f64.astype(np.float32).astype(np.float64), sp.Setup(d=2, N=16, L=8.0, kernel="maxwell", M=16))
    plan = qc.Plan(2, 16, 8.0, "maxwell", 16, precision=precision)
    assert plan.tile() == (16, 32)
    outs = {}
    for t in (16, 32):
        plan.set_tile(t)
        assert plan.tile() == (t, 48 - t)
        q = plan.eval(f)
        torch.cuda.synchronize()
        outs[t] = q
        err = np.linalg.norm(q.cpu().double().numpy() - ref) / np.linalg.norm(ref)
        print(f"16x16 {precision} on the {t}x{t} tile kernels: rel L2 {err:.3e}")
        assert err < tol
    cache = str(tmp_path / "tune.json")
    best = plan.autotune(f, reps=2, cache=cache)
    assert best["tile"] in (16, 32) and plan.tile()[0] == best["tile"]
    tuned = plan.eval(f)
    other = qc.Plan(2, 16, 8.0, "maxwell", 16, precision=precision)
    assert other.load_tuning(cache) and other.shape() == best
    again = other.eval(f)
    out_m = torch.empty_like(again)
    qc.eval_multi([other], [f], [out_m])
    torch.cuda.synchronize()
    assert torch.equal(tuned, outs[best["tile"]]) and torch.equal(again, tuned) and torch.equal(out_m, tuned)
    with pytest.raises(qc.QcollError):
        other.set_tile(64)
    plan.close()
    other.close()


def test_more_slots_than_one_table(qc):
    """Ten plans in one call (the slot table holds eight; the call spreads them
    over several launches on the same stream) still match the single launches."""
    specs = [(N, kern) for N in (16, 24, 32, 20, 48) for kern in ("maxwell", "hard_sphere")]
    plans = [qc.Plan(2, N, 8.0, kern, 8, precision="fx16") for N, kern in specs]
    fs = [torch.tensor(wl.mixture_cells(2, N, 8.0, 3 + i, 300 + i), dtype=torch.float32, device="cuda")
          for i, (N, _) in enumerate(specs)]
    singles = [p.eval(f) for p, f in zip(plans, fs)]
    outs = [torch.full_like(s, float("nan")) for s in singles]
    qc.eval_multi(plans, fs, outs)
    ref = [f.clone() for f in fs]
    for p, f in zip(plans, ref):
        p.step(f, 0.01, 1.0, "explicit")
    qc.step_multi(plans, fs, 0.01, 1.0, "explicit")
    torch.cuda.synchronize()
    for a, b in zip(singles, outs):
        assert torch.equal(a, b)
    for a, b in zip(ref, fs):
        assert torch.equal(a, b)
    for p in plans:
        p.close()


@pytest.mark.parametrize("cells", [1, 37, 4100])
def test_pingpong_shape_matches_default_shape(qc, cells):
    """Eight wavefronts per workgroup (the ping-pong FX16 32x32 kernel) give the
    default shape's results bitwise, for eval, the projection, both single-stage
    steps and a multi-stage step, including a partly filled last workgroup."""
    f0 = torch.tensor(wl.mixture_cells(2, 32, 8.0, cells, 50 + cells), dtype=torch.float32, device="cuda")
    outs = {}
    for ws in (4, 8):
        plan = qc.Plan(2, 32, 8.0, "hard_sphere", 8, precision="fx16")
        cons = qc.Plan(2, 32, 8.0, "hard_sphere", 8, precision="fx16", conserve=True)
        for p in (plan, cons):
            p.set_launch(ws, 2048 if ws == 8 else 1024)
        fe, fi, fr = f0.clone(), f0.clone(), f0.clone()
        st = torch.full((cells,), -1, dtype=torch.int32, device="cuda")
        plan.step(fe, 0.02, 0.5, "explicit", st)
        plan.step(fi, 0.02, 0.5, "imex")
        plan.step_rk(fr, 0.02, 0.5, "ars222")
        outs[ws] = [plan.eval(f0), cons.eval(f0), fe, fi, fr, st]
        plan.close()
        cons.close()
    torch.cuda.synchronize()
    for a, b in zip(outs[4], outs[8]):
        assert torch.equal(a, b)
    assert (outs[8][5] == 0).all()


@pytest.mark.parametrize("scheme", ["ars222", "bpr343"])
@pytest.mark.parametrize("N,precision", [(32, "fx16"), (32, "fp32"), (16, "fx16")])
def test_step_rk_grid_stride_matches_default_shape(qc, N, precision, scheme):
    """Three one-wavefront workgroups walk 37 cells (about twelve each): the
    moments of f^n that the first stage launch keeps per cell, and the later
    launches read back, belong to that cell whatever wavefront computed it, so
    two steps match the default launch shape's bitwise."""
    cells = 37
    f0 = torch.tensor(wl.mixture_cells(2, N, 8.0, cells, 90 + N), dtype=torch.float32, device="cuda")
    out = []
    for shape in (None, (1, 3)):
        plan = qc.Plan(2, N, 8.0, "hard_sphere", 8, precision=precision)
        if shape is not None:
            plan.set_launch(*shape)
        f = f0.clone()
        for _ in range(2):
            plan.step_rk(f, 0.02, 0.5, scheme)
        out.append(f)
        plan.close()
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])


def test_calls_on_a_side_stream_with_library_allocated_buffers(qc):
    """Calls queued on a stream other than the current one, with the binding
    allocating the output and work buffers: the buffers are recorded on that
    stream, and the results equal the same calls on the current stream."""
    f0 = wl.mixture_cells(2, 32, 8.0, 12, 21)
    plan = qc.Plan(2, 32, 8.0, "hard_sphere", 8, precision="fx16")
    ref_f = torch.tensor(f0, dtype=torch.float32, device="cuda")
    ref_q = plan.eval(ref_f)
    plan.step_rk(ref_f, 0.01, 1.0, "ars222")
    side = torch.cuda.Stream()
    f = torch.tensor(f0, dtype=torch.float32, device="cuda")
    side.wait_stream(torch.cuda.current_stream())
    q = plan.eval(f, stream=side)
    plan.step_rk(f, 0.01, 1.0, "ars222", stream=side)
    # allocations on the current stream while the side stream may still run
    junk = [torch.full((12, 32, 32), 7.0, device="cuda") for _ in range(4)]
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    assert torch.equal(q, ref_q)
    assert torch.equal(f, ref_f)
    del junk
    plan.close()


@pytest.mark.parametrize("N,kernel,M", [(32, "hard_sphere", 8), (18, "hard_sphere", 6), (32, "maxwell", 14),
                                        (26, "maxwell", 16), (32, "maxwell", 2)])
def test_few_cells_equal_the_full_batch_bitwise(qc, N, kernel, M):
    """Few cells run eight wavefronts per cell in rounds of eight transforms (here 21
    or more, 8, 9 and 2 entries with the loss): bitwise the results of the same cells
    in a batch that runs one wavefront per cell, for every output of such plans."""
    cells = 600
    f0 = torch.tensor(wl.mixture_cells(2, N, 8.0, cells, 60 + N), dtype=torch.float32, device="cuda")
    plan = qc.Plan(2, N, 8.0, kernel, M, precision="fx16", conserve=True)

    def outputs(f):
        fe, fr = f.clone(), f.clone()
        st = torch.full((f.shape[0],), -1, dtype=torch.int32, device="cuda")
        plan.step(fe, 0.02, 0.5, "imex", st)
        plan.step_rk(fr, 0.02, 0.5, "bpr343")
        return [plan.eval(f), fe, fr, st]

    full = outputs(f0)
    for lo, hi in ((0, 1), (5, 14), (17, 17 + 256)):
        for a, b in zip(outputs(f0[lo:hi].contiguous()), full):
            assert torch.equal(a, b[lo:hi])
    plan.close()
    gal = qc.Plan(2, 16, 8.0, kernel, M, precision="fx16", galerkin=True)   # fine grid of 24 points
    g0 = torch.tensor(wl.mixture_cells(2, 16, 8.0, cells, 61), dtype=torch.float32, device="cuda")
    assert torch.equal(gal.eval_galerkin(g0[3:20].contiguous()), gal.eval_galerkin(g0)[3:20])
    gal.close()


class _KernelNode(ctypes.Structure):   # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _workgroups(qc, call):
    """Workgroups of each kernel that call(stream) launches, from a captured graph
    (which is not run)."""
    lib, s, graph = qc.LIB, torch.cuda.Stream(), ctypes.c_void_p()
    call(s)
    s.synchronize()
    assert lib.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 2) == 0
    try:
        call(s)
    finally:
        assert lib.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    n = ctypes.c_size_t()
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes, out = (ctypes.c_void_p * n.value)(), []
    assert lib.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    for node in nodes:
        p = _KernelNode()
        assert lib.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        out.append(p.grid[0])
    assert lib.hipGraphDestroy(graph) == 0
    return out


@pytest.mark.parametrize("cap", [1, 2, 1 << 20])
def test_few_cells_keep_the_grid_cap(qc, cap):
    """The launch shape's cap holds for the form that gives a cell eight wavefronts as
    well: its workgroups then walk several cells, with the same digits."""
    cells = 5
    f0 = torch.tensor(wl.mixture_cells(2, 32, 8.0, cells, 92), dtype=torch.float32, device="cuda")
    plan = qc.Plan(2, 32, 8.0, "hard_sphere", 8, precision="fx16", conserve=True)
    want = plan.eval(f0)
    steps = plan.step(f0.clone(), 0.02, 0.5, "imex")
    plan.set_launch(4, cap)
    q, g = torch.empty_like(want), f0.clone()
    assert _workgroups(qc, lambda s: plan.eval(f0, q, stream=s)) == [min(cells, cap)]
    assert torch.equal(q, want)
    assert torch.equal(plan.step(g, 0.02, 0.5, "imex"), steps)
    plan.close()


@pytest.mark.parametrize("cap", [1, 2, 3, 100, 1 << 62])
@pytest.mark.parametrize("N", [4, 10, 16])
def test_many_small_cells_keep_the_grid_cap(qc, N, cap):
    """Four cells per wavefront, and the cells left over one per wavefront: both parts
    together stay within the cap, with the same digits."""
    cells = 16 * torch.cuda.get_device_properties(0).multi_processor_count + 5
    f0 = torch.tensor(wl.mixture_cells(2, N, 8.0, 7, 93 + N), dtype=torch.float32, device="cuda")
    f0 = f0[torch.arange(cells, device="cuda") % 7].contiguous()
    plan = qc.Plan(2, N, 8.0, "hard_sphere", 8, precision="fx16")
    want = plan.eval(f0)
    steps = plan.step(f0.clone(), 0.02, 0.5, "imex")
    plan.set_launch(4, cap)
    q, g = torch.empty_like(want), f0.clone()
    grid, = _workgroups(qc, lambda s: plan.eval(f0, q, stream=s))
    assert grid <= cap
    q.zero_()
    plan.eval(f0, q)
    assert torch.equal(q, want)
    assert torch.equal(plan.step(g, 0.02, 0.5, "imex"), steps)
    plan.close()


@pytest.mark.parametrize("N", [8, 16, 18, 20, 22, 24])
def test_classical_workgroup_widths(qc, N):
    """Four and sixteen (eight) cells per workgroup around the lines of the rule: the same
    digits, and the widths that the rule names."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    f = torch.tensor(wl.mixture_cells(2, N, 8.0, 7, 95 + N), dtype=torch.float32, device="cuda")
    plan = qc.Plan(2, N, 8.0, "hard_sphere", 6, classical=True, separable_modes=True, conserve=True)
    want = plan.eval(f)
    wide = 8 if N > 20 else 16
    for cells in (8 * cus, 8 * cus + 3, 16 * cus - 1, 16 * cus, 16 * cus + 3, 24 * cus + 5):
        at = torch.arange(cells, device="cuda") % 7
        many = f[at].contiguous()
        q = torch.empty(many.shape, dtype=torch.float64, device="cuda")
        grid, = _workgroups(qc, lambda s: plan.eval(many, q, stream=s))
        rounds = -(-cells // (8 * cus))
        width = wide if (rounds > 1 if N == 18 else rounds % 2 == 0 if N == 20 else cells >= 16 * cus) else 4
        assert grid == -(-cells // width), (N, cells)
        q.zero_()
        plan.eval(many, q)
        assert torch.equal(q, want[at]), (N, cells)
    plan.close()


def test_step_multi_takes_a_longer_status_list(qc):
    """Status entries beyond the plans are ignored (a caller may keep one list for all of
    its cells' groups and step only some of them)."""
    plan = qc.Plan(2, 16, 8.0, "maxwell", 8, precision="fx16")
    f = torch.tensor(wl.mixture_cells(2, 16, 8.0, 3, 94), dtype=torch.float32, device="cuda")
    st = [torch.full((3,), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
    qc.step_multi([plan], [f], 0.01, 1.0, "imex", statuses=[st[0], None, st[2]])
    assert st[0].cpu().tolist() == [0, 0, 0] and st[2].cpu().tolist() == [-1, -1, -1]
    plan.close()


@pytest.mark.parametrize("N,M,shared", [(28, 8, True), (20, 8, True), (24, 16, True), (28, 6, False), (20, 4, False)])
def test_two_cells_per_compute_unit_share_workgroups(qc, N, M, shared):
    """Between one and two cells per compute unit a cell has a workgroup of its own from
    four transforms (Maxwell, M = 8) on, with the digits of a wavefront per cell."""
    cells = torch.cuda.get_device_properties(0).multi_processor_count + 44
    f = torch.tensor(wl.mixture_cells(2, N, 8.0, 7, 97), dtype=torch.float32, device="cuda")
    at = torch.arange(2 * cells, device="cuda") % 7
    plan = qc.Plan(2, N, 8.0, "maxwell", M, precision="fx16")
    want = plan.eval(f[at].contiguous())[:cells]
    many = f[at[:cells]].contiguous()
    q = torch.empty_like(want)
    assert _workgroups(qc, lambda s: plan.eval(many, q, stream=s)) == [cells if shared else -(-cells // 4)]
    assert torch.equal(plan.eval(many), want)
    plan.close()


@pytest.mark.parametrize("N,conserve,cells", [(32, True, 5), (24, False, 5), (16, False, 5000)])
def test_autotune_keeps_what_the_launch_ignores(qc, N, conserve, cells):
    """Forms for few cells and for many small ones choose their own cells per workgroup
    (and FFT plans have one kernel for both tile families): the autotuner keeps the plan's
    values instead of choosing among equal launches."""
    f = torch.tensor(wl.mixture_cells(2, N, 8.0, cells, 98), dtype=torch.float32, device="cuda")
    for waves in (1, 2):
        plan = qc.Plan(2, N, 8.0, "hard_sphere", 8, precision="fx16", conserve=conserve)
        plan.set_launch(waves, 64)
        tile = plan.tile()
        want = plan.eval(f)
        best = plan.autotune(f, reps=2)
        assert best["waves_per_block"] == waves and plan.tile() == tile
        assert torch.equal(plan.eval(f), want)
        plan.close()


@pytest.mark.parametrize("N", [18, 20, 22, 24, 26])
def test_steps_of_projected_plans_bitwise(qc, N):
    """The steps of a plan with the projection (more cells than compute units, as fewer run
    on another kernel) give the digits of the batched call."""
    f = torch.rand(300, N, N, generator=torch.Generator().manual_seed(N)).cuda()
    plan = qc.Plan(2, N, 8.0, "hard_sphere", 4, precision="fx16", conserve=True)
    a, b = f.clone(), f.clone()
    plan.step(a, 0.01, 1.0, "imex")
    qc.step_multi([plan], [b], 0.01, 1.0, "imex")
    assert torch.equal(a, b)
    plan.close()


def test_more_plans_than_a_slot_table(qc):
    """Forty slots: three slot tables (concurrently on side streams: few cells), every
    result bitwise that of the single-plan call, twice in a row without a
    synchronisation in between."""
    plans, fs = [], []
    for i in range(40):
        N = (16, 24, 32, 48, 20)[i % 5]
        plans.append(qc.Plan(2, N, 8.0, "maxwell" if i % 2 else "hard_sphere", 8, precision="fx16", conserve=i % 7 == 0))
        fs.append(torch.tensor(wl.mixture_cells(2, N, 8.0, 1 + i % 3, 300 + i), dtype=torch.float32, device="cuda"))
    qs = [torch.empty(f.shape, dtype=torch.float64 if p.conserve else torch.float32, device="cuda")
          for p, f in zip(plans, fs)]
    qc.eval_multi(plans, fs, qs)
    qc.eval_multi(plans, fs, qs)
    for p, f, q in zip(plans, fs, qs):
        assert torch.equal(q, p.eval(f))
        p.close()


@pytest.mark.parametrize("precision", ["fx16", "fp32"])
@pytest.mark.parametrize("N", [34, 36, 44, 48, 50])
def test_64_point_tiles_without_their_empty_rows_bitwise(qc, N, precision):
    """Up to 48 points the single-plan kernels leave out the tile rows beyond the grid
    (the batched kernel does not): the same digits."""
    g = torch.Generator().manual_seed(N)
    f = torch.rand(5, N, N, generator=g).cuda()
    plan = qc.Plan(2, N, 8.0, "hard_sphere", 4, precision=precision, conserve=True)
    q = torch.empty(f.shape, dtype=torch.float64, device="cuda")
    qc.eval_multi([plan], [f], [q])
    assert torch.equal(plan.eval(f), q)
    plan.close()
    plan = qc.Plan(2, N, 8.0, "maxwell", 2, precision="fp32")
    a, b = f.clone(), f.clone()
    plan.step(a, 0.01, 1.0, "imex")
    qc.step_multi([plan], [b], 0.01, 1.0, "imex")
    assert torch.equal(a, b)
    plan.close()


@pytest.mark.parametrize("precision", ["fx16", "fp32"])
@pytest.mark.parametrize("N", [18, 20, 22, 24, 26])
def test_32_point_tiles_without_their_empty_rows_bitwise(qc, N, precision):
    """The same on the 32x32 tiles (up to 24 points; more cells than compute units, as
    fewer run on another kernel)."""
    g = torch.Generator().manual_seed(N)
    f = torch.rand(300, N, N, generator=g).cuda()
    plan = qc.Plan(2, N, 8.0, "hard_sphere", 4, precision=precision, conserve=True)
    q = torch.empty(f.shape, dtype=torch.float64, device="cuda")
    qc.eval_multi([plan], [f], [q])
    assert torch.equal(plan.eval(f), q)
    plan.close()
    if precision == "fp32":
        plan = qc.Plan(2, N, 8.0, "maxwell", 2, precision=precision)
        a, b = f.clone(), f.clone()
        plan.step(a, 0.01, 1.0, "imex")
        qc.step_multi([plan], [b], 0.01, 1.0, "imex")
        assert torch.equal(a, b)
        plan.close()
