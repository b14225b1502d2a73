"""The FP64 FFT kernels (FX16 plans without the projection) on every grid size they
have a body for, against the FP64 oracle.

Tolerance: spectra, transforms and sums are FP64 (their error relative to Q is of
the order of gain/Q x 1e-15 ~ 1e-13), so the float rounding of Q is what is left:
at most 2^-24 = 6e-8 of every value, hence of the 2-norm; 1.5e-7 leaves room for
the plan's filters, which the oracle computes separately.
"""

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import spectral as sp
from oracle import stepping
from paper_2103_14890_amd import qcoll

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SIZES = list(range(4, 33, 2)) + list(range(36, 65, 4))


def _case(N, cells):
    kernel = "maxwell" if N % 8 == 2 else "hard_sphere"
    L = 3.0 + 0.16 * N
    f = wl.mixture_cells(2, N, L, cells, 50 + N).astype(np.float32)
    # a different scale per cell, so that a mixed-up cell or slot shows
    f *= np.linspace(0.5, 2.0, cells, dtype=np.float32)[:, None, None]
    M = 6 if N % 4 == 0 else 8
    s = sp.Setup(d=2, N=N, L=L, kernel=kernel, M=M)
    return f, L, kernel, M, sp.q_fast(f.astype(np.float64), s)


def _rel(got, ref):
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("N", SIZES)
def test_every_grid_size(N):
    f, L, kernel, M, ref = _case(N, 7)   # 7 cells: the last workgroup is not full
    plan = qcoll.Plan(2, N, L, kernel, M)
    t = torch.tensor(f, device=DEV)
    for waves in (1, 4):
        plan.set_launch(waves, 1 if waves == 4 else 1 << 20)   # one workgroup walking the cells, or one per cell
        q = plan.eval(t).cpu().double().numpy()
        assert _rel(q, ref) < 1.5e-7, (N, waves)
    one = plan.eval(t[2:3].contiguous()).cpu().numpy()
    assert np.array_equal(one, q[2:3].astype(np.float32)), "a cell's result does not depend on the batch"
    status = torch.full((7,), -1, dtype=torch.int32, device=DEV)
    g = plan.step(t.clone(), 0.01, 1.0, "imex", status=status).cpu().double().numpy()
    want = stepping.imex_euler_penalized(f.astype(np.float64), ref, 0.01, 1.0, 2, L)
    assert np.abs(g - want).max() <= 1.2e-7 * np.abs(want).max()
    assert status.cpu().tolist() == [0] * 7
    if N > 16:   # the transforms of a cell shared by several workers: the FP64 sums in another order
        for split in ((4,) if N <= 32 else (2, 8)):
            plan.set_split(split)
            assert _rel(plan.eval(t).cpu().double().numpy(), ref) < 1.5e-7, (N, split)
    plan.close()


@pytest.mark.parametrize("N", range(4, 17, 2))
def test_many_cells_equal_few_bitwise(N):
    """Four cells per wavefront (whole rounds of 16 cells per compute unit, and what
    is left over, alone or four to a wavefront) against a cell per wavefront."""
    f, L, kernel, M, _ = _case(N, 7)
    plan = qcoll.Plan(2, N, L, kernel, M)
    few = torch.tensor(f, device=DEV)
    q = plan.eval(few)
    g, st = few.clone(), torch.empty(7, dtype=torch.int32, device=DEV)
    few[5, 1, 1] = float("nan")   # its four-cell neighbours keep status 0
    bad = few.clone()
    plan.step(g, 0.01, 1.0, "explicit")
    plan.step(bad, 0.01, 1.0, "explicit", status=st)
    assert st.cpu().tolist() == [0] * 5 + [1, 0]
    unit = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    for cells in (unit - 1, unit, unit + 5, 2 * unit + unit // 2 + 2, 2 * unit + unit - 3):
        idx = torch.arange(cells, device=DEV) % 7
        many = torch.tensor(f, device=DEV)[idx].contiguous()
        assert torch.equal(plan.eval(many), q[idx]), cells
        status = torch.full((cells,), -1, dtype=torch.int32, device=DEV)
        many = few[idx].contiguous()
        plan.step(many, 0.01, 1.0, "explicit", status=status)
        ok = idx != 5
        assert torch.equal(many[ok], g[idx][ok]), cells
        assert torch.equal(status, (~ok).int()), cells
    plan.set_launch(4, 3)   # a capped grid walks its cells
    many = torch.tensor(f, device=DEV)[idx].contiguous()
    assert torch.equal(plan.eval(many), q[idx])
    plan.close()


@pytest.mark.parametrize("N", range(18, 33, 2))
@pytest.mark.parametrize("M", [2, 4, 8])
def test_few_cells_share_a_workgroup_bitwise(N, M):
    """With few cells a workgroup of four wavefronts computes a cell (fewer groups of
    transforms than wavefronts for small M, a last round of one, or several rounds),
    with many one wavefront: the same digits."""
    f, L, kernel, _, _ = _case(N, 7)
    plan = qcoll.Plan(2, N, L, kernel, M)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    limit = 2 * cus
    src = torch.tensor(f, device=DEV)
    idx = torch.arange(limit + 1, device=DEV) % 7

    def run(cells, act):
        t = src[idx[:cells]].contiguous()
        return act(t)

    def rk(t):
        plan.step_rk(t, 0.01, 1.0, "bpr343")
        return t

    for act in (plan.eval, lambda t: plan.step(t, 0.01, 1.0, "imex"), rk):
        want = run(limit + 1, act)
        for cells in (1, 5, cus, limit):
            assert torch.equal(run(cells, act), want[:cells]), cells
    plan.set_launch(4, 2)   # a capped grid walks its cells
    assert torch.equal(run(5, plan.eval), run(limit + 1, plan.eval)[:5])
    plan.close()


@pytest.mark.parametrize("N", SIZES)
def test_batched_calls_equal_single_plan_calls_bitwise(N):
    """A slot of a batched call gives the digits of the single-plan call, alone and next
    to a slot of the matrix kernels (its workgroups full and ragged)."""
    f, L, kernel, M, _ = _case(N, 7)
    plan, other = qcoll.Plan(2, N, L, kernel, M), qcoll.Plan(2, 32, L, "maxwell", 4, conserve=True)
    t = torch.tensor(f, device=DEV)
    g = torch.tensor(wl.mixture_cells(2, 32, L, 3, 90), dtype=torch.float32, device=DEV)
    want, want_g = plan.eval(t), other.eval(g)
    stepped, stepped_g = plan.step(t.clone(), 0.01, 1.0, "imex"), other.step(g.clone(), 0.01, 1.0, "imex")
    for mixed in (False, True):
        plans, fs = ([plan, other], [t, g]) if mixed else ([plan], [t])
        qs = [torch.empty_like(want), torch.empty_like(want_g)][:len(plans)]
        qcoll.eval_multi(plans, fs, qs)
        assert torch.equal(qs[0], want) and (not mixed or torch.equal(qs[1], want_g))
        fs = [x.clone() for x in fs]
        qcoll.step_multi(plans, fs, 0.01, 1.0, "imex")
        assert torch.equal(fs[0], stepped) and (not mixed or torch.equal(fs[1], stepped_g))
    plan.close()
    other.close()
