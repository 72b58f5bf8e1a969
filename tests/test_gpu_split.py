"""The persistent chunk kernel on every split of a path that a plan may take,
whichever one timing would choose: workgroups per path, 512 and 1024 threads,
one launch of all paths and several.  It adds the same products in the same
order as the stage kernel, so every comparison with that is bitwise; the
gradient shares of the adjoint are summed in another order (each of their
4 x steps x rows terms rounds once: 1e-12 of the largest)."""
import numpy as np
import pytest
import torch

import paper_2403_04252_amd as W

pytestmark = pytest.mark.gpu

SPLITS = [1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 80, 96]
# n_max, l_max, n_bins: N = 4, 13, 68, 155, 366, 580, 86 (l_max 8), 1868
BASES = [(1, 0, 3), (2, 1, 2), (3, 2, 6), (5, 4, 4), (4, 3, 21), (6, 4, 20), (2, 8, 1), (8, 7, 26)]
FORMS = {"exact": {}, "interp": dict(interp=True), "fp32": dict(mixed=True, stage_cache=W.WPCCC_CACHE_OFF)}


def _basis(n_max, l_max, n_bins):
    return W.wpccc_basis(W.BasisSpec(n_max, l_max, n_bins, 3.0, 300, 60.0, 1.0))


def _run(plan, zg):
    X = torch.zeros((plan.n_traj, plan.n_pad), dtype=torch.complex128, device="cuda")
    X[:, 0] = 1.0
    W.wpccc_propagate(plan, zg, X)
    W.wpccc_plan_status(plan)
    torch.cuda.synchronize()
    return X.cpu().numpy()


def _splits(plan):
    """Every split of SPLITS that fits, set on the plan; then two of them a few paths at a time."""
    seen = []
    for g in SPLITS:
        try:
            W.wpccc_plan_set_stage_split(plan, g)
        except W.WpcccError as e:
            assert e.code == -6
            continue
        got, paths = W.wpccc_plan_stage_split(plan)
        assert 1 <= got <= g and 1 <= paths <= plan.n_traj
        if got in seen:
            continue
        seen.append(got)
        yield got, paths
    assert seen
    for g, paths in ((seen[0], 1), (seen[-1], 2)):
        W.wpccc_plan_set_stage_split(plan, g, paths)
        assert W.wpccc_plan_stage_split(plan) == (g, min(paths, plan.n_traj))
        yield g, paths


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n_max,l_max,n_bins", BASES)
def test_every_split_bitwise(n_max, l_max, n_bins, form):
    zg = np.linspace(-3.0, 0.5, 68) ** 3 / 9.0   # 67 ragged steps: a full chunk and a short one
    plan = W.wpccc_plan_create(_basis(n_max, l_max, n_bins), [0.4, 1.5, 6.0], [1.0, 2.0, 1.5], stage_rows=4,
                               stage_launch=W.WPCCC_LAUNCH_STAGES, **FORMS[form])
    assert W.wpccc_plan_stage_split(plan) == (0, 0)
    ref = _run(plan, zg)
    for g, paths in _splits(plan):
        print(f"N = {plan.n_states}, {form}: {g} workgroups, {paths} paths a launch", flush=True)
        assert np.array_equal(_run(plan, zg), ref), (g, paths)
    W.wpccc_plan_set_stage_split(plan, 0)
    assert W.wpccc_plan_stage_split(plan) == (0, 0)
    assert np.array_equal(_run(plan, zg), ref)


@pytest.mark.parametrize("n_max,l_max,n_bins", BASES[1:-1])
def test_every_split_adjoint(n_max, l_max, n_bins):
    zg = np.linspace(-3.0, 2.0, 68)
    b = np.array([0.6, 2.0, 4.0])
    plan = W.wpccc_plan_create(_basis(n_max, l_max, n_bins), b, 1.5, model_a=0.5, model_c=1.2, stage_rows=4,
                               stage_launch=W.WPCCC_LAUNCH_STAGES)
    X0 = torch.zeros((3, plan.n_pad), dtype=torch.complex128, device="cuda")
    X0[:, 0] = 1.0
    gX = torch.zeros_like(X0)
    gX[:, :plan.n_states] = torch.exp(1j * torch.arange(plan.n_states, device="cuda", dtype=torch.float64))

    def grads():
        X, grad = torch.empty_like(X0), torch.empty((3, 3), dtype=torch.float64, device="cuda")
        W.wpccc_adjoint(plan, zg, X0, gX, grad, X)
        W.wpccc_plan_status(plan)
        torch.cuda.synchronize()
        return X.cpu().numpy(), grad.cpu().numpy()

    X, g0 = grads()
    for g, paths in _splits(plan):
        print(f"adjoint, N = {plan.n_states}: {g} workgroups, {paths} paths a launch", flush=True)
        Xc, gc = grads()
        assert np.array_equal(Xc, X), (g, paths)
        assert np.abs(gc - g0).max() <= 1e-12 * np.abs(g0).max(), (g, paths)


def test_split_is_what_runs():
    """The launch query follows the kernel: a plan that asks for the persistent
    form of a basis no split fits reports one launch per stage, the FP32-table
    and interpolated forms tell their split, and refusals change nothing."""
    big = _basis(10, 7, 32)   # N = 2380
    try:
        plan = W.wpccc_plan_create(big, [1.0], [1.0], stage_launch=W.WPCCC_LAUNCH_PERSISTENT)
    except W.WpcccError as e:
        assert e.code == -6
        plan = W.wpccc_plan_create(big, [1.0], [1.0])
    assert W.wpccc_plan_stage_split(plan) == (0, 0)
    assert W.wpccc_plan_stage_launch(plan) == W.WPCCC_LAUNCH_STAGES
    with pytest.raises(W.WpcccError) as e:
        W.wpccc_plan_set_stage_split(plan, 96)
    assert e.value.code == -6
    lb = _basis(3, 2, 6)
    plan = W.wpccc_plan_create(lb, [1.0], [1.0], stage_launch=W.WPCCC_LAUNCH_PERSISTENT)
    g, n = W.wpccc_plan_stage_split(plan)
    assert g >= 1 and n == 1 and W.wpccc_plan_stage_launch(plan) == W.WPCCC_LAUNCH_PERSISTENT
    plan = W.wpccc_plan_create(lb, [1.0], [1.0], interp=True)
    W.wpccc_plan_set_stage_split(plan, 2)
    assert W.wpccc_plan_stage_split(plan) == (2, 1) and W.wpccc_plan_stage_launch(plan) == W.WPCCC_LAUNCH_STAGES
    plan = W.wpccc_plan_create(lb, [1.0], [1.0], mixed=True, stage_cache=W.WPCCC_CACHE_ON)
    for bad, code in ((2, -6), (-1, -1)):
        with pytest.raises(W.WpcccError) as e:
            W.wpccc_plan_set_stage_split(plan, bad)
        assert e.value.code == code and W.wpccc_plan_stage_split(plan) == (0, 0)


@pytest.mark.parametrize("n_max,l_max,n_bins,n_paths", [(2, 1, 3, 1), (3, 2, 8, 3), (6, 4, 20, 5)])
def test_mixed_plan_has_one_arithmetic(n_max, l_max, n_bins, n_paths):
    """An FP32-table plan with the default choices rounds alike in every call:
    steps one by one, a propagation and a second one on other chunk borders;
    the same for a graph plan, whose full chunks are replays and whose
    remainder is not."""
    lb = _basis(n_max, l_max, n_bins)
    b, zg = np.linspace(0.5, 4.0, n_paths), np.arange(76) / 8.0 - 4.0   # z + h is the next grid point exactly
    for kw in ({}, dict(graph=True)):
        plan = W.wpccc_plan_create(lb, b, 1.5, mixed=True, **kw)
        split, cache = W.wpccc_plan_stage_split(plan), W.wpccc_plan_stage_cache(plan)
        print(f"N = {plan.n_states} {kw}: split {split}, cache {cache}", flush=True)
        start = torch.zeros((n_paths, plan.n_pad), dtype=torch.complex128, device="cuda")
        start[:, 0] = 1.0
        whole, parts, steps = start.clone(), start.clone(), start.clone()
        W.wpccc_propagate(plan, zg, whole)
        W.wpccc_propagate(plan, zg[:4], parts)
        W.wpccc_propagate(plan, zg[3:], parts)
        for z in zg[:-1]:
            W.wpccc_step(plan, steps, z, 0.125)
        W.wpccc_plan_status(plan)
        torch.cuda.synchronize()
        assert torch.equal(whole, steps) and torch.equal(whole, parts)
        assert not (split[0] and cache)


def _adjoint(plan, zg):
    n = plan.n_traj
    X0 = torch.zeros((n, plan.n_pad), dtype=torch.complex128, device="cuda")
    X0[:, 0] = 1.0
    gX = torch.zeros_like(X0)
    gX[:, :plan.n_states] = torch.exp(1j * torch.arange(plan.n_states, device="cuda", dtype=torch.float64))
    X, grad = torch.empty_like(X0), torch.empty((n, 3), dtype=torch.float64, device="cuda")
    W.wpccc_adjoint(plan, zg, X0, gX, grad, X)
    W.wpccc_plan_status(plan)
    return X, grad


@pytest.mark.parametrize("every", [1, 5, 64, 70])
def test_adjoint_memory_follows_checkpoints(every):
    """What the adjoint by the persistent kernel holds beside the segments:
    four vectors per step of a run, which is no longer than the steps between
    checkpoints, and the 16 shares of each row tile and path for a chunk's
    steps; gradients as kernel by kernel (the bar above), also after a call on
    a longer grid grew the workspace."""
    lb, zg = _basis(3, 2, 8), np.linspace(-4.0, 4.0, 141)
    b = np.linspace(0.6, 4.0, 16)
    plan = W.wpccc_plan_create(lb, b, 1.5, model_a=0.5, model_c=1.2, checkpoint_every=every, stage_rows=4,
                               stage_launch=W.WPCCC_LAUNCH_STAGES)
    Xs, gs = _adjoint(plan, zg)
    held = W.wpccc_plan_info(plan)[3]
    W.wpccc_plan_set_stage_split(plan, 2)
    tables = W.wpccc_plan_info(plan)[3] - held
    for steps in (every, 140):   # one segment, then all
        X, g = _adjoint(plan, zg[:steps + 1])
    assert torch.equal(X, Xs) and (g - gs).abs().max() <= 1e-12 * gs.abs().max()
    grown = W.wpccc_plan_info(plan)[3] - held - tables
    tiles = sum((n + 7) // 8 for n in (11, 10, 9))
    assert grown <= 16 * plan.n_traj * plan.n_pad * 4 * min(every, 64) + 8 * plan.n_traj * 16 * 64 * tiles


def test_adjoint_without_memory_for_runs():
    """Where the device has room for the segments but not for the persistent
    kernel's runs, the sweeps go kernel by kernel, in this call and the next."""
    lb, zg, n = _basis(6, 4, 20), np.linspace(-1.0, 1.0, 65), 1700
    b = np.linspace(0.6, 4.0, n)
    make = lambda: W.wpccc_plan_create(lb, b, 1.5, model_a=0.5, model_c=1.2, checkpoint_every=64, stage_rows=8,
                                       stage_launch=W.WPCCC_LAUNCH_STAGES)
    ref = make()
    Xs, gs = _adjoint(ref, zg)
    W.wpccc_plan_set_stage_split(ref, 8)   # every kernel has run before memory gets short
    _adjoint(ref, zg)
    W.wpccc_plan_destroy(ref)
    plan = make()
    W.wpccc_plan_set_stage_split(plan, 8)
    torch.cuda.empty_cache()
    vector = 16 * n * plan.n_pad
    runs, segments = 256 * vector, (4 * 64 + 1 + 2 + 3 + 1) * vector
    free = torch.cuda.mem_get_info()[0]
    fill = torch.empty(free - segments - runs // 2, dtype=torch.uint8, device="cuda")
    print(f"{free >> 20} MiB free, {segments >> 20} for segments, {runs >> 20} for runs", flush=True)
    for rep in range(2):
        X, g = _adjoint(plan, zg)
        assert torch.equal(X, Xs) and torch.equal(g, gs), rep
    del fill
    torch.cuda.empty_cache()
    X, g = _adjoint(plan, zg)
    assert torch.equal(X, Xs) and (g - gs).abs().max() <= 1e-12 * gs.abs().max()


def test_short_calls_bitwise():
    """Calls of one to nine steps, which run one launch per stage where that is
    faster (many paths), and the short end of a longer one: as the stage kernel."""
    lb = _basis(6, 4, 20)
    b = np.linspace(0.3, 6.0, 256)
    zg = np.linspace(-3.0, 0.5, 68) ** 3 / 9.0
    auto = W.wpccc_plan_create(lb, b, 1.5)
    ref = W.wpccc_plan_create(lb, b, 1.5, stage_rows=4, stage_launch=W.WPCCC_LAUNCH_STAGES)
    print(f"split {W.wpccc_plan_stage_split(auto)}", flush=True)
    for steps in (1, 2, 3, 5, 9, 66):
        assert np.array_equal(_run(auto, zg[:steps + 1]), _run(ref, zg[:steps + 1])), steps


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_nonfinite_path_stays_alone(value):
    """A non-finite amplitude of one path, on every split: that path ends
    non-finite and is reported, the others are as without it, bitwise."""
    zg = np.linspace(-2.0, 1.0, 20)
    plan = W.wpccc_plan_create(_basis(5, 4, 4), [0.4, 1.5, 6.0], 1.5, stage_rows=4, stage_launch=W.WPCCC_LAUNCH_STAGES)
    ref = _run(plan, zg)
    for g, paths in _splits(plan):
        X = torch.zeros((3, plan.n_pad), dtype=torch.complex128, device="cuda")
        X[:, 0] = 1.0
        X[1, 7] = value
        W.wpccc_propagate(plan, zg, X)
        with pytest.raises(W.WpcccError) as e:
            W.wpccc_plan_status(plan)
        assert e.value.code == -5, (g, paths)
        X = X.cpu().numpy()
        assert np.array_equal(X[[0, 2]], ref[[0, 2]]) and not np.isfinite(X[1]).all(), (g, paths)


def test_chunks_among_other_calls():
    """Propagations by the persistent kernel with single steps, short calls and
    an adjoint between them (calls that do not advance its tags): bitwise the
    stage kernel's amplitudes throughout."""
    lb, b = _basis(6, 4, 20), np.array([0.5, 1.5, 3.0, 5.0])
    zg = np.arange(140) / 16.0 - 4.0
    out = []
    for split in (0, 8):
        plan = W.wpccc_plan_create(lb, b, 1.5, model_a=0.5, model_c=1.2, stage_rows=8, stage_launch=W.WPCCC_LAUNCH_STAGES)
        W.wpccc_plan_set_stage_split(plan, split)
        X = torch.zeros((4, plan.n_pad), dtype=torch.complex128, device="cuda")
        X[:, 0] = 1.0
        seen = []
        for lo, hi in ((0, 1), (1, 67), (67, 68), (68, 139)):
            W.wpccc_propagate(plan, zg[lo:hi + 1], X)
            seen.append(X.clone())
            for _ in range(3):
                W.wpccc_step(plan, X, zg[hi], 0.0625)
            seen.append(X.clone())
            seen.append(_adjoint(plan, zg[lo:hi + 1])[0])
        W.wpccc_plan_status(plan)
        out.append([t.cpu().numpy() for t in seen])
    assert all(np.array_equal(x, y) for x, y in zip(*out))
