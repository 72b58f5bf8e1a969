"""The persistent chunk kernel's wait for the other workgroups of a path: what
a give-up leaves behind, and other streams' work beside it.  The give-up is
forced from the host by a limit of no polls; every kernel ends normally."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import paper_2403_04252_amd as W

pytestmark = pytest.mark.gpu


def _basis(n_max, l_max, n_bins):
    return W.wpccc_basis(W.BasisSpec(n_max, l_max, n_bins, 3.0, 300, 60.0, 1.0))


def _start(plan):
    X = torch.zeros((plan.n_traj, plan.n_pad), dtype=torch.complex128, device="cuda")
    X[:, 0] = 1.0
    return X


def _spin(plan, polls):
    f = W.load_library().wpccc_internal_chunk_spin
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_int], ctypes.c_int
    assert f(plan.handle, polls) == 0


def _tune(plan):
    f = W.load_library().wpccc_internal_tune
    f.argtypes, f.restype = [ctypes.c_void_p, ctypes.c_void_p], ctypes.c_int
    assert f(plan.handle, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0


@pytest.fixture(scope="module")
def n580():
    return _basis(6, 4, 20)


def test_give_up_is_reported_once(n580):
    """A workgroup that gives up latches WPCCC_EHIP and leaves the amplitudes
    of its chunk as they were; the next call runs as if nothing had been."""
    zg = np.linspace(-3.0, 0.0, 71)
    plan = W.wpccc_plan_create(n580, [0.5, 2.0, 5.0], 1.5, stage_rows=8, stage_launch=W.WPCCC_LAUNCH_STAGES)
    ref = _start(plan)
    W.wpccc_propagate(plan, zg, ref)
    W.wpccc_plan_set_stage_split(plan, 8)
    _spin(plan, 0)
    X = _start(plan)
    W.wpccc_propagate(plan, zg, X)
    with pytest.raises(W.WpcccError) as e:
        W.wpccc_plan_status(plan)
    assert e.value.code == -3
    assert torch.equal(X, _start(plan))
    W.wpccc_plan_status(plan)   # read once
    _spin(plan, -1)
    W.wpccc_propagate(plan, zg, X)
    W.wpccc_plan_status(plan)
    assert torch.equal(X, ref)


def test_tuning_leaves_no_error(n580):
    """Splits whose workgroups gave up while they were timed are not chosen and
    leave no error on the plan."""
    zg = np.linspace(-3.0, 0.0, 71)
    plan = W.wpccc_plan_create(n580, [0.5, 2.0, 5.0], 1.5)
    _spin(plan, 0)
    _tune(plan)
    assert W.wpccc_plan_stage_split(plan)[0] <= 1
    W.wpccc_plan_status(plan)
    ref = _start(plan)
    W.wpccc_propagate(plan, zg, ref)
    W.wpccc_plan_status(plan)
    _spin(plan, -1)
    _tune(plan)
    X = _start(plan)
    W.wpccc_propagate(plan, zg, X)
    W.wpccc_plan_status(plan)
    assert torch.equal(X, ref)


def test_plans_on_their_own_streams(n580):
    """Three plans, each with workgroups that wait for each other, propagated
    from three threads on three streams."""
    zg = np.linspace(-3.0, 3.0, 101)
    specs = [(n580, 32, 8), (n580, 8, 24), (_basis(8, 7, 26), 2, 86)]
    plans, refs = [], []
    for lb, n, g in specs:
        plan = W.wpccc_plan_create(lb, np.linspace(0.3, 6.0, n), 1.5, stage_rows=4, stage_launch=W.WPCCC_LAUNCH_STAGES)
        ref = _start(plan)
        W.wpccc_propagate(plan, zg, ref)
        W.wpccc_plan_set_stage_split(plan, g)
        assert W.wpccc_plan_stage_split(plan)[0] > 1
        plans.append(plan)
        refs.append(ref)
    torch.cuda.synchronize()
    bad = []

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for rep in range(8):
                X = _start(plans[i])
                W.wpccc_propagate(plans[i], zg, X)
                stream.synchronize()
                try:
                    W.wpccc_plan_status(plans[i])
                except W.WpcccError as e:
                    bad.append((i, rep, str(e)))
                if not torch.equal(X, refs[i]):
                    bad.append((i, rep, "amplitudes differ"))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_beside_a_full_device(n580):
    """A propagation whose workgroups wait for each other, while another
    stream's propagation of 40000 paths keeps every CU occupied."""
    zg = np.linspace(-3.0, 3.0, 129)
    many = W.wpccc_plan_create(_basis(2, 1, 3), np.linspace(0.3, 6.0, 40000), 1.5, stage_rows=4,
                               stage_launch=W.WPCCC_LAUNCH_STAGES)
    W.wpccc_plan_set_stage_split(many, 1)
    plan = W.wpccc_plan_create(n580, np.linspace(0.3, 6.0, 32), 1.5, stage_rows=8, stage_launch=W.WPCCC_LAUNCH_STAGES)
    ref = _start(plan)
    W.wpccc_propagate(plan, zg, ref)
    W.wpccc_plan_set_stage_split(plan, 8)
    XM, X = _start(many), _start(plan)
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    W.wpccc_propagate(many, zg, XM, stream=s1)
    W.wpccc_propagate(plan, zg, X, stream=s2)
    torch.cuda.synchronize()
    W.wpccc_plan_status(plan)
    W.wpccc_plan_status(many)
    assert torch.equal(X, ref) and torch.isfinite(XM.abs()).all()


def test_captured_calls_do_not_wait(n580):
    """A propagation and an adjoint captured into the caller's graphs, replayed
    on two streams beside each other: no workgroup of them waits for another
    (with a limit of no polls any wait would be an error), and every replay
    gives the eager amplitudes bitwise."""
    zg = np.linspace(-3.0, 0.0, 71)
    plans, refs, graphs, outs, streams = [], [], [], [], []
    for n in (3, 5):
        plan = W.wpccc_plan_create(n580, np.linspace(0.5, 5.0, n), 1.5, model_a=0.4, model_c=1.1, stage_rows=8,
                                   stage_launch=W.WPCCC_LAUNCH_STAGES)
        W.wpccc_plan_set_stage_split(plan, 8)
        ref, Xa, grad = _start(plan), torch.empty_like(_start(plan)), torch.empty((n, 3), dtype=torch.float64, device="cuda")
        gX = _start(plan)
        W.wpccc_propagate(plan, zg, ref)
        W.wpccc_adjoint(plan, zg, _start(plan), gX, grad, Xa)   # allocates its workspace
        W.wpccc_plan_status(plan)
        assert torch.equal(Xa, ref)
        W.wpccc_plan_set_stage_split(plan, 0)
        W.wpccc_adjoint(plan, zg, _start(plan), gX, grad, Xa)   # as it will run in the graph
        want = grad.clone()
        W.wpccc_plan_set_stage_split(plan, 8)
        _spin(plan, 0)
        X0, X = _start(plan), _start(plan)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            W.wpccc_propagate(plan, zg, X)
            W.wpccc_adjoint(plan, zg, X0, gX, grad, Xa)
        plans.append(plan)
        refs.append(ref)
        graphs.append(graph)
        outs.append((X, Xa, grad, X0, gX, want))
        streams.append(torch.cuda.Stream())
    for rep in range(4):
        for X, Xa, grad, *_ in outs:
            grad.fill_(float("nan"))
            X.zero_()
            X[:, 0] = 1.0
            Xa.fill_(float("nan"))
        torch.cuda.synchronize()
        for graph, stream in zip(graphs, streams):
            with torch.cuda.stream(stream):
                graph.replay()
        torch.cuda.synchronize()
        for plan, ref, (X, Xa, grad, _, _, want) in zip(plans, refs, outs):
            W.wpccc_plan_status(plan)
            assert torch.equal(X, ref) and torch.equal(Xa, ref), rep
            assert torch.equal(grad, want), rep
