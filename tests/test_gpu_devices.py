"""Plans on two devices of one process: kernels that request more LDS than the
default must be allowed to on each device they run on."""
import numpy as np
import pytest
import torch

import paper_2403_04252_amd as W

pytestmark = pytest.mark.gpu


@pytest.mark.skipif(torch.cuda.device_count() < 2, reason="needs two devices")
def test_large_lds_on_the_second_device():
    lb = W.wpccc_basis(W.BasisSpec(6, 4, 20, 3.0, 300, 60.0, 1.0))
    rng = np.random.default_rng(1)
    A = np.eye(500) + (rng.standard_normal((500, 500)) + 1j * rng.standard_normal((500, 500))) * 0.02
    out = []
    for dev in range(2):
        with torch.cuda.device(dev):
            plan = W.wpccc_plan_create(lb, [0.5, 2.0], 1.5)
            X = torch.zeros((2, plan.n_pad), dtype=torch.complex128, device="cuda")
            X[:, 0] = 1.0
            W.wpccc_propagate(plan, np.linspace(-2.0, 2.0, 41), X)
            W.wpccc_plan_status(plan)
            At = torch.as_tensor(np.ascontiguousarray(A.T[None]), device="cuda")
            Y = torch.empty_like(At)
            W.wpccc_zgesv_batched(At, torch.ones_like(At), Y)
            out.append((X.cpu(), Y.cpu()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
