"""The FP64 contraction at the edges of its tiles: one radial function, counts
just below and above a group of eight and a tile of 32, tiles of unequal size,
every number of weights (2, 4, 6, 8 and 12 per block: one and two centres'
bases, prior and dagger form), odd numbers of nodes (no 16-byte rows) and node
ranges that end inside a chunk.

S and H element-wise against the oracle within 1e-11 max|X|, the bar of the
other coupling checks (same quadrature, other summation order); the FP32
products within their 1e-5."""
import numpy as np
import pytest
import torch

import paper_2403_04252_amd as W
from oracle.radial import BasisSpec as OSpec, build_basis
from oracle.twocentre import Q_DAGGER, Q_PRIOR, two_centre_matrices

pytestmark = pytest.mark.gpu

# (n_max, l_max, n_bins) of target and projectile: n_max - l + n_bins functions per l
CASES = [
    ((1, 0, 0), (1, 0, 0), Q_DAGGER, 9, 11),
    ((2, 0, 6), (3, 1, 6), Q_PRIOR, 17, 19),        # 8; 9 + 8
    ((3, 0, 30), (2, 0, 30), Q_DAGGER, 16, 20),     # 33 and 32
    ((4, 1, 14), (4, 1, 14), Q_PRIOR, 15, 21),      # 18 + 17 on both centres: two tiles of the diagonal blocks
    ((5, 2, 21), (4, 2, 5), Q_PRIOR, 24, 27),       # 75 = 3 uneven tiles against 24
    ((6, 2, 29), (6, 2, 29), Q_DAGGER, 16, 25),     # 102, 67 and 33 on both centres
]


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("tspec,pspec,ql,n_eta,n_tau", CASES)
def test_contraction_edges(tspec, pspec, ql, n_eta, n_tau, mixed):
    tail = (4.0, 400, 40.0, 1.0)
    lt, ot = W.wpccc_basis(W.BasisSpec(*tspec, *tail)), build_basis(OSpec(*tspec, *tail))
    lp, op = (lt, ot) if pspec == tspec else (W.wpccc_basis(W.BasisSpec(*pspec, *tail)), build_basis(OSpec(*pspec, *tail)))
    b, z, v = 1.3, -0.8, 1.2
    q = W.WPCCC_Q_PRIOR if ql == Q_PRIOR else W.WPCCC_Q_DAGGER
    plan = W.wpccc_plan_create_2c([lt], [lp], 0, [b], [v], q_lower=q, n_eta=n_eta, n_tau=n_tau, mixed=mixed)
    N, _ = W.wpccc_plan_path_info(plan, 0)
    print(f"{tspec} {pspec} {ql}: N = {N}, {n_eta} x {n_tau} nodes", flush=True)
    H = torch.empty((N, N), dtype=torch.complex128, device="cuda")
    S = torch.empty((N, N), dtype=torch.complex128, device="cuda")
    W.wpccc_couplings(plan, 0, z, H, S)
    torch.cuda.synchronize()
    W.wpccc_plan_status(plan)
    So, Ho = two_centre_matrices(ot, op, b, z, v, n_eta, n_tau, q_lower=ql)
    for name, g, o in (("S", S, So), ("H", H, Ho)):
        err = np.abs(g.cpu().numpy() - o).max() / np.abs(o).max()
        print(f"  {name} {err:.1e}", flush=True)
        assert err <= (1e-5 if mixed else 1e-11)


@pytest.mark.parametrize("pspec", [(6, 3, 20), (5, 2, 9)])
def test_contraction_tiles_of_three_row_groups(pspec):
    """Blocks of 98 functions, split into tiles of 32, 24, 24 and 18 rows, with
    two (above the diagonal of equal bases) and six weights: tiles of three
    row groups, next to others of the same block.  Bar as above."""
    tail, tspec = (4.0, 400, 40.0, 1.0), (6, 3, 20)
    lt, ot = W.wpccc_basis(W.BasisSpec(*tspec, *tail)), build_basis(OSpec(*tspec, *tail))
    lp, op = (lt, ot) if pspec == tspec else (W.wpccc_basis(W.BasisSpec(*pspec, *tail)), build_basis(OSpec(*pspec, *tail)))
    plan = W.wpccc_plan_create_2c([lt], [lp], 0, [1.3], [1.2], q_lower=W.WPCCC_Q_PRIOR, n_eta=12, n_tau=16)
    N, _ = W.wpccc_plan_path_info(plan, 0)
    print(f"{tspec} {pspec}: N = {N}", flush=True)
    H, S = (torch.empty((N, N), dtype=torch.complex128, device="cuda") for _ in range(2))
    W.wpccc_couplings(plan, 0, -0.8, H, S)
    W.wpccc_plan_status(plan)
    So, Ho = two_centre_matrices(ot, op, 1.3, -0.8, 1.2, 12, 16, q_lower=Q_PRIOR)
    for name, g, o in (("S", S, So), ("H", H, Ho)):
        err = np.abs(g.cpu().numpy() - o).max() / np.abs(o).max()
        print(f"  {name} {err:.1e}", flush=True)
        assert err <= 1e-11
