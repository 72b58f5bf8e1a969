"""The batched solve at the edges of its blocks: n at and beside 16 columns,
32 rows and the largest n whose columns stay on chip (544), odd batches, and a
singular matrix reported by its number.

Bar: LU with partial pivoting solves (A + E) X = B with |E| <= 3 n eps |L||U|,
and |L||U| of a random matrix is a small multiple of |A|: the residual is held
to 10 n eps (|A| |X| + |B|), row sums against the largest element."""
import numpy as np
import pytest
import torch

import paper_2403_04252_amd as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(2, 1), (15, 3), (16, 9), (17, 2), (31, 3), (32, 1), (33, 5), (543, 1), (544, 3), (545, 2)])
def test_solve_edges(n, batch):
    print(f"n = {n}, batch {batch}", flush=True)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((batch, n, n)) + 1j * rng.standard_normal((batch, n, n))
    B = rng.standard_normal((batch, n, n)) + 1j * rng.standard_normal((batch, n, n))
    At = torch.as_tensor(np.ascontiguousarray(A.transpose(0, 2, 1)), device="cuda")
    Bd = torch.as_tensor(B, device="cuda")
    X = torch.full_like(Bd, float("nan"))
    W.wpccc_zgesv_batched(At, Bd, X)
    X = X.cpu().numpy()
    assert np.array_equal(At.cpu().numpy(), A.transpose(0, 2, 1)) and np.array_equal(Bd.cpu().numpy(), B)
    for b in range(batch):
        res = np.abs(A[b] @ X[b] - B[b]).max()
        bar = 10 * n * np.finfo(float).eps * (np.abs(A[b]).sum(1).max() * np.abs(X[b]).max() + np.abs(B[b]).max())
        print(f"  residual {res:.1e}, bar {bar:.1e}", flush=True)
        assert res <= bar


def test_singular_matrix_is_named():
    A = np.stack([np.eye(40, dtype=complex) * (i + 1) for i in range(5)])
    A[3][:, 17] = 0.0
    At = torch.as_tensor(np.ascontiguousarray(A.transpose(0, 2, 1)), device="cuda")
    with pytest.raises(W.WpcccError) as e:
        W.wpccc_zgesv_batched(At, torch.ones_like(At), torch.empty_like(At))
    assert "matrix 3" in str(e.value) and "column 17" in str(e.value)


def _lu(A):
    """LU with the library's pivots (largest |a|^2) in panels of 16 columns."""
    A, n = A.copy(), len(A)
    p = np.arange(n)
    for k0 in range(0, n, 16):
        k1 = min(k0 + 16, n)
        for j in range(k0, k1):
            i = j + np.argmax(A[j:, j].real ** 2 + A[j:, j].imag ** 2)
            if i != j:
                A[[i, j]], p[[i, j]] = A[[j, i]], p[[j, i]]
            A[j + 1:, j] *= np.conj(A[j, j]) / (A[j, j].real ** 2 + A[j, j].imag ** 2)
            A[j + 1:, j + 1:k1] -= np.outer(A[j + 1:, j], A[j, j + 1:k1])
        for j in range(k0, k1):
            A[j + 1:k1, k1:] -= np.outer(A[j + 1:k1, j], A[j, k1:])
        A[k1:, k1:] -= A[k1:, k0:k1] @ A[k0:k1, k1:]
    return A, p


def _substitute(F, Y):
    """Both substitutions, every element rounded once per term."""
    Y, n = Y.copy(), len(F)
    for k in range(n):
        Y[k + 1:] -= F[k + 1:, k][:, None] * Y[k][None]
    for k in range(n - 1, -1, -1):
        Y[k] *= np.conj(F[k, k]) / (F[k, k].real ** 2 + F[k, k].imag ** 2)
        Y[:k] -= F[:k, k][:, None] * Y[k][None]
    return Y


def _exact(A, B, X):
    """Solution refined with residuals in extended precision."""
    Al, x = A.astype(np.clongdouble), X.astype(np.clongdouble)
    for _ in range(3):
        r = B.astype(np.clongdouble) - np.stack([(Al * x[:, c][None]).sum(1) for c in range(x.shape[1])], 1)
        x = x + np.linalg.solve(A, r.astype(complex))
    return x


@pytest.mark.parametrize("n", [128, 256, 442, 600])
def test_solve_error_of_one_rounding_per_term(n):
    """Overlap-like systems: the error of the solution is no larger than with
    the sums of the substitutions rounded once per term (in numpy, from
    factors with the same pivots; root mean square over 48 columns of four
    systems, 5% for the spread between systems)."""
    got, model = [], []
    for seed in range(4):
        rng = np.random.default_rng(seed)
        z = lambda s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
        A, B = np.eye(n) + z((n, n)) * (0.4 / np.sqrt(n)), z((n, n))
        At = torch.as_tensor(np.ascontiguousarray(A.T[None]), device="cuda")
        X = torch.empty_like(At)
        W.wpccc_zgesv_batched(At, torch.as_tensor(B[None], device="cuda"), X)
        X = X.cpu().numpy()[0][:, :48]
        F, p = _lu(A)
        V = _substitute(F, B[p][:, :48])
        x = _exact(A, B[:, :48], V)
        got.append(float((np.abs(X - x) ** 2).mean()))
        model.append(float((np.abs(V - x) ** 2).mean()))
    ratio = np.sqrt(np.sum(got) / np.sum(model))
    print(f"n = {n}: error {np.sqrt(np.mean(got)):.2e}, {ratio:.2f} of one rounding per term", flush=True)
    assert ratio <= 1.05


@pytest.mark.parametrize("n,batch", [(5, 3), (33, 2), (600, 1)])
def test_solve_of_arrays_at_any_place(n, batch):
    """Matrices that start 8 bytes past a multiple of 16, and X in the place of
    B or across it: the bits of the solve of arrays of their own."""
    rng = np.random.default_rng(n)
    z = lambda: rng.standard_normal((batch, n, n)) + 1j * rng.standard_normal((batch, n, n))
    A, B, size = z(), z(), 2 * batch * n * n
    At, Bt = (torch.as_tensor(np.ascontiguousarray(m), device="cuda") for m in (A.transpose(0, 2, 1), B))
    X = torch.empty_like(Bt)
    W.wpccc_zgesv_batched(At, Bt, X)
    ref = torch.view_as_real(X).flatten()
    flat = lambda t: torch.view_as_real(t).flatten()
    solve = W.load_library().wpccc_zgesv_batched
    stream = torch.cuda.current_stream().cuda_stream
    for a, b, x in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1)):
        bufs = [torch.full((size + 1,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(3)]
        va, vb, vx = (t[o:o + size] for t, o in zip(bufs, (a, b, x)))
        va.copy_(flat(At))
        vb.copy_(flat(Bt))
        assert solve(n, batch, va.data_ptr(), vb.data_ptr(), vx.data_ptr(), stream) == 0
        assert torch.equal(vx, ref) and torch.equal(vb, flat(Bt)), (a, b, x)
    for shift in (0, 1, 2, size // 2):
        both = torch.empty(size + shift, dtype=torch.float64, device="cuda")
        both[shift:].copy_(flat(Bt))
        assert solve(n, batch, At.data_ptr(), both[shift:].data_ptr(), both.data_ptr(), stream) == 0
        assert torch.equal(both[:size], ref), shift
