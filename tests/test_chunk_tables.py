"""Index tables of the persistent chunk kernel (chunk_split), checked and run on
the host: for every split that a plan may take, every position lies inside its
LDS array, every state, table entry and output is covered once, and the sums
that the tables describe, carried out here in numpy with the kernel's lane
layouts, give y = G F x' of the dense formula.

Tolerance: both are sums of the same products in another order, each of at
most a few thousand terms of order one: 1e-11 of the largest."""
import ctypes
import os

import numpy as np
import pytest

import paper_2403_04252_amd as W

CHAINS = 8
K_MAX_L = 10
K_RPOW = 2 * (2 * K_MAX_L + 1)
K_MAX_PB = (2 * K_MAX_L + 1) * (2 * K_MAX_L + 2) // 2
MAX_LDS = 160 * 1024 - 1024
SPLITS = [1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 80, 96]

# (n_max, l_max, n_bins): N_l = max(n_max - l, 0) + n_bins
BASES = [(1, 0, 0), (1, 0, 3), (2, 1, 2), (3, 2, 6), (3, 2, 8), (5, 4, 4), (4, 3, 21), (6, 4, 20), (7, 6, 10), (8, 7, 26),
         (10, 6, 32), (10, 7, 32), (2, 8, 1)]


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(W.library_path()):
        from paper_2403_04252_amd.build import build_library
        build_library()
    lib = W.load_library()
    pi = ctypes.POINTER(ctypes.c_int)
    lib.wpccc_internal_chunk_tables.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, pi, ctypes.c_int]
    lib.wpccc_internal_chunk_tables.restype = ctypes.c_int
    return lib


def _tables(lib, basis, G, threads):
    f = lib.wpccc_internal_chunk_tables
    n = f(basis.handle, G, threads, None, 0)
    if n == 0:
        return None
    a = np.zeros(n, dtype=np.int32)
    assert f(basis.handle, G, threads, a.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), n) == n
    t = dict(zip(("G", "nt", "fp", "smem", "n_xs"), a[:5].tolist()))
    at = 13
    for name, ln, cols in zip(("wgs", "ents", "jobs", "grps", "outs", "jlane", "gsrc", "xpos"), a[5:13].tolist(),
                              (32, 2, 4, 2, 4, 2, 1, 1)):
        part = a[at:at + ln]
        t[name] = part if cols == 1 else part.reshape(-1, cols)
        at += ln
    assert at == n
    return t


class Layout:
    """Row layouts of the moment table and the angular factors (struct Meta)."""

    def __init__(self, n_l):
        L = len(n_l) - 1
        self.n_l, self.l_max = n_l, L
        self.state_off = np.concatenate([[0], np.cumsum([(2 * l + 1) * n for l, n in enumerate(n_l)])])
        self.nV = [sum((min(l, p) + 1) * n_l[l] for l in range(L + 1)) for p in range(L + 1)]
        self.gcols = [sum((min(l, p) + 1) * (2 * l + 1) for l in range(L + 1)) for p in range(L + 1)]
        self.frow_off = np.concatenate([[0], np.cumsum([n_l[p] * self.nV[p] for p in range(L + 1)])])
        self.g_off = np.concatenate([[0], np.cumsum([(2 * p + 1) * self.gcols[p] for p in range(L + 1)])])

    def dense(self, F, G, x):
        """y by state, F[n_frow], G[n_g], x[n_states]; and lambda of every entry."""
        y = np.zeros(int(self.state_off[-1]))
        lam = np.zeros(int(self.frow_off[-1]), dtype=int)
        for p in range(self.l_max + 1):
            n = self.n_l[p]
            Fp = F[self.frow_off[p]:self.frow_off[p + 1]].reshape(n, self.nV[p])
            lp = lam[self.frow_off[p]:self.frow_off[p + 1]].reshape(n, self.nV[p])
            Gp = G[self.g_off[p]:self.g_off[p + 1]].reshape(2 * p + 1, self.gcols[p])
            Wp = np.zeros((n, self.gcols[p]))
            e = g = 0
            for l in range(self.l_max + 1):
                xl = x[self.state_off[l]:self.state_off[l + 1]].reshape(2 * l + 1, self.n_l[l])
                for k in range(min(l, p) + 1):
                    Wp[:, g:g + 2 * l + 1] = Fp[:, e:e + self.n_l[l]] @ xl.T
                    lp[:, e:e + self.n_l[l]] = abs(l - p) + 2 * k
                    e, g = e + self.n_l[l], g + 2 * l + 1
            y[self.state_off[p]:self.state_off[p + 1]] = (Gp @ Wp.T).ravel()
        return y, lam


def _u16(v):
    return v & 0xffff, (v >> 16) & 0xffff


def _run_workgroup(t, w, F, G, x, lay_lam):
    """One workgroup's sums by its tables; returns {state: y}."""
    nt, n_xs = t["nt"], t["n_xs"]
    (ent0, n_ent, job0, n_jobs, grp0, n_grp, out0, n_out, g0, n_g, rad0, n_rad, n_f, n_w, kb) = w[:15].tolist()
    wave_job = w[15:32]
    waves = nt // 64
    halves = waves // CHAINS
    # LDS layout as the kernel lays it out, in doubles
    lds = 2 * (n_xs + n_w + CHAINS * n_out + 2 * n_rad) + nt // CHAINS * n_grp + n_f + n_g
    assert lds % 2 == 0 and n_f % 2 == 0, "16-byte loads of F and of the R factors"
    assert (lds + K_RPOW + K_MAX_PB + 1) % 2 == 0, "16-byte loads of the job headers"
    assert 8 * (lds + K_RPOW + K_MAX_PB + 1 + 66 * n_jobs) <= t["smem"] <= MAX_LDS
    assert 0 < n_out <= nt and 0 < n_rad <= nt and n_ent <= t["fp"] * nt and n_f < 1 << 20 and n_w <= 0xffff
    # NaN past x': a product with it must not reach an output
    xs = np.zeros(n_xs)
    xs[t["xpos"]] = x
    Ws, Fs = np.zeros(n_w), np.zeros(n_f)
    ents = t["ents"][ent0:ent0 + n_ent]
    pos, lam = ents[:, 1] & 0xfffff, ents[:, 1] >> 20
    assert (ents[:, 1] >= 0).all() and (pos < n_f).all() and np.unique(pos).size == n_ent
    assert (lam == lay_lam[ents[:, 0]]).all()
    Fs[pos] = F[ents[:, 0]]
    assert wave_job[0] == 0 and (np.diff(wave_job[:waves + 1]) >= 0).all() and wave_job[waves] == n_jobs
    lane = np.arange(64)
    written = []
    for q in range(job0, job0 + n_jobs):
        fx, xy, z, nu = t["jobs"][q].tolist()
        stride, np_ = z & 0xffff, z >> 16
        assert 1 <= nu <= 4 and fx % 128 == 0 and fx + 128 * np_ <= n_f
        rows = 4 * (nu - 1) + 4
        if np_:
            assert xy + (rows - 1) * stride + 8 * np_ <= n_xs, "x' read past its array"
        A = Fs[fx:fx + 128 * np_].reshape(np_, 4, 16, 2).transpose(2, 0, 3, 1).reshape(16, 8 * np_)
        idx = xy + np.arange(rows)[:, None] * stride + np.arange(8 * np_)[None, :]
        Wj = A @ xs[idx].T if np_ else np.zeros((16, rows))
        jl = t["jlane"][64 * q:64 * q + 64]
        p4 = [*_u16(jl[:, 0]), *_u16(jl[:, 1])]
        for u in range(nu):
            assert (p4[u] < n_w).all()
            Ws[p4[u]] = Wj[4 * ((lane & 15) >> 2) + (lane >> 4), 4 * u + (lane & 3)]
            written.append(p4[u][p4[u] < n_w - 64])
    written = np.concatenate(written)
    assert np.unique(written).size == written.size, "a W position written twice"
    Ws[n_w - 64:] = np.nan   # the lanes' positions that nothing reads
    Gs = np.where(t["gsrc"][g0:g0 + n_g] >= 0, G[np.maximum(t["gsrc"][g0:g0 + n_g], 0)], 0.0)
    assert Gs.size == n_g
    y = np.zeros(n_out)
    hit = np.zeros(n_out, dtype=int)
    step = 16 * np.arange(CHAINS * kb)
    blk, k, r = (lane & 15) >> 2, lane >> 4, lane & 3
    for q in range(grp0, grp0 + halves * n_grp):
        g = t["grps"][64 * q:64 * q + 64]
        wp, gp = _u16(g[:, 0])
        live = g[:, 1] >= 0
        if not live.any():
            continue
        assert (wp + step[-1] < n_w).all() and (gp + step[-1] < n_g).all()
        Wv, Gv = Ws[wp[:, None] + step], Gs[gp[:, None] + step]
        a, b = np.zeros((4, 4, 4, step.size)), np.zeros((4, 4, 4, step.size))
        a[blk, r, k], b[blk, r, k] = Wv, Gv
        out = np.einsum("zrks,zcks->zrc", a, b)
        o = g[live, 1]
        assert (o < n_out).all()
        y[o] = out[blk, k, r][live]
        hit[o] += 1
    assert (hit == 1).all(), "an output summed not once"
    outs = t["outs"][out0:out0 + n_out]
    assert (outs[:, 1] < n_rad).all() and (outs[:, 2] == t["xpos"][outs[:, 0]]).all()
    return outs[:, 0], outs[:, 1] + rad0, y


def _bytes_of_grps(t):
    return (t["grps"].shape[0] % 64, t["jlane"].shape[0] % 64)


@pytest.mark.parametrize("threads", [512, 1024])
@pytest.mark.parametrize("n_max,l_max,n_bins", BASES)
def test_split_tables(lib, n_max, l_max, n_bins, threads):
    basis = W.wpccc_basis(W.BasisSpec(n_max, l_max, n_bins, 3.0, 60, 60.0, 1.0))
    st = W.wpccc_basis_export(basis)
    n_l = [int(((st["l"] == l) & (st["m"] == -l)).sum()) for l in range(l_max + 1)]
    lay = Layout(n_l)
    N = int(lay.state_off[-1])
    assert N == st["l"].size
    rng = np.random.default_rng(N)
    F, G, x = rng.standard_normal(int(lay.frow_off[-1])), rng.standard_normal(int(lay.g_off[-1])), rng.standard_normal(N)
    ref, lam = lay.dense(F, G, x)
    seen = set()
    for want in SPLITS:
        t = _tables(lib, basis, want, threads)
        if t is None or t["G"] in seen:
            continue
        seen.add(t["G"])
        assert t["G"] <= want and t["nt"] == threads and len(t["wgs"]) == t["G"] and _bytes_of_grps(t) == (0, 0)
        assert np.unique(t["xpos"]).size == N and t["xpos"].max() < t["n_xs"]
        y = np.full(N, np.nan)
        for w in t["wgs"]:
            s, rad, v = _run_workgroup(t, w, F, G, x, lam)
            assert np.isnan(y[s]).all(), "a state in two workgroups"
            assert (rad == st["a"][s]).all()
            y[s] = v
        assert np.abs(y - ref).max() <= 1e-11 * max(np.abs(ref).max(), 1.0)
    print(f"N = {N}, {threads} threads: splits {sorted(seen)}")
    assert seen or N > 1800   # large bases: entries per thread and LDS leave few splits or none
