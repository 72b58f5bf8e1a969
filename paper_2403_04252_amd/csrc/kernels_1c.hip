// HIP kernels of the one-centre path on gfx950 (64-wide waves, FP64).
//
// One RK4 stage of Algorithm 1 for every path of the batch is one launch of
// k_stage: from (b, z, v) and the basis tables it forms, per workgroup, the
// part of M(z) = -(i/v) Zp D_T(b, z) it needs and applies it to the stage
// input, then writes the RK4 combination of that stage.  k_chunk runs the
// same stages for up to 64 steps in one persistent launch on MFMA, forwards
// or, for the adjoint, backwards; k_apply and k_grad apply M and its
// derivatives for the adjoint.  D_T (Eq. D1) is
// never formed: its (l'm', lm) block is sum_lambda c Pbar_lambda^|m'-m| F_lambda
// with F_lambda the N_l' x N_l matrix of Eq. D2 radial integrals, so
//   y_{l'm'}[n'] = sum_{l, lambda, q} G_l'[m'][(l,lambda), q] sum_n F_l'[n'][(l,lambda), n] x'_{l q n}
// with x' = conj(phase) u (interaction picture).
//
// Radial integrals at the exact R.  For the grid quadrature of Eq. D2
//   F(R) = sum_i w_i r_i^2 f_a f_b min(r_i,R)^lam / max(r_i,R)^(lam+1)
//        = R^-(lam+1) A_k + R^lam B_(k+1),
//   A_k = sum_{i<=k} w_i r_i^(2+lam) f_a f_b,   B_k = sum_{i>=k} w_i r_i^(1-lam) f_a f_b,
// with k the last node r_k <= R: the multipole kernel factorises into a power
// of r times a power of R on either side of R.  k_moments tabulates A and B
// once per basis; per R each integral costs one 16-byte load and two
// multiplies instead of an n_r-term sum.  It is the same quadrature, summed
// in a different association order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "plan.h"

namespace wpccc {

namespace {

// The arithmetic that the stage kernels (one launch per stage) and the
// persistent chunk kernel share is written with explicit fused operations, so
// that both round alike whatever the compiler contracts around them.
__device__ inline double2 cmul(double2 a, double2 b) {
    return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.x, b.y, a.y * b.x));
}
// conj(ph) u
__device__ inline double2 dephase(double2 ph, double2 u) {
    return make_double2(__builtin_fma(ph.x, u.x, ph.y * u.y), __builtin_fma(ph.x, u.y, -(ph.y * u.x)));
}
// F at R from a table entry and the two R factors of its multipole
__device__ inline double radial_f(double a, double b, double fa, double fb) {
    return __builtin_fma(a, fa, b * fb);
}

// Partial moments, one thread per Frow entry d = (a, b, lambda); phiT is [n_r+1][n_f].
//   tab[k][d].x = A_k     = sum_{i=1..k}      w_i r_i^(2+lam) f_a(r_i) f_b(r_i)
//   tab[k][d].y = B_(k+1) = sum_{i=k+1..n_r}  w_i r_i^(1-lam) f_a(r_i) f_b(r_i)
__global__ void k_moments(const double* __restrict__ r, const double* __restrict__ w,
                          const double* __restrict__ phiT, const int* __restrict__ da,
                          const int* __restrict__ db, const int* __restrict__ dl, int n_r, int n_f,
                          int n_frow, double2* __restrict__ tab) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= n_frow) return;
    const int a = da[d], b = db[d], lam = dl[d];
    double A = 0.0;
    tab[d].x = 0.0;
    for (int i = 1; i <= n_r; ++i) {
        const double ri = r[i];
        double p = ri * ri;
        for (int q = 0; q < lam; ++q) p *= ri;
        A += w[i] * p * phiT[(size_t)i * n_f + a] * phiT[(size_t)i * n_f + b];
        tab[(size_t)i * n_frow + d].x = A;
    }
    double B = 0.0;
    tab[(size_t)n_r * n_frow + d].y = 0.0;
    for (int i = n_r; i >= 1; --i) {
        const double ri = r[i];
        double p;  // r^(1 - lam)
        if (lam == 0) {
            p = ri;
        } else {
            double q = 1.0;
            for (int s = 1; s < lam; ++s) q *= ri;
            p = 1.0 / q;
        }
        B += w[i] * p * phiT[(size_t)i * n_f + a] * phiT[(size_t)i * n_f + b];
        tab[(size_t)(i - 1) * n_frow + d].y = B;
    }
}

// Column mu of Pbar_l^mu = sqrt((l-mu)!/(l+mu)!) P_l^mu(x) (Condon-Shortley
// phase) for l = mu..lam_max, written to pb[pb_index(l, mu)].
__device__ void legendre_column(int lam_max, int mu, double x, double* pb) {
    const double s = sqrt(fmax(0.0, 1.0 - x * x));
    double pmm = 1.0;
    for (int i = 1; i <= mu; ++i) pmm *= -sqrt((2.0 * i - 1.0) / (2.0 * i)) * s;
    pb[pb_index(mu, mu)] = pmm;
    if (mu + 1 > lam_max) return;
    double p0 = pmm;
    double p1 = sqrt(2.0 * mu + 1.0) * x * pmm;
    pb[pb_index(mu + 1, mu)] = p1;
    for (int l = mu + 1; l < lam_max; ++l) {
        const double p2 = ((2.0 * l + 1.0) * x * p1 - sqrt((double)(l + mu) * (l - mu)) * p0) /
                          sqrt((double)(l + 1 + mu) * (l + 1 - mu));
        pb[pb_index(l + 1, mu)] = p2;
        p0 = p1;
        p1 = p2;
    }
}

// dPbar_l^mu/dx for l = mu..lam_max into pb[pb_index(l, mu)], from
// (x^2 - 1) dPbar_l^mu/dx = l x Pbar_l^mu - sqrt((l+mu)(l-mu)) Pbar_(l-1)^mu, |x| < 1.
__device__ void legendre_column_dx(int lam_max, int mu, double x, double* pb) {
    const double s = sqrt(fmax(0.0, 1.0 - x * x));
    const double den = x * x - 1.0;
    double pmm = 1.0;
    for (int i = 1; i <= mu; ++i) pmm *= -sqrt((2.0 * i - 1.0) / (2.0 * i)) * s;
    pb[pb_index(mu, mu)] = mu * x * pmm / den;
    if (mu + 1 > lam_max) return;
    double p0 = pmm;
    double p1 = sqrt(2.0 * mu + 1.0) * x * pmm;
    pb[pb_index(mu + 1, mu)] = ((mu + 1) * x * p1 - sqrt((double)(2 * mu + 1)) * p0) / den;
    for (int l = mu + 1; l < lam_max; ++l) {
        const double p2 = ((2.0 * l + 1.0) * x * p1 - sqrt((double)(l + mu) * (l - mu)) * p0) /
                          sqrt((double)(l + 1 + mu) * (l + 1 - mu));
        pb[pb_index(l + 1, mu)] = ((l + 1) * x * p2 - sqrt((double)(l + 1 + mu) * (l + 1 - mu)) * p1) / den;
        p0 = p1;
        p1 = p2;
    }
}

// Grid node r_k = r_max (k/n_r)^2, with the same arithmetic as the host grid.
__device__ inline double node_r(int k, double r_max, int n_r) {
    const double x = (double)k / n_r;
    return r_max * x * x;
}

// Last grid node with r_k <= R (nodes recomputed in registers).
__device__ inline int grid_index(double R, double r_max, int n_r) {
    int k = (int)floor(n_r * sqrt(fmin(R / r_max, 1.0)));
    k = max(0, min(k, n_r));
    auto rk = [&](int q) { return node_r(q, r_max, n_r); };
    while (k < n_r && rk(k + 1) <= R) ++k;
    while (k > 0 && rk(k) > R) --k;
    return k;
}

// F at R from the table entry (A_k, B_(k+1)).
__device__ inline double radial_at(double2 ab, double R, int lam) {
    double Rl = 1.0;
    for (int q = 0; q < lam; ++q) Rl *= R;
    return ab.x / (Rl * R) + ab.y * Rl;
}

// The R factors of the scaled FP32 table at node k <= R's interval:
// (r_k/R)^(lam+1) (0 at k = 0) and (R/r_(k+1))^lam (0 at k = n_r), both in
// [0, 1] because r_k <= R < r_(k+1).
__device__ inline void scaled_factors(double R, int k, int lam, double r_max, int n_r, double* fa, double* fb) {
    const double qa = k > 0 ? node_r(k, r_max, n_r) / R : 0.0;
    const double qb = k < n_r ? R / node_r(k + 1, r_max, n_r) : 0.0;
    double a = qa, b = 1.0;
    for (int q = 0; q < lam; ++q) {
        a *= qa;
        b *= qb;
    }
    *fa = a;
    *fb = k < n_r ? b : 0.0;
}

// Scaled single-precision copy of the moment table, one thread per (entry d,
// node k): x = A_k / r_k^(lam+1) (0 at k = 0), y = B_(k+1) r_(k+1)^lam (0 at
// k = n_r).  F(R) = x (r_k/R)^(lam+1) + y (R/r_(k+1))^lam is the same
// quadrature as the FP64 table's; the stored values are of the size of the
// integrals (no powers of r that leave FP32's range), rounded once.
__global__ void k_table_f32(const double2* __restrict__ tab, const int* __restrict__ dl, int n_frow, int n_r,
                            double r_max, float2* __restrict__ out) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    const int k = blockIdx.y;
    if (d >= n_frow) return;
    const int lam = dl[d];
    const size_t i = (size_t)k * n_frow + d;
    const double2 ab = tab[i];
    double x = 0.0, y = 0.0;
    if (k > 0) {
        const double rk = node_r(k, r_max, n_r);
        double p = rk;
        for (int q = 0; q < lam; ++q) p *= rk;
        x = ab.x / p;
    }
    if (k < n_r) {
        const double rk1 = node_r(k + 1, r_max, n_r);
        double p = 1.0;
        for (int q = 0; q < lam; ++q) p *= rk1;
        y = ab.y * p;
    }
    out[i] = make_float2((float)x, (float)y);
}

// F on the grid nodes, one thread per (entry d, node k): the quadrature of
// Eq. D2 at R = r_k, r_k^-(lam+1) A_k + r_k^lam B_(k+1) (at r_0 = 0 only the
// lam = 0 term B_1 survives).  The paper's production table (Sec. II).
__global__ void k_table_nodes(const double2* __restrict__ tab, const int* __restrict__ dl, int n_frow, int n_r,
                              double r_max, double* __restrict__ out) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    const int k = blockIdx.y;
    if (d >= n_frow) return;
    const int lam = dl[d];
    const size_t i = (size_t)k * n_frow + d;
    const double2 ab = tab[i];
    double f;
    if (k == 0) {
        f = lam == 0 ? ab.y : 0.0;
    } else {
        const double rk = node_r(k, r_max, n_r);
        double p = 1.0;
        for (int q = 0; q < lam; ++q) p *= rk;
        f = ab.x / (p * rk) + ab.y * p;
    }
    out[i] = f;
}

// Five-point interpolation of the node table at R (R < r_max): the stencil of
// the node j nearest to R in x = sqrt(r/r_max) (uniform in x), nodes j-2..j+2
// clamped to the grid, with the Lagrange weights in r.  Returns the first node.
__device__ inline int interp_stencil(double R, double r_max, int n_r, double* w) {
    int j = (int)rint(n_r * sqrt(R / r_max));
    j = min(max(j, 2), n_r - 2) - 2;
    double x[5];
    for (int i = 0; i < 5; ++i) x[i] = node_r(j + i, r_max, n_r);
    for (int i = 0; i < 5; ++i) {
        double p = 1.0;
        for (int k = 0; k < 5; ++k)
            if (k != i) p *= (R - x[k]) / (x[i] - x[k]);
        w[i] = p;
    }
    return j;
}

// F of entry d (multipole lam) from the node table: the stencil sum (kidx >= 0,
// weights rp[0..4]) or the multipole form beyond the grid, F(r_max) (r_max/R)^(lam+1)
// (kidx = -1, rp[lam] = (r_max/R)^(lam+1)).
__device__ inline double interp_value(const double* ftab, int n_frow, int n_r, int kidx, const double* rp, size_t d,
                                      int lam) {
    if (kidx < 0) return ftab[(size_t)n_r * n_frow + d] * rp[lam];
    double f = 0.0;
    for (int i = 0; i < 5; ++i) f = __builtin_fma(rp[i], ftab[(size_t)(kidx + i) * n_frow + d], f);
    return f;
}

__device__ inline double2 phase(double eps, double z, double v) {
    double sn, cs;
    sincos(eps * z / v, &sn, &cs);
    return make_double2(cs, sn);
}

// Per (path, z-point): grid node of R, powers of R, Pbar table and phases per
// radial function.  grid: x = point, y = path; one wave per block.
__global__ __launch_bounds__(64) void k_prologue(PrologueArgs a) {
    const Meta& m = *a.meta;
    const int j = a.traj0 + blockIdx.y;
    const int p = blockIdx.x;
    if (a.epoch && p == 0 && blockIdx.y == 0 && threadIdx.x == 0) *a.epoch += kChunkEpoch;
    const double z = a.zdev ? a.zdev[(size_t)(*a.chunk) * kChunkPoints + p] : a.z[p];
    const double b = a.tb.bvec[j], v = a.tb.vvec[j];
    const double R = sqrt(b * b + z * z);
    const size_t jp = (size_t)j * a.pt.n_pts + p;
    const int t = threadIdx.x;
    const int k = grid_index(R, m.r_max, m.n_r);
    if (a.tb.ftab) {
        // interpolated F: stencil and weights, or the multipole factors beyond the grid
        if (R < m.r_max) {
            if (t == 0) {
                double w[5];
                a.pt.kidx[jp] = interp_stencil(R, m.r_max, m.n_r, w);
                for (int i = 0; i < 5; ++i) a.pt.rpow[jp * kRpow + i] = w[i];
            }
        } else {
            if (t == 0) a.pt.kidx[jp] = -1;
            if (t <= m.lam_max) {
                const double q = m.r_max / R;
                double f = q;
                for (int i = 0; i < t; ++i) f *= q;
                a.pt.rpow[jp * kRpow + t] = f;
            }
        }
    } else if (t == 0) {
        a.pt.kidx[jp] = k;
    }
    if (t <= m.lam_max) {
        if (a.tb.ftab) {
            // factors written above
        } else if (a.tb.tab32) {
            scaled_factors(R, k, t, m.r_max, m.n_r, &a.pt.rpow[jp * kRpow + 2 * t], &a.pt.rpow[jp * kRpow + 2 * t + 1]);
        } else {
            double Rl = 1.0;
            for (int q = 0; q < t; ++q) Rl *= R;
            a.pt.rpow[jp * kRpow + 2 * t] = 1.0 / (Rl * R);
            a.pt.rpow[jp * kRpow + 2 * t + 1] = Rl;
        }
        legendre_column(m.lam_max, t, z / R, a.pt.pbar + jp * kMaxPb);
    }
    for (int f = t; f < m.n_f; f += blockDim.x) a.pt.ph[jp * m.n_f + f] = phase(a.tb.rad_eps[f], z, v);
}

// table entries per thread held in registers by a stage workgroup of `rows`
// rows (about 1.5 per row and thread; the rest is loaded where it is used)
constexpr int fbatch(int rows) { return rows >= 8 ? 12 : (rows * 3 + 1) / 2; }
constexpr int kXBatch = 4;   // amplitudes per thread held in registers
constexpr int kGBatch = 4;   // angular coefficients per thread held in registers

// RK4 combinations (Algorithm 1) of stage `stage` with slope K and step h:
// the next stage input (stages 1-3) and the new accumulator (stages 1-3) or
// the new amplitude (stage 4); w = rk4_weight(stage, h).
__device__ inline double rk4_weight(int stage, double h) { return (stage == 1 || stage == 4) ? h / 6.0 : h / 3.0; }
__device__ inline double2 rk4_next_input(int stage, double2 x0, double2 K, double h) {
    const double c = (stage == 3) ? h : 0.5 * h;
    return make_double2(__builtin_fma(c, K.x, x0.x), __builtin_fma(c, K.y, x0.y));
}
__device__ inline double2 rk4_accumulate(int stage, double2 x0, double2 xa, double2 K, double w) {
    const double2 x = stage == 1 ? x0 : xa;
    return make_double2(__builtin_fma(w, K.x, x.x), __builtin_fma(w, K.y, x.y));
}

// The RK4 combination of stage a.stage for output oi with slope K and step h.
__device__ inline void rk4_update(const StageArgs& a, size_t oi, double2 K, double2 x0, double2 xa, double h) {
    if (a.stage < 4) {
        a.u_out[oi] = rk4_next_input(a.stage, x0, K, h);
        a.Xacc[oi] = rk4_accumulate(a.stage, x0, xa, K, rk4_weight(a.stage, h));
    } else {
        const double2 xn = rk4_accumulate(4, x0, xa, K, rk4_weight(4, h));
        if (!isfinite(xn.x) || !isfinite(xn.y)) atomicOr(a.flag, 1);
        (a.Xout ? a.Xout : a.X)[oi] = xn;
    }
}

// phase 2 of a stage: W[r][g] = sum_n F_l'[r][e0(g) + n] x'[xoff(g) + n]
// for the workgroup's rows (LDS in, LDS out).  Each work item is one column g
// and half of the rows (ROWS / 2 accumulators), so that every x' load serves
// ROWS / 2 products; lanes of a wave take consecutive g (the F columns of one
// (l, lambda) block are read as a broadcast).
template <int ROWS>
__device__ inline void stage_phase2(const double* Fs, const double2* xs, const int2* gis, double2* Ws, int nrows,
                                    int gcols, int nV) {
    constexpr int RB = (ROWS + 1) / 2;
    const int B = blockDim.x, tid = threadIdx.x;
    for (int it = tid; it < 2 * gcols; it += B) {
        const int half = it >= gcols ? 1 : 0;
        const int g = it - half * gcols;
        const int r0 = half * RB;
        if (r0 >= nrows) continue;
        const int2 info = gis[g];
        const int e0 = info.x & 0xffff, nl = info.x >> 16;
        const double* f = Fs + r0 * nV + e0;
        const double2* x = xs + info.y;
        double re[RB], im[RB];
#pragma unroll
        for (int k = 0; k < RB; ++k) re[k] = im[k] = 0.0;
#pragma unroll 2
        for (int n = 0; n < nl; ++n) {
            const double2 y = x[n];
#pragma unroll
            for (int k = 0; k < RB; ++k) {
                // rows r0 + k >= nrows read rows of F that this stage did not
                // fill (inside the ROWS-row buffer); their sums are dropped
                const double fk = f[k * nV + n];
                re[k] = __builtin_fma(fk, y.x, re[k]);
                im[k] = __builtin_fma(fk, y.y, im[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < RB; ++k)
            if (r0 + k < nrows) Ws[(r0 + k) * gcols + g] = make_double2(re[k], im[k]);
    }
}

// Value of another lane of the wave's 16-lane rows (DPP, no LDS traffic).
template <int CTRL>
__device__ inline double dpp_move(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true));
}

// Sum over the S lanes (a power of two, S-aligned) of an output, every lane
// returning it.  Neighbours first: after the pairs and the quads hold equal
// values, mirroring half a row (row) brings the other quad's (half's) sum.
__device__ inline void lane_sum(double& re, double& im, int S) {
    if (S >= 2) {
        re += dpp_move<0xB1>(re);    // quad_perm [1, 0, 3, 2]
        im += dpp_move<0xB1>(im);
    }
    if (S >= 4) {
        re += dpp_move<0x4E>(re);    // quad_perm [2, 3, 0, 1]
        im += dpp_move<0x4E>(im);
    }
    if (S >= 8) {
        re += dpp_move<0x141>(re);   // row_half_mirror
        im += dpp_move<0x141>(im);
    }
    if (S >= 16) {
        re += dpp_move<0x140>(re);   // row_mirror
        im += dpp_move<0x140>(im);
    }
    for (int off = 16; off < S; off <<= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
    }
}

// An output's sum over the columns g is taken in kChains chains, g = c, c + 8,
// c + 16, ... for chain c, each in ascending order, whose sums are then added
// in pairs (0 + 1, 2 + 3, ...), the pairs in pairs and so on.  Every kernel
// that forms y = G W follows this order, so the split of the rows over
// workgroups and of the columns over lanes changes no bit of the result.
constexpr int kChains = 8;

// The sum for one output by S lanes, lane s taking chains s, s + S, ...; every
// lane of the wave takes part and returns the output's sum.
template <int S>
__device__ inline double2 phase3_sum(const double* g, const double2* w, int s, int gcols, bool valid) {
    constexpr int U = kChains / S;
    double re[U], im[U];
#pragma unroll
    for (int u = 0; u < U; ++u) re[u] = im[u] = 0.0;
    // whole rounds of the lane's chains without a test per column, then what
    // is left (k_stage, N = 1855, 4 paths, 5 rows: 22.4 us with a test per
    // column, 18.5 without)
    int c0 = s;
    const int n = valid ? gcols : 0;
    for (; c0 + (U - 1) * S < n; c0 += kChains) {
        double gv[U];
        double2 wv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            gv[u] = g[c0 + u * S];
            wv[u] = w[c0 + u * S];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            re[u] = __builtin_fma(gv[u], wv[u].x, re[u]);
            im[u] = __builtin_fma(gv[u], wv[u].y, im[u]);
        }
    }
#pragma unroll
    for (int u = 0; u + 1 < U; ++u)
        if (c0 + u * S < n) {
            const double gv = g[c0 + u * S];
            const double2 wv = w[c0 + u * S];
            re[u] = __builtin_fma(gv, wv.x, re[u]);
            im[u] = __builtin_fma(gv, wv.y, im[u]);
        }
#pragma unroll
    for (int u = 0; u < U; ++u) lane_sum(re[u], im[u], S);
#pragma unroll
    for (int d = 1; d < U; d *= 2)
#pragma unroll
        for (int u = 0; u + d < U; u += 2 * d) {
            re[u] += re[u + d];
            im[u] += im[u + d];
        }
    return make_double2(re[0], im[0]);
}

// phase 3 of a stage: y[r][q'] = sum_g G_l'[q'][g] W[r][g] for output o =
// (r, q') (o < n_out) by the S lanes s = 0..S-1 of the output.
__device__ inline double2 stage_phase3(const double* Gs, const double2* Ws, int o, int s, int S, int n_out, int nmp,
                                       int gcols) {
    const bool valid = o < n_out;
    const int r = valid ? o / nmp : 0, qp = valid ? o - r * nmp : 0;
    const double* g = Gs + qp * gcols;
    const double2* w = Ws + r * gcols;
    switch (S) {
        case 8: return phase3_sum<8>(g, w, s, gcols, valid);
        case 4: return phase3_sum<4>(g, w, s, gcols, valid);
        case 2: return phase3_sum<2>(g, w, s, gcols, valid);
        default: return phase3_sum<1>(g, w, s, gcols, valid);
    }
}

// phase 3 of the large-basis form: as stage_phase3, with the angular factor
// G_l'[q'][g] = c(g) Pbar[p(g)] formed from the coefficient tables (global
// memory, shared by every path and point: L2 hits) instead of staged in LDS.
__device__ inline double2 stage_phase3_global(const double* gc, const int* gp, const double* pbs, const double2* Ws,
                                              int o, int s, int S, int n_out, int nmp, int gcols) {
    double re = 0.0, im = 0.0;
    if (o < n_out) {
        const int r = o / nmp, qp = o - r * nmp;
        const double* c = gc + qp * gcols;
        const int* pp = gp + qp * gcols;
        const double2* w = Ws + r * gcols;
        // the coefficients of eight columns are loaded before the first is
        // used (their L2 latency bounded the stage: N = 2958, 8 paths, 122 ->
        // 80 us per launch); the order of the sum does not change
        constexpr int U = 8;
        for (int k0 = s; k0 < gcols; k0 += U * S) {
            int p[U];
            double cv[U];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int k = min(k0 + i * S, gcols - 1);
                p[i] = pp[k];
                cv[i] = c[k];
            }
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int k = k0 + i * S;
                if (k < gcols && p[i] >= 0) {
                    const double g = cv[i] * pbs[p[i]];
                    re += g * w[k].x;
                    im += g * w[k].y;
                }
            }
        }
    }
    for (int off = S >> 1; off > 0; off >>= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
    }
    return make_double2(re, im);
}

// Lanes per output of phase 3: the largest power of two S <= most with
// 2 n_out S <= B (so that every output keeps at least half the lanes busy),
// for the n_out = ROWS x (2 l' + 1) outputs of a full tile of the block.
// Every output has a lane group when n_out <= B (phase3_fits).
__device__ inline int phase3_lanes(int n_out, int B, int most) {
    int S = 1;
    while (S < most && n_out * S * 2 <= B) S *= 2;
    return S;
}

// Whether a tile of `rows` rows gives every output of blocks of up to
// nmp_max = 2 l_max + 1 values of m' a lane of the stage workgroup.
__host__ __device__ inline bool phase3_fits(int rows, int nmp_max) { return rows * nmp_max <= kStageThreads; }

// One stage for rows [row0, row0 + nrows) of the l' block, all nmp = 2l'+1 values of m'.
// KIND 0: RK4 stage (k_stage); KIND 1: operator application (k_apply, see
// StageArgs) with the same three phases.
//   phase 0: every independent global load of the stage is issued at once
//            (table entries or cached F, stage input, coefficients) and the
//            per-point tables (R powers, Pbar, phases) go to LDS;
//   phase 1: x' = conj(ph) u, F_l'[rows][:] = A R^-(lam+1) + B R^lam (or the
//            cached F), G_l' = c Pbar  -> LDS
//   phase 2: W[r][g] = sum_n F_l'[r][e0(g) + n] x'_{l(g), q(g), n}
//   phase 3: y[r][q'] = sum_g G_l'[q'][g] W[r][g];  K = -(i/v) Zp ph y; RK4 update.
//   phase 4 (FC with a.fc_next): F of the rows at point a.p_next from the
//            moment-table entries loaded in phase 0 -> a.fc_next.
// F32: the moment table is the scaled FP32 form.  FC: F at the stage's point
// comes from the radial-integral cache a.fc_cur (KIND 0 only).  GG (large
// bases, FC only): G_l' is not staged in LDS; phase 3 forms it from the
// coefficient tables.
template <int KIND, int ROWS, bool F32 = false, bool FC = false, bool GG = false>
__device__ void stage_body(const StageArgs& a, int j, const StageTile& t, char* smem) {
    // moment-table entries: FP64 (A_k, B_(k+1)) or the scaled FP32 form
    using TabT = typename std::conditional<F32, float2, double2>::type;
    const Meta& m = *a.meta;
    const Tables& T = a.tb;
    const int N = m.n_states;
    const int row0 = t.row0, nrows = t.nrows;
    const int nmp = t.nmp;
    const int nlp = t.n_l;
    const int nV = t.nV;
    const int gcols = t.gcols;
    const int B = blockDim.x;
    const int tid = threadIdx.x;
    const size_t jp = (size_t)j * a.pt.n_pts + a.p;

    double2* xs = reinterpret_cast<double2*>(smem);                       // [n_xs] (xs_off, xs_stride)
    double2* Ws = xs + m.n_xs;                                             // [rows][gcols]
    double2* phs = Ws + ROWS * gcols;                                      // [n_f]
    double* Fs = reinterpret_cast<double*>(phs + m.n_f);                  // [rows][nV]
    double* Gs = Fs + ROWS * nV;                                           // [nmp][gcols] (not with GG)
    double* rps = GG ? Gs : Gs + nmp * gcols;                              // [kRpow]
    double* pbs = rps + kRpow;                                             // [kMaxPb]
    int2* gis = reinterpret_cast<int2*>(pbs + kMaxPb);                     // [gcols]

    // phase 0
    // the moment-table rows are read at this stage's point (no cache) or at
    // the cache's next point (FC with fc_next)
    const bool tab_rows = !FC || a.fc_next != nullptr;
    const size_t jt = FC ? (size_t)j * a.pt.n_pts + a.p_next : jp;
    const int k = tab_rows ? a.pt.kidx[jt] : 0;
    const TabT* tab = nullptr;
    if constexpr (F32) tab = T.tab32;
    else tab = T.tab;
    const TabT* row = tab + (size_t)k * m.n_frow + t.frow_off + (size_t)row0 * nV;
    // cached F: FP64, or FP32 for the scaled FP32 table
    using FcT = typename std::conditional<F32, float, double>::type;
    const FcT* frow = FC ? static_cast<const FcT*>(a.fc_cur) + (size_t)j * m.n_frow + t.frow_off + (size_t)row0 * nV
                         : nullptr;
    const int* cl = T.col_lam + t.col_off;
    const int totF = nrows * nV;
    constexpr int FB = fbatch(ROWS);
    TabT tv[FB];
    int lv[FB];
    FcT fv[FC ? FB : 1];
    // Every lane loads (past the end: a clamped, in-bounds index whose value
    // is not used), so that all loads of a batch are issued back to back
    // before the first wait: one memory round trip instead of one per batch.
    auto load_table_rows = [&]() {
        int q = tid % nV;
        const int dq = B % nV;
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            tv[i] = row[min(tid + i * B, totF - 1)];
            lv[i] = cl[q];
            q += dq;
            if (q >= nV) q -= nV;
        }
    };
    if (FC) {
        // the next point's table rows are loaded after phase 1, so that they
        // arrive during phases 2 and 3 instead of delaying the first wait
#pragma unroll
        for (int i = 0; i < (FC ? FB : 0); ++i) fv[i] = frow[min(tid + i * B, totF - 1)];
    } else {
        load_table_rows();
    }
    // stage input (KIND 1: v = cu1 u_in + cu2 u_in2)
    const double2* u = a.u_in + (size_t)j * a.n_pad;
    const double2* u2 = (KIND == 1 && a.u_in2) ? a.u_in2 + (size_t)j * a.n_pad : nullptr;
    auto load_u = [&](int idx) -> double2 {
        if (KIND == 0) return u[idx];
        const double2 x = u[idx];
        double2 r = make_double2(a.cu1 * x.x, a.cu1 * x.y);
        if (u2) {
            const double2 y = u2[idx];
            r.x += a.cu2 * y.x;
            r.y += a.cu2 * y.y;
        }
        return r;
    };
    double2 uv[kXBatch];
    int sr[kXBatch], sx[kXBatch];  // radial index and LDS position of each amplitude
#pragma unroll
    for (int i = 0; i < kXBatch; ++i) {
        const int idx = min(tid + i * B, N - 1);
        uv[i] = load_u(idx);
        sr[i] = T.st_rad[idx];
        sx[i] = T.st_xs[idx];
    }
    const double* gc = T.gcoef + t.g_off;
    const int* gp = T.gpb + t.g_off;
    const int totG = nmp * gcols;
    double gcv[kGBatch];
    int gpv[kGBatch];
#pragma unroll
    for (int i = 0; i < kGBatch; ++i) {
        const int idx = min(tid + i * B, totG - 1);
        gcv[i] = GG ? 0.0 : gc[idx];
        gpv[i] = GG ? -1 : gp[idx];
    }
    // output-side values, prefetched by the thread that writes output o.
    // The lanes per output follow from the tiling's ROWS, not from this
    // tile's rows (the large-basis form's sums depend on them)
    const int n_out = nrows * nmp;
    const int S = phase3_lanes(ROWS * nmp, B, GG ? 64 : kChains);
    const int o = tid / S, s = tid - o * S;
    const bool writer = (o < n_out) && (s == 0);
    const double v = T.vvec[j];
    size_t oi = 0;
    int rad_o = 0;
    double2 x0 = make_double2(0.0, 0.0), xa = make_double2(0.0, 0.0);
    if (writer) {
        const int r = o / nmp, qp = o - r * nmp;
        oi = (size_t)j * a.n_pad + t.state_off + qp * nlp + row0 + r;
        rad_o = t.rad_off + row0 + r;
        if (KIND == 0) {
            if (a.stage < 4) x0 = a.X[oi];
            if (a.stage > 1) xa = a.Xacc[oi];
        } else {
            // x0 = sum of the added vectors, xa = d = cd1 dv + cd2 dv2
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (a.w[k]) {
                    const double2 t = a.w[k][oi];
                    x0.x += t.x;
                    x0.y += t.y;
                }
            if (a.dv) {
                const double2 t = a.dv[oi];
                xa = make_double2(a.cd1 * t.x, a.cd1 * t.y);
                if (a.dv2) {
                    const double2 t2 = a.dv2[oi];
                    xa.x += a.cd2 * t2.x;
                    xa.y += a.cd2 * t2.y;
                }
            }
        }
    }
    const int deriv = (KIND == 1) ? a.deriv : 0;
    const double bj = T.bvec[j];
    const double Rz = sqrt(bj * bj + a.z * a.z);
    // the point's tables and the column descriptors, one entry per thread
    // (larger tables: the rest is loaded below)
    const int n_rp = 2 * (m.lam_max + 1), n_pb = (m.lam_max + 1) * (m.lam_max + 2) / 2;
    const int2 gv = T.gcol_info[t.gcol_off + min(tid, gcols - 1)];
    const double rpv = tab_rows ? a.pt.rpow[jt * kRpow + min(tid, n_rp - 1)] : 0.0;
    const double pbv = a.pt.pbar[jp * kMaxPb + min(tid, n_pb - 1)];
    const double2 phv = a.pt.ph[jp * m.n_f + min(tid, m.n_f - 1)];
    // every load above is issued before any of their values is used
    __builtin_amdgcn_sched_barrier(0);
    if (deriv == 1) {
        // d/dR of R^-(lam+1) and R^lam
        if (tid <= m.lam_max) {
            double Rl = 1.0;
            for (int q = 0; q < tid; ++q) Rl *= Rz;
            rps[2 * tid] = -(tid + 1.0) / (Rl * Rz * Rz);
            rps[2 * tid + 1] = tid > 0 ? tid * Rl / Rz : 0.0;
        }
    } else if (tid < n_rp) {
        rps[tid] = rpv;
    }
    if (tid < gcols) gis[tid] = gv;
    for (int i = tid + B; i < gcols; i += B) gis[i] = T.gcol_info[t.gcol_off + i];
    if (deriv == 2) {
        if (tid <= m.lam_max) legendre_column_dx(m.lam_max, tid, a.z / Rz, pbs);
    } else {
        if (tid < n_pb) pbs[tid] = pbv;
        for (int i = tid + B; i < n_pb; i += B) pbs[i] = a.pt.pbar[jp * kMaxPb + i];
    }
    if (tid < m.n_f) phs[tid] = phv;
    for (int i = tid + B; i < m.n_f; i += B) phs[i] = a.pt.ph[jp * m.n_f + i];
    __syncthreads();

    // phase 1
#pragma unroll
    for (int i = 0; i < kXBatch; ++i) {
        const int idx = tid + i * B;
        if (idx < N) {
            const double2 ph = phs[sr[i]], x = uv[i];
            xs[sx[i]] = dephase(ph, x);
        }
    }
    for (int idx = tid + kXBatch * B; idx < N; idx += B) xs[T.st_xs[idx]] = dephase(phs[T.st_rad[idx]], load_u(idx));
    if (FC) {
#pragma unroll
        for (int i = 0; i < (FC ? FB : 0); ++i) {
            const int idx = tid + i * B;
            if (idx < totF) Fs[idx] = (double)fv[i];
        }
        for (int idx = tid + FB * B; idx < totF; idx += B) Fs[idx] = (double)frow[idx];
    } else {
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            const int idx = tid + i * B;
            if (idx < totF) Fs[idx] = radial_f((double)tv[i].x, (double)tv[i].y, rps[2 * lv[i]], rps[2 * lv[i] + 1]);
        }
        for (int idx = tid + FB * B; idx < totF; idx += B) {
            const TabT t0 = row[idx];
            const int l0 = cl[idx % nV];
            Fs[idx] = radial_f((double)t0.x, (double)t0.y, rps[2 * l0], rps[2 * l0 + 1]);
        }
    }
    if (!GG) {
#pragma unroll
        for (int i = 0; i < kGBatch; ++i) {
            const int idx = tid + i * B;
            if (idx < totG) Gs[idx] = gpv[i] >= 0 ? gcv[i] * pbs[gpv[i]] : 0.0;
        }
        for (int idx = tid + kGBatch * B; idx < totG; idx += B) {
            const int p = gp[idx];
            Gs[idx] = p >= 0 ? gc[idx] * pbs[p] : 0.0;
        }
    }
    __syncthreads();

    if (FC && tab_rows) load_table_rows();
    stage_phase2<ROWS>(Fs, xs, gis, Ws, nrows, gcols, nV);
    __syncthreads();
    const double2 y = GG ? stage_phase3_global(gc, gp, pbs, Ws, o, s, S, n_out, nmp, gcols)
                         : stage_phase3(Gs, Ws, o, s, S, n_out, nmp, gcols);
    double gval = 0.0, gma = 0.0, gmc = 0.0;
    if (writer) {
        const double2 py = cmul(phs[rad_o], y);
        const double sc = a.Zp / v;
        double2 K = make_double2(sc * py.y, -sc * py.x);  // -(i/v) Zp ph y
        const double h = a.h;
        if (KIND == 1) {
            if (deriv) {
                const double f = deriv == 1 ? bj / Rz : -a.z * bj / (Rz * Rz * Rz);
                K = make_double2(f * K.x, f * K.y);
            }
            if (a.out) a.out[oi] = make_double2(a.alpha * K.x + x0.x, a.alpha * K.y + x0.y);
            gval = 2.0 * a.gamma * (xa.x * K.x + xa.y * K.y);  // 2 gamma Re(conj(d) K)
            if (a.model) {
                // (dDeltaV/dtheta)_{n' n} x'_n over the radial block of (l', q'):
                // dM/dtheta v = -(i/v) ph (dDeltaV/dtheta) conj(ph) v and x' = conj(ph) v
                const int r = o / nmp, qp = o - r * nmp;
                const double* fa = a.va + t.vo + (size_t)(row0 + r) * nlp;
                const double* fc = a.vc + t.vo + (size_t)(row0 + r) * nlp;
                const double2* xq = xs + t.xs_off + qp * t.xs_stride;
                double2 ca = make_double2(0.0, 0.0), cc = make_double2(0.0, 0.0);
                for (int n = 0; n < nlp; ++n) {
                    const double2 x = xq[n];
                    ca.x += fa[n] * x.x;
                    ca.y += fa[n] * x.y;
                    cc.x += fc[n] * x.x;
                    cc.y += fc[n] * x.y;
                }
                const double2 p = phs[rad_o];
                const double2 t = make_double2(xa.x * p.x + xa.y * p.y, xa.x * p.y - xa.y * p.x);  // conj(d) p
                // 2 gamma Re(-(i/v) t c) = 2 gamma Im(t c) / v
                gma = 2.0 * a.gamma * (t.x * ca.y + t.y * ca.x) / v;
                gmc = 2.0 * a.gamma * (t.x * cc.y + t.y * cc.x) / v;
            }
        } else {
            // graph replays read the step length from device memory
            const double hh = a.hdev ? a.hdev[(size_t)(*a.chunk) * kChunkSteps + a.hidx] : h;
            rk4_update(a, oi, K, x0, xa, hh);
        }
    }
    if (FC && a.fc_next) {
        // phase 4: the cache's next point (rps holds its R factors)
        FcT* fout = static_cast<FcT*>(a.fc_next) + (size_t)j * m.n_frow + t.frow_off + (size_t)row0 * nV;
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            const int idx = tid + i * B;
            if (idx < totF)
                fout[idx] = (FcT)radial_f((double)tv[i].x, (double)tv[i].y, rps[2 * lv[i]], rps[2 * lv[i] + 1]);
        }
        for (int idx = tid + FB * B; idx < totF; idx += B) {
            const TabT t0 = row[idx];
            const int l0 = cl[idx % nV];
            fout[idx] = (FcT)radial_f((double)t0.x, (double)t0.y, rps[2 * l0], rps[2 * l0 + 1]);
        }
    }
    if (KIND == 1 && a.grad) {
        // this workgroup's shares, accumulated over the launches in its own
        // slots and summed in a fixed order by k_grad_sum
        __shared__ double red[3][kStageThreads / 64];
        for (int off = 32; off > 0; off >>= 1) {
            gval += __shfl_xor(gval, off, 64);
            gma += __shfl_xor(gma, off, 64);
            gmc += __shfl_xor(gmc, off, 64);
        }
        if ((tid & 63) == 0) {
            red[0][tid >> 6] = gval;
            red[1][tid >> 6] = gma;
            red[2][tid >> 6] = gmc;
        }
        __syncthreads();
        if (tid == 0) {
            double sb = 0.0, sa = 0.0, sc = 0.0;
            for (int w = 0; w < B / 64; ++w) {
                sb += red[0][w];
                sa += red[1][w];
                sc += red[2][w];
            }
            double* g = a.grad + (size_t)j * kGradSlots * a.gn + blockIdx.x;
            g[a.gslot * a.gn] += sb;
            if (a.model) {
                g[2 * a.gn] += sa;
                g[3 * a.gn] += sc;
            }
        }
    }
}

// k_apply's grid: x = row tile of a path (a.tiles, l' order), y = path.
template <int KIND, int ROWS, bool GG = false>
__device__ void stage_entry(const StageArgs& a, char* smem) {
    const StageTile t = a.tiles[blockIdx.x];
    if (t.nrows <= 0) return;
    stage_body<KIND, ROWS, false, false, GG>(a, a.traj0 + blockIdx.y, t, smem);
}

// One RK4 stage for a.n_paths paths from a.traj0.  Small
// row tiles ask for registers that leave room for four workgroups per CU
// (their LDS does), larger ones for three.
template <int ROWS, bool F32, bool FC, bool GG = false>
__global__ __launch_bounds__(GG ? kStageThreadsGG : kStageThreads, ROWS <= 4 ? 4 : 3) void k_stage(StageArgs a) {
    extern __shared__ double2 smem2[];
    // work item W of the path-major list of a.n_paths x a.nwg row tiles:
    // consecutive workgroup ids go to the eight XCDs in turn and the items of
    // XCD x are the x-th eighth of the list, so the workgroups of a path share
    // an XCD (and its L2, which then serves the path's stage input to all of
    // them).  The tile (one 64-byte load) holds the per-l' offsets, so no
    // loop over the basis blocks precedes the loads
    const int total = a.n_paths * a.nwg;
    const int per = (total + 7) / 8;
    const int W = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (W >= total) return;
    const int jl = W / a.nwg;
    const StageTile t = a.tiles[W - jl * a.nwg];
    stage_body<0, ROWS, F32, FC, GG>(a, a.traj0 + jl, t, reinterpret_cast<char*>(smem2));
}

// F of Eq. D2 at point slot p for every entry of the row layout and every path
// of the launch (grid: entries / 256 x paths), with the arithmetic of the
// stage kernels' phase 1 / phase 4.
template <bool F32>
__global__ __launch_bounds__(256) void k_fpoint(const Meta* __restrict__ mp_, Tables T, PointArrays pt, int p,
                                                int traj0, void* __restrict__ fc_) {
    const Meta& m = *mp_;
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= m.n_frow) return;
    const int j = traj0 + blockIdx.y;
    const size_t jp = (size_t)j * pt.n_pts + p;
    int lp = 0;
    while (lp < m.l_max && d >= m.frow_off[lp + 1]) ++lp;
    const int lam = T.col_lam[m.col_off[lp] + (d - m.frow_off[lp]) % m.nV[lp]];
    const double* rp = pt.rpow + jp * kRpow;
    if (T.ftab) {
        static_cast<double*>(fc_)[(size_t)j * m.n_frow + d] =
            interp_value(T.ftab, m.n_frow, m.n_r, pt.kidx[jp], rp, d, lam);
        return;
    }
    const size_t i = (size_t)pt.kidx[jp] * m.n_frow + d;
    if constexpr (F32) {
        const float2 t0 = T.tab32[i];
        static_cast<float*>(fc_)[(size_t)j * m.n_frow + d] =
            (float)radial_f((double)t0.x, (double)t0.y, rp[2 * lam], rp[2 * lam + 1]);
    } else {
        const double2 t0 = T.tab[i];
        static_cast<double*>(fc_)[(size_t)j * m.n_frow + d] = radial_f(t0.x, t0.y, rp[2 * lam], rp[2 * lam + 1]);
    }
}

// ---------------------------------------------------------------------------
// Persistent form of a propagation chunk.
//
// G workgroups hold one path for all steps of a chunk, each a run of its
// radial functions (ChunkWG).  A workgroup keeps in LDS the F rows
// of its functions at the current point and their angular factors, in
// registers the amplitude and RK4 accumulator of its outputs, and forms F and
// G again only when the point changes (twice per step); the moment-table
// entries of the next point are loaded into registers while the stage before
// sums y.
//
// A stage is a chain of four short dependent parts (x' arrives, W, y, update),
// so what bounds it is latency: few workgroups per path and the whole chip's
// issue slots beside each other.  16 waves where a workgroup has at most two
// table entries per thread (one path of a small basis), else 8 waves, whose
// register budget holds the entries without spilling: a spill in the loop
// waits for the table loads in flight (vector memory returns in order; 60
// bytes of it cost 4 us a step at N = 580).  Which G is best
// depends on basis and batch and is timed at plan creation.  Measured per
// pass on the propagation cases, one launch per stage -> this kernel:
// N = 86, 1 path, 800 steps: 12.8 -> 7.4 ms (G = 1); N = 580, 32 paths, 800:
// 35.5 -> 19.6 ms (G = 8); N = 580, 64 paths, 400, FP32 table: 28.9 ->
// 18.1 ms; N = 1855, 8 paths, 100, interpolated: 15.1 -> 9.2 ms (G = 48).
//
// Both sums of a stage run on v_mfma_f64_4x4x4 (four 4 x 4 products of four
// terms each, at the FP64 MFMA peak, with a granularity that fits 2l+1 and
// nearly any row count).  Its four terms are added one after another with a
// single rounding each, so a chain of them gives bitwise the sum that
// k_stage's chain of fused multiply-adds gives; F rows, W rows and angular
// factors are padded with zeros to whole blocks.
//   W = F x'  (jobs): F lies in LDS in operand order, so a wave reads 16 rows
//             x 8 n with one conflict-free 16-byte load per lane and reuses it
//             for all 2l+1 rows of x'; a 16-byte load of x' is the operand of
//             the real and of the imaginary product.
//   y = G W   (groups): wave c sums column chain c (kChains), the eight chain
//             sums are added by the output's thread.
//
// What the workgroups of a path exchange between stages is the next stage's
// x' = conj(ph) u, through global memory, in words that carry the stage
// number beside half a double (chunk_put, chunk_take): a reader polls the
// data itself, so there is no barrier, no fence and no second round trip, and
// each word is consistent by itself whatever order the words arrive in.  With
// G = 1 x' stays in LDS.  The wait is for workgroups of the same launch, which
// a cooperative launch brings onto the device together; kernels of other
// streams can hold their places up meanwhile, so it lasts as long as a queued
// launch would (kChunkSpin) before it ends with an error.
// ---------------------------------------------------------------------------

// Words [4][N] of one path and buffer: the two halves of an amplitude's
// components tagged with the stage number.  Every word is written and read by
// one 64-bit atomic access at agent scope, so it is never torn and needs no
// ordering with respect to the others.
__device__ inline void chunk_put(unsigned long long* buf, int N, int i, double2 x, unsigned tag) {
    const unsigned long long t = (unsigned long long)tag << 32;
    const unsigned h[4] = {(unsigned)__double2loint(x.x), (unsigned)__double2hiint(x.x), (unsigned)__double2loint(x.y),
                           (unsigned)__double2hiint(x.y)};
#pragma unroll
    for (int k = 0; k < 4; ++k)
        __hip_atomic_store(buf + (size_t)k * N + i, t | h[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// x' of every state of the path into xs once all its words carry `tag`.
// sx: x' positions of states tid and tid + NT; xpos: of every
// state.  Returns false if the words do not come within `spin` polls.
template <int NT>
__device__ inline bool chunk_take(const unsigned long long* buf, int N, unsigned tag, const int (&sx)[2],
                                  const int* __restrict__ xpos, double2* xs, int spin, int tid) {
    bool all = true;
    for (int base = 0; base < N; base += 2 * NT) {
        const bool two = N > base + NT;
        const int i0 = min(base + tid, N - 1), i1 = min(base + NT + tid, N - 1);
        const int p0 = base == 0 ? sx[0] : xpos[i0], p1 = base == 0 ? sx[1] : xpos[i1];
        unsigned long long w[2][4];
        bool ok = false;
        for (int it = 0; it < spin && !ok; ++it) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[0][k] = __hip_atomic_load(buf + k * N + i0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (two) w[1][k] = __hip_atomic_load(buf + k * N + i1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            ok = true;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ok = ok && (unsigned)(w[0][k] >> 32) == tag;
                if (two) ok = ok && (unsigned)(w[1][k] >> 32) == tag;
            }
        }
        all = all && ok;
        // threads past the last state hold a copy of it
        xs[p0] = make_double2(__hiloint2double((int)w[0][1], (int)w[0][0]), __hiloint2double((int)w[0][3], (int)w[0][2]));
        if (two)
            xs[p1] = make_double2(__hiloint2double((int)w[1][1], (int)w[1][0]), __hiloint2double((int)w[1][3], (int)w[1][2]));
    }
    return all;
}

__device__ inline int4 wave_uniform(int4 v) {
    return make_int4(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y),
                     __builtin_amdgcn_readfirstlane(v.z), __builtin_amdgcn_readfirstlane(v.w));
}

// W rows lie in groups of four: [row group][chain][column block][k][row % 4],
// column g = chain + 8 (4 block + k).
inline int chunk_column(int g, int blocks) { return ((g & 7) * blocks + (g >> 5)) * 16 + ((g >> 3) & 3) * 4; }

// NP pairs of n blocks of a job: re, im += F x' for NU groups of four rows of
// x'.  Straight-line code: every operand load is issued before the products
// that wait for it.
template <int NU, int NP>
__device__ inline void chunk_mac(const double2* f, const double2* x, int ustride, double (&re)[NU], double (&im)[NU]) {
    double2 a[NP], b[NP][NU][2];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        a[p] = f[64 * p];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            b[p][u][0] = x[u * ustride + 8 * p];
            b[p][u][1] = x[u * ustride + 8 * p + 4];
        }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            re[u] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[p].x, b[p][u][0].x, re[u], 0, 0, 0);
            im[u] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[p].x, b[p][u][0].y, im[u], 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            re[u] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[p].y, b[p][u][1].x, re[u], 0, 0, 0);
            im[u] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[p].y, b[p][u][1].y, im[u], 0, 0, 0);
        }
    }
}

// One job: W[row][q] = sum_n F[row][n] x'[q][n] for the job's 16 rows and 4 NU
// rows of x'.  Lane l reads row l % 16 of F and row l % 4 (+ 4 u) of x' at
// n = 4 block + l / 16; its results are row 4 ((l % 16) / 4) + l / 16, q =
// 4 u + l % 4, written to position u of jl (results past the rows or past
// 2l+1 go to a position of the lane's own that nothing reads).
template <int NU>
__device__ inline void chunk_job(const double2* F2, const double2* xs, double2* Ws, int4 job, int2 jl, int lane) {
    const int stride = job.z & 0xffff;
    int np = job.z >> 16;
    const double2* f = F2 + job.x / 2 + lane;
    const double2* x = xs + job.y + (lane & 3) * stride + (lane >> 4);
    double re[NU], im[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) re[u] = im[u] = 0.0;
    constexpr int MP = NU < 3 ? 2 : 1;   // pairs at once (operand registers)
    for (; np >= MP; np -= MP) {
        chunk_mac<NU, MP>(f, x, 4 * stride, re, im);
        f += MP * 64;
        x += MP * 8;
    }
    if (MP == 2 && np == 1) chunk_mac<NU, 1>(f, x, 4 * stride, re, im);
    const int w[4] = {jl.x & 0xffff, (int)((unsigned)jl.x >> 16), jl.y & 0xffff, (int)((unsigned)jl.y >> 16)};
#pragma unroll
    for (int u = 0; u < NU; ++u) Ws[w[u]] = make_double2(re[u], im[u]);
}

// KB column blocks of a chain for NG groups: re, im += G W
template <int KB, int NG>
__device__ inline void chunk_chain(const double2* const (&w)[NG], const double* const (&g)[NG], int at, double (&re)[NG],
                                   double (&im)[NG]) {
    double2 wv[KB][NG];
    double gv[KB][NG];
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            wv[b][i] = w[i][at + 16 * b];
            gv[b][i] = g[i][at + 16 * b];
        }
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            re[i] = __builtin_amdgcn_mfma_f64_4x4x4f64(wv[b][i].x, gv[b][i], re[i], 0, 0, 0);
            im[i] = __builtin_amdgcn_mfma_f64_4x4x4f64(wv[b][i].y, gv[b][i], im[i], 0, 0, 0);
        }
}

// Chain `wave` of NG groups, their sums to Ps.  q: W position | angular
// position << 16, output or -1.
template <int NG>
__device__ inline void chunk_groups(const int2* q, const double2* Ws, const double* Gs, double2* Ps, int wave, int n_out,
                                    int blocks) {
    const double2* w[NG];
    const double* g[NG];
    double re[NG], im[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        w[i] = Ws + (q[i].x & 0xffff) + wave * blocks * 16;
        g[i] = Gs + ((unsigned)q[i].x >> 16) + wave * blocks * 16;
        re[i] = im[i] = 0.0;
    }
    int at = 0;
    for (; blocks > 4; blocks -= 4, at += 64) chunk_chain<4>(w, g, at, re, im);
    if (blocks == 4) chunk_chain<4>(w, g, at, re, im);
    else if (blocks == 3) chunk_chain<3>(w, g, at, re, im);
    else if (blocks == 2) chunk_chain<2>(w, g, at, re, im);
    else chunk_chain<1>(w, g, at, re, im);
#pragma unroll
    for (int i = 0; i < NG; ++i)
        if (q[i].y >= 0) Ps[wave * n_out + q[i].y] = make_double2(re[i], im[i]);
}

// FORM: kRadialMoments (FP64 table), kRadialMoments32 (scaled FP32 table) or
// kRadialInterp (F interpolated from the node table where it is needed).
// NT: threads.  FP: table entries per thread.  ADJ: the adjoint's forms
// (ChunkArgs::adjoint).
template <int FORM, int NT, int FP, bool ADJ>
__global__ __launch_bounds__(NT) void k_chunk(ChunkArgs c) {
    extern __shared__ double2 smem2[];
    __shared__ int gave_up;
    using TabT = typename std::conditional<FORM == kRadialMoments32, float2, double2>::type;
    constexpr int GP = 2;   // angular coefficients per thread held in registers
    const StageArgs& a = c.s;
    const Meta& m = *a.meta;
    const Tables& T = a.tb;
    const int total = c.n_traj * c.G, per = (total + 7) / 8;
    // paths on one XCD each, as in k_stage
    const int Wi = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (Wi >= total) return;
    const int jl = Wi / c.G, j = a.traj0 + jl;
    const ChunkWG& wg = c.wgs[Wi - jl * c.G];
    int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), N = m.n_states;
    const int n_f = m.n_f, n_frow = m.n_frow, n_r = m.n_r, lam_max = m.lam_max;
    const int n_out = wg.n_out, n_g = wg.n_g, n_grp = wg.n_grp, g0 = wg.g0, ent0 = wg.ent0;
    const int n_rad = wg.n_rad, rad0 = wg.rad0;
    const bool local = c.G == 1;

    double2* xs = smem2;                                        // [c.n_xs]
    double2* Ws = xs + c.n_xs;                                  // [wg.n_w]
    double2* Ps = Ws + wg.n_w;                                  // [8][n_out] chain sums
    double2* phs = Ps + kChains * n_out;                        // [2][n_rad] phases of its functions, by parity of the point
    int2* grps = reinterpret_cast<int2*>(phs + 2 * n_rad);        // [n_grp][NT / 8]
    double* Fs = reinterpret_cast<double*>(grps + NT / kChains * n_grp); // [wg.n_f]
    double* Gs = Fs + wg.n_f;                                   // [n_g]
    double* rps = Gs + n_g;                                     // [kRpow]
    double* pbs = rps + kRpow;                                  // [kMaxPb]
    int4* jhs = reinterpret_cast<int4*>(pbs + kMaxPb + 1);      // [wg.n_jobs] job headers
    int2* jls = reinterpret_cast<int2*>(jhs + wg.n_jobs);       // [wg.n_jobs][64] and their lanes

    // this thread's share of the workgroup's constants
    int entf[FP];      // its table entries: F position | lambda << 20, and byte offset in a table row
    unsigned entx[FORM == kRadialInterp ? 1 : FP];
#pragma unroll
    for (int i = 0; i < FP; ++i) {
        const int e = tid + i * NT;
        const int2 v = e < wg.n_ent ? c.ents[wg.ent0 + e] : make_int2(0, -1);
        entf[i] = v.y;
        if constexpr (FORM != kRadialInterp) entx[i] = (unsigned)v.x * (unsigned)sizeof(TabT);
    }
    double gco[GP];    // angular coefficients and their Legendre factors
    int gpi[GP];
#pragma unroll
    for (int i = 0; i < GP; ++i) {
        const int e = tid + i * NT, q = e < n_g ? c.gsrc[wg.g0 + e] : -1;
        gpi[i] = q >= 0 ? T.gpb[q] : -1;
        gco[i] = gpi[i] >= 0 ? T.gcoef[q] : 0.0;
    }
    // output tid
    int4 out = c.outs[wg.out0 + min(tid, n_out - 1)];
    double2 x0 = a.X[(size_t)j * a.n_pad + out.x], xa = make_double2(0.0, 0.0);
    // groups halves * g + half for the chain of this wave
    constexpr int halves = NT / 64 / kChains;
    const int chain = wave & (kChains - 1), half = wave / kChains;
    int2 grp[kChunkGroups];
#pragma unroll
    for (int g = 0; g < kChunkGroups; ++g)
        grp[g] = c.grps[(size_t)64 * (wg.grp0 + halves * min(g, n_grp - 1) + half) + lane];
    for (int i = tid; i < 64 * halves * n_grp; i += NT) grps[i] = c.grps[(size_t)64 * wg.grp0 + i];
    const int kb = wg.kb;
    for (int i = tid; i < 64 * wg.n_jobs; i += NT) jls[i] = c.jlane[(size_t)64 * wg.job0 + i];
    for (int i = tid; i < wg.n_jobs; i += NT) jhs[i] = c.jobs[wg.job0 + i];
    for (int i = tid; i < wg.n_f; i += NT) Fs[i] = 0.0;
    for (int i = tid; i < c.n_xs + wg.n_w; i += NT) xs[i] = make_double2(0.0, 0.0);
    if (tid == 0) gave_up = 0;
    bool alive = true;
    const int sx[2] = {c.xpos[min(tid, N - 1)], c.xpos[min(tid + NT, N - 1)]};
    const int j_first = wg.wave_job[wave], j_end = wg.wave_job[wave + 1];
    // the wave's first job (the headers and lanes of the others are read from
    // LDS while the job before runs)
    int4 job0 = j_first < j_end ? c.jobs[wg.job0 + j_first] : make_int4(0, 0, 0, 0);
    job0 = wave_uniform(job0);
    const int2 jlv0 = j_first < j_end ? c.jlane[(size_t)64 * (wg.job0 + j_first) + lane] : make_int2(0, 0);
    const int n_rp = FORM == kRadialInterp ? max(5, lam_max + 1) : 2 * (lam_max + 1);
    const int n_pb = (lam_max + 1) * (lam_max + 2) / 2;
    const size_t j0 = (size_t)j * a.pt.n_pts;
    const double sc = a.Zp / T.vvec[j];
    const unsigned tag0 = (unsigned)*c.epoch;
    int spin = c.spin;
    asm volatile("" : "+s"(spin));   // stays in its register: no reload on the way to a poll
    unsigned long long* exch = c.exch + (size_t)j * 8 * N;   // [2][4][N]

    // What the next new point needs, in registers before its use: a stage
    // ahead its grid node, R factor tid, Legendre factor tid and the phase of
    // its radial function tid, while phase 3 runs its table entries.
    TabT tv[FORM == kRadialInterp ? 1 : FP];
    double rpv = 0.0, pbv = 0.0;
    double2 phv = make_double2(0.0, 0.0);
    int kload = 0, kcur = 0;
    auto load_factors = [&](int p) {
        kload = a.pt.kidx[j0 + p];
        if (tid < n_rp) rpv = a.pt.rpow[(j0 + p) * kRpow + tid];
        if (tid < n_pb) pbv = a.pt.pbar[(j0 + p) * kMaxPb + tid];
        if (tid < n_rad) phv = a.pt.ph[(j0 + p) * n_f + rad0 + tid];
    };
    auto load_table = [&]() {
        kcur = __builtin_amdgcn_readfirstlane(kload);
        if constexpr (FORM != kRadialInterp) {
            const TabT* tab;
            if constexpr (FORM == kRadialMoments32) tab = T.tab32;
            else tab = T.tab;
            const char* row = reinterpret_cast<const char*>(tab + (size_t)kcur * n_frow);
#pragma unroll
            for (int i = 0; i < FP; ++i) tv[i] = *reinterpret_cast<const TabT*>(row + entx[i]);
        }
    };
    // R factors and phases of point p to LDS (phases by parity of the point)
    auto store_factors = [&](int p) {
        if (tid < n_rp) rps[tid] = rpv;
        if (tid < n_rad) phs[(p & 1) * n_rad + tid] = phv;
    };
    auto form_F = [&]() {
#pragma unroll
        for (int i = 0; i < FP; ++i)
            if (entf[i] >= 0) {
                const int l = entf[i] >> 20;
                double f;
                if constexpr (FORM == kRadialInterp)
                    f = interp_value(T.ftab, n_frow, n_r, kcur, rps, c.ents[ent0 + tid + i * NT].x, l);
                else
                    {
                    const double2 rp = reinterpret_cast<const double2*>(rps)[l];
                    f = radial_f((double)tv[i].x, (double)tv[i].y, rp.x, rp.y);
                }
                Fs[entf[i] & 0xfffff] = f;
            }
        if (tid < n_pb) pbs[tid] = pbv;
    };
    auto form_G = [&]() {
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            const int e = tid + i * NT;
            if (e < n_g) Gs[e] = gpi[i] >= 0 ? gco[i] * pbs[gpi[i]] : 0.0;
        }
        for (int e = tid + GP * NT; e < n_g; e += NT) {
            const int q = c.gsrc[g0 + e], p = q >= 0 ? T.gpb[q] : -1;
            Gs[e] = p >= 0 ? T.gcoef[q] * pbs[p] : 0.0;
        }
    };

    // the first point: F, Pbar, x'
    load_factors(0);
    load_table();
    store_factors(0);
    __syncthreads();
    form_F();
    const bool rev = ADJ && c.adjoint == kChunkReverse;
    double2* const mu = rev ? c.mu + (size_t)j * a.n_pad : nullptr;
    {
        const double w = rev ? rk4_weight(1, c.h[0]) : 1.0;   // reverse: the first input is h/6 lambda
        for (int i = tid; i < N; i += NT) {
            double2 x = a.X[(size_t)j * a.n_pad + i];
            if (rev) x = make_double2(w * x.x, w * x.y);
            xs[c.xpos[i]] = dephase(a.pt.ph[j0 * n_f + T.st_rad[i]], x);
        }
        if (rev && tid < n_out) mu[out.x] = make_double2(w * x0.x, w * x0.y);
    }
    load_factors(1);

    for (int step = 0; step < c.n_steps; ++step) {
        const double h = c.h[step], h6 = rk4_weight(1, h), h3 = rk4_weight(2, h);
#pragma unroll 1
        for (int stage = 1; stage <= 4; ++stage) {
            const int p = stage == 1 ? 2 * step : (stage == 4 ? 2 * step + 2 : 2 * step + 1);
            // the point of the stage after this one
            const bool last = step + 1 == c.n_steps && stage == 4;
            const int pn = stage == 2 || stage == 4 ? p : p + 1;
            const unsigned tag = tag0 + 4 * step + stage;   // of the x' this stage writes
            // keeps the addresses derived from these out of the registers that
            // live across stages
            asm volatile("" : "+v"(tid), "+v"(lane), "+v"(out.x), "+v"(out.y), "+v"(out.z));
#pragma unroll
            for (int i = 0; i < GP; ++i) asm volatile("" : "+v"(gpi[i]));
#pragma unroll
            for (int g = 0; g < kChunkGroups; ++g) asm volatile("" : "+v"(grp[g].x), "+v"(grp[g].y));
#pragma unroll
            for (int i = 0; i < FP; ++i) asm volatile("" : "+v"(entf[i]));
            if constexpr (FORM != kRadialInterp)
#pragma unroll
                for (int i = 0; i < FP; ++i) asm volatile("" : "+v"(entx[i]));
            if (!local && !(step == 0 && stage == 1) &&
                !chunk_take<NT>(exch + (size_t)((tag - 1) & 1) * 4 * N, N, tag - 1, sx, c.xpos, xs, alive ? spin : 1, tid)) {
                alive = false;
                gave_up = 1;
            }
            __syncthreads();
            // a path whose words did not come ends at the next step: its flag
            // is latched and its amplitudes are not written
            if (!local && stage == 1 && *(volatile int*)&gave_up) {
                if (tid == 0) atomicOr(a.flag, 2);
                return;
            }
            // W = F x'
            {
                const double2* F2 = reinterpret_cast<const double2*>(Fs);
                int4 job = job0;
                int2 jlv = jlv0;
                for (int i = j_first; i < j_end; ++i) {
                    const int in = min(i + 1, j_end - 1);
                    const int4 next = jhs[in];
                    const int2 jln = jls[64 * in + lane];
                    if (job.w == 1) chunk_job<1>(F2, xs, Ws, job, jlv, lane);
                    else if (job.w == 2) chunk_job<2>(F2, xs, Ws, job, jlv, lane);
                    else if (job.w == 3) chunk_job<3>(F2, xs, Ws, job, jlv, lane);
                    else chunk_job<4>(F2, xs, Ws, job, jlv, lane);
                    job = wave_uniform(next);
                    jlv = jln;
                }
            }
            if (stage == 2 || stage == 4 || (step == 0 && stage == 1)) form_G();
            __syncthreads();
            if (pn != p) {
                store_factors(pn);
                if (NT == 512) load_table();   // 1024 threads: no registers for it yet
            }
            // the wave's chain of y = G W
            if (n_grp == 1) chunk_groups<1>(grp, Ws, Gs, Ps, chain, n_out, kb);
            else chunk_groups<2>(grp, Ws, Gs, Ps, chain, n_out, kb);
            for (int g = kChunkGroups; g < n_grp; g += 2) {
                const int2 q[2] = {grps[64 * (halves * g + half) + lane], grps[64 * (halves * min(g + 1, n_grp - 1) + half) + lane]};
                if (g + 1 == n_grp) chunk_groups<1>(q, Ws, Gs, Ps, chain, n_out, kb);
                else chunk_groups<2>(q, Ws, Gs, Ps, chain, n_out, kb);
            }
            if (NT != 512 && pn != p) load_table();
            __syncthreads();
            // the slope and the RK4 update of output tid
            if (tid < n_out) {
                double2 t[kChains];
#pragma unroll
                for (int k = 0; k < kChains; ++k) t[k] = Ps[k * n_out + tid];
#pragma unroll
                for (int d = 1; d < kChains; d *= 2)
#pragma unroll
                    for (int k = 0; k + d < kChains; k += 2 * d) {
                        t[k].x += t[k + d].x;
                        t[k].y += t[k + d].y;
                    }
                const double2 py = cmul(phs[(p & 1) * n_rad + out.y], t[0]);
                const double2 K = make_double2(sc * py.y, -sc * py.x);   // -(i/v) Zp ph y
                double2 u;
                if (!rev) {
                    xa = rk4_accumulate(stage, x0, xa, K, stage == 1 || stage == 4 ? h6 : h3);
                    u = xa;
                    if (stage < 4) u = rk4_next_input(stage, x0, K, h);
                } else {
                    // nu = M^H mu = -K; lambda of the step before is lambda + the
                    // four nu; next mu = h/3 lambda + h nu, h/3 lambda + h/2 nu,
                    // h/6 lambda + h/2 nu, then h'/6 of the new lambda
                    xa = stage == 1 ? x0 : xa;
                    xa = make_double2(xa.x - K.x, xa.y - K.y);
                    const double wn = stage == 1 ? h : 0.5 * h, wl = stage < 3 ? h3 : h6;
                    u = make_double2(wl * x0.x - wn * K.x, wl * x0.y - wn * K.y);
                    if (stage == 4 && !last) {
                        const double w = rk4_weight(1, c.h[step + 1]);
                        u = make_double2(w * xa.x, w * xa.y);
                    }
                    if (!last) mu[(size_t)(4 * step + stage) * c.v + out.x] = u;
                }
                if (ADJ && !rev) {
                    double2* keep = stage < 4 ? c.us + (size_t)(3 * step + stage - 1) * c.v : c.xs + (size_t)(step + 1) * c.v;
                    keep[(size_t)j * a.n_pad + out.x] = u;
                }
                if (!last) {
                    const double2 xn = dephase(phs[(pn & 1) * n_rad + out.y], u);
                    if (local) xs[out.z] = xn;
                    else chunk_put(exch + (size_t)(tag & 1) * 4 * N, N, out.x, xn, tag);
                }
                if (stage == 4) {
                    if (!rev && (!isfinite(xa.x) || !isfinite(xa.y))) atomicOr(a.flag, 1);
                    x0 = xa;
                    if (last && (!ADJ || rev) && !*(volatile int*)&gave_up) a.X[(size_t)j * a.n_pad + out.x] = xa;
                }
            }
            if (last && !local && tid == 0 && *(volatile int*)&gave_up) atomicOr(a.flag, 2);
            if (pn != p) form_F();
            if (stage == 2 || (stage == 4 && !last)) load_factors(p + 1);
        }
    }
}

// Operator application with the grid of k_stage (see StageArgs), ROWS rows
// per workgroup (kRowsPerBlock, or kApplyRowsLarge where that does not fit
// the LDS); GG: the large-basis form (angular factors formed in phase 3 from
// the coefficient tables, F from the moment table as in every k_apply).
template <int ROWS, bool GG = false>
__global__ __launch_bounds__(kStageThreads) void k_apply(ApplyArgs a) {
    extern __shared__ double2 smem2[];
    stage_entry<1, ROWS, GG>(a.s[blockIdx.z], reinterpret_cast<char*>(smem2));
}

// grad[j] = (dL/da, dL/dc, dL/db): the k_apply shares of path j (slots 2, 3
// and 0 + 1 of gpart[j][kGradSlots][n_part]) summed in a fixed order, so that
// the result does not depend on the order in which workgroups ran.
__global__ __launch_bounds__(192) void k_grad_sum(const double* __restrict__ gpart, int n_part,
                                                  double* __restrict__ grad) {
    // wave t: derivative by a, c, b (its two shares)
    const int j = blockIdx.x, t = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double* g = gpart + (size_t)j * kGradSlots * n_part + (t < 2 ? (size_t)(2 + t) * n_part : 0);
    double s = 0.0;
    for (int i = lane; i < (t < 2 ? n_part : 2 * n_part); i += 64) s += g[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) grad[(size_t)j * 3 + t] = s;
}

// The gradient shares of a run of reverse steps (GradArgs): grid x = row
// tiles, y = paths, z = 2 (4 s + r) + (first or second b term).  They feed
// nothing back, so the chain of stages (k_chunk in its reverse form) keeps
// its adjoint inputs and these launches fill the chip afterwards.
template <int ROWS>
__global__ __launch_bounds__(kStageThreads) void k_grad(GradArgs g) {
    extern __shared__ double2 smem2[];
    const int d = blockIdx.z & 1, r = (blockIdx.z >> 1) & 3, s = blockIdx.z >> 3;
    StageArgs a = g.s;
    a.p = 2 * s + (r == 0 ? 0 : (r == 3 ? 2 : 1));
    a.z = g.z[a.p];
    a.deriv = d + 1;
    a.gslot = d;
    a.model = d == 0;
    a.u_in = g.us[r] - (size_t)s * g.ustep[r];
    a.dv = g.mu + (size_t)(4 * s + r) * g.v;
    a.grad += (size_t)(g.q0 - 4 * s + r) * gridDim.x;
    stage_entry<1, ROWS, false>(a, reinterpret_cast<char*>(smem2));
}

__global__ __launch_bounds__(256) void k_clear(double* __restrict__ p, size_t n) {
    for (size_t i = blockIdx.x * size_t(256) + threadIdx.x; i < n; i += gridDim.x * size_t(256)) p[i] = 0.0;
}

__global__ void k_chunk_counter(int* chunk, int reset) {
    if (reset) *chunk = 0;
    else *chunk += 1;
}

// tab[k][idx[e]].y += val[e] for every grid node k; grid (entries, nodes)
__global__ void k_table_shift(double2* __restrict__ tab, int n_frow, const int* __restrict__ idx,
                              const double* __restrict__ val, int count) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    tab[(size_t)blockIdx.y * n_frow + idx[e]].y += val[e];
}

// Diagnostic path: Frow, G and phases of one (path, z) into scratch arrays.
// grid: x = [nbF Frow blocks | nbP phase blocks | G blocks].
__global__ __launch_bounds__(256) void k_slot_setup(SetupArgs a) {
    const Meta& m = *a.meta;
    const Tables& T = a.tb;
    const double z = a.z;
    const double b = T.bvec[a.j], v = T.vvec[a.j];
    const double R = sqrt(b * b + z * z);
    const int bx = blockIdx.x;
    if (bx < a.nbF) {
        const int d = bx * blockDim.x + threadIdx.x;
        if (d >= m.n_frow) return;
        int lp = 0;
        while (lp < m.l_max && d >= m.frow_off[lp + 1]) ++lp;
        const int e = (d - m.frow_off[lp]) % m.nV[lp];
        const int k = grid_index(R, m.r_max, m.n_r);
        const int lam = T.col_lam[m.col_off[lp] + e];
        if (T.ftab) {
            double rp[kRpow];
            int kk = -1;
            if (R < m.r_max) {
                kk = interp_stencil(R, m.r_max, m.n_r, rp);
            } else {
                double f = m.r_max / R;
                for (int q = 0; q <= lam; ++q) {
                    rp[q] = f;
                    f *= m.r_max / R;
                }
            }
            a.Frow[d] = interp_value(T.ftab, m.n_frow, m.n_r, kk, rp, d, lam);
        } else if (T.tab32) {
            const float2 ab = T.tab32[(size_t)k * m.n_frow + d];
            double fa, fb;
            scaled_factors(R, k, lam, m.r_max, m.n_r, &fa, &fb);
            a.Frow[d] = (double)ab.x * fa + (double)ab.y * fb;
        } else {
            a.Frow[d] = radial_at(T.tab[(size_t)k * m.n_frow + d], R, lam);
        }
        return;
    }
    if (bx < a.nbF + a.nbP) {
        const int i = (bx - a.nbF) * blockDim.x + threadIdx.x;
        if (i < m.n_states) a.PH[i] = phase(T.eps[i], z, v);
        return;
    }
    __shared__ double pb[kMaxPb];
    if ((int)threadIdx.x <= m.lam_max) legendre_column(m.lam_max, threadIdx.x, z / R, pb);
    __syncthreads();
    const int i = (bx - a.nbF - a.nbP) * blockDim.x + threadIdx.x;
    if (i < m.n_g) {
        const int p = T.gpb[i];
        a.G[i] = p >= 0 ? T.gcoef[i] * pb[p] : 0.0;
    }
}

// Dense D_T (Eq. D1) with phases: H[row][col] = Zp ph_row conj(ph_col) sum_lambda G F.
__global__ void k_couplings_dense(const Meta* __restrict__ mp_, const double* __restrict__ Frow,
                                  const double* __restrict__ G, const double2* __restrict__ PH, double Zp,
                                  double2* __restrict__ H) {
    const Meta& m = *mp_;
    const int N = m.n_states;
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = blockIdx.y;
    if (col >= N) return;
    int lp = 0, l = 0;
    while (lp < m.l_max && row >= m.state_off[lp + 1]) ++lp;
    while (l < m.l_max && col >= m.state_off[l + 1]) ++l;
    const int rp = row - m.state_off[lp], rc = col - m.state_off[l];
    const int qp = rp / m.n_l[lp], np = rp - qp * m.n_l[lp];
    const int q = rc / m.n_l[l], n = rc - q * m.n_l[l];
    int e0 = 0, g0 = 0;
    for (int ll = 0; ll < l; ++ll) {
        const int nlam = min(ll, lp) + 1;
        e0 += nlam * m.n_l[ll];
        g0 += nlam * (2 * ll + 1);
    }
    const double* Fr = Frow + m.frow_off[lp] + (size_t)np * m.nV[lp];
    const double* Gr = G + m.g_off[lp] + (size_t)qp * m.gcols[lp];
    double acc = 0.0;
    for (int lam = abs(l - lp); lam <= l + lp; lam += 2) {
        acc += Gr[g0 + q] * Fr[e0 + n];
        e0 += m.n_l[l];
        g0 += 2 * l + 1;
    }
    const double2 pr = PH[row], pc = PH[col];
    const double2 w = make_double2(pr.x * pc.x + pr.y * pc.y, pr.y * pc.x - pr.x * pc.y);  // pr conj(pc)
    H[(size_t)row * N + col] = make_double2(Zp * acc * w.x, Zp * acc * w.y);
}

__global__ void k_probabilities(const double2* __restrict__ X, int n_states, int n_pad,
                                double* __restrict__ P, double* __restrict__ norm) {
    const int j = blockIdx.x;
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n_states; i += blockDim.x) {
        const double2 x = X[(size_t)j * n_pad + i];
        const double p = x.x * x.x + x.y * x.y;
        if (P) P[(size_t)j * n_pad + i] = p;
        s += p;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0 && norm) norm[j] = red[0];
}

}  // namespace

int stage_chunks(const Meta& m, int rows) {
    int n = 0;
    for (int lp = 0; lp <= m.l_max; ++lp) n += (m.n_l[lp] + rows - 1) / rows;
    return n;
}

namespace {
// Rows [r0, r0 + nrows) of block l' of one path (vo: offset of the block's
// model-potential rows).
StageTile make_tile(const Meta& m, int lp, int r0, int nrows, int vo) {
    StageTile t{};
    t.lp = lp;
    t.row0 = r0;
    t.nrows = nrows;
    t.nmp = 2 * lp + 1;
    t.nV = m.nV[lp];
    t.gcols = m.gcols[lp];
    t.frow_off = m.frow_off[lp];
    t.col_off = m.col_off[lp];
    t.g_off = m.g_off[lp];
    t.gcol_off = m.gcol_off[lp];
    t.state_off = m.state_off[lp];
    t.rad_off = m.rad_off[lp];
    t.n_l = m.n_l[lp];
    t.xs_off = m.xs_off[lp];
    t.xs_stride = m.xs_stride[lp];
    t.vo = vo;
    return t;
}
}  // namespace

void stage_tiles(const Meta& m, int rows, std::vector<StageTile>& out) {
    out.clear();
    int vo = 0;
    for (int lp = 0; lp <= m.l_max; ++lp) {
        for (int r0 = 0; r0 < m.n_l[lp]; r0 += rows) out.push_back(make_tile(m, lp, r0, std::min(rows, m.n_l[lp] - r0), vo));
        vo += m.n_l[lp] * m.n_l[lp];
    }
}

void stage_tiles_balanced(const Meta& m, int rows, int n_launch, long long wg_slots, std::vector<StageTile>& out) {
    out.clear();
    int cap[kMaxL + 1];
    long long per_path = 0;
    for (int lp = 0; lp <= m.l_max; ++lp) {
        cap[lp] = rows;
        per_path += (m.n_l[lp] + rows - 1) / rows;
    }
    for (int lp = m.l_max; lp >= 0 && rows > 1; --lp) {
        const int extra = (m.n_l[lp] + rows - 2) / (rows - 1) - (m.n_l[lp] + rows - 1) / rows;
        if ((long long)n_launch * (per_path + extra) <= wg_slots) {
            cap[lp] = rows - 1;
            per_path += extra;
        }
    }
    int vo = 0;
    for (int lp = 0; lp <= m.l_max; ++lp) {
        const int n = m.n_l[lp], nt = (n + cap[lp] - 1) / cap[lp];
        for (int ti = 0, r0 = 0; ti < nt; ++ti) {
            const int nr = n / nt + (ti < n % nt ? 1 : 0);
            out.push_back(make_tile(m, lp, r0, nr, vo));
            r0 += nr;
        }
        vo += n * n;
    }
}

int stage_smem_bytes(const Meta& m, int rows, bool gg) {
    int best = 0;
    for (int lp = 0; lp <= m.l_max; ++lp) {
        const size_t nmp = gg ? 0 : 2 * lp + 1;
        const size_t bytes = m.n_xs * sizeof(double2) + (size_t)rows * m.gcols[lp] * sizeof(double2) +
                             (size_t)m.n_f * sizeof(double2) + (size_t)rows * m.nV[lp] * sizeof(double) +
                             nmp * m.gcols[lp] * sizeof(double) + (kRpow + kMaxPb) * sizeof(double) +
                             (size_t)m.gcols[lp] * sizeof(int2);
        if ((int)bytes > best) best = (int)bytes;
    }
    return best;
}

bool stage_rows_fit(const Meta& m, int rows) { return phase3_fits(rows, 2 * m.l_max + 1); }

hipError_t stage_set_smem_limit(int, int bytes) {
    static SmemLimit limit(0);
#define WPCCC_FN_PAIR(R)                                                                        \
    (const void*)k_stage<R, false, false>, (const void*)k_stage<R, false, true>,                 \
        (const void*)k_stage<R, true, true>, (const void*)k_stage<R, true, false>,
#define WPCCC_FN_GG(R) (const void*)k_stage<R, false, true, true>, (const void*)k_stage<R, true, true, true>,
    const void* fns[] = {WPCCC_STAGE_ROWS(WPCCC_FN_PAIR) WPCCC_STAGE_ROWS_GG(WPCCC_FN_GG)(const void*)k_apply<kRowsPerBlock>,
                         (const void*)k_apply<kApplyRowsLarge>, (const void*)k_grad<kRowsPerBlock>,
                         (const void*)k_grad<kApplyRowsLarge>, (const void*)k_apply<4, true>,
                         (const void*)k_apply<2, true>, (const void*)k_apply<1, true>};
#undef WPCCC_FN_PAIR
#undef WPCCC_FN_GG
    return limit.raise(bytes, [&]() {
        hipError_t e = hipSuccess;
        for (const void* f : fns)
            if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        return e;
    });
}

int stage_wgs_per_cu(int rows, int smem) {
    const void* f = nullptr;
    switch (rows) {
#define WPCCC_CASE(R) \
    case R: f = (const void*)k_stage<R, false, false>; break;
        WPCCC_STAGE_ROWS(WPCCC_CASE)
#undef WPCCC_CASE
        default: return 0;
    }
    int dev = 0, per_cu = 0, lds_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, kStageThreads, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    // the occupancy query without dynamic LDS (above 64 KiB it would need the
    // kernel attribute first), then the LDS bound
    return smem > 0 ? std::min(per_cu, lds_cu / smem) : per_cu;
}

// Whether the tiles of `rows` rows of all paths, with their F, could be resident
// at once at two workgroups per CU: the size up to which an explicit
// WPCCC_LAUNCH_PERSISTENT is taken.
bool tiles_resident(const Meta& m, int n_traj, int rows) {
    size_t smem = 0;
    for (int lp = 0; lp <= m.l_max; ++lp)
        smem = std::max(smem, (m.n_xs + (size_t)rows * m.gcols[lp] + m.n_f) * sizeof(double2) +
                                  ((size_t)rows * m.nV[lp] + (size_t)(2 * lp + 1) * m.gcols[lp] + kRpow + kMaxPb) * sizeof(double) +
                                  (size_t)m.gcols[lp] * sizeof(int2) + (size_t)m.nV[lp] * sizeof(int));
    int dev = 0, n_cu = 0, coop = 0, lds_cu = 0;
    if (smem > (size_t)kMaxDynLds || !stage_rows_fit(m, rows) || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
        hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const long long grid = 8 * (((long long)n_traj * stage_chunks(m, rows) + 7) / 8);
    return grid <= (long long)n_cu * std::min(2, (int)(lds_cu / smem));
}

namespace {

// k_chunk's instances: form, threads, table entries per thread
#define WPCCC_CHUNK_FORMS(X)                                                                               \
    X(kRadialMoments, 1024, 2) X(kRadialMoments, 512, 8) X(kRadialMoments, 512, 12) X(kRadialMoments, 512, 16)           \
    X(kRadialMoments32, 1024, 2) X(kRadialMoments32, 512, 8) X(kRadialMoments32, 512, 12) X(kRadialMoments32, 512, 16) \
    X(kRadialInterp, 1024, 2) X(kRadialInterp, 512, 8) X(kRadialInterp, 512, 12) X(kRadialInterp, 512, 16)

const void* chunk_fn(int form, int nt, int fp, bool adjoint = false) {
#define WPCCC_CASE(F, T, P) \
    if (form == F && nt == T && fp == P) return adjoint ? (const void*)k_chunk<F, T, P, F == kRadialMoments> : (const void*)k_chunk<F, T, P, false>;
    WPCCC_CHUNK_FORMS(WPCCC_CASE)
#undef WPCCC_CASE
    return nullptr;
}

}  // namespace

namespace {

// Splits the n_f radial functions of a path over at most G workgroups (runs
// of consecutive functions, the largest run's cost minimised) and writes the
// index tables k_chunk reads.  Returns false where a field, the entries per
// thread, the outputs or the LDS of a workgroup would not fit.  whole: no
// workgroup holds functions of two l'.
bool chunk_split(const Meta& m, int G, int threads, bool whole, ChunkTables& t) {
    t = ChunkTables{};
    t.nt = threads;
    const int waves = threads / 64, halves = waves / kChains;
    if ((long long)m.n_frow > (long long)G * threads * (threads == 1024 ? 2 : 16)) return false;   // entries per thread
    auto blocks4 = [](int n) { return (n + 3) / 4; };
    auto n_lam = [](int l, int lp) { return std::min(l, lp) + 1; };
    // x' rows in whole pairs of blocks of four n, at a stride of 4 modulo 8 (in
    // 16-byte units), which spreads the four rows x four n of a load over all
    // banks; the padding stays zero.  Three more rows follow the last: a group
    // of four rows may reach past those of its l (products that nothing uses).
    int xs_off[kMaxL + 1], xs_stride[kMaxL + 1];
    for (int l = 0; l <= m.l_max; ++l) {
        xs_off[l] = t.n_xs;
        xs_stride[l] = (m.n_l[l] + 7) / 8 * 8 + 4;
        t.n_xs += (2 * l + 1) * xs_stride[l];
        if (m.n_l[l] > 0x3fff) return false;
    }
    t.n_xs += 3 * xs_stride[m.l_max];
    if (m.n_frow > 0x7fffffff / 16 || m.l_max > 11) return false;
    int kbl[kMaxL + 1];           // column blocks of each chain
    double per_row[kMaxL + 1];    // cost of a row, in MFMAs
    for (int lp = 0; lp <= m.l_max; ++lp) {
        kbl[lp] = blocks4((m.gcols[lp] + kChains - 1) / kChains);
        if (m.gcols[lp] > 0x3ff || kbl[lp] > 31) return false;
        double sums = 0.0;
        for (int l = 0; l <= m.l_max; ++l) sums += n_lam(l, lp) * blocks4(m.n_l[l]) * 2.0 * blocks4(2 * l + 1);
        per_row[lp] = sums / 16 + kChains * kbl[lp] * 2.0 * blocks4(2 * lp + 1) / 16 + m.nV[lp] * 0.03;
    }
    struct Seg {
        int lp, r0, nr;
    };
    auto split = [&](double cap, std::vector<std::vector<Seg>>& out) {
        out.assign(1, {});
        double used = 0.0;
        for (int lp = 0; lp <= m.l_max; ++lp) {
            if (whole && !out.back().empty()) {
                if ((int)out.size() == G) return false;
                out.push_back({});
                used = 0.0;
            }
            for (int r0 = 0; r0 < m.n_l[lp];) {
                const int nr = std::min((int)((cap - used) / per_row[lp]), m.n_l[lp] - r0);
                if (nr > 0) {
                    out.back().push_back(Seg{lp, r0, nr});
                    used += nr * per_row[lp];
                    r0 += nr;
                }
                if (r0 < m.n_l[lp]) {
                    if (out.back().empty() || (int)out.size() == G) return false;
                    out.push_back({});
                    used = 0.0;
                }
            }
        }
        return true;
    };
    double lo = 0.0, hi = 1.0;
    std::vector<std::vector<Seg>> wgs, best;
    for (int lp = 0; lp <= m.l_max; ++lp) hi += (m.n_l[lp] + 1) * per_row[lp];
    for (int it = 0; it < 40; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (split(mid, wgs)) {
            hi = mid;
            best = wgs;
        } else {
            lo = mid;
        }
    }
    if (best.empty()) return false;
    t.G = (int)best.size();
    t.xpos.resize(m.n_states);
    for (int l = 0; l <= m.l_max; ++l)
        for (int q = 0; q <= 2 * l; ++q)
            for (int n = 0; n < m.n_l[l]; ++n)
                t.xpos[(size_t)m.state_off[l] + q * m.n_l[l] + n] = xs_off[l] + q * xs_stride[l] + n;
    size_t smem = 0;
    int most_ent = 0;
    for (const auto& segs : best) {
        ChunkWG w{};
        w.ent0 = (int)t.ents.size();
        w.job0 = (int)t.jobs.size();
        w.grp0 = (int)t.grps.size() / 64;
        w.out0 = (int)t.outs.size();
        w.rad0 = m.rad_off[segs[0].lp] + segs[0].r0;
        w.g0 = (int)t.gsrc.size();
        // W, angular factors and outputs of each segment, all with the block
        // count of the segment that needs most
        std::vector<int> seg_w;
        for (const Seg& s : segs) w.kb = std::max(w.kb, kbl[s.lp]);
        const int kb = w.kb;
        for (const Seg& s : segs) {
            const int lp = s.lp, nmp = 2 * lp + 1, nu = blocks4(nmp), nrg = blocks4(s.nr), per = kChains * kb * 16;
            const int out0 = w.n_out, w0 = w.n_w, g0 = w.n_g;
            seg_w.push_back(w0);
            for (int qp = 0; qp < nmp; ++qp)
                for (int r = 0; r < s.nr; ++r)
                    t.outs.push_back(make_int4(m.state_off[lp] + qp * m.n_l[lp] + s.r0 + r, w.n_rad + r,
                                               xs_off[lp] + qp * xs_stride[lp] + s.r0 + r, 0));
            w.n_out += nmp * s.nr;
            w.n_rad += s.nr;
            w.n_w += nrg * per;
            for (int u = 0; u < nu; ++u)
                for (int c = 0; c < kChains; ++c)
                    for (int b = 0; b < kb; ++b)
                        for (int k = 0; k < 4; ++k)
                            for (int i = 0; i < 4; ++i) {
                                const int qp = 4 * u + i, g = c + kChains * (4 * b + k);
                                t.gsrc.push_back(qp < nmp && g < m.gcols[lp] ? m.g_off[lp] + qp * m.gcols[lp] + g : -1);
                            }
            w.n_g += nu * per;
            // four (row group, m' group) pairs per MFMA
            const int pairs = nrg * nu;
            for (int p0 = 0; p0 < pairs; p0 += 4)
                for (int lane = 0; lane < 64; ++lane) {
                    const int blk = (lane & 15) >> 2, p = std::min(p0 + blk, pairs - 1), rg = p / nu, u = p - rg * nu;
                    const int row = 4 * rg + (lane >> 4), qp = 4 * u + (lane & 3);
                    const bool ok = p0 + blk < pairs && row < s.nr && qp < nmp;
                    const int at = (lane >> 4) * 4 + (lane & 3), gp = g0 + u * per + at;
                    if (gp > 0xffff) return false;
                    t.grps.push_back(make_int2((w0 + rg * per + at) | (gp << 16), ok ? out0 + qp * s.nr + row : -1));
                }
        }
        // the waves of a chain take every halves-th group each
        while (((int)t.grps.size() / 64 - w.grp0) % halves)
            for (int lane = 0; lane < 64; ++lane) t.grps.push_back(make_int2(0, -1));
        w.n_grp = ((int)t.grps.size() / 64 - w.grp0) / halves;
        // jobs: 16 rows (l' n', lambda) against the rows of one l
        struct Job {
            int4 h;
            std::vector<int2> lanes;
            int cost;
        };
        std::vector<Job> jobs;
        for (int l = 0; l <= m.l_max; ++l) {
            struct Row {
                int seg, r, e, g;   // segment, row of it, Frow column and G column of the block
                int lam;
            };
            std::vector<Row> rows;
            for (size_t si = 0; si < segs.size(); ++si) {
                const int lp = segs[si].lp;
                int e0 = 0, g0 = 0;
                for (int ll = 0; ll < l; ++ll) {
                    e0 += n_lam(ll, lp) * m.n_l[ll];
                    g0 += n_lam(ll, lp) * (2 * ll + 1);
                }
                for (int r = 0; r < segs[si].nr; ++r)
                    for (int k = 0; k < n_lam(l, lp); ++k)
                        rows.push_back(Row{(int)si, r, e0 + k * m.n_l[l], g0 + k * (2 * l + 1), std::abs(l - lp) + 2 * k});
            }
            const int np = (m.n_l[l] + 7) / 8;
            for (size_t r0 = 0; r0 < rows.size(); r0 += 16) {
                // operand order: [pair of n blocks][lane = (n % 4) * 16 + row][block of the
                // pair]; consecutive entries take four n of a row (a 64-byte run of the
                // table), then the next row (other banks of the LDS)
                for (int ks = 0; ks < blocks4(m.n_l[l]); ++ks)
                    for (int i = 0; i < 16 && r0 + i < rows.size(); ++i)
                        for (int n = 4 * ks; n < std::min(4 * ks + 4, m.n_l[l]); ++n) {
                            const Row& rw = rows[r0 + i];
                            const Seg& s = segs[rw.seg];
                            t.ents.push_back(make_int2(m.frow_off[s.lp] + (s.r0 + rw.r) * m.nV[s.lp] + rw.e + n,
                                                       (w.n_f + ((ks / 2) * 64 + (n & 3) * 16 + i) * 2 + (ks & 1)) |
                                                           (rw.lam << 20)));
                        }
                for (int q0 = 0; q0 <= 2 * l; q0 += 16) {
                    const int nu = std::min(4, blocks4(2 * l + 1 - q0));
                    Job jb;
                    jb.h = make_int4(w.n_f, xs_off[l] + q0 * xs_stride[l], xs_stride[l] | (np << 16), nu);
                    jb.cost = 12 + np * (2 + 4 * nu);
                    for (int lane = 0; lane < 64; ++lane) {
                        const size_t i = r0 + 4 * ((lane & 15) >> 2) + (lane >> 4);
                        int pos[4] = {0, 0, 0, 0};
                        for (int u = 0; u < nu; ++u) {
                            const int q = q0 + 4 * u + (lane & 3);
                            pos[u] = w.n_w + lane;   // read by nothing
                            if (i < rows.size() && q <= 2 * l) {
                                const Row& rw = rows[i];
                                pos[u] = seg_w[rw.seg] + (rw.r / 4) * kChains * kb * 16 + (rw.r & 3) +
                                         chunk_column(rw.g + q, kb);
                            }
                        }
                        jb.lanes.push_back(make_int2(pos[0] | (pos[1] << 16), pos[2] | (pos[3] << 16)));
                    }
                    jobs.push_back(jb);
                }
                w.n_f += np * 128;
            }
        }
        w.n_w += 64;
        if (w.n_w > 0xffff) return false;
        // jobs to waves: the longest first, each to the least loaded wave
        std::vector<int> order(jobs.size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return jobs[x].cost > jobs[y].cost; });
        std::vector<int> of_wave[kChunkWaves];
        int load[kChunkWaves] = {};
        for (int i : order) {
            const int v = (int)(std::min_element(load, load + waves) - load);
            of_wave[v].push_back(i);
            load[v] += jobs[i].cost;
        }
        for (int v = 0; v < waves; ++v) {
            w.wave_job[v] = w.n_jobs;
            for (int i : of_wave[v]) {
                t.jobs.push_back(jobs[i].h);
                t.jlane.insert(t.jlane.end(), jobs[i].lanes.begin(), jobs[i].lanes.end());
                ++w.n_jobs;
            }
        }
        w.wave_job[waves] = w.n_jobs;
        w.n_ent = (int)t.ents.size() - w.ent0;
        if (w.n_out > threads || w.n_rad > threads || w.n_f >= (1 << 20)) return false;
        most_ent = std::max(most_ent, w.n_ent);
        smem = std::max(smem, ((size_t)t.n_xs + w.n_w + kChains * (size_t)w.n_out + 2 * (size_t)w.n_rad + 32 * (size_t)halves * w.n_grp) *
                                      sizeof(double2) +
                                  ((size_t)w.n_f + w.n_g + kRpow + kMaxPb + 1 + 66 * (size_t)w.n_jobs) * sizeof(double));
        t.wgs.push_back(w);
    }
    if (smem > (size_t)kMaxDynLds) return false;
    t.smem = (int)smem;
    for (int fp : {2, 8, 12, 16})
        if (fp * threads >= most_ent && chunk_fn(kRadialMoments, threads, fp)) {
            t.fp = fp;
            return true;
        }
    return false;
}

}  // namespace

// A workgroup that holds functions of two l' holds the angular factors of
// both: large bases fit with one l' per workgroup only.
bool chunk_build(const Meta& m, int G, int threads, ChunkTables& t) {
    return chunk_split(m, G, threads, false, t) || chunk_split(m, G, threads, true, t);
}

// Paths per launch: those whose workgroups can be resident at once (with one
// workgroup per path nothing waits for another: any number).
int chunk_paths(const ChunkTables& t, int form, int n_traj, bool adjoint) {
    if (t.G == 1) return n_traj;
    int dev = 0, n_cu = 0, per_cu = 0, coop = 0;
    const void* f = chunk_fn(form, t.nt, t.fp, adjoint);
    if (!f || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, t.nt, t.smem) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    // the grid is rounded up to a multiple of eight workgroups (XCD order)
    const int resident = per_cu * n_cu;
    int n = std::min(n_traj, resident / t.G);
    while (n > 0 && 8 * ((n * t.G + 7) / 8) > resident) --n;
    return n;
}

hipError_t launch_chunk(const ChunkArgs& a, const ChunkTables& t, int form, hipStream_t st, const LaunchEv& ev) {
    const dim3 grid(8 * ((a.n_traj * a.G + 7) / 8)), block(t.nt);
    const void* f = chunk_fn(form, t.nt, t.fp, a.adjoint != 0);
    if (!f) return hipErrorInvalidValue;
    ChunkArgs arg = a;
    void* params[] = {&arg};
    if (ev.a) (void)hipEventRecord(ev.a, st);
    const hipError_t e = a.G > 1 ? hipLaunchCooperativeKernel(f, grid, block, params, t.smem, st)
                                 : hipLaunchKernel(f, grid, block, params, t.smem, st);
    if (ev.b) (void)hipEventRecord(ev.b, st);
    return e;
}

// The dynamic-LDS attribute of every k_chunk instance.
hipError_t chunk_set_smem_limit(int bytes) {
    static SmemLimit limit(64 * 1024);
    return limit.raise(bytes, [&]() {
        hipError_t e = hipSuccess;
#define WPCCC_CASE(F, T, P) \
    if (e == hipSuccess) \
        e = hipFuncSetAttribute((const void*)k_chunk<F, T, P, false>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); \
    if (e == hipSuccess && F == kRadialMoments) \
        e = hipFuncSetAttribute((const void*)k_chunk<F, T, P, F == kRadialMoments>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        WPCCC_CHUNK_FORMS(WPCCC_CASE)
#undef WPCCC_CASE
        return e;
    });
}

hipError_t launch_grad(const GradArgs& a, const Meta& hm, int n_traj, int n_steps, int smem, int rows, hipStream_t st,
                       const LaunchEv& ev) {
    const dim3 grid(stage_chunks(hm, rows), n_traj, 8 * n_steps);
    if (rows == kRowsPerBlock) WPCCC_LAUNCH(ev, k_grad<kRowsPerBlock>, grid, dim3(kStageThreads), smem, st, a);
    else if (rows == kApplyRowsLarge) WPCCC_LAUNCH(ev, k_grad<kApplyRowsLarge>, grid, dim3(kStageThreads), smem, st, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_apply(const ApplyArgs& a, int n_ops, const Meta& hm, int n_traj_launch, int smem, int rows,
                        bool gg, hipStream_t st, const LaunchEv& ev) {
    const dim3 grid(stage_chunks(hm, rows), n_traj_launch, n_ops);
    if (gg) {
        if (rows == 4) WPCCC_LAUNCH(ev, (k_apply<4, true>), grid, dim3(kStageThreads), smem, st, a);
        else if (rows == 2) WPCCC_LAUNCH(ev, (k_apply<2, true>), grid, dim3(kStageThreads), smem, st, a);
        else if (rows == 1) WPCCC_LAUNCH(ev, (k_apply<1, true>), grid, dim3(kStageThreads), smem, st, a);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    if (rows == kRowsPerBlock)
        WPCCC_LAUNCH(ev, k_apply<kRowsPerBlock>, grid, dim3(kStageThreads), smem, st, a);
    else if (rows == kApplyRowsLarge)
        WPCCC_LAUNCH(ev, k_apply<kApplyRowsLarge>, grid, dim3(kStageThreads), smem, st, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_chunk_counter(int* chunk, int reset, hipStream_t st) {
    hipLaunchKernelGGL(k_chunk_counter, dim3(1), dim3(1), 0, st, chunk, reset);
    return hipGetLastError();
}

hipError_t launch_clear(double* p, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_clear, dim3((unsigned)std::min<size_t>((n + 255) / 256, 2048)), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_grad_sum(const double* gpart, int n_part, double* grad, int n_traj, hipStream_t st) {
    hipLaunchKernelGGL(k_grad_sum, dim3(n_traj), dim3(192), 0, st, gpart, n_part, grad);
    return hipGetLastError();
}

hipError_t launch_table_nodes(const double2* tab, const int* dl, int n_frow, int n_r, double r_max, double* out,
                              hipStream_t st) {
    hipLaunchKernelGGL(k_table_nodes, dim3((n_frow + 255) / 256, n_r + 1), dim3(256), 0, st, tab, dl, n_frow, n_r,
                       r_max, out);
    return hipGetLastError();
}

hipError_t launch_table_f32(const double2* tab, const int* dl, int n_frow, int n_r, double r_max, float2* out,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_table_f32, dim3((n_frow + 255) / 256, n_r + 1), dim3(256), 0, st, tab, dl, n_frow, n_r, r_max,
                       out);
    return hipGetLastError();
}

hipError_t launch_table_shift(double2* tab, int n_frow, int n_r, const int* idx, const double* val, int count,
                              hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_table_shift, dim3((count + 255) / 256, n_r + 1), dim3(256), 0, st, tab, n_frow, idx, val,
                       count);
    return hipGetLastError();
}

hipError_t launch_moments(const double* r, const double* w, const double* phiT, const int* da, const int* db,
                          const int* dl, int n_r, int n_f, int n_frow, double2* tab, hipStream_t st) {
    const int nb = (n_frow + 127) / 128;
    hipLaunchKernelGGL(k_moments, dim3(nb), dim3(128), 0, st, r, w, phiT, da, db, dl, n_r, n_f, n_frow, tab);
    return hipGetLastError();
}

hipError_t launch_prologue(const PrologueArgs& a, int n_traj_launch, hipStream_t st, const LaunchEv& ev) {
    WPCCC_LAUNCH(ev, k_prologue, dim3(a.n, n_traj_launch), dim3(64), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_slot_setup(const SetupArgs& a, const Meta& hm, hipStream_t st, const LaunchEv& ev) {
    const int nbG = (hm.n_g + 255) / 256;
    WPCCC_LAUNCH(ev, k_slot_setup, dim3(a.nbF + a.nbP + nbG), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_stage(const StageArgs& a, const Meta& hm, int n_traj_launch, int smem, hipStream_t st, const LaunchEv& ev,
                        int rows) {
    const dim3 grid(8 * ((n_traj_launch * a.nwg + 7) / 8)), block(a.gg ? kStageThreadsGG : kStageThreads);
    StageArgs a1 = a;
    a1.n_paths = n_traj_launch;
    if (a.gg) {
        // large bases: cached F, angular factors from global memory
        if (!a.fc_cur) return hipErrorInvalidValue;
        switch (rows) {
#define WPCCC_CASE(R)                                                                                        \
    case R:                                                                                                  \
        if (a.tb.tab32) WPCCC_LAUNCH(ev, (k_stage<R, true, true, true>), grid, block, smem, st, a1);       \
        else WPCCC_LAUNCH(ev, (k_stage<R, false, true, true>), grid, block, smem, st, a1);                  \
        break;
            WPCCC_STAGE_ROWS_GG(WPCCC_CASE)
#undef WPCCC_CASE
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (rows) {
#define WPCCC_CASE(R)                                                                    \
    case R:                                                                              \
        if (a.tb.tab32 && a.fc_cur) WPCCC_LAUNCH(ev, (k_stage<R, true, true>), grid, block, smem, st, a1); \
        else if (a.tb.tab32) WPCCC_LAUNCH(ev, (k_stage<R, true, false>), grid, block, smem, st, a1);       \
        else if (a.fc_cur) WPCCC_LAUNCH(ev, (k_stage<R, false, true>), grid, block, smem, st, a1);       \
        else WPCCC_LAUNCH(ev, (k_stage<R, false, false>), grid, block, smem, st, a1);                    \
        break;
        WPCCC_STAGE_ROWS(WPCCC_CASE)
#undef WPCCC_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fpoint(const Meta* m, const Meta& hm, const Tables& tb, const PointArrays& pt, int p, int traj0,
                         int n_paths, void* fc, hipStream_t st, const LaunchEv& ev) {
    const dim3 grid((hm.n_frow + 255) / 256, n_paths);
    if (tb.tab32) WPCCC_LAUNCH(ev, k_fpoint<true>, grid, dim3(256), 0, st, m, tb, pt, p, traj0, fc);
    else WPCCC_LAUNCH(ev, k_fpoint<false>, grid, dim3(256), 0, st, m, tb, pt, p, traj0, fc);
    return hipGetLastError();
}

hipError_t launch_couplings_dense(const Meta* m, const Meta& hm, const double* Frow, const double* G,
                                  const double2* PH, double Zp, double2* H, hipStream_t st, const LaunchEv& ev) {
    WPCCC_LAUNCH(ev, k_couplings_dense, dim3((hm.n_states + 127) / 128, hm.n_states), dim3(128), 0, st, m, Frow,
                       G, PH, Zp, H);
    return hipGetLastError();
}

hipError_t launch_probabilities(const double2* X, int n_traj, int n_states, int n_pad, double* P, double* norm,
                                hipStream_t st, const LaunchEv& ev) {
    WPCCC_LAUNCH(ev, k_probabilities, dim3(n_traj), dim3(256), 0, st, X, n_states, n_pad, P, norm);
    return hipGetLastError();
}

}  // namespace wpccc
