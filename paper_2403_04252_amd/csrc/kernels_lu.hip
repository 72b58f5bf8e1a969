// Batched complex LU with partial pivoting (the overlap matrices S of Eq. 1)
// on gfx950.  Right-looking, one panel of kLUPanel columns per pass and one
// launch of each kernel per pass for every matrix of the batch:
//   k_lu_panel      the N - k0 rows of the panel in registers (one to four
//                   rows per thread, 512 threads): per column an argmax (largest
//                   |a|^2, ties to the lowest row), the row swap, the scaling
//                   of L and the rank-1 update of the remaining panel columns,
//                   behind one barrier
//   k_lu_swap_trsm  the panel's swaps on every other column (LAPACK getrf
//                   order) and U12 = L11^-1 A12, one thread per column
//   k_lu_update     A22 -= L21 U12 on MFMA (v_mfma_f64_16x16x4f64), 64 x 64
//                   output tiles, complex product as four real products
// and, for the explicit form of the derivative matrix, k_lu_rhs: M = S^-1 H
// from the finished factors.
#include <hip/hip_runtime.h>

#include "plan2c.h"

namespace wpccc {

namespace {

constexpr int kPanelThreads = 512;

typedef double dbl4 __attribute__((ext_vector_type(4)));

// Matrix y of a launch: slot `slot` of path pl (n_sub 0: the matrices lie one
// after another, without slots).
__device__ inline void job_of(const Jobs& J, int y, int& pl, int& slot) {
    if (J.n_sub == 0) {
        pl = 0;
        slot = y;
        return;
    }
    pl = J.path0 + y / J.n_sub;
    slot = J.slot[y % J.n_sub];
}

// Whether a launch's kernel has nothing to do for this matrix (LUStepArgs::skip_mode).
__device__ inline bool skipped(const LUStepArgs& a, size_t ms) {
    if (a.skip_mode == 0) return false;
    const bool s = a.skip[ms] != 0;
    return a.skip_mode == 1 ? s : !s;
}

__device__ inline double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Keeps the better of this lane's pivot candidate and that of the lane a DPP
// control moves here: the larger magnitude, the lower row on ties (lanes
// without a source compare with themselves).
template <int CTRL>
__device__ inline void better_pivot(double& m, int& i) {
    const int lo = __double2loint(m), hi = __double2hiint(m);
    const double om = __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                                       __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
    const int oi = __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false);
    if (om > m || (om == m && oi < i)) {
        m = om;
        i = oi;
    }
}

// ROWS rows per thread (N - k0 <= ROWS x 512), panels of up to NB columns: the
// panel's N - k0 rows live in registers (ROWS x NB complex values per thread).
//
// A column is a chain: argmax, the pivot row to everyone, reciprocal, update.
// Each wave finds its own candidate with DPP moves and puts its row beside its
// magnitude, so one barrier serves the choice and the row; two sets of the
// LDS arrays, taken in turn, need no barrier between columns.  Measured at
// N = 442, 16 matrices, per panel of 16 columns: 39 us (with shuffles, the row
// published after the choice and three barriers) -> 30 us.
template <int ROWS, int NB>
__global__ __launch_bounds__(kPanelThreads) void k_lu_panel(LUStepArgs a) {
    constexpr int kPanelRows = ROWS;
    constexpr int kWaves = kPanelThreads / 64;
    __shared__ double2 cand[2][kWaves][NB], xrows[2][NB];   // the waves' candidate rows, row j
    __shared__ double2 recip[2][kWaves];                    // reciprocals of the candidates
    __shared__ double redv[2][kWaves];
    __shared__ int redi[2][kWaves];
    int pl, slot;
    job_of(a.jobs, blockIdx.x, pl, slot);
    const int N = a.N, k0 = a.k0, nb = a.nb;
    const size_t ms = (size_t)pl * kSlots2C + slot;
    if (skipped(a, ms)) return;
    double2* A = a.LU + ms * (size_t)N * N;
    int* piv = a.piv + ms * N;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (k0 == 0) {
        int* perm = a.perm + ms * N;
        for (int i = t; i < N; i += kPanelThreads) perm[i] = i;
    }
    double2 v[kPanelRows][NB];
#pragma unroll
    for (int q = 0; q < kPanelRows; ++q) {
        const int i = k0 + t + kPanelThreads * q;
#pragma unroll
        for (int c = 0; c < NB; ++c)
            v[q][c] = (i < N && c < nb) ? A[i + (size_t)(k0 + c) * N] : make_double2(0.0, 0.0);
    }
    // Four columns per pass of a rolled loop, after which the registers rotate
    // by four: v[.][c] holds column (c + jj0) % NB.  Sixteen columns written
    // out are some 100 KB of code that runs once, bound by instruction fetch.
    constexpr int U = 4;
    static_assert(NB % U == 0, "whole passes");
#pragma unroll 1
    for (int jj0 = 0; jj0 < NB; jj0 += U) {
#pragma unroll
    for (int uu = 0; uu < U; ++uu) {
        const int jj = jj0 + uu;
        if (jj < nb) {
        const int j = k0 + jj;
        double best = -1.0;
        int bi = 0x7fffffff;
#pragma unroll
        for (int q = 0; q < kPanelRows; ++q) {
            const int i = k0 + t + kPanelThreads * q;
            const double m = v[q][uu].x * v[q][uu].x + v[q][uu].y * v[q][uu].y;
            if (i >= j && i < N && m > best) {
                best = m;
                bi = i;
            }
        }
        // every lane's own reciprocal fills the waits of the argmax; the
        // pivot's is published with its row
        double2 own[kPanelRows];
#pragma unroll
        for (int q = 0; q < kPanelRows; ++q) {
            const double2 d = v[q][uu];
            const double dn = d.x * d.x + d.y * d.y;
            own[q] = make_double2(d.x / dn, -d.y / dn);
        }
        better_pivot<0x111>(best, bi);   // row_shr 1, 2, 4, 8, then row_bcast 15, 31
        better_pivot<0x112>(best, bi);
        better_pivot<0x114>(best, bi);
        better_pivot<0x118>(best, bi);
        better_pivot<0x142>(best, bi);
        better_pivot<0x143>(best, bi);
        best = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(best), 63),
                                __builtin_amdgcn_readlane(__double2loint(best), 63));
        bi = __builtin_amdgcn_readlane(bi, 63);
        const int set = uu & 1, oj = (j - k0) % kPanelThreads, qj = (j - k0) / kPanelThreads;
        if (lane == 0) {
            redv[set][wave] = best;
            redi[set][wave] = bi;
        }
#pragma unroll
        for (int q = 0; q < kPanelRows; ++q) {
            if (k0 + t + kPanelThreads * q == bi) {
#pragma unroll
                for (int c = 0; c < NB; ++c) cand[set][wave][c] = v[q][c];
                recip[set][wave] = own[q];
            }
            if (t == oj && q == qj)
#pragma unroll
                for (int c = 0; c < NB; ++c) xrows[set][c] = v[q][c];
        }
        __syncthreads();
        // the best of the waves' candidates: lanes w % 8 compare them, which
        // wave it came from follows from its row
        static_assert(kWaves == 8, "three steps over eight candidates");
        double pmag = redv[set][lane & 7];
        int p = redi[set][lane & 7];
        better_pivot<0xb1>(pmag, p);     // quad_perm 1 0 3 2, 2 3 0 1, row_half_mirror
        better_pivot<0x4e>(pmag, p);
        better_pivot<0x141>(pmag, p);
        pmag = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(pmag)),
                                __builtin_amdgcn_readfirstlane(__double2loint(pmag)));
        p = __builtin_amdgcn_readfirstlane(p);
        const int pw = ((p - k0) % kPanelThreads) >> 6;
        const double2 *prow = cand[set][pw], *xrow = xrows[set];
        if (!(pmag > 0.0)) {
            // exact zero column: record, leave it (LAPACK continues the same way)
            if (t == 0) {
                piv[j] = j;
                if (atomicCAS(&a.flag[1], 0, (a.paths ? a.paths[pl] : (int)blockIdx.x) + 1) == 0) a.flag[2] = j;
            }
        } else {
        if (t == 0) piv[j] = p;
        const int op = (p - k0) % kPanelThreads, qp = (p - k0) / kPanelThreads;
        if (p != j) {
#pragma unroll
            for (int q = 0; q < kPanelRows; ++q) {
                if (t == oj && q == qj)
#pragma unroll
                    for (int c = 0; c < NB; ++c) v[q][c] = prow[c];
                if (t == op && q == qp)
#pragma unroll
                    for (int c = 0; c < NB; ++c) v[q][c] = xrow[c];
            }
        }
        const double2 inv = recip[set][pw];
#pragma unroll
        for (int q = 0; q < kPanelRows; ++q) {
            const int i = k0 + t + kPanelThreads * q;
            if (i > j && i < N) {
                const double2 l = cmul(v[q][uu], inv);
                v[q][uu] = l;
                // columns after jj: those of this pass, then groups of four
                // until the rotated-in finished ones
#pragma unroll
                for (int g = 0; g < NB; g += U)
                    if (g < NB - jj0)
#pragma unroll
                        for (int c = g; c < g + U; ++c)
                            if (c > uu) {
                                const double2 u = prow[c];
                                v[q][c].x -= l.x * u.x - l.y * u.y;
                                v[q][c].y -= l.x * u.y + l.y * u.x;
                            }
            }
        }
        }
        }
    }
#pragma unroll
        for (int q = 0; q < kPanelRows; ++q) {
            double2 first[U];
#pragma unroll
            for (int c = 0; c < U; ++c) first[c] = v[q][c];
#pragma unroll
            for (int c = 0; c < NB; ++c) v[q][c] = c + U < NB ? v[q][(c + U) % NB] : first[(c + U - NB) < 0 ? 0 : c + U - NB];
        }
    }
#pragma unroll
    for (int q = 0; q < kPanelRows; ++q) {
        const int i = k0 + t + kPanelThreads * q;
        if (i < N)
#pragma unroll
            for (int c = 0; c < NB; ++c)
                if (c < nb) A[i + (size_t)(k0 + c) * N] = v[q][c];
    }
}

// grid: x = column blocks of 256, y = matrix.
__global__ __launch_bounds__(256) void k_lu_swap_trsm(LUStepArgs a) {
    constexpr int NB = kLUPanel;
    __shared__ double2 L11[NB][NB];
    __shared__ int pv[NB];
    int pl, slot;
    job_of(a.jobs, blockIdx.y, pl, slot);
    const int N = a.N, k0 = a.k0, nb = a.nb;
    const size_t ms = (size_t)pl * kSlots2C + slot;
    if (skipped(a, ms)) return;
    double2* A = a.LU + ms * (size_t)N * N;
    const int* piv = a.piv + ms * N;
    const int t = threadIdx.x;
    for (int e = t; e < nb * nb; e += blockDim.x) {
        const int r = e % nb, c = e / nb;
        L11[r][c] = A[(k0 + r) + (size_t)(k0 + c) * N];
    }
    if (t < nb) pv[t] = piv[k0 + t];
    __syncthreads();
    if (blockIdx.x == 0 && t == 0) {
        int* perm = a.perm + ms * N;
        for (int jj = 0; jj < nb; ++jj) {
            const int p = pv[jj];
            if (p != k0 + jj) {
                const int x = perm[k0 + jj];
                perm[k0 + jj] = perm[p];
                perm[p] = x;
            }
        }
    }
    const int c = blockIdx.x * blockDim.x + t;
    if (c >= N || (c >= k0 && c < k0 + nb)) return;
    double2* col = A + (size_t)c * N;
    for (int jj = 0; jj < nb; ++jj) {
        const int p = pv[jj];
        if (p != k0 + jj) {
            const double2 x = col[k0 + jj];
            col[k0 + jj] = col[p];
            col[p] = x;
        }
    }
    if (c < k0 + nb) return;
    double2 x[NB];
#pragma unroll
    for (int jj = 0; jj < NB; ++jj) x[jj] = (jj < nb) ? col[k0 + jj] : make_double2(0.0, 0.0);
#pragma unroll
    for (int jj = 1; jj < NB; ++jj) {
        if (jj < nb) {
#pragma unroll
            for (int m = 0; m < jj; ++m) {
                const double2 l = L11[jj][m];
                x[jj].x -= l.x * x[m].x - l.y * x[m].y;
                x[jj].y -= l.x * x[m].y + l.y * x[m].x;
            }
        }
    }
#pragma unroll
    for (int jj = 0; jj < NB; ++jj)
        if (jj < nb) col[k0 + jj] = x[jj];
}

// grid: x = 64 x 64 tiles of the trailing matrix (T x T), y = matrix.
// Computed as the transposed product D'[jj][ii] = sum_k U12[k][jj] L21[ii][k],
// so that the 16 lanes of an output row address consecutive rows of the
// column-major matrix.
__global__ __launch_bounds__(256) void k_lu_update(LUStepArgs a) {
    constexpr int NB = kLUPanel;
    __shared__ double Ur[NB][64], Ui[NB][64], Lr[NB][64], Li[NB][64];
    int pl, slot;
    job_of(a.jobs, blockIdx.y, pl, slot);
    const int N = a.N, k0 = a.k0, nb = a.nb, k1 = k0 + nb;
    const int T = (N - k1 + 63) / 64;
    const int bi = blockIdx.x % T, bj = blockIdx.x / T;
    const int r0 = k1 + 64 * bi, c0 = k1 + 64 * bj;
    const size_t ms = (size_t)pl * kSlots2C + slot;
    if (skipped(a, ms)) return;
    double2* A = a.LU + ms * (size_t)N * N;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int jsub = (wave >> 1) * 32, isub = (wave & 1) * 32;
    const int li = lane & 15, lk = lane >> 4;
    dbl4 re[2][2], im[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            re[x][y] = dbl4{0.0, 0.0, 0.0, 0.0};
            im[x][y] = dbl4{0.0, 0.0, 0.0, 0.0};
        }
    // the k range k0 .. k0 + nb - 1 in chunks of NB (one chunk for a panel)
    for (int kc = 0; kc < nb; kc += NB) {
    if (kc) __syncthreads();
    for (int e = t; e < 64 * NB; e += blockDim.x) {
        const int ii = e % 64, k = e / 64;
        const int row = r0 + ii;
        const double2 x = (row < N && kc + k < nb) ? A[row + (size_t)(k0 + kc + k) * N] : make_double2(0.0, 0.0);
        Lr[k][ii] = x.x;
        Li[k][ii] = x.y;
    }
    for (int e = t; e < 64 * NB; e += blockDim.x) {
        const int k = e % NB, jj = e / NB;
        const int col = c0 + jj;
        const double2 x = (col < N && kc + k < nb) ? A[(k0 + kc + k) + (size_t)col * N] : make_double2(0.0, 0.0);
        Ur[k][jj] = x.x;
        Ui[k][jj] = x.y;
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < NB / 4; ++ks) {
        const int kr = ks * 4 + lk;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const double ur = Ur[kr][jsub + 16 * x + li], ui = Ui[kr][jsub + 16 * x + li];
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const double lr = Lr[kr][isub + 16 * y + li], lm = Li[kr][isub + 16 * y + li];
                re[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ur, lr, re[x][y], 0, 0, 0);
                re[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ui, lm, re[x][y], 0, 0, 0);
                im[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ur, lm, im[x][y], 0, 0, 0);
                im[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(ui, lr, im[x][y], 0, 0, 0);
            }
        }
    }
    }
    // D'[row][col] of a 16 x 16 tile: lane l, register r -> row 4 r + l / 16, col l % 16
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int col = c0 + jsub + 16 * x + 4 * r + lk;
                const int row = r0 + isub + 16 * y + li;
                if (row < N && col < N) {
                    double2* p = A + row + (size_t)col * N;
                    double2 val = *p;
                    val.x -= re[x][y][r];
                    val.y -= im[x][y][r];
                    *p = val;
                }
            }
}

// One workgroup per matrix: skip = (every |A[i][j]| <= 1 for rows i >= nt,
// columns j < nt, i.e. |K^dagger| <= 1); where set, the identity permutation
// and the diagonal pivots of the first nt columns are written here (the panel
// steps that would write them return at once).
__global__ __launch_bounds__(1024) void k_lu_check(LUStepArgs a) {
    __shared__ int bad;
    int pl, slot;
    job_of(a.jobs, blockIdx.x, pl, slot);
    const int N = a.N, nt = a.nt;
    const size_t ms = (size_t)pl * kSlots2C + slot;
    const double2* A = a.LU + ms * (size_t)N * N;
    const int t = threadIdx.x;
    if (t == 0) bad = 0;
    __syncthreads();
    // every element of the block independent of the others (all loads in
    // flight at once; consecutive threads read consecutive rows of a column)
    int b = 0;
    const int nr = N - nt;
    const long long n_el = (long long)nt * nr;
    for (long long e = t; e < n_el; e += blockDim.x) {
        const int j = (int)(e / nr), i = nt + (int)(e - (long long)j * nr);
        const double2 x = A[i + (size_t)j * N];
        b |= !(x.x * x.x + x.y * x.y <= 1.0);
    }
    if (b) atomicOr(&bad, 1);
    __syncthreads();
    const int ok = bad ? 0 : 1;
    if (t == 0) a.skip[ms] = ok;
    if (ok) {
        int* perm = a.perm + ms * N;
        int* piv = a.piv + ms * N;
        for (int i = t; i < N; i += blockDim.x) perm[i] = i;
        for (int j = t; j < nt; j += blockDim.x) piv[j] = j;
    }
}


// M = S^{-1} H = U^{-1} L^{-1} (P H) for every matrix of the launch from the
// factors above: the explicit form of Eq. INV, N right-hand sides.
//
// A workgroup of eight waves takes 16 columns of one matrix through both
// substitutions, right-looking by blocks of 32 rows: solve the diagonal block,
// then subtract its products from the rows still to come, 16 rows x 16 columns
// per wave at a time on v_mfma_f64_16x16x4.  The factor is the A operand as it
// lies in memory (16 consecutive rows of a column), read straight into
// registers a tile ahead; the 16 columns stay in LDS (ONCHIP, up to kRhsRows
// rows; beyond that in M), where one 16-byte read gives the real and imaginary
// B operand.  In the diagonal block a lane holds one element (32 rows x two
// columns per wave) and the solved row is broadcast by lane reads.  The four
// real products of a block are summed from zero, each by itself, and
// subtracted from Y once: with the products added to Y one after another Y is
// rounded twice per term (root mean square error of overlap-like systems of
// n = 442: 2.5e-15 that way, 1.8e-15 rounded once per term, 0.83e-15 this way).
//
// The chain of 2 N such rows bounds small batches, the products large ones.
// Column blocks of 32 staged in LDS and solved with vector FMAs, one launch
// -> this one: N = 442, 16 matrices: 1.86 -> 0.62 ms; N = 115, ten matrices:
// 223 -> 58 us.
constexpr int kRhsB = 32;          // rows of a block
constexpr int kRhsC = 16;          // columns of a workgroup
constexpr int kRhsThreads = 512;
constexpr int kRhsRows = 544;      // 16 columns of as many rows fit the LDS beside the diagonal block

__device__ inline double lane_read(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

template <bool ONCHIP>
__global__ __launch_bounds__(kRhsThreads) void k_lu_rhs(RhsArgs a, int n_jobs) {
    extern __shared__ double2 rhs_lds[];
    double2* ft = rhs_lds;                    // [k][row] diagonal block of the factors
    double2* Y = rhs_lds + kRhsB * kRhsB;     // ONCHIP: [row][column]
    const int N = a.N, t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // the column blocks of a matrix on one XCD, whose L2 then holds its factors
    const int n_cb = (N + kRhsC - 1) / kRhsC, total = n_cb * n_jobs, per = (total + 7) / 8;
    const int W = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (W >= total) return;
    const int job = W / n_cb;
    int pl, slot;
    job_of(a.jobs, job, pl, slot);
    const size_t ms = (size_t)pl * kSlots2C + slot, NN = (size_t)N * N;
    const double2* LU = a.LU + ms * NN;
    const double2* H = a.H + ms * NN;
    const int* perm = a.perm + ms * N;
    double2* M = a.M + ms * NN;
    const int c0 = (W - job * n_cb) * kRhsC, nc = min(kRhsC, N - c0), nb = (N + kRhsB - 1) / kRhsB;
    auto get = [&](int row, int col) {
        if (ONCHIP) return Y[row * kRhsC + col];
        return row < N && col < nc ? M[(size_t)row * N + c0 + col] : make_double2(0.0, 0.0);
    };
    auto put = [&](int row, int col, double2 v) {
        if (ONCHIP) Y[row * kRhsC + col] = v;
        else if (row < N && col < nc) M[(size_t)row * N + c0 + col] = v;
    };
    for (int e = t; e < nb * kRhsB * kRhsC; e += kRhsThreads) {
        const int row = e / kRhsC, col = e % kRhsC;
        put(row, col, row < N && col < nc ? H[(size_t)perm[row] * N + c0 + col] : make_double2(0.0, 0.0));
    }
    const int li = lane & 15, lk = lane >> 4;
    // rows [row0, row0 + 16) x columns [kb0, kb0 + 32) of the factors as A operands
    auto load_tile = [&](int row0, int kb0, double2 (&f)[8]) {
        const int row = row0 + li;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int col = kb0 + 4 * s + lk;
            f[s] = LU[min(row, N - 1) + (size_t)min(col, N - 1) * N];
            if (row >= N || col >= N) f[s] = make_double2(0.0, 0.0);
        }
    };
    // Y[rows of tiles] -= factors x Y[block kb0], the tiles q = q0, q0 + 8, .. < q1 of 16 rows
    auto update = [&](int q0, int q1, int kb0) {
        int q = q0 + wave;
        if (q >= q1) return;
        double2 y[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) y[s] = get(kb0 + 4 * s + lk, li);
        double2 f[8];
        load_tile(16 * q, kb0, f);
        for (; q < q1; q += kRhsThreads / 64) {
            double2 fn[8];
            load_tile(16 * min(q + kRhsThreads / 64, q1 - 1), kb0, fn);
            double2 v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = get(16 * q + 4 * r + lk, li);
            const dbl4 zero = {0.0, 0.0, 0.0, 0.0};
            dbl4 xx = zero, xy = zero, yy = zero, yx = zero;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                xx = __builtin_amdgcn_mfma_f64_16x16x4f64(f[s].x, y[s].x, xx, 0, 0, 0);
                xy = __builtin_amdgcn_mfma_f64_16x16x4f64(f[s].x, y[s].y, xy, 0, 0, 0);
                yy = __builtin_amdgcn_mfma_f64_16x16x4f64(f[s].y, y[s].y, yy, 0, 0, 0);
                yx = __builtin_amdgcn_mfma_f64_16x16x4f64(f[s].y, y[s].x, yx, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                put(16 * q + 4 * r + lk, li, make_double2(v[r].x - (xx[r] - yy[r]), v[r].y - (xy[r] + yx[r])));
#pragma unroll
            for (int s = 0; s < 8; ++s) f[s] = fn[s];
        }
    };
    // the diagonal block's factors: two elements per thread
    double2 dg[2];
    auto load_diag = [&](int rb0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = t + i * kRhsThreads, row = rb0 + e % kRhsB, col = rb0 + e / kRhsB;
            dg[i] = row < N && col < N ? LU[row + (size_t)col * N] : make_double2(0.0, 0.0);
        }
    };
    auto store_diag = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i) ft[t + i * kRhsThreads] = dg[i];
    };
    // this lane's element of a diagonal block
    const int r = lane & 31, col = 2 * wave + (lane >> 5);
    auto solved_row = [&](double2 v, int k) {
        const double ax = lane_read(v.x, k), ay = lane_read(v.y, k), bx = lane_read(v.x, k + 32), by = lane_read(v.y, k + 32);
        return lane < 32 ? make_double2(ax, ay) : make_double2(bx, by);
    };
    load_diag(0);
    __syncthreads();
    // forward: L (unit diagonal) Y = P H
    for (int rb = 0; rb < nb; ++rb) {
        const int rb0 = rb * kRhsB;
        store_diag();
        __syncthreads();
        if (rb + 1 < nb) load_diag(rb0 + kRhsB);
        double2 v = get(rb0 + r, col);
#pragma unroll 4
        for (int k = 0; k + 1 < kRhsB; ++k) {
            const double2 f = ft[k * kRhsB + r], y = solved_row(v, k);
            if (r > k) {
                v.x -= f.x * y.x - f.y * y.y;
                v.y -= f.x * y.y + f.y * y.x;
            }
        }
        put(rb0 + r, col, v);
        __syncthreads();
        update(2 * (rb + 1), 2 * nb, rb0);
        __syncthreads();
    }
    // backward: U M = Y
    load_diag((nb - 1) * kRhsB);
    for (int rb = nb - 1; rb >= 0; --rb) {
        const int rb0 = rb * kRhsB;
        store_diag();
        __syncthreads();
        if (rb > 0) load_diag(rb0 - kRhsB);
        double2 v = get(rb0 + r, col);
        const double2 d = ft[r * kRhsB + r];
        const double rdn = rb0 + r < N ? 1.0 / (d.x * d.x + d.y * d.y) : 0.0;
        const double2 id = make_double2(d.x * rdn, -d.y * rdn);   // 1 / d
#pragma unroll 4
        for (int k = min(kRhsB, N - rb0) - 1; k >= 0; --k) {
            const double2 f = ft[k * kRhsB + r];
            if (r == k) v = cmul(v, id);
            const double2 y = solved_row(v, k);
            if (r < k) {
                v.x -= f.x * y.x - f.y * y.y;
                v.y -= f.x * y.y + f.y * y.x;
            }
        }
        put(rb0 + r, col, v);
        __syncthreads();
        update(0, 2 * rb, rb0);
        __syncthreads();
    }
    if (ONCHIP)
        for (int e = t; e < N * kRhsC; e += kRhsThreads) {
            const int row = e / kRhsC, c = e % kRhsC;
            if (c < nc) M[(size_t)row * N + c0 + c] = Y[e];
        }
}

}  // namespace

hipError_t launch_lu_check(const LUStepArgs& a, int n_jobs, hipStream_t st, const LaunchEv& ev) {
    WPCCC_LAUNCH(ev, k_lu_check, dim3(n_jobs), dim3(1024), 0, st, a);
    return hipGetLastError();
}

int lu_panel_width(int N) { return N <= 2 * kPanelThreads ? kLUPanel : kLUPanel / 2; }

hipError_t launch_lu_panel(const LUStepArgs& a, int n_jobs, hipStream_t st, const LaunchEv& ev) {
    if (a.N > kLUMaxN || a.nb > lu_panel_width(a.N)) return hipErrorInvalidValue;
    // rows per thread from the rows left below k0 (the pivot is the same
    // whatever the split: largest |a|^2, lowest row on ties)
    const int rows = (a.N - a.k0 + kPanelThreads - 1) / kPanelThreads;
    if (lu_panel_width(a.N) == kLUPanel) {
        if (rows <= 1)
            WPCCC_LAUNCH(ev, (k_lu_panel<1, kLUPanel>), dim3(n_jobs), dim3(kPanelThreads), 0, st, a);
        else
            WPCCC_LAUNCH(ev, (k_lu_panel<2, kLUPanel>), dim3(n_jobs), dim3(kPanelThreads), 0, st, a);
    } else if (rows <= 1) {
        WPCCC_LAUNCH(ev, (k_lu_panel<1, kLUPanel / 2>), dim3(n_jobs), dim3(kPanelThreads), 0, st, a);
    } else if (rows <= 2) {
        WPCCC_LAUNCH(ev, (k_lu_panel<2, kLUPanel / 2>), dim3(n_jobs), dim3(kPanelThreads), 0, st, a);
    } else {
        WPCCC_LAUNCH(ev, (k_lu_panel<4, kLUPanel / 2>), dim3(n_jobs), dim3(kPanelThreads), 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_lu_swap_trsm(const LUStepArgs& a, int n_jobs, hipStream_t st, const LaunchEv& ev) {
    WPCCC_LAUNCH(ev, k_lu_swap_trsm, dim3((a.N + 255) / 256, n_jobs), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_lu_update(const LUStepArgs& a, int n_jobs, hipStream_t st, const LaunchEv& ev) {
    const int T = (a.N - a.k0 - a.nb + 63) / 64;
    if (T <= 0) return hipSuccess;
    WPCCC_LAUNCH(ev, k_lu_update, dim3(T * T, n_jobs), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_lu_rhs(const RhsArgs& a, int n_jobs, hipStream_t st, const LaunchEv& ev) {
    const int n = (a.N + kRhsC - 1) / kRhsC * n_jobs;
    const dim3 grid(8 * ((n + 7) / 8)), block(kRhsThreads);
    constexpr int diag = kRhsB * kRhsB * (int)sizeof(double2), most = diag + kRhsRows * kRhsC * (int)sizeof(double2);
    const int rows = (a.N + kRhsB - 1) / kRhsB * kRhsB;
    if (rows <= kRhsRows) {
        const int smem = diag + rows * kRhsC * (int)sizeof(double2);
        static SmemLimit limit(64 * 1024);
        const hipError_t e = limit.raise(most, [] {
            return hipFuncSetAttribute((const void*)k_lu_rhs<true>, hipFuncAttributeMaxDynamicSharedMemorySize, most);
        });
        if (e != hipSuccess) return e;
        WPCCC_LAUNCH(ev, k_lu_rhs<true>, grid, block, smem, st, a, n_jobs);
    } else {
        WPCCC_LAUNCH(ev, k_lu_rhs<false>, grid, block, diag, st, a, n_jobs);
    }
    return hipGetLastError();
}

}  // namespace wpccc
