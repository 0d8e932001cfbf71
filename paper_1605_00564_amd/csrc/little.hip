// The little Dirac operator A (N_s x N_s blocks coupling a deflation block with
// itself and its eight neighbours) and the little solve A^{-1} by GCR on the
// block even-odd Schur complement, in FP64.
//
// Blocks are coloured by the parity of their coordinates on the deflation-block
// grid (an even number of blocks along every axis), so every coupling joins
// blocks of opposite colour and A_EE, A_OO are block diagonal.  With
//   M1 = A_OO^{-1} A_OE A_EE^{-1}   (formed when A is built),
//   g_O = A_OO^{-1} u_O,   u' = u_E - A_EO g_O,
// the Schur system preconditioned from the right by A_EE^{-1} is
//   (1 - A_EO M1) y = u',   x_E = A_EE^{-1} y,   x_O = g_O - M1 y:
// two products of eight couplings an iteration.  The search direction z_k =
// A_EE^{-1} r_k is never formed; the residuals r_k are kept instead, and y is
// their combination.
//
// Vectors of the iteration hold the even blocks only, [rhs][rank][N_s] (rank of a
// block among its colour).  On small systems the solve is a chain of short
// launches, so an iteration is five of them (two products, dot products,
// subtraction, update; each sums up the partial sums of the one before by
// itself), and the host looks at the norms only every few iterations: y is formed
// from the steps up to the first that converged, so steps beyond it do no harm.
#include <algorithm>
#include <cmath>

#include "blas.h"
#include "dflint.h"
#include "little_rules.h"

namespace dfl {

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

// out[r][orow(i)] = base[r][brow(i)] + sgn sum_{d < nd} M[mrow(i)][d0 + d] v[r][slot[i][d]]
// for rows i < nrows; null tables are the identity, a null base is zero.  Each
// vector has its own number of slots per right-hand side.
struct Rows {
    const double2 *M;
    const int *mrow;
    int ND, d0, nd;
    const double2 *v;
    const int *slot;
    int nv;
    const double2 *base;
    const int *brow;
    int nb;
    double2 *out;
    const int *orow;
    int no;
    double sgn;
};

// A complex GEMM (N_s x nd N_s) (nd N_s x n) per row on the FP64 matrix cores, in
// tiles of 16 of a row's N_s by some right-hand sides.  With M = a + ib, v = c + id,
// Re = ac - bd and Im = ad + bc as real 16x16x4 products.  Wide tile: 16 right-hand
// sides, four products; narrow tile: 8, whose real and imaginary parts are
// neighbouring columns, two products.  Lane L supplies M[row L % 16][k L / 16] and
// v[k L / 16][column L % 16] and receives out[row L / 16 + 4 i][column L % 16].
// RW = 4: few tiles, bound by the latency of their loads (slot, then vector).  The
// waves of a workgroup share a tile, each taking every fourth group of four columns
// (of all nd couplings in one list) with the loads of four steps before their
// products, and are added through LDS in order.
// RW = 1: tiles enough to fill the device, bound by the matrix cores and the L2.  A
// workgroup takes four tiles (one wave per workgroup left the launch of workgroups
// as the bound), a wave walks coupling by coupling, the loads of three steps before
// their products.
// All nine couplings, us, one wave per row and one step's loads at a time / now:
//   16^3 x 32, 4^4, N_s = 12: n = 1 10.6 / 9.0, n = 24 11.6 / 9.7
//   24^3 x 48, 4^4, N_s = 12: n = 1 22.7 / 13.9, n = 12 24.7 / 19.9, n = 25 34.1 / 33.9, n = 40 57.0 / 45.4
//   24^3 x 48, 4^4, N_s = 20: n = 1 49.7 / 32.9, n = 12 51.2 / 49.3, n = 25 87.6 / 84.4, n = 40 133 / 121
//   24^3 x 48, 6^4, N_s = 20: n = 1 22.8 / 10.3, n = 24 29.9 / 23.3
constexpr int RU = 4, RU1 = 3;   // steps in flight
template <int RW, bool WIDE>
__global__ void __launch_bounds__(64 * ROW_WAVES) k_little_rows(Rows a, int nrows, int Ns, int n, int nmt, int ng) {
    constexpr int TR = WIDE ? 16 : 8;   // right-hand sides of a tile
    __shared__ double red[ROW_WAVES][WIDE ? 2 : 1][16][17];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = wv % RW;
    const RowTile t = row_tile(blockIdx.x, wv / RW, ROW_WAVES / RW, nmt, ng);
    const bool live = t.row < nrows;
    const int i = live ? t.row : nrows - 1, m0 = t.m * 16, r0 = t.r * TR;
    const int row = lane & 15, kk = lane >> 4;
    const bool mv = m0 + row < Ns, im = row & 1;
    const size_t NN = (size_t)Ns * Ns;
    const double2 *M = a.M + ((size_t)(a.mrow ? a.mrow[i] : i) * a.ND + a.d0) * NN + (size_t)(mv ? m0 + row : 0) * Ns;
    const double2 *v = a.v + (size_t)min(r0 + (WIDE ? row : row / 2), n - 1) * a.nv * Ns;   // from n on: not used
    const int *slot = a.slot ? a.slot + (size_t)i * a.nd : nullptr;
    d4v x = {0, 0, 0, 0}, y = {0, 0, 0, 0}, z = {0, 0, 0, 0}, w = {0, 0, 0, 0};
    auto products = [&](const double2 &m, const double2 &b) {
        x = __builtin_amdgcn_mfma_f64_16x16x4f64(m.x, !WIDE && im ? b.y : b.x, x, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(m.y, !WIDE && im ? b.x : -b.y, y, 0, 0, 0);
        if constexpr (WIDE) {
            z = __builtin_amdgcn_mfma_f64_16x16x4f64(m.x, b.y, z, 0, 0, 0);
            w = __builtin_amdgcn_mfma_f64_16x16x4f64(m.y, b.x, w, 0, 0, 0);
        }
    };
    if constexpr (RW == 1) {
        for (int d = 0; d < a.nd; ++d) {
            const double2 *Md = M + d * NN, *vd = v + (size_t)(slot ? slot[d] : i) * Ns;
            for (int l0 = 0; l0 < Ns; l0 += 4 * RU1) {
                double2 ma[RU1], vb[RU1];
#pragma unroll
                for (int u = 0; u < RU1; ++u) {
                    const int l = l0 + 4 * u + kk;
                    ma[u] = vb[u] = make_double2(0.0, 0.0);
                    if (l < Ns) {
                        if (mv) ma[u] = Md[l];
                        vb[u] = vd[l];
                    }
                }
#pragma unroll
                for (int u = 0; u < RU1; ++u)
                    if (l0 + 4 * u < Ns) products(ma[u], vb[u]);
            }
        }
    } else {
        const int nl = (Ns + 3) / 4, steps = a.nd * nl;
        for (int s0 = wave; s0 < steps; s0 += RW * RU) {
            double2 ma[RU], vb[RU];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                const int st = s0 + u * RW;
                ma[u] = vb[u] = make_double2(0.0, 0.0);
                if (st < steps) {
                    const int d = st / nl, l = (st - d * nl) * 4 + kk;
                    if (l < Ns) {
                        if (mv) ma[u] = M[d * NN + l];
                        vb[u] = v[(size_t)(slot ? slot[d] : i) * Ns + l];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) products(ma[u], vb[u]);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        red[wv][0][kk + 4 * q][row] = x[q] + y[q];
        if constexpr (WIDE) red[wv][1][kk + 4 * q][row] = z[q] + w[q];
    }
    __syncthreads();
    for (int e = wave * 64 + lane; e < 16 * TR; e += 64 * RW) {
        const int mo = e & 15, ro = e >> 4;   // consecutive threads along N_s
        if (!live || m0 + mo >= Ns || r0 + ro >= n) continue;
        double2 o = make_double2(0, 0);
#pragma unroll
        for (int p = 0; p < RW; ++p) {
            const auto &part = red[wv - wave + p];
            o.x += part[0][mo][WIDE ? ro : 2 * ro];
            o.y += WIDE ? part[WIDE][mo][ro] : part[0][mo][2 * ro + 1];
        }
        o.x *= a.sgn;
        o.y *= a.sgn;
        if (a.base) {
            const double2 b = a.base[((size_t)(r0 + ro) * a.nb + (a.brow ? a.brow[i] : i)) * Ns + m0 + mo];
            o.x += b.x;
            o.y += b.y;
        }
        a.out[((size_t)(r0 + ro) * a.no + (a.orow ? a.orow[i] : i)) * Ns + m0 + mo] = o;
    }
}

int rows_launch(const Rows &a, int nrows, int Ns, int n, hipStream_t s) {
    const RowTiles t = row_tiles(nrows, Ns, n);
    // nd N_s complex multiply-adds per row entry and right-hand side; M read once
    // per group of right-hand sides
    ProfScope ps(PROF_LITTLE, s, 8.0 * a.nd * Ns * Ns * nrows * n,
                 16.0 * Ns * nrows * ((double)a.nd * Ns * t.ng + 2.0 * n), (double)Ns * nrows * n);
    const unsigned grid = row_workgroups(nrows, ROW_WAVES / t.waves, t.nmt, t.ng);
#define DFL_ROWS(RW, WIDE) k_little_rows<RW, WIDE><<<grid, 64 * ROW_WAVES, 0, s>>>(a, nrows, Ns, n, t.nmt, t.ng)
    if (t.waves == 1) {
        if (t.wide)
            DFL_ROWS(1, true);
        else
            DFL_ROWS(1, false);
    } else {
        if (t.wide)
            DFL_ROWS(ROW_WAVES, true);
        else
            DFL_ROWS(ROW_WAVES, false);
    }
#undef DFL_ROWS
    DFL_HIP(hipGetLastError());
    return 0;
}

// C[i][d] = X[xrow(i)] Y with one N_s x N_s product per coupling: LEFT = false:
// C = A[mrow(i)][1 + d] Dinv[erow[slot[i][d]]], LEFT = true: C = Dinv[mrow(i)] T[i][d]
template <bool LEFT>
__global__ void k_fold(const double2 *__restrict__ A, const double2 *__restrict__ D, const int *__restrict__ mrow,
                       const int *__restrict__ slot, const int *__restrict__ erow, double2 *__restrict__ C, int nh,
                       int Ns) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t NN = (size_t)Ns * Ns;
    if (t >= (long)nh * 8 * NN) return;
    const int q = (int)(t % Ns), p = (int)((t / Ns) % Ns), d = (int)((t / NN) % 8), i = (int)(t / (8 * NN));
    const double2 *X = LEFT ? D + (size_t)mrow[i] * NN : A + ((size_t)mrow[i] * 9 + 1 + d) * NN;
    const double2 *Y = LEFT ? A + ((size_t)i * 8 + d) * NN : D + (size_t)erow[slot[i * 8 + d]] * NN;
    double re = 0, im = 0;
    for (int l = 0; l < Ns; ++l) {
        const double2 x = X[(size_t)p * Ns + l], y = Y[(size_t)l * Ns + q];
        re = ffma(x.x, y.x, ffma(-x.y, y.y, re));
        im = ffma(x.x, y.y, ffma(x.y, y.x, im));
    }
    C[t] = make_double2(re, im);
}

// ---------------------------------------------------------------------------
// One GCR step after the products: with w = W_k (set by the product) and r = r_k,
//   beta_j = (W_j, w), w -= sum beta_j W_j, w /= |w|, c = (w, r), r_{k+1} = r - c w
// (classical Gram-Schmidt, sums in FP64), in three launches of G workgroups per
// right-hand side, each on its stretch of the vector.  A launch leaves G partial
// sums per value; every workgroup of the next adds them up by itself, in one
// fixed order.  All three are bound by latency (3 to 8 us each at the sizes where
// the solve is slow).  Before: ten launches and a wait of the host per iteration
// and 77 us; a solve to 1e-10 (14 iterations, 16^3 x 32, N_s = 12) 1130 -> 500 us
// for one right-hand side, 1240 -> 540 for twelve.  One workgroup per right-hand
// side for the whole step needs 27 us (its registers spill).
// ---------------------------------------------------------------------------
constexpr int LB = 256, LWV = LB / 64;   // threads and waves of a workgroup
constexpr int GMAX = 64;                 // partial sums per value, at most

__device__ inline double lane_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// NV sums over the workgroup into part[v * GMAX] (v < nv)
template <int NV>
__device__ inline void leave(double (&v)[NV], double (*sh)[LWV], double *part, int nv) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if constexpr (NV == 16) {
        // halving exchange: 15 + 2 exchanges instead of 6 for each of 16 values;
        // lane l ends with value l / 4 of the wave
#pragma unroll
        for (int h = 8, o = 32; h > 0; h >>= 1, o >>= 1) {
            const bool up = lane & o;
#pragma unroll
            for (int i = 0; i < h; ++i) {
                const double keep = up ? v[i + h] : v[i], send = up ? v[i] : v[i + h];
                v[i] = keep + __shfl_xor(send, o, 64);
            }
        }
        v[0] += __shfl_xor(v[0], 2, 64);
        v[0] += __shfl_xor(v[0], 1, 64);
        if ((lane & 3) == 0) sh[lane >> 2][w] = v[0];
    } else {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const double t = lane_sum(v[q]);
            if (lane == 0) sh[q][w] = t;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nv)
        part[threadIdx.x * GMAX] = (sh[threadIdx.x][0] + sh[threadIdx.x][1]) + (sh[threadIdx.x][2] + sh[threadIdx.x][3]);
    __syncthreads();
}

// workgroup (g, r): elements [g len, (g + 1) len) of right-hand side r
struct Stretch {
    int lo, hi;
};
__device__ inline Stretch stretch(int ne) {
    const int len = (ne + (int)gridDim.x - 1) / (int)gridDim.x;
    const int lo = min((int)blockIdx.x * len, ne);
    return {lo, min(lo + len, ne)};
}

// partial (W_j, w), eight j < k per workgroup: dots[r][2 j + (0 re, 1 im)][g]
__global__ void __launch_bounds__(LB) k_little_dots(const double2 *__restrict__ W, int ne, int n, int k,
                                                    double *__restrict__ dots) {
    __shared__ double sh[16][LWV];
    const int r = blockIdx.y;
    const size_t vec = (size_t)n * ne;
    const double2 *w0 = W + (size_t)r * ne, *wk = w0 + k * vec;
    const Stretch t = stretch(ne);
    const int j0 = blockIdx.z * 8;
    double acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0;
    for (int i = t.lo + threadIdx.x; i < t.hi; i += LB) {
        const double2 b = wk[i];
        double2 a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = w0[min(j0 + j, k) * vec + i];   // from k on: not used
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            acc[2 * j] += a[j].x * b.x + a[j].y * b.y;
            acc[2 * j + 1] += a[j].x * b.y - a[j].y * b.x;
        }
    }
    leave<16>(acc, sh, dots + ((size_t)r * 2 * NKV_MAX + 2 * j0) * GMAX + blockIdx.x, 2 * min(8, k - j0));
}

// w -= sum beta_j W_j; partial |w|^2, (w, r) in three[r][3][g]; column k of R
__global__ void __launch_bounds__(LB) k_little_sub(double2 *__restrict__ W, const double2 *__restrict__ Rv, int ne,
                                                   int n, int k, const double *__restrict__ dots,
                                                   double *__restrict__ Rm, double *__restrict__ three) {
    __shared__ double sh[3][LWV];
    __shared__ double beta[2 * NKV_MAX];
    const int r = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, G = gridDim.x;
    const size_t vec = (size_t)n * ne;
    for (int v = wave; v < 2 * k; v += LWV) {
        const double b = lane_sum(lane < G ? dots[((size_t)r * 2 * NKV_MAX + v) * GMAX + lane] : 0.0);
        if (lane == 0) {
            beta[v] = b;
            if (blockIdx.x == 0) Rm[(((size_t)r * NKV_MAX + v / 2) * NKV_MAX + k) * 2 + v % 2] = b;
        }
    }
    __syncthreads();
    double2 *w0 = W + (size_t)r * ne, *wk = w0 + k * vec;
    const double2 *rk = Rv + k * vec + (size_t)r * ne;
    const Stretch t = stretch(ne);
    double acc[3] = {0, 0, 0};
    for (int i = t.lo + threadIdx.x; i < t.hi; i += LB) {
        double2 a = wk[i];
        const double2 b = rk[i];
        for (int j0 = 0; j0 < k; j0 += 8) {
            double2 c[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) c[j] = w0[min(j0 + j, k - 1) * vec + i];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j0 + j < k) {
                    const double tr = beta[2 * (j0 + j)], ti = beta[2 * (j0 + j) + 1];
                    a.x -= tr * c[j].x - ti * c[j].y;
                    a.y -= tr * c[j].y + ti * c[j].x;
                }
        }
        wk[i] = a;
        acc[0] += a.x * a.x + a.y * a.y;
        acc[1] += a.x * b.x + a.y * b.y;
        acc[2] += a.x * b.y - a.y * b.x;
    }
    leave<3>(acc, sh, three + (size_t)r * 3 * GMAX + blockIdx.x, 3);
}

// w /= |w|, c = (w, r), r_{k+1} = r - c w; partial |r_{k+1}|^2 in one[r][g]
__global__ void __launch_bounds__(LB) k_little_update(double2 *__restrict__ W, double2 *__restrict__ Rv, int ne, int n,
                                                      int k, const double *__restrict__ three, double *__restrict__ Rm,
                                                      double *__restrict__ cvec, double *__restrict__ one) {
    __shared__ double sh[1][LWV];
    __shared__ double s3[3];
    const int r = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, G = gridDim.x;
    const size_t vec = (size_t)n * ne;
    if (wave < 3) {
        const double b = lane_sum(lane < G ? three[((size_t)r * 3 + wave) * GMAX + lane] : 0.0);
        if (lane == 0) s3[wave] = b;
    }
    __syncthreads();
    const double g = sqrt(s3[0]);
    const bool fine = g > 0 && isfinite(g);
    const double ig = fine ? 1.0 / g : 0.0, cr = fine ? s3[1] * ig : 0.0, ci = fine ? s3[2] * ig : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        double *o = Rm + (((size_t)r * NKV_MAX + k) * NKV_MAX + k) * 2;
        o[0] = fine ? g : 1.0;
        o[1] = 0;
        cvec[((size_t)r * NKV_MAX + k) * 2] = cr;
        cvec[((size_t)r * NKV_MAX + k) * 2 + 1] = ci;
    }
    double2 *wk = W + k * vec + (size_t)r * ne;
    const double2 *rk = Rv + k * vec + (size_t)r * ne;
    double2 *rn = Rv + (k + 1) * vec + (size_t)r * ne;
    const Stretch t = stretch(ne);
    double acc[1] = {0};
    for (int i = t.lo + threadIdx.x; i < t.hi; i += LB) {
        double2 a = wk[i], b = rk[i];
        a.x *= ig;
        a.y *= ig;
        b.x -= cr * a.x - ci * a.y;
        b.y -= cr * a.y + ci * a.x;
        wk[i] = a;
        rn[i] = b;
        acc[0] += b.x * b.x + b.y * b.y;
    }
    leave<1>(acc, sh, one + (size_t)r * GMAX + blockIdx.x, 1);
}

// y (+)= sum_j alpha_j r_j over k steps, R alpha = c: every workgroup's first wave
// solves the triangular system by itself, lane i holding row i
__global__ void __launch_bounds__(LB) k_little_accum(double2 *__restrict__ y, const double2 *__restrict__ Rv, int ne,
                                                     int n, int k, const double *__restrict__ Rm,
                                                     const double *__restrict__ cvec, int first) {
    __shared__ double2 Rs[NKV_MAX * NKV_MAX];
    __shared__ double2 al[NKV_MAX];
    const int r = blockIdx.y;
    for (int e = threadIdx.x; e < k * k; e += LB)
        Rs[e] = reinterpret_cast<const double2 *>(Rm)[((size_t)r * NKV_MAX + e / k) * NKV_MAX + e % k];
    __syncthreads();
    if (threadIdx.x < 64) {
        const int i = threadIdx.x;
        double2 c = make_double2(0, 0);
        double d = 1;
        if (i < k) {
            c = reinterpret_cast<const double2 *>(cvec)[(size_t)r * NKV_MAX + i];
            d = 1.0 / Rs[i * k + i].x;   // real and positive
        }
        for (int j = k - 1; j >= 0; --j) {
            const double ar = __shfl(c.x * d, j, 64), ai = __shfl(c.y * d, j, 64);
            if (i == j) al[j] = make_double2(ar, ai);
            if (i < j) {
                const double2 q = Rs[i * k + j];
                c.x -= q.x * ar - q.y * ai;
                c.y -= q.x * ai + q.y * ar;
            }
        }
    }
    __syncthreads();
    const int i = blockIdx.x * LB + threadIdx.x;
    if (i >= ne) return;
    const size_t vec = (size_t)n * ne;
    const double2 *z = Rv + (size_t)r * ne + i;
    double2 a = first ? make_double2(0, 0) : y[(size_t)r * ne + i];
#pragma unroll 4
    for (int j = 0; j < k; ++j) {
        const double2 v = z[j * vec], t = al[j];
        a.x += t.x * v.x - t.y * v.y;
        a.y += t.x * v.y + t.y * v.x;
    }
    y[(size_t)r * ne + i] = a;
}

// out[v] = sum of part[v][0 .. G) (one wave per value)
__global__ void __launch_bounds__(LB) k_little_norms(const double *__restrict__ part, int G, int nv,
                                                     double *__restrict__ out) {
    const int v = blockIdx.x * LWV + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (v >= nv) return;
    const double t = lane_sum(lane < G ? part[(size_t)v * GMAX + lane] : 0.0);
    if (lane == 0) out[v] = t;
}
int little_norms(const double *part, int G, int nv, double *out, hipStream_t s) {
    k_little_norms<<<(nv + LWV - 1) / LWV, LB, 0, s>>>(part, G, nv, out);
    DFL_HIP(hipGetLastError());
    return 0;
}

__global__ void k_little_minus(const double2 *__restrict__ a, const double2 *__restrict__ b, double2 *__restrict__ c,
                               long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) c[i] = make_double2(a[i].x - b[i].x, a[i].y - b[i].y);
}

}  // namespace

int little_apply_dev(qcd_dfl d, const double2 *v, double2 *w, int n, hipStream_t s) {
    Rows a{d->A, nullptr, 9, 0, 9, v, d->bnbr, d->Nb, nullptr, nullptr, 0, w, nullptr, d->Nb, 1.0};
    return rows_launch(a, d->Nb, d->Ns, n, s);
}

// M1 from A and the inverse diagonal blocks; work: as large as M1
int little_fold(qcd_dfl d, double2 *work, hipStream_t s) {
    const int nh = d->Nb / 2;
    const int *erow = d->brow, *orow = d->brow + nh, *slot = d->brank + (size_t)nh * 8;
    const long t = (long)nh * 8 * d->Ns * d->Ns;
    k_fold<false><<<nblocks(t, 256), 256, 0, s>>>(d->A, d->Dinv, orow, slot, erow, work, nh, d->Ns);
    k_fold<true><<<nblocks(t, 256), 256, 0, s>>>(work, d->Dinv, orow, slot, erow, d->M1, nh, d->Ns);
    DFL_HIP(hipGetLastError());
    return 0;
}

// x = A^{-1} u (FP64).  The residual of the full system equals that of the Schur
// system (x_O is exact given x_E); it is reported relative to ||u||.  poll: stop
// when every right-hand side is at tol (at most maxit iterations, restarted
// every 24); otherwise run one cycle of min(maxit, 24) iterations without host
// synchronisation.  No iterations (maxit <= 0): x_O = A_OO^{-1} u_O, x_E = 0.
int little_solve(qcd_dfl d, const double2 *u, double2 *x, int n, double tol, int maxit, bool poll, int *iters_out,
                 double *relres_out, hipStream_t s) {
    // polled norms pass through the handle's pinned buffer of 4096 doubles
    if (n > 4096) return set_error(QCD_EINVAL, "too many right-hand sides in one little solve (max 4096)");
    const int Ns = d->Ns, Nb = d->Nb, nh = Nb / 2, ne = nh * Ns;
    const int nkv = std::max(1, std::min(maxit, 24)), look = n <= 4096 / LOOK ? LOOK : 1;
    const size_t vec = (size_t)ne * n;
    // doubles per right-hand side: partial dots, three, one (per step of a look),
    // norms (per step of a look), R, c
    const size_t per = (2 * NKV_MAX + 3 + LOOK) * GMAX + LOOK + 2 * (NKV_MAX * NKV_MAX + NKV_MAX);
    const size_t need = sizeof(double2) * vec * (2 * (size_t)nkv + 5) +
                        std::max(sizeof(double) * per * n, poll ? scalar_bytes(n) : 0);
    void *p;
    DFL_TRY(dfl_work(d, need, &p));
    double2 *W = static_cast<double2 *>(p);
    double2 *Rv = W + (size_t)nkv * vec;          // residuals r_0 .. r_nkv
    double2 *y = Rv + (size_t)(nkv + 1) * vec, *g = y + vec, *q = g + vec, *us = q + vec;
    double *dots = reinterpret_cast<double *>(us + vec), *three = dots + (size_t)n * 2 * NKV_MAX * GMAX;
    double *one = three + (size_t)n * 3 * GMAX, *norms = one + (size_t)LOOK * n * GMAX;
    double *Rm = norms + (size_t)LOOK * n, *cvec = Rm + (size_t)n * NKV_MAX * NKV_MAX * 2;
    // workgroups per right-hand side: a thread takes one element as long as the
    // partial sums of a value fit one wave
    const int G = std::min((ne + LB - 1) / LB, GMAX);
    const int *erow = d->brow, *orow = d->brow + nh;
    const int *e_nb = d->brank, *o_nb = d->brank + (size_t)nh * 8;   // ranks of a row's neighbours
    auto rows = [&](const Rows &a) { return rows_launch(a, nh, Ns, n, s); };
    std::vector<double> bn(poll ? n : 0, 0.0);
    auto fetch = [&](const double *dev, int count) -> int {
        DFL_HIP(hipMemcpyAsync(d->hp, dev, count * sizeof(double), hipMemcpyDeviceToHost, s));
        DFL_HIP(hipStreamSynchronize(s));
        return 0;
    };
    if (poll) {
        // ||u|| (its sums pass through the room of the step's)
        Scal sc;
        DFL_TRY(scalar_buffers_at(us + vec, n, sc));
        DFL_TRY(blas_norm2<double2>(u, (long)Nb * Ns, n, sc.part, sc.red, s));
        DFL_TRY(fetch(sc.red, n));
        for (int i = 0; i < n; ++i) bn[i] = std::sqrt(d->hp[i]);
    }
    // g = A_OO^{-1} u_O; r_0 = u' = u_E - A_EO g
    DFL_TRY(rows(Rows{d->Dinv, orow, 1, 0, 1, u, orow, Nb, nullptr, nullptr, 0, g, nullptr, nh, 1.0}));
    DFL_TRY(rows(Rows{d->A, erow, 9, 1, 8, g, e_nb, nh, u, erow, Nb, Rv, nullptr, nh, -1.0}));
    if (poll && maxit > nkv) DFL_HIP(hipMemcpyAsync(us, Rv, sizeof(double2) * vec, hipMemcpyDeviceToDevice, s));
    int iters = 0;
    double worst = 0;
    bool done = false, first = true;
    int at = 0, want = std::min(look, first_look(tol));   // steps since the last look, until the next one
    // y = the combination of k residuals (the first time), += it (after a restart)
    auto accum = [&](int k) -> int {
        k_little_accum<<<dim3(nblocks(ne, LB), n), LB, 0, s>>>(y, Rv, ne, n, k, Rm, cvec, first ? 1 : 0);
        DFL_HIP(hipGetLastError());
        first = false;
        return 0;
    };
    while (!done && iters < maxit) {
        int k = 0;
        while (!done && k < nkv && iters < maxit) {
            double2 *rk = Rv + (size_t)k * vec, *wk = W + (size_t)k * vec;
            // w = r - A_EO M1 r
            DFL_TRY(rows(Rows{d->M1, nullptr, 8, 0, 8, rk, o_nb, nh, nullptr, nullptr, 0, q, nullptr, nh, 1.0}));
            DFL_TRY(rows(Rows{d->A, erow, 9, 1, 8, q, e_nb, nh, rk, nullptr, nh, wk, nullptr, nh, -1.0}));
            double *mine = one + (size_t)(poll ? at : 0) * n * GMAX;   // its place among the steps of the look
            {
                ProfScope ps(PROF_BLAS, s);
                const dim3 grid(G, n);
                if (k > 0) k_little_dots<<<dim3(G, n, (k + 7) / 8), LB, 0, s>>>(W, ne, n, k, dots);
                k_little_sub<<<grid, LB, 0, s>>>(W, Rv, ne, n, k, dots, Rm, three);
                k_little_update<<<grid, LB, 0, s>>>(W, Rv, ne, n, k, three, Rm, cvec, mine);
                DFL_HIP(hipGetLastError());
            }
            ++k;
            ++iters;
            ++at;
            if (poll && (at == want || k == nkv || iters == maxit)) {
                DFL_TRY(little_norms(one, G, n * at, norms, s));
                DFL_TRY(fetch(norms, n * at));
                for (int c = 0; c < at && !done; ++c) {
                    done = true;
                    worst = 0;
                    for (int i = 0; i < n; ++i) {
                        const double rel = bn[i] > 0 ? std::sqrt(d->hp[c * n + i]) / bn[i] : 0.0;
                        worst = std::max(worst, rel);
                        if (!(rel <= tol)) done = false;
                    }
                    if (done) {   // the steps after this one do not count
                        iters -= at - 1 - c;
                        k -= at - 1 - c;
                    }
                }
                at = 0;
                want = std::min(look, next_look(iters, worst, tol));
            }
        }
        DFL_TRY(accum(k));
        if (!poll) break;
        if (!done && iters < maxit) {   // restart from the true residual u' - (y - A_EO M1 y)
            DFL_TRY(rows(Rows{d->M1, nullptr, 8, 0, 8, y, o_nb, nh, nullptr, nullptr, 0, q, nullptr, nh, 1.0}));
            DFL_TRY(rows(Rows{d->A, erow, 9, 1, 8, q, e_nb, nh, y, nullptr, nh, W, nullptr, nh, -1.0}));
            k_little_minus<<<nblocks((long)vec, 256), 256, 0, s>>>(us, W, Rv, (long)vec);
            DFL_HIP(hipGetLastError());
        }
    }
    if (first) DFL_TRY(accum(0));   // no steps (maxit <= 0): y = 0, x_E = 0 and x_O = g_O
    // x_O = g_O - M1 y, x_E = A_EE^{-1} y
    DFL_TRY(rows(Rows{d->M1, nullptr, 8, 0, 8, y, o_nb, nh, g, nullptr, nh, x, orow, Nb, -1.0}));
    DFL_TRY(rows(Rows{d->Dinv, erow, 1, 0, 1, y, nullptr, nh, nullptr, nullptr, 0, x, erow, Nb, 1.0}));
    if (iters_out) *iters_out = iters;
    if (relres_out) *relres_out = worst;
    return (poll && !done) ? QCD_NOCONV : 0;
}

}  // namespace dfl
