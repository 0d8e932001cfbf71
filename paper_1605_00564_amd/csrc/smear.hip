// Source and sink smearing (section 2.3): Gaussian smearing of quark fields
// with APE-smeared spatial links in the Laplacian.  The paper takes the
// parameters from earlier work; here they are arguments.
//
// APE step, for each spatial direction i and site x:
//   V = (1 - alpha) U_i(x) + (alpha / 4) sum_{j != i spatial}
//         [ U_j(x) U_i(x + j) U_j(x + i)^+ + U_j(x - j)^+ U_i(x - j) U_j(x - j + i) ],
//   U'_i(x) = W / det(W)^(1/3),  W = V (V^+ V)^(-1/2)  (polar factor; the cube
//   root is exp(i arg(det W) / 3), arg in (-pi, pi]).
// W is found by the Newton iteration W <- (W + W^{-+}) / 2, which converges
// quadratically to the polar factor of a nonsingular matrix; for 3 x 3
// matrices W^{-+} = conj(cof(W) / det(W)) with cof(W) the cofactor matrix,
// whose rows are cross products of the other two rows.
//
// Gaussian step: psi'(x) = [psi(x) + kappa sum_{i spatial} (U'_i(x) psi(x + i)
//   + U'_i(x - i)^+ psi(x - i))] / (1 + 6 kappa), colour only, each timeslice
// on its own.
//
// Both run in the lexicographic site order of the caller's vectors, links as
// [3][9][V] FP64 entries: the lanes of a wave are neighbours along z, so every
// load of a site or of its x, y, z neighbours is one contiguous run.  (In the
// solver's block order, 16-byte entries of the y and z neighbours lie 4 and 8
// apart, and each pulls a whole line.)
#include <cmath>

#include "internal.h"
#include "smear_rules.h"

namespace dfl {

namespace {

using cd = cx<double>;

__device__ inline void m_load(const double2 *U, long V, int i, unsigned x, cd m[9]) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const double2 t = U[((size_t)i * 9 + k) * V + x];
        m[k] = {t.x, t.y};
    }
}
// c = a b, a b^+, a^+ b
__device__ inline void m_mul(const cd a[9], const cd b[9], cd c[9]) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) c[3 * r + q] = cmac(cmac(a[3 * r] * b[q], a[3 * r + 1], b[3 + q]), a[3 * r + 2], b[6 + q]);
}
__device__ inline void m_mul_dag(const cd a[9], const cd b[9], cd c[9]) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            c[3 * r + q] = cmac(cmac(a[3 * r] * conj(b[3 * q]), a[3 * r + 1], conj(b[3 * q + 1])), a[3 * r + 2],
                                conj(b[3 * q + 2]));
}
__device__ inline void m_dag_mul(const cd a[9], const cd b[9], cd c[9]) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) c[3 * r + q] = cmacc(cmacc(cmulc(a[r], b[q]), a[3 + r], b[3 + q]), a[6 + r], b[6 + q]);
}

// projection onto SU(3): polar factor (Newton) divided by a cube root of its determinant
__device__ inline void project_su3(cd w[9]) {
    for (int it = 0; it < 40; ++it) {
        cd cof[9];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const cd *u = w + 3 * ((r + 1) % 3), *v = w + 3 * ((r + 2) % 3);
            cof[3 * r] = cmac(u[1] * v[2], -u[2], v[1]);
            cof[3 * r + 1] = cmac(u[2] * v[0], -u[0], v[2]);
            cof[3 * r + 2] = cmac(u[0] * v[1], -u[1], v[0]);
        }
        const cd det = cmac(cmac(w[0] * cof[0], w[1], cof[1]), w[2], cof[2]);
        const double dn = 1.0 / norm2(det);
        // conj(cof / det) = conj(cof) det / |det|^2
        double change = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const cd inv = dn * (conj(cof[k]) * det);
            const cd nw = 0.5 * (w[k] + inv);
            change += norm2(nw - w[k]);
            w[k] = nw;
        }
        // quadratic convergence: the error left is at most half of `change`
        // (1e-17) times |w^-1|, about 1
        if (change < 1e-17) break;
    }
    cd c0[3];
    const cd *u = w + 3, *v = w + 6;
    c0[0] = cmac(u[1] * v[2], -u[2], v[1]);
    c0[1] = cmac(u[2] * v[0], -u[0], v[2]);
    c0[2] = cmac(u[0] * v[1], -u[1], v[0]);
    const cd det = cmac(cmac(w[0] * c0[0], w[1], c0[1]), w[2], c0[2]);
    const double th = atan2(det.im, det.re) / 3.0;
    const cd ph = {cos(th), -sin(th)};
#pragma unroll
    for (int k = 0; k < 9; ++k) w[k] = w[k] * ph;
}

// Ends a hop or a staple: its sums are due here and later loads stay behind it
// (their pointers are not marked restrict, or they could pass).  Otherwise the
// compiler issues all loads first and adds up at the end, with 300 to 420
// registers.
template <int N>
__device__ inline void settle(cd (&acc)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) asm volatile("" : "+v"(acc[k].re), "+v"(acc[k].im) : : "memory");
}

// lexicographic index of the neighbours of site x = ((t X + x) Y + y) Z + z
struct Box {
    int X, Y, Z;
};
struct Site {
    unsigned x;
    int c[3];
};
__device__ inline Site site_of(const Box &b, unsigned x) {
    Site s;
    s.x = x;
    unsigned r = x / (unsigned)b.Z;
    s.c[2] = (int)(x - r * b.Z);
    const unsigned q = r / (unsigned)b.Y;
    s.c[1] = (int)(r - q * b.Y);
    s.c[0] = (int)(q % (unsigned)b.X);
    return s;
}
__device__ inline unsigned fwd(const Box &b, const Site &s, int i) {
    const int L = i == 0 ? b.X : i == 1 ? b.Y : b.Z, st = i == 0 ? b.Y * b.Z : i == 1 ? b.Z : 1;
    const int c = i == 0 ? s.c[0] : i == 1 ? s.c[1] : s.c[2];
    return s.x + (unsigned)(c + 1 == L ? -(L - 1) * st : st);
}
__device__ inline unsigned bwd(const Box &b, const Site &s, int i) {
    const int L = i == 0 ? b.X : i == 1 ? b.Y : b.Z, st = i == 0 ? b.Y * b.Z : i == 1 ? b.Z : 1;
    const int c = i == 0 ? s.c[0] : i == 1 ? s.c[1] : s.c[2];
    return s.x + (unsigned)(c == 0 ? (L - 1) * st : -st);
}

// One APE step on the spatial links Uin -> Uout.  FP64 arithmetic (about 3000
// instructions a link, half of them in the projection) and 13 link reads a link:
// one thread per link, the three directions of a tile of sites next to each
// other on one XCD, whose L2 they share.  32^3 x 64: 0.87 ms a step, 0.48 of it
// FP64 issue at 3 waves per SIMD (2.46 ms with one thread per site on the block
// order).
template <int I>
__device__ inline void ape_link(const double2 *Uin, double2 *Uout, const Box &box, long V, unsigned x,
                                double alpha) {
    const Site s = site_of(box, x);
    cd acc[9], a[9], b[9], t[9];
    m_load(Uin, V, I, x, a);
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[k] = (1.0 - alpha) * a[k];
    const unsigned xpi = fwd(box, s, I);
#pragma unroll
    for (int jj = 1; jj < 3; ++jj) {
        constexpr int J1 = I == 0 ? 1 : 0, J2 = I == 2 ? 1 : 2;   // the other directions, ascending
        const int j = jj == 1 ? J1 : J2;
        const unsigned xpj = fwd(box, s, j), xmj = bwd(box, s, j);
        const unsigned xmjpi = xmj + (xpi - x);   // the step along i does not depend on the coordinate along j
        // U_j(x) U_i(x + j) U_j(x + i)^+
        m_load(Uin, V, j, x, a);
        m_load(Uin, V, I, xpj, b);
        m_mul(a, b, t);
        m_load(Uin, V, j, xpi, b);
        m_mul_dag(t, b, a);
#pragma unroll
        for (int k = 0; k < 9; ++k) acc[k] = rmac(acc[k], 0.25 * alpha, a[k]);
        settle(acc);
        // U_j(x - j)^+ U_i(x - j) U_j(x - j + i)
        m_load(Uin, V, j, xmj, a);
        m_load(Uin, V, I, xmj, b);
        m_dag_mul(a, b, t);
        m_load(Uin, V, j, xmjpi, b);
        m_mul(t, b, a);
#pragma unroll
        for (int k = 0; k < 9; ++k) acc[k] = rmac(acc[k], 0.25 * alpha, a[k]);
        settle(acc);
    }
    project_su3(acc);
#pragma unroll
    for (int k = 0; k < 9; ++k) Uout[((size_t)I * 9 + k) * V + x] = make_double2(acc[k].re, acc[k].im);
}
__global__ void __launch_bounds__(128) k_ape_step(const double2 *Uin, double2 *Uout, Box box, long V,
                                                  double alpha) {
    unsigned bx, by;
    xcd_order(bx, by);
    const long x = (long)bx * blockDim.x + threadIdx.x;
    if (x >= V) return;
    switch (by) {
        case 0: ape_link<0>(Uin, Uout, box, V, (unsigned)x, alpha); break;
        case 1: ape_link<1>(Uin, Uout, box, V, (unsigned)x, alpha); break;
        default: ape_link<2>(Uin, Uout, box, V, (unsigned)x, alpha);
    }
}

// One Gaussian step on FP64 vectors [n][12][V] in lexicographic site order: one
// thread per site and vector, so that each of its 138 loads of 16 bytes is one
// contiguous kilobyte of the wave; the vectors of a tile of sites run back to
// back on one XCD and share its links through the L2.  24^3 x 48: 0.165 ms a
// vector and step, bound by the L2 (2.2 KB a site and vector at 16 TB/s).
__global__ void __launch_bounds__(256, 3) k_gauss_step(const double2 *in, double2 *out, const double2 *U, Box box,
                                                       long V, double kappa, double norm) {
    unsigned bx, by;
    xcd_order(bx, by);
    const unsigned x = bx * 256 + threadIdx.x;
    const Site s = site_of(box, x);
    const double2 *src = in + (size_t)by * 12 * V;
    cd acc[12], p[12], w[9];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const double2 t = src[(size_t)k * V + x];
        acc[k] = {t.x, t.y};
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const unsigned yf = fwd(box, s, i), yb = bwd(box, s, i);
        m_load(U, V, i, x, w);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const double2 t = src[(size_t)k * V + yf];
            p[k] = {t.x, t.y};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const cd t = cmac(cmac(w[3 * a] * p[3 * q], w[3 * a + 1], p[3 * q + 1]), w[3 * a + 2], p[3 * q + 2]);
                acc[3 * q + a] = rmac(acc[3 * q + a], kappa, t);
            }
        settle(acc);
        m_load(U, V, i, yb, w);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const double2 t = src[(size_t)k * V + yb];
            p[k] = {t.x, t.y};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const cd t = cmacc(cmacc(cmulc(w[a], p[3 * q]), w[3 + a], p[3 * q + 1]), w[6 + a], p[3 * q + 2]);
                acc[3 * q + a] = rmac(acc[3 * q + a], kappa, t);
            }
        settle(acc);
    }
    double2 *dst = out + (size_t)by * 12 * V;
#pragma unroll
    for (int k = 0; k < 12; ++k) dst[(size_t)k * V + x] = make_double2(norm * acc[k].re, norm * acc[k].im);
}

// The same for groups of four vectors (2 GW colour-vector pairs; the operator
// does not mix spins).  A workgroup stages the six links of each of 64 sites in
// LDS once (55 KB, two workgroups per CU) and each of its eight waves takes two
// colour vectors, so that one LDS read of a link serves both.  Groups run one
// after the other: the planes x - 1, x, x + 1 of four vectors (2.4 MB at 32^2
// sites) stay in an XCD's L2, those of twelve do not, and their neighbours came
// from HBM three times.  24^3 x 48, 12 vectors: 1.0 ms a step (2.03 ms on the
// block order; 1.13 with all twelve at once), again the L2's 16 TB/s.
constexpr int GW = 8;   // waves per workgroup
__global__ void __launch_bounds__(64 * GW, 4) k_gauss_step4(const double2 *in, double2 *out, const double2 *U, Box box,
                                                            long V, double kappa, double norm) {
    __shared__ double2 lk[6 * 9 * 64];
    // XCD k takes the k-th eighth of the list (group, tile), tiles fastest
    const unsigned gx = gridDim.x, tot = gx * gridDim.y;
    unsigned w = blockIdx.x + blockIdx.y * gx;
    if (tot % 8u == 0) w = (w & 7u) * (tot >> 3) + (w >> 3);
    const unsigned grp = w / gx, bx = w - grp * gx;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned x = bx * 64 + lane;
    const Site s = site_of(box, x);
    unsigned y[6];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        y[2 * i] = fwd(box, s, i);
        y[2 * i + 1] = bwd(box, s, i);
    }
    for (int e = wave; e < 54; e += GW) {
        const int d = e / 9;   // forward links at the site, backward ones at its neighbour
        const unsigned at = (d & 1) ? (d == 1 ? y[1] : d == 3 ? y[3] : y[5]) : x;
        lk[e * 64 + lane] = U[(size_t)((d >> 1) * 9 + (e - 9 * d)) * V + at];
    }
    const size_t off = ((size_t)grp * GW + wave) * 6 * V;
    const double2 *src = in + off;
    // the next direction's neighbours are on their way while one is computed
    cd acc[6], p[2][6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double2 t = src[(size_t)k * V + x], n = src[(size_t)k * V + y[0]];
        acc[k] = {t.x, t.y};
        p[0][k] = {n.x, n.y};
    }
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        if (d < 5)
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const double2 t = src[(size_t)k * V + y[d + 1]];
                p[(d + 1) & 1][k] = {t.x, t.y};
            }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            cd u[3];   // row a of the link, or column a of its adjoint's source
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double2 t = lk[(d * 9 + ((d & 1) ? 3 * c + a : 3 * a + c)) * 64 + lane];
                u[c] = {t.x, t.y};
            }
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const cd *h = p[d & 1] + 3 * v;
                const cd t = (d & 1) ? cmacc(cmacc(cmulc(u[0], h[0]), u[1], h[1]), u[2], h[2])
                                     : cmac(cmac(u[0] * h[0], u[1], h[1]), u[2], h[2]);
                acc[3 * v + a] = rmac(acc[3 * v + a], kappa, t);
            }
        }
        settle(acc);
    }
    double2 *dst = out + off;
#pragma unroll
    for (int k = 0; k < 6; ++k) dst[(size_t)k * V + x] = make_double2(norm * acc[k].re, norm * acc[k].im);
}

// canonical [n][V][12] <-> [n][12][V], 64 sites per workgroup through LDS, both
// sides in contiguous runs
template <class CT>
__global__ void __launch_bounds__(256) k_split(const CT *__restrict__ in, double2 *__restrict__ out, long V) {
    __shared__ CT sh[64 * 13];
    const long x0 = (long)blockIdx.x * 64;
    const CT *src = in + ((size_t)blockIdx.y * V + x0) * 12;
#pragma unroll
    for (int e = threadIdx.x; e < 64 * 12; e += 256) sh[(e / 12) * 13 + e % 12] = src[e];
    __syncthreads();
    double2 *dst = out + (size_t)blockIdx.y * 12 * V + x0;
#pragma unroll
    for (int e = threadIdx.x; e < 64 * 12; e += 256) {
        const CT t = sh[(e & 63) * 13 + (e >> 6)];
        dst[(size_t)(e >> 6) * V + (e & 63)] = make_double2(t.x, t.y);
    }
}
template <class CT>
__global__ void __launch_bounds__(256) k_join(const double2 *__restrict__ in, CT *__restrict__ out, long V) {
    __shared__ CT sh[64 * 13];
    const long x0 = (long)blockIdx.x * 64;
    const double2 *src = in + (size_t)blockIdx.y * 12 * V + x0;
#pragma unroll
    for (int e = threadIdx.x; e < 64 * 12; e += 256) {
        const double2 t = src[(size_t)(e >> 6) * V + (e & 63)];
        CT c;
        c.x = t.x;
        c.y = t.y;
        sh[(e & 63) * 13 + (e >> 6)] = c;
    }
    __syncthreads();
    CT *dst = out + ((size_t)blockIdx.y * V + x0) * 12;
#pragma unroll
    for (int e = threadIdx.x; e < 64 * 12; e += 256) dst[e] = sh[(e / 12) * 13 + e % 12];
}

// spatial links of the block-ordered FP64 copy -> lexicographic [3][9][V].  A
// workgroup's 256 consecutive sites are whole rows along z of a few y: together
// its lanes use the whole lines that they gather.
__global__ void __launch_bounds__(256) k_ape_import(const double2 *__restrict__ U, double2 *__restrict__ out,
                                                    const int *__restrict__ int_of, long V) {
    const long lex = (long)blockIdx.x * 256 + threadIdx.x;
    const unsigned idx = int_of[lex];
#pragma unroll
    for (int k = 0; k < 27; ++k) out[(size_t)k * V + lex] = U[(size_t)(9 + k) * V + idx];
}

// [3][9][V] -> canonical [V][3][3][3] (spatial direction i = mu - 1), 64 sites
// per workgroup through LDS, both sides in contiguous runs
__global__ void __launch_bounds__(256) k_ape_export(const double2 *__restrict__ U, double2 *__restrict__ out, long V) {
    __shared__ double2 sh[64 * 27];
    const long x0 = (long)blockIdx.x * 64;
    for (int e = threadIdx.x; e < 64 * 27; e += 256) {
        const int k = e >> 6, i = e & 63;
        sh[i * 27 + k] = U[(size_t)k * V + x0 + i];
    }
    __syncthreads();
    double2 *o = out + (size_t)x0 * 27;
    for (int e = threadIdx.x; e < 64 * 27; e += 256) o[e] = sh[e];
}

// n_iter steps from the caller's vectors to the caller's vectors, FP64 in
// between (scratch, so in and out may coincide)
template <class CT>
int gauss_run(qcd_field f, const CT *in, CT *out, int n, double kappa, int n_iter, hipStream_t s) {
    const long V = f->g.V;
    const size_t ne = (size_t)12 * V * n;
    const double norm = 1.0 / (1 + 6 * kappa);
    const Box box{f->g.L[1], f->g.L[2], f->g.L[3]};
    const double2 *U = static_cast<const double2 *>(f->Uape);
    void *ws;
    DFL_TRY(field_buffer(f, BUF_SAP_IO, 2 * sizeof(double2) * ne, &ws));
    double2 *a = static_cast<double2 *>(ws), *b = a + ne;
    ProfScope ps(PROF_OTHER, s);
    k_split<<<dim3((unsigned)(V / 64), n), 256, 0, s>>>(in, a, V);
    for (int it = 0; it < n_iter; ++it) {
        // groups of four vectors, then the others
        const int n4 = gauss_groups(V, n), rest = n - 4 * n4;
        if (n4)
            k_gauss_step4<<<dim3((unsigned)(V / 64), n4), 64 * GW, 0, s>>>(a, b, U, box, V, kappa, norm);
        if (rest) {
            const size_t done = (size_t)48 * V * n4;
            k_gauss_step<<<dim3((unsigned)(V / 256), rest), 256, 0, s>>>(a + done, b + done, U, box, V, kappa, norm);
        }
        std::swap(a, b);
    }
    k_join<<<dim3((unsigned)(V / 64), n), 256, 0, s>>>(a, out, V);
    DFL_HIP(hipGetLastError());
    return 0;
}

}  // namespace
}  // namespace dfl

using namespace dfl;

extern "C" int qcd_field_ape_smear(qcd_field f, double alpha, int n_iter, hipStream_t s) {
    if (!f || n_iter < 0 || !std::isfinite(alpha)) return set_error(QCD_EINVAL, "bad arguments to qcd_field_ape_smear");
    const long V = f->g.V;
    const size_t bytes = sizeof(double2) * 27 * (size_t)V;
    // the scratch first, and new links reach the handle once they are on their
    // way: a call that fails leaves what it had (links, or none)
    void *w = nullptr, *links = f->Uape;
    if (n_iter > 0) DFL_TRY(field_buffer(f, BUF_APPLY, bytes, &w));
    if (!links && !dev_alloc(f->device, &links, bytes))
        return set_error(QCD_ENOMEM, "device allocation of the smeared links failed");
    // spatial links of the FP64 copy, then n_iter steps ping-ponging through
    // the handle's scratch, so that the last one lands in the kept links
    const double2 *U64 = static_cast<const double2 *>(f->U[LNK_F64]);
    const Box box{f->g.L[1], f->g.L[2], f->g.L[3]};
    double2 *a = static_cast<double2 *>(links), *b = static_cast<double2 *>(w);
    if (n_iter % 2) std::swap(a, b);
    ProfScope ps(PROF_OTHER, s);
    k_ape_import<<<(unsigned)(V / 256), 256, 0, s>>>(U64, a, f->int_of, V);
    for (int it = 0; it < n_iter; ++it) {
        k_ape_step<<<dim3(nblocks(V, 128), 3), 128, 0, s>>>(a, b, box, V, alpha);
        std::swap(a, b);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        if (!f->Uape) (void)hipFree(links);
        return set_error(QCD_EHIP, std::string("APE smearing: ") + hipGetErrorString(e));
    }
    f->Uape = links;
    return 0;
}

extern "C" int qcd_field_get_ape_links(qcd_field f, void *links, hipStream_t s) {
    if (!f || !links) return set_error(QCD_EINVAL, "bad arguments to qcd_field_get_ape_links");
    if (!f->Uape) return set_error(QCD_ENOTSET, "no smeared links: call qcd_field_ape_smear first");
    k_ape_export<<<(unsigned)(f->g.V / 64), 256, 0, s>>>(static_cast<const double2 *>(f->Uape),
                                                         static_cast<double2 *>(links), f->g.V);
    DFL_HIP(hipGetLastError());
    return 0;
}

extern "C" int gauss_smear(qcd_field f, const void *in, void *out, int nrhs, qcd_prec io, double kappa_g, int n_iter,
                           hipStream_t s) {
    if (!f || !in || !out || nrhs <= 0 || n_iter < 0 || !std::isfinite(kappa_g))
        return set_error(QCD_EINVAL, "bad arguments to gauss_smear");
    if (io != QCD_F64 && io != QCD_F32) return set_error(QCD_EINVAL, "io precision must be F64 or F32");
    if (!f->Uape) return set_error(QCD_ENOTSET, "no smeared links: call qcd_field_ape_smear first");
    if (1 + 6 * kappa_g == 0) return set_error(QCD_EINVAL, "kappa_g = -1/6 is singular");
    if (io == QCD_F64)
        return gauss_run(f, static_cast<const double2 *>(in), static_cast<double2 *>(out), nrhs, kappa_g, n_iter, s);
    return gauss_run(f, static_cast<const float2 *>(in), static_cast<float2 *>(out), nrhs, kappa_g, n_iter, s);
}
