// Kernels that read and write vectors in the caller's canonical layout
// ([rhs][V][4 spin][3 colour] complex, lexicographic sites): the Dirac operator
// on canonical vectors, and the canonical <-> internal conversions.
//
// Internal positions pos and V/2 + pos are the two sites 2j, 2j + 1 of one
// block row (j = local lexicographic index >> 1, even block extents), so
// together they are one contiguous, even-aligned pair of canonical sites.  A
// workgroup takes up to 128 consecutive positions (256 sites); its canonical
// data are read and written as the pairs' 16-byte pieces, consecutive lanes on
// consecutive pieces, and change hands with the one-thread-per-site work in
// LDS.  A thread that reads its own site's 96 or 192 bytes instead touches a
// third of each line per instruction, and each line twice (once per parity).
#include <type_traits>

#include "block_tables.h"
#include "internal.h"

namespace dfl {

namespace {

constexpr int TP = CANON_TILE;   // 2 TP threads
typedef float q4 __attribute__((ext_vector_type(4)));   // one 16-byte piece

// LDS slot of a site, bytes: one 16-byte unit more than the site's own, so
// that consecutive slots start 4 banks times an odd number apart (16 lanes'
// 16-byte accesses at one offset then hit all 64 banks once)
template <class CT>
constexpr int slot_bytes() { return 12 * (int)sizeof(CT) + 16; }
template <class CT>
constexpr int pieces() { return 24 * (int)sizeof(CT) / 16; }   // 16-byte pieces of a pair

// first site (canonical index) of each pair of the tile; bit 31: its odd site
// comes first
__device__ inline void pair_table(const int *__restrict__ lex_of, long Vh, long pos0, int P, unsigned *lexp) {
    if ((int)threadIdx.x < P) {
        const unsigned e = lex_of[pos0 + threadIdx.x], o = lex_of[Vh + pos0 + threadIdx.x];
        lexp[threadIdx.x] = e < o ? e : (o | 0x80000000u);
    }
}

// Piece e of the tile: byte offset in a canonical vector and in LDS (site
// slots in the order even half, odd half)
template <class CT>
__device__ inline void piece_at(int e, const unsigned *lexp, unsigned &goff, unsigned &loff) {
    constexpr int NP = pieces<CT>(), H = NP / 2;
    const int pair = e / NP, k = e - pair * NP;
    const unsigned lp = lexp[pair];
    const int second = k >= H ? 1 : 0;
    const int par = second ^ (int)(lp >> 31);
    goff = (lp & 0x7fffffffu) * (12u * sizeof(CT)) + (unsigned)k * 16u;
    loff = (unsigned)(par * TP + pair) * slot_bytes<CT>() + (unsigned)(k - second * H) * 16u;
}

// canonical vector -> LDS slots, all threads (a tile of fewer pieces: the
// threads beyond them repeat its last piece)
template <class CT>
__device__ inline void tile_in(const char *__restrict__ src, unsigned char *lds, const unsigned *lexp, int P) {
    constexpr int NP = pieces<CT>(), PER = TP * NP / (2 * TP);
    q4 t[PER];
    unsigned lo[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        unsigned go;
        piece_at<CT>(min((int)threadIdx.x + k * 2 * TP, P * NP - 1), lexp, go, lo[k]);
        t[k] = *reinterpret_cast<const q4 *>(src + go);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) *reinterpret_cast<q4 *>(lds + lo[k]) = t[k];
}

// LDS slots -> canonical vector, all threads
template <class CT>
__device__ inline void tile_out(char *__restrict__ dst, const unsigned char *lds, const unsigned *lexp, int P) {
    constexpr int NP = pieces<CT>(), PER = TP * NP / (2 * TP);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        unsigned go, lo;
        piece_at<CT>(min((int)threadIdx.x + k * 2 * TP, P * NP - 1), lexp, go, lo);
        *reinterpret_cast<float4 *>(dst + go) = *reinterpret_cast<const float4 *>(lds + lo);
    }
}

// one site's spinor from 16-byte units at p (LDS or global memory)
template <class CT, class R>
__device__ inline void site_load(const char *p, cx<R> v[12]) {
    if constexpr (sizeof(CT) == 8) {
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            const float4 t = *reinterpret_cast<const float4 *>(p + 16 * c);
            v[2 * c] = {R(t.x), R(t.y)};
            v[2 * c + 1] = {R(t.z), R(t.w)};
        }
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const double2 t = *reinterpret_cast<const double2 *>(p + 16 * c);
            v[c] = {R(t.x), R(t.y)};
        }
    }
}
template <class CT, class R>
__device__ inline void site_store(unsigned char *p, const cx<R> v[12]) {
    if constexpr (sizeof(CT) == 8) {
#pragma unroll
        for (int c = 0; c < 6; ++c)
            *reinterpret_cast<float4 *>(p + 16 * c) = make_float4(float(v[2 * c].re), float(v[2 * c].im),
                                                                  float(v[2 * c + 1].re), float(v[2 * c + 1].im));
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c)
            *reinterpret_cast<double2 *>(p + 16 * c) = make_double2(double(v[c].re), double(v[c].im));
    }
}

// canonical -> internal
template <class CT, class S>
__global__ void __launch_bounds__(2 * TP) k_pack_tile(const CT *__restrict__ canon, void *__restrict__ out,
                                                      const int *__restrict__ lex_of, long V) {
    extern __shared__ unsigned char lds[];
    __shared__ unsigned lexp[TP];
    const long Vh = V / 2, pos0 = (long)blockIdx.x * TP;
    const int r = blockIdx.y;
    pair_table(lex_of, Vh, pos0, TP, lexp);
    __syncthreads();
    tile_in<CT>(reinterpret_cast<const char *>(canon + (size_t)r * V * 12), lds, lexp, TP);
    __syncthreads();
    using R = decltype(CT::x);
    cx<R> v[12];
    site_load<CT>(reinterpret_cast<const char *>(lds) + threadIdx.x * slot_bytes<CT>(), v);
    const int par = threadIdx.x / TP;
    Spin<S>::store(static_cast<char *>(out) + (size_t)r * Spin<S>::BYTES * V, V,
                   (unsigned)(par * Vh + pos0 + (threadIdx.x - par * TP)), v);
}

// internal -> canonical
template <class CT, class S>
__global__ void __launch_bounds__(2 * TP) k_unpack_tile(const void *__restrict__ in, CT *__restrict__ canon,
                                                        const int *__restrict__ lex_of, long V) {
    extern __shared__ unsigned char lds[];
    __shared__ unsigned lexp[TP];
    const long Vh = V / 2, pos0 = (long)blockIdx.x * TP;
    const int r = blockIdx.y;
    pair_table(lex_of, Vh, pos0, TP, lexp);
    using R = decltype(CT::x);
    cx<R> v[12];
    const int par = threadIdx.x / TP;
    Spin<S>::load(static_cast<const char *>(in) + (size_t)r * Spin<S>::BYTES * V, V,
                  (unsigned)(par * Vh + pos0 + (threadIdx.x - par * TP)), v);
    site_store<CT>(lds + threadIdx.x * slot_bytes<CT>(), v);
    __syncthreads();
    tile_out<CT>(reinterpret_cast<char *>(canon + (size_t)r * V * 12), lds, lexp, TP);
}

// ---------------------------------------------------------------------------
// the Dirac operator on canonical vectors
// ---------------------------------------------------------------------------

// The operator's raw data of one site, kept in registers over the right-hand
// sides of a workgroup (half-precision links and clover): forward links of the
// site, forward links of its four backward neighbours, clover.
template <class H4>
struct OpRegs {
    u32x2_t lf[4][3], lb[4][3], c[18];
};
// The compiler must not convert these once before the loop and keep the wide
// values instead: each use goes through an opaque copy.
__device__ inline u32x2_t opaque(u32x2_t t) {
    asm volatile("" : "+v"(t));
    return t;
}
template <class H4, class R>
__device__ inline void link_raw(const u32x2_t raw[3], cx<R> w[9]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const H4 t = __builtin_bit_cast(H4, opaque(raw[c]));
        w[2 * c] = {R(to_f(t.v[0])), R(to_f(t.v[1]))};
        w[2 * c + 1] = {R(to_f(t.v[2])), R(to_f(t.v[3]))};
    }
    rebuild_row2(w);
}

// One workgroup per tile; the tile's spinors are staged in LDS, neighbours
// outside it are read from the canonical vector, where a site is 96 (192)
// contiguous bytes: a 4^4 tile's 512 halo sites cost 1.1 times their own bytes,
// where the internal chunk-major layout pulls whole lines for the 16 to 32
// bytes of them that the y and z faces use.  At 32^3 x 64, FP16 links, 24
// right-hand sides: 17.7 GB of fetches and writes instead of 31.6 GB, and no
// conversion passes: 4.24 ms instead of 11.2 ms (2.72 pack, 4.80 stencil, 3.69
// unpack).  What is left is latency, eight hops each waiting for its halo lanes
// at 2 waves per SIMD (VALU busy 47%).  Measured and not kept: the halo staged
// in LDS as projected half-spinors (7.0 ms: per-lane 96-byte reads of all waves
// at once evict each other from the 32 KB cache), the next hop loaded ahead
// through branches (10 ms: spills), the next tile loaded ahead (4.3 ms).
//
// HALF: half-precision links and clover in registers (84 of the 246), the
// workgroup loops over `chunk` right-hand sides; otherwise they are read where
// they are used and a workgroup takes one right-hand side, 4 waves per SIMD.
template <class CT, class R, int LF, int CF, bool HALF>
__global__ void __launch_bounds__(2 * TP, HALF ? 2 : 1)
    k_dirac_canon(const CT *__restrict__ in, CT *__restrict__ out, const void *__restrict__ U,
                  const void *__restrict__ clo, const int *__restrict__ nbr, const int *__restrict__ lex_of,
                  const int *__restrict__ border, long V, int Vbh, int P, int tpb, R kappa, int nrhs, int chunk) {
    using H4 = std::conditional_t<LF == LNK_BF16, b4, h4>;
    constexpr int SB = slot_bytes<CT>();
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ unsigned lexp[TP];
    const long Vh = V / 2;
    unsigned bx, by;
    xcd_order(bx, by);
    // tpb tiles per Schwarz block, blocks in lexicographic order (tpb = 0:
    // tiles of several whole blocks, memory order)
    long pos0;
    if (tpb > 0) {
        const unsigned b = bx / (unsigned)tpb;
        pos0 = (long)border[b] * Vbh + (long)(bx - b * tpb) * P;
    } else {
        pos0 = (long)bx * P;
    }
    pair_table(lex_of, Vh, pos0, P, lexp);
    const int par = threadIdx.x / TP, j = threadIdx.x - par * TP;
    const unsigned x = (unsigned)(par * Vh + pos0 + (j < P ? j : 0));
    // neighbours: LDS offset of one inside the tile, canonical byte offset of
    // one outside; the boundary sign of the time hops
    unsigned where[8];
    unsigned inside = 0, neg = 0;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const int e = nbr_at(nbr, d, V, x);
        const unsigned y = nb_index(e);
        const unsigned q = y - (unsigned)((1 - par) * Vh + pos0);
        const bool is_in = q < (unsigned)P;
        where[d] = is_in ? ((unsigned)((1 - par) * TP) + q) * SB : (unsigned)lex_of[y] * (12u * sizeof(CT));
        inside |= is_in ? 1u << d : 0u;
        if (d < 2) neg |= e < 0 ? 1u << d : 0u;
    }
    OpRegs<H4> op;
    if constexpr (HALF) {
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const unsigned yb = nb_index(nbr_at(nbr, 2 * mu + 1, V, x));
            const u32x2_t *b = static_cast<const u32x2_t *>(U) + (size_t)mu * 3 * V;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                op.lf[mu][c] = ld<u32x2_t>(b, c, V, x);
                op.lb[mu][c] = ld<u32x2_t>(b, c, V, yb);
            }
        }
#pragma unroll
        for (int k = 0; k < 18; ++k)
            op.c[k] = ld<u32x2_t>(static_cast<const u32x2_t *>(clo) + (size_t)(k / 9) * 9 * V, k % 9, V, x);
    }
    // not HALF: one right-hand side in a single pass, so that nothing is hoisted
    // out of a loop
    const int r0 = HALF ? by * chunk : by, r1 = HALF ? min(nrhs, r0 + chunk) : r0 + 1;
    int r = r0;
    do {
        const char *src = reinterpret_cast<const char *>(in) + (size_t)r * V * 12 * sizeof(CT);
        __syncthreads();
        tile_in<CT>(src, lds, lexp, P);
        __syncthreads();
        cx<R> acc[12], w[9], p[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
        // a neighbour's spinor comes through a generic pointer: LDS inside the
        // tile, the canonical vector outside, in one instruction and without a
        // divergent branch; each direction ends in a scheduling fence, which
        // keeps the other directions' loads from being held in registers
#define DFL_CANON_HOP(MU, FWD)                                                                           \
    {                                                                                                   \
        constexpr int d = 2 * MU + (FWD ? 0 : 1);                                                       \
        site_load<CT>((inside >> d) & 1u ? reinterpret_cast<const char *>(lds) + where[d] : src + where[d], p); \
        if constexpr (HALF)                                                                             \
            link_raw<H4>(FWD ? op.lf[MU] : op.lb[MU], w);                                               \
        else                                                                                            \
            Link<LF>::load(U, V, MU, FWD ? x : nb_index(nbr_at(nbr, d, V, x)), w);                      \
        hop<R, MU, FWD>(w, p, MU == 0 ? ((neg >> d) & 1u ? R(-1) : R(1)) : R(1), acc);                  \
        __builtin_amdgcn_sched_barrier(0);                                                              \
    }
        DFL_CANON_HOP(0, true)
        DFL_CANON_HOP(0, false)
        DFL_CANON_HOP(1, true)
        DFL_CANON_HOP(1, false)
        DFL_CANON_HOP(2, true)
        DFL_CANON_HOP(2, false)
        DFL_CANON_HOP(3, true)
        DFL_CANON_HOP(3, false)
#undef DFL_CANON_HOP
        unsigned char *own = lds + threadIdx.x * SB;
        cx<R> o[12];
        site_load<CT>(reinterpret_cast<const char *>(own), p);
        if constexpr (HALF) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                R a[36];
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    const h4 t = __builtin_bit_cast(h4, opaque(op.c[9 * h + k]));
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[4 * k + e] = R(__half2float(t.v[e]));
                }
                herm6_apply(a, p + 6 * h, o + 6 * h);
            }
        } else {
            clover_apply<CF, R, false>(clo, V, x, p, o);
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) o[k] = rmac(o[k], -kappa, acc[k]);
        __syncthreads();
        site_store<CT>(own, o);   // a thread without a site writes its unused slot
        __syncthreads();
        tile_out<CT>(reinterpret_cast<char *>(out) + (size_t)r * V * 12 * sizeof(CT), lds, lexp, P);
        ++r;
    } while (HALF && r < r1);
}

template <class CT, class R, int LF, int CF, bool HALF>
int launch_canon(qcd_field f, const void *in, void *out, int nrhs, hipStream_t s) {
    const Geom &g = f->g;
    const int P = f->tile_pos;
    const int tpb = g.Vbh % P == 0 ? g.Vbh / P : 0;
    const unsigned tiles = (unsigned)(g.Vh / P);
    // right-hand sides per workgroup: all of them when the tiles alone fill
    // the device several times (512 workgroups are resident), fewer otherwise
    int chunk = 1;
    if (HALF) {
        const int split = std::max(1, std::min(nrhs, (int)(3072 / tiles)));
        chunk = (nrhs + split - 1) / split;
    }
    const double lbytes = LF == LNK_F64 ? 144 : LF == LNK_F32 ? 48 : 24;
    const double cbytes = CF == CLO_F64 ? 576 : CF == CLO_F32 ? 288 : 144;
    ProfScope ps(PROF_DIRAC, s, 1872.0 * g.V * nrhs, g.V * (4 * lbytes + cbytes + nrhs * 24.0 * sizeof(CT)),
                 1.0 * g.V * nrhs);
    k_dirac_canon<CT, R, LF, CF, HALF><<<dim3(tiles, (unsigned)((nrhs + chunk - 1) / chunk)), 2 * TP,
                                         (size_t)2 * TP * slot_bytes<CT>(), s>>>(
        static_cast<const CT *>(in), static_cast<CT *>(out), f->U[LF], f->clo[CF], f->nbr, f->lex_of, f->border, g.V,
        g.Vbh, P, tpb, (R)f->lat.kappa, nrhs, chunk);
    DFL_HIP(hipGetLastError());
    return 0;
}

template <class CT, class S>
int launch_pack(qcd_field f, const void *canon, void *internal, int nrhs, hipStream_t s) {
    const long V = f->g.V;
    k_pack_tile<CT, S><<<dim3((unsigned)(V / (2 * TP)), nrhs), 2 * TP, (size_t)2 * TP * slot_bytes<CT>(), s>>>(
        static_cast<const CT *>(canon), internal, f->lex_of, V);
    DFL_HIP(hipGetLastError());
    return 0;
}
template <class CT, class S>
int launch_unpack(qcd_field f, const void *internal, void *canon, int nrhs, hipStream_t s) {
    const long V = f->g.V;
    k_unpack_tile<CT, S><<<dim3((unsigned)(V / (2 * TP)), nrhs), 2 * TP, (size_t)2 * TP * slot_bytes<CT>(), s>>>(
        internal, static_cast<CT *>(canon), f->lex_of, V);
    DFL_HIP(hipGetLastError());
    return 0;
}

}  // namespace

// canonical pointers on which the tile kernels' 16-byte accesses are aligned
bool canon_aligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Whether the operator runs on the canonical vectors themselves: they hold the
// stencil's own vector type, are 16-byte aligned and do not overlap (staged
// copies would make an overlap harmless), the block shape gives tiles that fill a
// workgroup, and the handle asks for it or leaves every launch choice of the
// internal-layout stencils at its default.
bool canon_route(qcd_field f, const void *in, const void *out, int nrhs, qcd_prec io, qcd_prec storage, qcd_prec vin,
                 qcd_prec vout) {
    if (vin != io || vout != io || (io == QCD_F64) != (storage == QCD_F64)) return false;
    if (storage != QCD_F64 && storage != QCD_F32 && storage != QCD_F16 && storage != QCD_BF16) return false;
    const bool defaults = f->st_block == 1 && f->st_rg == 0 && f->st_order == 1 && f->st_nr == 0 && f->st_linklds == 1;
    if (f->st_canon == 2 || (f->st_canon == 0 && !defaults)) return false;
    if (!tiles_fill(f->tile_pos, CANON_TILE)) return false;
    if (!canon_aligned(in) || !canon_aligned(out)) return false;
    const size_t bytes = (size_t)nrhs * f->g.V * (io == QCD_F64 ? 192 : 96);
    const char *a = static_cast<const char *>(in), *b = static_cast<const char *>(out);
    return a + bytes <= b || b + bytes <= a;
}

int pack_tiles(qcd_field f, const void *canon, qcd_prec io, void *internal, qcd_prec vec, int nrhs, hipStream_t s) {
    if (io == QCD_F64) {
        if (vec == QCD_F64) return launch_pack<double2, double>(f, canon, internal, nrhs, s);
        if (vec == QCD_F32) return launch_pack<double2, float>(f, canon, internal, nrhs, s);
        return launch_pack<double2, __half>(f, canon, internal, nrhs, s);
    }
    if (vec == QCD_F64) return launch_pack<float2, double>(f, canon, internal, nrhs, s);
    if (vec == QCD_F32) return launch_pack<float2, float>(f, canon, internal, nrhs, s);
    return launch_pack<float2, __half>(f, canon, internal, nrhs, s);
}

int unpack_tiles(qcd_field f, const void *internal, qcd_prec vec, void *canon, qcd_prec io, int nrhs, hipStream_t s) {
    if (io == QCD_F64) {
        if (vec == QCD_F64) return launch_unpack<double2, double>(f, internal, canon, nrhs, s);
        if (vec == QCD_F32) return launch_unpack<double2, float>(f, internal, canon, nrhs, s);
        return launch_unpack<double2, __half>(f, internal, canon, nrhs, s);
    }
    if (vec == QCD_F64) return launch_unpack<float2, double>(f, internal, canon, nrhs, s);
    if (vec == QCD_F32) return launch_unpack<float2, float>(f, internal, canon, nrhs, s);
    return launch_unpack<float2, __half>(f, internal, canon, nrhs, s);
}

// The operator is worth keeping in registers (2 waves per SIMD instead of 4)
// from some right-hand sides per tile and some thousand tile passes on; FP16
// links, in registers / not: 32^3 x 64 n = 1 0.34 / 0.27 ms, n = 7 1.35 / 1.52,
// n = 24 4.24 / 5.06; 24^3 x 48 in 6^4 blocks n = 1 0.125 / 0.102, n = 7
// 0.49 / 0.58; 16^3 x 32 n = 12 0.169 / 0.158, n = 24 0.302 / 0.316.
template <int LF>
static int canon_half(qcd_field f, const void *in, void *out, int nrhs, hipStream_t s) {
    const long passes = f->g.Vh / f->tile_pos * nrhs;
    if (nrhs >= 4 && passes >= 8192) return launch_canon<float2, float, LF, CLO_F16, true>(f, in, out, nrhs, s);
    return launch_canon<float2, float, LF, CLO_F16, false>(f, in, out, nrhs, s);
}

int dirac_canon(qcd_field f, const void *in, void *out, int nrhs, qcd_prec storage, hipStream_t s) {
    switch (storage) {
        case QCD_F64: return launch_canon<double2, double, LNK_F64, CLO_F64, false>(f, in, out, nrhs, s);
        case QCD_F32: return launch_canon<float2, float, LNK_F32, CLO_F32, false>(f, in, out, nrhs, s);
        case QCD_F16: return canon_half<LNK_F16>(f, in, out, nrhs, s);
        case QCD_BF16: return canon_half<LNK_BF16>(f, in, out, nrhs, s);
        default: return set_error(QCD_EINVAL, "bad operator storage");
    }
}

}  // namespace dfl
