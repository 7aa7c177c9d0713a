// Wilson-Dirac stencil H_W(mu) = gamma5 D_W(mu) on gfx950.
//
// One thread per lattice site, 256 threads (4 wavefronts) per block, blocks
// ordered per XCD (xcd_block).  Each of the 8 hops projects the neighbour
// spinor to a half spinor with (1 -+ gamma_nu) (DeGrand-Rossi basis), applies
// U or U^H to the two colour vectors, scales by -kappa * weight * boundary
// factor, and adds the reconstructed 4-spinor.  The chemical potential enters
// only as the weights e^{-mu} (forward time hop) and e^{+mu} (backward time
// hop); the adjoint H_W(mu)^H = H_W(-mu) is the same kernel with mu -> -mu.
// Single-RHS stencil: HBM-bound, 1368 flop per site.  On small lattices, and for fields in the canonical
// layout, one wavefront per hop (the split kernel) instead of one thread per site.
#include "field_io.h"
#include "launch.h"

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <type_traits>

#ifndef SGN_STENCIL_WAVES
#define SGN_STENCIL_WAVES 1
#endif
#ifndef SGN_STENCIL_THREADS
#define SGN_STENCIL_THREADS 256
#endif
#ifndef SGN_XCD_REMAP
#define SGN_XCD_REMAP 1
#endif
#ifndef SGN_T_MINOR
#define SGN_T_MINOR 1   // t-fastest block order inside each XCD's t-slab when the shape allows
#endif
#ifndef SGN_PIN_PAIR
#define SGN_PIN_PAIR 0   // 1: both hops of a direction in flight together
#endif
#ifndef SGN_STENCIL_LDS
#define SGN_STENCIL_LDS 1   // single-RHS stencil with the block's own spinors staged in LDS
#endif
#ifndef SGN_STAGED_STRIP
#define SGN_STAGED_STRIP 1   // staged kernel block order: 0 = z-fastest XCD t-slabs, W > 0 = t-fastest strips of W blocks
#endif
#ifndef SGN_NT_OUT
#define SGN_NT_OUT 1     // non-temporal stores of the stencil output
#endif
#ifndef SGN_LDS_MAXBYTES
#define SGN_LDS_MAXBYTES 64512   // dynamic LDS budget of one block of the staged stencil (64 KiB less the reduction scratch)
#endif

namespace sgn {

namespace {

}  // namespace
// right-hand sides of one multi-RHS application (one block walks all of them; a
// StencilParams holding this many is 2 KiB, within the kernel-argument limit)
constexpr int kMaxRhs = 16;
namespace {

struct RhsParams {
    const void *in;
    void *out;
    double wf_t, wb_t;  // time-hop weights e^{-mu}, e^{+mu} of this right-hand side
    float s5_in;        // -1: apply gamma5 to the input first
    float s5_out;       // -1: apply gamma5 to the result
    // epilogue  out = a * in_scale * Op(in) + b * z ;  partials of conj(w) . out
    double a;
    z64 b;
    const z64 *b_dev;
    const void *z;
    const void *w;
    z64 *partials;
    const z64 *in_scale;
    int norm;  // with w: partials hold {conj(w) . out, ||out||^2} per block
};

struct StencilParams {
    const void *links;
    int V;  // sites
    int S;  // component stride
    int L[4];
    int stride[4];
    float bcf[4];  // boundary factor per direction (hops that wrap)
    double kappa;
    // block schedule: when sched_T > 0, XCD k owns the t-slab [k*T, (k+1)*T) and
    // walks it region by region with t fastest (sched_R spatial regions per slice)
    int sched_T, sched_R;
    int nblk_sites;  // blocks covering the V sites; later blocks zero the padding sites [V, S)
    int blk_sites;   // staged kernel: sites per block and t-slice (whole x-rows)
    int tslices;     // staged kernel: t-slices per block (1, or 2: a brick of the same B sites at t and t + 1)
    int nblk_total;  // blocks of this application (sites + padding); batched launches skip the rest
    // split kernel with a dot product: the blocks are the wavefronts of the staged kernel's blocks (grp_n blocks of
    // grp_sites sites, grp_waves wavefronts each; grp_waves = 0: 64 consecutive sites per block)
    int grp_sites, grp_waves, grp_n;
    int link_ne;     // complex entries stored per link (6 or 9)
    int tgauge;      // temporal gauge: U_t = 1 off the last time slice (the staged and split kernels skip those links)
    int nrhs;        // right-hand sides of this application (staged kernel; the unstaged one uses NR)
    RhsParams rhs[kMaxRhs];
};

// Complex arithmetic of the hops written as fused multiply-adds: a complex
// multiply-accumulate is four FMAs (the plain expression s + a * b compiles to
// two multiplies, two FMAs and two adds, as the compiler may not reassociate).

// s = a b, or s = conj(a) b with CONJ
template <bool CONJ, typename R>
__device__ __forceinline__ cpx<R> cmul_f(cpx<R> a, cpx<R> b)
{
    cpx<R> s;
    s.r = a.r * b.r;
    s.r = fma(CONJ ? a.i : -a.i, b.i, s.r);
    s.i = a.r * b.i;
    s.i = fma(CONJ ? -a.i : a.i, b.r, s.i);
    return s;
}

// s += a b, or s += conj(a) b with CONJ
template <bool CONJ, typename R>
__device__ __forceinline__ void cmac_f(cpx<R> &s, cpx<R> a, cpx<R> b)
{
    s.r = fma(a.r, b.r, s.r);
    s.r = fma(CONJ ? a.i : -a.i, b.i, s.r);
    s.i = fma(a.r, b.i, s.i);
    s.i = fma(CONJ ? -a.i : a.i, b.r, s.i);
}

// a + f * (ph b) for the phase ph in {+1, -1, +i, -i} (PH = 0, 1, 2, 3) and a real f
template <int PH, typename R>
__device__ __forceinline__ cpx<R> add_ph(cpx<R> a, R f, cpx<R> b)
{
    if constexpr (PH == 0) return {fma(f, b.r, a.r), fma(f, b.i, a.i)};
    else if constexpr (PH == 1) return {fma(-f, b.r, a.r), fma(-f, b.i, a.i)};
    else if constexpr (PH == 2) return {fma(-f, b.i, a.r), fma(f, b.r, a.i)};
    else return {fma(f, b.i, a.r), fma(-f, b.r, a.i)};
}

constexpr int kP1 = 0, kM1 = 1, kPI = 2, kMI = 3;

// Half-spinor projection (1 - gamma_nu) for FWD, (1 + gamma_nu) otherwise, of
// the spinor p with its lower two spins multiplied by s5 (the input gamma5
// sign, folded into the adds): h[0..2] = colour vector of the upper-spin-0
// row, h[3..5] = spin-1 row.
template <int NU, bool FWD, typename R>
__device__ __forceinline__ void project(const cpx<R> p[12], cpx<R> h[6], R s5)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        cpx<R> p0 = p[c], p1 = p[3 + c], p2 = p[6 + c], p3 = p[9 + c];
        if constexpr (NU == 0) {
            h[c] = FWD ? add_ph<kMI>(p0, s5, p3) : add_ph<kPI>(p0, s5, p3);
            h[3 + c] = FWD ? add_ph<kMI>(p1, s5, p2) : add_ph<kPI>(p1, s5, p2);
        } else if constexpr (NU == 1) {
            h[c] = FWD ? add_ph<kP1>(p0, s5, p3) : add_ph<kM1>(p0, s5, p3);
            h[3 + c] = FWD ? add_ph<kM1>(p1, s5, p2) : add_ph<kP1>(p1, s5, p2);
        } else if constexpr (NU == 2) {
            h[c] = FWD ? add_ph<kMI>(p0, s5, p2) : add_ph<kPI>(p0, s5, p2);
            h[3 + c] = FWD ? add_ph<kPI>(p1, s5, p3) : add_ph<kMI>(p1, s5, p3);
        } else {
            h[c] = FWD ? add_ph<kM1>(p0, s5, p2) : add_ph<kP1>(p0, s5, p2);
            h[3 + c] = FWD ? add_ph<kM1>(p1, s5, p3) : add_ph<kP1>(p1, s5, p3);
        }
    }
}

// acc += coef * reconstruct(chi): upper spins are chi0, chi1; lower spins follow
// from the rank-2 structure of (1 -+ gamma_nu).  Every real component is one FMA.
template <int NU, bool FWD, typename R>
__device__ __forceinline__ void accumulate(cpx<R> acc[12], const cpx<R> chi[6], R coef)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cpx<R> h0 = chi[c], h1 = chi[3 + c];
        acc[c] = add_ph<kP1>(acc[c], coef, h0);
        acc[3 + c] = add_ph<kP1>(acc[3 + c], coef, h1);
        if constexpr (NU == 0) {
            acc[6 + c] = FWD ? add_ph<kPI>(acc[6 + c], coef, h1) : add_ph<kMI>(acc[6 + c], coef, h1);
            acc[9 + c] = FWD ? add_ph<kPI>(acc[9 + c], coef, h0) : add_ph<kMI>(acc[9 + c], coef, h0);
        } else if constexpr (NU == 1) {
            acc[6 + c] = FWD ? add_ph<kM1>(acc[6 + c], coef, h1) : add_ph<kP1>(acc[6 + c], coef, h1);
            acc[9 + c] = FWD ? add_ph<kP1>(acc[9 + c], coef, h0) : add_ph<kM1>(acc[9 + c], coef, h0);
        } else if constexpr (NU == 2) {
            acc[6 + c] = FWD ? add_ph<kPI>(acc[6 + c], coef, h0) : add_ph<kMI>(acc[6 + c], coef, h0);
            acc[9 + c] = FWD ? add_ph<kMI>(acc[9 + c], coef, h1) : add_ph<kPI>(acc[9 + c], coef, h1);
        } else {
            acc[6 + c] = FWD ? add_ph<kM1>(acc[6 + c], coef, h0) : add_ph<kP1>(acc[6 + c], coef, h0);
            acc[9 + c] = FWD ? add_ph<kM1>(acc[9 + c], coef, h1) : add_ph<kP1>(acc[9 + c], coef, h1);
        }
    }
}

// chi = U h (forward) or U^H h (backward), on both colour vectors
template <bool ADJ, typename R>
__device__ __forceinline__ void link_mul(const cpx<R> u[9], const cpx<R> h[6], cpx<R> chi[6])
{
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            cpx<R> s = cmul_f<ADJ>(ADJ ? u[a] : u[a * 3], h[3 * v]);
#pragma unroll
            for (int b = 1; b < 3; ++b) cmac_f<ADJ>(s, ADJ ? u[b * 3 + a] : u[a * 3 + b], h[3 * v + b]);
            chi[3 * v + a] = s;
        }
}

template <typename R>
using SpT = typename SpinorStore<R>::type;

// One component's terms of the partial sums conj(w) . out and ||out||^2, in FP64.  The products are contracted here
// and not by the compiler, in one place for every kernel, so that the sums have the same bits whichever one runs
// (the order within a term differs between the precisions, as it always has).
template <typename R>
__device__ __forceinline__ void dot_terms(cpx<R> w, cpx<R> out, double &dr, double &di, double &dn)
{
    constexpr bool kRealFirst = sizeof(R) == 8;
    const z64 a = cast<double>(w), o = cast<double>(out);
    dr += kRealFirst ? fma(a.i, o.i, a.r * o.r) : fma(a.r, o.r, a.i * o.i);
    di += fma(a.r, o.i, -(a.i * o.r));
    dn += kRealFirst ? fma(o.i, o.i, o.r * o.r) : fma(o.r, o.r, o.i * o.i);
}

// Output side of one site: gamma5 on the result, the epilogue
// out = a * in_scale * Op(in) + b * z, the store, and the site's terms of the
// partial sums conj(w) . out and ||out||^2 (FP64).  The scales are real unless
// in_scale / b_dev / Im b say otherwise (wave-uniform branches), and a dot
// partner equal to z is not read twice.
template <typename R, bool kEpi, bool kDot>
__device__ __forceinline__ void finish_site(cpx<R> (&acc)[12], const RhsParams &Q, int S, int s, double &dr,
                                            double &di, double &dn)
{
    const R s5o = static_cast<R>(Q.s5_out);
    cpx<R> zz[12];
    if constexpr (!kEpi) {
#pragma unroll
        for (int k = 6; k < 12; ++k) acc[k] = s5o * acc[k];
    } else {
        if (Q.in_scale) {
            const z64 t = *Q.in_scale;
            const cpx<R> sc = {static_cast<R>(Q.a * t.r), static_cast<R>(Q.a * t.i)};
            const cpx<R> sl = {s5o * sc.r, s5o * sc.i};
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = cmul_f<false>(k < 6 ? sc : sl, acc[k]);
        } else {
            const R a = static_cast<R>(Q.a), al = s5o * a;
#pragma unroll
            for (int k = 0; k < 12; ++k) acc[k] = (k < 6 ? a : al) * acc[k];
        }
        if (Q.z) {
            load_spinor(static_cast<const SpT<R> *>(Q.z), S, s, zz);
            if (!Q.b_dev && Q.b.i == 0.0) {
                const R b = static_cast<R>(Q.b.r);
#pragma unroll
                for (int k = 0; k < 12; ++k) acc[k] = add_ph<kP1>(acc[k], b, zz[k]);
            } else {
                z64 bb = Q.b;
                if (Q.b_dev) {
                    const z64 t = *Q.b_dev;
                    bb = {bb.r * t.r - bb.i * t.i, bb.r * t.i + bb.i * t.r};
                }
                const cpx<R> b = {static_cast<R>(bb.r), static_cast<R>(bb.i)};
#pragma unroll
                for (int k = 0; k < 12; ++k) cmac_f<false>(acc[k], b, zz[k]);
            }
        }
    }
    if (SGN_NT_OUT)
        store_spinor_nt(static_cast<SpT<R> *>(Q.out), S, s, acc);
    else
        store_spinor(static_cast<SpT<R> *>(Q.out), S, s, acc);
    if constexpr (kDot) {
        if (Q.w) {
            cpx<R> ww[12];
            if (kEpi && Q.w == Q.z) {
#pragma unroll
                for (int k = 0; k < 12; ++k) ww[k] = zz[k];
            } else {
                load_spinor(static_cast<const SpT<R> *>(Q.w), S, s, ww);
            }
#pragma unroll
            for (int k = 0; k < 12; ++k) dot_terms<R>(ww[k], acc[k], dr, di, dn);
        }
    }
}

// Ordering fence between hops: the accumulator must be complete here and no
// later load may move above it.  Without it the compiler issues all 8
// neighbour gathers up front and the kernel needs >300 VGPRs (spills, one
// wave per SIMD).
template <typename R>
__device__ __forceinline__ void pin(cpx<R> acc[12])
{
#pragma unroll
    for (int k = 0; k < 12; ++k) asm volatile("" : "+v"(acc[k].r), "+v"(acc[k].i)::"memory");
}

template <int NU, int NR, typename R, typename LT>
__device__ __forceinline__ void hop_pair(cpx<R> (&acc)[NR][12], const StencilParams &P, int s, int coord)
{
    const LT *U = static_cast<const LT *>(P.links);
    const int L = P.L[NU], st = P.stride[NU];
    const R kap = static_cast<R>(P.kappa);
    cpx<R> u[9];
    // forward hop: (1 - gamma) U_nu(x) psi(x + nu), the link shared by all right-hand sides
    {
        const bool wrap = coord == L - 1;
        const int n = wrap ? s - (L - 1) * st : s + st;
        const R bcf = wrap ? static_cast<R>(P.bcf[NU]) : R(1);
        load_link<R>(U, P.S, P.link_ne, NU, s, u);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            cpx<R> p[12], h[6], chi[6];
            load_spinor(static_cast<const SpT<R> *>(P.rhs[r].in), P.S, n, p);
            project<NU, true>(p, h, static_cast<R>(P.rhs[r].s5_in));
            link_mul<false>(u, h, chi);
            const R w = NU == 3 ? static_cast<R>(P.rhs[r].wf_t) : R(1);
            accumulate<NU, true>(acc[r], chi, -kap * w * bcf);
        }
    }
    if (!SGN_PIN_PAIR) {
#pragma unroll
        for (int r = 0; r < NR; ++r) pin(acc[r]);
    }
    // backward hop: (1 + gamma) U_nu(x - nu)^H psi(x - nu)
    {
        const bool wrap = coord == 0;
        const int n = wrap ? s + (L - 1) * st : s - st;
        const R bcb = wrap ? static_cast<R>(P.bcf[NU]) : R(1);
        load_link<R>(U, P.S, P.link_ne, NU, n, u);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            cpx<R> p[12], h[6], chi[6];
            load_spinor(static_cast<const SpT<R> *>(P.rhs[r].in), P.S, n, p);
            project<NU, false>(p, h, static_cast<R>(P.rhs[r].s5_in));
            link_mul<true>(u, h, chi);
            const R w = NU == 3 ? static_cast<R>(P.rhs[r].wb_t) : R(1);
            accumulate<NU, false>(acc[r], chi, -kap * w * bcb);
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) pin(acc[r]);
}

template <typename R, typename LT, int NR, bool kEpi, bool kDot>
__global__ void __launch_bounds__(SGN_STENCIL_THREADS) __attribute__((amdgpu_waves_per_eu(SGN_STENCIL_WAVES))) stencil_kernel(StencilParams P)
{
    if ((int)blockIdx.x >= P.nblk_sites) {  // padding of the component arrays: keep it zero
        const int s = P.V + ((int)blockIdx.x - P.nblk_sites) * SGN_STENCIL_THREADS + threadIdx.x;
        if (s < P.S) {
            cpx<R> zero[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) zero[k] = {R(0), R(0)};
#pragma unroll
            for (int r = 0; r < NR; ++r) store_spinor(static_cast<SpT<R> *>(P.rhs[r].out), P.S, s, zero);
        }
        if constexpr (kDot) {
            if (threadIdx.x == 0)
                for (int r = 0; r < NR; ++r)
                    if (P.rhs[r].w) {
                        if (P.rhs[r].norm) {
                            P.rhs[r].partials[2 * blockIdx.x] = {0.0, 0.0};
                            P.rhs[r].partials[2 * blockIdx.x + 1] = {0.0, 0.0};
                        } else {
                            P.rhs[r].partials[blockIdx.x] = {0.0, 0.0};
                        }
                    }
        }
        return;
    }
    int blk;
    if (P.sched_T > 0) {
        // t-minor order inside each XCD's slab: the t-neighbours of a block are the
        // blocks just before and after it
        const int k = blockIdx.x % 8, j = blockIdx.x / 8;
        const int tl = j % P.sched_T, r = j / P.sched_T;
        blk = (k * P.sched_T + tl) * P.sched_R + r;
    } else {
        blk = SGN_XCD_REMAP ? xcd_block(blockIdx.x, P.nblk_sites) : (int)blockIdx.x;
    }
    const int s = blk * SGN_STENCIL_THREADS + threadIdx.x;
    const bool valid = s < P.V;
    double dr[NR], di[NR], dn[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) dr[r] = di[r] = dn[r] = 0.0;
    if (valid) {
        int c0 = s % P.L[0];
        int q = s / P.L[0];
        int c1 = q % P.L[1];
        q /= P.L[1];
        int c2 = q % P.L[2];
        int c3 = q / P.L[2];
        cpx<R> acc[NR][12];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            load_spinor(static_cast<const SpT<R> *>(P.rhs[r].in), P.S, s, acc[r]);
            const R s5 = static_cast<R>(P.rhs[r].s5_in);
#pragma unroll
            for (int k = 6; k < 12; ++k) acc[r][k] = s5 * acc[r][k];
        }
        hop_pair<0, NR, R, LT>(acc, P, s, c0);
        hop_pair<1, NR, R, LT>(acc, P, s, c1);
        hop_pair<2, NR, R, LT>(acc, P, s, c2);
        hop_pair<3, NR, R, LT>(acc, P, s, c3);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            finish_site<R, kEpi, kDot>(acc[r], P.rhs[r], P.S, s, dr[r], di[r], dn[r]);
        }
    }
    if constexpr (kDot) {
        __shared__ double lds[3 * (SGN_STENCIL_THREADS / 64)];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (!P.rhs[r].w) continue;  // uniform
            double v[3] = {dr[r], di[r], dn[r]};
            block_sum<3>(v, lds);
            if (threadIdx.x == 0) {
                if (P.rhs[r].norm) {
                    P.rhs[r].partials[2 * blockIdx.x] = {v[0], v[1]};
                    P.rhs[r].partials[2 * blockIdx.x + 1] = {v[2], 0.0};
                } else {
                    P.rhs[r].partials[blockIdx.x] = {v[0], v[1]};
                }
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------- staged stencil
// Single right-hand side.  A block owns B consecutive sites made of whole
// x-rows (whole x-y planes when they fit), so the +-x neighbours of every site
// and, for whole planes, the +-y neighbours too lie inside the block.  Each
// thread loads its own spinor once (it is needed for the diagonal term anyway)
// and stores it in LDS; a neighbour inside the block is then read from LDS and
// only the others (+-z, +-t, block-edge rows) are gathered from memory.

// largest block of the staged kernel (the LDS budget allows at most 64512/192 = 336 FP64 and
// 672 FP32 sites): FP64 needs ~180 VGPRs, so at most 2 waves per SIMD; the FP32 bound leaves up
// to 168 VGPRs for the multi-RHS form that holds every link of a site in registers
template <typename R> constexpr int kStagedMaxThreads = sizeof(R) == 8 ? 512 : 704;
// the multi-RHS form with the links in registers (FP16 links): 8 waves per block at most, so
// up to 256 VGPRs (two waves per SIMD)
constexpr int kRegsMaxThreads = 512;
// the split kernel leaves one partial sum per wavefront of such a block, or of the unstaged kernel's
static_assert((std::max(kStagedMaxThreads<float>, kStagedMaxThreads<double>) + 63) / 64 <= kMaxPartialWidth &&
                  (SGN_STENCIL_THREADS + 63) / 64 <= kMaxPartialWidth,
              "the readers of the partial sums add kMaxPartialWidth entries at most");

template <typename R>
__device__ __forceinline__ void lds_store_spinor(SpT<R> *l, int B, int i, const cpx<R> v[12]);
template <>
__device__ __forceinline__ void lds_store_spinor<double>(double2 *l, int B, int i, const cpx<double> v[12])
{
#pragma unroll
    for (int c = 0; c < 12; ++c) l[c * B + i] = make_double2(v[c].r, v[c].i);
}
template <>
__device__ __forceinline__ void lds_store_spinor<float>(float4 *l, int B, int i, const cpx<float> v[12])
{
#pragma unroll
    for (int c = 0; c < 6; ++c) l[c * B + i] = make_float4(v[2 * c].r, v[2 * c].i, v[2 * c + 1].r, v[2 * c + 1].i);
}

template <typename R>
__device__ __forceinline__ void lds_load_spinor(const SpT<R> *l, int B, int i, cpx<R> v[12]);
template <>
__device__ __forceinline__ void lds_load_spinor<double>(const double2 *l, int B, int i, cpx<double> v[12])
{
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        double2 t = l[c * B + i];
        v[c] = {t.x, t.y};
    }
}
template <>
__device__ __forceinline__ void lds_load_spinor<float>(const float4 *l, int B, int i, cpx<float> v[12])
{
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        float4 t = l[c * B + i];
        v[2 * c] = {t.x, t.y};
        v[2 * c + 1] = {t.z, t.w};
    }
}

// neighbour spinor n of right-hand side Q: from LDS when it belongs to this block
// (stored already multiplied by the input gamma5 sign), else from memory.  Returns
// the gamma5 sign the projection still has to apply to the lower spins.
template <typename R>
__device__ __forceinline__ R fetch_neighbour(const RhsParams &Q, const StencilParams &P, const SpT<R> *lds, int base,
                                             int n, cpx<R> p[12])
{
    const int B = P.blk_sites, NB = B * P.tslices;
    int ln = n - base;
    if ((unsigned)ln < (unsigned)B) {
        lds_load_spinor<R>(lds, NB, ln, p);
        return R(1);
    }
    if (P.tslices == 2) {  // the brick's second slice (uniform branch)
        ln = n - base - P.stride[3];
        if ((unsigned)ln < (unsigned)B) {
            lds_load_spinor<R>(lds, NB, B + ln, p);
            return R(1);
        }
    }
    load_spinor(static_cast<const SpT<R> *>(Q.in), P.S, n, p);
    return static_cast<R>(Q.s5_in);
}

// The eight links a site needs (U_nu(x) and U_nu(x - nu) for nu = 0..3, entry 2 nu + d),
// loaded once in their stored two-row form and shared by every right-hand side of the
// block (kRegs), or read from memory at each hop (kRegs false: L2 serves the repeats).
template <typename R, typename LT, bool kRegs>
struct SiteLinks {
    LT e[kRegs ? 8 : 1][kRegs ? 6 : 1];

    __device__ __forceinline__ void load(const StencilParams &P, int s, const int (&c)[4])
    {
        if constexpr (kRegs) {
            const LT *U = static_cast<const LT *>(P.links);
#pragma unroll
            for (int nu = 0; nu < 4; ++nu) {
                const int L = P.L[nu], st = P.stride[nu];
                const int nb = c[nu] == 0 ? s + (L - 1) * st : s - st;
                const LT *b = U + (size_t)nu * 6 * P.S;
                // temporal gauge: the unit time links are neither loaded nor used
                const bool fwd = !(nu == 3 && P.tgauge && c[3] != L - 1), bwd = !(nu == 3 && P.tgauge && c[3] != 0);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    if (fwd) e[2 * nu][k] = ld_off(b + (size_t)k * P.S, (uint32_t)s * (uint32_t)sizeof(LT));
                    if (bwd) e[2 * nu + 1][k] = ld_off(b + (size_t)k * P.S, (uint32_t)nb * (uint32_t)sizeof(LT));
                }
            }
        }
    }

    // link K = 2 nu + d as a full 3x3 matrix; n: the site it belongs to (s, or x - nu)
    template <int K>
    __device__ __forceinline__ void get(const StencilParams &P, int n, cpx<R> u[9]) const
    {
        if constexpr (kRegs) {
#pragma unroll
            for (int k = 0; k < 6; ++k) u[k] = to_cpx<R>(e[K][k]);
            su3_third_row(u);
        } else {
            load_link<R>(static_cast<const LT *>(P.links), P.S, P.link_ne, K / 2, n, u);
        }
    }
};

template <int NU, typename R, typename LT, bool kRegs>
__device__ __forceinline__ void hop_pair_staged(cpx<R> (&acc)[12], const StencilParams &P, const RhsParams &Q,
                                                const SpT<R> *lds, int base, int s, int coord,
                                                const SiteLinks<R, LT, kRegs> &lk)
{
    const int L = P.L[NU], st = P.stride[NU];
    const R kap = static_cast<R>(P.kappa);
    cpx<R> u[9];
    {
        const bool wrap = coord == L - 1;
        const int n = wrap ? s - (L - 1) * st : s + st;
        const R bcf = wrap ? static_cast<R>(P.bcf[NU]) : R(1);
        cpx<R> p[12], h[6], chi[6];
        const bool unit = NU == 3 && P.tgauge && !wrap;  // temporal gauge: U_t(x) = 1
        if (!unit) lk.template get<2 * NU>(P, s, u);
        const R s5 = fetch_neighbour<R>(Q, P, lds, base, n, p);
        project<NU, true>(p, h, s5);
        if (unit) {
#pragma unroll
            for (int k = 0; k < 6; ++k) chi[k] = h[k];
        } else {
            link_mul<false>(u, h, chi);
        }
        const R w = NU == 3 ? static_cast<R>(Q.wf_t) : R(1);
        accumulate<NU, true>(acc, chi, -kap * w * bcf);
    }
    pin(acc);
    {
        const bool wrap = coord == 0;
        const int n = wrap ? s + (L - 1) * st : s - st;
        const R bcb = wrap ? static_cast<R>(P.bcf[NU]) : R(1);
        cpx<R> p[12], h[6], chi[6];
        const bool unit = NU == 3 && P.tgauge && !wrap;  // temporal gauge: U_t(x - t) = 1
        if (!unit) lk.template get<2 * NU + 1>(P, n, u);
        const R s5 = fetch_neighbour<R>(Q, P, lds, base, n, p);
        project<NU, false>(p, h, s5);
        if (unit) {
#pragma unroll
            for (int k = 0; k < 6; ++k) chi[k] = h[k];
        } else {
            link_mul<true>(u, h, chi);
        }
        const R w = NU == 3 ? static_cast<R>(Q.wb_t) : R(1);
        accumulate<NU, false>(acc, chi, -kap * w * bcb);
    }
    pin(acc);
}

// One block: B sites for each right-hand side in turn (kMulti: right-hand sides r0 .. r1 - 1
// of P, all on P's lattice; else the single one, P.rhs[0]); the block's own spinors of
// the current right-hand side are staged in LDS.  The single form indexes P.rhs only with
// constants: P is then a kernel argument, and a runtime index into it would copy it to private
// memory.
template <typename R, typename LT, bool kEpi, bool kDot, bool kRegs, bool kMulti>
__device__ __forceinline__ void staged_body(const StencilParams &P, const int bx, const int r0 = 0, const int r1 = 1)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    SpT<R> *lds = reinterpret_cast<SpT<R> *>(smem_raw);
    if (bx >= P.nblk_sites) {  // padding of the component arrays: keep it zero
        const int s = P.V + (bx - P.nblk_sites) * (int)blockDim.x + (int)threadIdx.x;
        for (int r = r0; r < r1; ++r) {
            const RhsParams &Q = P.rhs[kMulti ? r : 0];
            if (s < P.S) {
                cpx<R> zero[12];
#pragma unroll
                for (int k = 0; k < 12; ++k) zero[k] = {R(0), R(0)};
                store_spinor(static_cast<SpT<R> *>(Q.out), P.S, s, zero);
            }
            if constexpr (kDot) {
                if (threadIdx.x == 0 && Q.w) {
                    if (Q.norm) {
                        Q.partials[2 * bx] = {0.0, 0.0};
                        Q.partials[2 * bx + 1] = {0.0, 0.0};
                    } else {
                        Q.partials[bx] = {0.0, 0.0};
                    }
                }
            }
        }
        return;
    }
    const int B = P.blk_sites, NB = B * P.tslices;
    int blk;
    if (P.sched_T > 0) {
        // XCD k owns the t-slab [k T, (k+1) T) of sched_R blocks per t-slice (per pair of
        // t-slices for bricks) and walks it in strips of W consecutive blocks with t fastest, so
        // the t-neighbours of a block run on the same XCD at about the same time
        const int W = SGN_STAGED_STRIP;
        const int k = bx % 8, j = bx / 8;
        const int per_strip = P.sched_T * W;
        const int strip = j / per_strip, rem = j - strip * per_strip;
        const int tl = rem / W, wi = rem - tl * W;
        blk = (k * P.sched_T + tl) * P.sched_R + strip * W + wi;
    } else {
        blk = SGN_XCD_REMAP ? xcd_block(bx, P.nblk_sites) : bx;
    }
    // first site of the block: B consecutive sites of one t-slice, for bricks the same B sites
    // of the next slice too (threads B.. 2B-1); blocks tile the V sites exactly
    int base;
    if (P.tslices == 2) {
        const int nreg = P.stride[3] / B, g = blk / nreg;
        base = 2 * g * P.stride[3] + (blk - g * nreg) * B;
    } else {
        base = blk * B;
    }
    const int i = threadIdx.x;
    const bool valid = i < NB;
    const int s = i < B ? base + i : base + P.stride[3] + (i - B);
    int c[4] = {0, 0, 0, 0};
    if (valid) {
        c[0] = s % P.L[0];
        int q = s / P.L[0];
        c[1] = q % P.L[1];
        q /= P.L[1];
        c[2] = q % P.L[2];
        c[3] = q / P.L[2];
    }
    SiteLinks<R, LT, kRegs> lk;
    if (valid) lk.load(P, s, c);
    for (int r = r0; r < r1; ++r) {
        const RhsParams &Q = P.rhs[kMulti ? r : 0];
        if (r > r0) __syncthreads();  // the previous right-hand side's LDS reads are done
        cpx<R> acc[12];
        if (valid) {
            load_spinor(static_cast<const SpT<R> *>(Q.in), P.S, s, acc);
            const R s5 = static_cast<R>(Q.s5_in);
#pragma unroll
            for (int k = 6; k < 12; ++k) acc[k] = s5 * acc[k];
            lds_store_spinor<R>(lds, NB, i, acc);
        }
        __syncthreads();
        double dr = 0.0, di = 0.0, dn = 0.0;
        if (valid) {
            hop_pair_staged<0, R, LT, kRegs>(acc, P, Q, lds, base, s, c[0], lk);
            hop_pair_staged<1, R, LT, kRegs>(acc, P, Q, lds, base, s, c[1], lk);
            hop_pair_staged<2, R, LT, kRegs>(acc, P, Q, lds, base, s, c[2], lk);
            hop_pair_staged<3, R, LT, kRegs>(acc, P, Q, lds, base, s, c[3], lk);
            finish_site<R, kEpi, kDot>(acc, Q, P.S, s, dr, di, dn);
        }
        if constexpr (kDot) {
            __shared__ double red[3 * 16];
            if (Q.w) {  // uniform
                double v[3] = {dr, di, dn};
                block_sum<3>(v, red);
                if (threadIdx.x == 0) {
                    if (Q.norm) {
                        Q.partials[2 * bx] = {v[0], v[1]};
                        Q.partials[2 * bx + 1] = {v[2], 0.0};
                    } else {
                        Q.partials[bx] = {v[0], v[1]};
                    }
                }
            }
        }
    }
}

// Waves per SIMD the compiler must allow the single-RHS staged kernel: with FP16 links 5 (at most 96
// VGPRs; the epilogue form spills a few bytes and still gains 3% inside the solves); otherwise what
// the largest block already implies (FP32 and FP64 lost time to spills when pushed further).
template <typename R, typename LT>
constexpr int kStagedWaves = std::is_same<LT, __half2>::value ? 5 : (sizeof(R) == 8 ? 2 : 3);

template <typename R, typename LT, bool kEpi, bool kDot>
__global__ void __launch_bounds__(kStagedMaxThreads<R>) __attribute__((amdgpu_waves_per_eu(kStagedWaves<R, LT>)))
    stencil_staged_kernel(StencilParams P)
{
    staged_body<R, LT, kEpi, kDot, false, false>(P, (int)blockIdx.x);
}

// Batched form: blockIdx.y selects one of several independent applications
// (own lattice, right-hand sides and epilogues) whose parameters live in device
// memory.  gridDim.x is a multiple of 8, so the XCD of block (x, y) is x mod 8 as
// in the single form.
template <typename R, typename LT, bool kEpi, bool kDot, bool kRegs>
__global__ void __launch_bounds__(kRegs ? kRegsMaxThreads : kStagedMaxThreads<R>)
    stencil_staged_batch(const StencilParams *__restrict__ plist)
{
    const StencilParams &P = plist[blockIdx.y];
    if ((int)blockIdx.x >= P.nblk_total) return;
    staged_body<R, LT, kEpi, kDot, kRegs, true>(P, (int)blockIdx.x, 0, P.nrhs);
}

// ---------------------------------------------------------------------------- split stencil
// Small lattices, where one thread per site leaves most of the chip idle and a launch is bound by the
// latency of one thread's 16 loads and 8 hops in sequence: 64 sites per block of eight wavefronts, one
// hop each (direction and sense are wave-uniform).  A wavefront loads its hop's neighbour spinor and
// link, all in flight at once, and leaves the transported half spinor in LDS; after the barrier six
// wavefronts take one pair of components of the 64 sites each, add the eight hops to the diagonal term in
// the order and with the operations of the staged kernel (so the result has the same bits) and run the
// epilogue.  Neighbours come through L2: no reuse inside the block.  One FP64 application on 8^4: 7.7 us as
// 16 staged blocks, 4.1 us here.
// The form for canonical fields is used at every size: on 24^3 x 48 it is 5-8% behind the staged kernel on internal
// fields (FP64 146 us against 135, FP32 61 against 58) and needs no pack and unpack passes (with them 267 and 130 us).
constexpr int kSplitSites = 64, kSplitThreads = 512;

// component pair C (components 2C, 2C + 1) of site s, internal layout
__device__ __forceinline__ void load_pair(const double2 *__restrict__ p, int S, int s, int C, cpx<double> v[2])
{
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const double2 t = ld_off(p + (size_t)(2 * C + q) * S, (uint32_t)s * 16u);
        v[q] = {t.x, t.y};
    }
}
__device__ __forceinline__ void load_pair(const float4 *__restrict__ p, int S, int s, int C, cpx<float> v[2])
{
    const float4 t = ld_off(p + (size_t)C * S, (uint32_t)s * 16u);
    v[0] = {t.x, t.y};
    v[1] = {t.z, t.w};
}
__device__ __forceinline__ void store_pair(double2 *__restrict__ p, int S, int s, int C, const cpx<double> v[2])
{
#pragma unroll
    for (int q = 0; q < 2; ++q) st_off(p + (size_t)(2 * C + q) * S, (uint32_t)s * 16u, make_double2(v[q].r, v[q].i));
}
__device__ __forceinline__ void store_pair(float4 *__restrict__ p, int S, int s, int C, const cpx<float> v[2])
{
    st_off(p + (size_t)C * S, (uint32_t)s * 16u, make_float4(v[0].r, v[0].i, v[1].r, v[1].i));
}

// Canonical fields hold a site's 12 components together (192 or 96 bytes).  A lane that loads its own site
// 16 bytes at a time makes every load of a wavefront touch 64 cache lines, and the address unit then takes 64
// cycles where the data would take 16.  So neighbouring lanes load consecutive 16-byte pieces of one site,
// for each of their sites in turn, and exchange the pieces in registers (DPP within four lanes): four lanes
// and 64-byte segments in FP64, two lanes and 32-byte segments in FP32.  Every lane must be active.
template <int CTRL>
__device__ __forceinline__ int dpp_quad(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E;               // lane ^ 1, lane ^ 2
constexpr int kPairFirst = 0xA0, kPairSecond = 0xF5;            // the even and the odd lane of each pair
typedef int piece __attribute__((ext_vector_type(4)));          // 16 bytes

// lanes with up = 0 keep a and receive the partner's a in b; lanes with up = 1 keep b and receive its b in a
template <int CTRL>
__device__ __forceinline__ void exchange(piece &a, piece &b, bool up)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int t = dpp_quad<CTRL>(up ? a[k] : b[k]);
        if (up) a[k] = t;
        else b[k] = t;
    }
}

__device__ __forceinline__ void load_site_canon(const double2 *__restrict__ p, int n, cpx<double> v[12])
{
    const int q = threadIdx.x & 3;
    const size_t n0 = (size_t)dpp_quad<0x00>(n) * 12 + q, n1 = (size_t)dpp_quad<0x55>(n) * 12 + q,
                 n2 = (size_t)dpp_quad<0xAA>(n) * 12 + q, n3 = (size_t)dpp_quad<0xFF>(n) * 12 + q;
    const piece *b = reinterpret_cast<const piece *>(p);
    piece a[12];
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        a[4 * g] = ld_off(b + n0 + 4 * g, 0u);
        a[4 * g + 1] = ld_off(b + n1 + 4 * g, 0u);
        a[4 * g + 2] = ld_off(b + n2 + 4 * g, 0u);
        a[4 * g + 3] = ld_off(b + n3 + 4 * g, 0u);
    }
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        piece *r = a + 4 * g;
        exchange<kQuadXor1>(r[0], r[1], q & 1);
        exchange<kQuadXor1>(r[2], r[3], q & 1);
        exchange<kQuadXor2>(r[0], r[2], q & 2);
        exchange<kQuadXor2>(r[1], r[3], q & 2);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[4 * g + c] = __builtin_bit_cast(cpx<double>, r[c]);
    }
}

__device__ __forceinline__ void split_piece(piece t, cpx<float> v[2])
{
    const float4 f = __builtin_bit_cast(float4, t);
    v[0] = {f.x, f.y};
    v[1] = {f.z, f.w};
}

__device__ __forceinline__ void load_site_canon(const float4 *__restrict__ p, int n, cpx<float> v[12])
{
    const int q = threadIdx.x & 1;
    const size_t n0 = (size_t)dpp_quad<kPairFirst>(n) * 6 + q, n1 = (size_t)dpp_quad<kPairSecond>(n) * 6 + q;
    const piece *b = reinterpret_cast<const piece *>(p);
    piece a[6];
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        a[2 * g] = ld_off(b + n0 + 2 * g, 0u);
        a[2 * g + 1] = ld_off(b + n1 + 2 * g, 0u);
    }
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        exchange<kQuadXor1>(a[2 * g], a[2 * g + 1], q);
        split_piece(a[2 * g], v + 4 * g);
        split_piece(a[2 * g + 1], v + 4 * g + 2);
    }
}

// component pair C of this lane's site s
__device__ __forceinline__ void load_pair_canon(const double2 *__restrict__ p, int s, int C, cpx<double> v[2])
{
    const int q = threadIdx.x & 1;
    const piece *b = reinterpret_cast<const piece *>(p) + 2 * C + q;
    piece a0 = ld_off(b + (size_t)dpp_quad<kPairFirst>(s) * 12, 0u);
    piece a1 = ld_off(b + (size_t)dpp_quad<kPairSecond>(s) * 12, 0u);
    exchange<kQuadXor1>(a0, a1, q);
    v[0] = __builtin_bit_cast(cpx<double>, a0);
    v[1] = __builtin_bit_cast(cpx<double>, a1);
}
__device__ __forceinline__ void load_pair_canon(const float4 *__restrict__ p, int s, int C, cpx<float> v[2])
{
    split_piece(ld_off(reinterpret_cast<const piece *>(p) + (size_t)s * 6 + C, 0u), v);
}

// neighbour of s in direction NU (forward or backward); wrap: the hop crosses the boundary
template <int NU, bool FWD>
__device__ __forceinline__ int hop_site(const StencilParams &P, int s, int coord, bool &wrap)
{
    const int L = P.L[NU], st = P.stride[NU];
    wrap = coord == (FWD ? L - 1 : 0);
    return FWD ? (wrap ? s - (L - 1) * st : s + st) : (wrap ? s + (L - 1) * st : s - st);
}

// chi = U (1 - gamma) psi(x + nu) or U^H (1 + gamma) psi(x - nu), the operations of hop_pair_staged
template <int NU, bool FWD, bool kCanon, typename R, typename LT>
__device__ __forceinline__ void split_hop(const StencilParams &P, const RhsParams &Q, int s, int coord, cpx<R> chi[6])
{
    bool wrap;
    const int n = hop_site<NU, FWD>(P, s, coord, wrap);
    const bool unit = NU == 3 && P.tgauge && !wrap;
    cpx<R> u[9], p[12], h[6];
    if (!unit) load_link<R>(static_cast<const LT *>(P.links), P.S, P.link_ne, NU, FWD ? s : n, u);
    if constexpr (kCanon) load_site_canon(static_cast<const SpT<R> *>(Q.in), n, p);
    else load_spinor(static_cast<const SpT<R> *>(Q.in), P.S, n, p);
    project<NU, FWD>(p, h, static_cast<R>(Q.s5_in));
    if (unit) {
#pragma unroll
        for (int k = 0; k < 6; ++k) chi[k] = h[k];
    } else {
        link_mul<!FWD>(u, h, chi);
    }
}

// what component (spin SP, colour c) takes from a hop: the half spinor's row and phase, as in accumulate()
template <int NU, bool FWD, int SP>
struct HopRow {
    static constexpr int row = SP < 2 ? SP : (NU < 2 ? 3 - SP : SP - 2);
    static constexpr int phase = SP < 2    ? kP1
                                 : NU == 0 ? (FWD ? kPI : kMI)
                                 : NU == 1 ? ((SP == 2) == FWD ? kM1 : kP1)
                                 : NU == 2 ? ((SP == 2) == FWD ? kPI : kMI)
                                           : (FWD ? kM1 : kP1);
};

template <int NU, int C, typename R>
__device__ __forceinline__ void split_add(cpx<R> (&acc)[2], const StencilParams &P, const RhsParams &Q, int coord,
                                          const cpx<R> *chi /* [hop][6][kSplitSites], at this site */)
{
    const R kap = static_cast<R>(P.kappa);
    const R bf = coord == P.L[NU] - 1 ? static_cast<R>(P.bcf[NU]) : R(1);
    const R bb = coord == 0 ? static_cast<R>(P.bcf[NU]) : R(1);
    const R wf = NU == 3 ? static_cast<R>(Q.wf_t) : R(1), wb = NU == 3 ? static_cast<R>(Q.wb_t) : R(1);
    const cpx<R> *f = chi + (2 * NU) * 6 * kSplitSites, *b = f + 6 * kSplitSites;
    constexpr int S0 = (2 * C) / 3, c0 = (2 * C) % 3, S1 = (2 * C + 1) / 3, c1 = (2 * C + 1) % 3;
    using F0 = HopRow<NU, true, S0>;
    using F1 = HopRow<NU, true, S1>;
    using B0 = HopRow<NU, false, S0>;
    using B1 = HopRow<NU, false, S1>;
    acc[0] = add_ph<F0::phase>(acc[0], -kap * wf * bf, f[(3 * F0::row + c0) * kSplitSites]);
    acc[1] = add_ph<F1::phase>(acc[1], -kap * wf * bf, f[(3 * F1::row + c1) * kSplitSites]);
    acc[0] = add_ph<B0::phase>(acc[0], -kap * wb * bb, b[(3 * B0::row + c0) * kSplitSites]);
    acc[1] = add_ph<B1::phase>(acc[1], -kap * wb * bb, b[(3 * B1::row + c1) * kSplitSites]);
}

// acc (the diagonal term's pair C, gamma5 of the input not yet applied) += the eight hops, in the staged
// kernel's order
template <int C, typename R>
__device__ __forceinline__ void split_sum(cpx<R> (&acc)[2], const StencilParams &P, const RhsParams &Q,
                                          const int (&c)[4], const cpx<R> *chi)
{
    if constexpr (C >= 3) {
        const R s5 = static_cast<R>(Q.s5_in);
        acc[0] = s5 * acc[0];
        acc[1] = s5 * acc[1];
    }
    split_add<0, C, R>(acc, P, Q, c[0], chi);
    split_add<1, C, R>(acc, P, Q, c[1], chi);
    split_add<2, C, R>(acc, P, Q, c[2], chi);
    split_add<3, C, R>(acc, P, Q, c[3], chi);
}

template <typename R, typename LT, bool kEpi, bool kDot, bool kCanon, bool kMulti>
__device__ __forceinline__ void split_body(const StencilParams &P, const int bx, const int r0 = 0, const int r1 = 1)
{
    if (bx >= P.nblk_sites) {  // padding of the component arrays (internal layout): keep it zero
        const int s = P.V + (bx - P.nblk_sites) * kSplitThreads + (int)threadIdx.x;
        for (int r = r0; r < r1; ++r) {
            const RhsParams &Q = P.rhs[kMulti ? r : 0];
            if (s < P.S) {
                cpx<R> zero[12];
#pragma unroll
                for (int k = 0; k < 12; ++k) zero[k] = {R(0), R(0)};
                store_spinor(static_cast<SpT<R> *>(Q.out), P.S, s, zero);
            }
        }
        return;
    }
    __shared__ __align__(16) cpx<R> chi_lds[8 * 6 * kSplitSites];
    __shared__ __align__(16) cpx<R> out_lds[kCanon || kDot ? 13 * kSplitSites : 1];  // rows of 12, padded by one
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    // block bx0 of the launch; with a dot product one wavefront `part` of the staged kernel's block bx0 (on the
    // same XCD)
    int bx0 = bx, part = 0, sites = kSplitSites, nblk = P.nblk_sites, stride = kSplitSites;
    if (kDot && P.grp_waves > 0) {
        bx0 = bx / (8 * P.grp_waves) * 8 + bx % 8;
        part = bx / 8 % P.grp_waves;
        nblk = P.grp_n;
        stride = P.grp_sites;
        sites = min(kSplitSites, P.grp_sites - part * kSplitSites);
        if (bx0 >= nblk) return;  // uniform
    }
    int blk;
    if (P.sched_T > 0) {  // t fastest inside each XCD's t-slab (as the staged kernel)
        const int k = bx0 % 8, j = bx0 / 8;
        blk = (k * P.sched_T + j % P.sched_T) * P.sched_R + j / P.sched_T;
    } else {
        blk = xcd_block(bx0, nblk);
    }
    // lanes past the last site work on it too (the register exchanges of the canonical form need every
    // lane) and store nothing
    const int s0 = blk * stride + part * kSplitSites, s = min(s0 + lane, P.V - 1);
    const bool valid = lane < sites && s0 + lane < P.V;
    int c[4];
    {
        c[0] = s % P.L[0];
        int q = s / P.L[0];
        c[1] = q % P.L[1];
        q /= P.L[1];
        c[2] = q % P.L[2];
        c[3] = q / P.L[2];
    }
    for (int r = r0; r < r1; ++r) {
        const RhsParams &Q = P.rhs[kMulti ? r : 0];
        if (r > r0) __syncthreads();  // the previous right-hand side's LDS reads are done
        const bool mine = wave < 6;  // this wavefront finishes component pair `wave`
        // wavefront 7 takes the dot product: the 12 components of its sites in order, as the staged kernel does
        const bool dots = kDot && wave == 7;
        cpx<R> acc[2] = {{R(0), R(0)}, {R(0), R(0)}}, zz[2], ww[kDot ? 12 : 1];
        // the operands of the second part: in flight during the hops, or, where the registers do not hold them
        // as well, from the end of the hop on
        if (mine) {
            if constexpr (kCanon) load_pair_canon(static_cast<const SpT<R> *>(Q.in), s, wave, acc);
            else load_pair(static_cast<const SpT<R> *>(Q.in), P.S, s, wave, acc);
            if (kEpi && sizeof(R) == 4 && Q.z) load_pair(static_cast<const SpT<R> *>(Q.z), P.S, s, wave, zz);
        }
        {
            cpx<R> chi[6];
            switch (wave) {
            case 0: split_hop<0, true, kCanon, R, LT>(P, Q, s, c[0], chi); break;
            case 1: split_hop<0, false, kCanon, R, LT>(P, Q, s, c[0], chi); break;
            case 2: split_hop<1, true, kCanon, R, LT>(P, Q, s, c[1], chi); break;
            case 3: split_hop<1, false, kCanon, R, LT>(P, Q, s, c[1], chi); break;
            case 4: split_hop<2, true, kCanon, R, LT>(P, Q, s, c[2], chi); break;
            case 5: split_hop<2, false, kCanon, R, LT>(P, Q, s, c[2], chi); break;
            case 6: split_hop<3, true, kCanon, R, LT>(P, Q, s, c[3], chi); break;
            default: split_hop<3, false, kCanon, R, LT>(P, Q, s, c[3], chi); break;
            }
#pragma unroll
            for (int k = 0; k < 6; ++k) chi_lds[(wave * 6 + k) * kSplitSites + lane] = chi[k];
            if constexpr (kEpi || kDot) asm volatile("" ::: "memory");  // not during the hops: they would spill
            if (kEpi && sizeof(R) == 8 && mine && Q.z) load_pair(static_cast<const SpT<R> *>(Q.z), P.S, s, wave, zz);
            if constexpr (kDot) {
                if (dots && Q.w) load_spinor(static_cast<const SpT<R> *>(Q.w), P.S, s, ww);
            }
        }
        __syncthreads();
        if (mine) {
            const cpx<R> *chi = chi_lds + lane;
            switch (wave) {
            case 0: split_sum<0, R>(acc, P, Q, c, chi); break;
            case 1: split_sum<1, R>(acc, P, Q, c, chi); break;
            case 2: split_sum<2, R>(acc, P, Q, c, chi); break;
            case 3: split_sum<3, R>(acc, P, Q, c, chi); break;
            case 4: split_sum<4, R>(acc, P, Q, c, chi); break;
            default: split_sum<5, R>(acc, P, Q, c, chi); break;
            }
            // gamma5 of the result (components 6..11) and the epilogue, as in finish_site
            const R s5o = wave < 3 ? R(1) : static_cast<R>(Q.s5_out);
            if constexpr (!kEpi) {
                acc[0] = s5o * acc[0];
                acc[1] = s5o * acc[1];
            } else {
                if (Q.in_scale) {
                    const z64 t = *Q.in_scale;
                    const cpx<R> sc = {static_cast<R>(Q.a * t.r), static_cast<R>(Q.a * t.i)};
                    const cpx<R> sl = {s5o * sc.r, s5o * sc.i};
#pragma unroll
                    for (int k = 0; k < 2; ++k) acc[k] = cmul_f<false>(sl, acc[k]);
                } else {
                    const R a = s5o * static_cast<R>(Q.a);
#pragma unroll
                    for (int k = 0; k < 2; ++k) acc[k] = a * acc[k];
                }
                if (Q.z) {
                    if (!Q.b_dev && Q.b.i == 0.0) {
                        const R b = static_cast<R>(Q.b.r);
#pragma unroll
                        for (int k = 0; k < 2; ++k) acc[k] = add_ph<kP1>(acc[k], b, zz[k]);
                    } else {
                        z64 bb = Q.b;
                        if (Q.b_dev) {
                            const z64 t = *Q.b_dev;
                            bb = {bb.r * t.r - bb.i * t.i, bb.r * t.i + bb.i * t.r};
                        }
                        const cpx<R> b = {static_cast<R>(bb.r), static_cast<R>(bb.i)};
#pragma unroll
                        for (int k = 0; k < 2; ++k) cmac_f<false>(acc[k], b, zz[k]);
                    }
                }
            }
            if constexpr (kCanon || kDot) {
                out_lds[lane * 13 + 2 * wave] = acc[0];
                out_lds[lane * 13 + 2 * wave + 1] = acc[1];
            }
            if (!kCanon && valid) store_pair(static_cast<SpT<R> *>(Q.out), P.S, s, wave, acc);
        }
        if constexpr (kCanon) {
            // the block's sites are one contiguous piece of the canonical output: written in order
            __syncthreads();
            const int n = min(kSplitSites, P.V - s0) * 12;
            SGN_GLOBAL cpx<R> *o = (SGN_GLOBAL cpx<R> *)Q.out + (size_t)s0 * 12;
            for (int e = threadIdx.x; e < n; e += kSplitThreads) o[e] = out_lds[e / 12 * 13 + e % 12];
        }
        if constexpr (kDot) {
            __syncthreads();
            if (dots && Q.w) {
                double v[3] = {0.0, 0.0, 0.0};
                if (valid) {
#pragma unroll
                    for (int k = 0; k < 12; ++k) dot_terms<R>(ww[k], out_lds[lane * 13 + k], v[0], v[1], v[2]);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) v[k] = wave_sum(v[k]);
                if (lane == 0) {
                    const int e = bx0 * P.grp_waves + part;
                    if (Q.norm) {
                        Q.partials[2 * e] = {v[0], v[1]};
                        Q.partials[2 * e + 1] = {v[2], 0.0};
                    } else {
                        Q.partials[e] = {v[0], v[1]};
                    }
                }
            }
        }
    }
}

// Four waves per SIMD, i.e. two blocks per CU, for FP64 too (128 VGPRs); the batched FP64 epilogues would spill
// there (up to 116 registers) and get two.
template <typename R, bool kEpi, bool kMulti>
constexpr int kSplitWaves = sizeof(R) == 8 && kEpi && kMulti ? 2 : 4;

template <typename R, typename LT, bool kEpi, bool kDot, bool kCanon>
__global__ void __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(kSplitWaves<R, kEpi, false>)))
    stencil_split_kernel(StencilParams P)
{
    split_body<R, LT, kEpi, kDot, kCanon, false>(P, (int)blockIdx.x);
}

template <typename R, typename LT, bool kEpi, bool kDot>
__global__ void __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(kSplitWaves<R, kEpi, true>)))
    stencil_split_batch(const StencilParams *__restrict__ plist)
{
    const StencilParams &P = plist[blockIdx.y];
    if ((int)blockIdx.x >= P.nblk_total) return;
    split_body<R, LT, kEpi, kDot, false, true>(P, (int)blockIdx.x, 0, P.nrhs);
}

// Several right-hand sides on one lattice without an epilogue, the parameters as a kernel argument: blockIdx.y
// takes `per` of the P.nrhs right-hand sides.  P is read through the kernel-argument segment, because a
// run-time index into a by-value argument would copy it to private memory.  With the parameters in device memory
// each call with other fields than the last cost a wait for the device and a copy (8^4, 2 right-hand sides, fields
// swapped between calls: 34 us a call, now 15; 16^3 x 32 FP16, 12: 128, now 91).
#if defined(__HIP_DEVICE_COMPILE__)
#define SGN_KERNARG(P) (*(const StencilParams *)__builtin_amdgcn_kernarg_segment_ptr())
#else
#define SGN_KERNARG(P) (P)
#endif
template <typename R, typename LT, bool kRegs>
__global__ void __launch_bounds__(kRegs ? kRegsMaxThreads : kStagedMaxThreads<R>)
    stencil_staged_multi(StencilParams P, int per)
{
    const StencilParams &A = SGN_KERNARG(P);
    if ((int)blockIdx.x >= A.nblk_total) return;
    staged_body<R, LT, false, false, kRegs, true>(A, (int)blockIdx.x, (int)blockIdx.y * per,
                                                  min(A.nrhs, ((int)blockIdx.y + 1) * per));
}
template <typename R, typename LT>
__global__ void __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(kSplitWaves<R, false, true>)))
    stencil_split_multi(StencilParams P, int per)
{
    const StencilParams &A = SGN_KERNARG(P);
    if ((int)blockIdx.x >= A.nblk_total) return;
    split_body<R, LT, false, false, false, true>(A, (int)blockIdx.x, (int)blockIdx.y * per,
                                                 min(A.nrhs, ((int)blockIdx.y + 1) * per));
}
// Two right-hand sides, one per blockIdx.y, with epilogues (a dot product only where w is set).  A small lattice
// leaves the chip short of blocks and each launch costs more than its work: 8^4 FP64, A v with its dot product and
// A^H w, 6.2 + 5.0 us as two launches, 6.9 as one.
template <typename R, typename LT, bool kEpi, bool kDot>
__global__ void __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(kSplitWaves<R, kEpi, false>)))
    stencil_split_pair(StencilParams P)
{
    const StencilParams &A = SGN_KERNARG(P);
    split_body<R, LT, kEpi, kDot, false, true>(A, (int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.y + 1);
}
static_assert(offsetof(StencilParams, links) == 0 && sizeof(StencilParams) + 64 <= 4096,
              "the first kernel argument, within the argument segment");

template <typename R, typename LT>
void launch_multi_kernarg(const StencilParams &P, int nblk, int threads, size_t lds, int per, bool split, bool regs,
                          hipStream_t s, const LaunchStamp &ev)
{
    const dim3 g((nblk + 7) / 8 * 8, (P.nrhs + per - 1) / per);
    if (split) {
        launch_k(ev, stencil_split_multi<R, LT>, g, dim3(kSplitThreads), 0u, s, P, per);
        return;
    }
    if constexpr (std::is_same<LT, __half2>::value) {
        if (regs) {
            launch_k(ev, stencil_staged_multi<R, LT, true>, g, dim3(threads), (uint32_t)lds, s, P, per);
            return;
        }
    }
    launch_k(ev, stencil_staged_multi<R, LT, false>, g, dim3(threads), (uint32_t)lds, s, P, per);
}

template <typename R, typename LT>
void launch_split(const StencilParams &P, int nblk, bool epi, bool dot, bool canon, hipStream_t s,
                  const LaunchStamp &ev)
{
    dim3 g(nblk), b(kSplitThreads);
    if (canon)  // no padding sites in the canonical layout
        launch_k(ev, stencil_split_kernel<R, LT, false, false, true>, dim3(P.nblk_sites), b, 0u, s, P);
    else if (dot)
        launch_k(ev, stencil_split_kernel<R, LT, true, true, false>, g, b, 0u, s, P);
    else if (epi)
        launch_k(ev, stencil_split_kernel<R, LT, true, false, false>, g, b, 0u, s, P);
    else
        launch_k(ev, stencil_split_kernel<R, LT, false, false, false>, g, b, 0u, s, P);
}

template <typename R, typename LT>
void launch_staged(const StencilParams &P, int nblk, int threads, size_t lds, bool epi, bool dot, hipStream_t s,
                   const LaunchStamp &ev)
{
    dim3 g(nblk), b(threads);
    if (dot)
        launch_k(ev, stencil_staged_kernel<R, LT, true, true>, g, b, (uint32_t)lds, s, P);
    else if (epi)
        launch_k(ev, stencil_staged_kernel<R, LT, true, false>, g, b, (uint32_t)lds, s, P);
    else
        launch_k(ev, stencil_staged_kernel<R, LT, false, false>, g, b, (uint32_t)lds, s, P);
}

template <typename R, typename LT, int NR>
void launch_typed(const StencilParams &P, int nblk, bool epi, bool dot, hipStream_t s, const LaunchStamp &ev)
{
    dim3 g(nblk), b(SGN_STENCIL_THREADS);
    if (dot)
        launch_k(ev, stencil_kernel<R, LT, NR, true, true>, g, b, 0u, s, P);
    else if (epi)
        launch_k(ev, stencil_kernel<R, LT, NR, true, false>, g, b, 0u, s, P);
    else
        launch_k(ev, stencil_kernel<R, LT, NR, false, false>, g, b, 0u, s, P);
}

// unstaged kernel (lattices too small for a staged block shape): one launch per right-hand side;
// a stamp is only taken for one right-hand side (one launch)
template <typename R, typename LT>
void launch_nr(const StencilParams &P, int nr, int nblk, bool epi, bool dot, hipStream_t s, const LaunchStamp &ev)
{
    if (nr == 1) {
        launch_typed<R, LT, 1>(P, nblk, epi, dot, s, ev);
        return;
    }
    for (int r = 0; r < nr; ++r) {
        StencilParams Q = P;
        Q.rhs[0] = P.rhs[r];
        Q.nrhs = 1;
        launch_typed<R, LT, 1>(Q, nblk, epi, dot, s, LaunchStamp{});
    }
}

}  // namespace

namespace {

// Block shape of the staged kernel: B sites of whole x-rows (whole x-y planes
// when they fit the LDS budget), B dividing V; not used when B < 64.
struct StagedPlan {
    bool ok = false;
    int B = 0, T = 1, threads = 0, nblk_sites = 0, nblk = 0;  // B sites per t-slice, T slices per block
    size_t lds = 0;
};

// max_threads > 0 caps the block (the register-link multi-RHS form), max_sites > 0 the sites of
// a block (a tuned shape); tslices = 2 asks for bricks of two t-slices (even L_t; B then divides
// one slice, so a brick never straddles a time boundary)
StagedPlan staged_plan(const Lattice &lat, sgn_prec p, int max_threads = 0, int max_sites = 0, int tslices = 1)
{
    StagedPlan pl;
    if (!SGN_STENCIL_LDS) return pl;
    const int T = tslices == 2 ? 2 : 1;
    if (T == 2 && lat.L[3] % 2) return pl;
    const int64_t site_bytes = p == SGN_PREC_F64 ? 192 : 96;
    int64_t tmax = p == SGN_PREC_F64 ? kStagedMaxThreads<double> : kStagedMaxThreads<float>;
    if (max_threads > 0) tmax = std::min<int64_t>(tmax, max_threads);
    if (max_sites > 0) tmax = std::min<int64_t>(tmax, max_sites);
    const int64_t bmax = std::min<int64_t>(tmax, SGN_LDS_MAXBYTES / site_bytes) / T;
    const int64_t Lx = lat.L[0], A = (int64_t)lat.L[0] * lat.L[1];
    const int64_t nplane = (int64_t)lat.L[2] * (T == 2 ? 1 : lat.L[3]);
    int64_t B = 0;
    if (A <= bmax) {
        int64_t P = bmax / A;
        while (nplane % P) --P;
        B = P * A;
    } else {
        int64_t rows = bmax / Lx;
        const int64_t nrows = (int64_t)lat.L[1] * nplane;
        while (rows > 0 && nrows % rows) --rows;
        B = rows * Lx;
    }
    if (B * T < 64) return pl;
    pl.ok = true;
    pl.B = (int)B;
    pl.T = T;
    pl.threads = (int)((B * T + 63) / 64 * 64);
    pl.nblk_sites = (int)(lat.V / (B * T));
    const int64_t pad = lat.S > lat.V ? (lat.S - lat.V + pl.threads - 1) / pl.threads : 0;
    pl.nblk = pl.nblk_sites + (int)pad;
    pl.lds = (size_t)B * T * site_bytes;
    return pl;
}

}  // namespace

// An upper bound of the partial sums of any dotting stencil launch on lat, whatever shape is chosen (tuned or
// default): one per block, every staged block holds at least 64 sites, the unstaged kernel 256, and the padding
// sites [V, S) take blocks of at least 64 threads; the split kernel leaves one per wavefront of such a block,
// at most two per 64 sites.
int dslash_blocks(const Lattice &lat)
{
    const int64_t valid = 2 * ((lat.V + 63) / 64) + 4;
    const int64_t pad = lat.S > lat.V ? (lat.S - lat.V + 63) / 64 : 0;
    return (int)(valid + pad);
}

namespace {

// Internal fields up to this size take the split kernel unless a staged shape was tuned or pinned for their
// lattice (49152 FP64 or 98304 FP32 sites): beyond it the chip is full either way and the staged kernel's
// reuse of neighbours wins.  One application of many in a row, split / default staged / best staged shape, us:
// FP64 4^4 3.8 / 6.9 / 6.4, 8^4 4.1 / 7.7 / 6.8, 12^4 5.8 / 10.2 / 8.0, 40320 sites 9.3 / 11.7 / 9.5, 49152
// 10.5 / 10.9 / 10.9, 16^4 13.1 / 12.6 / 12.6, 70200 15.5 / 14.6 / 14.3; FP32 8^4 3.5 / 7.4 / 6.4, 16^4
// 7.8 / 9.1 / 8.4, 70200 8.3 / 10.3 / 8.9, 98304 9.9 / 9.7 / 9.7, 16^3 x 32 13.0 / 10.6 / 10.6 (FP16 links as FP32).
constexpr int64_t kSplitMaxBytes = 9 << 20;

// nr fields of the lattice together
bool split_takes(const Lattice &lat, sgn_prec p, int nr)
{
    return nr * lat.V * (p == SGN_PREC_F64 ? 192 : 96) <= kSplitMaxBytes;
}

bool split_fits(const Lattice &lat, sgn_prec p) { return split_takes(lat, p, 1); }

bool use_split(const Lattice &lat, sgn_prec p, bool multi)
{
    if (!split_fits(lat, p)) return false;
    auto it = lat.ctx->tuned.find({lat.L[0], lat.L[1], lat.L[2], lat.L[3], (int)p, multi ? 1 : 0});
    return it == lat.ctx->tuned.end() || it->second.unstaged;
}

// The staged shape set for a lattice.  Where the split kernel serves the lattice's own applications, `unstaged`
// stands for that kernel and says nothing about launches of more fields than it takes: the default shape there,
// so that they stay one launch.  Without it each took a launch of its own: on tuned lattices 32 FP64 solves on 8^4 in
// one call 76.6 ms, now 30.5 (untuned 30.6); 16 FP32 right-hand sides on 12^4 95 us, now 46.
Context::TunedShape staged_shape(const Lattice &lat, sgn_prec p, bool multi)
{
    Context::TunedShape ts = lat.ctx->tuned_shape(lat.L, p, multi);
    if (ts.unstaged && split_fits(lat, p)) ts.unstaged = ts.max_sites = 0, ts.tslices = 1;
    return ts;
}

// whether a staged shape (or the unstaged kernel on a large lattice) was set for the multi-RHS form
bool multi_shape_set(const Lattice &lat, sgn_prec p)
{
    return lat.ctx->tuned.count({lat.L[0], lat.L[1], lat.L[2], lat.L[3], (int)p, 1}) && !use_split(lat, p, true);
}

// Everything about one stencil application except the launch itself.
struct PreparedStencil {
    StencilParams P{};
    StagedPlan pl;
    bool split = false;  // the split kernel (pl is then not used)
    int nblk = 0;       // blocks of the launch
    int partials = 0;   // partials written when dotting (packed)
    double bytes = 0.0;         // algorithmic bytes (links as nine entries) and flops
    double flops = 0.0;
    double bytes_stored = 0.0;  // bytes in the stored format (two-row links where the lattice keeps them)
    bool epi = false, dot = false;
};

enum KernelPick { kAuto, kStaged, kSplit };

bool has_epilogue(const Epilogue &e) { return e.w || e.z || e.a != 1.0 || e.in_scale; }

// max_threads > 0 caps the staged block (the register-link multi-RHS form)
PreparedStencil prepare_stencil(const Lattice &lat, sgn_prec p, int nr, const OpSpec *op, const void *const *in,
                                void *const *out, const Epilogue *ep, int max_threads = 0, KernelPick pick = kAuto)
{
    if (nr < 1 || nr > kMaxRhs) throw Failure{SGN_ERR_INVALID, "stencil: 1..16 right-hand sides per launch"};
    PreparedStencil ps;
    StencilParams &P = ps.P;
    P.V = (int)lat.V;
    P.S = (int)lat.S;
    for (int d = 0; d < 4; ++d) {
        P.L[d] = lat.L[d];
        P.bcf[d] = (float)lat.bc[d];
    }
    P.stride[0] = 1;
    P.stride[1] = lat.L[0];
    P.stride[2] = lat.L[0] * lat.L[1];
    P.stride[3] = lat.L[0] * lat.L[1] * lat.L[2];
    P.kappa = lat.kappa;
    double extra_bytes = 0.0, extra_flops = 0.0;
    const double sb = (p == SGN_PREC_F64) ? 192.0 : 96.0;
    for (int r = 0; r < nr; ++r) {
        RhsParams &Q = P.rhs[r];
        Q.in = in[r];
        Q.out = out[r];
        Q.wf_t = std::exp(-op[r].mu);
        Q.wb_t = std::exp(op[r].mu);
        Q.s5_in = op[r].g5_in ? -1.f : 1.f;
        Q.s5_out = op[r].g5_out ? -1.f : 1.f;
        Q.a = ep[r].a;
        Q.b = ep[r].b;
        Q.b_dev = ep[r].b_dev;
        Q.z = ep[r].z;
        Q.w = ep[r].w;
        Q.partials = ep[r].partials;
        Q.in_scale = ep[r].in_scale;
        Q.norm = ep[r].norm ? 1 : 0;
        if (ep[r].w && !ep[r].partials) throw Failure{SGN_ERR_INVALID, "stencil dot without partial buffer"};
        ps.dot = ps.dot || ep[r].w != nullptr;
        ps.epi = ps.epi || has_epilogue(ep[r]);
        // an epilogue operand counts once: a dot partner equal to z is not read again
        extra_bytes += (ep[r].z ? sb : 0.0) + (ep[r].w && ep[r].w != ep[r].z ? sb : 0.0);
        extra_flops += (ep[r].z ? 96.0 : 0.0) + (ep[r].w ? 96.0 : 0.0) + 24.0;
    }
    {
        const int64_t t = SGN_STENCIL_THREADS;
        ps.nblk = (int)((lat.V + t - 1) / t + (lat.S > lat.V ? (lat.S - lat.V + t - 1) / t : 0));
    }
    P.nblk_sites = (int)((lat.V + SGN_STENCIL_THREADS - 1) / SGN_STENCIL_THREADS);
    {
        const int64_t vxyz = (int64_t)lat.L[0] * lat.L[1] * lat.L[2];
        P.sched_T = P.sched_R = 0;
        if (SGN_T_MINOR && vxyz % SGN_STENCIL_THREADS == 0 && lat.L[3] % 8 == 0) {
            P.sched_T = lat.L[3] / 8;
            P.sched_R = (int)(vxyz / SGN_STENCIL_THREADS);
            if ((int64_t)8 * P.sched_T * P.sched_R != P.nblk_sites) P.sched_T = P.sched_R = 0;
        }
    }
    // algorithmic bytes: every input and output spinor once, the 4 links of each
    // site once (shared by the right-hand sides) as nine complex entries, plus the
    // epilogue operands; 1368 flop per site and right-hand side for the stencil itself
    P.link_ne = lat.link_ne;
    P.tgauge = 0;
    const double eb = (p == SGN_PREC_F64) ? 16.0 : (p == SGN_PREC_F32 ? 8.0 : 4.0);
    ps.bytes = (2 * sb * nr + 4 * 9 * eb + extra_bytes) * lat.V;
    ps.bytes_stored = (2 * sb * nr + 4 * lat.link_ne * eb + extra_bytes) * lat.V;
    ps.flops = (1368.0 * nr + extra_flops) * lat.V;
    P.nrhs = nr;
    P.tslices = 1;
    ps.split = pick == kSplit || (pick == kAuto && use_split(lat, p, nr > 1));
    P.grp_sites = P.grp_waves = P.grp_n = 0;
    if (ps.split && ps.dot) {
        // the blocks and wavefronts whose sums the staged kernel (or without a staged shape the unstaged one)
        // would leave, in its block order: the dot products of a solve do not depend on the kernel
        const StagedPlan pl = staged_plan(lat, p, max_threads);
        const int64_t v3 = (int64_t)lat.L[0] * lat.L[1] * lat.L[2];
        P.grp_sites = pl.ok ? pl.B : SGN_STENCIL_THREADS;
        P.grp_waves = (P.grp_sites + kSplitSites - 1) / kSplitSites;
        P.grp_n = (int)((lat.V + P.grp_sites - 1) / P.grp_sites);
        P.sched_T = P.sched_R = 0;
        if (v3 % P.grp_sites == 0 && lat.L[3] % 8 == 0) {
            P.sched_T = lat.L[3] / 8;
            P.sched_R = (int)(v3 / P.grp_sites);
        }
        P.nblk_sites = (P.grp_n + 7) / 8 * 8 * P.grp_waves;
        ps.nblk = P.nblk_sites + (int)((lat.S - lat.V + kSplitThreads - 1) / kSplitThreads);
        ps.partials = pack_partials(P.grp_n, P.grp_waves);
    } else if (ps.split) {
        P.sched_T = P.sched_R = 0;
        const int64_t v3 = (int64_t)lat.L[0] * lat.L[1] * lat.L[2];
        if (v3 % kSplitSites == 0 && lat.L[3] % 8 == 0) {
            P.sched_T = lat.L[3] / 8;
            P.sched_R = (int)(v3 / kSplitSites);
        }
        P.nblk_sites = (int)((lat.V + kSplitSites - 1) / kSplitSites);
        ps.nblk = P.nblk_sites + (int)((lat.S - lat.V + kSplitThreads - 1) / kSplitThreads);
    } else {
        const Context::TunedShape ts = staged_shape(lat, p, nr > 1);
        if (!ts.unstaged) {
            ps.pl = staged_plan(lat, p, max_threads, ts.max_sites, ts.tslices);
            if (!ps.pl.ok && ts.tslices == 2) ps.pl = staged_plan(lat, p, max_threads, ts.max_sites, 1);
        }
    }
    if (ps.pl.ok) {
        P.blk_sites = ps.pl.B;
        P.tslices = ps.pl.T;
        P.nblk_sites = ps.pl.nblk_sites;
        ps.nblk = ps.pl.nblk;
        P.sched_T = P.sched_R = 0;
        const int64_t v3 = (int64_t)lat.L[0] * lat.L[1] * lat.L[2];
        const int tg = lat.L[3] / ps.pl.T;  // t-slices, or pairs of them for bricks
        if (SGN_STAGED_STRIP > 0 && v3 % ps.pl.B == 0 && tg % 8 == 0 && (v3 / ps.pl.B) % SGN_STAGED_STRIP == 0) {
            P.sched_T = tg / 8;
            P.sched_R = (int)(v3 / ps.pl.B);
        }
    }
    P.nblk_total = ps.nblk;
    if (!ps.partials) ps.partials = pack_partials(ps.nblk, 1);
    if (lat.gauge && (ps.pl.ok || ps.split)) {  // these kernels read the time links of the last slice only
        P.tgauge = 1;
        ps.bytes_stored -= (1.0 - 1.0 / lat.L[3]) * lat.link_ne * ((p == SGN_PREC_F64) ? 16.0 : (p == SGN_PREC_F32 ? 8.0 : 4.0)) * lat.V;
    }
    switch (p) {
    case SGN_PREC_F64: P.links = lat.links64; break;
    case SGN_PREC_F32: P.links = lat.links32; break;
    case SGN_PREC_F32_H16: P.links = lat.links16; break;
    default: throw Failure{SGN_ERR_INVALID, "unknown precision"};
    }
    if (!P.links)
        throw Failure{SGN_ERR_INVALID, p == SGN_PREC_F64 ? "lattice has no FP64 links"
                                                         : (p == SGN_PREC_F32 ? "lattice has no FP32 links"
                                                                              : "lattice has no FP16 links")};
    return ps;
}

int kclass(sgn_prec p)
{
    return p == SGN_PREC_F64 ? SGN_K_STENCIL_F64 : (p == SGN_PREC_F32 ? SGN_K_STENCIL_F32 : SGN_K_STENCIL_H16);
}

template <typename R, typename LT, bool kRegs>
void launch_staged_batch_r(const StencilParams *dev, int count, int gx, int threads, size_t lds, bool epi, bool dot,
                           hipStream_t s, const LaunchStamp &ev)
{
    dim3 g(gx, count), b(threads);
    if (dot)
        launch_k(ev, stencil_staged_batch<R, LT, true, true, kRegs>, g, b, (uint32_t)lds, s, dev);
    else if (epi)
        launch_k(ev, stencil_staged_batch<R, LT, true, false, kRegs>, g, b, (uint32_t)lds, s, dev);
    else
        launch_k(ev, stencil_staged_batch<R, LT, false, false, kRegs>, g, b, (uint32_t)lds, s, dev);
}

template <typename R, typename LT>
void launch_split_batch(const StencilParams *dev, int count, int gx, bool epi, bool dot, hipStream_t s,
                        const LaunchStamp &ev)
{
    dim3 g(gx, count), b(kSplitThreads);
    if (dot)
        launch_k(ev, stencil_split_batch<R, LT, true, true>, g, b, 0u, s, dev);
    else if (epi)
        launch_k(ev, stencil_split_batch<R, LT, true, false>, g, b, 0u, s, dev);
    else
        launch_k(ev, stencil_split_batch<R, LT, false, false>, g, b, 0u, s, dev);
}

template <typename R, typename LT>
void launch_staged_batch(const StencilParams *dev, int count, int gx, int threads, size_t lds, bool epi, bool dot,
                         bool regs, hipStream_t s, const LaunchStamp &ev)
{
    if constexpr (std::is_same<LT, __half2>::value) {
        if (regs) {
            launch_staged_batch_r<R, LT, true>(dev, count, gx, threads, lds, epi, dot, s, ev);
            return;
        }
    }
    launch_staged_batch_r<R, LT, false>(dev, count, gx, threads, lds, epi, dot, s, ev);
}

}  // namespace

namespace {

// Right-hand sides per block of a launch of nr of them over nblk blocks of sites: as many as leave the launch
// 1024 blocks (four per CU), or as many blocks as groups of one would
int rhs_per_block(int nr, int64_t nblk)
{
    const int64_t want = std::min<int64_t>(1024, nr * nblk);
    int g = kMaxRhs;
    while (g > 1 && (nr + g - 1) / g * nblk < want) --g;
    return g;
}

// whether an application of several right-hand sides holds the links in registers: FP16 two-row links, unless
// tuned otherwise or the environment asks for re-reads (SGN_MULTI_LINK_REGS=0)
bool link_regs(const Lattice &lat, sgn_prec p)
{
    if (p != SGN_PREC_F32_H16 || lat.link_ne != 6) return false;
    const char *e = std::getenv("SGN_MULTI_LINK_REGS");
    return !(e && e[0] == '0') && staged_shape(lat, p, true).regs != 0;
}

// 2..16 right-hand sides without an epilogue in one launch; false if no kernel takes them together
bool launch_rhs_block(const Lattice &lat, sgn_prec p, int nr, const OpSpec *op, const void *const *in,
                      void *const *out, hipStream_t s)
{
    const std::vector<Epilogue> ep(nr);
    const KernelPick pick = split_takes(lat, p, nr) && use_split(lat, p, true) ? kSplit : kStaged;
    bool regs = pick == kStaged && link_regs(lat, p);
    int cap = regs ? kRegsMaxThreads : 0;
    if (regs && !multi_shape_set(lat, p)) {
        // Two waves per SIMD hide little latency: below 1024 blocks half the block is faster where it fills its
        // wavefronts as well (12 right-hand sides, 512 against 256 sites per block: 16^4 59 against 53 us,
        // 16^3 x 32 98 against 91), and slower where it does not (20^4, 400 of 448 against 200 of 256 lanes: 141
        // against 152 us; 12^3 x 24, 432 of 448 against 144 of 192: 40 against 56).
        const StagedPlan full = staged_plan(lat, p, cap), half = staged_plan(lat, p, cap / 2);
        if (full.ok && half.ok && full.nblk_sites < 1024 && half.B * full.threads >= full.B * half.threads) cap /= 2;
    }
    PreparedStencil ps = prepare_stencil(lat, p, nr, op, in, out, ep.data(), cap, pick);
    if (pick == kStaged && !ps.pl.ok) return false;
    const int per = rhs_per_block(nr, ps.P.nblk_sites);
    if (per < 2) regs = false;
    const int prof = lat.ctx->prof_start(s, kclass(p), true);
    const LaunchStamp ev = lat.ctx->prof_stamp(prof);
    switch (p) {
    case SGN_PREC_F64:
        launch_multi_kernarg<double, double2>(ps.P, ps.nblk, ps.pl.threads, ps.pl.lds, per, ps.split, regs, s, ev);
        break;
    case SGN_PREC_F32:
        launch_multi_kernarg<float, float2>(ps.P, ps.nblk, ps.pl.threads, ps.pl.lds, per, ps.split, regs, s, ev);
        break;
    default:
        launch_multi_kernarg<float, __half2>(ps.P, ps.nblk, ps.pl.threads, ps.pl.lds, per, ps.split, regs, s, ev);
        break;
    }
    SGN_HIP(hipGetLastError());
    lat.ctx->prof_stop(prof, s, kclass(p), ps.bytes, ps.flops, false, ps.bytes_stored);
    return true;
}

// canon: one right-hand side without an epilogue, in and out in the canonical layout (split kernel only)
int launch_multi(const Lattice &lat, sgn_prec p, int nr, const OpSpec *op, const void *const *in, void *const *out,
                 const Epilogue *ep, hipStream_t s, bool canon)
{
    if (nr > 1 && std::none_of(ep, ep + nr, has_epilogue) && launch_rhs_block(lat, p, nr, op, in, out, s)) return 0;
    const PreparedStencil ps = prepare_stencil(lat, p, nr, op, in, out, ep, 0, canon ? kSplit : kAuto);
    if (nr > 1 && (ps.split || ps.pl.ok)) {
        int partials = 0;  // the same for each
        for (int r = 0; r < nr; ++r) partials = launch_multi(lat, p, 1, op + r, in + r, out + r, ep + r, s, false);
        return partials;
    }
    // one launch unless the unstaged kernel runs several right-hand sides
    const int prof = lat.ctx->prof_start(s, kclass(p), ps.pl.ok || nr == 1);
    const LaunchStamp ev = lat.ctx->prof_stamp(prof);
    switch (p) {
    case SGN_PREC_F64:
        if (ps.split)
            launch_split<double, double2>(ps.P, ps.nblk, ps.epi, ps.dot, canon, s, ev);
        else if (ps.pl.ok)
            launch_staged<double, double2>(ps.P, ps.nblk, ps.pl.threads, ps.pl.lds, ps.epi, ps.dot, s, ev);
        else
            launch_nr<double, double2>(ps.P, nr, ps.nblk, ps.epi, ps.dot, s, ev);
        break;
    case SGN_PREC_F32:
        if (ps.split)
            launch_split<float, float2>(ps.P, ps.nblk, ps.epi, ps.dot, canon, s, ev);
        else if (ps.pl.ok)
            launch_staged<float, float2>(ps.P, ps.nblk, ps.pl.threads, ps.pl.lds, ps.epi, ps.dot, s, ev);
        else
            launch_nr<float, float2>(ps.P, nr, ps.nblk, ps.epi, ps.dot, s, ev);
        break;
    default:
        if (ps.split)
            launch_split<float, __half2>(ps.P, ps.nblk, ps.epi, ps.dot, canon, s, ev);
        else if (ps.pl.ok)
            launch_staged<float, __half2>(ps.P, ps.nblk, ps.pl.threads, ps.pl.lds, ps.epi, ps.dot, s, ev);
        else
            launch_nr<float, __half2>(ps.P, nr, ps.nblk, ps.epi, ps.dot, s, ev);
        break;
    }
    SGN_HIP(hipGetLastError());
    lat.ctx->prof_stop(prof, s, kclass(p), ps.bytes, ps.flops, false, ps.bytes_stored);
    return ps.partials;
}

}  // namespace

int dslash_launch_multi(const Lattice &lat, sgn_prec p, int nr, const OpSpec *op, const void *const *in,
                        void *const *out, const Epilogue *ep, hipStream_t s)
{
    return launch_multi(lat, p, nr, op, in, out, ep, s, false);
}

namespace {

template <typename R, typename LT>
void launch_split_pair(const PreparedStencil &ps, hipStream_t s, const LaunchStamp &ev)
{
    const dim3 g(ps.nblk, 2), b(kSplitThreads);
    if (ps.dot)
        launch_k(ev, stencil_split_pair<R, LT, true, true>, g, b, 0u, s, ps.P);
    else if (ps.epi)
        launch_k(ev, stencil_split_pair<R, LT, true, false>, g, b, 0u, s, ps.P);
    else
        launch_k(ev, stencil_split_pair<R, LT, false, false>, g, b, 0u, s, ps.P);
}

}  // namespace

bool dslash_pairs(const Lattice &lat, sgn_prec p)
{
    return use_split(lat, p, false);
}

int dslash_launch_pair(const Lattice &lat, sgn_prec p, const OpSpec *op, const void *const *in, void *const *out,
                       const Epilogue *ep, hipStream_t s)
{
    if (!dslash_pairs(lat, p)) {
        const int n0 = dslash_launch(lat, p, op[0], in[0], out[0], ep[0], s);
        dslash_launch(lat, p, op[1], in[1], out[1], ep[1], s);
        return n0;
    }
    const PreparedStencil ps = prepare_stencil(lat, p, 2, op, in, out, ep, 0, kSplit);
    const int prof = lat.ctx->prof_start(s, kclass(p), true);
    const LaunchStamp ev = lat.ctx->prof_stamp(prof);
    switch (p) {
    case SGN_PREC_F64: launch_split_pair<double, double2>(ps, s, ev); break;
    case SGN_PREC_F32: launch_split_pair<float, float2>(ps, s, ev); break;
    default: launch_split_pair<float, __half2>(ps, s, ev); break;
    }
    SGN_HIP(hipGetLastError());
    lat.ctx->prof_stop(prof, s, kclass(p), ps.bytes, ps.flops, false, ps.bytes_stored);
    return ps.partials;
}

bool dslash_launch_canon(const Lattice &lat, sgn_prec p, const OpSpec &op, const void *in, void *out, hipStream_t s)
{
    const size_t bytes = (size_t)lat.V * (p == SGN_PREC_F64 ? 192 : 96);
    const uintptr_t a = reinterpret_cast<uintptr_t>(in), b = reinterpret_cast<uintptr_t>(out);
    if (lat.gauge || (a | b) % 16 != 0 || (a < b + bytes && b < a + bytes)) return false;
    const Epilogue ep;
    launch_multi(lat, p, 1, &op, &in, &out, &ep, s, true);
    return true;
}

StencilBatch::~StencilBatch()
{
    if (dev_) (void)hipFree(dev_);
}

void StencilBatch::prepare(const std::vector<StencilJob> &jobs, sgn_prec p)
{
    jobs_ = jobs;
    prec_ = p;
    partials_.assign(jobs.size(), 0);
    batched_ = !jobs.empty();
    epi_ = dot_ = false;
    gx_ = threads_ = 0;
    lds_ = 0;
    bytes_ = flops_ = bytes_stored_ = 0.0;
    // applications on the same lattice become multi-RHS groups (right-hand sides sharing every
    // link load); the groups are the launch's blockIdx.y.  A group's block walks its right-hand
    // sides one after another, so the group size is the largest (up to kMaxRhs) that still leaves
    // the launch 1024 blocks of sites (four per CU), or as many as groups of one would: small
    // lattices trade link sharing for parallelism
    // The split kernel serves a launch whose fields together are small; with more of them the chip is full and
    // the staged kernel's reuse wins (24 right-hand sides on 8^4, 12^4 and 16^4, FP32 with a dot product: 66 us
    // staged, 77 split).  Dot products have the same bits either way.
    double fields = 0.0;
    for (const StencilJob &j : jobs) fields += (double)j.lat->V * (p == SGN_PREC_F64 ? 192 : 96);
    const bool small = fields <= (double)kSplitMaxBytes;
    int gsize = kMaxRhs;
    bool multi = false;  // whether the staged kernel would see a group of several right-hand sides
    {
        std::vector<const Lattice *> lats;
        std::vector<int64_t> cnt, per, per_staged;
        for (const StencilJob &j : jobs) {
            size_t l = 0;
            while (l < lats.size() && lats[l] != j.lat) ++l;
            if (l == lats.size()) {
                lats.push_back(j.lat);
                cnt.push_back(0);
                const Context::TunedShape ts = staged_shape(*j.lat, p, true);
                const StagedPlan pl = staged_plan(*j.lat, p, 0, ts.max_sites, ts.tslices);
                per_staged.push_back(pl.ok ? pl.nblk_sites : (j.lat->V + 255) / 256);
                per.push_back(small && use_split(*j.lat, p, true) ? (j.lat->V + kSplitSites - 1) / kSplitSites
                                                                  : per_staged.back());
            }
            ++cnt[l];
        }
        auto group_size = [&](const std::vector<int64_t> &blk) {
            auto blocks = [&](int g) {
                int64_t b = 0;
                for (size_t l = 0; l < lats.size(); ++l) b += (cnt[l] + g - 1) / g * blk[l];
                return b;
            };
            int g = kMaxRhs;
            const int64_t want = std::min<int64_t>(1024, blocks(1));
            while (g > 1 && blocks(g) < want) --g;
            return g;
        };
        gsize = group_size(per);
        const int staged = group_size(per_staged);
        for (int64_t c : cnt) multi = multi || std::min<int64_t>(c, staged) > 1;
    }
    std::vector<std::vector<size_t>> groups;
    for (size_t k = 0; k < jobs.size(); ++k) {
        size_t g = 0;
        for (; g < groups.size(); ++g)
            if (jobs[groups[g][0]].lat == jobs[k].lat && (int)groups[g].size() < gsize) break;
        if (g == groups.size()) groups.emplace_back();
        groups[g].push_back(k);
    }
    // the split kernel's groups first: two launches where a lattice has a staged shape tuned or pinned
    auto split_group = [&](const std::vector<size_t> &g) {
        return small && use_split(*jobs[g[0]].lat, p, g.size() > 1);
    };
    nsplit_ = (int)(std::stable_partition(groups.begin(), groups.end(), split_group) - groups.begin());
    gx_split_ = 0;
    // links in registers (FP16 two-row links, some group with several right-hand sides, and the
    // environment does not ask for re-reads: SGN_MULTI_LINK_REGS=0)
    regs_ = p == SGN_PREC_F32_H16;
    for (size_t g = 0; g < groups.size(); ++g) regs_ = regs_ && jobs[groups[g][0]].lat->link_ne == 6;
    {
        const char *e = std::getenv("SGN_MULTI_LINK_REGS");
        const int tuned = jobs.empty() ? -1 : staged_shape(*jobs[0].lat, p, true).regs;
        regs_ = regs_ && multi && !(e && e[0] == '0') && tuned != 0;
    }
    // The full block, also where half of it would be faster (FP16 launches of BiCGStab batches, full against half:
    // 24 on 16^4 106 / 102 us, 12 on 16^3 x 32 102 / 97, 8 on 20^4 110 / 94, 32 on 12^4 60 / 60): the block decides
    // how the dot products are summed, and with it the iterates of a mixed solve.
    const int cap = regs_ ? kRegsMaxThreads : 0;
    // the blocks whose sums a split dot product leaves (without a staged shape for some lattice every
    // application would be a launch of its own, without the cap)
    int dot_cap = cap;
    for (size_t g = 0; g < groups.size(); ++g)
        if (!staged_plan(*jobs[groups[g][0]].lat, p, cap).ok) dot_cap = 0;
    std::vector<StencilParams> host(groups.size());
    for (size_t g = 0; g < groups.size(); ++g) {
        const int nr = (int)groups[g].size();
        std::vector<OpSpec> op(nr);
        std::vector<const void *> in(nr);
        std::vector<void *> out(nr);
        std::vector<Epilogue> ep(nr);
        for (int r = 0; r < nr; ++r) {
            const StencilJob &j = jobs[groups[g][r]];
            op[r] = j.op;
            in[r] = j.in;
            out[r] = j.out;
            ep[r] = j.ep;
        }
        const Lattice &lat = *jobs[groups[g][0]].lat;
        const PreparedStencil ps = prepare_stencil(lat, p, nr, op.data(), in.data(), out.data(), ep.data(),
                                                   (int)g < nsplit_ ? dot_cap : cap, (int)g < nsplit_ ? kSplit : kStaged);
        host[g] = ps.P;
        for (size_t k : groups[g]) partials_[k] = ps.partials;
        batched_ = batched_ && (ps.pl.ok || ps.split);
        epi_ = epi_ || ps.epi;
        dot_ = dot_ || ps.dot;
        if (ps.split) {
            gx_split_ = std::max(gx_split_, ps.nblk);
        } else {
            gx_ = std::max(gx_, ps.nblk);
            threads_ = std::max(threads_, ps.pl.threads);
            lds_ = std::max(lds_, ps.pl.lds);
        }
        bytes_ += ps.bytes;
        bytes_stored_ += ps.bytes_stored;
        flops_ += ps.flops;
    }
    ngroups_ = (int)groups.size() - nsplit_;
    gx_ = (gx_ + 7) / 8 * 8;
    gx_split_ = (gx_split_ + 7) / 8 * 8;
    if (!batched_) {  // launches of their own (see launch), and so the partials of those
        for (size_t k = 0; k < jobs.size(); ++k) {
            const StencilJob &j = jobs[k];
            partials_[k] = prepare_stencil(*j.lat, p, 1, &j.op, &j.in, &j.out, &j.ep).partials;
        }
        return;
    }
    const size_t need = sizeof(StencilParams) * host.size();
    // unchanged parameters stay on the device; new ones wait until no launch reads the old
    if (need == uploaded_.size() && std::memcmp(uploaded_.data(), host.data(), need) == 0) return;
    SGN_HIP(hipDeviceSynchronize());
    if (need > dev_bytes_) {
        if (dev_) SGN_HIP(hipFree(dev_));
        dev_ = nullptr;
        dev_bytes_ = 0;
        if (hipMalloc(&dev_, need) != hipSuccess) throw Failure{SGN_ERR_NOMEM, "stencil batch parameters"};
        dev_bytes_ = need;
    }
    SGN_HIP(hipMemcpy(dev_, host.data(), need, hipMemcpyHostToDevice));
    uploaded_.assign(reinterpret_cast<const char *>(host.data()), reinterpret_cast<const char *>(host.data()) + need);
}

void StencilBatch::launch(hipStream_t s) const
{
    if (jobs_.empty()) return;
    if (!batched_) {  // some lattice has no staged block shape: one launch per application
        for (const StencilJob &j : jobs_) dslash_launch(*j.lat, prec_, j.op, j.in, j.out, j.ep, s);
        return;
    }
    Context *ctx = jobs_[0].lat->ctx;
    const int prof = ctx->prof_start(s, kclass(prec_), !nsplit_ || !ngroups_);  // a stamp takes one kernel
    const LaunchStamp ev = ctx->prof_stamp(prof);
    const StencilParams *d = static_cast<const StencilParams *>(dev_);
    if (nsplit_) {
        switch (prec_) {
        case SGN_PREC_F64: launch_split_batch<double, double2>(d, nsplit_, gx_split_, epi_, dot_, s, ev); break;
        case SGN_PREC_F32: launch_split_batch<float, float2>(d, nsplit_, gx_split_, epi_, dot_, s, ev); break;
        default: launch_split_batch<float, __half2>(d, nsplit_, gx_split_, epi_, dot_, s, ev); break;
        }
    }
    if (ngroups_) {
        d += nsplit_;
        switch (prec_) {
        case SGN_PREC_F64:
            launch_staged_batch<double, double2>(d, ngroups_, gx_, threads_, lds_, epi_, dot_, false, s, ev);
            break;
        case SGN_PREC_F32:
            launch_staged_batch<float, float2>(d, ngroups_, gx_, threads_, lds_, epi_, dot_, regs_, s, ev);
            break;
        default: launch_staged_batch<float, __half2>(d, ngroups_, gx_, threads_, lds_, epi_, dot_, regs_, s, ev); break;
        }
    }
    SGN_HIP(hipGetLastError());
    ctx->prof_stop(prof, s, kclass(prec_), bytes_, flops_, false, bytes_stored_);
}

int dslash_launch(const Lattice &lat, sgn_prec p, const OpSpec &op, const void *in, void *out,
                  const Epilogue &ep, hipStream_t s)
{
    return dslash_launch_multi(lat, p, 1, &op, &in, &out, &ep, s);
}

}  // namespace sgn

// ----------------------------------------------------------------------------- no-allocation scratch
// Staging of the two fields of wilson_apply_noalloc: one file-scope device array, a copy of
// which every GPU holds from the time the library's code is loaded on it until the process
// ends.  Host code never passes the array's name (a host-side stand-in) to a kernel or copy:
// noalloc_scratch() takes its address on each device once, with that device current, and
// kernels receive that address.
static __device__ __align__(256) unsigned char scratch[SGN_NOALLOC_MAX_BYTES];

namespace sgn {

void *noalloc_scratch(int device)
{
    static std::mutex mu;
    static std::map<int, void *> addr;
    std::lock_guard<std::mutex> lock(mu);
    auto it = addr.find(device);
    if (it != addr.end()) return it->second;
    int cur = -1;
    SGN_HIP(hipGetDevice(&cur));
    SGN_REQUIRE(cur == device, "no-allocation scratch: the device must be current");
    void *ptr = nullptr;
    SGN_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    SGN_REQUIRE(ptr != nullptr, "no-allocation scratch: no device address");
    addr[device] = ptr;
    return ptr;
}

}  // namespace sgn

// ----------------------------------------------------------------------------- C ABI
using namespace sgn;

static sgn_status apply_common(sgn_lattice l, double mu, const void *in, void *out, sgn_prec p,
                               unsigned flags, void *stream, bool dag)
{
    return guard([&] {
        SGN_REQUIRE(l != nullptr && in != nullptr && out != nullptr, "wilson_apply: null argument");
        SGN_REQUIRE(in != out, "wilson_apply: in and out must differ");
        SGN_REQUIRE(std::isfinite(mu), "wilson_apply: mu is not finite");
        Lattice &lat = *as_lattice(l);
        SGN_HIP(hipSetDevice(lat.ctx->device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        OpSpec op;
        const bool g5 = !(flags & SGN_NO_GAMMA5);
        if (!dag) {
            op.mu = mu;
            op.g5_out = g5;
            op.g5_in = false;
        } else if (g5) {   // H(mu)^H = H(-mu)
            op.mu = -mu;
            op.g5_out = true;
            op.g5_in = false;
        } else {           // D(mu)^H = gamma5 D(-mu) gamma5
            op.mu = -mu;
            op.g5_out = true;
            op.g5_in = true;
        }
        Epilogue ep;
        if (flags & SGN_INTERNAL_LAYOUT) {
            dslash_launch(lat, p, op, in, out, ep, s);
        } else {
            if (dslash_launch_canon(lat, p, op, in, out, s)) return;
            const size_t bytes = spinor_bytes(lat.S, p);
            lat.ensure_stage(bytes);
            pack_spinor(lat, in, lat.stage_in, p, s);
            dslash_launch(lat, p, op, lat.stage_in, lat.stage_out, ep, s);
            unpack_spinor(lat, lat.stage_out, out, p, s);
        }
    });
}

extern "C" sgn_status wilson_apply(sgn_lattice lat, double mu, const void *in, void *out, sgn_prec p,
                                   unsigned flags, void *stream)
{
    return apply_common(lat, mu, in, out, p, flags, stream, false);
}

extern "C" sgn_status wilson_apply_dag(sgn_lattice lat, double mu, const void *in, void *out, sgn_prec p,
                                       unsigned flags, void *stream)
{
    return apply_common(lat, mu, in, out, p, flags, stream, true);
}

extern "C" sgn_status wilson_apply_noalloc(sgn_lattice l, double mu, const void *in, void *out, sgn_prec p,
                                           unsigned flags, void *stream)
{
    return guard([&] {
        SGN_REQUIRE(l != nullptr && in != nullptr && out != nullptr, "wilson_apply_noalloc: null argument");
        SGN_REQUIRE(in != out, "wilson_apply_noalloc: in and out must differ");
        SGN_REQUIRE(std::isfinite(mu), "wilson_apply_noalloc: mu is not finite");
        SGN_REQUIRE(p == SGN_PREC_F64 || p == SGN_PREC_F32 || p == SGN_PREC_F32_H16,
                    "wilson_apply_noalloc: unknown precision");
        Lattice &lat = *as_lattice(l);
        SGN_HIP(hipSetDevice(lat.ctx->device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        OpSpec op;
        op.mu = mu;
        op.g5_out = !(flags & SGN_NO_GAMMA5);
        Epilogue ep;
        if (flags & SGN_INTERNAL_LAYOUT) {  // no staging needed
            dslash_launch(lat, p, op, in, out, ep, s);
            return;
        }
        const size_t bytes = spinor_bytes(lat.S, p);
        const size_t off = (bytes + 255) / 256 * 256;  // second field 256-byte aligned
        if (off + bytes > (size_t)SGN_NOALLOC_MAX_BYTES)
            throw Failure{SGN_ERR_INVALID, "wilson_apply_noalloc: the lattice needs " + std::to_string(off + bytes) +
                                               " staging bytes, more than SGN_NOALLOC_MAX_BYTES = " +
                                               std::to_string((size_t)SGN_NOALLOC_MAX_BYTES)};
        SGN_REQUIRE(lat.ctx->noalloc != nullptr, "wilson_apply_noalloc: scratch address not set up");
        if (dslash_launch_canon(lat, p, op, in, out, s)) return;
        char *stage_in = static_cast<char *>(lat.ctx->noalloc);
        char *stage_out = stage_in + off;
        pack_spinor(lat, in, stage_in, p, s);
        dslash_launch(lat, p, op, stage_in, stage_out, ep, s);
        unpack_spinor(lat, stage_out, out, p, s);
    });
}

extern "C" sgn_status sgn_autotune(sgn_lattice l, sgn_prec p, int nrhs, int reps, sgn_tune_candidate *out,
                                   int max_out, int *n_out, void *stream)
{
    return guard([&] {
        SGN_REQUIRE(l != nullptr, "sgn_autotune: null lattice");
        SGN_REQUIRE(p == SGN_PREC_F64 || p == SGN_PREC_F32 || p == SGN_PREC_F32_H16, "sgn_autotune: unknown precision");
        SGN_REQUIRE(nrhs >= 1 && nrhs <= kMaxRhs, "sgn_autotune: nrhs must be 1..16");
        SGN_REQUIRE(max_out >= 0 && (max_out == 0 || out != nullptr), "sgn_autotune: bad output array");
        Lattice &lat = *as_lattice(l);
        Context &ctx = *lat.ctx;
        SGN_HIP(hipSetDevice(ctx.device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (reps <= 0) reps = 20;
        const bool multi = nrhs > 1;
        const std::vector<int> key = {lat.L[0], lat.L[1], lat.L[2], lat.L[3], (int)p, multi ? 1 : 0};
        // candidate shapes: distinct blocks of the staged plan under decreasing site caps, as one
        // t-slice or as bricks of two, and for several right-hand sides with FP16 two-row links both
        // link modes
        struct Cand {
            int cap, B, T, regs;
            double us;
            int unstaged;
        };
        std::vector<Cand> cands;
        // the unstaged kernel, or on small lattices the split one (for several right-hand sides if it takes them)
        if (!multi || split_takes(lat, p, nrhs)) cands.push_back({0, 0, 1, -1, 0.0, 1});
        const bool can_regs = multi && p == SGN_PREC_F32_H16 && lat.link_ne == 6;
        for (int regs : can_regs ? std::vector<int>{1, 0} : std::vector<int>{-1}) {
            for (int T : {1, 2}) {
                std::vector<int> seen;
                for (int cap : {0, 576, 432, 384, 288, 192, 96}) {
                    const StagedPlan pl = staged_plan(lat, p, regs == 1 ? kRegsMaxThreads : 0, cap, T);
                    if (!pl.ok && T == 2) continue;
                    const int B = pl.ok ? pl.B : 0;
                    if (std::find(seen.begin(), seen.end(), B) != seen.end()) continue;
                    seen.push_back(B);
                    cands.push_back({cap, B, pl.ok ? pl.T : 1, regs, 0.0, 0});
                }
            }
        }
        // fields: nrhs inputs (zero) and outputs in the internal layout
        const size_t bytes = spinor_bytes(lat.S, p);
        std::vector<void *> buf(2 * nrhs, nullptr);
        struct Free {
            std::vector<void *> &b;
            ~Free()
            {
                for (void *q : b)
                    if (q) (void)hipFree(q);
            }
        } freer{buf};
        for (void *&q : buf) {
            if (hipMalloc(&q, bytes) != hipSuccess) throw Failure{SGN_ERR_NOMEM, "sgn_autotune: fields"};
            SGN_HIP(hipMemsetAsync(q, 0, bytes, s));
        }
        std::vector<OpSpec> op(nrhs);
        std::vector<Epilogue> ep(nrhs);
        std::vector<const void *> in(nrhs);
        std::vector<void *> outp(nrhs);
        for (int r = 0; r < nrhs; ++r) {
            op[r].mu = 0.2;
            in[r] = buf[r];
            outp[r] = buf[nrhs + r];
        }
        hipEvent_t e0, e1;
        SGN_HIP(hipEventCreate(&e0));
        SGN_HIP(hipEventCreate(&e1));
        const auto set = ctx.tuned.find(key);
        const bool was_set = set != ctx.tuned.end();
        const Context::TunedShape before = was_set ? set->second : Context::TunedShape{};
        try {
            for (Cand &c : cands) {
                ctx.tuned[key] = {c.cap, c.regs, c.T, c.unstaged};
                for (int w = 0; w < 3; ++w) dslash_launch_multi(lat, p, nrhs, op.data(), in.data(), outp.data(), ep.data(), s);
                SGN_HIP(hipEventRecord(e0, s));
                for (int k = 0; k < reps; ++k)
                    dslash_launch_multi(lat, p, nrhs, op.data(), in.data(), outp.data(), ep.data(), s);
                SGN_HIP(hipEventRecord(e1, s));
                SGN_HIP(hipEventSynchronize(e1));
                float ms = 0.f;
                SGN_HIP(hipEventElapsedTime(&ms, e0, e1));
                c.us = 1e3 * ms / reps;
            }
        } catch (...) {
            // (an entry where there was none would keep the split kernel from lattices of these dimensions)
            if (was_set) ctx.tuned[key] = before;
            else ctx.tuned.erase(key);
            (void)hipEventDestroy(e0);
            (void)hipEventDestroy(e1);
            throw;
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        const Cand *best = &cands[0];
        for (const Cand &c : cands)
            if (c.us < best->us) best = &c;
        ctx.tuned[key] = {best->cap, best->regs, best->T, best->unstaged};
        SGN_HIP(hipDeviceSynchronize());
        const int n = std::min<int>((int)cands.size(), max_out);
        for (int k = 0; k < n; ++k)
            out[k] = {cands[k].B * cands[k].T, cands[k].regs < 0 ? 0 : cands[k].regs, cands[k].us,
                      &cands[k] == best ? 1 : 0, cands[k].T};
        if (n_out) *n_out = (int)cands.size();
    });
}

extern "C" sgn_status sgn_tune_set(sgn_lattice l, sgn_prec p, int multi, int max_sites, int t_slices,
                                   int links_in_registers)
{
    return guard([&] {
        SGN_REQUIRE(l != nullptr, "sgn_tune_set: null lattice");
        SGN_REQUIRE(p == SGN_PREC_F64 || p == SGN_PREC_F32 || p == SGN_PREC_F32_H16, "sgn_tune_set: unknown precision");
        SGN_REQUIRE(max_sites >= -1, "sgn_tune_set: max_sites must be >= -1");
        SGN_REQUIRE(t_slices == 1 || t_slices == 2, "sgn_tune_set: t_slices must be 1 or 2");
        SGN_REQUIRE(links_in_registers >= -1 && links_in_registers <= 1, "sgn_tune_set: links_in_registers is -1, 0 or 1");
        Lattice &lat = *as_lattice(l);
        const bool unstaged = max_sites == -1;
        if (!unstaged) {
            const StagedPlan pl = staged_plan(lat, p, 0, max_sites, t_slices);
            SGN_REQUIRE(pl.ok && pl.T == t_slices, "sgn_tune_set: no staged block of this shape fits the lattice");
        }
        SGN_HIP(hipSetDevice(lat.ctx->device));
        SGN_HIP(hipDeviceSynchronize());
        lat.ctx->tuned[{lat.L[0], lat.L[1], lat.L[2], lat.L[3], (int)p, multi ? 1 : 0}] =
            Context::TunedShape{unstaged ? 0 : max_sites, links_in_registers, t_slices, unstaged ? 1 : 0};
    });
}

extern "C" sgn_status wilson_apply_multi(sgn_lattice l, int nrhs, const double *mu, const void *const *in,
                                         void *const *out, sgn_prec p, unsigned flags, void *stream)
{
    return guard([&] {
        SGN_REQUIRE(l != nullptr && mu != nullptr && in != nullptr && out != nullptr && nrhs >= 0,
                    "wilson_apply_multi: null argument");
        SGN_REQUIRE(flags & SGN_INTERNAL_LAYOUT, "wilson_apply_multi: fields must be in the internal layout");
        Lattice &lat = *as_lattice(l);
        SGN_HIP(hipSetDevice(lat.ctx->device));
        hipStream_t s = static_cast<hipStream_t>(stream);
        for (int i = 0; i < nrhs; ++i) {
            SGN_REQUIRE(in[i] && out[i] && std::isfinite(mu[i]), "wilson_apply_multi: bad right-hand side");
            for (int j = 0; j < nrhs; ++j)
                SGN_REQUIRE(in[i] != out[j], "wilson_apply_multi: inputs and outputs must not alias");
        }
        for (int i0 = 0; i0 < nrhs; i0 += kMaxRhs) {
            const int nr = std::min(kMaxRhs, nrhs - i0);
            OpSpec op[kMaxRhs];
            Epilogue ep[kMaxRhs];
            for (int r = 0; r < nr; ++r) {
                op[r].mu = mu[i0 + r];
                op[r].g5_out = !(flags & SGN_NO_GAMMA5);
            }
            dslash_launch_multi(lat, p, nr, op, in + i0, out + i0, ep, s);
        }
    });
}
