// Device helpers shared by the forward and adjoint kernels.
#pragma once

#include "btl_internal.h"

namespace btl {

__device__ __forceinline__ double2 ld2(const float2* p) {
    const float2 v = *p;
    return make_double2((double)v.x, (double)v.y);
}
__device__ __forceinline__ double2 ld2(const double2* p) { return *p; }
__device__ __forceinline__ void store2(float2* p, double2 v) {
    *p = make_float2((float)v.x, (float)v.y);
}
__device__ __forceinline__ void store2(double2* p, double2 v) { *p = v; }
// Streaming stores: the next step reads the whole state back, which does not
// fit in the caches, so the written lines are not kept.
__device__ __forceinline__ void store2_stream(float2* p, double2 v) {
    __builtin_nontemporal_store((float)v.x, &p->x);
    __builtin_nontemporal_store((float)v.y, &p->y);
}
__device__ __forceinline__ void store2_stream(double2* p, double2 v) {
    __builtin_nontemporal_store(v.x, &p->x);
    __builtin_nontemporal_store(v.y, &p->y);
}

// Value that is the same in every lane, kept in scalar registers.
__device__ __forceinline__ double uniform(double v) {
    const unsigned long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(u & 0xffffffffu));
    const int hi = __builtin_amdgcn_readfirstlane((int)(u >> 32));
    return __longlong_as_double(((long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double2 uniform2(double2 v) {
    return make_double2(uniform(v.x), uniform(v.y));
}

// Workgroups are dealt to the 8 XCDs round-robin (workgroup i to XCD
// i mod 8), each XCD with its own L2.  xcd_tile renumbers them so that every
// XCD walks one contiguous range of tiles: neighbouring tiles, which read
// each other's edge rows, then run on the same XCD close in time and share
// those rows through its L2.  A bijection of [0, G).
constexpr int kXcd = 8;
__device__ __forceinline__ int32_t xcd_tile(int32_t bid, int32_t G) {
    const int32_t k = bid % kXcd, i = bid / kXcd;
    const int32_t q = G / kXcd, r = G % kXcd;
    return (k < r ? k * (q + 1) : r * (q + 1) + (k - r) * q) + i;
}

// The products and sums of a site update are spelled out as fused operations,
// so that every kernel that updates a site rounds alike (k_step and k_pair
// give the same populations bit for bit).
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(__builtin_fma(a.x, b.x, -(a.y * b.y)),
                        __builtin_fma(a.x, b.y, a.y * b.x));
}

// Site word (StepArgs::words): four bits for each pull link, a membrane's
// 8 + the phase beyond it, 0 where there is none.
__device__ __forceinline__ uint32_t link_code(uint32_t word, int d) { return (word >> (4 * d)) & 0xfu; }
__device__ __forceinline__ bool link_membrane(uint32_t word, int d) { return (word >> (4 * d + 3)) & 1u; }
__device__ __forceinline__ int link_phase(uint32_t word, int d) { return (int)((word >> (4 * d)) & 0x7u); }

// Half-link membranes (Eqs. B5, P_def, permeability_BC): what enters across
// one is own + t (in - own), own the node's own outgoing population and t the
// transmitted share.  In this form the share keeps its relative precision
// however small it is (kappa = 0 lets nothing through), and the two sides of a
// link exchange exactly opposite amounts.  A share of 1 (no membrane) takes
// own as 0, which leaves the entering population exactly as it is whatever own
// holds, so that a site with any membrane can take its six links without a
// branch on each: k_pair does (128^3 x 24: 814 us per step; the form in + (1 -
// t) (own - in) needs no selection and took 805, 2 % less than with branches,
// but holds t to an absolute 1e-16 only); k_step, which runs at the bandwidth
// and whose loads of the own populations are then waited for at every site, is
// faster with the branches (960 against 1010).
// c_trans: [n_phase][16] transmitted shares by phase and link code, 1 where
// there is no membrane.
constexpr int kTransSize = kMaxPhase * 16;
__device__ __forceinline__ void fill_transmitted(double* c_trans, const double* trans, int P, int t) {
    if (t < P * 16) {
        const int n = t & 15;
        c_trans[t] = n >= 8 && n - 8 < P ? trans[(t >> 4) * P + (n - 8)] : 1.0;
    }
}
template <typename V>
__device__ __forceinline__ double2 half_link(double2 in, V own, double t) {
    const V o = V{t < 1.0 ? own.x : 0, t < 1.0 ? own.y : 0};
    const double ox = (double)o.x, oy = (double)o.y;
    return make_double2(__builtin_fma(t, in.x - ox, ox), __builtin_fma(t, in.y - oy, oy));
}

// Reaction by exp(-i fdt (c.j + cu)) = e and the decay dec, moment and
// collision of one site; g becomes the post-collision populations.  Returns
// the moment M.
template <int NQ>
__device__ __forceinline__ double2 react_collide(double2 (&g)[NQ], double2 e, double dec, double w) {
    const double2 rf = make_double2(e.x * dec, e.y * dec);
#pragma unroll
    for (int d = 0; d < NQ; ++d) g[d] = cmul(g[d], rf);
    double2 M = g[0];
#pragma unroll
    for (int d = 1; d < NQ; ++d) {
        M.x += g[d].x;
        M.y += g[d].y;
    }
#pragma unroll
    for (int d = 0; d < NQ; ++d) {
        const double wd = d == 0 ? lattice_w0(NQ) : lattice_w1(NQ);
        g[d].x = __builtin_fma(w, __builtin_fma(wd, M.x, -g[d].x), g[d].x);
        g[d].y = __builtin_fma(w, __builtin_fma(wd, M.y, -g[d].y), g[d].y);
    }
    return M;
}

// A copy made here and now: the register that v was loaded into is free for
// the next load (left to itself the compiler loads elsewhere and copies at the
// end of the loop, which waits for the load).
template <typename V>
__device__ __forceinline__ V copied(V v) {
    asm("" : "+v"(v.x), "+v"(v.y));
    return v;
}

// Workgroup barrier that orders LDS accesses alone: loads and stores of
// global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Weights of the six populations that make up the population entering a
// node across a membrane at distance d (units of dx) from it, for a straight
// membrane normal to the link (Eqs. B2a_text/B2b_text with theta = 0,
// Eqs. B4a-B4c).  The Dirichlet (c_d) and Neumann (c_n) coefficients of the
// node's own side use d (Eqs. c_d, c_n), those of the far side 1 - d.
// Output order: own side A[0..2] for ghat_ibar(x), ghat_ibar(x + e_i),
// ghat_i(x); far side B[0..2] for ghat_i(x - e_i), ghat_i(x - 2 e_i),
// ghat_ibar(x - e_i).  kdt = kappa dt, edx = eps_D dx.
struct MembCoef {
    double A[3], B[3];
};
__device__ __forceinline__ MembCoef membrane_coefficients(double d, double kdt, double edx) {
    const double e = 1.0 - d;
    // one division for the three reciprocals ro = 1/(2d + 1), rf = 1/(2e + 1)
    // and rF below: with Do = 3 - 2d, Df = 3 - 2e the denominator of rF is
    // ro rf Qd, Qd = Do Df edx + 2 (Do + Df) kdt
    const double Ao = 2.0 * d + 1.0, Af = 2.0 * e + 1.0;
    const double Do = 3.0 - 2.0 * d, Df = 3.0 - 2.0 * e;
    const double Qd = Do * Df * edx + 2.0 * (Do + Df) * kdt;
    const double AA = Ao * Af;
    const double R = 1.0 / (AA * Qd);
    const double ro = Af * Qd * R, rf = Ao * Qd * R;
    const double ho = 2.0 * d - 1.0, hf = 2.0 * e - 1.0;
    // own side
    const double n2 = -ho * ro, n3 = ho * ro, n4 = 2.0 * ro;
    const double d1 = 2.0 * d - 2.0, d2 = -ho * ho * ro, d3 = 2.0 * ho * ro, d4 = (3.0 - 2.0 * d) * ro;
    // far side
    const double fn2 = -hf * rf, fn3 = hf * rf, fn4 = 2.0 * rf;
    const double fd1 = 2.0 * e - 2.0, fd2 = -hf * hf * rf, fd3 = 2.0 * hf * rf, fd4 = (3.0 - 2.0 * e) * rf;
    const double diff = d4 * fd4 * edx;
    const double perm_own = fd4 * n4 * kdt, perm_far = fn4 * d4 * kdt;
    const double rF = AA * AA * R;   // 1 / (diff + (d4 fn4 + n4 fd4) kdt)
    MembCoef c;
    c.A[0] = (diff + perm_own * d1 + perm_far) * rF;
    c.A[1] = (diff * n2 + perm_own * d2 + perm_far * n2) * rF;
    c.A[2] = (diff * n3 + perm_own * d3 + perm_far * n3) * rF;
    const double bk = d4 * n4 * kdt * rF;
    c.B[0] = bk * (1.0 - fd1);
    c.B[1] = bk * (fn2 - fd2);
    c.B[2] = bk * (fn3 - fd3);
    return c;
}

// exp(i th) in FP64 (library sincos; used only by the table kernel).
__device__ __forceinline__ double2 expi(double th) {
    double sn, cs;
    sincos(th, &sn, &cs);
    return make_double2(cs, sn);
}

}  // namespace btl
