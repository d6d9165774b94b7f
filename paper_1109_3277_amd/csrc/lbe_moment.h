// The step at tau = 1 in moments (FP64): device functions shared by the step
// kernel, the conversions from and to populations, and kill / fill.
//
// With tau = 1 the BGK collision (Eq. (2)) replaces every population by its
// equilibrium, f*_i = f_i^eq(rho^c, u^eq_c): all that a node carries from one
// step to the next are rho^A, rho^B and the common velocity u' =
// (j^A + j^B) / (rho^A + rho^B). The state of a node is then
//   plane 0, 1   rho^A, rho^B
//   plane 2..4   u'
//   plane 5, 6   Psi^A, Psi^B   (the shell fills write solid nodes)
// in seven planes of N doubles per copy, two copies. The populations are formed
// on the fly and only summed.
//
// FP64 only: the float forms relax as h - (h - h^eq) with the difference
// rounded, which at tau = 1 is h^eq up to that rounding; without the h their
// results could not stay what they are (1e-7 in the domain sizes).
//
// Every sum over the 19 populations runs in one order: the directions with
// c_iz = +1 (from plane z - 1), then 0, then -1, as the step kernel meets the
// planes. Contraction is off here and every fused multiply-add is written out,
// so that a population has the same bits wherever it is formed: a saved and
// reloaded run continues bit for bit.
#pragma once

#include "lbe_internal.h"

namespace lbe {

// k-th direction of the summation order: 0..4 c_iz = +1, 5..13 c_iz = 0, 14..18
// c_iz = -1, each by the in-plane position of its source: the node's own, then
// those with c = +x, +y, -x, -y (and the diagonals).
__host__ __device__ constexpr int sum_dir(int k) {
    constexpr int t[Q] = {3, 6, 8, 16, 18, 0, 1, 2, 10, 11, 4, 5, 13, 14, 12, 7, 9, 15, 17};
    return t[k];
}

// One component of a node after the collision: a = rho (1 - 1.5 u.u) and the
// velocity times three, so that population i is w_i (a + rho s (1 + s / 2)) with
// s = 3 c_i . u (constants that fit an instruction).
struct Post {
    double a, rho, ux, uy, uz;
};
__device__ inline Post post_of(double rho, double ux, double uy, double uz) {
#pragma clang fp contract(off)
    const double x = 3.0 * ux, y = 3.0 * uy, z = 3.0 * uz;
    return Post{fma_r(rho, (-1.0 / 6.0) * fma_r(x, x, fma_r(y, y, z * z)), rho), rho, x, y, z};
}
__device__ inline double pop_eq(int i, double a, double rho, double s) {
#pragma clang fp contract(off)
    return wq(i) * fma_r(rho * s, fma_r(0.5, s, 1.0), a);
}
__device__ inline double pop_of(const Post& p, int i) {
    return i == 0 ? pop_eq(0, p.a, p.rho, 0.0) : pop_eq(i, p.a, p.rho, dir_dot<double>(i, p.ux, p.uy, p.uz));
}

// Neighbour sums S = sum_i Psi(n + c_i) c_i of Eq. (3); p(i) gives Psi^A and
// Psi^B of neighbour i as a double2.
template <class F>
__device__ inline void mom_psi_sums(F p, double (&S0)[3], double (&S1)[3]) {
    for (int d = 0; d < 3; d++) S0[d] = S1[d] = 0.0;
#pragma unroll
    for (int i = 1; i < Q; i++) {
        const double2 v = p(i);
        if (cx(i) > 0) { S0[0] += v.x; S1[0] += v.y; }
        if (cx(i) < 0) { S0[0] -= v.x; S1[0] -= v.y; }
        if (cy(i) > 0) { S0[1] += v.x; S1[1] += v.y; }
        if (cy(i) < 0) { S0[1] -= v.x; S1[1] -= v.y; }
        if (cz(i) > 0) { S0[2] += v.x; S1[2] += v.y; }
        if (cz(i) < 0) { S0[2] -= v.x; S1[2] -= v.y; }
    }
}

// Post-collision components of a node: densities r0, r1, velocity u', Psi p0,
// p1, neighbour sums of Psi^A, Psi^B, body acceleration acc.
__device__ inline void collide_moments(const Box& bx, double r0, double r1, double ux, double uy, double uz, double p0,
                                       double p1, const double (&S0)[3], const double (&S1)[3], const double (&acc)[3],
                                       Post& A, Post& B) {
#pragma clang fp contract(off)
    // Psi / rho (1 at rho = 0 and for Psi = rho)
    double q0 = 1.0, q1 = 1.0;
    if (bx.psi_kind != 0) {
        q0 = r0 == 0.0 ? 1.0 : p0 / r0;
        q1 = r1 == 0.0 ? 1.0 : p1 / r1;
    }
    const double k0 = -bx.g * q0, k1 = -bx.g * q1;
    A = post_of(r0, ux + fma_r(k0, S1[0], acc[0]), uy + fma_r(k0, S1[1], acc[1]), uz + fma_r(k0, S1[2], acc[2]));
    B = post_of(r1, ux + fma_r(k1, S0[0], acc[0]), uy + fma_r(k1, S0[1], acc[1]), uz + fma_r(k1, S0[2], acc[2]));
}

// Running sums of the populations of a node, both components.
struct MomSum {
    double d0, d1, jx, jy, jz;
    __device__ void clear() { d0 = d1 = jx = jy = jz = 0.0; }
    __device__ void add(int i, double v0, double v1) {
#pragma clang fp contract(off)
        d0 = d0 + v0;
        d1 = d1 + v1;
        const double s = v0 + v1;
        if (cx(i) > 0) jx = jx + s;
        if (cx(i) < 0) jx = jx - s;
        if (cy(i) > 0) jy = jy + s;
        if (cy(i) < 0) jy = jy - s;
        if (cz(i) > 0) jz = jz + s;
        if (cz(i) < 0) jz = jz - s;
    }
};

// The seven numbers of a node from the sums of its populations; true when a
// density is negative or not a number.
__device__ inline bool finish_node(const Box& bx, const MomSum& m, double (&v)[kMomPlanes]) {
#pragma clang fp contract(off)
    const double irt = 1.0 / (m.d0 + m.d1);
    v[0] = m.d0;
    v[1] = m.d1;
    v[2] = m.jx * irt;
    v[3] = m.jy * irt;
    v[4] = m.jz * irt;
    v[5] = psi_of(m.d0, bx.psi_kind);
    v[6] = psi_of(m.d1, bx.psi_kind);
    return !(m.d0 >= 0.0) || !(m.d1 >= 0.0);
}

// A filled node (kill / fill, initial fields): every population of both components
// is the equilibrium of its density at velocity u. True for a bad density.
__device__ inline bool fill_node(const Box& bx, double r0, double r1, const double (&u)[3], double (&v)[kMomPlanes]) {
    const Post A = post_of(r0, u[0], u[1], u[2]), B = post_of(r1, u[0], u[1], u[2]);
    MomSum m;
    m.clear();
#pragma unroll
    for (int k = 0; k < Q; k++) m.add(sum_dir(k), pop_of(A, sum_dir(k)), pop_of(B, sum_dir(k)));
    return finish_node(bx, m, v);
}

// C of Eq. (4) per unit density for a link along c_l into a surface moving at U.
__device__ inline double bounce_c(int l, double Ux, double Uy, double Uz) {
#pragma clang fp contract(off)
    return -6.0 * wq(l) * dir_dot<double>(l, Ux, Uy, Uz);
}

// A step whose sums left a bad density somewhere raises *suspect; the nodes
// that are fluid before and after the re-rasterisation are then looked at
// (a node the step killed does not count). Copies: v the new state, o0 / o1
// the owner maps before and after.
__device__ inline void check_suspect(const Box& bx, const double* __restrict__ v, const uint32_t* __restrict__ o0,
                                     const uint32_t* __restrict__ o1, const int* __restrict__ suspect,
                                     int* __restrict__ health, int blk, int nblk) {
    if (*suspect == 0) return;
    const int64_t N = bx.N;
    for (int64_t n = (int64_t)blk * 256 + threadIdx.x; n < N; n += (int64_t)nblk * 256)
        if (o0[n] == OWN_FLUID && o1[n] == OWN_FLUID && (!(v[n] >= 0.0) || !(v[N + n] >= 0.0))) atomicOr(health, 1);
}

// Sums over this thread's nodes first, first + step, ...: masses, momentum, fluid
// count and the number of nodes with a bad density.
__device__ inline void mom_stats_acc(const Box& bx, const double* __restrict__ v, const uint32_t* __restrict__ owner,
                                     int64_t first, int64_t step, double (&acc)[7]) {
    const int64_t N = bx.N;
    for (int64_t n = first; n < N; n += step) {
        if (owner[n] != OWN_FLUID) continue;
        const double r0 = v[n], r1 = v[N + n], rt = r0 + r1;
        acc[0] += r0;
        acc[1] += r1;
        for (int d = 0; d < 3; d++) acc[2 + d] += rt != 0.0 ? rt * v[(2 + d) * N + n] : 0.0;
        acc[5] += 1.0;
        if (!(r0 >= 0.0) || !(r1 >= 0.0)) acc[6] += 1.0;
    }
}

}  // namespace lbe
