// The step at tau = 1 in moments (gfx950, FP64): see lbe_moment.h for the state.
//
// k_mstep advances the fluid by one whole step in one pass over the seven numbers of
// every node: 112 B per node and step at the least, where populations that are
// streamed and re-read for the densities take 928. It moves 1.7 to 1.8 times that:
// a block of 32 x 8 nodes reads rho and u' at 340 positions of a plane and Psi at 432,
// and three planes more than it writes.
#include <algorithm>
#include <type_traits>

#include "lbe_moment.h"

#pragma clang fp contract(off)

namespace lbe {

// Block b of nb, with each of the 8 XCDs (round-robin dispatch) walking a
// contiguous range: the halos that neighbouring columns share sit in one L2.
__device__ inline int xcd_range(int b, int nb) {
    const int x = b & 7, q = nb >> 3, r = nb & 7;
    return x * q + min(x, r) + (b >> 3);
}

// ---------------------------------------------------------------- step
// A block owns a column of TX x TY nodes and marches zc planes up z. At plane k
// it forms the post-collision moments (`Post`, both components) of the column
// and a one-node ring around it into LDS: Psi of three planes with a two-node
// ring is staged there for the force stencil, rho and u' come straight from
// memory. Then every thread sums the populations that stream to its node: of
// node k the directions coming from plane k - 1 (still in LDS) and within plane
// k, of node k - 1 the ones coming from plane k, which completes it. So each
// node's 38 equilibria are formed from at most two resident planes, and two
// blocks fit a CU. The next plane's loads are in flight meanwhile.
// Without solids a thread reads its nine sources of plane k once, for the three
// nodes they stream to, and carries the sums of plane k + 1 along: the order of
// each node's sum is the same, one plane of moments suffices, and three blocks fit
// a CU (128^3: 95 us per step in two planes, 81 in one).
//
// With solids, a source n - c_i that is solid stands for a link of n into it:
// the population is the node's own f*_l, l = ibar, bounced (Eq. (4)), plus
// C = -6 w_l rho^c (U_n . c_l), U_n = V + W x r_n of that particle; its momentum
// exchange (2 f*_l + C) c_l over both components adds to the node's force on the
// particle, written into the node's record as the link force pass expects.
// Waves without links, waves whose nodes touch one body each, and the rest take
// separate paths. U_n comes from wave-uniform loads: the wave visits the distinct
// bodies one at a time; a node's third and further bodies are read per lane.
template <bool SOLID, int TX, int TY>
__device__ inline void mstep_body(const Box& bx, const double* __restrict__ vin, double* __restrict__ vout,
                                  const uint32_t* __restrict__ owner, const double* __restrict__ pfast,
                                  double* __restrict__ rec, int rstride, int* __restrict__ bad, int tiles_x, int tiles_y,
                                  int zc, int blk) {
    static_assert(TX * TY == 256, "one node of the column per thread");
    constexpr int MX = TX + 2, MY = TY + 2, MP = MX * MY;      // column with a one-node ring
    constexpr int PX_ = TX + 4, PY_ = TY + 4, PP = PX_ * PY_;  // with a two-node ring
    constexpr int NP = (PP + 255) / 256;                       // staged Psi per thread and component
    static_assert((MP + 255) / 256 == 2, "the ring fits one extra round");
    __shared__ double s_psi[3][2][PP];
    __shared__ double s_m[SOLID ? 2 : 1][10][MP];
    __shared__ uint32_t s_own[SOLID ? 4 : 1][SOLID ? MP : 1];

    const int nx = bx.nx, ny = bx.ny, nz = bx.nz;
    const uint32_t N = (uint32_t)bx.N;
    const uint32_t pl = (uint32_t)nx * (uint32_t)ny;
    const int tx = blk % tiles_x, tq = blk / tiles_x;
    const int ty = tq % tiles_y, zbeg = (tq / tiles_y) * zc;
    const int zend = min(zbeg + zc, nz);
    const int x0 = tx * TX, y0 = ty * TY;
    const int t = threadIdx.x;
    const int lx = t % TX, ly = t / TX;
    const int x = x0 + lx, y = y0 + ly;
    const bool active = x < nx && y < ny;
    const double accv[3] = {bx.ax, bx.ay, bx.az};

    // in-plane node offset of column position (px, py), counted from the
    // column's corner: periodic; positions past a ragged edge (never used by an
    // active node) are clamped into the box
    auto at_xy = [&](int px, int py) -> uint32_t {
        int gx = x0 + px, gy = y0 + py;
        gx = gx < 0 ? gx + nx : (gx >= nx ? gx - nx : gx);
        gy = gy < 0 ? gy + ny : (gy >= ny ? gy - ny : gy);
        gx = gx < nx ? gx : 0;
        gy = gy < ny ? gy : 0;
        return (uint32_t)(gx + nx * gy);
    };
    auto plane = [&](int k) -> uint32_t { return (uint32_t)(k < 0 ? k + nz : (k >= nz ? k - nz : k)) * pl; };

    // this thread's one or two nodes of the ringed column: its own, and for the
    // first MP - 256 threads a ring node (rows below and above, then the sides)
    const bool ring = t < MP - 256;
    int rx = 0, ry = 0;
    if (ring) {
        if (t < 2 * MX) {
            rx = t % MX;
            ry = t < MX ? 0 : MY - 1;
        } else {
            const int s = t - 2 * MX;
            rx = s < TY ? 0 : MX - 1;
            ry = 1 + (s < TY ? s : s - TY);
        }
    }
    const int mi[2] = {(ly + 1) * MX + lx + 1, ry * MX + rx};              // in the ringed column
    const int pi[2] = {(ly + 2) * PX_ + lx + 2, (ry + 1) * PX_ + rx + 1};  // in the Psi plane
    const uint32_t mo[2] = {at_xy(lx, ly), at_xy(rx - 1, ry - 1)};         // in-plane node offsets
    uint32_t po[NP];
#pragma unroll
    for (int j = 0; j < NP; j++) {
        const int e = min(t + 256 * j, PP - 1);
        po[j] = at_xy(e % PX_ - 2, e / PX_ - 2);
    }
    const bool psi2 = t + 256 * (NP - 1) < PP;  // the last round is partial

    double pv[2][5], pp0[NP], pp1[NP];
    uint32_t pown[2] = {OWN_FLUID, OWN_FLUID};
    auto load_v = [&](int k) {
        const uint32_t z = plane(k);
#pragma unroll
        for (int r = 0; r < 2; r++) {
            if (r == 1 && !ring) break;
            const uint32_t b = (z + mo[r]) * 8u;
#pragma unroll
            for (int f = 0; f < 5; f++) pv[r][f] = *at(vin + (size_t)f * N, b);
        }
    };
    auto load_psi = [&](int k) {
        const uint32_t z = plane(k);
#pragma unroll
        for (int j = 0; j < NP; j++) {
            if (j == NP - 1 && !psi2) break;
            const uint32_t b = (z + po[j]) * 8u;
            pp0[j] = *at(vin + (size_t)5 * N, b);
            pp1[j] = *at(vin + (size_t)6 * N, b);
        }
    };
    auto put_psi = [&](int slot) {
#pragma unroll
        for (int j = 0; j < NP; j++) {
            if (j == NP - 1 && !psi2) break;
            s_psi[slot][0][t + 256 * j] = pp0[j];
            s_psi[slot][1][t + 256 * j] = pp1[j];
        }
    };
    auto load_own = [&](int k) {
        if constexpr (SOLID) {
            const uint32_t z = plane(k);
            pown[0] = owner[z + mo[0]];
            if (ring) pown[1] = owner[z + mo[1]];
        }
    };
    auto put_own = [&](int k) {
        if constexpr (SOLID) {
            s_own[k & 3][mi[0]] = pown[0];
            if (ring) s_own[k & 3][mi[1]] = pown[1];
        }
    };

    // planes before the loop: Psi zbeg - 2 .. zbeg, owners zbeg - 1 and zbeg
    for (int j = 0; j < 3; j++) {
        load_psi(zbeg - 2 + j);
        put_psi(j);
    }
    if constexpr (SOLID) {
        load_own(zbeg - 1);
        put_own(zbeg - 1);
        load_own(zbeg);
        put_own(zbeg);
    }
    load_v(zbeg - 1);

    const int c = mi[0];
    MomSum sum;               // of the node of plane k - 1, then of plane k
    sum.clear();
    MomSum ahead;             // without solids: of the node of plane k + 1, what leaves plane k
    ahead.clear();
    uint32_t mask = 0u;       // bit i: source n - c_i of the node is solid
    bool fluid = false;
    double b0[5], b1[5];      // its bounced populations from the plane above
    int sm = 0, s0 = 1, sp = 2;  // Psi slots of planes k - 1, k, k + 1
    for (int k = zbeg - 1; k <= zend; k++) {
        __syncthreads();
        // post-collision moments of plane k
        double(*mk)[MP] = s_m[SOLID ? k & 1 : 0];
#pragma unroll
        for (int r = 0; r < 2; r++) {
            if (r == 1 && !ring) break;
            if (SOLID && s_own[k & 3][mi[r]] != OWN_FLUID) continue;
            const int e = pi[r];
            double S0[3], S1[3];
            mom_psi_sums(
                [&](int i) {
                    const int slot = cz(i) == 0 ? s0 : (cz(i) > 0 ? sp : sm);
                    const int q = e + cy(i) * PX_ + cx(i);
                    return make_double2(s_psi[slot][0][q], s_psi[slot][1][q]);
                },
                S0, S1);
            Post A, B;
            collide_moments(bx, pv[r][0], pv[r][1], pv[r][2], pv[r][3], pv[r][4], s_psi[s0][0][e], s_psi[s0][1][e], S0,
                            S1, accv, A, B);
            const int m = mi[r];
            mk[0][m] = A.a;
            mk[1][m] = A.rho;
            mk[2][m] = A.ux;
            mk[3][m] = A.uy;
            mk[4][m] = A.uz;
            mk[5][m] = B.a;
            mk[6][m] = B.rho;
            mk[7][m] = B.ux;
            mk[8][m] = B.uy;
            mk[9][m] = B.uz;
        }
        // the next plane's loads, in flight while the populations are summed
        const bool more = k < zend;
        if (more) {
            load_v(k + 1);
            load_psi(k + 2);
            load_own(k + 2);
        }
        __syncthreads();

        double(*mb)[MP] = s_m[SOLID ? (k + 1) & 1 : 0];  // plane k - 1 (with solids)
        // both components' population i from the moments at position e of plane buffer m
        auto from = [&](double(*m)[MP], int e, int i, double& v0, double& v1) {
            v0 = pop_eq(i, m[0][e], m[1][e], i == 0 ? 0.0 : dir_dot<double>(i, m[2][e], m[3][e], m[4][e]));
            v1 = pop_eq(i, m[5][e], m[6][e], i == 0 ? 0.0 : dir_dot<double>(i, m[7][e], m[8][e], m[9][e]));
        };
        MomSum here = ahead;  // without solids: of the node of plane k
        if constexpr (!SOLID) {
            // each of the nine sources in plane k is read once, for the nodes of planes
            // k - 1, k and k + 1 that it streams to
            ahead.clear();
#pragma unroll
            for (int j = 0; j < 9; j++) {
                double v0, v1;
                const int ih = sum_dir(5 + j), e = c - cy(ih) * MX - cx(ih);
                if (j < 5) {
                    const int id = sum_dir(14 + j % 5), iu = sum_dir(j % 5);
                    from(mk, e, id, v0, v1);
                    sum.add(id, v0, v1);
                    from(mk, e, iu, v0, v1);
                    ahead.add(iu, v0, v1);
                }
                from(mk, e, ih, v0, v1);
                here.add(ih, v0, v1);
                // one source at a time: all nine read ahead cost more registers than
                // three waves per SIMD leave
                asm volatile("" : "+v"(here.d0), "+v"(here.d1), "+v"(here.jx), "+v"(here.jy), "+v"(here.jz),
                             "+v"(sum.d0), "+v"(sum.d1), "+v"(sum.jx), "+v"(sum.jy), "+v"(sum.jz), "+v"(ahead.d0),
                             "+v"(ahead.d1), "+v"(ahead.jx), "+v"(ahead.jy), "+v"(ahead.jz)
                             :
                             : "memory");
            }
        }
        // node of plane k - 1: the directions with c_iz = -1 come from plane k
        if (k > zbeg) {
#pragma unroll
            for (int j = 14; SOLID && j < Q; j++) {
                const int i = sum_dir(j);
                double v0, v1;
                from(mk, c - cy(i) * MX - cx(i), i, v0, v1);
                if ((mask >> i) & 1u) {
                    v0 = b0[j - 14];
                    v1 = b1[j - 14];
                }
                sum.add(i, v0, v1);
            }
            if (active) {
                double v[kMomPlanes];
                const bool wrong = finish_node(bx, sum, v);
                const uint32_t b = (plane(k - 1) + mo[0]) * 8u;
                if (SOLID && !fluid) {
#pragma unroll
                    for (int f = 0; f < kMomPlanes; f++) v[f] = 0.0;  // every line is written whole
                } else if (wrong) {
                    atomicOr(bad, 1);
                }
#pragma unroll
                for (int f = 0; f < kMomPlanes; f++) *atw(vout + (size_t)f * N, b) = v[f];
            }
        }
        if (SOLID && k >= zbeg && more) {
            // node of plane k: the directions with c_iz = +1 (from plane k - 1) and 0
            sum.clear();
            auto own_at = [&](int i) -> uint32_t { return s_own[(k - cz(i)) & 3][c - cy(i) * MX - cx(i)]; };
            uint32_t top = 0u;
            if constexpr (SOLID) {
                // codes plus one: 0 for fluid, so the largest tells whether any is solid
                fluid = active && s_own[k & 3][c] == OWN_FLUID;
#pragma unroll
                for (int i = 1; i < Q; i++) top = max(top, own_at(i) + 1u);
                top = fluid ? top : 0u;
            }
            mask = 0u;
            if (__ballot(top != 0u) == 0ull) {
#pragma unroll
                for (int j = 0; j < 14; j++) {
                    const int i = sum_dir(j);
                    double v0, v1;
                    from(cz(i) > 0 ? mb : mk, c - cy(i) * MX - cx(i), i, v0, v1);
                    sum.add(i, v0, v1);
                }
            } else if constexpr (SOLID) {
                // the links, and the bodies behind them (the walls count as one): the one
                // with the smallest code, the one with the largest, whether there are more
                uint32_t p1 = OWN_FLUID;
#pragma unroll
                for (int i = 1; i < Q; i++) {
                    const uint32_t o = own_at(i);
                    mask |= min(o + 1u, 1u) << i;
                    p1 = min(p1, o);
                }
                mask = fluid ? mask : 0u;
                asm("" : "+v"(mask));  // kept as bits: 18 lane masks would not fit the scalar registers
                p1 = fluid ? p1 : OWN_FLUID;
                const uint32_t p2 = top != 0u && top - 1u != p1 ? top - 1u : OWN_FLUID;
                const bool two = __ballot(p2 != OWN_FLUID) != 0ull;
                bool more_bodies = false;
                if (two) {
#pragma unroll
                    for (int i = 1; i < Q; i++) {
                        const uint32_t o = own_at(i);
                        more_bodies = more_bodies || (p2 != OWN_FLUID && o != OWN_FLUID && o != p1 && o != p2);
                    }
                }
                const int xyz[3] = {x, y, k}, Ls[3] = {nx, ny, nz};
                // surface velocity of body q at the node, and the node's cell in its records
                auto body = [&](uint32_t q, double(&U)[3], int& cb) {
                    cb = -1;
                    if (q == OWN_WALL) {
                        for (int d = 0; d < 3; d++) U[d] = bx.walls == 2 ? bx.uw[d] : 0.0;
                        return;
                    }
                    const double* pq = pfast + (size_t)q * kPF;
                    surface_velocity(bx, pq, x, y, k, U[0], U[1], U[2]);
                    cb = rec_cell(xyz, pq, Ls);
                };
                // U of body p (per lane, OWN_FLUID: none) for all lanes: the wave visits
                // the distinct bodies one at a time
                auto visit = [&](uint32_t p, double(&U)[3], int& cb) {
                    bool need = p != OWN_FLUID;
                    while (true) {
                        const unsigned long long w = __ballot(need);
                        if (w == 0ull) break;
                        const int lead = __ffsll(w) - 1;
                        const uint32_t q = __builtin_amdgcn_readfirstlane(__shfl(p, lead, 64));
                        double V[3];
                        int cq;
                        body(q, V, cq);
                        if (need && p == q) {
                            for (int d = 0; d < 3; d++) U[d] = V[d];
                            cb = cq;
                            need = false;
                        }
                    }
                };
                // population i of a link from the node's own f*_l (e0, e1), l = ibar, its
                // densities and the body's U; the momentum exchange goes to F
                auto link = [&](int i, double e0, double e1, double r0, double r1, const double(&U)[3], double(&F)[3],
                                double& v0, double& v1) {
                    const int l = opp(i);
                    const double C = bounce_c(l, U[0], U[1], U[2]);
                    const double C0 = C * r0, C1 = C * r1;
                    v0 = e0 + C0;
                    v1 = e1 + C1;
                    const double mag = 2.0 * (e0 + e1) + (C0 + C1);
                    if (cx(l) > 0) F[0] += mag;
                    if (cx(l) < 0) F[0] -= mag;
                    if (cy(l) > 0) F[1] += mag;
                    if (cy(l) < 0) F[1] -= mag;
                    if (cz(l) > 0) F[2] += mag;
                    if (cz(l) < 0) F[2] -= mag;
                };
                auto record = [&](uint32_t p, int cb, const double(&F)[3]) {
                    if (cb < 0) return;
                    double* r = rec + ((size_t)p * rstride + cb) * kRec;
                    for (int d = 0; d < 3; d++) r[d] = F[d];
                };
                // at most one body per node, or two
                auto sums = [&](auto how) {
                    constexpr bool TWO = decltype(how)::value;
                    double U1[3] = {0.0, 0.0, 0.0}, F1[3] = {0.0, 0.0, 0.0};
                    double U2[3] = {0.0, 0.0, 0.0}, F2[3] = {0.0, 0.0, 0.0};
                    int cb1 = -1, cb2 = -1;
                    visit(p1, U1, cb1);
                    if constexpr (TWO) visit(p2, U2, cb2);
                    auto hit_link = [&](int i, double e0, double e1, double r0, double r1, double& v0, double& v1) {
                        if (!TWO || own_at(i) == p1)
                            link(i, e0, e1, r0, r1, U1, F1, v0, v1);
                        else
                            link(i, e0, e1, r0, r1, U2, F2, v0, v1);
                    };
                    // a solid source is replaced by the node itself: its own moments, the
                    // opposite direction (s changes sign)
#pragma unroll
                    for (int j = 0; j < 14; j++) {
                        const int i = sum_dir(j);
                        const bool hit = (mask >> i) & 1u;
                        double(*m)[MP] = (cz(i) > 0 && !hit) ? mb : mk;
                        const int e = hit ? c : c - cy(i) * MX - cx(i);
                        double sa = 0.0, sb = 0.0;
                        if (i != 0) {
                            sa = dir_dot<double>(i, m[2][e], m[3][e], m[4][e]);
                            sb = dir_dot<double>(i, m[7][e], m[8][e], m[9][e]);
                            sa = hit ? -sa : sa;
                            sb = hit ? -sb : sb;
                        }
                        const double r0 = m[1][e], r1 = m[6][e];
                        double v0 = pop_eq(i, m[0][e], r0, sa), v1 = pop_eq(i, m[5][e], r1, sb);
                        if (i != 0 && hit) hit_link(i, v0, v1, r0, r1, v0, v1);
                        sum.add(i, v0, v1);
                    }
#pragma unroll
                    for (int j = 14; j < Q; j++) {
                        const int i = sum_dir(j);
                        if ((mask >> i) & 1u) {
                            double e0, e1;
                            from(mk, c, opp(i), e0, e1);
                            hit_link(i, e0, e1, mk[1][c], mk[6][c], b0[j - 14], b1[j - 14]);
                        }
                    }
                    record(p1, cb1, F1);
                    if constexpr (TWO) record(p2, cb2, F2);
                };
                if (__ballot(more_bodies) != 0ull) {
                    // some node touches three bodies or more: one direction at a time, its
                    // body read per lane and its record updated in place (this lane
                    // alone writes it, and it starts at zero)
#pragma unroll 1
                    for (int j = 0; j < Q; j++) {
                        const int i = sum_dir(j);
                        const bool hit = (mask >> i) & 1u;
                        double(*m)[MP] = (j < 5 && !hit) ? mb : mk;
                        const int e = hit ? c : c - cy(i) * MX - cx(i);
                        const double sg = hit ? -1.0 : 1.0;
                        const double dx = sg * cx(i), dy = sg * cy(i), dz = sg * cz(i), w = wq(i);
                        auto dot = [&](double a, double b, double z) { return (dx * a + dy * b) + dz * z; };
                        const double r0 = m[1][e], r1 = m[6][e];
                        const double sa = dot(m[2][e], m[3][e], m[4][e]), sb = dot(m[7][e], m[8][e], m[9][e]);
                        double v0 = w * fma_r(r0 * sa, fma_r(0.5, sa, 1.0), m[0][e]);
                        double v1 = w * fma_r(r1 * sb, fma_r(0.5, sb, 1.0), m[5][e]);
                        if (hit) {
                            const uint32_t o = own_at(i);
                            double U[3];
                            int cb;
                            body(o, U, cb);
                            const double C = -6.0 * w * dot(U[0], U[1], U[2]);
                            const double C0 = C * r0, C1 = C * r1;
                            const double mag = 2.0 * (v0 + v1) + (C0 + C1);
                            v0 = v0 + C0;
                            v1 = v1 + C1;
                            if (cb >= 0) {
                                double* r = rec + ((size_t)o * rstride + cb) * kRec;
                                r[0] += mag * dx;
                                r[1] += mag * dy;
                                r[2] += mag * dz;
                            }
                        }
                        if (j < 14) {
                            sum.d0 = sum.d0 + v0;
                            sum.d1 = sum.d1 + v1;
                            const double s = sg * (v0 + v1);  // (dx, dy, dz are those of the link where hit)
                            sum.jx = sum.jx + dx * s;
                            sum.jy = sum.jy + dy * s;
                            sum.jz = sum.jz + dz * s;
                        } else {
#pragma unroll
                            for (int q = 0; q < 5; q++) {
                                b0[q] = j == 14 + q ? v0 : b0[q];
                                b1[q] = j == 14 + q ? v1 : b1[q];
                            }
                        }
                    }
                } else if (!two) {
                    sums(std::false_type{});
                } else {
                    sums(std::true_type{});
                }
            }
        }
        if constexpr (!SOLID) sum = here;
        if (more) {
            put_psi(sm);  // plane k + 2 takes the slot of plane k - 1, read before the last barrier
            put_own(k + 2);
        }
        const int s = sm;
        sm = s0;
        s0 = sp;
        sp = s;
    }
}
// What the step leaves on record for a checkpoint (one thread per system), and
// the verdict on a state that was set instead of stepped to.
__device__ inline void begin_mstep(const Box& bx, int* __restrict__ status) {
    if (status[ST_FROM] != FROM_STEP && status[ST_BAD_START] != 0) atomicOr(status + ST_HEALTH, 1);
    status[ST_FROM] = FROM_STEP;
    double* acc = (double*)(status + ST_ACC);
    acc[0] = bx.ax;
    acc[1] = bx.ay;
    acc[2] = bx.az;
}
template <bool SOLID, int TX>
__global__ __launch_bounds__(256, SOLID ? 2 : 3) void k_mstep(Box bx, const double* __restrict__ vin, double* __restrict__ vout,
                                                  const uint32_t* __restrict__ owner, const double* __restrict__ pfast,
                                                  double* __restrict__ rec, int rstride, int* __restrict__ status,
                                                  int bad, int tiles_x, int tiles_y, int zc) {
    if (blockIdx.x == 0 && threadIdx.x == 0) begin_mstep(bx, status);
    mstep_body<SOLID, TX, 256 / TX>(bx, vin, vout, owner, pfast, rec, rstride, status + bad, tiles_x, tiles_y, zc,
                                    xcd_range(blockIdx.x, gridDim.x));
}
// Batched: item = (system, column); moment, owner and packed-particle copy c.
template <bool SOLID, int TX>
__global__ __launch_bounds__(256, SOLID ? 2 : 3) void k_mstep_batch(const SysDev* __restrict__ sd,
                                                        const WorkItem* __restrict__ items, int c, int zc) {
    const WorkItem w = items[xcd_range(blockIdx.x, gridDim.x)];
    const SysDev& d = sd[w.sys];
    if (w.local == 0 && threadIdx.x == 0) begin_mstep(d.box, d.health);
    mstep_body<SOLID, TX, 256 / TX>(d.box, d.mv[c], d.mv[1 - c], d.owner[c], d.pfast[c], d.rec,
                                    d.kext * d.kext * d.kext, d.health + ST_SUSPECT, d.tiles_x, d.tiles_y, zc, w.local);
}

// ---------------------------------------------------------------- conversions
// Moments from fields: every population of a fluid node is the equilibrium of its
// density at velocity u, of which the sums are kept, as of a filled node; its
// densities and velocity as given go to the other copy, v0, for a checkpoint that
// is taken before the first step. 140 B per node, where populations take 352, and 368
// more to sum them later.
__global__ __launch_bounds__(256) void k_mom_init(Box bx, const double* __restrict__ ra, const double* __restrict__ rb,
                                                  const double* __restrict__ u, const uint32_t* __restrict__ owner,
                                                  double* __restrict__ v, double* __restrict__ v0,
                                                  int* __restrict__ status) {
    const size_t N = (size_t)bx.N;
    const uint32_t n = blockIdx.x * 256u + threadIdx.x;
    if (n >= N) return;
    double out[kMomPlanes] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const double r0 = ra[n], r1 = rb[n];
    double un[3] = {0.0, 0.0, 0.0};
    if (u)
        for (int d = 0; d < 3; d++) un[d] = u[3 * (size_t)n + d];
    if (owner[n] == OWN_FLUID && fill_node(bx, r0, r1, un, out)) atomicOr(status + ST_BAD_START, 1);
#pragma unroll
    for (int p = 0; p < kMomPlanes; p++) v[(size_t)p * N + n] = out[p];
    v0[n] = r0;
    v0[N + n] = r1;
    for (int d = 0; d < 3; d++) v0[(2 + d) * N + n] = un[d];
}

// Moments from populations in plain form (a loaded state).
__global__ __launch_bounds__(256) void k_mom_from_pops(Box bx, const double* __restrict__ f,
                                                       const uint32_t* __restrict__ owner, double* __restrict__ v,
                                                       int* __restrict__ status) {
    const uint32_t N = (uint32_t)bx.N;
    const uint32_t n = blockIdx.x * 256u + threadIdx.x;
    if (n >= N) return;
    double out[kMomPlanes] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (owner[n] == OWN_FLUID) {
        MomSum m;
        m.clear();
#pragma unroll
        for (int k = 0; k < Q; k++) {
            const int i = sum_dir(k);
            m.add(i, f[(size_t)i * N + n], f[(size_t)(Q + i) * N + n]);
        }
        if (finish_node(bx, m, out)) atomicOr(status + ST_BAD_START, 1);
    }
#pragma unroll
    for (int p = 0; p < kMomPlanes; p++) v[(size_t)p * N + n] = out[p];
}

// Post-collision components of node (x, y, z) of moment copy v.
__device__ inline void post_at(const Box& bx, const double* __restrict__ v, int x, int y, int z,
                               const double (&acc)[3], Post& A, Post& B) {
    const size_t N = (size_t)bx.N;
    const size_t n = (size_t)x + (size_t)bx.nx * ((size_t)y + (size_t)bx.ny * z);
    double S0[3], S1[3];
    mom_psi_sums(
        [&](int i) {
            const size_t e = upstream(bx.nx, bx.ny, bx.nz, x, y, z, opp(i));  // n + c_i
            return make_double2(v[5 * N + e], v[6 * N + e]);
        },
        S0, S1);
    collide_moments(bx, v[n], v[N + n], v[2 * N + n], v[3 * N + n], v[4 * N + n], v[5 * N + n], v[6 * N + n], S0, S1,
                    acc, A, B);
}

// Populations of the current state in plain form, from the state one step
// before (moment copy v0, owner map o0, packed particles pf0, acceleration in the
// status words): each is formed as the step formed it for its sums. Nodes filled
// since then hold the equilibrium of the densities and velocity that kill / fill
// left in v0, and so do all nodes of a state set from fields. Populations that
// were loaded are there already, but for nodes that particles have covered since.
// Rare (checkpoints): nothing is staged. The directions are split over gridDim.y.
__global__ __launch_bounds__(256) void k_expand(Box bx, const double* __restrict__ v0, const uint32_t* __restrict__ o0,
                                                const uint32_t* __restrict__ o1, const double* __restrict__ pf0,
                                                const int* __restrict__ status, double* __restrict__ f) {
    const size_t N = (size_t)bx.N;
    const uint32_t n = blockIdx.x * 256u + threadIdx.x;
    if (n >= N) return;
    int x, y, z;
    node_xyz(bx, n, x, y, z);
    const int from = status[ST_FROM];
    const bool fluid = o1[n] == OWN_FLUID;
    if (from == FROM_POPS && fluid) return;
    const bool filled = fluid && (from == FROM_FIELDS || o0[n] != OWN_FLUID);
    const double* accp = (const double*)(status + ST_ACC);
    const double acc[3] = {accp[0], accp[1], accp[2]};
#pragma unroll 1
    for (int i = blockIdx.y; i < Q; i += gridDim.y) {
        double e0 = 0.0, e1 = 0.0;
        if (filled) {
            const double ux = v0[2 * N + n], uy = v0[3 * N + n], uz = v0[4 * N + n];
            e0 = pop_of(post_of(v0[n], ux, uy, uz), i);
            e1 = pop_of(post_of(v0[N + n], ux, uy, uz), i);
        } else if (fluid) {
            const uint32_t src = upstream(bx.nx, bx.ny, bx.nz, x, y, z, i);
            const uint32_t o = o0[src];
            Post A, B;
            int sx = x, sy = y, sz = z;
            if (o == OWN_FLUID) node_xyz(bx, src, sx, sy, sz);
            post_at(bx, v0, sx, sy, sz, acc, A, B);
            const int l = o == OWN_FLUID ? i : opp(i);
            e0 = pop_of(A, l);
            e1 = pop_of(B, l);
            if (o != OWN_FLUID) {
                double C = 0.0;
                if (o == OWN_WALL) {
                    if (bx.walls == 2) C = bounce_c(l, bx.uw[0], bx.uw[1], bx.uw[2]);
                } else {
                    double ux, uy, uz;
                    surface_velocity(bx, pf0 + (size_t)o * kPF, x, y, z, ux, uy, uz);
                    C = bounce_c(l, ux, uy, uz);
                }
                e0 = e0 + C * A.rho;
                e1 = e1 + C * B.rho;
            }
        }
        f[(size_t)i * N + n] = e0;
        f[(size_t)(Q + i) * N + n] = e1;
    }
}

// One block per system: the health check of a batched step (a lone handle's runs
// in its kill / fill pass). It clears the flag for the next step.
__global__ __launch_bounds__(256) void k_check_batch(const SysDev* __restrict__ sd, int c) {
    const SysDev& d = sd[blockIdx.x];
    if (!d.mom || d.health[ST_SUSPECT] == 0) return;
    check_suspect(d.box, d.mv[1 - c], d.owner[c], d.owner[1 - c], d.health + ST_SUSPECT, d.health, 0, 1);
    __syncthreads();
    if (threadIdx.x == 0) d.health[ST_SUSPECT] = 0;
}

// ---------------------------------------------------------------- readout
// Fields straight into the destination arrays (any may be null); a fluid node
// without fluid reads velocity 0.
__global__ __launch_bounds__(256) void k_mom_fields(Box bx, const double* __restrict__ v,
                                                    const uint32_t* __restrict__ owner, double* __restrict__ ra,
                                                    double* __restrict__ rb, double* __restrict__ u) {
    const int64_t N = bx.N;
    const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    const bool fluid = owner[n] == OWN_FLUID;
    const double r0 = fluid ? v[n] : 0.0, r1 = fluid ? v[N + n] : 0.0;
    if (ra) ra[n] = r0;
    if (rb) rb[n] = r1;
    if (u) {
        const bool has = fluid && r0 + r1 != 0.0;
        for (int d = 0; d < 3; d++) u[3 * n + d] = has ? v[(2 + d) * N + n] : 0.0;
    }
}

// Masses, momentum, fluid count and health of the fluid nodes: the partials
// of k_stats_final, fixed grid and order.
__global__ __launch_bounds__(256) void k_mom_stats(Box bx, const double* __restrict__ v,
                                                   const uint32_t* __restrict__ owner, double* __restrict__ red) {
    double acc[7] = {0, 0, 0, 0, 0, 0, 0}, tot[7];
    mom_stats_acc(bx, v, owner, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)gridDim.x * 256, acc);
    block_sum<7>(acc, tot);
    if (threadIdx.x == 0) {
        for (int k = 0; k < 6; k++) red[blockIdx.x * 8 + k] = tot[k];
        red[blockIdx.x * 8 + 6] = tot[6] > 0.0 ? 1.0 : 0.0;
    }
}

// ---------------------------------------------------------------- launchers
static inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

// Planes a block marches: the fewest rounds of resident blocks (two per CU with
// solids, three without) times the planes each works through (two more than it
// writes, and a start-up worth about one). Looked for once per box, over the
// values that ceil(nz / chunks) takes (some 2 sqrt(nz): going through every number of
// chunks took 3.9 ms at nz = 2^20).
int mstep_planes(int64_t columns, int nz, bool solids) {
    const int64_t resident = solids ? 512 : 768;
    int best = nz;
    double cost = 1e300;
    for (int zc = nz;; zc = (nz - 1) / ((nz + zc - 2) / (zc - 1)) + 1) {
        const int64_t blocks = columns * ((nz + zc - 1) / zc);
        const double c = (double)((blocks + resident - 1) / resident) * (zc + 3);
        if (c < cost) {
            cost = c;
            best = zc;
        }
        if (zc == 1) break;
    }
    return best;
}

// Where the state comes from, and no bad density in it so far.
__global__ void k_set_from(int* __restrict__ status, int from) {
    status[ST_FROM] = from;
    status[ST_BAD_START] = 0;
}
hipError_t launch_set_from(lb_handle* h, int from) {
    hipLaunchKernelGGL(k_set_from, dim3(1), dim3(1), 0, h->stream, h->b.health, from);
    return hipGetLastError();
}

hipError_t launch_mom_init(lb_handle* h, const double* ra, const double* rb, const double* u) {
    const hipError_t e = launch_set_from(h, FROM_FIELDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mom_init, dim3(nblk(h->box.N)), dim3(256), 0, h->stream, h->box, ra, rb, u,
                       h->b.owner[h->ocur], h->b.mv[h->mc], h->b.mv[1 - h->mc], h->b.health);
    return hipGetLastError();
}

hipError_t launch_mom_from_pops(lb_handle* h) {
    hipLaunchKernelGGL(k_mom_from_pops, dim3(nblk(h->box.N)), dim3(256), 0, h->stream, h->box,
                       (const double*)h->b.f[h->cur], h->b.owner[h->ocur], h->b.mv[h->mc], h->b.health);
    return hipGetLastError();
}

hipError_t launch_expand(lb_handle* h) {
    // a small box leaves most CUs idle with one thread per node, which works through
    // 19 chains of loads (16^3: a save took 240 us, 180 in populations)
    const unsigned nb = nblk(h->box.N);
    hipLaunchKernelGGL(k_expand, dim3(nb, nb < 1024 ? Q : 1), dim3(256), 0, h->stream, h->box, h->b.mv[1 - h->mc],
                       h->b.owner[h->oprev], h->b.owner[h->ocur], h->b.pfast[h->oprev], h->b.health,
                       (double*)h->b.f[h->cur]);
    return hipGetLastError();
}

hipError_t launch_mstep(lb_handle* h) {
    constexpr int W = kMomTileX;
    const int tx = (h->box.nx + W - 1) / W, ty = (h->box.ny + 256 / W - 1) / (256 / W);
    const int zc = h->zc[h->has_solid ? 1 : 0];
    const dim3 grid((unsigned)(tx * ty * ((h->box.nz + zc - 1) / zc)));
    const int ke = h->np > 0 ? kill_ext(h) : 0;
    const int bad = h->np > 0 ? ST_SUSPECT : ST_HEALTH;
    const double* vin = h->b.mv[h->mc];
    double* vout = h->b.mv[1 - h->mc];
    if (h->has_solid)
        hipLaunchKernelGGL((k_mstep<true, W>), grid, dim3(256), 0, h->stream, h->box, vin, vout, h->b.owner[h->ocur],
                           h->b.pfast[h->ocur], h->b.rec, ke * ke * ke, h->b.health, bad, tx, ty, zc);
    else
        hipLaunchKernelGGL((k_mstep<false, W>), grid, dim3(256), 0, h->stream, h->box, vin, vout, h->b.owner[h->ocur],
                           h->b.pfast[h->ocur], h->b.rec, 0, h->b.health, bad, tx, ty, zc);
    return hipGetLastError();
}

hipError_t launch_mom_fields(lb_handle* h, double* ra, double* rb, double* u) {
    hipLaunchKernelGGL(k_mom_fields, dim3(nblk(h->box.N)), dim3(256), 0, h->stream, h->box, h->b.mv[h->mc],
                       h->b.owner[h->ocur], ra, rb, u);
    return hipGetLastError();
}

hipError_t launch_mom_stats(lb_handle* h) {
    hipLaunchKernelGGL(k_mom_stats, dim3(kRedBlocks), dim3(256), 0, h->stream, h->box, h->b.mv[h->mc],
                       h->b.owner[h->ocur], h->b.red);
    return hipGetLastError();
}

// ---------------------------------------------------------------- batched
template <bool SOLID>
static void launch_batch_mstep_t(const BatchLaunch& bl, hipStream_t st, int c) {
    const int k = SOLID ? BI_MTILE : BI_MTILE_PLAIN, zc = bl.zc[SOLID ? 1 : 0];
    if (bl.n[k] == 0) return;
    const dim3 grid(bl.n[k]);
    if (bl.bx == 64)
        hipLaunchKernelGGL((k_mstep_batch<SOLID, 64>), grid, dim3(256), 0, st, bl.sys, bl.items[k], c, zc);
    else if (bl.bx == 32)
        hipLaunchKernelGGL((k_mstep_batch<SOLID, 32>), grid, dim3(256), 0, st, bl.sys, bl.items[k], c, zc);
    else
        hipLaunchKernelGGL((k_mstep_batch<SOLID, 16>), grid, dim3(256), 0, st, bl.sys, bl.items[k], c, zc);
}
hipError_t launch_batch_mstep(const BatchLaunch& bl, hipStream_t st, int c) {
    launch_batch_mstep_t<true>(bl, st, c);
    launch_batch_mstep_t<false>(bl, st, c);
    return hipGetLastError();
}
hipError_t launch_batch_check(const BatchLaunch& bl, int nsys, hipStream_t st, int c) {
    hipLaunchKernelGGL(k_check_batch, dim3(nsys), dim3(256), 0, st, bl.sys, c);
    return hipGetLastError();
}

}  // namespace lbe
