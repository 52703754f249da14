// lbm_kernels.h -- the fused collide-and-stream kernel and its helpers.
//
// Included by one translation unit per (Q, precision); each instantiates the
// launchers declared in lbm_internal.h.
//
// In-place streaming: the AA pattern (named in Sec. 2.3 of the paper as the
// single-array, thread-safe alternative to the two-population scheme).
// With h_i(x) the population of direction i at node x stored in slot i:
//   even step  : read slot i at x; collide; write h*_i to slot opp(i) at x.
//   odd step   : read h_i(x) from slot opp(i) at x - c_i; collide; write h*_i
//                to slot i at x + c_i.
// After an even step the array holds the next state "in reverse"; after the
// odd step it is back in natural layout.  Each (node, slot) is read and
// written by exactly one thread per step, so the update is race-free.
// Half-way bounce-back (Sec. 3 intro, after Ladd) closes the loop next to a
// non-fluid node y = x + c_i: the post-collision h*_i returns to node x as
// direction opp(i), minus 6 w_i rho0 (c_i . u_wall) for a moving wall; in
// the even step that value already sits in slot opp(i) at x (so the wall
// term is applied there), in the odd step it is written to slot opp(i) at x,
// and the odd step's read of direction i from a wall neighbour x - c_i
// takes slot i at x instead.
//
// Node update (Sec. 2.3 push-pull scheme): the Q populations of a node are
// pulled into registers, the tag selects the collision model among the
// compiled model set (BGK, TRT, BGK with Smagorinsky or the learned eddy
// viscosity, regularized BGK, regularized open boundaries), and the results
// are pushed back (slot addresses from pop_base / slot_off).  Populations are
// stored shifted, h_i = f_i - w_i rho0 (Sec. 3 intro, Skordos' offset
// stripping), which the collision is written for directly:
//   drho = sum h_i, rho = rho0 + drho, j = sum c_i h_i, u = (j + F/2) / rho
//   heq_i = w_i (drho + rho (3 c.u + 9/2 (c.u)^2 - 3/2 u.u))
// and the collision works on pairs (i, opp(i)) split into even and odd parts
// (TRT; BGK is the case omega- = omega+), with the Guo forcing term split
// the same way.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_device.h"
#include "lbm_internal.h"
#include "lbm_mlp_device.h"

namespace lbmd {

// Per-node neighbour mask layout.  Fluid node: bits 1..26 wall bits (bit i
// set when node x + c_i is not fluid), bit 27 set when a neighbour is a moving
// wall, bits 28..31 the node's own fluid tag.  Non-fluid node (tag bits 0):
// zero, or a filler (see the step kernel) with bit 0 set and bit i set when
// node x + (0, c_iy, c_iz) is not fluid.
constexpr uint32_t kMaskWalls = (1u << 27) - 1u;
constexpr int kMaskMovingBit = 27;
constexpr int kMaskTagShift = 28;

__device__ __forceinline__ int wrap_idx(int v, int n) { return v < 0 ? v + n : (v >= n ? v % n : v); }

// FP64 reduction terms of one node's loaded (time-t) populations, added to red.
template <int Q, typename C>
__device__ __forceinline__ void node_reduce(const C (&h)[Q], bool live, const StepParams &p, double (&red)[NRED]) {
    double dr = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        const double v = (double)h[i];
        dr += v;
        if constexpr (Vi::x != 0) jx += Vi::x * v;
        if constexpr (Vi::y != 0) jy += Vi::y * v;
        if constexpr (Vi::z != 0) jz += Vi::z * v;
    });
    const double rho = p.rho0 + dr;
    const double px = jx + 0.5 * p.force[0], py = jy + 0.5 * p.force[1], pz = jz + 0.5 * p.force[2];
    const double ux = px / rho, uy = py / rho, uz = pz / rho;
    const double uu = ux * ux + uy * uy + uz * uz;
    const bool ok = isfinite(rho) && isfinite(uu);
    const bool use = live && ok;
    red[0] += use ? dr : 0.0;
    red[1] += use ? px : 0.0;
    red[2] += use ? py : 0.0;
    red[3] += use ? pz : 0.0;
    red[4] += use ? ux : 0.0;
    red[5] += use ? uy : 0.0;
    red[6] += use ? uz : 0.0;
    red[7] += use ? 0.5 * uu : 0.0;
    red[8] += use ? 0.5 * rho * uu : 0.0;
    red[9] += (live && !ok) ? 1.0 : 0.0;
}

// Regularized open boundary on an x plane (the conditions of Latt et al. 2008
// the paper uses for the Berea runs, Sec. 3.3), shifted form: f_i = h_i + w_i rho0.
// On the x = 0 plane the populations with c_x = +1 come from outside, on
// x = nx-1 those with c_x = -1.  Mass and x-momentum over the known populations
// give, with s = -1 on x = 0 and s = +1 on x = nx-1,
//   rho (1 + s u_x) = sum_{c_x=0} f + 2 sum_{c_x=s} f = s0 + 2 s_s + rho0 = K
// (the weights of c_x = 0 plus twice those of c_x = s sum to 1): a velocity
// boundary (u imposed) has rho = K / (1 + s u_x), a pressure boundary (rho
// imposed, u_y = u_z = 0) has u_x = s (K / rho - 1).  Each unknown population
// is equilibrium plus its opposite's non-equilibrium part; the node is then
// regularized (Hermite projection of its momentum flux) and relaxed with omega.
// No body force on these nodes.
template <int Q, typename C>
__device__ __forceinline__ void open_boundary(const C (&h)[Q], int tag, const StepParams &p, C (&hs)[Q]) {
    const bool low = tag == LBM_TAG_VEL_IN || tag == LBM_TAG_PRES_IN;  // the x = 0 plane
    const bool vel = tag == LBM_TAG_VEL_IN || tag == LBM_TAG_VEL_OUT;  // velocity imposed
    C s0 = C(0), sp = C(0), sm = C(0);
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        if constexpr (Vi::x == 0) s0 += h[i];
        if constexpr (Vi::x > 0) sp += h[i];
        if constexpr (Vi::x < 0) sm += h[i];
    });
    const C rho0 = (C)p.rho0;
    const C sg = low ? C(-1) : C(1);
    const C K = s0 + C(2) * (low ? sm : sp) + rho0;
    C rb, ux, uy, uz;
    if (vel) {
        ux = (C)p.bc_u[0];
        uy = (C)p.bc_u[1];
        uz = (C)p.bc_u[2];
        rb = K / (C(1) + sg * ux);
    } else {
        rb = (C)p.bc_rho[low ? 0 : 1];
        ux = sg * (K / rb - C(1));
        uy = C(0);
        uz = C(0);
    }
    const C drb = rb - rho0;
    const C uu = ux * ux + uy * uy + uz * uz;
    C he[Q];
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        C cu = C(0);
        if constexpr (Vi::x != 0) cu += C(Vi::x) * ux;
        if constexpr (Vi::y != 0) cu += C(Vi::y) * uy;
        if constexpr (Vi::z != 0) cu += C(Vi::z) * uz;
        he[i] = C(Vi::w) * (drb + rb * (C(3) * cu + C(4.5) * cu * cu - C(1.5) * uu));
    });
    // non-equilibrium part of the completed node; an unknown population takes
    // its opposite's
    C pxx = C(0), pyy = C(0), pzz = C(0), pxy = C(0), pxz = C(0), pyz = C(0);
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        if constexpr (i > 0) {
            constexpr int o = Vi::opp;
            C ne = h[i] - he[i];
            if constexpr (Vi::x != 0) {
                const bool unknown = low ? (Vi::x > 0) : (Vi::x < 0);
                if (unknown) ne = h[o] - he[o];
            }
            if constexpr (Vi::x != 0) pxx += ne;
            if constexpr (Vi::y != 0) pyy += ne;
            if constexpr (Vi::z != 0) pzz += ne;
            if constexpr (Vi::x * Vi::y != 0) pxy += C(Vi::x * Vi::y) * ne;
            if constexpr (Vi::x * Vi::z != 0) pxz += C(Vi::x * Vi::z) * ne;
            if constexpr (Vi::y * Vi::z != 0) pyz += C(Vi::y * Vi::z) * ne;
        }
    });
    const C tr = (pxx + pyy + pzz) * C(1.0 / 3.0);
    const C a = (C(1) - (C)p.omega) * C(4.5);
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        C cpc = C(0);
        if constexpr (Vi::x != 0) cpc += pxx;
        if constexpr (Vi::y != 0) cpc += pyy;
        if constexpr (Vi::z != 0) cpc += pzz;
        if constexpr (Vi::x * Vi::y != 0) cpc += C(2 * Vi::x * Vi::y) * pxy;
        if constexpr (Vi::x * Vi::z != 0) cpc += C(2 * Vi::x * Vi::z) * pxz;
        if constexpr (Vi::y * Vi::z != 0) cpc += C(2 * Vi::y * Vi::z) * pyz;
        hs[i] = he[i] + a * C(Vi::w) * (cpc - tr);
    });
}

// A kernel parameter as the two-step kernel uses it.  FRESH ties it to a value of the
// node, so that what is computed from parameters alone (weights times forces and
// rates) is formed for each node and not kept in registers across the march over
// planes: there it is spilled, and its reload waits for the populations in flight.
template <bool FRESH, typename C>
__device__ __forceinline__ C node_param(double v, C h) {
    if constexpr (FRESH) asm("" : "+s"(v) : "v"(h));
    return (C)v;
}

// Collision of one node in shifted form (pair split, Guo forcing).  Every lane
// of the wave must call it (the learned closure is evaluated wave-wide).
// Regularized and recursive-regularized update for lattices whose fluid nodes
// all use one of those two models.  Both relax to a state built from the
// moments alone (rho, u and the non-equilibrium momentum flux), so the update
// needs the populations only for the moment sums: the flux comes from the
// second moment of h minus that of the equilibrium,
//   Pi_ab = sum c_a c_b h - drho / 3 delta_ab - rho u_a u_b
// (h = f - w rho0; the second-order equilibrium's second moment is
// rho / 3 delta + rho u u on D3Q19 and D3Q27), and the post-collision pair
// (k, k + H) is feq_k + F_k / 2 + the regularized (and third-order) terms,
// with the odd parts entering with opposite signs.  The same algebra as the
// general path with omega = 1 in its relaxation, where h cancels; only the
// rounding differs.  Keeping no population live across the update frees the
// registers the general path needs.
// Every product-sum is an explicit fused multiply-add and nothing else is fused, so
// the rounding does not depend on the kernel around it: steps in place and two at a
// time agree bit for bit.  The forms are those that FP64 and FP16 lattices always had,
// among them: untagged D3Q19 lattices add u.u, u.F and the cross terms of u and F from x
// on, all others from y on, and so do the even steps of FP16 lattices with two nodes a
// lane (pair), which fuse the odd equilibrium and not the force's term.  FORCE: as in
// collide_pairs.
// P: storage precision.  FP32 lattices sum the moments pair by pair: the second moments
// see only the even parts, ten times smaller in a flow at u = 0.05 than the odd ones that
// cancel in a plain sum.  Their error against FP64 (rms over 72 flows of 48^3 to 128^3
// nodes, 10 to 200 steps) is 0.966 (recursive) and 0.955 (regularized) times that of the
// general update below; with plain sums it was up to 1.06 times.
template <int Q, int P, typename C, int MS, bool TAGGED, bool FORCE, bool TWO>
__device__ __forceinline__ void collide_regularized(const C (&h)[Q], int tag, const StepParams &p, C (&hs)[Q],
                                                    bool pair) {
#pragma clang fp contract(off)
    constexpr int H = (Q - 1) / 2;
    constexpr bool RR = MS == MS_RR;
    auto fm = [](C a, C b, C c) { return __builtin_elementwise_fma(a, b, c); };
    C drho = C(0), jx = C(0), jy = C(0), jz = C(0);
    C sxx = C(0), syy = C(0), szz = C(0), sxy = C(0), sxz = C(0), syz = C(0);
    if constexpr (P == 1) {
        drho = h[0];
        sfor<H>([&](auto K) {
            constexpr int k = decltype(K)::value + 1;
            using Vk = V<Q, k>;
            const C e = h[k] + h[k + H], o = h[k] - h[k + H];
            drho += e;
            if constexpr (Vk::x != 0) jx += C(Vk::x) * o, sxx += e;
            if constexpr (Vk::y != 0) jy += C(Vk::y) * o, syy += e;
            if constexpr (Vk::z != 0) jz += C(Vk::z) * o, szz += e;
            if constexpr (Vk::x * Vk::y != 0) sxy += C(Vk::x * Vk::y) * e;
            if constexpr (Vk::x * Vk::z != 0) sxz += C(Vk::x * Vk::z) * e;
            if constexpr (Vk::y * Vk::z != 0) syz += C(Vk::y * Vk::z) * e;
        });
    } else {
        sfor<Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            using Vi = V<Q, i>;
            drho += h[i];
            if constexpr (Vi::x == 1) jx += h[i];
            if constexpr (Vi::x == -1) jx -= h[i];
            if constexpr (Vi::y == 1) jy += h[i];
            if constexpr (Vi::y == -1) jy -= h[i];
            if constexpr (Vi::z == 1) jz += h[i];
            if constexpr (Vi::z == -1) jz -= h[i];
            if constexpr (Vi::x != 0) sxx += h[i];
            if constexpr (Vi::y != 0) syy += h[i];
            if constexpr (Vi::z != 0) szz += h[i];
            if constexpr (Vi::x * Vi::y == 1) sxy += h[i];
            if constexpr (Vi::x * Vi::y == -1) sxy -= h[i];
            if constexpr (Vi::x * Vi::z == 1) sxz += h[i];
            if constexpr (Vi::x * Vi::z == -1) sxz -= h[i];
            if constexpr (Vi::y * Vi::z == 1) syz += h[i];
            if constexpr (Vi::y * Vi::z == -1) syz -= h[i];
        });
    }
    // (parameters formed anew where their products would spill: as in collide_pairs)
    auto par = [&](double v) { return node_param<TWO && (TAGGED || (FORCE && Q == 27))>(v, h[0]); };
    const C Fx = FORCE ? par(p.force[0]) : C(0), Fy = FORCE ? par(p.force[1]) : C(0), Fz = FORCE ? par(p.force[2]) : C(0);
    const C rho = par(p.rho0) + drho;
    const C inv_rho = C(1) / rho;
    C px = jx, py = jy, pz = jz;
    if constexpr (FORCE) px = fm(C(0.5), Fx, jx), py = fm(C(0.5), Fy, jy), pz = fm(C(0.5), Fz, jz);
    const C ux = px * inv_rho, uy = py * inv_rho, uz = pz * inv_rho;
    const bool from_x = Q == 19 && !TAGGED && !pair;
    const C uu = fm(uz, uz, from_x ? fm(uy, uy, ux * ux) : fm(ux, ux, uy * uy));
    C uF = C(0);
    if constexpr (FORCE) uF = fm(uz, Fz, from_x ? fm(uy, Fy, ux * Fx) : fm(ux, Fx, uy * Fy));
    auto cross = [&](C ua, C Fb, C ub, C Fa, bool from_a) {
#pragma clang fp contract(off)
        return from_a ? fm(ub, Fa, ua * Fb) : fm(ua, Fb, ub * Fa);
    };
    const C third = C(1.0 / 3.0);
    // Pi1 = Pi + (uF + Fu) / 2
    const C jux = rho * ux, juy = rho * uy, juz = rho * uz;
    C rxx = fm(-jux, ux, fm(-drho, third, sxx)), ryy = fm(-juy, uy, fm(-drho, third, syy));
    C rzz = fm(-juz, uz, fm(-drho, third, szz));
    C rxy = fm(-jux, uy, sxy), rxz = fm(-jux, uz, sxz), ryz = fm(-juy, uz, syz);
    if constexpr (FORCE) {
        rxx = fm(ux, Fx, rxx);
        ryy = fm(uy, Fy, ryy);
        rzz = fm(uz, Fz, rzz);
        rxy = fm(C(0.5), cross(ux, Fy, uy, Fx, from_x), rxy);
        rxz = fm(C(0.5), cross(ux, Fz, uz, Fx, from_x), rxz);
        ryz = fm(C(0.5), cross(uy, Fz, uz, Fy, from_x && !RR), ryz);
    }
    const C rsum = (rxx + ryy) + rzz;
    const C rtr = rsum * third;
    const bool on = tag == (RR ? LBM_TAG_RR : LBM_TAG_REG);
    const C om1 = C(1) - par(p.omega);
    const C reg = on ? om1 * C(4.5) : C(0);
    // third-order coefficients, each the product of t and its norm
    C t1p = C(0), t1m = C(0), t2p = C(0), t2m = C(0), t3p = C(0), t3m = C(0), t7 = C(0);
    constexpr double np_ = Q == 19 ? 27.0 / 2.0 : 27.0 / 4.0;  // 1 / norm of a sum
    constexpr double nm_ = Q == 19 ? 27.0 / 6.0 : 27.0 / 4.0;  // 1 / norm of a difference
    if constexpr (RR) {
        // A2 = (1 - omega) dev Pi1, A3 recursive, T = rho u u u + A3
        const C axx = om1 * fm(-rsum, third, rxx), ayy = om1 * fm(-rsum, third, ryy), azz = om1 * fm(-rsum, third, rzz);
        const C axy = om1 * rxy, axz = om1 * rxz, ayz = om1 * ryz;
        const C x2 = ux + ux, y2 = uy + uy, z2 = uz + uz;
        const C juxy = jux * uy;
        const C txxy = fm(uy, axx, fm(jux * ux, uy, x2 * axy));
        const C tyzz = fm(z2, ayz, fm(juy * uz, uz, uy * azz));
        const C txzz = fm(z2, axz, fm(jux * uz, uz, ux * azz));
        const C txyy = fm(y2, axy, fm(juxy, uy, ux * ayy));
        const C tyyz = fm(uz, ayy, fm(juy * uy, uz, y2 * ayz));
        const C txxz = fm(uz, axx, fm(jux * ux, uz, x2 * axz));
        const C g = on ? C(1) : C(0);
        t1p = g * (txxy + tyzz);
        t1m = g * (txxy - tyzz);
        t2p = g * (txzz + txyy);
        t2m = g * (txzz - txyy);
        t3p = g * (tyyz + txxz);
        t3m = g * (tyyz - txxz);
        if constexpr (Q == 27) t7 = g * fm(uz, axy, fm(uy, axz, fm(juxy, uz, ux * ayz)));
    }

    // rest population: regularized keeps the trace term, recursive relaxes it with 1
    C r0 = fm(C(-1.5) * rho, uu, drho);
    if constexpr (FORCE) r0 = fm(C(-1.5), uF, r0);
    if constexpr (RR) hs[0] = C(V<Q, 0>::w) * r0;
    else hs[0] = fm(C(V<Q, 0>::w), r0, -((reg * C(V<Q, 0>::w)) * rtr));
    sfor<H>([&](auto K) {
#pragma clang fp contract(off)
        constexpr int k = decltype(K)::value + 1;
        using Vk = V<Q, k>;
        C cu = C(0), cF = C(0), cpc = C(0);
        if constexpr (Vk::x != 0) cu = C(Vk::x) * ux, cF += C(Vk::x) * Fx, cpc += rxx;
        if constexpr (Vk::y != 0) {
            cu = Vk::x == 0 ? C(Vk::y) * uy : fm(C(Vk::y) * py, inv_rho, cu);
            cF += C(Vk::y) * Fy, cpc += ryy;
        }
        if constexpr (Vk::z != 0) {
            cu = Vk::x == 0 && Vk::y == 0 ? C(Vk::z) * uz : fm(C(Vk::z) * pz, inv_rho, cu);
            cF += C(Vk::z) * Fz, cpc += rzz;
        }
        if constexpr (Vk::x * Vk::y != 0) cpc = fm(C(2 * Vk::x * Vk::y), rxy, cpc);
        if constexpr (Vk::x * Vk::z != 0) cpc = fm(C(2 * Vk::x * Vk::z), rxz, cpc);
        if constexpr (Vk::y * Vk::z != 0) cpc = fm(C(2 * Vk::y * Vk::z), ryz, cpc);
        C ev = C(Vk::w) * fm(rho, fm(cu, C(4.5) * cu, C(-1.5) * uu), drho);
        C B = ((C(Vk::w) * C(3)) * rho) * cu;
        if constexpr (FORCE) {
            ev = fm(C(0.5), C(Vk::w) * fm(cF, C(9) * cu, C(-3) * uF), ev);
            const C Fo = (C(Vk::w) * C(3)) * cF;
            B = pair ? fm((C(Vk::w) * C(3)) * rho, cu, C(0.5) * Fo) : fm(C(0.5), Fo, B);
        }
        // regularized: |c|^2 -> 1 (tr Q = 0 projection); recursive: |c|^2 (deviatoric)
        constexpr int nt = RR ? Vk::n2 : 1;
        const C dev = nt == 1 ? fm(-rsum, third, cpc) : fm(-rtr, C(nt), cpc);
        const C A = fm(reg * C(Vk::w), dev, ev);
        if constexpr (RR) {
            constexpr int cx = Vk::x, cy = Vk::y, cz = Vk::z;
            C E = C(0);
            // E += p norm t, p a polynomial of c_k: of its two products the one with p is fused,
            // or, where p is 1 or -1, the one with the norm
            auto add = [&](double p, double norm, C t) {
#pragma clang fp contract(off)
                if (p == 1.0 || p == -1.0) E = fm(C(p) * t, C(norm), E);
                else if (p != 0.0) E = fm(C(p), t * C(norm), E);
            };
            add(cy * (cx * cx + cz * cz - 2.0 / 3.0), np_, t1p);
            add(cy * (cx * cx - cz * cz), nm_, t1m);
            add(cx * (cy * cy + cz * cz - 2.0 / 3.0), np_, t2p);
            add(cx * (cz * cz - cy * cy), nm_, t2m);
            add(cz * (cx * cx + cy * cy - 2.0 / 3.0), np_, t3p);
            add(cz * (cy * cy - cx * cx), nm_, t3m);
            if constexpr (Q == 27) add(cx * cy * cz, 27.0, t7);
            B = fm(E, C(Vk::w), B);
        }
        hs[k] = A + B;
        hs[k + H] = A - B;
    });
}

// BGK with a per-node relaxation time from the eddy-viscosity closure (tag
// BGK+MLP), from Smagorinsky (tag BGK+Smagorinsky, and the closure's
// fallback) or the plain one (tag BGK), for lattices whose fluid nodes use
// only these three models.  The non-equilibrium momentum flux comes from the
// second moment of h minus that of the second-order equilibrium (dRho/3 I +
// rho u u, exact on D3Q19 and D3Q27), and the network is evaluated before the
// equilibrium is formed, pair by pair where it is used: only the populations
// and a few moments are live across the matrix-core products.
template <int Q, typename C, int MS>
__device__ __forceinline__ void collide_closure(const C (&h)[Q], int tag, bool live, const StepParams &p,
                                                C (&hs)[Q]) {
    constexpr int H = (Q - 1) / 2;
    // moments from the pair sums and differences (the second moments see only
    // the even parts, the momentum only the odd ones)
    C drho = h[0], jx = C(0), jy = C(0), jz = C(0);
    C sxx = C(0), syy = C(0), szz = C(0), sxy = C(0), sxz = C(0), syz = C(0);
    C E[H + 1], O[H + 1];  // pair halves (h_k + h_k') / 2 and (h_k - h_k') / 2; h is not used again
    sfor<H>([&](auto K) {
        constexpr int k = decltype(K)::value + 1;
        using Vk = V<Q, k>;
        const C e = h[k] + h[k + H], o = h[k] - h[k + H];
        E[k] = C(0.5) * e;
        O[k] = C(0.5) * o;
        drho += e;
        if constexpr (Vk::x != 0) jx += C(Vk::x) * o, sxx += e;
        if constexpr (Vk::y != 0) jy += C(Vk::y) * o, syy += e;
        if constexpr (Vk::z != 0) jz += C(Vk::z) * o, szz += e;
        if constexpr (Vk::x * Vk::y != 0) sxy += C(Vk::x * Vk::y) * e;
        if constexpr (Vk::x * Vk::z != 0) sxz += C(Vk::x * Vk::z) * e;
        if constexpr (Vk::y * Vk::z != 0) syz += C(Vk::y * Vk::z) * e;
    });
    const C Fx = (C)p.force[0], Fy = (C)p.force[1], Fz = (C)p.force[2];
    const C rho = (C)p.rho0 + drho;
    const C inv_rho = C(1) / rho;
    const C ux = (jx + C(0.5) * Fx) * inv_rho;
    const C uy = (jy + C(0.5) * Fy) * inv_rho;
    const C uz = (jz + C(0.5) * Fz) * inv_rho;
    const C d3 = drho * C(1.0 / 3.0);
    const C pxx = sxx - d3 - rho * ux * ux, pyy = syy - d3 - rho * uy * uy, pzz = szz - d3 - rho * uz * uz;
    const C pxy = sxy - rho * ux * uy, pxz = sxz - rho * ux * uz, pyz = syz - rho * uy * uz;

    const C qn = sqrt(pxx * pxx + pyy * pyy + pzz * pzz + C(2) * (pxy * pxy + pxz * pxz + pyz * pyz));
    const C tau0 = (C)p.tau;
    C tau_eff = C(0.5) * (tau0 + sqrt(tau0 * tau0 + (C)p.smag_c * qn * inv_rho));
    const bool want = live && tag == LBM_TAG_BGK_MLP;
    if (p.has_mlp && __any(want)) {
        const float feat[7] = {(float)pxx, (float)pyy, (float)pzz, (float)pxy, (float)pxz, (float)pyz, (float)rho};
        const float sp = mlp_wave_eval(p.mlp, feat);
        const C nu0 = (C)p.nu0;
        const C nut = nu0 * (C)sp;
        if (want && isfinite(nut) && nut <= C(10) * nu0) tau_eff = C(3) * (nu0 + nut) + C(0.5);
    }
    const C w = (tag == LBM_TAG_BGK_SMAG || tag == LBM_TAG_BGK_MLP) ? C(1) / tau_eff : (C)p.omega;

    const C uu = ux * ux + uy * uy + uz * uz;
    const C uF = ux * Fx + uy * Fy + uz * Fz;
    const C g = C(1) - C(0.5) * w;
    hs[0] = h[0] - w * (h[0] - C(V<Q, 0>::w) * (drho - C(1.5) * rho * uu)) + g * C(V<Q, 0>::w) * C(-3) * uF;
    sfor<H>([&](auto K) {
        constexpr int k = decltype(K)::value + 1;
        using Vk = V<Q, k>;
        C cu = C(0), cF = C(0);
        if constexpr (Vk::x != 0) cu += C(Vk::x) * ux, cF += C(Vk::x) * Fx;
        if constexpr (Vk::y != 0) cu += C(Vk::y) * uy, cF += C(Vk::y) * Fy;
        if constexpr (Vk::z != 0) cu += C(Vk::z) * uz, cF += C(Vk::z) * Fz;
        const C ev = C(Vk::w) * (drho + rho * (C(4.5) * cu * cu - C(1.5) * uu));
        const C od = C(Vk::w) * C(3) * rho * cu;
        const C Fe = C(Vk::w) * (C(9) * cu * cF - C(3) * uF);
        const C Fo = C(Vk::w) * C(3) * cF;
        const C hp = E[k], hm = O[k];
        const C A = g * Fe - w * (hp - ev);
        const C B = g * Fo - w * (hm - od);
        hs[k] = (hp + hm) + A + B;
        hs[k + H] = (hp - hm) + A - B;
    });
}

// BGK, BGK + Smagorinsky and two-relaxation-time updates for lattices whose fluid
// nodes use only these, pair by pair: h* = h - omega+ (even part of h - heq) -+
// omega- (odd part), plus the Guo terms.  The same sums and products, in the same
// order and fused the same way, as the general update above compiles to in FP32;
// every product-sum here is an explicit fused multiply-add, so the rounding does
// not depend on the kernel around it (steps in place and two at a time agree bit
// for bit).  FORCE: the Guo terms are compiled in.  Without a body force they are
// exactly zero, so both forms give the same result.  TAGGED: untagged D3Q19 BGK and
// TRT lattices add u.u and u.F from x on, all others from y on (the order their
// kernels always had), and so do the even steps of FP16 lattices with two nodes a
// lane (pair).
template <int Q, typename C, int MS, bool TAGGED, bool FORCE, bool TWO>
__device__ __forceinline__ void collide_pairs(const C (&h)[Q], int tag, const StepParams &p, C (&hs)[Q], bool pair) {
    constexpr int H = (Q - 1) / 2;
    auto fm = [](C a, C b, C c) { return __builtin_elementwise_fma(a, b, c); };
    C drho = C(0), px = C(0), py = C(0), pz = C(0);
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        drho += h[i];
        if constexpr (Vi::x == 1) px += h[i];
        if constexpr (Vi::x == -1) px -= h[i];
        if constexpr (Vi::y == 1) py += h[i];
        if constexpr (Vi::y == -1) py -= h[i];
        if constexpr (Vi::z == 1) pz += h[i];
        if constexpr (Vi::z == -1) pz -= h[i];
    });
    // Untagged kernels have the registers, but for the force's on D3Q27.  256 x 256 x 200
    // Smagorinsky with a force, us a step, one step a pass / kept / formed anew: D3Q27 periodic
    // FP32 525 / 1015 / 356, FP64 1026 / 1528 / 692, cavity FP32 560 / 1240 / 462; D3Q19 cavity
    // FP32 384 / 432 / 310
    auto par = [&](double v) { return node_param<TWO && (TAGGED || (FORCE && Q == 27))>(v, h[0]); };
    const C Fx = FORCE ? par(p.force[0]) : C(0), Fy = FORCE ? par(p.force[1]) : C(0), Fz = FORCE ? par(p.force[2]) : C(0);
    const C rho = par(p.rho0) + drho;
    C inv_rho = C(1) / rho;
    if constexpr (FORCE) {
        px = fm(C(0.5), Fx, px);
        py = fm(C(0.5), Fy, py);
        pz = fm(C(0.5), Fz, pz);
    }
    const C ux = px * inv_rho, uy = py * inv_rho, uz = pz * inv_rho;
    constexpr bool kFromX = Q == 19 && !TAGGED && (MS == MS_BGK || MS == MS_TRT);
    const C uu = fm(uz, uz, kFromX && !pair ? fm(uy, uy, ux * ux) : fm(ux, ux, uy * uy));
    C uu15 = C(-1.5) * uu;
    // c.u and the even part of the equilibrium of pair k
    auto cu_of = [&](auto K) {
        using Vk = V<Q, decltype(K)::value>;
        C cu = C(0);
        if constexpr (Vk::x != 0) cu = C(Vk::x) * ux;
        if constexpr (Vk::y != 0) cu = Vk::x == 0 ? C(Vk::y) * uy : fm(C(Vk::y) * py, inv_rho, cu);
        if constexpr (Vk::z != 0) cu = Vk::x == 0 && Vk::y == 0 ? C(Vk::z) * uz : fm(C(Vk::z) * pz, inv_rho, cu);
        return cu;
    };
    auto ev_of = [&](auto K, C cu) {
        return C(V<Q, decltype(K)::value>::w) * fm(rho, fm(cu, C(4.5) * cu, uu15), drho);
    };
    C wp = par(p.omega), wm = wp;
    if constexpr ((MS & MS_TRT) != 0) {
        if (tag == LBM_TAG_TRT) wm = par(p.omega_minus);
    }
    if constexpr ((MS & MS_SMAG) != 0) {
        C pxx = C(0), pyy = C(0), pzz = C(0), pxy = C(0), pxz = C(0), pyz = C(0);
        sfor<H>([&](auto K) {
            constexpr int k = decltype(K)::value + 1;
            using Vk = V<Q, k>;
            const std::integral_constant<int, k> kc{};
            const C ne = fm(C(-2), ev_of(kc, cu_of(kc)), h[k] + h[k + H]);
            if constexpr (Vk::x != 0) pxx += ne;
            if constexpr (Vk::y != 0) pyy += ne;
            if constexpr (Vk::z != 0) pzz += ne;
            if constexpr (Vk::x * Vk::y != 0) pxy += C(Vk::x * Vk::y) * ne;
            if constexpr (Vk::x * Vk::z != 0) pxz += C(Vk::x * Vk::z) * ne;
            if constexpr (Vk::y * Vk::z != 0) pyz += C(Vk::y * Vk::z) * ne;
        });
        const C qn = sqrt(fm(C(2), fm(pyz, pyz, fm(pxy, pxy, pxz * pxz)), fm(pzz, pzz, fm(pxx, pxx, pyy * pyy))));
        const C tau0 = par(p.tau);
        const C tau_s = C(0.5) * (tau0 + sqrt(fm(tau0, tau0, (qn * par(p.smag_c)) * inv_rho)));
        if (tag == LBM_TAG_BGK_SMAG) {
            wp = C(1) / tau_s;
            wm = wp;
        }
    }
    // in the two-step kernel, whose registers are short: form the equilibria again
    // rather than keep them from the momentum flux
    if constexpr (TWO && (TAGGED || !FORCE || Q == 27) && (MS & MS_SMAG) != 0) asm("" : "+v"(inv_rho), "+v"(uu15));
    hs[0] = fm(-fm(C(-V<Q, 0>::w), fm(C(-1.5) * rho, uu, drho), h[0]), wp, h[0]);
    C gp = C(0), gm = C(0), uF3 = C(0);
    if constexpr (FORCE) {
        gp = fm(wp, C(-0.5), C(1));
        gm = fm(wm, C(-0.5), C(1));
        const C uF = fm(uz, Fz, kFromX ? fm(uy, Fy, ux * Fx) : fm(ux, Fx, uy * Fy));
        uF3 = C(-3) * uF;
        hs[0] = fm(gp, C(-3.0 * V<Q, 0>::w) * uF, hs[0]);
    }
    sfor<H>([&](auto K) {
#pragma clang fp contract(off)  // A and B are rounded before they are added
        constexpr int k = decltype(K)::value + 1;
        using Vk = V<Q, k>;
        const std::integral_constant<int, k> kc{};
        const C cu = cu_of(kc);
        const C ev = ev_of(kc, cu);
        const C od = (C(3.0 * Vk::w) * rho) * cu;
        C A = -(fm(h[k] + h[k + H], C(0.5), -ev) * wp);
        C B = -(fm(h[k] - h[k + H], C(0.5), -od) * wm);
        if constexpr (FORCE) {
            C cF = C(0);
            if constexpr (Vk::x != 0) cF += C(Vk::x) * Fx;
            if constexpr (Vk::y != 0) cF += C(Vk::y) * Fy;
            if constexpr (Vk::z != 0) cF += C(Vk::z) * Fz;
            A = fm(gp, C(Vk::w) * fm(cF, C(9) * cu, uF3), A);
            B = fm(C(3.0 * Vk::w) * cF, gm, B);
        }
        hs[k] = (h[k] + A) + B;
        hs[k + H] = (h[k + H] + A) - B;
    });
}

// Regularized / recursive-regularized lattices take the moment-only update
// (collide_regularized).
// P: storage precision; TWO: in the two-step kernel; pair: with the rounding of the even
// step with two nodes a lane.
template <int Q, int P, typename C, int MS, bool TAGGED, bool FORCE = true, bool TWO = false>
__device__ __forceinline__ void collide_node(const C (&h)[Q], int tag, bool live, const StepParams &p, C (&hs)[Q],
                                             bool pair = false) {
    if constexpr (MS == MS_STREAM) {
        // collision switched off: the step only streams (and bounces back)
        sfor<Q>([&](auto I) { hs[decltype(I)::value] = h[decltype(I)::value]; });
        return;
    }
    if constexpr (MS == MS_REG || MS == MS_RR) {
        collide_regularized<Q, P, C, MS, TAGGED, FORCE, TWO>(h, tag, p, hs, pair);
        return;
    }
    // FP32 and FP16 lattices a step at a time keep the general update below: the same bits
    // as collide_pairs, and the compiler's own order is the faster one there (us a step, this
    // / collide_pairs: 64^3 D3Q19 FP32 TRT cavity 9.9 / 10.5, 101^3 D3Q27 FP32 TRT with a force
    // 34.7 / 36.3, FP16 TRT 23.0 / 25.8); in FP64 the slower one (101^3 D3Q19 BGK cavity 1.09)
    if constexpr ((P == 0 || TWO) && (MS == MS_BGK || MS == MS_TRT || MS == (MS_BGK | MS_SMAG))) {
        collide_pairs<Q, C, MS, TAGGED, FORCE, TWO>(h, tag, p, hs, pair);
        return;
    }
    if constexpr (MS == (MS_BGK | MS_SMAG | MS_MLP)) {
        collide_closure<Q, C, MS>(h, tag, live, p, hs);
        return;
    }
    constexpr int H = (Q - 1) / 2;
    C drho = C(0), jx = C(0), jy = C(0), jz = C(0);
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        drho += h[i];
        if constexpr (Vi::x == 1) jx += h[i];
        if constexpr (Vi::x == -1) jx -= h[i];
        if constexpr (Vi::y == 1) jy += h[i];
        if constexpr (Vi::y == -1) jy -= h[i];
        if constexpr (Vi::z == 1) jz += h[i];
        if constexpr (Vi::z == -1) jz -= h[i];
    });
    const C Fx = (C)p.force[0], Fy = (C)p.force[1], Fz = (C)p.force[2];
    const C rho = (C)p.rho0 + drho;
    const C inv_rho = C(1) / rho;
    const C ux = (jx + C(0.5) * Fx) * inv_rho;
    const C uy = (jy + C(0.5) * Fy) * inv_rho;
    const C uz = (jz + C(0.5) * Fz) * inv_rho;
    const C uu = ux * ux + uy * uy + uz * uz;
    const C uF = ux * Fx + uy * Fy + uz * Fz;

    // equilibrium, even/odd parts per pair k = 1..H (direction k, opposite k+H)
    C ev[H + 1], od[H + 1], cuk[H + 1];
    ev[0] = C(V<Q, 0>::w) * (drho - C(1.5) * rho * uu);
    od[0] = C(0);
    cuk[0] = C(0);
    sfor<H>([&](auto K) {
        constexpr int k = decltype(K)::value + 1;
        using Vk = V<Q, k>;
        C cu = C(0);
        if constexpr (Vk::x != 0) cu += C(Vk::x) * ux;
        if constexpr (Vk::y != 0) cu += C(Vk::y) * uy;
        if constexpr (Vk::z != 0) cu += C(Vk::z) * uz;
        cuk[k] = cu;
        ev[k] = C(Vk::w) * (drho + rho * (C(4.5) * cu * cu - C(1.5) * uu));
        od[k] = C(Vk::w) * C(3) * rho * cu;
    });

    // relaxation rates from the node's model
    C wp = (C)p.omega, wm = (C)p.omega;
    if constexpr ((MS & MS_TRT) != 0) {
        if (tag == LBM_TAG_TRT) wm = (C)p.omega_minus;
    }
    // Pi_ab = sum c_a c_b (h - heq): only even parts contribute.
    C pxx = C(0), pyy = C(0), pzz = C(0), pxy = C(0), pxz = C(0), pyz = C(0);
    if constexpr ((MS & (MS_SMAG | MS_MLP | MS_REG | MS_RR)) != 0) {
        sfor<H>([&](auto K) {
            constexpr int k = decltype(K)::value + 1;
            using Vk = V<Q, k>;
            const C ne = (h[k] + h[k + H]) - C(2) * ev[k];
            if constexpr (Vk::x != 0) pxx += ne;
            if constexpr (Vk::y != 0) pyy += ne;
            if constexpr (Vk::z != 0) pzz += ne;
            if constexpr (Vk::x * Vk::y != 0) pxy += C(Vk::x * Vk::y) * ne;
            if constexpr (Vk::x * Vk::z != 0) pxz += C(Vk::x * Vk::z) * ne;
            if constexpr (Vk::y * Vk::z != 0) pyz += C(Vk::y * Vk::z) * ne;
        });
    }
    if constexpr ((MS & (MS_SMAG | MS_MLP)) != 0) {
        const C qn = sqrt(pxx * pxx + pyy * pyy + pzz * pzz + C(2) * (pxy * pxy + pxz * pxz + pyz * pyz));
        const C tau0 = (C)p.tau;
        const C tau_s = C(0.5) * (tau0 + sqrt(tau0 * tau0 + (C)p.smag_c * qn * inv_rho));
        C tau_eff = tau_s;
        if constexpr ((MS & MS_MLP) != 0) {
            const bool want = live && tag == LBM_TAG_BGK_MLP;
            if (p.has_mlp && __any(want)) {
                const float feat[7] = {(float)pxx, (float)pyy, (float)pzz, (float)pxy,
                                       (float)pxz, (float)pyz, (float)rho};
                const float sp = mlp_wave_eval(p.mlp, feat);
                const C nu0 = (C)p.nu0;
                const C nut = nu0 * (C)sp;
                if (isfinite(nut) && nut <= C(10) * nu0) {
                    if (tag == LBM_TAG_BGK_MLP) tau_eff = C(3) * (nu0 + nut) + C(0.5);
                }
            }
        }
        if (tag == LBM_TAG_BGK_SMAG || tag == LBM_TAG_BGK_MLP) {
            wp = C(1) / tau_eff;
            wm = wp;
        }
    }

    // Regularized BGK (second-order Hermite projection of the first-order
    // non-equilibrium part, Guo forcing).  The populations read
    // f = feq + f1 - F_i/2, f1 having the momentum flux Pi1 = Pi + (uF + Fu)/2;
    // relaxing feq + w_i Q_i:Pi1 / (2 cs^4) - F_i/2 gives
    //   f*_i = feq_i + (1 - omega) w_i (9/2) (c_i.Pi1.c_i - tr Pi1 / 3) + F_i / 2,
    // which is the omega = 1 update below (A, B) plus the regularized term added
    // to the even part of each pair.
    // Recursive regularized (the paper's RR model, Sec. 3.1-3.2): the same with
    // the deviatoric part of Pi1 only (bulk relaxation 1), i.e. the even term
    // (1 - omega) w_i (9/2) (c_i.Pi1.c_i - |c_i|^2 tr Pi1 / 3), plus the odd
    // third-order Hermite term of T = rho u u u + A3, A3 the recursive
    // non-equilibrium coefficient A3_abc = u_a A2_bc + u_b A2_ac + u_c A2_ab of
    // A2 = (1 - omega) dev Pi1.  Third-order polynomials: the sums and
    // differences of H_xxy and H_yzz, H_xzz and H_xyy, H_yyz and H_xxz
    // (orthogonal on D3Q19 and D3Q27) and, on D3Q27, H_xyz; each projected with
    // its lattice norm (D3Q19: 2/27 for sums, 6/27 for differences; D3Q27: 4/27,
    // and 1/27 for H_xyz).
    C reg = C(0);      // (1 - omega) * 9/2 on regularized nodes, else 0
    C trm = C(1);      // 1 (regularized) or 0 (recursive: its trace is relaxed with 1)
    bool rr = false;   // recursive regularized node
    C rxx = C(0), ryy = C(0), rzz = C(0), rxy = C(0), rxz = C(0), ryz = C(0), rtr = C(0);
    C t1p = C(0), t1m = C(0), t2p = C(0), t2m = C(0), t3p = C(0), t3m = C(0), t7 = C(0);
    if constexpr ((MS & (MS_REG | MS_RR)) != 0) {
        if constexpr ((MS & MS_REG) != 0) {
            if (tag == LBM_TAG_REG) {
                reg = (C(1) - (C)p.omega) * C(4.5);
                wp = C(1);
                wm = C(1);
            }
        }
        if constexpr ((MS & MS_RR) != 0) {
            if (tag == LBM_TAG_RR) {
                reg = (C(1) - (C)p.omega) * C(4.5);
                trm = C(0);
                rr = true;
                wp = C(1);
                wm = C(1);
            }
        }
        rxx = pxx + ux * Fx;
        ryy = pyy + uy * Fy;
        rzz = pzz + uz * Fz;
        rxy = pxy + C(0.5) * (ux * Fy + uy * Fx);
        rxz = pxz + C(0.5) * (ux * Fz + uz * Fx);
        ryz = pyz + C(0.5) * (uy * Fz + uz * Fy);
        rtr = (rxx + ryy + rzz) * C(1.0 / 3.0);
        if constexpr ((MS & MS_RR) != 0) {
            // A2 = (1 - omega) dev Pi1, A3 recursive, T = rho u u u + A3
            const C om1 = C(1) - (C)p.omega;
            const C axx = om1 * (rxx - rtr), ayy = om1 * (ryy - rtr), azz = om1 * (rzz - rtr);
            const C axy = om1 * rxy, axz = om1 * rxz, ayz = om1 * ryz;
            const C txxy = rho * ux * ux * uy + C(2) * ux * axy + uy * axx;
            const C tyzz = rho * uy * uz * uz + uy * azz + C(2) * uz * ayz;
            const C txzz = rho * ux * uz * uz + ux * azz + C(2) * uz * axz;
            const C txyy = rho * ux * uy * uy + ux * ayy + C(2) * uy * axy;
            const C tyyz = rho * uy * uy * uz + C(2) * uy * ayz + uz * ayy;
            const C txxz = rho * ux * ux * uz + C(2) * ux * axz + uz * axx;
            constexpr double np_ = Q == 19 ? 27.0 / 2.0 : 27.0 / 4.0;  // 1 / norm of a sum
            constexpr double nm_ = Q == 19 ? 27.0 / 6.0 : 27.0 / 4.0;  // 1 / norm of a difference
            t1p = (txxy + tyzz) * C(np_);
            t1m = (txxy - tyzz) * C(nm_);
            t2p = (txzz + txyy) * C(np_);
            t2m = (txzz - txyy) * C(nm_);
            t3p = (tyyz + txxz) * C(np_);
            t3m = (tyyz - txxz) * C(nm_);
            if constexpr (Q == 27) t7 = (rho * ux * uy * uz + ux * ayz + uy * axz + uz * axy) * C(27.0);
        }
    }

    const C gp = C(1) - C(0.5) * wp, gm = C(1) - C(0.5) * wm;
    const C F0 = C(V<Q, 0>::w) * C(-3) * uF;
    hs[0] = h[0] - wp * (h[0] - ev[0]) + gp * F0;
    if constexpr ((MS & (MS_REG | MS_RR)) != 0) hs[0] -= reg * C(V<Q, 0>::w) * rtr * trm;
    sfor<H>([&](auto K) {
        constexpr int k = decltype(K)::value + 1;
        using Vk = V<Q, k>;
        C cF = C(0);
        if constexpr (Vk::x != 0) cF += C(Vk::x) * Fx;
        if constexpr (Vk::y != 0) cF += C(Vk::y) * Fy;
        if constexpr (Vk::z != 0) cF += C(Vk::z) * Fz;
        const C Fe = C(Vk::w) * (C(9) * cuk[k] * cF - C(3) * uF);
        const C Fo = C(Vk::w) * C(3) * cF;
        const C hp = C(0.5) * (h[k] + h[k + H]);
        const C hm = C(0.5) * (h[k] - h[k + H]);
        C A = gp * Fe - wp * (hp - ev[k]);
        const C B = gm * Fo - wm * (hm - od[k]);
        C Bx = B;
        if constexpr ((MS & (MS_REG | MS_RR)) != 0) {
            C cpc = C(0);  // c_k . Pi1 . c_k
            if constexpr (Vk::x != 0) cpc += rxx;
            if constexpr (Vk::y != 0) cpc += ryy;
            if constexpr (Vk::z != 0) cpc += rzz;
            if constexpr (Vk::x * Vk::y != 0) cpc += C(2 * Vk::x * Vk::y) * rxy;
            if constexpr (Vk::x * Vk::z != 0) cpc += C(2 * Vk::x * Vk::z) * rxz;
            if constexpr (Vk::y * Vk::z != 0) cpc += C(2 * Vk::y * Vk::z) * ryz;
            // regularized: |c|^2 -> 1 (tr Q = 0 projection); recursive: |c|^2 (deviatoric)
            const C cc = trm + (C(1) - trm) * C(Vk::n2);
            A += reg * C(Vk::w) * (cpc - rtr * cc);
        }
        if constexpr ((MS & MS_RR) != 0) {
            // odd third-order Hermite term (both equilibrium and non-equilibrium)
            constexpr int cx = Vk::x, cy = Vk::y, cz = Vk::z;
            constexpr double p1p = cy * (cx * cx + cz * cz - 2.0 / 3.0), p1m = cy * (cx * cx - cz * cz);
            constexpr double p2p = cx * (cy * cy + cz * cz - 2.0 / 3.0), p2m = cx * (cz * cz - cy * cy);
            constexpr double p3p = cz * (cx * cx + cy * cy - 2.0 / 3.0), p3m = cz * (cy * cy - cx * cx);
            constexpr double p7 = cx * cy * cz;
            C e3 = C(0);
            if constexpr (p1p != 0.0) e3 += C(p1p) * t1p;
            if constexpr (p1m != 0.0) e3 += C(p1m) * t1m;
            if constexpr (p2p != 0.0) e3 += C(p2p) * t2p;
            if constexpr (p2m != 0.0) e3 += C(p2m) * t2m;
            if constexpr (p3p != 0.0) e3 += C(p3p) * t3p;
            if constexpr (p3m != 0.0) e3 += C(p3m) * t3m;
            if constexpr (Q == 27 && p7 != 0.0) e3 += C(p7) * t7;
            if (rr) Bx += C(Vk::w) * e3;
        }
        hs[k] = h[k] + A + Bx;
        hs[k + H] = h[k + H] + A - Bx;
    });

    if constexpr ((MS & MS_OPEN) != 0) {
        if (tag >= LBM_TAG_VEL_IN && tag <= LBM_TAG_VEL_OUT) open_boundary<Q, C>(h, tag, p, hs);
    }
}

// The fused collide-and-stream step: one thread per node, 256-thread blocks
// covering a tile of (1 << tx_log2) x (256 >> tx_log2) nodes of one z-plane.
// Wall handling selects addresses rather than branching around loads, so the
// Q loads of a thread are all in flight together.
template <int Q, int P, int MS, bool TAGGED, int MODE, int PARITY, int ADDR>
__global__ __launch_bounds__(256) void k_collide_stream(StepParams p) {
    using S = typename Prec<P>::S;
    using C = typename Prec<P>::C;
    // ADDR 0: row layout, node-form addresses; 1: row layout, row-form
    // addresses; 2: brick layout (tagged kernels), node-form addresses; 3: brick
    // layout, 32-bit byte offsets into an array below 4 GiB
    constexpr bool ROWS = ADDR == 1;
    constexpr bool BRICK = ADDR >= 2;
    constexpr bool B32 = ADDR == 3;

    // XCD-aware tile order: hardware deals workgroups round-robin over the 8
    // XCDs, so workgroup w runs on XCD w % 8; give each XCD a contiguous run
    // of tiles (whole z-slabs) so neighbouring rows share that XCD's L2.
    const int wg = blockIdx.x;
    const int L = (wg & 7) * p.tiles_per_xcd + (wg >> 3);
    if (L >= p.n_tiles) return;  // uniform for the block

    const int nx = p.nx, ny = p.ny, nz = p.nz;
    int x, y, z;
    bool brick_none = false;  // brick layout: a padding wave past the last listed brick
    int xo[3], yo[3], zo[3];  // storage-index terms of the neighbours, index 1 + c for c in {-1, 0, 1}
    if constexpr (!BRICK) {
        // row layout: a tile of (1 << tx_log2) x (256 >> tx_log2) nodes of one plane
        const int txl = p.tx_log2;
        const int TX = 1 << txl, TY = 256 >> txl;
        const int tix = L % p.tiles_x;
        const int rem = L / p.tiles_x;
        const int tiy = rem % p.tiles_y;
        z = rem / p.tiles_y;
        x = (tix << txl) + (threadIdx.x & (TX - 1));
        y = tiy * TY + (threadIdx.x >> txl);
        // neighbour offsets with periodic wrap
        const bool in = (x < nx) && (y < ny);
        const int xc = in ? x : 0, yc = in ? y : 0;
        xo[0] = xc == 0 ? nx - 1 : xc - 1, xo[1] = xc, xo[2] = xc + 1 == nx ? 0 : xc + 1;
        yo[0] = (yc == 0 ? ny - 1 : yc - 1) * nx, yo[1] = yc * nx, yo[2] = (yc + 1 == ny ? 0 : yc + 1) * nx;
        const int nxy = nx * ny;
        zo[0] = (z == 0 ? nz - 1 : z - 1) * nxy, zo[1] = z * nxy, zo[2] = (z + 1 == nz ? 0 : z + 1) * nxy;
    } else {
        // brick layout: wave w of tile L updates the brick listed at [L][w] (the
        // bricks that hold fluid, in storage order, so solid rock launches no
        // wave), lane l the node (l % 4, l / 4 % 4, l / 16) of that brick; brick
        // b is brick b % 64 of 16^3 block b / 64 (every axis a multiple of 16)
        typedef const __attribute__((address_space(4))) int const_int;
        const int l = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int b = ((const_int *)p.tile_tag)[L * 4 + wave];
        brick_none = b < 0;
        const int bb = brick_none ? 0 : b;
        const int blk = bb >> 6, bib = bb & 63;
        const Layout &ly = p.lay;
        const int bz = blk / ly.nbxy, brem = blk - bz * ly.nbxy;
        const int by = brem / ly.nbx, bx = brem - by * ly.nbx;
        x = bx * 16 + (bib & 3) * 4 + (l & 3);
        y = by * 16 + ((bib >> 2) & 3) * 4 + ((l >> 2) & 3);
        z = bz * 16 + (bib >> 4) * 4 + (l >> 4);
        xo[0] = ly.x(x == 0 ? nx - 1 : x - 1), xo[1] = ly.x(x), xo[2] = ly.x(x + 1 == nx ? 0 : x + 1);
        yo[0] = ly.y(y == 0 ? ny - 1 : y - 1), yo[1] = ly.y(y), yo[2] = ly.y(y + 1 == ny ? 0 : y + 1);
        zo[0] = ly.z(z == 0 ? nz - 1 : z - 1), zo[1] = ly.z(z), zo[2] = ly.z(z + 1 == nz ? 0 : z + 1);
    }
    // B32: population 0 of a neighbour is at byte px + py + pz (the three terms of a
    // storage index share no bit within a block, so pop_base is additive in them)
    unsigned px[3] = {}, py[3] = {}, pz[3] = {};
    if constexpr (B32) {
        auto bytes = [](int s) {
            return ((__umul24((unsigned)s >> kBlockLog2, (unsigned)Q) << kBlockLog2) + ((unsigned)s & (kBlockNodes - 1))) *
                   (unsigned)sizeof(S);
        };
#pragma unroll
        for (int k = 0; k < 3; ++k) px[k] = bytes(xo[k]), py[k] = bytes(yo[k]), pz[k] = bytes(zo[k]);
    }
    const bool active = (x < nx) && (y < ny);
    const int n = zo[1] + yo[1] + xo[1];  // storage index of the node

    // Node class.  Waves whose 64 nodes and their one-node halo are a single
    // fluid model (the interior of a walled domain) need nothing; waves with no
    // fluid or filler node (solid rock) skip the update; the other waves read
    // each node's precomputed neighbour mask (wave-uniform branches).
    S *__restrict__ f = static_cast<S *>(p.pops);
    const long long pb = pop_base<Q>(n);
    int tag = p.uniform_tag;
    uint32_t wall = 0;   // bit i: node x + c_i is not fluid
    bool moving = false; // some neighbour is a moving wall
    bool plain = !TAGGED;
    bool skip = false;
    if constexpr (TAGGED) {
        // wave-uniform entry read through the constant address space (scalar load)
        typedef const __attribute__((address_space(4))) int const_int;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int tile_tag = BRICK ? (brick_none ? -1 : 0) : ((const_int *)p.tile_tag)[L * 4 + wave];
        if (tile_tag > 0) {
            tag = tile_tag;
            plain = true;
        } else if (tile_tag < 0) {
            tag = 0;
            skip = true;
        } else {
            const uint32_t m = active ? p.mask[n] : 0u;
            wall = m & kMaskWalls;
            moving = (m >> kMaskMovingBit) & 1u;
            tag = (int)(m >> kMaskTagShift);
        }
    }
    const bool live = active && (!TAGGED || tag != 0);
    // Filler stores.  A non-fluid node that shares a 64-byte storage sector with
    // fluid nodes stores into slots no fluid node reads or writes, so that the
    // sectors the step writes are written whole instead of partially (partial
    // sectors cost the memory a read-modify-write): in the even step its own
    // slots; in the odd step slot i of node x + (0, c_iy, c_iz) when that node
    // is not fluid (the row the wave's other lanes write for direction i).
    // Its loaded values are zero and its stored values are never read.
    const bool filler = TAGGED && active && tag == 0 && (wall & 1u);

    double red[NRED];
    if constexpr (MODE != MODE_STEP) {
#pragma unroll
        for (int k = 0; k < NRED; ++k) red[k] = 0.0;
    }

    // The node update with either of two address forms.  Row form (ROWS
    // variants; which waves use it is chosen below): whole rows tile the
    // 4096-node blocks and the tile is at least a wave wide (the host checks
    // both), so the wave's 64 nodes lie in one row and each population row it
    // reads or writes starts at a wave-uniform address: a scalar base plus the
    // lane's x offset, no per-lane 64-bit address arithmetic (wall waves
    // select per lane between two such addresses).  Node form: every address
    // computed per node, with wall selection.
    auto update = [&](auto rows_c, auto walls_c) {
        constexpr bool RF = decltype(rows_c)::value;     // row form
        constexpr bool WALLS = decltype(walls_c)::value; // wall, filler and moving-wall code
        // row form: population 0 at x = 0 of row (y + dy, z + dz), index [1 + dz][1 + dy],
        // and the lane's byte offsets of x - 1, x, x + 1 (periodic)
        const S *rp[3][3] = {};
        unsigned xb[3] = {0u, 0u, 0u};
        if constexpr (RF) {
            const int ys = __builtin_amdgcn_readfirstlane(y);
            const int yv[3] = {ys == 0 ? ny - 1 : ys - 1, ys, ys + 1 == ny ? 0 : ys + 1};
            const int zv[3] = {z == 0 ? nz - 1 : z - 1, z, z + 1 == nz ? 0 : z + 1};
            const int rl = p.row_log2;
            sfor<3>([&](auto DZ) {
                sfor<3>([&](auto DY) {
                    constexpr int dz = decltype(DZ)::value, dy = decltype(DY)::value;
                    if (PARITY == 1 || (dz == 1 && dy == 1)) {
                        const int r = zv[dz] * ny + yv[dy];
                        rp[dz][dy] = f + (long long)(r >> rl) * (long long)(Q << kBlockLog2) +
                                     (long long)((r & ((1 << rl) - 1)) * nx);
                    }
                });
            });
#pragma unroll
            for (int k = 0; k < 3; ++k) xb[k] = (unsigned)xo[k] * (unsigned)sizeof(S);
        }
        // Slot base in scalar registers (wave-uniform: the row bases derive from
        // the wave's row; the empty asm keeps the compiler from re-associating
        // the slot offset into per-lane 64-bit adds), plus the lane's 32-bit
        // offset: one global access with a scalar base.
        typedef __attribute__((address_space(1))) S gS;
        typedef __attribute__((address_space(1))) char gchar;
        auto at = [&](const S *row, int slot, unsigned xoff) -> gS * {
            gS *b = (gS *)(row + slot_off(slot));
            asm("" : "+s"(b));
            return (gS *)((gchar *)b + xoff);
        };
        // B32: the node's byte offset, that of slot i at x + (dx, dy, dz) (offsets 1 + d),
        // and a select by a mask bit without a compare
        const unsigned pn = pz[1] + py[1] + px[1];
        auto nb32 = [&](int dz, int dy, int dx, int slot) {
            return pz[1 + dz] + py[1 + dy] + px[1 + dx] + (unsigned)(slot << kBlockLog2) * (unsigned)sizeof(S);
        };
        auto own32 = [&](int slot) { return pn + (unsigned)(slot << kBlockLog2) * (unsigned)sizeof(S); };
        auto pick32 = [&](int bit, unsigned set, unsigned clear) {
            const unsigned m = (unsigned)((int)(wall << (31 - bit)) >> 31);
            return (set & m) | (clear & ~m);
        };
        auto at32 = [&](unsigned off) { return (gS *)((gchar *)f + off); };

        // ---- pull the node's populations.  The registers are zeroed first and the
        // loads sit in a branch with no else: a divergent else that overwrote
        // registers with loads in flight would force a wait on those loads.
        C h[Q];
        sfor<Q>([&](auto I) { h[decltype(I)::value] = C(0); });
        if (live) {
            sfor<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                using Vi = V<Q, i>;
                if constexpr (RF) {
                    if constexpr (PARITY == 0 || i == 0) {
                        h[i] = (C)*at(rp[1][1], i, xb[1]);
                    } else {
                        gS *a = at(rp[1 - Vi::z][1 - Vi::y], Vi::opp, xb[1 - Vi::x]);
                        if constexpr (WALLS) {
                            // a wall at x - c_i: the node's own slot i instead
                            gS *own = at(rp[1][1], i, xb[1]);
                            a = ((wall >> Vi::opp) & 1u) ? own : a;
                        }
                        h[i] = (C)*a;
                    }
                } else if constexpr (B32) {
                    if constexpr (PARITY == 0 || i == 0)
                        h[i] = (C)*at(f, i, pn);
                    else
                        h[i] = (C)*at32(pick32(Vi::opp, own32(i), nb32(-Vi::z, -Vi::y, -Vi::x, Vi::opp)));
                } else {
                    long long off;
                    if constexpr (PARITY == 0 || i == 0) {
                        off = pb + slot_off(i);
                    } else {
                        // direction i arrives from x - c_i (slot opp), or from the node's
                        // own slot i when x - c_i is a wall
                        const long long o_nb =
                            pop_base<Q>(zo[1 - Vi::z] + yo[1 - Vi::y] + xo[1 - Vi::x]) + slot_off(Vi::opp);
                        if constexpr (TAGGED) {
                            off = ((wall >> Vi::opp) & 1u) ? pb + slot_off(i) : o_nb;
                        } else {
                            off = o_nb;
                        }
                    }
                    h[i] = (C)f[off];
                }
            });
        }

        if constexpr (MODE != MODE_STEP) node_reduce<Q, C>(h, live, p, red);

        if constexpr (MODE != MODE_REDUCE) {
            C hs[Q];
            collide_node<Q, P, C, MS, TAGGED>(h, tag, live, p, hs);

            // moving-wall term where x + c_i is a moving wall (nodes next to one only)
            if constexpr (TAGGED && WALLS) {
                if (moving) {
                    sfor<Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        using Vi = V<Q, i>;
                        if constexpr (i > 0) {
                            if ((wall >> i) & 1u) {
                                int dst;
                                if constexpr (B32) {
                                    // from the byte offset: three terms to keep, not six
                                    const unsigned e = nb32(Vi::z, Vi::y, Vi::x, 0) / (unsigned)sizeof(S);
                                    dst = (int)(((e >> kBlockLog2) / (unsigned)Q << kBlockLog2) |
                                                (e & (kBlockNodes - 1)));
                                } else {
                                    dst = zo[1 + Vi::z] + yo[1 + Vi::y] + xo[1 + Vi::x];
                                }
                                const int t = p.tags[dst];
                                if (t >= LBM_TAG_WALL0) {
                                    const double *uw = p.wall_u + 3 * (t - LBM_TAG_WALL0);
                                    C cu = C(0);
                                    if constexpr (Vi::x != 0) cu += C(Vi::x) * (C)uw[0];
                                    if constexpr (Vi::y != 0) cu += C(Vi::y) * (C)uw[1];
                                    if constexpr (Vi::z != 0) cu += C(Vi::z) * (C)uw[2];
                                    hs[i] -= C(6.0 * Vi::w) * (C)p.rho0 * cu;
                                }
                            }
                        }
                    });
                }
            }

            // ---- push
            if constexpr (RF) {
                if (live || (WALLS && filler)) {
                    sfor<Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        using Vi = V<Q, i>;
                        if constexpr (i == 0) {
                            *at(rp[1][1], 0, xb[1]) = (S)hs[0];
                        } else if constexpr (PARITY == 0) {
                            *at(rp[1][1], Vi::opp, xb[1]) = (S)hs[i];
                        } else if constexpr (!WALLS) {
                            *at(rp[1 + Vi::z][1 + Vi::y], i, xb[1 + Vi::x]) = (S)hs[i];
                        } else {
                            // a wall at x + c_i: back to the node's own slot opp(i), or
                            // (filler) slot i of x + (0, c_iy, c_iz)
                            gS *a = at(rp[1 + Vi::z][1 + Vi::y], i, xb[1 + Vi::x]);
                            const bool wi = (wall >> i) & 1u;
                            gS *alt = live ? at(rp[1][1], Vi::opp, xb[1]) : at(rp[1 + Vi::z][1 + Vi::y], i, xb[1]);
                            a = wi ? alt : a;
                            if (live || wi) *a = (S)hs[i];
                        }
                    });
                }
            } else if constexpr (B32) {
                if (live || filler) *at(f, 0, pn) = (S)hs[0];
                // the push forms its addresses anew: kept from the pull, the sums hold 14 to
                // 18 registers across the collision
                if constexpr (PARITY == 1) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) asm("" : "+v"(px[k]), "+v"(py[k]), "+v"(pz[k]));
                }
                // (no odd-step fillers in this layout: its own slots written as well left
                // 0.3 instead of 1.5 million of the 6.4 million sector writes partial,
                // and the step where it was, 188.9 us against 188.8)
                if (live || (PARITY == 0 && filler))
                    sfor<Q - 1>([&](auto I) {
                        constexpr int i = 1 + decltype(I)::value;
                        using Vi = V<Q, i>;
                        if constexpr (PARITY == 0)
                            *at(f, Vi::opp, pn) = (S)hs[i];
                        else
                            *at32(pick32(i, own32(Vi::opp), nb32(Vi::z, Vi::y, Vi::x, i))) = (S)hs[i];
                    });
            } else if (live || filler) {
                sfor<Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    using Vi = V<Q, i>;
                    long long off;
                    bool ok = true;
                    if constexpr (i == 0) {
                        off = pb;
                    } else if constexpr (PARITY == 0) {
                        // even step: h*_i goes to slot opp(i) of the node itself
                        off = pb + slot_off(Vi::opp);
                    } else {
                        // odd step: h*_i goes to slot i of x + c_i, or back to slot
                        // opp(i) of the node itself when x + c_i is a wall
                        off = pop_base<Q>(zo[1 + Vi::z] + yo[1 + Vi::y] + xo[1 + Vi::x]) + slot_off(i);
                        if constexpr (TAGGED) {
                            const bool wi = (wall >> i) & 1u;
                            if (wi) off = live ? pb + slot_off(Vi::opp)
                                               : pop_base<Q>(zo[1 + Vi::z] + yo[1 + Vi::y] + xo[1]) + slot_off(i);
                            ok = live || wi;
                        }
                    }
                    if (ok) f[off] = (S)hs[i];
                });
            }
        }
    };
    using yes = std::true_type;
    using no = std::false_type;
    if constexpr (ROWS && !TAGGED) {
        update(yes{}, no{});
    } else if (skip) {
        // no fluid or filler node: nothing to load, update or store
    } else if constexpr (ROWS && P == 2) {
        if (plain) update(yes{}, no{});
        else update(yes{}, yes{});
    } else if constexpr (ROWS) {
        if (plain) update(no{}, yes{});
        else update(yes{}, yes{});
    } else {
        update(no{}, std::integral_constant<bool, TAGGED>{});
    }

    // ---- per-tile reduction partials (fixed order: shuffle tree, then waves 0..3)
    if constexpr (MODE != MODE_STEP) {
        __shared__ double s_red[4][NRED];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int k = 0; k < NRED; ++k) {
            double v = red[k];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if (lane == 0) s_red[wave][k] = v;
        }
        __syncthreads();
        if (threadIdx.x < NRED) {
            const int k = threadIdx.x;
            p.partials[(long long)k * p.partial_stride + L] = (s_red[0][k] + s_red[1][k]) + (s_red[2][k] + s_red[3][k]);
        }
    }
}

// ---- FP16 storage, two nodes per lane (even step)
//
// Lattices of one fluid model without walls (untagged), stored in FP16, whose
// rows of 128..4096 nodes tile the 4096-node blocks.  Wave w of tile L updates
// the 128-node row segment 4 L + w, lane l its nodes x0 = 2 l and x0 + 1 from
// the segment start, reading and writing each population row with aligned
// 4-byte accesses (a wave moves 256 contiguous bytes per row instead of 128).
// The even step only: every access stays at the nodes themselves (an odd step
// in this form, its x-shifted rows combined across lanes with DPP shifts, ran
// slower than the one-node odd step at two waves per SIMD).  The node update is
// the one-node code run twice; where the compiler shares a product between the
// two nodes it may fuse one multiply-add fewer, so a rare population differs
// from the one-node kernels' by one FP16 rounding.
__device__ __forceinline__ float half_lo(uint32_t v) {
    return (float)__builtin_bit_cast(_Float16, (unsigned short)(v & 0xffffu));
}
__device__ __forceinline__ float half_hi(uint32_t v) { return (float)__builtin_bit_cast(_Float16, (unsigned short)(v >> 16)); }
__device__ __forceinline__ uint32_t half_bits(float v) { return (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)v); }

template <int Q, int MS>
__global__ __launch_bounds__(256) void k_collide_pair_even(StepParams p) {
    using C = float;
    // tiles of four segments, dealt to the XCDs in contiguous runs (as k_collide_stream)
    const int n_tiles = (p.n_segs + 3) >> 2;
    const int per_xcd = (n_tiles + 7) >> 3;
    const int wg = blockIdx.x;
    const int L = (wg & 7) * per_xcd + (wg >> 3);
    if (L >= n_tiles) return;  // uniform for the block
    const int sg = L * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (sg >= p.n_segs) return;  // uniform for the wave (the last tile may be short)
    const int lane = threadIdx.x & 63;
    const int nx = p.nx;
    const long long s0 = (long long)sg * 128;  // natural index of the segment's first node
    const int nxl = __builtin_ctz((unsigned)nx);
    const int xs = (int)(s0 & (nx - 1));
    const int r = (int)(s0 >> nxl);            // row z ny + y
    const int rl = p.row_log2;
    // population 0 at x = 0 of the row, and the lane's byte offset in it
    _Float16 *__restrict__ f = static_cast<_Float16 *>(p.pops);
    const _Float16 *row =
        f + (long long)(r >> rl) * (long long)(Q << kBlockLog2) + (long long)((r & ((1 << rl) - 1)) * nx);
    const unsigned xb = (unsigned)(xs + 2 * lane) * 2u;
    typedef __attribute__((address_space(1))) uint32_t gU32;
    typedef __attribute__((address_space(1))) char gchar;
    auto at = [&](int slot) -> gU32 * {
        gchar *b = (gchar *)(row + slot_off(slot));
        asm("" : "+s"(b));  // scalar base, lane offset added per access
        return (gU32 *)(b + xb);
    };

    // u[i]: h_i of both nodes (low half: x0, high half: x0 + 1)
    uint32_t u[Q], o[Q];
    sfor<Q>([&](auto I) { u[decltype(I)::value] = *at(decltype(I)::value); });
    const int tag = p.uniform_tag;
    sfor<2>([&](auto K) {
        constexpr int k = decltype(K)::value;
        C h[Q], hs[Q];
        sfor<Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            h[i] = k == 0 ? half_lo(u[i]) : half_hi(u[i]);
        });
        collide_node<Q, 2, C, MS, false>(h, tag, true, p, hs, true);
        sfor<Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (k == 0) o[i] = half_bits(hs[i]);
            else o[i] |= half_bits(hs[i]) << 16;
        });
    });
    // h*_i to slot opp(i) of the nodes themselves
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        *at(V<Q, i>::opp) = o[i];
    });
}

// Neighbour mask of every node (see kMask*): wall bits, moving-wall flag and
// the node's own fluid tag (0 for non-fluid nodes); tags and masks in storage
// order (lay).
template <int Q>
__global__ __launch_bounds__(256) void k_build_mask(const uint8_t *tags, int nx, int ny, int nz, Layout lay,
                                                    int sector_log2, int odd_fill, uint32_t *mask) {
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long N = (long long)nx * ny * nz;
    if (t >= N) return;
    const int x = (int)(t % nx), y = (int)((t / nx) % ny), z = (int)(t / ((long long)nx * ny));
    auto fluid_at = [&](int gx, int gy, int gz) { return is_fluid_tag(tags[lay.at(gx, gy, gz)]); };
    const long long s = lay.at(x, y, z);
    const int own = tags[s];
    uint32_t m = 0;
    if (is_fluid_tag(own)) {
        m = (uint32_t)own << kMaskTagShift;
        sfor<Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if constexpr (i > 0) {
                using Vi = V<Q, i>;
                const int gx = wrap_idx(x + Vi::x, nx), gy = wrap_idx(y + Vi::y, ny), gz = wrap_idx(z + Vi::z, nz);
                const int tn = tags[lay.at(gx, gy, gz)];
                if (!is_fluid_tag(tn)) m |= 1u << i;
                if (tn >= LBM_TAG_WALL0) m |= 1u << kMaskMovingBit;
            }
        });
    } else {
        // filler: a non-fluid node in a storage sector that also holds fluid nodes
        const long long g = 1ll << sector_log2;
        const long long a = s & ~(g - 1), b = a + g < N ? a + g : N;
        bool any = false;
        for (long long k = a; k < b; ++k) any |= is_fluid_tag(tags[k]);
        if (any) {
            m = 1u;
            if (odd_fill) {
                sfor<Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    if constexpr (i > 0) {
                        using Vi = V<Q, i>;
                        if (!fluid_at(x, wrap_idx(y + Vi::y, ny), wrap_idx(z + Vi::z, nz))) m |= 1u << i;
                    }
                });
            }
        }
    }
    mask[s] = m;
}

// ------------------------------------------------------------- helpers

// Storage index of the node with natural index n = (z ny + y) nx + x.
__device__ __forceinline__ int storage_index(const AuxParams &a, long long n) {
    if (!a.lay.brick) return (int)n;
    const int x = (int)(n % a.nx), y = (int)((n / a.nx) % a.ny), z = (int)(n / ((long long)a.nx * a.ny));
    return a.lay.at(x, y, z);
}

// Equilibrium initialisation (FP64 arithmetic, rounded once to storage).
template <int Q, int P>
__global__ __launch_bounds__(256) void k_init(AuxParams a) {
    using S = typename Prec<P>::S;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= a.count) return;
    const int n = storage_index(a, a.cell0 + t);
    if (!is_fluid_tag(a.tags[n])) return;
    const double rho = a.in_rho ? a.in_rho[t] : a.rho0;
    const double ux = a.in_u ? a.in_u[t] : 0.0;
    const double uy = a.in_u ? a.in_u[a.count + t] : 0.0;
    const double uz = a.in_u ? a.in_u[2 * a.count + t] : 0.0;
    const double drho = rho - a.rho0;
    const double uu = ux * ux + uy * uy + uz * uz;
    S *f = static_cast<S *>(a.pops);
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        const double cu = Vi::x * ux + Vi::y * uy + Vi::z * uz;
        const double heq = Vi::w * (drho + rho * (3.0 * cu + 4.5 * cu * cu - 1.5 * uu));
        f[pop_base<Q>(n) + slot_off(i)] = (S)heq;
    });
}

// Natural state of the node at (x, y, z): f_i (or h_i) for every i (slot map of
// the layout parity).
template <int Q, int P>
__device__ __forceinline__ void load_natural(const AuxParams &a, int x, int y, int z, double (&fo)[Q]) {
    using S = typename Prec<P>::S;
    const S *f = static_cast<const S *>(a.pops);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const long long own = pop_base<Q>(a.lay.at(x, y, z));
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        long long off = own + slot_off(i);
        if (a.parity != 0 && i != 0) {
            const int sx = wrap_idx(x - Vi::x, nx), sy = wrap_idx(y - Vi::y, ny), sz = wrap_idx(z - Vi::z, nz);
            const int src = a.lay.at(sx, sy, sz);
            if (a.all_fluid || is_fluid_tag(a.tags[src])) off = pop_base<Q>(src) + slot_off(Vi::opp);
        }
        fo[i] = a.shifted ? (double)f[off] : (double)f[off] + Vi::w * a.rho0;
    });
}

// Density and velocity from the unshifted populations.
template <int Q>
__device__ __forceinline__ void node_fields(const AuxParams &a, const double (&fo)[Q], double &rho, double (&u)[3]) {
    double jx = 0.0, jy = 0.0, jz = 0.0;
    rho = 0.0;
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        rho += fo[i];
        jx += Vi::x * fo[i];
        jy += Vi::y * fo[i];
        jz += Vi::z * fo[i];
    });
    const double inv = 1.0 / rho;
    u[0] = (jx + 0.5 * a.force[0]) * inv;
    u[1] = (jy + 0.5 * a.force[1]) * inv;
    u[2] = (jz + 0.5 * a.force[2]) * inv;
}

// Box filter: a block takes 256 / factor consecutive coarse nodes, a thread one fine
// column of x (every 256th beyond a factor of 256), whose factor^2 nodes it sums; the
// columns of a coarse node are then added through LDS.  Coarse rows do not end a block:
// short ones (64 nodes, factor 8: eight coarse nodes of 32) would leave it mostly idle, and
// one block a row is more than a launch takes on flat lattices.  Bound by memory:
// one read of the populations, where a gather of the fields to FP64 planes and a
// filter of those moved them to memory and back (256^3 D3Q27 FP32, factor 4, the
// whole call: 15.1 ms with those and their 580 MB allocated and freed, 0.35 ms now).
template <int Q, int P>
__global__ __launch_bounds__(256) void k_filter(AuxParams a, int factor, int cx, int cy, int cz, double *coarse) {
    __shared__ double s[kCoarsePlanes][256];
    const int cols = factor < 256 ? factor : 256, per = 256 / cols;  // columns of a coarse node, coarse nodes a block
    const unsigned nc = (unsigned)cx * cy * cz, first = blockIdx.x * (unsigned)per;
    const int t = threadIdx.x, c = t / cols, xi = t - c * cols;
    const unsigned n = first + c, row = n / (unsigned)cx;  // of this thread's columns
    const int X = (int)(n - row * cx), Z = (int)(row / (unsigned)cy), Y = (int)(row - (unsigned)Z * cy);
    double v[kCoarsePlanes] = {};
    if (c < per && n < nc) {
        for (int dz = 0; dz < factor; ++dz)
            for (int dy = 0; dy < factor; ++dy)
                for (int dx = xi; dx < factor; dx += cols) {
                    const int x = X * factor + dx, y = Y * factor + dy, z = Z * factor + dz;
                    if (!a.all_fluid && !is_fluid_tag(a.tags[a.lay.at(x, y, z)])) continue;
                    double fo[Q], r, u[3];
                    load_natural<Q, P>(a, x, y, z, fo);
                    node_fields<Q>(a, fo, r, u);
                    v[0] += r;
                    v[1] += r * u[0];
                    v[2] += r * u[1];
                    v[3] += r * u[2];
                    v[4] += r * u[0] * u[0];
                    v[5] += r * u[1] * u[1];
                    v[6] += r * u[2] * u[2];
                    v[7] += r * u[0] * u[1];
                    v[8] += r * u[0] * u[2];
                    v[9] += r * u[1] * u[2];
                }
    }
#pragma unroll
    for (int k = 0; k < kCoarsePlanes; ++k) s[k][t] = v[k];
    __syncthreads();
    for (int q = t; q < per * kCoarsePlanes; q += 256) {
        const int k = q / per, e = (q - k * per) * cols;
        double sum = 0.0;
        for (int j = 0; j < cols; ++j) sum += s[k][e + j];
        s[k][e] = sum;
    }
    __syncthreads();
    const long long o = first + (unsigned)t;
    if (t >= per || o >= nc) return;
    const int e = t * cols;
    const double vol = (double)factor * factor * factor, sr = s[0][e];
    const double Ux = s[1][e] / sr, Uy = s[2][e] / sr, Uz = s[3][e] / sr;
    coarse[o] = sr / vol;
    coarse[nc + o] = Ux;
    coarse[2ll * nc + o] = Uy;
    coarse[3ll * nc + o] = Uz;
    coarse[4ll * nc + o] = s[4][e] / sr - Ux * Ux;
    coarse[5ll * nc + o] = s[5][e] / sr - Uy * Uy;
    coarse[6ll * nc + o] = s[6][e] / sr - Uz * Uz;
    coarse[7ll * nc + o] = s[7][e] / sr - Ux * Uy;
    coarse[8ll * nc + o] = s[8][e] / sr - Ux * Uz;
    coarse[9ll * nc + o] = s[9][e] / sr - Uy * Uz;
}

template <int Q, int P>
__global__ __launch_bounds__(256) void k_gather(AuxParams a, int gmode) {
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= a.count) return;
    const long long n = gmode == G_CELLS ? a.cells[t] : a.cell0 + t;
    // n < 2^31 (lbm_config), so 32-bit divisions do
    const unsigned row = (unsigned)n / (unsigned)a.nx;
    const int x = (int)((unsigned)n - row * (unsigned)a.nx), y = (int)(row % (unsigned)a.ny), z = (int)(row / (unsigned)a.ny);
    const bool fl = a.all_fluid || is_fluid_tag(a.tags[a.lay.at(x, y, z)]);
    if (gmode == G_FIELDS) a.shifted = 0;
    double fo[Q];
    if (fl) {
        load_natural<Q, P>(a, x, y, z, fo);
    } else {
        sfor<Q>([&](auto I) { fo[decltype(I)::value] = 0.0; });
    }
    if (gmode == G_POPS) {
        sfor<Q>([&](auto I) { a.out[(long long)decltype(I)::value * a.count + t] = fo[decltype(I)::value]; });
    } else if (gmode == G_CELLS) {
        sfor<Q>([&](auto I) { a.out[t * Q + decltype(I)::value] = fo[decltype(I)::value]; });
    } else {
        double rho = 0.0, u[3] = {0.0, 0.0, 0.0};
        if (fl) node_fields<Q>(a, fo, rho, u);
        a.out[t] = rho;
        a.out[a.count + t] = u[0];
        a.out[2 * a.count + t] = u[1];
        a.out[3 * a.count + t] = u[2];
    }
}

// Write natural-layout populations (unshifted FP64 in, shifted storage out).
template <int Q, int P>
__global__ __launch_bounds__(256) void k_scatter(AuxParams a) {
    using S = typename Prec<P>::S;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= a.count) return;
    const int n = storage_index(a, a.cell0 + t);
    if (!is_fluid_tag(a.tags[n])) return;
    S *f = static_cast<S *>(a.pops);
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        using Vi = V<Q, i>;
        const double v = a.in_f[(long long)i * a.count + t];
        f[pop_base<Q>(n) + slot_off(i)] = (S)(a.shifted ? v : v - Vi::w * a.rho0);
    });
}

// Slab-face copy: one thread per node of the plane; each copies the slots of
// the directions crossing the face (c_z = +1 on face 0, c_z = -1 on face 1),
// the j-th of them to buf[j][y][x].  Coalesced along x on both sides.
template <int Q, int P>
__global__ __launch_bounds__(256) void k_face(AuxParams a, int face, int unpack, void *buf) {
    using S = typename Prec<P>::S;
    const long long nxy = (long long)a.nx * a.ny;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= nxy) return;
    const int plane = face == 0 ? 0 : a.nz - 1;
    const int n = storage_index(a, (long long)plane * nxy + t);
    S *f = static_cast<S *>(a.pops);
    S *b = static_cast<S *>(buf);
    const long long base = pop_base<Q>(n);
    const int cz = face == 0 ? 1 : -1;
    int j = 0;
    sfor<Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (V<Q, i>::z != 0) {
            if (V<Q, i>::z == cz) {
                S *slot = f + base + slot_off(i);
                S *e = b + (long long)j * nxy + t;
                if (unpack) *slot = *e;
                else *e = *slot;
                ++j;
            }
        }
    });
}

// ------------------------------------------------------------- launchers

// Dynamic LDS that the even-step kernel of FP32/FP64 row-form (walled,
// mostly fluid) lattices does not use: it caps a CU's 160 KB of LDS at three
// workgroups, i.e. three waves per SIMD.  Measured on the 256^3 cavity: FP32
// +1.0% (two waves per SIMD: -2%), FP64 +0.2%, regularized +0.4-0.6%; FP16
// and the odd step lose with any cap.
constexpr unsigned kEvenLdsCap = 41u << 10;

// The same for both parities of FP32 brick-layout lattices, at four workgroups a
// CU: 256^3 porous D3Q19 TRT 188.5 us a step against 195.5 without a cap (five workgroups
// 191.0, three 191.2).
constexpr unsigned kBrickLdsCap = 40000u;

template <int Q, int P, int MS, bool TG, int MODE, int ADDR>
static hipError_t launch_step_rows(const StepParams &p, int parity, hipStream_t s) {
    const dim3 grid(8 * p.tiles_per_xcd), block(256);
    constexpr unsigned lds_brick = (ADDR >= 2 && P == 1) ? kBrickLdsCap : 0u;
    constexpr unsigned lds_even = (ADDR == 1 && TG && P != 2) ? kEvenLdsCap : lds_brick;
    if (parity == 0)
        k_collide_stream<Q, P, MS, TG, MODE, 0, ADDR><<<grid, block, lds_even, s>>>(p);
    else
        k_collide_stream<Q, P, MS, TG, MODE, 1, ADDR><<<grid, block, lds_brick, s>>>(p);
    return hipGetLastError();
}

// Row-form variants (see k_collide_stream) where the lattice allows them: in
// FP16 storage for every wave (there the node form's per-lane address
// arithmetic limits the step, the odd step most), in FP32/FP64 for the wall
// waves of tagged lattices only (their selects get cheaper; for plain waves
// and untagged lattices, bound by memory alone, the row form measured 0.5-3%
// slower than the node form).
template <int Q, int P, int MS, bool TG, int MODE>
static hipError_t launch_step_par(const StepParams &p, int parity, hipStream_t s) {
    if constexpr (TG) {
        if (p.lay.brick) {
            // 32-bit offsets where they reach the whole array: a third fewer vector
            // instructions in the odd step.  256^3 rock, us a step, node form / these:
            // D3Q19 FP32 190.5 / 188.5, FP16 117 / 107, FP64 354 / 351; D3Q27 FP32
            // 307 / 300, FP16 183 / 171.  (What is left of the FP32 odd step, 228 us
            // against 150 for the even one with the same bytes, is its 2.1 times as
            // many sector accesses: a brick shifted in x and y touches four bricks.)
            const unsigned long long bytes = (unsigned long long)p.nx * p.ny * p.nz * Q * sizeof(typename Prec<P>::S);
            if (bytes <= 1ull << 32) return launch_step_rows<Q, P, MS, TG, MODE, 3>(p, parity, s);
            return launch_step_rows<Q, P, MS, TG, MODE, 2>(p, parity, s);
        }
    }
    if constexpr (P == 2 && !TG && (MS & MS_MLP) == 0 && MODE == MODE_STEP) {
        // the even step of FP16 lattices of one model: two nodes per lane
        if (p.pair && parity == 0) {
            const int n_tiles = (p.n_segs + 3) / 4;
            k_collide_pair_even<Q, MS><<<dim3(8 * ((n_tiles + 7) / 8)), dim3(256), 0, s>>>(p);
            return hipGetLastError();
        }
    }
    constexpr bool kRows = P == 2 || TG;
    if constexpr (kRows) {
        if (p.row_log2 >= 0) return launch_step_rows<Q, P, MS, TG, MODE, 1>(p, parity, s);
    }
    return launch_step_rows<Q, P, MS, TG, MODE, 0>(p, parity, s);
}

template <int Q, int P, int MS, bool TG>
static hipError_t launch_step_mode(const StepParams &p, int mode, int parity, hipStream_t s) {
    switch (mode) {
        case MODE_STEP: return launch_step_par<Q, P, MS, TG, MODE_STEP>(p, parity, s);
        case MODE_STEP_REDUCE: return launch_step_par<Q, P, MS, TG, MODE_STEP_REDUCE>(p, parity, s);
        default: return launch_step_par<Q, P, MS_BGK, TG, MODE_REDUCE>(p, parity, s);
    }
}

template <int Q, int P, bool TG>
static hipError_t launch_step_ms(const StepParams &p, int ms, int mode, int parity, hipStream_t s) {
    switch (ms) {
        case MS_BGK: return launch_step_mode<Q, P, MS_BGK, TG>(p, mode, parity, s);
        case MS_TRT: return launch_step_mode<Q, P, MS_TRT, TG>(p, mode, parity, s);
        case MS_BGK | MS_SMAG: return launch_step_mode<Q, P, MS_BGK | MS_SMAG, TG>(p, mode, parity, s);
        case MS_BGK | MS_SMAG | MS_MLP: return launch_step_mode<Q, P, MS_BGK | MS_SMAG | MS_MLP, TG>(p, mode, parity, s);
        case MS_REG: return launch_step_mode<Q, P, MS_REG, TG>(p, mode, parity, s);
        case MS_TRT | MS_OPEN: return launch_step_mode<Q, P, MS_TRT | MS_OPEN, TG>(p, mode, parity, s);
        case MS_RR: return launch_step_mode<Q, P, MS_RR, TG>(p, mode, parity, s);
        case kAllModels: return launch_step_mode<Q, P, kAllModels, TG>(p, mode, parity, s);
        case MS_STREAM: return launch_step_mode<Q, P, MS_STREAM, TG>(p, mode, parity, s);
        default: return hipErrorInvalidValue;
    }
}

template <int Q, int P>
hipError_t launch_step(const StepParams &p, int ms, bool tagged, int mode, int parity, hipStream_t s) {
    return tagged ? launch_step_ms<Q, P, true>(p, ms, mode, parity, s)
                  : launch_step_ms<Q, P, false>(p, ms, mode, parity, s);
}

template <int Q>
hipError_t launch_build_mask(const uint8_t *tags, int nx, int ny, int nz, Layout lay, int sector_log2,
                             int odd_fill, uint32_t *mask, hipStream_t s) {
    const long long N = (long long)nx * ny * nz;
    k_build_mask<Q><<<(unsigned)((N + 255) / 256), 256, 0, s>>>(tags, nx, ny, nz, lay, sector_log2, odd_fill, mask);
    return hipGetLastError();
}

template <int Q, int P>
hipError_t launch_init(const AuxParams &a, hipStream_t s) {
    const unsigned blocks = (unsigned)((a.count + 255) / 256);
    k_init<Q, P><<<blocks, 256, 0, s>>>(a);
    return hipGetLastError();
}

template <int Q, int P>
hipError_t launch_gather(const AuxParams &a, int gmode, hipStream_t s) {
    const unsigned blocks = (unsigned)((a.count + 255) / 256);
    k_gather<Q, P><<<blocks, 256, 0, s>>>(a, gmode);
    return hipGetLastError();
}

template <int Q, int P>
hipError_t launch_filter(const AuxParams &a, int factor, double *coarse, hipStream_t s) {
    const int cx = a.nx / factor, cy = a.ny / factor, cz = a.nz / factor;
    const int per = 256 / (factor < 256 ? factor : 256);
    const long long blocks = ((long long)cx * cy * cz + per - 1) / per;
    k_filter<Q, P><<<(unsigned)blocks, 256, 0, s>>>(a, factor, cx, cy, cz, coarse);
    return hipGetLastError();
}

template <int Q, int P>
hipError_t launch_scatter(const AuxParams &a, hipStream_t s) {
    const unsigned blocks = (unsigned)((a.count + 255) / 256);
    k_scatter<Q, P><<<blocks, 256, 0, s>>>(a);
    return hipGetLastError();
}

template <int Q, int P>
hipError_t launch_face(const AuxParams &a, int face, int unpack, void *buf, hipStream_t s) {
    const long long nxy = (long long)a.nx * a.ny;
    k_face<Q, P><<<(unsigned)((nxy + 255) / 256), 256, 0, s>>>(a, face, unpack, buf);
    return hipGetLastError();
}

#define LBMD_INSTANTIATE(Q, P)                                                                           \
    template hipError_t launch_step<Q, P>(const StepParams &, int, bool, int, int, hipStream_t);          \
    template hipError_t launch_init<Q, P>(const AuxParams &, hipStream_t);                                \
    template hipError_t launch_gather<Q, P>(const AuxParams &, int, hipStream_t);                         \
    template hipError_t launch_scatter<Q, P>(const AuxParams &, hipStream_t);                             \
    template hipError_t launch_filter<Q, P>(const AuxParams &, int, double *, hipStream_t);               \
    template hipError_t launch_face<Q, P>(const AuxParams &, int, int, void *, hipStream_t);

}  // namespace lbmd
