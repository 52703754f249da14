// lbm_two.h -- two time steps in one pass over memory.
//
// A step alone is bound by memory: it reads and writes every population once
// (one 512^3 D3Q27 FP32 step moves 29 GB, 5.2 ms at the 5.6 TB/s a copy of that
// size reaches).  k_two_steps does two steps for one read and one write.  It
// reads the populations from one array and writes the state two steps later, in
// the same layout parity, to a second one (in place, a block could not know
// whether its neighbours had read their halo yet).
//
// A block takes a tile of nodes in x and y and marches over a chunk of planes.
// Per plane it collides the tile and a one-node halo around it (first step),
// leaves the post-collision populations in LDS, and streams and collides the
// plane below from there (second step): upward populations are kept for three
// planes, horizontal ones for two, downward ones for one, and each thread keeps
// its own rest population.  Loads of the next plane are in flight during the
// second step.  FP16 populations are rounded to FP16 in between as a stored
// state is, so the result does not depend on how steps are grouped.
//
// Tile: the halo columns cost whole 128-byte lines in 2 (TY + 2) of the lines a
// plane takes, so tiles are wide: measured on the 512^3 D3Q27 FP32 Taylor-Green
// flow per step, one step per pass 5.21 ms; two per pass with 32 x 8 tiles (two
// blocks a CU) 3.89, 64 x 8 3.44, 128 x 4 3.0 to 3.3 ms from box to box (1.27x the
// ideal reads from the L2s at 64 x 8).  More blocks a CU are slower (their tiles no longer share
// halos through a 4 MB L2): 3 a CU 4.96 ms.  Prefetching a plane earlier, or
// two, gained nothing.
#pragma once

#include "lbm_kernels.h"

namespace lbmd {

// Directions with c_z = cz, and the rank of direction I among those of its c_z.
template <int Q>
constexpr int dir_z(int i) {
    constexpr int H = (Q - 1) / 2;
    return i == 0 ? 0 : (i <= H ? kHalfDirs[i - 1][2] : -kHalfDirs[i - 1 - H][2]);
}
template <int Q>
constexpr int count_z(int cz) {
    int n = 0;
    for (int i = 0; i < Q; ++i) n += dir_z<Q>(i) == cz;
    return n;
}
template <int Q, int I>
constexpr int rank_z() {
    int n = 0;
    for (int i = 0; i < I; ++i) n += dir_z<Q>(i) == dir_z<Q>(I);
    return n;
}

template <int Q, int P, int MS, bool TAGGED, int PARITY, bool FORCE>
__global__ __launch_bounds__(two_region(P) / 64 * 64 + 64) void k_two_steps(StepParams p, void *dst, TwoTiles w) {
    using S = typename Prec<P>::S;
    using C = typename Prec<P>::C;
    constexpr int NU = count_z<Q>(1), NM = count_z<Q>(0);
    constexpr int RS = two_region(P);
    // D3Q27 FP64 populations of three planes do not fit in 160 KB: there the second
    // step reads what it takes from the planes below before the first step of this
    // plane overwrites them (a barrier more between, two planes kept)
    constexpr bool RING3 = !(Q == 27 && P == 0);
    __shared__ S lds[(RING3 ? 4 * NU + 2 * (NM - 1) : 3 * NU + (NM - 1)) * RS];
    typedef __attribute__((address_space(1))) S gS;
    typedef __attribute__((address_space(1))) char gchar;

    const int wg = blockIdx.x;
    const int L = (wg & 7) * w.per_xcd + (wg >> 3);
    if (L >= w.n_blocks) return;  // uniform for the block
    const int nx = p.nx, ny = p.ny, nz = p.nz, nxy = nx * ny;
    const int tix = __builtin_amdgcn_readfirstlane(L % w.tiles_x), rem = L / w.tiles_x;
    const int tiy = __builtin_amdgcn_readfirstlane(rem % w.tiles_y);
    const int z0 = __builtin_amdgcn_readfirstlane(rem / w.tiles_y) * w.chunk;
    const int planes = min(w.chunk, nz - z0);
    const int TX = w.tx, TY = w.ty, RX = TX + 2, RY = TY + 2;

    // region node of this thread: the tile's nodes first, then its halo (rows
    // below and above, columns left and right)
    const int tid = threadIdx.x;
    const bool in_tile = tid < TX * TY;
    int rx, ry;
    if (in_tile) {
        ry = tid / TX;
        rx = tid - ry * TX + 1, ry += 1;
    } else {
        const int k = tid - TX * TY;
        if (k < 2 * RX) rx = k < RX ? k : k - RX, ry = k < RX ? 0 : RY - 1;
        else rx = k < 2 * RX + TY ? 0 : RX - 1, ry = (k - 2 * RX) % TY + 1;
    }
    const int rn[3] = {(ry - 1) * RX + rx, ry * RX + rx, (ry + 1) * RX + rx};  // rows y - 1, y, y + 1
    const int r = rn[1];
    int x = tix * TX + rx - 1, y = tiy * TY + ry - 1;
    const bool tile = in_tile && x < nx && y < ny;
    const bool act = tid < RX * RY && x <= nx && y <= ny;
    x = !act ? 0 : (x < 0 ? x + nx : (x >= nx ? x - nx : x));
    y = !act ? 0 : (y < 0 ? y + ny : (y >= ny ? y - ny : y));
    const int m0 = y * nx + x;
    // byte offsets within a plane of columns x - 1, x, x + 1 and rows y - 1, y, y + 1
    const unsigned xb[3] = {(unsigned)(x == 0 ? nx - 1 : x - 1) * (unsigned)sizeof(S), (unsigned)x * (unsigned)sizeof(S),
                            (unsigned)(x + 1 == nx ? 0 : x + 1) * (unsigned)sizeof(S)};
    const unsigned yb[3] = {(unsigned)((y == 0 ? ny - 1 : y - 1) * nx) * (unsigned)sizeof(S),
                            (unsigned)(y * nx) * (unsigned)sizeof(S),
                            (unsigned)((y + 1 == ny ? 0 : y + 1) * nx) * (unsigned)sizeof(S)};

    auto wrapz = [&](int z) { return z < 0 ? z + nz : (z >= nz ? z - nz : z); };
    // A population's address: the scalar base of the block its plane starts in
    // and of its slot, plus the lane's 32-bit byte offset from there, which is
    // t + (t / block) (Q - 1) block for the node t bytes into the plane's blocks
    // (pop_base).
    constexpr int kBlockBytesLog2 = kBlockLog2 + (sizeof(S) == 8 ? 3 : (sizeof(S) == 4 ? 2 : 1));
    auto plane_base = [&](const void *f, int z) -> const S * {
        return static_cast<const S *>(f) + (((long long)z * nxy) >> kBlockLog2) * (long long)(Q << kBlockLog2);
    };
    auto lane_off = [&](int z, unsigned yo, unsigned xo) -> unsigned {
        const unsigned t = (unsigned)(((long long)z * nxy) & (kBlockNodes - 1)) * (unsigned)sizeof(S) + yo + xo;
        return __umul24(t >> kBlockBytesLog2, (unsigned)((Q - 1) << kBlockBytesLog2)) + t;
    };
    auto at = [&](const S *base, int slot, unsigned off) -> gS * {
        gS *b = (gS *)(base + slot_off(slot));
        asm("" : "+s"(b));  // scalar base, lane offset added per access
        return (gS *)((gchar *)b + off);
    };
    auto mask_of = [&](int z) -> uint32_t { return act ? p.mask[(long long)z * nxy + m0] : 0u; };
    auto is_live = [&](uint32_t m) { return act && (!TAGGED || (m >> kMaskTagShift) != 0u); };
    auto tag_of = [&](uint32_t m) { return TAGGED ? (int)(m >> kMaskTagShift) : p.uniform_tag; };

    // the stored populations of the thread's node on plane z
    auto load = [&](int z, uint32_t m, S (&v)[Q]) {
        if (!is_live(m)) return;
        const S *b1 = plane_base(p.pops, z);
        const unsigned own = lane_off(z, yb[1], xb[1]);
        if constexpr (PARITY == 0) {
            sfor<Q>([&](auto I) { v[decltype(I)::value] = *at(b1, decltype(I)::value, own); });
        } else {
            const int zv[3] = {wrapz(z - 1), z, wrapz(z + 1)};
            const S *b[3] = {plane_base(p.pops, zv[0]), b1, plane_base(p.pops, zv[2])};
            auto pull = [&](auto walls_c) {
                sfor<Q>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    using Vi = V<Q, i>;
                    if constexpr (i == 0) {
                        v[0] = *at(b1, 0, own);
                    } else {
                        gS *a = at(b[1 - Vi::z], Vi::opp, lane_off(zv[1 - Vi::z], yb[1 - Vi::y], xb[1 - Vi::x]));
                        if constexpr (decltype(walls_c)::value) {
                            gS *o = at(b1, i, own);
                            a = ((m >> Vi::opp) & 1u) ? o : a;
                        }
                        v[i] = *a;
                    }
                });
            };
            if (TAGGED && __any((m & kMaskWalls) != 0u)) pull(std::integral_constant<bool, TAGGED>{});
            else pull(std::false_type{});
        }
    };
    // moving-wall term of the directions that leave towards a moving wall
    auto wall_term = [&](uint32_t m, int z, C (&hs)[Q]) {
        if ((m >> kMaskMovingBit) & 1u) {
            const int yo[3] = {y == 0 ? ny - 1 : y - 1, y, y + 1 == ny ? 0 : y + 1};
            const int xo[3] = {x == 0 ? nx - 1 : x - 1, x, x + 1 == nx ? 0 : x + 1};
            sfor<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                using Vi = V<Q, i>;
                if constexpr (i > 0) {
                    if ((m >> i) & 1u) {
                        const int t = p.tags[(long long)wrapz(z + Vi::z) * nxy + yo[1 + Vi::y] * nx + xo[1 + Vi::x]];
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
    };
    // a rest population is rounded to FP32 before it is to FP16, as in the one-step kernels
    // of the models whose last product-sum is that of the force, also of a zero one
    auto round_rest = [](C &h0) {
        if constexpr (P == 2 && MS != MS_REG && MS != MS_RR) asm("" : "+v"(h0));
    };
    // orders LDS accesses only: loads and stores of global memory stay in flight
    auto barrier = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    S v[Q];
    sfor<Q>([&](auto I) { v[decltype(I)::value] = S(0); });
    uint32_t m_own = 0, m_cur = 0, m_next = 0;  // masks of planes ze - 1, ze, ze + 1
    int ze = wrapz(z0 - 1);
    if constexpr (TAGGED) m_cur = mask_of(ze);
    load(ze, m_cur, v);
    if constexpr (TAGGED) m_next = mask_of(wrapz(ze + 1));
    C rest = C(0);  // the thread's own rest population of plane ze - 1 (rounded as stored)
    int iu = 0;     // ring position of plane ze
    for (int k = 0; k < planes + 2; ++k) {
        // upward populations of planes ze, ze - 1, ze - 2, horizontal ones of ze and
        // ze - 1, downward ones of ze
        const int iu1 = RING3 ? (iu == 0 ? 2 : iu - 1) : iu ^ 1, iu2 = RING3 ? (iu1 == 0 ? 2 : iu1 - 1) : iu;
        S *up0 = lds + iu * (NU * RS), *up1 = lds + iu1 * (NU * RS), *up2 = lds + iu2 * (NU * RS);
        S *mid0 = lds + ((RING3 ? 3 * NU : 2 * NU) + (RING3 ? (k & 1) * (NM - 1) : 0)) * RS;
        S *mid1 = lds + ((RING3 ? 3 * NU : 2 * NU) + (RING3 ? ((k & 1) ^ 1) * (NM - 1) : 0)) * RS;
        S *down0 = lds + (RING3 ? 3 * NU + 2 * (NM - 1) : 2 * NU + (NM - 1)) * RS;
        iu = RING3 ? (iu == 2 ? 0 : iu + 1) : iu ^ 1;
        const int zo = wrapz(ze - 1), zn = wrapz(ze + 1);
        const bool second = k >= 2 && in_tile;
        // waves next to no wall take the code without it
        const bool walls = TAGGED && __any(tile && (m_own & kMaskWalls) != 0u);
        C g[Q];
        auto gather = [&](auto down_c, auto walls_c) {
            sfor<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                using Vi = V<Q, i>;
                if constexpr (i > 0 && (Vi::z < 0) == decltype(down_c)::value) {
                    const S *slot = Vi::z > 0 ? up2 : (Vi::z == 0 ? mid1 : down0);
                    int a = (rank_z<Q, i>() - (Vi::z == 0)) * RS + rn[1 - Vi::y] - Vi::x;
                    if constexpr (decltype(walls_c)::value && Vi::z <= 0) {
                        // a wall at x - c_i: the node's own opposite population
                        const S *own = Vi::z == 0 ? mid1 : up1;
                        const bool wi = (m_own >> Vi::opp) & 1u;
                        slot = wi ? own : slot;
                        a = wi ? (rank_z<Q, Vi::opp>() - (Vi::z == 0)) * RS + r : a;
                    }
                    g[i] = (C)slot[a];
                }
            });
        };
        auto gather_part = [&](auto down_c) {
            if (walls) gather(down_c, std::integral_constant<bool, TAGGED>{});
            else gather(down_c, std::false_type{});
        };

        // ---- first step of plane ze
        const bool live = is_live(m_cur);
        C hs[Q];
        {
            C h[Q];
            sfor<Q>([&](auto I) { h[decltype(I)::value] = live ? (C)v[decltype(I)::value] : C(0); });
            collide_node<Q, P, C, MS, TAGGED, FORCE, true>(h, tag_of(m_cur), live, p, hs, P == 2 && PARITY == 0 && p.pair);
            if constexpr (TAGGED) wall_term(m_cur, ze, hs);
        }
        g[0] = rest;
        round_rest(hs[0]);
        rest = (C)(S)hs[0];
        if constexpr (!RING3) {
            sfor<Q>([&](auto I) {
                if constexpr (decltype(I)::value > 0) g[decltype(I)::value] = C(0);
            });
            if (second) gather_part(std::false_type{});
            barrier();
        }
        if (live) {
            sfor<Q>([&](auto I) {
                constexpr int i = decltype(I)::value;
                using Vi = V<Q, i>;
                if constexpr (i > 0) {
                    S *slot = Vi::z > 0 ? up0 : (Vi::z == 0 ? mid0 : down0);
                    slot[(rank_z<Q, i>() - (Vi::z == 0)) * RS + r] = (S)hs[i];
                }
            });
            if constexpr (TAGGED) {
                // a wall below: what returns from it goes where the second step looks for it
                if (tile && (m_cur & kMaskWalls)) {
                    sfor<Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        using Vi = V<Q, i>;
                        if constexpr (Vi::z > 0) {
                            if ((m_cur >> Vi::opp) & 1u) up1[rank_z<Q, i>() * RS + rn[1 - Vi::y] - Vi::x] = (S)hs[Vi::opp];
                        }
                    });
                }
            }
        }
        uint32_t m_after = 0;
        if (k <= planes) {
            load(zn, m_next, v);
            if constexpr (TAGGED) m_after = mask_of(wrapz(zn + 1));
        }
        barrier();
        // ---- second step of plane ze - 1
        if (second) {
            const bool on = tile && (!TAGGED || (m_own >> kMaskTagShift) != 0u);
            if constexpr (RING3) gather_part(std::false_type{});
            gather_part(std::true_type{});
            C gs[Q];
            collide_node<Q, P, C, MS, TAGGED, FORCE, true>(g, tag_of(m_own), on, p, gs, P == 2 && PARITY == 1 && p.pair);
            if constexpr (TAGGED) wall_term(m_own, zo, gs);
            round_rest(gs[0]);
            const unsigned own = lane_off(zo, yb[1], xb[1]);
            const int zv[3] = {wrapz(zo - 1), zo, wrapz(zo + 1)};
            const S *b[3] = {plane_base(dst, zv[0]), plane_base(dst, zv[1]), plane_base(dst, zv[2])};
            if (!walls) {
                if (on) {
                    sfor<Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        using Vi = V<Q, i>;
                        if constexpr (i == 0 || PARITY == 1)
                            *at(b[1], Vi::opp, own) = (S)gs[i];
                        else
                            *at(b[1 + Vi::z], i, lane_off(zv[1 + Vi::z], yb[1 + Vi::y], xb[1 + Vi::x])) = (S)gs[i];
                    });
                }
            } else if constexpr (TAGGED) {
                if (on) {
                    sfor<Q>([&](auto I) {
                        constexpr int i = decltype(I)::value;
                        using Vi = V<Q, i>;
                        const S out = (S)gs[i];
                        if constexpr (i == 0 || PARITY == 1) {
                            *at(b[1], Vi::opp, own) = out;
                        } else {
                            const bool wi = (m_own >> i) & 1u;
                            gS *a = at(b[1 + Vi::z], i, lane_off(zv[1 + Vi::z], yb[1 + Vi::y], xb[1 + Vi::x]));
                            gS *o = at(b[1], Vi::opp, own);
                            a = wi ? o : a;
                            *a = out;
                        }
                    });
                }
            }
        }
        if constexpr (RING3) barrier();
        m_own = m_cur, m_cur = m_next, m_next = m_after;
        ze = zn;
    }
}

template <int Q, int P, int MS, bool TG, bool FORCE = true>
static hipError_t launch_two_par(const StepParams &p, void *dst, const TwoTiles &w, int parity, hipStream_t s) {
    const dim3 grid(8 * w.per_xcd), block(((w.tx + 2) * (w.ty + 2) + 63) / 64 * 64);
    if (parity == 0) k_two_steps<Q, P, MS, TG, 0, FORCE><<<grid, block, 0, s>>>(p, dst, w);
    else k_two_steps<Q, P, MS, TG, 1, FORCE><<<grid, block, 0, s>>>(p, dst, w);
    return hipGetLastError();
}

// Without a body force the Guo terms are left out (collide_pairs, collide_regularized):
// fewer registers.
template <int Q, int P, int MS, bool TG>
static hipError_t launch_two_force(const StepParams &p, void *dst, const TwoTiles &w, int parity, hipStream_t s) {
    if constexpr (two_built(Q, P, MS, TG, false)) {
        if (!p.has_force) return launch_two_par<Q, P, MS, TG, false>(p, dst, w, parity, s);
    }
    if constexpr (two_built(Q, P, MS, TG, true)) {
        if (p.has_force) return launch_two_par<Q, P, MS, TG, true>(p, dst, w, parity, s);
    }
    return hipErrorInvalidValue;
}

template <int Q, int P, bool TG>
static hipError_t launch_two_ms(const StepParams &p, void *dst, const TwoTiles &w, int ms, int parity, hipStream_t s) {
    switch (ms) {
        case MS_BGK: return launch_two_force<Q, P, MS_BGK, TG>(p, dst, w, parity, s);
        case MS_TRT: return launch_two_force<Q, P, MS_TRT, TG>(p, dst, w, parity, s);
        case MS_BGK | MS_SMAG: return launch_two_force<Q, P, MS_BGK | MS_SMAG, TG>(p, dst, w, parity, s);
        case MS_RR: return launch_two_force<Q, P, MS_RR, TG>(p, dst, w, parity, s);
        case MS_REG: return launch_two_force<Q, P, MS_REG, TG>(p, dst, w, parity, s);
        default: return hipErrorInvalidValue;
    }
}

template <int Q, int P>
hipError_t launch_two_steps(const StepParams &p, void *dst, const TwoTiles &w, int ms, bool tagged, int parity, hipStream_t s) {
    return tagged ? launch_two_ms<Q, P, true>(p, dst, w, ms, parity, s)
                  : launch_two_ms<Q, P, false>(p, dst, w, ms, parity, s);
}

}  // namespace lbmd
