// lbm_plane.hpp -- the two-pass D2Q9 step in one launch.
//
// The separate passes of a D2Q9 step each move little and mostly wait (memory latency and the drain
// between dependent launches): a workgroup here takes the whole step of a tile of the plane
// instead.  It forms the records (rho, v^(1)) of the tile and kRM rings around it from the
// populations, the corrected velocities of the tile and kRV rings from those, and collides the
// tile, all through LDS; ring cells are computed again by the neighbouring tiles.  As a tile reads
// its neighbours' populations, the step reads one population buffer and writes the other (slot for
// slot what the in-place passes write).  Every expression is the separate passes' own, so results
// are bitwise the same.
//
// Bounded by vector arithmetic on large planes (FP32 1019 x 977: 84 B per cell and step, 14 us at
// the copy rate, against 26 us) and by one tile's chain of load latencies and barriers on small
// ones.  us per step, separate passes and one launch: FP64 channel with walls 128 x 64 13.6 -> 7.3,
// FP32 box 1019 x 977 44.5 -> 26.5.
#pragma once

#include "lbm_device.hpp"

namespace lbm {

// Shape of a workgroup: a TX x TY tile on NT threads.  Rings: the collision reads the corrected
// velocity of the face neighbours, the correction the records of its own face neighbours; with
// solids the one-sided derivatives reach one cell further in both.
template <typename T, bool S, int TX, int TY, int NT>
struct PlaneCfg {
    static constexpr int kX = TX, kY = TY, kThreads = NT;
    static constexpr int kRV = S ? 2 : 1, kRM = S ? 4 : 2, kRE = kRM + 1;
    static constexpr int kVX = TX + 2 * kRV, kVY = TY + 2 * kRV, kV = kVX * kVY;
    static constexpr int kMX = TX + 2 * kRM, kMY = TY + 2 * kRM, kM = kMX * kMY;
    static constexpr int kEX = TX + 2 * kRE, kEY = TY + 2 * kRE, kE = kEX * kEY;
    // rounds of NT threads that cover the tile's own cells, whose populations stay in registers
    // from the moments to the collision
    static constexpr int kOwn = (TX * TY + NT - 1) / NT;
    static_assert(TX * TY % NT == 0 || TX * TY < NT, "whole rounds of own cells");
};

// q / W for 0 <= q < LIMIT by a 24-bit multiply (full rate, unlike the 32-bit multiplies of a
// division by a constant).
template <int W, int LIMIT>
__device__ __forceinline__ int div_small(int q) {
    constexpr int K = 1 << 19, M = K / W + 1;
    static_assert((M * W - K) * LIMIT < K && LIMIT <= 4096, "exact below LIMIT");
    return (int)((uint32_t)__umul24((unsigned)q, (unsigned)M) >> 19);
}

// Cell number q of a TX x TY tile with a ring of width R: the tile's own cells first, then the
// ring (lower rows, upper rows, left and right columns); position relative to the tile origin.
template <int TX, int TY, int R>
__device__ __forceinline__ void ring_cell(int q, int &lx, int &ly) {
    constexpr int WX = TX + 2 * R;
    if (q < TX * TY) {
        lx = q % TX;
        ly = q / TX;
        return;
    }
    q -= TX * TY;
    if (q < 2 * R * WX) {
        const int row = div_small<WX, 2 * R * WX>(q);
        ly = row < R ? row - R : TY + row - R;
        lx = q - row * WX - R;
    } else {
        q -= 2 * R * WX;
        const int c = q % (2 * R);
        ly = q / (2 * R);
        lx = c < R ? c - R : TX + c - R;
    }
}

// Second neighbours along an axis from the records, porosity and solid flags staged in LDS.
template <typename T, int WX, int EX>
struct FarPlane {
    const P4<T> *m;    // the cell's own record, row length WX
    const T *e;        // its porosity, row length EX
    const uint8_t *s;  // its solid flag, row length EX
    __device__ __forceinline__ bool get(int a, int k, Rec<T> &q) const {
        if (s[a == 0 ? k : k * EX]) return false;
        const P4<T> r = m[a == 0 ? k : k * WX];
        q.r = r.x;
        q.w[0] = r.y;
        q.w[1] = r.z;
        q.w[2] = r.w;
        q.e = e[a == 0 ? k : k * EX];
        return true;
    }
};

template <typename T>
__device__ __forceinline__ Rec<T> rec_of(const P4<T> &q, T e) {
    Rec<T> o;
    o.r = q.x;
    o.w[0] = q.y;
    o.w[1] = q.z;
    o.w[2] = q.w;
    o.e = e;
    return o;
}

template <typename T, typename P, bool S, int PH, int TX, int TY, int NT>
__global__ __launch_bounds__(NT) void k_plane_step(const P *__restrict__ fin, P *__restrict__ fout,
                                                   const T *__restrict__ eps,
                                                   const T *__restrict__ muD,
                                                   const T *__restrict__ muF,
                                                   const uint8_t *__restrict__ mask, Grid g,
                                                   uint32_t ntx, uint32_t nt, uint32_t per,
                                                   Phys<T> ph) {
    constexpr int D = 2, Q = 9;
    using C = PlaneCfg<T, S, TX, TY, NT>;
    constexpr int kMX = C::kMX, kVX = C::kVX, kEX = C::kEX, kRM = C::kRM, kRV = C::kRV,
                  kRE = C::kRE;
    __shared__ T es[C::kE];
    __shared__ P4<T> ms[C::kM];
    __shared__ P4<T> vs[C::kV];
    __shared__ uint8_t ss[S ? C::kE : 1];
    // the eight XCDs take contiguous ranges of the tiles, so that the rings of neighbouring
    // tiles are shared through the XCD's L2
    const uint32_t t = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if (t >= nt) return;  // whole workgroup
    const int x0 = (int)(t % ntx) * TX, y0 = (int)(t / ntx) * TY;
    const int tid = (int)threadIdx.x;
    // periodic coordinate; grids narrower than a tile and its rings take more than one correction
    const bool narrow = g.nx < TX + kRE || g.ny < TY + kRE;
    auto wrap = [&](int c, int n) {
        c = c < 0 ? c + n : (c >= n ? c - n : c);
        if (narrow) {
            while (c < 0) c += n;
            while (c >= n) c -= n;
        }
        return c;
    };
    auto at_e = [&](int lx, int ly) { return (ly + kRE) * kEX + lx + kRE; };
    auto eview = [&](int lx, int ly) {
        return EpsTile<D, T>{es + at_e(lx, ly), kEX, 0};
    };
    auto nbr = [&](int lx, int ly) {
        Nbr<D> nb;
        nb.init(g, wrap(x0 + lx, g.nx), wrap(y0 + ly, g.ny), 0);
        return nb;
    };

    // Slot of f_i of a cell as the AA pattern reads it; with solids the swapped phase finds a
    // population that was bounced back in the cell's own slot.
    auto slot = [&](auto ii, const Nbr<D> &nb, bool bounced) {
        constexpr int i = decltype(ii)::value;
        constexpr int cx = Lat<D>::c[i][0], cy = Lat<D>::c[i][1];
        if constexpr (PH == 0 || i == 0) {
            return at(plane(fin, i, g.N), nb.self());
        } else {
            return at(plane(fin, bounced ? i : Lat<D>::opp[i], g.N),
                      bounced ? nb.self() : nb.at(-cx, -cy, 0));
        }
    };
    // solid flag of the source cell of f_i, from the staged flags
    auto src_solid = [&](auto ii, int e) {
        constexpr int i = decltype(ii)::value;
        return S && i != 0 && ss[S ? e - Lat<D>::c[i][1] * kEX - Lat<D>::c[i][0] : 0];
    };
    auto sigma = [&](auto ii, const EpsTile<D, T> &ev, bool bounced) {
        constexpr int i = decltype(ii)::value;
        constexpr int cx = Lat<D>::c[i][0], cy = Lat<D>::c[i][1];
        if constexpr (!PopFmt<P>::shifted) return 0.0f;
        else return shift_sigma<D, i, P>(bounced ? ev.at(0, 0, 0) : ev.at(-cx, -cy, 0), ph);
    };

    // Own cells' populations (a cell past the grid's edge is the periodic image that the last
    // cells' stencils read), in flight while porosity and solid flags are staged: with solids
    // both candidate slots of the swapped phase, as the flags are not known yet.
    constexpr bool kBoth = S && PH == 1;
    P raw[C::kOwn][Q], own_slot[kBoth ? C::kOwn : 1][Q];
#pragma unroll
    for (int r = 0; r < C::kOwn; ++r) {
        int lx, ly;
        ring_cell<TX, TY, kRM>(tid + r * NT, lx, ly);
        if (tid + r * NT < C::kM) {
            const Nbr<D> nb = nbr(lx, ly);
            unroll<0, Q>([&](auto ii) {
                constexpr int i = decltype(ii)::value;
                raw[r][i] = *slot(ii, nb, false);
                if constexpr (kBoth) own_slot[r][i] = *slot(ii, nb, true);
            });
        }
    }
    constexpr int kItE = (C::kE + NT - 1) / NT;
    T te[kItE];
    uint8_t ts[kItE];
#pragma unroll
    for (int k = 0; k < kItE; ++k) {
        const int e = tid + k * NT;
        te[k] = T(0);
        ts[k] = 0;
        if (e < C::kE) {
            const int ey = div_small<kEX, C::kE>(e), ex = e - ey * kEX;
            const uint32_t c = (uint32_t)wrap(x0 + ex - kRE, g.nx) +
                               (uint32_t)g.nx * (uint32_t)wrap(y0 + ey - kRE, g.ny);
            te[k] = ld(eps, c);
            if constexpr (S) ts[k] = mask[c];
        }
    }
#pragma unroll
    for (int k = 0; k < kItE; ++k)
        if (tid + k * NT < C::kE) {
            es[tid + k * NT] = te[k];
            if constexpr (S) ss[tid + k * NT] = ts[k];
        }
    __syncthreads();
    if constexpr (kBoth) {
#pragma unroll
        for (int r = 0; r < C::kOwn; ++r) {
            int lx, ly;
            ring_cell<TX, TY, kRM>(tid + r * NT, lx, ly);
            if (tid + r * NT < C::kM) {
                unroll<0, Q>([&](auto ii) {
                    constexpr int i = decltype(ii)::value;
                    if (src_solid(ii, at_e(lx, ly))) raw[r][i] = own_slot[r][i];
                });
            }
        }
    }

    // records (rho, v^(1)) of the tile and kRM rings
    auto record = [&](int lx, int ly, const Nbr<D> &nb, const P (&rw)[Q]) {
        const int am = (ly + kRM) * kMX + lx + kRM, e = at_e(lx, ly);
        if constexpr (S) {
            if (ss[e]) {
                ms[am] = pack(T(0), T(0), T(0), T(0));
                return;
            }
        }
        const auto ev = eview(lx, ly);
        T fi[Q];
        unroll<0, Q>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            fi[i] = decode<D, i, T>(rw[i], sigma(ii, ev, src_solid(ii, e)));
        });
        const Rec<T> q = cell_moments<D, false>(fi, ev, muD, muF, nb, ph);
        ms[am] = pack(q.r, q.w[0], q.w[1], T(0));
    };
#pragma unroll
    for (int r = 0; r < C::kOwn; ++r) {
        int lx, ly;
        ring_cell<TX, TY, kRM>(tid + r * NT, lx, ly);
        if (tid + r * NT < C::kM) record(lx, ly, nbr(lx, ly), raw[r]);
    }
    for (int q = tid + C::kOwn * NT; q < C::kM; q += NT) {
        int lx, ly;
        ring_cell<TX, TY, kRM>(q, lx, ly);
        const Nbr<D> nb = nbr(lx, ly);
        P rw[Q];
        unroll<0, Q>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            rw[i] = *slot(ii, nb, src_solid(ii, at_e(lx, ly)));
        });
        record(lx, ly, nb, rw);
    }
    __syncthreads();

    // corrected velocities (v_final) of the tile and kRV rings
    auto stencil = [&](const P4<T> *m, int row, const EpsTile<D, T> &ev, const uint8_t *s,
                       Rec<T> rec[3][2], bool fl[3][2]) {
        rec[0][0] = rec_of(m[-1], ev.at(-1, 0, 0));
        rec[0][1] = rec_of(m[1], ev.at(1, 0, 0));
        rec[1][0] = rec_of(m[-row], ev.at(0, -1, 0));
        rec[1][1] = rec_of(m[row], ev.at(0, 1, 0));
        fl[0][0] = S ? !s[-1] : true;
        fl[0][1] = S ? !s[1] : true;
        fl[1][0] = S ? !s[-kEX] : true;
        fl[1][1] = S ? !s[kEX] : true;
    };
    for (int q = tid; q < C::kV; q += NT) {
        int lx, ly;
        ring_cell<TX, TY, kRV>(q, lx, ly);
        const int am = (ly + kRM) * kMX + lx + kRM, e = S ? at_e(lx, ly) : 0;
        P4<T> *out = vs + (ly + kRV) * kVX + lx + kRV;
        if constexpr (S) {
            if (ss[e]) {
                *out = pack(T(0), T(0), T(0), T(0));
                continue;
            }
        }
        const auto ev = eview(lx, ly);
        const Rec<T> own = rec_of(ms[am], ev.at(0, 0, 0));
        const CellStatic<D, T> cs = cell_static<D, false>(ev, ph, 0u, own.e);
        const bool flat = porosity_flat<D, T>(cs);
        Rec<T> rec[3][2];
        bool fl[3][2];
        if (!flat) stencil(ms + am, kMX, ev, ss + e, rec, fl);
        T v[3];
        const FarPlane<T, kMX, kEX> far{ms + am, ev.lds, ss + e};
        velocity_from_stencil<D, T, S>(far, own, rec, fl, cs, flat, v);
        *out = pack(own.r, v[0], v[1], T(0));
    }
    __syncthreads();

    // forcing, collision and streaming of the tile's own cells
#pragma unroll
    for (int r = 0; r < C::kOwn; ++r) {
        const int q = tid + r * NT;
        const int lx = q % TX, ly = q / TX;
        if (q >= TX * TY || x0 + lx >= g.nx || y0 + ly >= g.ny) continue;
        const int e = S ? at_e(lx, ly) : 0;
        if constexpr (S) {
            if (ss[e]) continue;
        }
        const int av = (ly + kRV) * kVX + lx + kRV;
        const auto ev = eview(lx, ly);
        Nbr<D> nb;
        nb.init(g, x0 + lx, y0 + ly, 0);
        const Rec<T> own = rec_of(vs[av], ev.at(0, 0, 0));
        const CellStatic<D, T> cs = cell_static<D, false>(ev, ph, 0u, own.e);
        Rec<T> rec[3][2];
        bool fl[3][2];
        stencil(vs + av, kVX, ev, ss + e, rec, fl);
        const FarPlane<T, kVX, kEX> far{vs + av, ev.lds, ss + e};
        T xi[3], Pa[3], xs[3], Ps[3];
        forcing_args_stencil<D, T, S>(far, muD, muF, ph, nb, own, rec, fl, cs.ge, cs.H, cs.vs, xi,
                                      Pa, xs, Ps);
        ProductForm<D, T> peq, pst;
        const T er = own.e * own.r;
        peq.init(er, xi, Pa);
        pst.init(er, xs, Ps);
        const T two_beta = T(2) * cs.vs.beta;
        const T omb = T(1) - cs.vs.beta;
        const float base = own_base<P>(own.e, ph);
        unroll<0, Q>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            constexpr int cx = Lat<D>::c[i][0], cy = Lat<D>::c[i][1], o = Lat<D>::opp[i];
            const T fi = decode<D, i, T>(raw[r][i], sigma(ii, ev, src_solid(ii, e)));
            const T feq = peq.template at<i>();
            const T fst = pst.template at<i>();
            const T fpc = (fi + two_beta * (feq - fi)) + omb * (fst - feq);
            const P out = encode<D, i, P>(fpc, base * weight<D, i>());
            if constexpr (PH == 0 || i == 0) {
                *at(plane(fout, o, g.N), nb.self()) = out;
            } else {  // bounced back where the destination is solid
                const bool back = S && ss[S ? e + cy * kEX + cx : 0];
                *at(plane(fout, back ? o : i, g.N), back ? nb.self() : nb.at(cx, cy, 0)) = out;
            }
        });
    }
}

}  // namespace lbm
