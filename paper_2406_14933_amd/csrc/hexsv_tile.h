// hexsv_tile.h — one explicit step of one TQ x TR tile of the raster.
//
// A tile step has three phases, kept apart so that a persistent kernel can
// overlap the loads of the next tile with the arithmetic of the current one:
//   load:    every thread loads (h, v1, v2, z, theta, alpha_p) of the cells it
//            owns (coalesced rows of the tile) and the halo slots of the tile
//            rim it is responsible for, into registers;
//   stage:   registers -> one 4-word LDS record per staged position,
//              {mass, w = g (z + h), v1/2, v2/2},
//            with mass = theta*h (FP64) or l*theta*h (FP32), plus an edge
//            code per position when the tile touches the raster boundary or
//            an inactive cell.  Interface velocities of eq. fvm_2D_eq.04 are
//            then one add (v_i/2 + v_j/2 equals (v_i + v_j)/2 exactly) and a
//            neighbour is one 16-byte LDS read;
//   compute: per owned cell, the six edge terms of eq. fvm_2D_eq_frac.01 with
//            the interface rules of eqs. fvm_2D_eq.05-.06, the mass update
//            with rain at t^{n+1} and clamping (eqs. .05-1/.06-1), and the
//            closed-form friction solve (Appendix A, miu-formula).
//
// FP64 evaluates the equations operation for operation as the CPU reference
// (contraction off); FP32 regroups them (J + S in one accumulator, l folded
// into the staged mass, depth updated by its increment) to save instructions
// and keep still water exactly still.
#pragma once

#include <type_traits>

#include "hexsv_device.h"

namespace hexsv {

template <typename T>
struct Rec;
template <>
struct Rec<float> {
    using type = float4;
};
template <>
struct Rec<double> {
    using type = double4;
};

// V: the step adds the artificial viscosity of the augmented momentum flux
// (eqs. eq_artif_visc, eq_visc1), which needs c = |v| + sqrt(g h) of every
// staged position as well.
template <typename T, int TQ, int TR, bool V = false>
struct TileLDS {
    static constexpr int W = TQ + 2, H = TR + 2, NS = W * H;
    typename Rec<T>::type rec[NS];
    uint8_t code[NS];
    T c[V ? NS : 1];
};

// Map ring index t (0 <= t < 2*(TQ+2) + 2*TR) to a halo slot (lq, lr) in
// staged coordinates (the tile's cells occupy lq in [1,TQ], lr in [1,TR]).
template <int TQ, int TR>
__device__ inline void ring_slot(int t, int &lq, int &lr) {
    constexpr int W = TQ + 2;
    if (t < W) { lq = t; lr = 0; }
    else if (t < 2 * W) { lq = t - W; lr = TR + 1; }
    else if (t < 2 * W + TR) { lq = 0; lr = 1 + (t - 2 * W); }
    else { lq = TQ + 1; lr = 1 + (t - 2 * W - TR); }
}

// Where a staged position lies: a cell of the tile, a raster cell reached
// through the halo (or a periodic wrap), or outside the raster.
enum : uint8_t { POS_OWN = 0, POS_NEIGHBOUR = 1, POS_OUTSIDE = 2 };

// SUB > 1: the tile is a stack of SUB sub-tiles of TQ x TR/SUB cells; each belongs to 256
// threads (real ones, or a second set that the same NT threads stand for), which own the
// cells that a workgroup of 256 threads with that tile alone would give them.
template <typename T, int TQ, int TR, int NT, int SUB = 1>
struct TileRegs {
    static constexpr int CPT = (TQ * TR) / NT;
    static constexpr int M = SUB == 1 ? NT : 256;        // threads of a sub-tile
    static constexpr int CPS = TQ * (TR / SUB) / M;      // cells of one of them
    // sub-tile of thread tid's k-th cell, and the cell's column and row in the tile
    __device__ static inline int sub_of(int tid, int k) {
        return SUB == 1 ? 0 : tid / M + (k / CPS) * (NT / M);
    }
    __device__ static inline void cell(int tid, int k, int &lq, int &lr) {
        const int sub = sub_of(tid, k);
        const int cc = (SUB == 1 ? tid : tid % M) + (k % CPS) * M;
        lr = cc / TQ;
        lq = cc - lr * TQ;
        lr += sub * (TR / SUB);
    }
    static constexpr int NRING = 2 * (TQ + 2) + 2 * TR;
    static constexpr int RPT = (NRING + NT - 1) / NT;
    static_assert(CPT * NT == TQ * TR, "tile must be a multiple of the workgroup");
    T h[CPT], th[CPT], ap[CPT], z[CPT], v1[CPT], v2[CPT];
    uint8_t pos[CPT];
    T rh[RPT], rth[RPT], rz[RPT], rv1[RPT], rv2[RPT];
    uint8_t rpos[RPT];
};

template <typename T>
__device__ inline typename Rec<T>::type make_rec(T m_or_M, T w, T vh1, T vh2) {
    typename Rec<T>::type r;
    r.x = m_or_M;
    r.y = w;
    r.z = vh1;
    r.w = vh2;
    return r;
}

template <typename T, bool NT_STORE>
__device__ inline void put(T *p, T v) {
    if constexpr (NT_STORE) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Per-thread accumulators of the step's reductions (c_max and FP64 books).
struct Acc {
    double c, s, o, cl;
};

__device__ inline bool tile_inner(const KGrid &g, int q0, int r0, int TQ, int TR) {
    return q0 >= 1 && q0 + TQ + 1 <= g.nq && r0 >= 1 && r0 + TR + 1 <= g.nr;
}

// ------------------------------------------------------------------ load

template <typename T, int TQ, int TR, int NT, int SUB = 1>
__device__ inline void tile_load(TileRegs<T, TQ, TR, NT, SUB> &R, const KDom<T> &d,
                                 const KGrid &g, int par, int tq, int tr) {
    using Regs = TileRegs<T, TQ, TR, NT, SUB>;
    const int q0 = tq * TQ, r0 = tr * TR;
    const T *__restrict__ hin = d.buf(par, 0);
    const T *__restrict__ v1in = d.buf(par, 1);
    const T *__restrict__ v2in = d.buf(par, 2);
    const bool inner = tile_inner(g, q0, r0, TQ, TR);
    // The state is read once per step.  Tiles 128 cells wide read their own cells with
    // streaming loads, which leave the L2 to the halo reads of neighbouring tiles; on
    // narrower tiles a larger share of each row is a neighbour's halo, and the ordinary
    // policy keeps those lines for it.
    constexpr bool STREAM = TQ >= 128;
#pragma unroll
    for (int k = 0; k < Regs::CPT; ++k) {
        int lq, lr;
        Regs::cell(threadIdx.x, k, lq, lr);
        int q = q0 + lq, r = r0 + lr;
        uint8_t pos = POS_OWN;
        if (!(inner || (q < g.nq && r < g.nr)))
            pos = wrap_pos(g, q, r) ? POS_NEIGHBOUR : POS_OUTSIDE;
        R.pos[k] = pos;
        if (pos != POS_OUTSIDE) {
            const uint32_t i = (uint32_t)(r * g.pitch + q);
            // the static fields always use the ordinary cache policy
            R.h[k] = STREAM ? ld_stream(hin, i) : ld(hin, i);
            R.th[k] = ld(d.th, i);
            R.ap[k] = ld(d.ap, i);
            R.z[k] = ld(d.z, i);
            R.v1[k] = STREAM ? ld_stream(v1in, i) : ld(v1in, i);
            R.v2[k] = STREAM ? ld_stream(v2in, i) : ld(v2in, i);
        }
    }
#pragma unroll
    for (int k = 0; k < Regs::RPT; ++k) {
        const int t = threadIdx.x + k * NT;
        R.rpos[k] = POS_OUTSIDE;
        if (t < Regs::NRING) {
            int lq, lr;
            ring_slot<TQ, TR>(t, lq, lr);
            int q = q0 + lq - 1, r = r0 + lr - 1;
            if (inner || wrap_pos(g, q, r)) {
                R.rpos[k] = POS_NEIGHBOUR;
                const uint32_t i = (uint32_t)(r * g.pitch + q);
                R.rh[k] = ld(hin, i);
                R.rth[k] = ld(d.th, i);
                R.rz[k] = ld(d.z, i);
                R.rv1[k] = ld(v1in, i);
                R.rv2[k] = ld(v2in, i);
            }
        }
    }
}

// ----------------------------------------------------------------- stage

// The staged record of a raster cell, {mass, w, v1/2, v2/2} (see the file's head).
// EXT: the cell may be a boundary cell: Dirichlet (-theta: |theta| h) or given flux
// (-2: the discharge's depth, and the bed only, as the edge adds the cell's depth).
template <typename T, bool EXT>
__device__ inline typename Rec<T>::type cell_rec(T h, T th, T z, T v1, T v2, T G, T mscale) {
    if constexpr (EXT) {
        const bool fl = th < T(-1.5);
        const T m = fl ? h : __builtin_fabs(th) * h;
        const T w = fl ? z : G * (z + h);
        return make_rec<T>(mscale * m, w, v1 * T(0.5), v2 * T(0.5));
    } else {
        const T m = th * h;
        return make_rec<T>(mscale * m, G * (z + h), v1 * T(0.5), v2 * T(0.5));
    }
}

// Its edge code as its neighbours see it.
template <typename T, bool EXT>
__device__ inline uint8_t cell_code(T th, const KGrid &g) {
    if constexpr (EXT)
        return th > T(0) ? (uint8_t)CODE_INTERIOR
                         : (th < T(-1.5) ? (uint8_t)CODE_FLUX
                                         : th < T(0) ? (uint8_t)CODE_DIRICHLET
                                                     : (uint8_t)g.mask_bc);
    else
        return th > T(0) ? (uint8_t)CODE_INTERIOR : (uint8_t)g.mask_bc;
}

// Its wave speed for the viscous flux.
template <typename T>
__device__ inline T cell_wave(T h, T v1, T v2, T G) {
    T vv;  // the fused square is named, so that every kernel rounds c alike
    if constexpr (sizeof(T) == 4) vv = __builtin_fmaf(v1, v1, v2 * v2);
    else vv = v1 * v1 + v2 * v2;
    return p_sqrt(vv) + p_sqrt(G * h);
}

// Write the LDS records; returns true if a staged raster cell is inactive.
// EXT: the extended scheme: the raster may hold Dirichlet or given-flux cells
// (theta < 0), and the mass source may lose infiltration; the plain instance keeps
// the plain records and mass update.
template <typename T, int TQ, int TR, int NT, bool EXT = false, bool V, int SUB>
__device__ inline bool tile_stage(TileLDS<T, TQ, TR, V> &L,
                                  const TileRegs<T, TQ, TR, NT, SUB> &R, const KGrid &g,
                                  const KConst &kc, int tq, int tr) {
    using Regs = TileRegs<T, TQ, TR, NT, SUB>;
    constexpr int W = TQ + 2;
    constexpr bool F32 = sizeof(T) == 4;
    const int q0 = tq * TQ, r0 = tr * TR;
    const bool inner = tile_inner(g, q0, r0, TQ, TR);
    const bool need_codes = !inner || g.has_mask;
    const T G = (T)kc.g;
    const T mscale = F32 ? (T)kc.a : T(1);
    bool bad = false;
    auto put_cell = [&](int s, uint8_t pos, T h, T th, T z, T v1, T v2, int q, int r) {
        if (pos != POS_OUTSIDE) {
            L.rec[s] = cell_rec<T, EXT>(h, th, z, v1, v2, G, mscale);
            if (need_codes) L.code[s] = cell_code<T, EXT>(th, g);
            if constexpr (V) L.c[s] = cell_wave(h, v1, v2, G);
            bad |= !(th > T(0));
        } else {
            wrap_pos(g, q, r);
            L.rec[s] = make_rec<T>(T(0), T(0), T(0), T(0));
            if constexpr (V) L.c[s] = T(0);
            L.code[s] = (uint8_t)side_code(g, q, r);
        }
    };
#pragma unroll
    for (int k = 0; k < Regs::CPT; ++k) {
        int lq, lr;
        Regs::cell(threadIdx.x, k, lq, lr);
        put_cell((lr + 1) * W + (lq + 1), R.pos[k], R.h[k], R.th[k], R.z[k], R.v1[k], R.v2[k],
                 q0 + lq, r0 + lr);
    }
#pragma unroll
    for (int k = 0; k < Regs::RPT; ++k) {
        const int t = threadIdx.x + k * NT;
        if (t >= Regs::NRING) continue;
        int lq, lr;
        ring_slot<TQ, TR>(t, lq, lr);
        put_cell(lr * W + lq, R.rpos[k], R.rh[k], R.rth[k], R.rz[k], R.rv1[k], R.rv2[k],
                 q0 + lq - 1, r0 + lr - 1);
    }
    return bad;
}

// Where a step's results go: into the other buffer, with the first non-finite cell
// of the step named in the control block.
template <typename T, bool NT_STORE>
struct StoreSink {
    T *__restrict__ hout;
    T *__restrict__ v1out;
    T *__restrict__ v2out;
    int32_t *err_flag, *err_cell;
    __device__ inline void put_state(int, uint32_t i, T h, T v1, T v2) {
        put<T, NT_STORE>(at(hout, i), h);
        put<T, NT_STORE>(at(v1out, i), v1);
        put<T, NT_STORE>(at(v2out, i), v2);
    }
    __device__ inline void nonfinite(uint32_t i) {
        if (atomicOr(err_flag, 1) == 0) *err_cell = (int32_t)i;
    }
    // rare: was this one of the offending cells?  (the values this thread just stored)
    __device__ inline void rescan(uint32_t i) {
        if (!__builtin_isfinite(ld(hout, i)) || !__builtin_isfinite(ld(v1out, i)) ||
            !__builtin_isfinite(ld(v2out, i)))
            nonfinite(i);
    }
};

// --------------------------------------------------------------- compute

// What a step's cells share.
template <typename T>
struct StepConst {
    T dt, dts, r, alpha_s, ftau, h_dry;
    bool lin;
};
template <typename T>
__device__ inline StepConst<T> step_const(const KConst &kc, double dt, double r_next) {
    StepConst<T> c;
    c.dt = (T)dt;
    c.dts = (T)(dt / kc.sigma);
    c.r = (T)r_next;
    c.alpha_s = (T)kc.alpha_s;
    // linear soil resistance theta tau h v, implicit in v^{n+1}: the coefficient of
    // v is m^{n+1} + dt tau m^{n+1} = m^{n+1} (1 + dt tau) (exactly m^{n+1} at tau = 0)
    c.lin = kc.tau_lin != 0.0;
    c.ftau = T(1) + c.dt * (T)kc.tau_lin;
    c.h_dry = (T)kc.h_dry;
    return c;
}

// Edge sums of a cell's step (what does not depend on dt): L, J (with V, J^v) + S, and
// the outward flux of open edges; with them the cell's staged half velocity.
template <typename T>
struct EdgeSums {
    T Ls, A1, A2, Fout, vh1, vh2;
};

// A thread's partial reductions that FP32 keeps in FP32 until its last cell: c_max, the sum
// of theta h, and a sum that any non-finite h or v makes non-finite.
struct Partial32 {
    float cmax = 0.f, m = 0.f, any = 0.f;
};

// The step of thread tid's cells of the tile staged in L: edges, then finish.  SHORT: FP64
// leaves the products by 0 and 1 of edges 0 and 3 out (same results).  That is less arithmetic,
// which the on-chip kernels (1024 x 1024: 2582 -> 2541 us per 100 steps) and the viscous steps
// gain from; in the launches of one step it costs registers: the plain 64 x 16 step takes 131,
// three waves per SIMD, against 121 and four, and the persistent ensemble kernel spills 61
// against 27 (256 rasters of 128 x 128: 181 against 119 us a step).
template <typename T, int TQ, int TR, int NT, bool V, bool EXT, int SUB, bool SHORT>
struct TileCells {
    using Regs = TileRegs<T, TQ, TR, NT, SUB>;
    static constexpr int W = TQ + 2;
    static constexpr bool F32 = sizeof(T) == 4;
    const TileLDS<T, TQ, TR, V> &L;
    const Regs &R;
    const KDom<T> &d;
    const KGrid &g;
    const KConst &kc;
    int q0, r0;
    T G, l, half_l;

    __device__ inline TileCells(const TileLDS<T, TQ, TR, V> &L_, const Regs &R_, const KDom<T> &d_,
                                const KGrid &g_, const KConst &kc_, int tq, int tr)
        : L(L_), R(R_), d(d_), g(g_), kc(kc_), q0(tq * TQ), r0(tr * TR), G((T)kc_.g),
          l((T)kc_.a), half_l((T)(0.5 * kc_.a)) {}

    // GEN: edges may be walls, open, or lead to boundary cells (codes are staged).  LIKE_GEN:
    // FP32 rounds as the general path does (see edge_vn), for interior cells beside those.
    template <bool GEN, bool LIKE_GEN = false>
    __device__ inline EdgeSums<T> edges(int tid, int k) const {
        const T S3H = (T)0.86602540378443864676;
        const T NX[6] = {T(1), T(0.5), T(-0.5), T(-1), T(-0.5), T(0.5)};
        const T NY[6] = {T(0), S3H, S3H, T(0), -S3H, -S3H};
        const T NXh[6] = {T(0.5), T(0.25), T(-0.25), T(-0.5), T(-0.25), T(0.25)};
        const T NYh[6] = {T(0), T(0.5) * S3H, T(0.5) * S3H, T(0), -T(0.5) * S3H, -T(0.5) * S3H};
        constexpr int OFF[6] = {1, W, W - 1, -1, -W, -W + 1};
        int lq, lr;
        Regs::cell(tid, k, lq, lr);
        const int s = (lr + 1) * W + (lq + 1);
        const int q = q0 + lq, r = r0 + lr;
        const T hi = R.h[k];
        const T mi = R.th[k] * hi;
        // the cell's own staged record (the values its neighbours see, formed by the same
        // operations), so that the bed register is free after staging; FP32 also takes
        // its velocity as twice the staged half, FP64 keeps the loaded one
        const typename Rec<T>::type me = L.rec[s];
        const T Mi = me.x, wi = me.y, vh1i = me.z, vh2i = me.w;
        T Ls = T(0), A1 = T(0), A2 = T(0), S1 = T(0), S2 = T(0), Fout = T(0);
        T V1 = T(0), V2 = T(0);
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            const int sn = s + OFF[e];
            T mj, wj, vh1j, vh2j;
            int cd = CODE_INTERIOR;
            if constexpr (GEN) {
                cd = L.code[sn];
                if (cd == CODE_WALL) continue;
            }
            // a cell: interior (or, EXT, a Dirichlet or flux cell)
            if (!GEN || (EXT ? cd != CODE_OUTFLOW : cd == CODE_INTERIOR)) {
                const typename Rec<T>::type nb = L.rec[sn];
                mj = nb.x;
                wj = nb.y;
                vh1j = nb.z;
                vh2j = nb.w;
            } else {
                // free outflow ghost: the cell's h, v, theta; terrain extrapolated linearly
                // through the opposite neighbour (read from memory: rim cells only)
                wj = wi;
                if (L.code[s - OFF[e]] == CODE_INTERIOR) {
                    int qo = q - dq_of(e), ro = r - dr_of(e);
                    wrap_pos(g, qo, ro);
                    const T zi = ld(d.z, (uint32_t)(r * g.pitch + q));
                    const T zg = T(2) * zi - d.z[(int64_t)ro * g.pitch + qo];
                    wj = G * (zg + hi);
                }
                mj = Mi;
                vh1j = vh1i;
                vh2j = vh2i;
            }
            // interface velocity; an edge to a Dirichlet or flux cell carries the prescribed one
            T vb1 = vh1i + vh1j;
            T vb2 = vh2i + vh2j;
            if (EXT && GEN && cd >= CODE_DIRICHLET) {
                vb1 = vh1j + vh1j;
                vb2 = vh2j + vh2j;
            }
            if (EXT && GEN && cd == CODE_FLUX) {
                // given mass flux: the discharge h_j v_j crosses the edge whatever the cell
                // holds; the pressure term sees the cell's own depth over the neighbour's
                // bed (wj holds that bed level)
                if constexpr (F32) {
                    const T vn = edge_vn(e, vb1, vb2);
                    T F = mj * vn;  // mj holds l h_j
                    edge_mass(Ls, F, mj, vn);
                    A1 = __builtin_fmaf(-F, vb1, A1);
                    A2 = __builtin_fmaf(-F, vb2, A2);
                    const T Q = __builtin_fmaf(G, wj + hi, -wi) * Mi;
                    A1 = __builtin_fmaf(-Q, NXh[e], A1);
                    if (e != 0 && e != 3) A2 = __builtin_fmaf(-Q, NYh[e], A2);
                    Fout = __builtin_fmaf(mj, vn, Fout);
                } else {
                    const T vn = vb1 * NX[e] + vb2 * NY[e];
                    const T F = l * mj * vn;
                    Ls -= F;
                    A1 -= F * vb1;
                    A2 -= F * vb2;
                    const T P = half_l * (G * (wj + hi) - wi) * mi;
                    S1 -= P * NX[e];
                    S2 -= P * NY[e];
                    Fout += F;
                }
                continue;
            }
            if constexpr (F32) {
                // mj holds l*theta_j*h_j
                T vn;
                if constexpr (GEN || LIKE_GEN) vn = edge_vn(e, vb1, vb2);
                else vn = (e == 0) ? vb1 : ((e == 3) ? -vb1 : vb1 * NX[e] + vb2 * NY[e]);
                const T dw = wj - wi;
                // one selected mass serves both terms: the upwind mass of the flux
                // (at vn = 0 the flux vanishes whatever it is) and the pressure mass,
                // which at vn = 0 follows the free-surface tie rule
                const T key = (vn != T(0)) ? vn : -dw;  // w_i > w_j decides at vn = 0
                const T msel = key > T(0) ? Mi : mj;
                T F = msel * vn;
                const T Q = dw * msel;
                if constexpr (GEN || LIKE_GEN) {
                    edge_mass(Ls, F, msel, vn);
                    A1 = __builtin_fmaf(-F, vb1, A1);
                    A2 = __builtin_fmaf(-F, vb2, A2);
                    A1 = __builtin_fmaf(-Q, NXh[e], A1);
                    if (e != 0 && e != 3) A2 = __builtin_fmaf(-Q, NYh[e], A2);
                } else {
                    Ls -= F;
                    A1 -= F * vb1;
                    A2 -= F * vb2;
                    A1 -= Q * NXh[e];
                    if (e != 0 && e != 3) A2 -= Q * NYh[e];
                }
                if (GEN && (EXT ? cd != CODE_INTERIOR : cd == CODE_OUTFLOW))
                    Fout = __builtin_fmaf(msel, vn, Fout);  // outflow or Dirichlet edge
            } else {
                const bool flat = SHORT && (e == 0 || e == 3);
                const T vn = flat ? (e == 0 ? vb1 : -vb1) : vb1 * NX[e] + vb2 * NY[e];
                // one selected mass, as above: at vn = 0 the flux vanishes whatever it is
                bool own;
                if constexpr (SHORT) {
                    own = vn > T(0) || (vn == T(0) && wi > wj);
                } else {
                    const T key = vn != T(0) ? vn : wi - wj;
                    own = key > T(0);
                }
                const T msel = own ? mi : mj;
                const T F = l * msel * vn;
                Ls -= F;
                A1 -= F * vb1;
                A2 -= F * vb2;
                const T P = half_l * (wj - wi) * msel;
                S1 -= P * NX[e];
                if (!flat) S2 -= P * NY[e];
                if (GEN && (EXT ? cd != CODE_INTERIOR : cd == CODE_OUTFLOW))
                    Fout += F;  // outflow or Dirichlet edge
            }
            if constexpr (V) {
                // artificial viscosity l c_ij mu_ij (v_j - v_i) of an interior edge (an
                // outflow ghost carries the cell's own velocity); (v_j - v_i) is twice the
                // difference of the staged halves, exactly.  FP32 masses carry the l.
                if (!GEN || cd == CODE_INTERIOR) {
                    const T ci = L.c[s], cj = L.c[sn];
                    const T cij = ci > cj ? ci : cj;
                    const T ms = Mi + mj;
                    const T mu = ms > T(0) ? p_div(T(2) * Mi * mj, ms) : T(0);
                    const T lc = F32 ? cij : l * cij;
                    V1 += lc * mu * (T(2) * (vh1j - vh1i));
                    V2 += lc * mu * (T(2) * (vh2j - vh2i));
                }
            }
        }
        if constexpr (V) {
            A1 = A1 + V1;
            A2 = A2 + V2;
        }
        if constexpr (!F32) {  // FP32 sums the pressure part with J
            A1 = A1 + S1;
            A2 = A2 + S2;
        }
        return EdgeSums<T>{Ls, A1, A2, Fout, vh1i, vh2i};
    }

    // A cell's edge codes as a word, three bits each, for kernels that keep it over many
    // steps; the beds of its outflow ghosts go to consecutive entries of a table in LDS (at
    // most three per cell), the first one's number to the word's upper bits.
    static constexpr uint32_t CODE_FLAT = 6;  // outflow without extrapolation
    __device__ inline uint32_t edge_codes(int tid, int k, T *ghosts, int *count) const {
        constexpr int OFF[6] = {1, W, W - 1, -1, -W, -W + 1};
        int lq, lr;
        Regs::cell(tid, k, lq, lr);
        const int s = (lr + 1) * W + (lq + 1);
        const int q = q0 + lq, r = r0 + lr;
        uint32_t ec = 0;
        int n = 0;
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            const uint32_t cd = L.code[s + OFF[e]], op = L.code[s - OFF[e]];
            const bool bed = cd == CODE_OUTFLOW && op == CODE_INTERIOR;
            n += bed ? 1 : 0;
            ec |= (cd == CODE_OUTFLOW && !bed ? CODE_FLAT : cd) << (3 * e);
        }
        if (n > 0) {
            uint32_t at = (uint32_t)atomicAdd(count, n);
            ec |= at << 18;
#pragma unroll 1
            for (int e = 0; e < 6; ++e)
                if (((ec >> (3 * e)) & 7) == CODE_OUTFLOW) {
                    int qo = q - dq_of(e), ro = r - dr_of(e);
                    wrap_pos(g, qo, ro);
                    const T zi = ld(d.z, (uint32_t)(r * g.pitch + q));
                    ghosts[at++] = T(2) * zi - d.z[(int64_t)ro * g.pitch + qo];
                }
        }
        return ec;
    }

    // The normal velocity of edge e and the flux's part in the mass sum of the general path.
    // FP32's fused multiply-adds are written out there, so that all its forms (edges<true>,
    // edges_fixed, edges<false, true>) round alike whatever the compiler would fuse.
    __device__ static inline T edge_vn(int e, T vb1, T vb2) {
        const T S3H = (T)0.86602540378443864676;
        const T NX[6] = {T(1), T(0.5), T(-0.5), T(-1), T(-0.5), T(0.5)};
        const T NY[6] = {T(0), S3H, S3H, T(0), -S3H, -S3H};
        if (e == 0) return vb1;
        if (e == 3) return -vb1;
        if constexpr (F32)
            return e == 5 ? __builtin_fmaf(vb1, NX[e], vb2 * NY[e])
                          : __builtin_fmaf(vb2, NY[e], vb1 * NX[e]);
        else return vb1 * NX[e] + vb2 * NY[e];
    }
    __device__ static inline void edge_mass(T &Ls, T &F, T m, T vn) {
        if constexpr (EXT) {  // F = m vn, rounded
            asm("" : "+v"(F));
            Ls -= F;
        } else {
            Ls = __builtin_fmaf(-m, vn, Ls);
        }
    }

    // edges<true> with the codes of edge_codes: the same sums bit for bit.  Every kind of edge
    // is a choice of values here, not of paths: the staged codes' way costs a chain of LDS
    // reads per edge (the code, then the record) and two reads of memory per open edge, which
    // the many-step kernels would wait for in every step.
    __device__ inline EdgeSums<T> edges_fixed(int tid, int k, uint32_t ec, const T *ghosts) const {
        const T S3H = (T)0.86602540378443864676;
        const T NX[6] = {T(1), T(0.5), T(-0.5), T(-1), T(-0.5), T(0.5)};
        const T NY[6] = {T(0), S3H, S3H, T(0), -S3H, -S3H};
        const T NXh[6] = {T(0.5), T(0.25), T(-0.25), T(-0.5), T(-0.25), T(0.25)};
        const T NYh[6] = {T(0), T(0.5) * S3H, T(0.5) * S3H, T(0), -T(0.5) * S3H, -T(0.5) * S3H};
        constexpr int OFF[6] = {1, W, W - 1, -1, -W, -W + 1};
        int lq, lr;
        Regs::cell(tid, k, lq, lr);
        const int s = (lr + 1) * W + (lq + 1);
        const T hi = R.h[k];
        const T mi = R.th[k] * hi;
        const typename Rec<T>::type me = L.rec[s];
        const T Mi = me.x, wi = me.y, vh1i = me.z, vh2i = me.w;
        typename Rec<T>::type nbs[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) nbs[e] = L.rec[s + OFF[e]];
        uint32_t ghost = ec >> 18;
        T Ls = T(0), A1 = T(0), A2 = T(0), S1 = T(0), S2 = T(0), Fout = T(0);
        T V1 = T(0), V2 = T(0);
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            const uint32_t cd = (ec >> (3 * e)) & 7;
            const bool in = cd == CODE_INTERIOR, wall = cd == CODE_WALL, bed = cd == CODE_OUTFLOW;
            const bool held = EXT && (cd == CODE_DIRICHLET || cd == CODE_FLUX);
            const bool flux = EXT && cd == CODE_FLUX;
            const bool cell = in || held;
            const T mj = cell ? nbs[e].x : Mi;
            const T vh1j = cell ? nbs[e].z : vh1i, vh2j = cell ? nbs[e].w : vh2i;
            T wj = cell ? nbs[e].y : wi;
            if (__any(bed)) {
                const T wg = G * (ghosts[bed ? ghost : 0] + hi);
                wj = bed ? wg : wj;
                ghost += bed ? 1 : 0;
            }
            const T vb1 = (held ? vh1j : vh1i) + vh1j;
            const T vb2 = (held ? vh2j : vh2i) + vh2j;
            T vn = edge_vn(e, vb1, vb2);
            T dw = wj - wi;
            if constexpr (EXT) {
                T wf;
                if constexpr (F32) wf = __builtin_fmaf(G, wj + hi, -wi);
                else wf = G * (wj + hi) - wi;
                dw = flux ? wf : dw;
            }
            vn = wall ? T(0) : vn;  // no flux and no pressure difference
            dw = wall ? T(0) : dw;
            if constexpr (F32) {
                const T key = (vn != T(0)) ? vn : -dw;
                const T msel = key > T(0) ? Mi : mj;
                const T mf = flux ? mj : msel, mp = flux ? Mi : msel;
                T F = mf * vn;
                edge_mass(Ls, F, mf, vn);
                A1 = __builtin_fmaf(-F, vb1, A1);
                A2 = __builtin_fmaf(-F, vb2, A2);
                const T Q = dw * mp;
                A1 = __builtin_fmaf(-Q, NXh[e], A1);
                if (e != 0 && e != 3) A2 = __builtin_fmaf(-Q, NYh[e], A2);
                const T Fo = __builtin_fmaf(mf, vn, Fout);
                Fout = in || wall ? Fout : Fo;
            } else {
                const bool own = vn > T(0) || (vn == T(0) && wi > wj);
                const T msel = own ? mi : mj;
                const T mf = flux ? mj : msel, mp = flux ? mi : msel;
                const T F = l * mf * vn;
                Ls -= F;
                A1 -= F * vb1;
                A2 -= F * vb2;
                const T P = half_l * dw * mp;
                S1 -= P * NX[e];
                if (e != 0 && e != 3) S2 -= P * NY[e];
                Fout = in || wall ? Fout : Fout + F;
            }
            if constexpr (V) {
                const T ci = L.c[s], cj = L.c[s + OFF[e]];
                const T cij = ci > cj ? ci : cj;
                const T ms = Mi + mj;
                T mu = ms > T(0) ? p_div(T(2) * Mi * mj, ms) : T(0);
                mu = in ? mu : T(0);
                const T lc = F32 ? cij : l * cij;
                V1 += lc * mu * (T(2) * (vh1j - vh1i));
                V2 += lc * mu * (T(2) * (vh2j - vh2i));
            }
        }
        if constexpr (V) {
            A1 = A1 + V1;
            A2 = A2 + V2;
        }
        if constexpr (!F32) {
            A1 = A1 + S1;
            A2 = A2 + S2;
        }
        return EdgeSums<T>{Ls, A1, A2, Fout, vh1i, vh2i};
    }

    // The new state from the sums: mass and depth, friction solve, reductions.
    template <bool GEN, typename Sink>
    __device__ inline void finish(int tid, int k, const EdgeSums<T> &es, const StepConst<T> &sc,
                                  double dt, Acc &acc, Partial32 &p32, Sink &sink) const {
        const T dtT = sc.dt, dts = sc.dts, rT = sc.r, ftau = sc.ftau, h_dry = sc.h_dry;
        const T Ls = es.Ls, A1 = es.A1, A2 = es.A2, Fout = es.Fout;
        int lq, lr;
        Regs::cell(tid, k, lq, lr);
        const int q = q0 + lq, r = r0 + lr;
        const T hi = R.h[k], thi = R.th[k];
        const T mi = thi * hi;
        const T vh1i = es.vh1, vh2i = es.vh2;
        const T v1i = F32 ? vh1i + vh1i : R.v1[k], v2i = F32 ? vh2i + vh2i : R.v2[k];
        T m1, h1, g1, g2;
        if constexpr (F32) {
            // fused multiply-adds are written out where the compiler could place them
            // otherwise from one kernel to the next (a factor formed outside the block, a
            // product with one use or several), so that every kernel of a tile shape
            // rounds alike; with one cell per thread the rain term is the fused one
            const T dm = Regs::CPS == 1 ? __builtin_fmaf(dtT, rT, dts * Ls)
                                        : __builtin_fmaf(dts, Ls, dtT * rT);
            m1 = __builtin_fmaf(thi, hi, dm);
            if (m1 < T(0)) {
                acc.cl += kc.sigma * (-(double)m1);
                m1 = T(0);
                h1 = T(0);
            } else {
                h1 = __builtin_fmaf(dm, __builtin_amdgcn_rcpf(thi), hi);  // hi + p_div(dm, thi)
                h1 = h1 > T(0) ? h1 : T(0);
            }
            g1 = __builtin_fmaf(mi, v1i, dts * A1);
            g2 = __builtin_fmaf(mi, v2i, dts * A2);
        } else {
            const T ms = mi + dts * Ls;
            m1 = ms + dtT * rT;
            if (m1 < T(0)) {
                acc.cl += kc.sigma * (-(double)m1);
                m1 = T(0);
            }
            h1 = p_div(m1, thi);
            g1 = mi * v1i + dts * A1;
            g2 = mi * v2i + dts * A2;
        }
        if constexpr (EXT) {
            if (kc.f_inf > 0.0 && m1 > T(0)) {
                // the mass source r - i(h^{n+1}) with i(h) = f h / (h + c) turns the mass
                // update into theta x + dt f x / (x + c) = m1 for x = h^{n+1}.  With
                // x = h1 - e (h1: the depth without infiltration, which FP32 keeps as an
                // increment) the loss e is the smaller root of theta e^2 - P e + dt f h1,
                // P = theta (h1 + c) + dt f; the soil's water is booked with the outflow
                const T c = (T)kc.h_inf, fd = dtT * (T)kc.f_inf, hs = h1;
                T x, lost;
                if constexpr (F32) {
                    const T P = __builtin_fmaf(thi, hs + c, fd);
                    const T Q = __builtin_fmaf(thi, hs + c, -fd);
                    const T Dq = __builtin_fmaf(T(4) * thi * fd, c, Q * Q);
                    x = __builtin_fmaf(-(T(2) * fd * hs), __builtin_amdgcn_rcpf(P + p_sqrt(Dq)), hs);
                    lost = __builtin_fmaf(-thi, x, m1);
                } else {
                    const T P = thi * (hs + c) + fd;
                    const T Q = thi * (hs + c) - fd;
                    const T Dq = Q * Q + T(4) * thi * fd * c;
                    const T e = p_div(T(2) * fd * hs, P + p_sqrt(Dq));
                    x = hs - e;
                    lost = m1 - thi * x;
                }
                const T mx = thi * x;
                acc.o += kc.sigma * (double)lost;
                m1 = mx;
                h1 = x;
            }
        }
        const uint32_t i = (uint32_t)(r * g.pitch + q);
        T as_i = sc.alpha_s;
        if constexpr (EXT) {
            if (d.as) as_i = ld(d.as, i);  // a soil coefficient per cell
        }
        T K;
        if constexpr (F32 && EXT) K = __builtin_fmaf(R.ap[k] * h1, T(1) - thi, thi * as_i);
        else if constexpr (F32) K = __builtin_fmaf(thi, as_i, R.ap[k] * h1 * (T(1) - thi));
        else K = R.ap[k] * h1 * (T(1) - thi) + thi * as_i;
        const T beta = dtT * K;
        T gg;
        if constexpr (F32) gg = GEN ? __builtin_fmaf(g2, g2, g1 * g1) : __builtin_fmaf(g1, g1, g2 * g2);
        else gg = g1 * g1 + g2 * g2;
        const T Gm = p_sqrt(gg);
        T alpha = m1;
        if (sc.lin) alpha = m1 * ftau;
        T disc;
        if constexpr (F32) disc = __builtin_fmaf(alpha, alpha, T(4) * beta * Gm);
        else disc = alpha * alpha + T(4) * beta * Gm;
        const T D = alpha + p_sqrt(disc);
        T mu = (D == T(0)) ? T(0) : p_div(T(2), D);
        if (h_dry > T(0) && h1 < h_dry) mu = T(0);
        const T v1n = mu * g1, v2n = mu * g2;
        sink.put_state(k, i, h1, v1n, v2n);
        // wave speed of the new state (eq. fvm_2D_eq_frac.13); FP32 takes |v^{n+1}| as
        // mu |gamma| (the same value up to rounding), FP64 the oracle's sqrt(v1^2 + v2^2)
        T cc2;
        if constexpr (F32) cc2 = __builtin_fmaf(Gm, mu, p_sqrt(G * h1));
        else cc2 = p_sqrt(v1n * v1n + v2n * v2n) + p_sqrt(G * h1);
        if constexpr (F32) {
            // FP32 partials over this thread's cells, folded into the FP64 books below;
            // p32.any carries any non-finite h or v of the thread's cells to one check
            p32.cmax = cc2 > p32.cmax ? cc2 : p32.cmax;
            p32.m = __builtin_fmaf(thi, h1, p32.m);
            p32.any += cc2;
        } else {
            acc.c = (double)cc2 > acc.c ? (double)cc2 : acc.c;
            acc.s += kc.sigma * ((double)thi * (double)h1);
            if (!__builtin_isfinite(h1) || !__builtin_isfinite(v1n) || !__builtin_isfinite(v2n))
                sink.nonfinite(i);
        }
        if (GEN) acc.o += dt * (double)Fout;
    }

    // FP32: the thread's partials into the FP64 accumulators, after the last of the cells
    // (k0 to k1) that they cover.
    template <typename Sink>
    __device__ inline void fold32(int tid, int k0, int k1, Acc &acc, const Partial32 &p32,
                                  Sink &sink) const {
        if constexpr (F32) {
            acc.c = (double)p32.cmax > acc.c ? (double)p32.cmax : acc.c;
            acc.s += kc.sigma * (double)p32.m;
            if (!__builtin_isfinite(p32.m + p32.any)) {
                // rare: find the offending cell among the thread's
#pragma unroll
                for (int k = k0; k < k1; ++k) {
                    if (R.pos[k] != POS_OWN) continue;
                    int lq, lr;
                    Regs::cell(tid, k, lq, lr);
                    sink.rescan((uint32_t)((r0 + lr) * g.pitch + q0 + lq));
                }
            }
        }
    }
};

// The step of a tile into the other buffer.
template <typename T, int TQ, int TR, int NT, bool NT_STORE, bool V, bool EXT = false>
__device__ inline void tile_compute(const TileLDS<T, TQ, TR, V> &L, const TileRegs<T, TQ, TR, NT> &R,
                                    bool general, const KDom<T> &d, const KGrid &g,
                                    const KConst &kc, int par, int tq, int tr, double dt,
                                    double r_next, Acc &acc, int32_t *err_flag,
                                    int32_t *err_cell) {
    using Regs = TileRegs<T, TQ, TR, NT>;
    StoreSink<T, NT_STORE> sink{d.buf(par ^ 1, 0), d.buf(par ^ 1, 1), d.buf(par ^ 1, 2), err_flag,
                                err_cell};
    const TileCells<T, TQ, TR, NT, V, EXT, 1, V> cells(L, R, d, g, kc, tq, tr);
    const StepConst<T> sc = step_const<T>(kc, dt, r_next);
    Partial32 p32;
    const int tid = threadIdx.x;
    auto cell = [&](int k, auto gen) {
        constexpr bool GEN = decltype(gen)::value;
        const EdgeSums<T> es = cells.template edges<GEN>(tid, k);
        // FP32 with 1024 threads (128 registers each): the cell's place is formed again after its
        // edges rather than kept through them: 27 registers spill instead of 33 with two
        // cells a thread (FP64 would spill 63 instead of 27 with one)
        int again = tid;
        if constexpr (NT == 1024 && sizeof(T) == 4) asm volatile("" : "+v"(again));
        cells.template finish<GEN>(again, k, es, sc, dt, acc, p32, sink);
    };
    if (general) {
#pragma unroll
        for (int k = 0; k < Regs::CPT; ++k)
            if (R.pos[k] == POS_OWN && R.th[k] > T(0)) cell(k, std::true_type{});
    } else {
#pragma unroll
        for (int k = 0; k < Regs::CPT; ++k) cell(k, std::false_type{});
    }
    cells.fold32(tid, 0, Regs::CPT, acc, p32, sink);
}

}  // namespace hexsv
