// hexsv_resident.h — many steps of a raster that fits on the chip, in one launch.
//
// A step of a small raster is bound by what surrounds it: a launch per step, whose
// workgroups load the tile, wait for the control block, reduce and drain (7.5 us for 64 x 64
// cells, 8.5 us for 512 x 512, 14 us for 1024 x 1024, of which the arithmetic and the cached
// traffic are a few).  When the tiles of the raster can all be resident at once, one launch
// keeps each tile's state and static fields in registers for up to ring_len steps, and per
// step exchanges only what other workgroups need: the rim cells of every tile, and every
// tile's largest wave speed, from which each workgroup derives the next time step by itself.
//
// Exchange.  Each 32-bit half of a value travels in a 64-bit word with the step's tag, stored
// and loaded as relaxed agent-scope atomics (write-through, read past the XCD's own L2): a
// reader polls the word until the tag is the one it waits for, so no fence, no cache
// write-back and no separate flag orders the data.  Words are double-buffered by the tag's
// parity: a workgroup that writes step n + 2 has seen every workgroup's wave speed of step
// n + 1, which each published after it had read all it needs of step n.
//
// Residency.  Nothing in the launch itself guarantees that all workgroups run at the same
// time, so the first exchange is a roll call with a bounded wait; whoever waits too long (or
// finds a non-finite value, or a wave speed that overflows) marks the launch as given up and
// leaves, and so do all others.  The launch's start state is never written: the result goes
// to the other buffer, and the fold that follows commits it only if every workgroup has
// reached the end.  Otherwise it sets the abort word of the launch queued behind this one, whose
// roll call then fails at the first look at that word (256 polls) if it has to wait again; a test
// of a flag at the kernel's start cost 1 to 3 % of a small raster's step.  The host then repeats
// the steps with one launch each, which also names a non-finite cell.  Every wait is bounded.
//
// The arithmetic, the tiles whose books are recorded and the threads that sum them are those
// of k_step with the same tile variant, so state and books are the same bit for bit.
//
// Bound by the chain of a step: rim words out, a poll that sees them (about 1.5 us across
// XCDs), edges, wave speeds out and polled again, cells, two barriers; for 1024 x 1024 by the
// arithmetic of four tiles per CU as well.  Share of a SIMD's cycles in which it issues vector
// arithmetic, and of the waves' time spent waiting: 64 x 64 FP64 0.37 and 0.42 (one wave per
// SIMD), 1024 x 1024 FP32 0.66 and 0.63 (four), FP64 0.48 and 0.53 (two).
// Per step of a whole run, setup and books included, single launches -> resident: 64 x 64 FP64
// 8.3 -> 4.2 us, 1159 x 72 viscous 10.6 -> 5.4, 512 x 512 FP32 10.6 -> 5.5, 1024 x 1024 FP32
// 16.1 -> 12.6 and FP64 27.8 -> 25.4; 45 flumes in FP64, a group of workgroups each,
// 24.9 -> 11.7.  Of that, edge codes kept in registers and the early first read of the wave
// speeds gave 15 % on 64 x 64 and 7 % on 512 x 512 cells.
#pragma once

#include "hexsv_ensemble.h"
#include "hexsv_internal.h"
#include "hexsv_tile.h"

namespace hexsv {

// Halo words of one value: FP32 one, FP64 two.
template <typename T>
constexpr int RES_WORDS = sizeof(T) / 4;

template <typename T>
__device__ inline uint32_t word_of(T v, int w) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(uint32_t, v);
    else return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> (32 * w));
}
template <typename T>
__device__ inline T value_of(const uint32_t *w) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, w[0]);
    else return __builtin_bit_cast(T, (uint64_t)w[1] << 32 | w[0]);
}
__device__ inline void send(unsigned long long *p, uint32_t tag, uint32_t bits) {
    __hip_atomic_store(p, (unsigned long long)tag << 32 | bits, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned long long recv(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A value all lanes hold, in scalar registers.
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline float uniform(float v) {
    return __builtin_bit_cast(float, uniform(__builtin_bit_cast(int, v)));
}
__device__ inline double uniform(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)uniform((int)(uint32_t)b), hi = (uint32_t)uniform((int)(b >> 32));
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Rim cell (lq, lr) of a TQ x TR tile in its halo block: bottom and top rows, then
// the left and right columns; -1 inside.
template <int TQ, int TR>
constexpr int RIM = 2 * (TQ + TR);
template <int TQ, int TR>
__device__ inline int rim_entry(int lq, int lr) {
    if (lr == 0) return lq;
    if (lr == TR - 1) return TQ + lq;
    if (lq == 0) return 2 * TQ + lr;
    if (lq == TQ - 1) return 2 * TQ + TR + lr;
    return -1;
}

// The new state stays in the tile's registers; rim cells go out at once.
template <typename T, int TQ, int TR, int NT, int SUB>
struct KeepSink {
    TileRegs<T, TQ, TR, NT, SUB> &R;
    unsigned long long *rim;  // this tile's halo block of the step's parity
    uint32_t tag;
    int tid;
    bool bad = false;
    __device__ inline void put_state(int k, uint32_t, T h, T v1, T v2) {
        constexpr int W = RES_WORDS<T>;
        R.h[k] = h;
        R.v1[k] = v1;
        R.v2[k] = v2;
        int lq, lr;
        TileRegs<T, TQ, TR, NT, SUB>::cell(tid, k, lq, lr);
        const int e = rim_entry<TQ, TR>(lq, lr);
        if (e < 0) return;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            send(rim + (0 * W + w) * RIM<TQ, TR> + e, tag, word_of(h, w));
            send(rim + (1 * W + w) * RIM<TQ, TR> + e, tag, word_of(v1, w));
            send(rim + (2 * W + w) * RIM<TQ, TR> + e, tag, word_of(v2, w));
        }
    }
    // which cell it was, the repetition with single launches finds out
    __device__ inline void nonfinite(uint32_t) { bad = true; }
    __device__ inline void rescan(uint32_t) { bad = true; }
};

// Polls before a wait is given up (a poll takes about a microsecond): the roll call, which
// other kernels on the device can delay, and a step's exchange, which nothing can once
// everybody has answered.
constexpr int RES_ROLL_POLLS = 1 << 12;
constexpr int RES_STEP_POLLS = 1 << 20;

// Sets of 256 threads that one thread stands for: FP64's four stacked tiles would leave a
// thread of 1024 too few registers for its cells (128; 200 spilled), so 512 take two each.
template <typename T, int SUB>
constexpr int RES_PER = (sizeof(T) == 8 && SUB == 4) ? 2 : 1;
template <typename T, int SUB>
constexpr int RES_NT = 256 * SUB / RES_PER<T, SUB>;

// Up to max_steps steps from control slot 0 (no step pending).  One workgroup per tile of
// TQ x TRS * SUB cells: SUB tiles of variant VAR (256 threads each) on top of each other.
// ntq, nwg: the raster's tiles per row and in all; ntiles: its tiles of variant VAR (records
// per ring slot).  Tags of this launch are tag0 (roll call) to tag0 + max_steps.
//
// The edge sums of a step do not depend on its dt, so they are formed as soon as the
// neighbours' rim cells are there, while the wave speeds that dt needs are on their way.
//
// Inlined by force: where both kernels below have the instance, the viscous FP32 64 x 16 tile
// became a function of its own, with its arguments and arrays in scratch memory.
template <typename T, int VAR, int SUB, bool VISC, bool EXT>
__device__ __attribute__((always_inline)) inline void resident_steps(
    const KDom<T> &dd, const KGrid &g, const KConst &kc, const KRain &rn, const Ctl *in, Ctl *out,
    Part *ring, const ResSync &rs, const ResGroup &grp, int max_steps, uint32_t tag0) {
    // FP64 time and books: rounded as written in every translation unit (the cells' own
    // arithmetic is in TileCells, under the unit's setting)
#pragma clang fp contract(off)
    constexpr int PER = RES_PER<T, SUB>;
    constexpr int TQ = TILES[VAR].tq, TRS = TILES[VAR].tr, TR = TRS * SUB, NT = 256 * SUB / PER;
    constexpr int W = RES_WORDS<T>, NW = NT / 64, SW = TQ + 2, E = RIM<TQ, TR>;
    using Regs = TileRegs<T, TQ, TR, NT, SUB>;
    constexpr int CPT = Regs::CPT, CPS = CPT / PER, NSETS = NT / 256;
    static_assert(TQ == 64 && TILES[VAR].nt == 256, "a wave holds one row of the tile");
    __shared__ TileLDS<T, TQ, TR, VISC> L;
    __shared__ T wmax[NW], fmax[NW];
    __shared__ double red[3][4 * SUB], book[3];
    __shared__ int sbad, nghost;
    // Workgroups of up to 8 KB a field have the registers to keep their cells' edge codes
    // (edges_fixed); those of larger ones would spill.
    constexpr bool FIXED = TQ * TR * sizeof(T) <= 8192;
    __shared__ T ghosts[FIXED ? 3 * TQ * TR : 1];  // beds of outflow ghosts
    const int nwg = grp.count, ntq = grp.ntq;      // of the group
    const int wg = grp.wg, me_wg = grp.first + wg;  // in the group, in the launch
    const int tr = wg / ntq, tq = wg - tr * ntq;
    const int q0 = tq * TQ, r0 = tr * TR;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, set = tid >> 8;
    Regs R;
    tile_load<T, TQ, TR, NT, SUB>(R, dd, g, 0, tq, tr);
    const uint32_t given_up = tag0;
    // this workgroup answers the roll call
    const size_t fstride = (size_t)W * rs.flag_cap;
    if (tid < W) send(rs.flags + (tag0 & 1) * fstride + tid * rs.flag_cap + me_wg, tag0, 0u);
    if (tid == 0) sbad = nghost = 0;
    __syncthreads();
    tile_stage<T, TQ, TR, NT, EXT>(L, R, g, kc, tq, tr);
    // sub-tiles that see an inactive cell take the general path, as a tile of their own would
    {
        int bits = 0;
        auto see = [&](int sr, bool inactive) {
            if (inactive)
                for (int s = 0; s < SUB; ++s)
                    if (sr >= s * TRS && sr <= s * TRS + TRS + 1) bits |= 1 << s;
        };
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            int lq, lr;
            Regs::cell(tid, k, lq, lr);
            see(lr + 1, R.pos[k] != POS_OUTSIDE && !(R.th[k] > T(0)));
        }
#pragma unroll
        for (int k = 0; k < Regs::RPT; ++k) {
            const int t = tid + k * NT;
            int lq = 0, lr = 0;
            if (t < Regs::NRING) ring_slot<TQ, TR>(t, lq, lr);
            see(lr, t < Regs::NRING && R.rpos[k] != POS_OUTSIDE && !(R.rth[k] > T(0)));
        }
        if (bits) atomicOr(&sbad, bits);
    }
    // cells this thread updates
    int act = 0;
#pragma unroll
    for (int k = 0; k < CPT; ++k)
        if (R.pos[k] == POS_OWN && R.th[k] > T(0)) act |= 1 << k;
    // where this thread's ring cells come from: their owner's halo block (cells that are
    // never updated keep the staged record)
    const unsigned long long *src[Regs::RPT];
#pragma unroll
    for (int k = 0; k < Regs::RPT; ++k) {
        const int t = tid + k * NT;
        src[k] = nullptr;
        if (t < Regs::NRING && R.rpos[k] != POS_OUTSIDE && R.rth[k] > T(0)) {
            int lq, lr;
            ring_slot<TQ, TR>(t, lq, lr);
            const int q = q0 + lq - 1, r = r0 + lr - 1;
            const int otq = q / TQ, otr = r / TR;
            src[k] = rs.halo + (size_t)(grp.first + otr * ntq + otq) * (3 * W * E) +
                     rim_entry<TQ, TR>(q - otq * TQ, r - otr * TR);
        }
    }
    const size_t hstride = (size_t)rs.flag_cap * (3 * W * E);
    const T G = (T)kc.g;
    const T mscale = sizeof(T) == 4 ? (T)kc.a : T(1);

    // another poll?  (not if somebody gave the launch up, or after too many)
    int polls = 0;
    bool ok = true;
    auto again = [&](int limit) {
        ++polls;
        if (polls >= limit ||
            ((polls & 255) == 0 && __hip_atomic_load(grp.abort_word, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT) == given_up))
            ok = false;
        return ok;
    };
    // the ring cells of `tag`, staged as they come
    auto wait_ring = [&](uint32_t tag) {
        polls = 0;
#pragma unroll
        for (int k = 0; k < Regs::RPT; ++k) {
            if (!src[k]) continue;
            const unsigned long long *p = src[k] + (tag & 1) * hstride;
            uint32_t b[3 * W];
            bool got = false;
            do {
                unsigned long long v[3 * W];
#pragma unroll
                for (int w = 0; w < 3 * W; ++w) v[w] = recv(p + w * E);
                got = true;
#pragma unroll
                for (int w = 0; w < 3 * W; ++w) {
                    got = got && (uint32_t)(v[w] >> 32) == tag;
                    b[w] = (uint32_t)v[w];
                }
            } while (!got && ok && again(RES_STEP_POLLS));
            const T h = value_of<T>(b), v1 = value_of<T>(b + W), v2 = value_of<T>(b + 2 * W);
            int lq, lr;
            ring_slot<TQ, TR>(tid + k * NT, lq, lr);
            const int s = lr * SW + lq;
            L.rec[s] = cell_rec<T, EXT>(h, R.rth[k], R.rz[k], v1, v2, G, mscale);
            if constexpr (VISC) L.c[s] = cell_wave(h, v1, v2, G);
        }
    };
    // the largest of all workgroups' wave speeds of `tag` (infinite: give up); a barrier.  The
    // first read of a word is issued early by ask_speeds, ahead of the edges: a read takes most
    // of a microsecond whether or not it finds the word.
    const int flag0 = NT - 1 - tid;  // from the other end than ring cells
    unsigned long long asked[W];
    auto ask_speeds = [&](uint32_t tag) {
        if (flag0 < nwg) {
            const unsigned long long *p = rs.flags + (tag & 1) * fstride + grp.first + flag0;
#pragma unroll
            for (int w = 0; w < W; ++w) asked[w] = recv(p + w * rs.flag_cap);
        }
    };
    auto wait_speeds = [&](uint32_t tag, int limit) -> T {
        T c = T(0);
        polls = 0;
        for (int f = flag0; f < nwg; f += NT) {
            const unsigned long long *p = rs.flags + (tag & 1) * fstride + grp.first + f;
            uint32_t b[W];
            bool got = f == flag0;  // asked for
            if (got) {
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    got = got && (uint32_t)(asked[w] >> 32) == tag;
                    b[w] = (uint32_t)asked[w];
                }
            }
            while (!got && ok && again(limit)) {
                got = true;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const unsigned long long v = recv(p + w * rs.flag_cap);
                    got = got && (uint32_t)(v >> 32) == tag;
                    b[w] = (uint32_t)v;
                }
            }
            const T u = value_of<T>(b);
            c = u > c ? u : c;
        }
        if (!ok) {
            c = (T)__builtin_inf();
            __hip_atomic_store(grp.abort_word, given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        c = wave_max_last(c);
        if (lane == 63) fmax[wave] = c;
        __syncthreads();
        c = fmax[0];
#pragma unroll
        for (int i = 1; i < NW; ++i) c = fmax[i] > c ? fmax[i] : c;
        return c;
    };
    TileCells<T, TQ, TR, NT, VISC, EXT, SUB, true> cells(L, R, dd, g, kc, tq, tr);
    cells.G = uniform(cells.G);
    cells.l = uniform(cells.l);
    cells.half_l = uniform(cells.half_l);
    // General sub-tiles: the rows (a wave's k-th cells) whose cells are all updated and have
    // six neighbours in the domain take the short path all the same.
    bool general[PER];
    int rows = 0;
    uint32_t ec[FIXED ? CPT : 1];
    EdgeSums<T> es[CPT];
    auto edges = [&](int me) {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            if (general[p]) {
#pragma unroll
                for (int k = p * CPS; k < (p + 1) * CPS; ++k) {
                    if constexpr (FIXED) {
                        if ((rows >> k) & 1) {
                            uint32_t codes = ec[k];  // opaque: its tests are not worth carrying
                            asm volatile("" : "+v"(codes));
                            es[k] = cells.edges_fixed(me, k, codes, ghosts);
                        } else {
                            es[k] = cells.template edges<false, sizeof(T) == 4>(me, k);
                        }
                    } else {
                        if ((act >> k) & 1) es[k] = cells.template edges<true>(me, k);
                    }
                }
            } else {
#pragma unroll
                for (int k = p * CPS; k < (p + 1) * CPS; ++k)
                    es[k] = cells.template edges<false>(me, k);
            }
        }
    };

    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int sub = set + p * NSETS;
        general[p] =
            uniform((int)(!tile_inner(g, q0, r0 + sub * TRS, TQ, TRS) || ((sbad >> sub) & 1))) != 0;
    }
    if constexpr (FIXED) {
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            ec[k] = 0;
            bool special = false;
            if (general[k / CPS]) {
                const bool mine = (act >> k) & 1;
                if (mine) ec[k] = cells.edge_codes(tid, k, ghosts, &nghost);
                special = !mine || ec[k] != 0;
            }
            if (__any(special)) rows |= 1 << k;
        }
        rows = uniform(rows);
        __syncthreads();  // the ghosts' beds are there
    }
    edges(tid);
    ask_speeds(tag0);
    if (!__builtin_isfinite(wait_speeds(tag0, RES_ROLL_POLLS))) return;

    // time and CFL bound, the same in every workgroup; the rain book and the time steps'
    // range are kept by the first one
    double t = uniform(in->t), tau = uniform(in->tau), lc = in->last_cmax;
    if (wg == 0 && tid == 0) {
        book[0] = in->rain;
        book[1] = in->dt_min;
        book[2] = in->dt_max_seen;
    }
    const double t_end = in->t_end, dt_max = in->dt_max;
    const int64_t left = in->err ? 0 : in->step_limit - in->steps;
    const int nmax = left < max_steps ? (int)left : max_steps;
    int n = 0;
    for (; n < nmax; ++n) {
        double dt = dt_max;
        if (tau < dt) dt = tau;
        if (t_end - t < dt) dt = t_end - t;
        if (!(dt > 0.0)) break;
        const double t_next = (dt == t_end - t) ? t_end : t + dt;
        const double r_next = uniform(rain_rate(rn, t_next));
        const uint32_t tag = tag0 + 1 + n;
        // an opaque thread index keeps the cells' addresses from being carried, one set per
        // cell, across the loop (they are cheaper to form again than to hold)
        int me = tid;
        asm volatile("" : "+v"(me));
        StepConst<T> sc = step_const<T>(kc, dt, r_next);
        sc.dt = uniform(sc.dt);
        sc.dts = uniform(sc.dts);
        sc.r = uniform(sc.r);
        sc.alpha_s = uniform(sc.alpha_s);
        sc.ftau = uniform(sc.ftau);
        sc.h_dry = uniform(sc.h_dry);
        Acc acc[PER];
        KeepSink<T, TQ, TR, NT, SUB> sink{
            R, rs.halo + (tag & 1) * hstride + (size_t)me_wg * (3 * W * E), tag, me};
        T c = T(0);
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            acc[p] = Acc{0.0, 0.0, 0.0, 0.0};
            Partial32 p32;
            if (general[p]) {
#pragma unroll
                for (int k = p * CPS; k < (p + 1) * CPS; ++k)
                    if ((act >> k) & 1)
                        cells.template finish<true>(me, k, es[k], sc, dt, acc[p], p32, sink);
            } else {
#pragma unroll
                for (int k = p * CPS; k < (p + 1) * CPS; ++k)
                    cells.template finish<false>(me, k, es[k], sc, dt, acc[p], p32, sink);
            }
            cells.fold32(me, p * CPS, (p + 1) * CPS, acc[p], p32, sink);
            c = (T)acc[p].c > c ? (T)acc[p].c : c;
        }
        if (sink.bad) c = (T)__builtin_inf();
        c = wave_max_last(c);
        if (lane == 63) wmax[wave] = c;
        __syncthreads();  // the records of the old state have been read
        if (wave == 0) {
            c = lane < NW ? wmax[lane] : T(0);
            c = wave_max_last(c);
            if (lane == 63) {
#pragma unroll
                for (int w = 0; w < W; ++w)
                    send(rs.flags + (tag & 1) * fstride + w * rs.flag_cap + me_wg, tag, word_of(c, w));
            }
        }
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            int lq, lr;
            Regs::cell(me, k, lq, lr);
            const int s = (lr + 1) * SW + (lq + 1);
            if ((act >> k) & 1) {
                L.rec[s] = cell_rec<T, EXT>(R.h[k], R.th[k], R.z[k], R.v1[k], R.v2[k], G, mscale);
                if constexpr (VISC) L.c[s] = cell_wave(R.h[k], R.v1[k], R.v2[k], G);
            }
        }
        // the books' sums, in block_reduce's order, while the words travel
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const double ss = wave_sum(acc[p].s), so = wave_sum(acc[p].o), sl = wave_sum(acc[p].cl);
            if (lane == 0) {
                red[0][wave + p * NW] = ss;
                red[1][wave + p * NW] = so;
                red[2][wave + p * NW] = sl;
            }
        }
        wait_ring(tag);
        __syncthreads();  // the new state's records are staged
        ask_speeds(tag);
        edges(me);
        const T cm = wait_speeds(tag, RES_STEP_POLLS);
        if (!__builtin_isfinite(cm)) return;
        if (tid < SUB) {
            const int ptr = tr * SUB + tid;  // row of this sub-tile among the tiles of VAR
            if (ptr * TRS < g.nr) {
                Part p{0.0, red[0][4 * tid], red[1][4 * tid], red[2][4 * tid]};
#pragma unroll
                for (int i = 1; i < 4; ++i) {
                    p.stored += red[0][4 * tid + i];
                    p.outflow += red[1][4 * tid + i];
                    p.clamp += red[2][4 * tid + i];
                }
                ring[(size_t)n * grp.ring_stride + ptr * ntq + tq] = p;
            }
        }
        // close the step (as open_step and write_slot do)
        const double cmax = (double)cm > kc.c_floor ? (double)cm : kc.c_floor;
        if (wg == 0 && tid == 0) {
            book[0] += kc.area_active * dt * r_next;
            if (dt < book[1]) book[1] = dt;
            if (dt > book[2]) book[2] = dt;
        }
        lc = uniform(cmax);
        t = uniform(t_next);
        tau = uniform(cmax > 0.0 ? kc.cfl_phi / cmax : __builtin_inf());
    }
    if (n > 0) {
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            if (!((act >> k) & 1)) continue;
            int lq, lr;
            Regs::cell(tid, k, lq, lr);
            const uint32_t i = (uint32_t)((r0 + lr) * g.pitch + q0 + lq);
            *at(dd.st[1][0], i) = R.h[k];
            *at(dd.st[1][1], i) = R.v1[k];
            *at(dd.st[1][2], i) = R.v2[k];
        }
    }
    if (tid == 0) {
        rs.done[me_wg] = tag0;
        if (wg == 0) {  // the proposed control block, for the fold
            out->t = t;
            out->tau = tau;
            out->t_end = t_end;
            out->dt_max = dt_max;
            out->steps = in->steps + n;
            out->step_limit = in->step_limit;
            out->parity = n > 0 ? in->parity ^ 1 : in->parity;
            out->open = n;
            out->initial = in->initial;
            out->stored = in->stored;
            out->rain = book[0];
            out->outflow = in->outflow;
            out->clamp = in->clamp;
            out->dt_min = book[1];
            out->dt_max_seen = book[2];
            out->last_cmax = lc;
            out->p_live = 0;
            out->p_dt = 0.0;
            out->p_tnext = 0.0;
        }
    }
}

// The resident steps of a single domain: slot 0 of the control block in, slot 1 out.
template <typename T, int VAR, int SUB, bool VISC, bool EXT>
__global__ __launch_bounds__((RES_NT<T, SUB>)) void k_resident(
    KDom<T> d, KGrid g, KConst kc, KRain rn, Ctl *ctl, KClose cl, ResSync rs, int ntq, int nwg,
    int ntiles, int max_steps, uint32_t tag0) {
    const int par = ctl->parity;
    KDom<T> dd = d;
    if (par)
        for (int f = 0; f < 3; ++f) {
            dd.st[0][f] = d.st[1][f];
            dd.st[1][f] = d.st[0][f];
        }
    const ResGroup grp{0, nwg, xcd_tile(blockIdx.x, gridDim.x, nwg, 0), ntq, ntiles, rs.abort_word};
    resident_steps<T, VAR, SUB, VISC, EXT>(dd, g, kc, rn, ctl, ctl + 1, cl.ring, rs, grp, max_steps,
                                           tag0);
}

// The resident steps of an ensemble: the workgroups of a scenario are a group of their own,
// which meets only its own members, so scenarios advance side by side at their own pace.
template <typename T, int VAR, int SUB, bool VISC, bool EXT>
__global__ __launch_bounds__((RES_NT<T, SUB>)) void k_ens_resident(
    KDom<T> base, const EnsScen *__restrict__ scen, const ResEnsWg *__restrict__ wgs,
    const Ctl *__restrict__ ctl, Ctl *out, Part *ring, ResSync rs, int btotal, int max_steps,
    uint32_t tag0) {
    const ResEnsWg w = wgs[blockIdx.x];
    const KGrid &g = scen[w.s].g;  // by reference (see k_ensemble)
    const ResGroup grp{w.first, w.count, (int)blockIdx.x - w.first, scen[w.s].bntq, btotal,
                       rs.abort_word + w.s};
    resident_steps<T, VAR, SUB, VISC, EXT>(dom_at(base, scen[w.s].off, ctl[w.s].parity), g,
                                           scen[w.s].kc, scen[w.s].rn, ctl + w.s, out + w.s,
                                           ring + scen[w.s].bbase, rs, grp, max_steps, tag0);
}

template <typename T, int VAR, int SUB>
static hipError_t launch_resident_vs(const KDom<T> &d, const KGrid &g, const KConst &kc,
                                     const KRain &rn, Ctl *ctl, const KClose &cl,
                                     const ResSync &rs, int ntq, int nwg, int ntiles,
                                     int max_steps, uint32_t tag0, int grid,
                                     hipStream_t stream) {
#define HEXSV_RES(VI, EX)                                                                      \
    hipLaunchKernelGGL((k_resident<T, VAR, SUB, VI, EX>), dim3(grid), dim3(RES_NT<T, SUB>), 0, \
                       stream, d, g, kc, rn, ctl, cl, rs, ntq, nwg, ntiles, max_steps, tag0)
    if (kc.visc) {
        if constexpr (resident_fits(sizeof(T), VAR, SUB, true)) HEXSV_RES(true, true);
        else return hipErrorInvalidValue;
    } else if (kc.ext) {
        HEXSV_RES(false, true);
    } else {
        HEXSV_RES(false, false);
    }
#undef HEXSV_RES
    return hipGetLastError();
}

template <typename T>
hipError_t launch_resident(int variant, int sub, const KDom<T> &d, const KGrid &g,
                           const KConst &kc, const KRain &rn, Ctl *ctl, const KClose &cl,
                           const ResSync &rs, int ntq, int nwg, int ntiles, int max_steps,
                           uint32_t tag0, int grid, hipStream_t stream) {
#define HEXSV_CASE(V, S)                                                                       \
    if (variant == V && sub == S)                                                              \
        return launch_resident_vs<T, V, S>(d, g, kc, rn, ctl, cl, rs, ntq, nwg, ntiles,        \
                                           max_steps, tag0, grid, stream);
    HEXSV_CASE(0, 1) HEXSV_CASE(0, 2) HEXSV_CASE(0, 4)
    HEXSV_CASE(1, 1) HEXSV_CASE(1, 2) HEXSV_CASE(1, 4)
    HEXSV_CASE(2, 1) HEXSV_CASE(2, 2) HEXSV_CASE(2, 4)
#undef HEXSV_CASE
    return hipErrorInvalidValue;
}

template <typename T, int VAR, int SUB>
static hipError_t launch_ens_resident_vs(bool visc, bool bc, const KDom<T> &base,
                                         const EnsScen *scen, const ResEnsWg *wgs, const Ctl *ctl,
                                         Ctl *out, Part *ring, const ResSync &rs, int nwg,
                                         int btotal, int max_steps, uint32_t tag0,
                                         hipStream_t stream) {
#define HEXSV_RES(VI, EX)                                                                      \
    hipLaunchKernelGGL((k_ens_resident<T, VAR, SUB, VI, EX>), dim3(nwg), dim3(RES_NT<T, SUB>), \
                       0, stream, base, scen, wgs, ctl, out, ring, rs, btotal, max_steps, tag0)
    if (visc) {
        if constexpr (resident_fits(sizeof(T), VAR, SUB, true)) HEXSV_RES(true, true);
        else return hipErrorInvalidValue;
    } else if (bc) HEXSV_RES(false, true);
    else HEXSV_RES(false, false);
#undef HEXSV_RES
    return hipGetLastError();
}

template <typename T>
hipError_t launch_ens_resident(int variant, int sub, bool visc, bool bc, const KDom<T> &base,
                               const EnsScen *scen, const ResEnsWg *wgs, const Ctl *ctl, Ctl *out,
                               Part *ring, const ResSync &rs, int nwg, int btotal, int max_steps,
                               uint32_t tag0, hipStream_t stream) {
#define HEXSV_CASE(V, S)                                                                       \
    if (variant == V && sub == S)                                                              \
        return launch_ens_resident_vs<T, V, S>(visc, bc, base, scen, wgs, ctl, out, ring, rs,  \
                                               nwg, btotal, max_steps, tag0, stream);
    HEXSV_CASE(0, 1) HEXSV_CASE(0, 2) HEXSV_CASE(0, 4) HEXSV_CASE(2, 1)
#undef HEXSV_CASE
    return hipErrorInvalidValue;
}

#define HEXSV_INSTANTIATE_RESIDENT(T)                                                          \
    template hipError_t launch_resident<T>(int, int, const KDom<T> &, const KGrid &,           \
                                           const KConst &, const KRain &, Ctl *,               \
                                           const KClose &, const ResSync &, int, int, int, int, \
                                           uint32_t, int, hipStream_t);                        \
    template hipError_t launch_ens_resident<T>(int, int, bool, bool, const KDom<T> &,          \
                                               const EnsScen *, const ResEnsWg *, const Ctl *, \
                                               Ctl *, Part *, const ResSync &, int, int, int,  \
                                               uint32_t, hipStream_t);

}  // namespace hexsv
