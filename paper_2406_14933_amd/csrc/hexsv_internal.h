// hexsv_internal.h — interface between the host library and the per-precision
// kernel translation units (FP64 built without contraction, FP32 with it).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hexsv_device.h"
#include "hexsv_nn.h"

namespace hexsv {

struct TileShape {
    int tq, tr, nt;
};

// Tile variants the step kernels are built for (the autotuner picks one).
constexpr TileShape TILES[] = {
    {64, 4, 256}, {64, 8, 256}, {64, 16, 256}, {128, 4, 256},
    {128, 8, 256}, {128, 8, 512}, {64, 32, 256}, {64, 8, 512},
};
constexpr int NUM_TILES = sizeof(TILES) / sizeof(TILES[0]);
#define HEXSV_TILE_SWITCH(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7)

// Tile variants of the persistent ensemble kernel (one 1024-thread workgroup
// sweeps a whole scenario).
constexpr TileShape ENS_TILES[] = {{64, 16, 1024}, {64, 32, 1024}, {128, 16, 1024}};
constexpr int NUM_ENS_TILES = sizeof(ENS_TILES) / sizeof(ENS_TILES[0]);

struct EnsScen;
struct EnsTile;
// Batched-step mode of the ensemble: the tile kernel over the tiles of all
// scenarios (one workgroup each) followed by the per-scenario finalize.
// Tile t loads the buffers of parity par_hint ^ tpar[t] first (tpar: the
// scenarios' parities relative to the launch hint).
template <typename T>
hipError_t launch_ens_step(int variant, bool visc, bool bc, const KDom<T> &base,
                           const EnsScen *scen, const EnsTile *tiles, const uint8_t *tpar,
                           Ctl *ctl, Part *part, int ntiles_total, int nscen, int par_hint,
                           hipStream_t stream);
hipError_t launch_ens_finalize(const EnsScen *scen, Ctl *ctl, const Part *part, int nscen,
                               hipStream_t stream);
// Reset the ensemble's scenario queue (a one-thread kernel, safe inside graphs).
hipError_t launch_queue_reset(uint32_t *queue, hipStream_t stream);
// One launch of the persistent ensemble kernel: nwg workgroups take the
// scenarios in `order` from the queue and advance each by up to ksteps steps.
template <typename T>
hipError_t launch_ensemble(int variant, const KDom<T> &base, const EnsScen *scen, Ctl *ctl,
                           const int32_t *order, int nscen, uint32_t *queue, int ksteps, int nwg,
                           hipStream_t stream);
constexpr int DEFAULT_TILE = 2;
// Step tile of a single domain when the tuning cache has no entry: in FP32, 128 x 8
// cells (256 threads) for rasters at least 2048 cells wide, whose long row
// segments it streams fastest; else the tallest of 64 x 16, 64 x 8 and 64 x 4
// (variants 2, 1, 0) that still makes 512 workgroups, two per CU (on smaller
// rasters a step is bound by latency, which more workgroups in flight hide),
// and 64 x 4 below that.
constexpr int WIDE_TILE = 4;
inline int default_step_tile(int nq, int nr, bool fp32) {
    if (fp32 && nq >= 2048) return WIDE_TILE;
    for (int v = DEFAULT_TILE; v > 0; --v) {
        const int64_t n = (int64_t)((nq + TILES[v].tq - 1) / TILES[v].tq) *
                          ((nr + TILES[v].tr - 1) / TILES[v].tr);
        if (n >= 512) return v;
    }
    return 0;
}

// Number of tiles covering an nq x nr raster with variant v.
inline void tile_grid(int v, int nq, int nr, int *ntq, int *ntiles) {
    const TileShape s = TILES[v];
    *ntq = (nq + s.tq - 1) / s.tq;
    *ntiles = *ntq * ((nr + s.tr - 1) / s.tr);
}

// One step launch (nwg == ntiles workgroups): closes the step of the
// previous launch and starts the next (see k_step, Ctl and KClose).  ctl
// points at the two control slots; `in` is the slot this launch reads and
// `set` its accumulator set (launch k after a fold: in = k % 2, set = k % 3).
// par_hint: the buffer parity the step is expected to read (its loads start
// before the control block is read; a wrong hint only costs a reload).
template <typename T>
hipError_t launch_step(int variant, const KDom<T> &d, const KGrid &g, const KConst &kc,
                       const KRain &rn, Ctl *ctl, const KClose &cl, int ntq, int ntiles, int nwg,
                       int par_hint, int in, int set, hipStream_t stream);

// Exchange memory of the resident steps (k_resident): halo words of every tile and
// wave-speed words of every workgroup (both twice, by the tag's parity), the word
// that gives a launch up, and each workgroup's mark that it reached the end.
struct ResSync {
    unsigned long long *halo, *flags;
    uint32_t *abort_word, *done;
    int flag_cap;  // workgroups the flags and marks are sized for
};
// The workgroups of a resident launch that advance one domain together: the first one's
// index in the launch, their number, this one's index among them, tiles per row, records per
// ring slot and the word that gives their part of the launch up.
struct ResGroup {
    int first, count, wg, ntq, ring_stride;
    uint32_t *abort_word;
};
// A workgroup of an ensemble's resident launch: its scenario and that scenario's group.
struct ResEnsWg {
    int s, first, count;
};
// After a resident launch that was given up although single launches got further (another
// stream's kernels held compute units), the wait at its roll call (about 4 ms) is not paid
// again at once: the next 1 runs go without, after a second one in a row the next 3, then 7,
// up to 63.  Back to none after a run that ended on chip.
struct ResBackoff {
    int fails = 0, left = 0;
    bool skip() { return left > 0 && left-- > 0; }
    void add() {
        fails = fails < 6 ? fails + 1 : 6;
        left = (1 << fails) - 1;
    }
    void clear() { fails = left = 0; }
};
constexpr int RES_MAX_SUB = 4;
// Does a resident workgroup fit a CU: its LDS (records, codes, with the viscous flux wave
// speeds, and the reduction scratch) the 160 KB, and its cells the registers?  The FP64 viscous
// edge sums of four cells per thread do not: 344 to 487 registers spill, with the sums in
// scratch memory, and the 64 x 32 tiles then lost some of them; single launches do those.
constexpr bool resident_fits(size_t esz, int variant, int sub, bool visc) {
    if (visc && esz == 8 && !(variant == 0 || (variant == 1 && sub <= 2))) return false;
    const size_t ns = (size_t)(TILES[variant].tq + 2) * (TILES[variant].tr * sub + 2);
    return ns * (4 * esz + 1 + (visc ? esz : 0)) + 2048 <= 160 * 1024;
}
// Fewest steps of a run for which a resident launch of a single domain is the faster way (0:
// none is): the tiling, its workgroups, and whether the raster has a mask or boundary cells.
// Times of the same run on chip / in single launches, short and long (4 and 300 steps):
//   one tile of 4 rows a workgroup: below 1 from the first step on (64 x 64: 0.8, 0.5)
//   up to 16 rows: 300 x 300 FP32 0.89, 0.50; 512 x 512 FP64 0.97, 0.75, viscous 1.03, 0.81
//   32 rows FP32: 600 x 600 0.90, 0.65, viscous 1.01, 0.76
//   64 rows FP32: 1024 x 1024 0.99, 0.77, masked 1.05, 0.86, viscous 1.11, 0.94; viscous with
//     idle compute units 2000 x 260 1.20, 1.08
//   FP64 stacks of four 8- or 16-row tiles, two of which a thread stands for, keep up only
//     where they fill the chip: 1000 x 1000 1.12, 0.87 (16 steps 0.94), 1024 x 800 1.18, 1.00,
//     800 x 800 1.33, 1.17; with a mask, where the tiles inside it are too few to fill it,
//     1000 x 1000 1.24, 1.02 and 600 x 600 1.13, 1.06
inline int resident_min_steps(size_t esz, int variant, int sub, int nwg, int ncu, bool masked,
                              bool visc) {
    const int rows = TILES[variant].tr * sub;
    if (esz == 8 && sub == 4 && variant > 0) return masked || 8 * nwg < 7 * ncu ? 0 : 16;
    if (visc && rows == 64 && 4 * nwg < 3 * ncu) return 0;
    if (rows <= 4) return 1;
    const int n = rows >= 64 ? (masked ? 16 : 8) : rows >= 32 || esz == 8 ? 4 : 2;
    return visc ? (4 * n < 16 ? 4 * n : 16) : n;
}
// 64-bit halo words of one tile (both parities).
inline size_t resident_halo_words(size_t esz, int variant, int sub) {
    return (size_t)2 * 3 * (esz / 4) * 2 * (TILES[variant].tq + TILES[variant].tr * sub);
}
// Up to max_steps steps in one launch of nwg workgroups, each a stack of `sub` tiles of
// `variant` (0, 1 or 2); the launch_fold_resident that follows commits them.  grid: nwg, or one
// fewer, which leaves the others to wait for the missing one in vain (a test's launch).
template <typename T>
hipError_t launch_resident(int variant, int sub, const KDom<T> &d, const KGrid &g,
                           const KConst &kc, const KRain &rn, Ctl *ctl, const KClose &cl,
                           const ResSync &rs, int ntq, int nwg, int ntiles, int max_steps,
                           uint32_t tag0, int grid, hipStream_t stream);
// The same for the scenarios of an ensemble, side by side: nwg workgroups (`wgs`, grouped by
// scenario), control blocks in `ctl` and proposed ones in `out`, btotal records per ring slot;
// variant 0 with any sub, or variant 2 with one.  launch_ens_fold commits the scenarios all of
// whose workgroups reached the end.
template <typename T>
hipError_t launch_ens_resident(int variant, int sub, bool visc, bool bc, const KDom<T> &base,
                               const EnsScen *scen, const ResEnsWg *wgs, const Ctl *ctl, Ctl *out,
                               Part *ring, const ResSync &rs, int nwg, int btotal, int max_steps,
                               uint32_t tag0, hipStream_t stream);
hipError_t launch_ens_fold(const EnsScen *scen, Ctl *ctl, const Ctl *out, const Part *ring,
                           const ResSync &rs, const int2 *groups, int nscen, int btotal,
                           uint32_t tag0, uint32_t next, hipStream_t stream);
// Commit the resident launch of tag0 (control slot 1, up to `slots` steps in the ring)
// if all nwg workgroups reached its end; otherwise only set the abort word of the next launch
// (whose tag0 is `slots` + 1 on).  tag0 = 0: neither (a timed trial).
hipError_t launch_fold_resident(Ctl *ctl, const KClose &cl, int ntiles, const KConst &kc,
                                const KRain &rn, int slots, const ResSync &rs, int nwg,
                                uint32_t tag0, hipStream_t stream);

// After a run of `launches` step launches since the previous fold, the last of
// which read slot `in` with accumulator set `set`: close its pending step, add
// the books of every closed step in the ring to ctl[0] in step order, empty the
// ring and clear the accumulators (one workgroup per ring slot the run can have
// filled, at most `launches`: the first launch after a fold has nothing to close,
// then one wave).
hipError_t launch_fold(Ctl *ctl, const KClose &cl, int ntiles, const KConst &kc, const KRain &rn,
                       int in, int set, int launches, hipStream_t stream);
// Close a priming pass over nparts partial records: tau (and, with
// reset_books, the initial books) of the current state.
hipError_t launch_prime_finalize(Ctl *ctl, const Part *part, int nparts, const KConst &kc,
                                 int reset_books, hipStream_t stream);
constexpr int PRIME_BLOCKS = 1024;

template <typename T>
hipError_t launch_prime(const KDom<T> &d, int64_t n, const KConst &kc, Ctl *ctl, Part *part,
                        int nblocks, int reset_books, hipStream_t stream);
// The caller's FP64 state into both buffers (zero outside the domain), primed (with the books).
template <typename T>
hipError_t launch_set_state(const KDom<T> &d, const double *h, const double *v1, const double *v2,
                            const uint8_t *active, int64_t n, const KConst &kc, Ctl *ctl,
                            Part *part, int nblocks, hipStream_t stream);

// FP64 caller arrays -> internal precision (theta forced to 0 outside the mask).
// nq, pitch: the internal rows are `pitch` cells apart (0: the caller's layout).
template <typename T>
hipError_t launch_import(const double *src, T *dst, const uint8_t *active, int zero_inactive,
                         int64_t n, hipStream_t stream, int64_t nq = 0, int64_t pitch = 0);
// internal state -> FP64 caller arrays (each output nullable); nq, pitch as above.
template <typename T>
hipError_t launch_export(const KDom<T> &d, const Ctl *ctl, int64_t n, double *h, double *v1,
                         double *v2, double *q1, double *q2, hipStream_t stream,
                         int64_t nq = 0, int64_t pitch = 0);

// Validation of caller inputs: counts offending active cells and records the
// lowest offending index in chk[0] (count) / chk[1] (index) / chk[2] (reason).
hipError_t launch_check_fields(const double *z, const double *th, const double *ap,
                               const uint8_t *active, int64_t n, int32_t *chk,
                               hipStream_t stream);
hipError_t launch_check_state(const double *h, const double *v1, const double *v2,
                              const uint8_t *active, int64_t n, double g, int32_t *chk,
                              hipStream_t stream);

// ------------------------------------------------------ surrogate windows
//
// A window advances the state by a fixed span with one network call; it is
// kept only if the predicted state keeps the water balance.  Everything of a
// window runs on the device (so windows chain inside a graph); the host only
// reads this record after a chain.
struct alignas(64) SurWin {
    double t_stop, window, tol;     // set by the host for a run
    double depth, R, t0, S0, rho;   // of the current window
    int32_t k;                      // rain sub-steps of a window
    int32_t live;                   // the current window runs
    int32_t alive;                  // every window of this chain so far was accepted
    int32_t rejected;               // a window of this chain was refused
    int32_t accepted;               // windows accepted in this chain
    int32_t project;                // 1: rescale an accepted state onto the balance
    int32_t scale_live;             // the current state waits for its rescaling by `scale`:
                                    // the windows of a chain read it scaled, and one
                                    // k_win_scale after the chain stores it
    int32_t perr, perr_cell;        // non-finite value met by a probe step
    double scale;                   // factor of that rescaling
    double c0;                      // reference c_max: of the last state the solver made
                                    // (run start, end of a refused span); < 0: take it
                                    // from the next window's start state
    int32_t why;                    // reason of the last refusal: 1 residual, 2 wave speed, 4 non-finite
    int32_t pad2;
};

constexpr int FEATURES = nn::FEATURES;
constexpr int WIN_PARTS = 1024;  // partial records of the window reductions

// Feature scales: H (depth), Q (discharge), Z (elevation), S (slope), and the
// window changes of depth and discharge dH, dQ.
struct FeatScale {
    float H, Q, Z, S, dH, dQ;
};

hipError_t launch_win_reset(SurWin *sw, hipStream_t stream);
// Gate of a window: part holds n_part records of the predicted state, op0 the
// probe's n_op0 records of the start state's outflow rate.
hipError_t launch_win_gate(Ctl *ctl, SurWin *sw, const Part *part, int n_part, const Part *op0,
                           int n_op0, const KConst &kc, hipStream_t stream);
// Window kernels on the current state (buffer ctl->parity), each a no-op unless sw->live
// (which the probe, the first of them, decides).
// scr holds 3 x cells values of T (the probe step's h, v1, v2).  The probe also
// writes the network's features of the current state into fout (feat 1: packed
// bf16; 2: FP32; 0: none) and one record per probe tile of the current state's
// outflow rate into op0[].stored (win_probe_tiles of them).
template <typename T>
hipError_t launch_win_probe(const KDom<T> &d, const KGrid &g, const KConst &kc, const KRain &rn,
                            const Ctl *ctl, SurWin *sw, T *scr, double dt_max,
                            const float2 *slope, FeatScale fs, int feat, void *fout, Part *op0,
                            hipStream_t stream);
// Tile of a window's probe launch: 64 x 4 cells, one per thread, so that the
// features the probe writes are spread over four times the workgroups of the
// step's default tile (a 512 x 512 raster: 1024).
constexpr int PROBE_TILE = 0;
// Workgroups (tiles) of a window's probe launch on an nq x nr raster.
inline int win_probe_tiles(int nq, int nr) {
    int ntq, ntiles;
    tile_grid(PROBE_TILE, nq, nr, &ntq, &ntiles);
    return ntiles;
}
// Terrain slope of every cell (float2), static for a simulation.
template <typename T>
hipError_t launch_win_slope(const KDom<T> &d, const KGrid &g, double a, float2 *slope,
                            hipStream_t stream);
// Predicted state into the other buffer, with its reductions (WIN_PARTS partials
// {c_max, stored, outflow rate, non-finite count}).
template <typename T>
hipError_t launch_win_apply(const KDom<T> &d, const KGrid &g, double l, const KConst &kc,
                            const Ctl *ctl, const SurWin *sw, const T *scr, double dt_max,
                            const float *out, int out_stride, float dH, float dQ, double m_min,
                            Part *part, hipStream_t stream);
// The network's last layer (input x: 32 channels per cell, weights wm, bias) with
// the predicted state as its epilogue, as launch_win_apply computes it from the
// stored network output; one record per conv tile (nn::conv_tiles of them) in part.
template <typename T>
hipError_t launch_win_last(const __bf16 *x, const __bf16 *wm, const float *bias,
                           const nn::ConvMask &cm, const KDom<T> &d, const KGrid &g, double l,
                           const KConst &kc, const Ctl *ctl, const SurWin *sw, const T *scr,
                           double dt_max, float dH, float dQ, double m_min, Part *part,
                           hipStream_t stream);
// Rescaling of the current state onto the water balance (no-op unless sw->scale_live),
// once after a chain of windows; the next chain's reset clears the flag.
template <typename T>
hipError_t launch_win_scale(const KDom<T> &d, int64_t n, const Ctl *ctl, const SurWin *sw,
                            hipStream_t stream);
// Neighbour and edge-code tables and the axial index arrays (each output nullable).
hipError_t launch_tables(const KGrid &g, const uint8_t *active, int32_t *nbr, uint8_t *code,
                         int32_t *q, int32_t *r, hipStream_t stream);

}  // namespace hexsv
