// hexsv_capi.hip — the C-ABI declared in include/hexsv.h: handles, input
// validation, graph capture of the step loop, books and error reporting.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>
#include <string>
#include <vector>

#include "hexsv.h"
#include "hexsv_internal.h"
#include "hexsv_host.h"

using namespace hexsv;

// ------------------------------------------------------------------ errors

thread_local std::string g_msg;

int hexsv_fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_msg = buf;
    return code;
}

extern "C" const char *hexsv_last_error(void) { return g_msg.c_str(); }
extern "C" const char *hexsv_version(void) { return "hexsv 0.1 gfx950"; }

// ------------------------------------------------------------------ raster

static bool valid_side(int c) {
    return c == HEXSV_WALL || c == HEXSV_OUTFLOW || c == HEXSV_PERIODIC;
}

extern "C" int hexsv_grid_create(const hexsv_grid_desc *desc, hexsv_grid **out) {
    if (!desc || !out) return fail(HEXSV_EINVAL, "grid_create: null argument");
    *out = nullptr;
    if (desc->nq < 1 || desc->nr < 1)
        return fail(HEXSV_EINVAL, "grid_create: nq=%d nr=%d must be >= 1", desc->nq, desc->nr);
    const int64_t n = (int64_t)desc->nq * desc->nr;
    if (n > 0x7fffffffLL) return fail(HEXSV_EINVAL, "grid_create: %lld cells exceed 2^31-1", (long long)n);
    if (!(desc->edge > 0.0) || !isfinite(desc->edge))
        return fail(HEXSV_EINVAL, "grid_create: edge length must be finite and > 0");
    for (int s = 0; s < 4; ++s)
        if (!valid_side(desc->side_bc[s]))
            return fail(HEXSV_EINVAL, "grid_create: side %d has invalid code %d", s, desc->side_bc[s]);
    const bool perq = desc->side_bc[HEXSV_E] == HEXSV_PERIODIC;
    const bool perr = desc->side_bc[HEXSV_S] == HEXSV_PERIODIC;
    if (perq != (desc->side_bc[HEXSV_W] == HEXSV_PERIODIC) ||
        perr != (desc->side_bc[HEXSV_N] == HEXSV_PERIODIC))
        return fail(HEXSV_EINVAL, "grid_create: opposite sides must both be PERIODIC or neither");
    if (desc->nseg < 0 || desc->nseg > HEXSV_MAX_SEGMENTS)
        return fail(HEXSV_EINVAL, "grid_create: nseg=%d outside [0,%d]", desc->nseg, HEXSV_MAX_SEGMENTS);
    if (desc->mask_bc != HEXSV_WALL && desc->mask_bc != HEXSV_OUTFLOW)
        return fail(HEXSV_EINVAL, "grid_create: mask_bc must be WALL or OUTFLOW");
    KGrid kg;
    memset(&kg, 0, sizeof kg);
    kg.nq = desc->nq;
    kg.nr = desc->nr;
    kg.pitch = desc->nq;
    kg.perq = perq;
    kg.perr = perr;
    for (int s = 0; s < 4; ++s) kg.side[s] = desc->side_bc[s];
    kg.nseg = desc->nseg;
    kg.mask_bc = desc->mask_bc;
    for (int s = 0; s < desc->nseg; ++s) {
        const hexsv_segment &g = desc->seg[s];
        if (g.side < 0 || g.side > 3 || (g.code != HEXSV_WALL && g.code != HEXSV_OUTFLOW) || g.lo > g.hi)
            return fail(HEXSV_EINVAL, "grid_create: segment %d malformed", s);
        if (desc->side_bc[g.side] == HEXSV_PERIODIC)
            return fail(HEXSV_EINVAL, "grid_create: segment %d lies on a periodic side", s);
        kg.seg_side[s] = g.side;
        kg.seg_lo[s] = g.lo;
        kg.seg_hi[s] = g.hi;
        kg.seg_code[s] = g.code;
    }
    hexsv_grid *gr = new (std::nothrow) hexsv_grid();
    if (!gr) return fail(HEXSV_ENOMEM, "grid_create: out of host memory");
    gr->kg = kg;
    gr->edge = desc->edge;
    gr->n = n;
    gr->n_active = n;
    gr->n_dirichlet = 0;
    gr->d_active = nullptr;
    if (desc->active) {
        int64_t na = 0, nd = 0;
        for (int64_t i = 0; i < n; ++i) {
            const uint8_t v = desc->active[i];
            if (v > 3) {
                delete gr;
                return fail(HEXSV_EINVAL, "grid_create: active[%lld]=%d is not 0, 1, 2 or 3", (long long)i, v);
            }
            na += v == 1;
            nd += v >= 2;
        }
        gr->n_active = na;
        gr->n_dirichlet = nd;
        if (na < n) {
            gr->kg.has_mask = 1;
            std::vector<uint8_t> a01(desc->active, desc->active + n);
            hipError_t e = hipMalloc(&gr->d_active, n);
            if (e != hipSuccess) {
                delete gr;
                return fail(HEXSV_ENOMEM, "grid_create: hipMalloc(active): %s", hipGetErrorString(e));
            }
            e = hipMemcpy(gr->d_active, a01.data(), n, hipMemcpyHostToDevice);
            if (e != hipSuccess) {
                (void)hipFree(gr->d_active);
                delete gr;
                return fail(HEXSV_EHIP, "grid_create: hipMemcpy(active): %s", hipGetErrorString(e));
            }
        }
    }
    *out = gr;
    return HEXSV_OK;
}

extern "C" void hexsv_grid_destroy(hexsv_grid *grid) {
    if (!grid) return;
    if (grid->d_active) (void)hipFree(grid->d_active);
    delete grid;
}

extern "C" int hexsv_grid_counts(const hexsv_grid *grid, int64_t *cells, int64_t *active) {
    if (!grid) return fail(HEXSV_EINVAL, "grid_counts: null grid");
    if (cells) *cells = grid->n;
    if (active) *active = grid->n_active;
    return HEXSV_OK;
}

extern "C" int hexsv_grid_tables_device(const hexsv_grid *grid, int32_t *d_nbr, uint8_t *d_code,
                                        int32_t *d_q, int32_t *d_r, hipStream_t stream) {
    if (!grid) return fail(HEXSV_EINVAL, "grid_tables_device: null grid");
    if (!d_nbr && !d_code && !d_q && !d_r) return HEXSV_OK;
    HIP_TRY(launch_tables(grid->kg, grid->d_active, d_nbr, d_code, d_q, d_r, stream));
    return HEXSV_OK;
}

extern "C" int hexsv_grid_tables(const hexsv_grid *grid, int32_t *nbr, uint8_t *code, int32_t *q,
                                 int32_t *r) {
    if (!grid) return fail(HEXSV_EINVAL, "grid_tables: null grid");
    if (!nbr && !code && !q && !r) return HEXSV_OK;
    const int64_t n = grid->n;
    // device staging of the requested tables, computed by the same kernel
    const size_t b_nbr = nbr ? sizeof(int32_t) * 6 * n : 0, b_code = code ? 6 * (size_t)n : 0;
    const size_t b_q = q ? sizeof(int32_t) * n : 0, b_r = r ? sizeof(int32_t) * n : 0;
    char *buf = nullptr;
    hipError_t e = hipMalloc(&buf, b_nbr + b_code + b_q + b_r);
    if (e != hipSuccess) return fail(HEXSV_ENOMEM, "grid_tables: %s", hipGetErrorString(e));
    int32_t *dn = nbr ? (int32_t *)buf : nullptr;
    int32_t *dq = q ? (int32_t *)(buf + b_nbr) : nullptr;
    int32_t *dr = r ? (int32_t *)(buf + b_nbr + b_q) : nullptr;
    uint8_t *dc = code ? (uint8_t *)(buf + b_nbr + b_q + b_r) : nullptr;
    e = launch_tables(grid->kg, grid->d_active, dn, dc, dq, dr, nullptr);
    if (e == hipSuccess && nbr) e = hipMemcpy(nbr, dn, b_nbr, hipMemcpyDeviceToHost);
    if (e == hipSuccess && code) e = hipMemcpy(code, dc, b_code, hipMemcpyDeviceToHost);
    if (e == hipSuccess && q) e = hipMemcpy(q, dq, b_q, hipMemcpyDeviceToHost);
    if (e == hipSuccess && r) e = hipMemcpy(r, dr, b_r, hipMemcpyDeviceToHost);
    (void)hipFree(buf);
    if (e != hipSuccess) return fail(HEXSV_EHIP, "grid_tables: %s", hipGetErrorString(e));
    return HEXSV_OK;
}

// ------------------------------------------------------------- simulation

// Steps per replay of the short graph used for spans of a few steps (the
// fallback of a refused surrogate window): the long graph would replay its
// whole length of no-op steps past the span's end.
static const int SHORT_STEPS = 8;
// Short graphs of 1, 2, 4, 8 and 16 steps (each ends with its fold) for spans of
// a few steps; a span is replayed as the set of them that costs least (see
// short_plan).
constexpr int N_SHORT = 5;
static const int SHORT_LEN[N_SHORT] = {1, 2, 4, 8, 16};
// Surrogate runs: after n >= 2 windows refused in a row the plain solver also
// advances the next min(2^(n-1), w_backoff) spans before windows are tried
// again, so phases in which the network fails (a wetting front) cost solver
// steps only; w_backoff starts at this value (hexsv_sim_set_surrogate_backoff).
static const int WIN_BACKOFF_MAX = 8;
// Most closed steps whose books wait in the step ring before a fold.
static const int RING_MAX = 128;
static const size_t ACC_BYTES = sizeof(unsigned long long) * ACC_SETS * ACC_SET_WORDS;

struct hexsv_sim {
    const hexsv_grid *grid;
    hexsv_params p;
    int prec;
    size_t esz;
    void *buf;  // [h0 v10 v20 h1 v11 v21 z th ap], n elements each
    void *d_as;     // soil coefficient per cell (n elements), allocated on first use
    bool as_field;  // d_as holds the soil coefficient (else the scalar kc.alpha_s)
    KConst kc;
    KRain rn;
    Ctl *d_ctl;
    Ctl *h_ctl;  // pinned mirror
    Part *d_part;  // partial records of the priming pass (PRIME_BLOCKS)
    // step results (see KClose): ring of ring_len steps x ntiles tile records,
    // per-slot totals and the wave-speed maximum; the ring is sized for the
    // current tile variant when a graph is captured or a kernel timed
    Part *d_ring, *d_slots;
    unsigned long long *d_acc;
    size_t ring_cap;  // tile records the ring holds
    int ring_len;
    int32_t *d_chk;
    int32_t *h_chk;  // pinned
    int tile, ntq, ntiles, nwg;
    int gsteps;
    int ncu;  // compute units: the most workgroups of a resident launch
    bool res_on;          // hexsv_sim_set_resident
    int64_t res_launches;  // resident launches so far
    int64_t res_drop;      // launches before the one a test wants given up (< 0: none)
    ResBackoff res_wait;   // runs left to single launches after a give-up
    // resident steps (k_resident): exchange memory sized for the current tiling, and the
    // next launch's tag
    char *d_res;
    size_t res_bytes;
    ResSync res;
    uint32_t res_tag;
    hipStream_t cap;
    hipGraph_t graph[2];    // gsteps steps, starting from buffer parity 0 / 1
    hipGraphExec_t gexec[2];
    hipGraph_t sgraph[N_SHORT][2];  // short graphs (SHORT_LEN[j] steps), per start parity
    hipGraphExec_t sexec[N_SHORT][2];
    bool graph_ok, fields_set, state_set;
    // surrogate windows: control record (device + pinned mirror), outflow
    // partials of both ends, and a graph of WIN_CHAIN chained windows
    SurWin *d_sw, *h_sw;
    Part *d_op;   // window partial records: start-state outflow, predicted-state sums
    void *d_scr;  // probe state: 3 x cells of the state's precision
    float2 *d_slope;  // terrain slope per cell (static; rebuilt after set_fields)
    bool slope_ok;
    hipGraph_t wgraph[6];     // chains of WIN_CHAINS[j] windows
    hipGraphExec_t wexec[6];
    const hexsv_surrogate *w_sur;
    uint64_t w_gen;
    float w_scales[8];
    int64_t w_stats[4];  // windows kept; refused for the residual, the wave speed, non-finite
    int32_t w_backoff;   // most spans solved after a run of refusals (0: none)
    // optional device timing of graph replays (hipEvents on the run stream)
    bool timing;
    hipEvent_t ev0, ev1;
    double timed_ms;
    int64_t timed_steps, timed_replays;
};

template <typename T>
static KDom<T> dom_of(const hexsv_sim *s) {
    KDom<T> d;
    T *b = (T *)s->buf;
    const int64_t n = s->grid->n;
    for (int p = 0; p < 2; ++p)
        for (int f = 0; f < 3; ++f) d.st[p][f] = b + (int64_t)(3 * p + f) * n;
    d.z = b + 6 * n;
    d.th = b + 7 * n;
    d.ap = b + 8 * n;
    d.as = s->as_field ? (const T *)s->d_as : nullptr;
    return d;
}

static void drop_graph(hexsv_sim *s) {
    for (int p = 0; p < 2; ++p) {
        if (s->gexec[p]) (void)hipGraphExecDestroy(s->gexec[p]);
        if (s->graph[p]) (void)hipGraphDestroy(s->graph[p]);
        for (int j = 0; j < N_SHORT; ++j) {
            if (s->sexec[j][p]) (void)hipGraphExecDestroy(s->sexec[j][p]);
            if (s->sgraph[j][p]) (void)hipGraphDestroy(s->sgraph[j][p]);
            s->sexec[j][p] = nullptr;
            s->sgraph[j][p] = nullptr;
        }
        s->gexec[p] = nullptr;
        s->graph[p] = nullptr;
    }
    s->graph_ok = false;
}

static void drop_win_graph(hexsv_sim *s) {
    for (int j = 0; j < 6; ++j) {
        if (s->wexec[j]) (void)hipGraphExecDestroy(s->wexec[j]);
        if (s->wgraph[j]) (void)hipGraphDestroy(s->wgraph[j]);
        s->wexec[j] = nullptr;
        s->wgraph[j] = nullptr;
    }
    s->w_sur = nullptr;
}

extern "C" int hexsv_tile_count(void) { return NUM_TILES; }

extern "C" int hexsv_tile_shape(int32_t v, int32_t *tq, int32_t *tr, int32_t *threads) {
    if (v < 0 || v >= NUM_TILES) return fail(HEXSV_EINVAL, "tile_shape: variant %d out of range", v);
    if (tq) *tq = TILES[v].tq;
    if (tr) *tr = TILES[v].tr;
    if (threads) *threads = TILES[v].nt;
    return HEXSV_OK;
}

extern "C" int hexsv_sim_create(const hexsv_grid *grid, const hexsv_params *params, hexsv_sim **out) {
    if (!grid || !params || !out) return fail(HEXSV_EINVAL, "sim_create: null argument");
    *out = nullptr;
    const hexsv_params &p = *params;
    if (!(p.g > 0.0) || !isfinite(p.g)) return fail(HEXSV_EDOMAIN, "sim_create: g must be > 0");
    if (!(p.cfl > 0.0 && p.cfl < 1.0)) return fail(HEXSV_EDOMAIN, "sim_create: cfl=%g not in (0,1)", p.cfl);
    if (!(p.dt_max > 0.0)) return fail(HEXSV_EDOMAIN, "sim_create: dt_max must be > 0");
    if (!(p.h_dry >= 0.0)) return fail(HEXSV_EDOMAIN, "sim_create: h_dry must be >= 0");
    if (p.precision != HEXSV_FP64 && p.precision != HEXSV_FP32)
        return fail(HEXSV_EINVAL, "sim_create: precision %d unknown", p.precision);
    if (p.tile >= NUM_TILES) return fail(HEXSV_EINVAL, "sim_create: tile %d not built", p.tile);
    if (p.wg_per_cu != 0) return fail(HEXSV_EUNSUPPORTED, "sim_create: wg_per_cu must be 0");
    if ((uint64_t)grid->n * (p.precision == HEXSV_FP64 ? 8u : 4u) >= (1ull << 32))
        return fail(HEXSV_EUNSUPPORTED, "sim_create: %lld cells exceed 4 GiB per field",
                    (long long)grid->n);
    hexsv_sim *s = new (std::nothrow) hexsv_sim();
    if (!s) return fail(HEXSV_ENOMEM, "sim_create: out of host memory");
    s->grid = grid;
    s->p = p;
    s->prec = p.precision;
    s->esz = p.precision == HEXSV_FP64 ? sizeof(double) : sizeof(float);
    s->tile = p.tile >= 0 ? p.tile
                          : tuned_tile("step", p.precision, grid->n,
                                       default_step_tile(grid->kg.nq, grid->kg.nr,
                                                         p.precision == HEXSV_FP32));
    tile_grid(s->tile, grid->kg.nq, grid->kg.nr, &s->ntq, &s->ntiles);
    s->gsteps = p.steps_per_graph > 0 ? p.steps_per_graph : 100;
    s->w_backoff = WIN_BACKOFF_MAX;
    s->res_on = true;
    s->res_drop = -1;
    s->ring_len = s->gsteps < RING_MAX ? s->gsteps : RING_MAX;
    if (s->ring_len < SHORT_STEPS) s->ring_len = SHORT_STEPS;
    const double a = grid->edge;
    s->kc.g = p.g;
    s->kc.a = a;
    hexsv_geometry(a, p.cfl, &s->kc.sigma, &s->kc.cfl_phi);
    s->kc.h_dry = p.h_dry;
    s->kc.alpha_s = 0.0;
    s->kc.tau_lin = 0.0;
    s->kc.c_floor = 0.0;
    s->kc.ext = grid->n_dirichlet > 0 ? 1 : 0;
    s->kc.f_inf = 0.0;
    s->kc.h_inf = 0.0;
    s->kc.visc = 0;
    s->kc.area_active = s->kc.sigma * (double)grid->n_active;
    s->rn.kind = 0;
    s->rn.i_a = 0.0;
    s->rn.t_a = 0.0;
    s->rn.T_d = INFINITY;
    s->nwg = s->ntiles;
    int dev = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&s->ncu, hipDeviceAttributeMultiprocessorCount, dev);
    hipError_t e = hipMalloc(&s->buf, s->esz * 9 * (size_t)grid->n);
    if (e == hipSuccess) e = hipMalloc(&s->d_ctl, 2 * sizeof(Ctl));  // two control slots
    if (e == hipSuccess) e = hipMalloc(&s->d_part, sizeof(Part) * PRIME_BLOCKS);
    if (e == hipSuccess) e = hipMalloc(&s->d_chk, 8 * sizeof(int32_t));
    if (e == hipSuccess) e = hipMalloc(&s->d_acc, ACC_BYTES);
    if (e == hipSuccess) e = hipMalloc(&s->d_slots, sizeof(Part) * s->ring_len);
    if (e == hipSuccess) e = hipMemset(s->d_acc, 0, ACC_BYTES);
    if (e == hipSuccess) e = hipHostMalloc(&s->h_ctl, sizeof(Ctl), hipHostMallocDefault);
    if (e == hipSuccess) e = hipHostMalloc(&s->h_chk, 8 * sizeof(int32_t), hipHostMallocDefault);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&s->cap, hipStreamNonBlocking);
    if (e != hipSuccess) {
        hexsv_sim_destroy(s);
        return fail(HEXSV_ENOMEM, "sim_create: allocation failed: %s", hipGetErrorString(e));
    }
    memset(s->h_ctl, 0, sizeof(Ctl));
    *out = s;
    return HEXSV_OK;
}

extern "C" void hexsv_sim_destroy(hexsv_sim *s) {
    if (!s) return;
    drop_graph(s);
    if (s->cap) (void)hipStreamDestroy(s->cap);
    if (s->ev0) (void)hipEventDestroy(s->ev0);
    if (s->ev1) (void)hipEventDestroy(s->ev1);
    if (s->buf) (void)hipFree(s->buf);
    if (s->d_as) (void)hipFree(s->d_as);
    if (s->d_ctl) (void)hipFree(s->d_ctl);
    if (s->d_part) (void)hipFree(s->d_part);
    if (s->d_ring) (void)hipFree(s->d_ring);
    if (s->d_slots) (void)hipFree(s->d_slots);
    if (s->d_acc) (void)hipFree(s->d_acc);
    if (s->d_res) (void)hipFree(s->d_res);
    if (s->d_chk) (void)hipFree(s->d_chk);
    if (s->h_ctl) (void)hipHostFree(s->h_ctl);
    if (s->h_chk) (void)hipHostFree(s->h_chk);
    drop_win_graph(s);
    if (s->d_sw) (void)hipFree(s->d_sw);
    if (s->h_sw) (void)hipHostFree(s->h_sw);
    if (s->d_op) (void)hipFree(s->d_op);
    if (s->d_scr) (void)hipFree(s->d_scr);
    if (s->d_slope) (void)hipFree(s->d_slope);
    delete s;
}

extern "C" int hexsv_sim_info(const hexsv_sim *s, int32_t *workgroups, int32_t *tile, int32_t *tq,
                              int32_t *tr, int32_t *threads) {
    if (!s) return fail(HEXSV_EINVAL, "sim_info: null sim");
    if (workgroups) *workgroups = s->nwg;
    if (tile) *tile = s->tile;
    return hexsv_tile_shape(s->tile, tq, tr, threads);
}

// Run a device check; returns the count of offending cells (chk[0]) and, for a
// state check, the largest wave speed of the Dirichlet cells (c_dirichlet, nullable).
static int run_check(hexsv_sim *s, hipStream_t stream, bool fields, const double *a, const double *b,
                     const double *c, int32_t *count, int32_t *first, int32_t *reason,
                     double *c_dirichlet = nullptr) {
    const int32_t init[8] = {0, 0x7fffffff, 0, 0, 0, 0, 0, 0};
    memcpy(s->h_chk, init, sizeof init);
    HIP_TRY(hipMemcpyAsync(s->d_chk, s->h_chk, sizeof init, hipMemcpyHostToDevice, stream));
    if (fields) HIP_TRY(launch_check_fields(a, b, c, s->grid->d_active, s->grid->n, s->d_chk, stream));
    else HIP_TRY(launch_check_state(a, b, c, s->grid->d_active, s->grid->n, s->kc.g, s->d_chk, stream));
    HIP_TRY(hipMemcpyAsync(s->h_chk, s->d_chk, sizeof init, hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    *count = s->h_chk[0];
    *first = s->h_chk[1];
    *reason = s->h_chk[2];
    if (c_dirichlet) memcpy(c_dirichlet, s->h_chk + 4, sizeof(double));
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_fields(hexsv_sim *s, const double *d_z, const double *d_theta,
                                    const double *d_alpha_p, const double *d_alpha_s,
                                    double alpha_s, hipStream_t stream) {
    if (!s || !d_z || !d_theta || !d_alpha_p) return fail(HEXSV_EINVAL, "set_fields: null argument");
    if (!d_alpha_s && (!(alpha_s >= 0.0) || !isfinite(alpha_s)))
        return fail(HEXSV_EDOMAIN, "set_fields: alpha_s must be >= 0");
    int32_t cnt, first, why;
    int rc = run_check(s, stream, true, d_z, d_theta, d_alpha_p, &cnt, &first, &why);
    if (rc) return rc;
    if (cnt)
        return fail(HEXSV_EDOMAIN,
                    "set_fields: %d active cells invalid; first cell %d (%s%s%s)", cnt, first,
                    (why & 1) ? "theta not in (0,1] " : "", (why & 2) ? "alpha_p < 0 " : "",
                    (why & 4) ? "z not finite" : "");
    if (d_alpha_s) {  // the same check with the soil field in the plant field's place
        rc = run_check(s, stream, true, d_z, d_theta, d_alpha_s, &cnt, &first, &why);
        if (rc) return rc;
        if (cnt)
            return fail(HEXSV_EDOMAIN, "set_fields: %d active cells invalid; first cell %d (%s)",
                        cnt, first, (why & 2) ? "alpha_s < 0 or not finite" : "?");
    }
    const int64_t n = s->grid->n;
    const uint8_t *act = s->grid->d_active;
    if (d_alpha_s && !s->d_as) {
        hipError_t e = hipMalloc(&s->d_as, s->esz * (size_t)n);
        if (e != hipSuccess) {
            s->d_as = nullptr;
            return fail(HEXSV_ENOMEM, "set_fields: soil field: %s", hipGetErrorString(e));
        }
    }
    if (d_alpha_s) {
        if (s->prec == HEXSV_FP64)
            HIP_TRY(launch_import<double>(d_alpha_s, (double *)s->d_as, act, 1, n, stream));
        else
            HIP_TRY(launch_import<float>(d_alpha_s, (float *)s->d_as, act, 1, n, stream));
    }
    s->as_field = d_alpha_s != nullptr;
    s->kc.ext = (s->grid->n_dirichlet > 0 || s->kc.f_inf > 0.0 || s->as_field) ? 1 : 0;
    if (s->prec == HEXSV_FP64) {
        KDom<double> d = dom_of<double>(s);
        HIP_TRY(launch_import<double>(d_z, (double *)d.z, act, 0, n, stream));
        HIP_TRY(launch_import<double>(d_theta, (double *)d.th, act, 2, n, stream));
        HIP_TRY(launch_import<double>(d_alpha_p, (double *)d.ap, act, 0, n, stream));
    } else {
        KDom<float> d = dom_of<float>(s);
        HIP_TRY(launch_import<float>(d_z, (float *)d.z, act, 0, n, stream));
        HIP_TRY(launch_import<float>(d_theta, (float *)d.th, act, 2, n, stream));
        HIP_TRY(launch_import<float>(d_alpha_p, (float *)d.ap, act, 0, n, stream));
    }
    s->kc.alpha_s = alpha_s;
    s->fields_set = true;
    s->slope_ok = false;
    drop_graph(s);
    drop_win_graph(s);
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_viscosity(hexsv_sim *s, int32_t on) {
    if (!s) return fail(HEXSV_EINVAL, "set_viscosity: null sim");
    if (on != 0 && on != 1) return fail(HEXSV_EINVAL, "set_viscosity: on must be 0 or 1");
    s->kc.visc = on;
    drop_graph(s);
    drop_win_graph(s);
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_linear_friction(hexsv_sim *s, double tau) {
    if (!s) return fail(HEXSV_EINVAL, "set_linear_friction: null sim");
    if (!(tau >= 0.0) || !isfinite(tau))
        return fail(HEXSV_EDOMAIN, "set_linear_friction: tau=%g must be finite and >= 0", tau);
    s->kc.tau_lin = tau;
    drop_graph(s);
    drop_win_graph(s);
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_infiltration(hexsv_sim *s, double f_inf, double h_inf) {
    if (!s) return fail(HEXSV_EINVAL, "set_infiltration: null sim");
    if (!(f_inf >= 0.0) || !isfinite(f_inf) || !isfinite(h_inf) || (f_inf > 0.0 && !(h_inf > 0.0)))
        return fail(HEXSV_EDOMAIN, "set_infiltration: f_inf=%g must be >= 0 and h_inf=%g > 0", f_inf,
                    h_inf);
    s->kc.f_inf = f_inf;
    s->kc.h_inf = f_inf > 0.0 ? h_inf : 0.0;
    s->kc.ext = (s->grid->n_dirichlet > 0 || f_inf > 0.0 || s->as_field) ? 1 : 0;
    drop_graph(s);
    drop_win_graph(s);
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_rain(hexsv_sim *s, const hexsv_rain *rain) {
    if (!s || !rain) return fail(HEXSV_EINVAL, "set_rain: null argument");
    if (rain->kind != 0 && rain->kind != 1) return fail(HEXSV_EINVAL, "set_rain: kind %d unknown", rain->kind);
    if (!(rain->i_a >= 0.0) || !isfinite(rain->i_a)) return fail(HEXSV_EDOMAIN, "set_rain: i_a must be >= 0");
    if (rain->kind == 1 && !(rain->t_a > 0.0 && rain->T_d > rain->t_a && isfinite(rain->T_d)))
        return fail(HEXSV_EDOMAIN, "set_rain: triangular rain needs 0 < t_a < T_d < inf");
    if (rain->kind == 0 && !(rain->T_d >= 0.0)) return fail(HEXSV_EDOMAIN, "set_rain: T_d must be >= 0");
    s->rn.kind = rain->kind;
    s->rn.i_a = rain->i_a;
    s->rn.t_a = rain->t_a;
    s->rn.T_d = rain->T_d;
    drop_graph(s);
    drop_win_graph(s);
    return HEXSV_OK;
}

template <typename T>
static hipError_t prime(hexsv_sim *s, int reset, hipStream_t stream) {
    return launch_prime<T>(dom_of<T>(s), s->grid->n, s->kc, s->d_ctl, s->d_part, PRIME_BLOCKS, reset,
                           stream);
}

extern "C" int hexsv_sim_set_state(hexsv_sim *s, double t0, const double *d_h, const double *d_v1,
                                   const double *d_v2, hipStream_t stream) {
    if (!s || !d_h || !d_v1 || !d_v2) return fail(HEXSV_EINVAL, "set_state: null argument");
    if (!s->fields_set) return fail(HEXSV_ESTATE, "set_state: call set_fields first");
    if (!isfinite(t0)) return fail(HEXSV_EDOMAIN, "set_state: t0 must be finite");
    int32_t cnt, first, why;
    double c_dirichlet = 0.0;
    int rc = run_check(s, stream, false, d_h, d_v1, d_v2, &cnt, &first, &why, &c_dirichlet);
    if (rc) return rc;
    if (cnt)
        return fail(HEXSV_EDOMAIN, "set_state: %d active cells invalid; first cell %d (%s%s)", cnt,
                    first, (why & 1) ? "h < 0 or not finite " : "", (why & 2) ? "v not finite" : "");
    if (c_dirichlet != s->kc.c_floor) {  // captured launches hold the old value
        s->kc.c_floor = c_dirichlet;
        drop_graph(s);
        drop_win_graph(s);
    }
    const int64_t n = s->grid->n;
    const uint8_t *act = s->grid->d_active;
    Ctl &c = *s->h_ctl;
    memset(&c, 0, sizeof c);
    c.t = t0;
    c.t_end = t0;
    c.dt_max = s->p.dt_max;
    c.steps = 0;
    c.step_limit = 0;
    c.parity = 0;
    c.err_cell = -1;
    HIP_TRY(hipMemcpyAsync(s->d_ctl, s->h_ctl, sizeof(Ctl), hipMemcpyHostToDevice, stream));
    HIP_TRY(hipMemsetAsync(s->d_acc, 0, ACC_BYTES, stream));
    HIP_TRY(s->prec == HEXSV_FP64
                ? launch_set_state<double>(dom_of<double>(s), d_h, d_v1, d_v2, act, n, s->kc, s->d_ctl,
                                           s->d_part, PRIME_BLOCKS, stream)
                : launch_set_state<float>(dom_of<float>(s), d_h, d_v1, d_v2, act, n, s->kc, s->d_ctl,
                                          s->d_part, PRIME_BLOCKS, stream));
    HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    s->state_set = true;
    return HEXSV_OK;
}

// The step ring sized for the current tile variant.
static int ensure_ring(hexsv_sim *s) {
    const size_t need = (size_t)s->ntiles * s->ring_len;
    if (s->d_ring && s->ring_cap >= need) return HEXSV_OK;
    if (s->d_ring) HIP_TRY(hipFree(s->d_ring));
    s->d_ring = nullptr;
    s->ring_cap = 0;
    if (hipMalloc(&s->d_ring, sizeof(Part) * need) != hipSuccess) {
        s->d_ring = nullptr;
        return fail(HEXSV_ENOMEM, "step ring of %zu records: allocation failed", need);
    }
    s->ring_cap = need;
    return HEXSV_OK;
}

static KClose close_of(const hexsv_sim *s) { return KClose{s->d_ring, s->d_slots, s->d_acc, s->ring_len}; }

static hipError_t step_launch(hexsv_sim *s, const KClose &cl, int hint, int in, int set,
                              hipStream_t stream) {
    if (s->prec == HEXSV_FP64)
        return launch_step<double>(s->tile, dom_of<double>(s), s->grid->kg, s->kc, s->rn, s->d_ctl,
                                   cl, s->ntq, s->ntiles, s->nwg, hint, in, set, stream);
    return launch_step<float>(s->tile, dom_of<float>(s), s->grid->kg, s->kc, s->rn, s->d_ctl, cl,
                              s->ntq, s->ntiles, s->nwg, hint, in, set, stream);
}

// Capture nsteps step launches (with a fold after every ring_len of them and
// at the end) into one executable graph.  Step k of the graph reads buffer
// parity (par0 + k) % 2 (live steps are consecutive from the start of a
// replay); the j-th launch after a fold reads control slot j % 2 and
// accumulates into set j % 3.
static int capture_steps(hexsv_sim *s, int nsteps, int par0, hipGraph_t *graph,
                         hipGraphExec_t *exec) {
    int rc = ensure_ring(s);
    if (rc) return rc;
    const KClose cl = close_of(s);
    HIP_TRY(hipStreamBeginCapture(s->cap, hipStreamCaptureModeThreadLocal));
    hipError_t e = hipSuccess;
    int j = 0;  // launches since the last fold
    for (int k = 0; k < nsteps && e == hipSuccess; ++k, ++j) {
        e = step_launch(s, cl, (par0 + k) & 1, j & 1, j % ACC_SETS, s->cap);
        if (e == hipSuccess && (j + 1 == s->ring_len || k + 1 == nsteps)) {
            e = launch_fold(s->d_ctl, cl, s->ntiles, s->kc, s->rn, (j + 1) & 1, j % ACC_SETS, j + 1,
                            s->cap);
            j = -1;
        }
    }
    hipGraph_t g = nullptr;
    hipError_t e2 = hipStreamEndCapture(s->cap, &g);
    if (e != hipSuccess || e2 != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return fail(HEXSV_EHIP, "graph capture failed: %s",
                    hipGetErrorString(e != hipSuccess ? e : e2));
    }
    *graph = g;
    HIP_TRY(hipGraphInstantiate(exec, g, nullptr, nullptr, 0));
    return HEXSV_OK;
}

static int capture(hexsv_sim *s) {
    drop_graph(s);
    for (int p = 0; p < 2; ++p) {
        int rc = capture_steps(s, s->gsteps, p, &s->graph[p], &s->gexec[p]);
        if (rc) return rc;
        for (int j = 0; j < N_SHORT && !rc; ++j)
            rc = capture_steps(s, SHORT_LEN[j], p, &s->sgraph[j][p], &s->sexec[j][p]);
        if (rc) return rc;
    }
    s->graph_ok = true;
    return HEXSV_OK;
}

// Short graphs (indices into SHORT_LEN, longest first) that replay at least n
// steps at the least cost: 16-step graphs while 16 or more steps remain, then the
// cheapest set for the rest, a graph's fold counting as two steps that find the
// run over (each such step still issues its loads).  Returns the count (<= cap).
static int short_plan(int n, int *plan, int cap) {
    int m = 0;
    while (n >= SHORT_LEN[N_SHORT - 1] && m < cap) {
        plan[m++] = N_SHORT - 1;
        n -= SHORT_LEN[N_SHORT - 1];
    }
    if (n <= 0) return m;
    int best = 0, best_cost = 1 << 30;
    for (int set = 1; set < (1 << N_SHORT); ++set) {
        int sum = 0, cnt = 0;
        for (int j = 0; j < N_SHORT; ++j)
            if (set >> j & 1) {
                sum += SHORT_LEN[j];
                ++cnt;
            }
        const int cost = 2 * cnt + (sum - n);
        if (sum >= n && cost < best_cost) {
            best_cost = cost;
            best = set;
        }
    }
    for (int j = N_SHORT - 1; j >= 0; --j)
        if ((best >> j & 1) && m < cap) plan[m++] = j;
    return m;
}

// Tiling of the resident steps: workgroups of `sub` stacked tiles of the current variant,
// the fewest per workgroup that leave at most one workgroup per compute unit (all of them
// then fit on the device at once, which the launch needs).  False: the raster is too large,
// or periodic (a seam's ring cells need not lie on the rim of a ragged tile), or the tile
// is not one of the 64-wide, 256-thread variants the kernel stacks, or single launches are
// faster however long the run.  min_steps: the shortest run for which they are not.
struct ResPlan {
    int sub, ntq, nwg, min_steps;
};
static bool resident_plan(const hexsv_sim *s, ResPlan *p) {
    const KGrid &g = s->grid->kg;
    if (!s->res_on || s->tile > 2 || g.perq || g.perr) return false;
    for (int sub = 1; sub <= RES_MAX_SUB; sub *= 2) {
        const int tr = TILES[s->tile].tr * sub;
        const int64_t nwg = (int64_t)s->ntq * ((g.nr + tr - 1) / tr);
        if (nwg > s->ncu) continue;
        if (!resident_fits(s->esz, s->tile, sub, s->kc.visc != 0)) return false;
        const int least = resident_min_steps(s->esz, s->tile, sub, (int)nwg, s->ncu,
                                             g.has_mask != 0, s->kc.visc != 0);
        *p = ResPlan{sub, s->ntq, (int)nwg, least};
        return least > 0;
    }
    return false;
}

// Exchange memory for a plan; all words zero (no tag is) before its first use.
static int ensure_resident(hexsv_sim *s, const ResPlan &p, hipStream_t st) {
    const size_t halo = sizeof(unsigned long long) * p.nwg * resident_halo_words(s->esz, s->tile, p.sub);
    const size_t flags = sizeof(unsigned long long) * 2 * (s->esz / 4) * p.nwg;
    const size_t bytes = halo + flags + sizeof(uint32_t) * (64 + p.nwg);
    const bool wrap = s->res_tag > 0xffff0000u;
    if (s->d_res && s->res_bytes == bytes && s->res.flag_cap == p.nwg && !wrap) return HEXSV_OK;
    if (s->res_bytes != bytes) {
        if (s->d_res) HIP_TRY(hipFree(s->d_res));
        s->d_res = nullptr;
        s->res_bytes = 0;
        if (hipMalloc(&s->d_res, bytes) != hipSuccess) {
            (void)hipGetLastError();
            s->d_res = nullptr;
            return HEXSV_ENOMEM;  // the caller steps without
        }
        s->res_bytes = bytes;
    }
    HIP_TRY(hipMemsetAsync(s->d_res, 0, bytes, st));
    s->res.halo = (unsigned long long *)s->d_res;
    s->res.flags = (unsigned long long *)(s->d_res + halo);
    s->res.abort_word = (uint32_t *)(s->d_res + halo + flags);
    s->res.done = s->res.abort_word + 64;
    s->res.flag_cap = p.nwg;
    s->res_tag = 1;
    return HEXSV_OK;
}

// A resident launch of up to ring_len steps and its fold, which commits them (trial: does not).
// drop: it is to be given up: a workgroup is missing, or all of it.
static hipError_t resident_issue(hexsv_sim *s, const ResPlan &p, bool drop, bool trial,
                                 hipStream_t st) {
    const KClose cl = close_of(s);
    const uint32_t tag0 = s->res_tag;
    s->res_tag += (uint32_t)s->ring_len + 1;
    const int grid = drop ? p.nwg - 1 : p.nwg;
    hipError_t e = hipSuccess;
    if (grid > 0)
        e = s->prec == HEXSV_FP64
                ? launch_resident<double>(s->tile, p.sub, dom_of<double>(s), s->grid->kg, s->kc,
                                          s->rn, s->d_ctl, cl, s->res, p.ntq, p.nwg, s->ntiles,
                                          s->ring_len, tag0, grid, st)
                : launch_resident<float>(s->tile, p.sub, dom_of<float>(s), s->grid->kg, s->kc,
                                         s->rn, s->d_ctl, cl, s->res, p.ntq, p.nwg, s->ntiles,
                                         s->ring_len, tag0, grid, st);
    if (e != hipSuccess) return e;
    return launch_fold_resident(s->d_ctl, cl, s->ntiles, s->kc, s->rn, s->ring_len, s->res, p.nwg,
                                trial ? 0 : tag0, st);
}

// One of a run's.
static hipError_t resident_launch(hexsv_sim *s, const ResPlan &p, hipStream_t st) {
    const bool drop = s->res_drop == 0;
    if (s->res_drop >= 0) s->res_drop -= 1;
    s->res_launches += 1;
    return resident_issue(s, p, drop, false, st);
}

// Steps a run to t_end is expected to take from here: at the current dt bound, or up to the
// step limit.
static double steps_left(const hexsv_sim *s, double t_end) {
    const Ctl &c = *s->h_ctl;
    const double dt = c.tau < s->p.dt_max ? c.tau : s->p.dt_max;
    const double need = dt > 0.0 ? (t_end - c.t) / dt + 1.0 : 1.0;
    const double by_limit = (double)(c.step_limit - c.steps);
    return by_limit < need ? by_limit : need;
}

static int sim_run(hexsv_sim *s, double t_end, int64_t max_steps, bool shortg, bool ctl_fresh,
                   hipStream_t stream);

extern "C" int hexsv_sim_run(hexsv_sim *s, double t_end, int64_t max_steps, hipStream_t stream) {
    return sim_run(s, t_end, max_steps, false, false, stream);
}

// ctl_fresh: the pinned host copy of the control block is already current
// (the caller has just read it), which saves a round trip.
static int sim_run(hexsv_sim *s, double t_end, int64_t max_steps, bool shortg, bool ctl_fresh,
                   hipStream_t stream) {
    if (!s) return fail(HEXSV_EINVAL, "run: null sim");
    if (!s->state_set) return fail(HEXSV_ESTATE, "run: call set_state first");
    if (!ctl_fresh) {
        HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
    }
    Ctl &c = *s->h_ctl;
    if (!(t_end >= c.t)) return fail(HEXSV_EDOMAIN, "run: t_end=%g before t=%g", t_end, c.t);
    c.t_end = t_end;
    c.dt_max = s->p.dt_max;
    c.step_limit = max_steps > 0 ? c.steps + max_steps : INT64_MAX;
    const int64_t limit = c.step_limit;
    HIP_TRY(hipMemcpyAsync(s->d_ctl, s->h_ctl, sizeof(Ctl), hipMemcpyHostToDevice, stream));
    // a raster that fits on the chip steps in resident launches; one that was given up
    // (see k_resident) leaves the rest of the run, and some of the next runs, to single launches
    ResPlan plan_r;
    bool resident = resident_plan(s, &plan_r) && steps_left(s, t_end) >= plan_r.min_steps &&
                    !s->res_wait.skip();
    int64_t gave_up = -1;  // steps taken when a launch was given up
    int64_t last_steps = -1;
    for (;;) {
        const int64_t before = c.steps;
        if (resident) {
            int rc = ensure_ring(s);
            if (rc) return rc;
            rc = ensure_resident(s, plan_r, stream);
            if (rc == HEXSV_ENOMEM) resident = false;
            else if (rc) return rc;
        }
        if (!resident && !s->graph_ok) {
            int rc = capture(s);
            if (rc) return rc;
        }
        // A launch past the end of the run still issues its tile loads before it
        // finds out, so each batch of replays is sized from the steps expected to
        // remain (the current dt bound, or the step limit): whole long graphs
        // while two or more of them remain, then short graphs for the rest (a
        // span of a few steps costs one host round trip).
        // A step limit that leaves a whole number of long graphs before t_end (as a
        // benchmark's step count does) is replayed as exactly those graphs.
        const double need = steps_left(s, t_end);
        const int64_t by_limit = limit - c.steps;
        const bool exact = !shortg && need == (double)by_limit && by_limit % s->gsteps == 0;
        const bool use_short = !exact && (shortg || need < 2.0 * s->gsteps);
        int reps;
        int plan[48];  // short graphs of this batch
        if (resident) {  // a launch stops where the run does
            reps = (int)fmin(64.0, ceil(fmax(need, 1.0) / s->ring_len));
        } else if (exact) {
            reps = (int)(by_limit / s->gsteps < 64 ? by_limit / s->gsteps : 64);
        } else if (use_short) {
            const double n = ceil(fmin(need, 512.0));
            reps = short_plan(n < 1.0 ? 1 : (int)n, plan, 48);
        } else {
            reps = (int)fmin(64.0, floor(need / s->gsteps) - 1.0);
        }
        if (s->timing) HIP_TRY(hipEventRecord(s->ev0, stream));
        // replays after the first start from a parity the host no longer knows: for a
        // live step the graph's hint is right while the steps before it were live (the
        // short graphs go longest first, so the odd ones come last)
        int64_t launched = 0;
        for (int k = 0; k < reps; ++k) {
            const int p = (int)((c.parity + launched) & 1);
            if (resident) {
                HIP_TRY(resident_launch(s, plan_r, stream));
            } else if (use_short) {
                HIP_TRY(hipGraphLaunch(s->sexec[plan[k]][p], stream));
                launched += SHORT_LEN[plan[k]];
            } else {
                HIP_TRY(hipGraphLaunch(s->gexec[p], stream));
                launched += s->gsteps;
            }
        }
        if (s->timing) HIP_TRY(hipEventRecord(s->ev1, stream));
        HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        if (s->timing) {
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, s->ev0, s->ev1));
            s->timed_ms += ms;
            s->timed_steps += c.steps - before;
            s->timed_replays += 1;
        }
        if (c.err)
            return fail(HEXSV_ENUMERIC, "run: non-finite value at cell %d in step %lld (t=%g)",
                        c.err_cell, (long long)c.steps + 1, c.t);
        // (a committed launch short of the run's end takes ring_len steps)
        const bool dropped = resident && c.steps - before < (int64_t)reps * s->ring_len;
        if (c.t >= t_end || c.steps >= limit) {
            if (resident) s->res_wait.clear();
            break;
        }
        if (dropped) {
            resident = false;
            gave_up = c.steps;
            continue;
        }
        if (c.steps == last_steps) break;
        last_steps = c.steps;
    }
    // single launches got further: it was not the state that could not go on
    if (gave_up >= 0 && c.steps > gave_up) s->res_wait.add();
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_resident(hexsv_sim *s, int32_t on) {
    if (!s) return fail(HEXSV_EINVAL, "set_resident: null sim");
    if (on != 0 && on != 1) return fail(HEXSV_EINVAL, "set_resident: on must be 0 or 1");
    s->res_on = on != 0;
    s->res_wait.clear();
    return HEXSV_OK;
}

extern "C" int hexsv_sim_drop_resident(hexsv_sim *s, int64_t launch) {
    if (!s || launch < 0) return fail(HEXSV_EINVAL, "drop_resident: bad argument");
    s->res_drop = launch;
    return HEXSV_OK;
}

extern "C" int64_t hexsv_sim_resident_launches(const hexsv_sim *s) { return s ? s->res_launches : -1; }

extern "C" int hexsv_sim_get_state(const hexsv_sim *sc, double *d_h, double *d_v1, double *d_v2,
                                   double *d_q1, double *d_q2, hipStream_t stream) {
    hexsv_sim *s = const_cast<hexsv_sim *>(sc);
    if (!s) return fail(HEXSV_EINVAL, "get_state: null sim");
    if (!s->state_set) return fail(HEXSV_ESTATE, "get_state: no state set");
    if (s->prec == HEXSV_FP64)
        HIP_TRY(launch_export<double>(dom_of<double>(s), s->d_ctl, s->grid->n, d_h, d_v1, d_v2, d_q1, d_q2, stream));
    else
        HIP_TRY(launch_export<float>(dom_of<float>(s), s->d_ctl, s->grid->n, d_h, d_v1, d_v2, d_q1, d_q2, stream));
    return HEXSV_OK;
}

extern "C" int hexsv_sim_timing(hexsv_sim *s, int32_t enable, double *gpu_ms, int64_t *steps,
                                int64_t *replays) {
    if (!s) return fail(HEXSV_EINVAL, "timing: null sim");
    if (gpu_ms) *gpu_ms = s->timed_ms;
    if (steps) *steps = s->timed_steps;
    if (replays) *replays = s->timed_replays;
    if (enable >= 0) {
        if (enable && !s->ev0) {
            HIP_TRY(hipEventCreate(&s->ev0));
            HIP_TRY(hipEventCreate(&s->ev1));
        }
        s->timing = enable != 0;
        s->timed_ms = 0.0;
        s->timed_steps = 0;
        s->timed_replays = 0;
    }
    return HEXSV_OK;
}

extern "C" int hexsv_sim_time_kernel(hexsv_sim *s, int32_t nlaunch, double *avg_ms,
                                     hipStream_t stream) {
    if (!s || !avg_ms || nlaunch < 1) return fail(HEXSV_EINVAL, "time_kernel: bad argument");
    if (!s->state_set) return fail(HEXSV_ESTATE, "time_kernel: no state set");
    HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    Ctl &c = *s->h_ctl;
    // make the current step live without advancing it: every launch recomputes the
    // same step from the same buffer, so the state is untouched afterwards
    const double t_end = c.t_end, dtm = c.dt_max;
    const int64_t lim = c.step_limit;
    c.t_end = INFINITY;
    c.step_limit = c.steps + 1;
    HIP_TRY(hipMemcpyAsync(s->d_ctl, s->h_ctl, sizeof(Ctl), hipMemcpyHostToDevice, stream));
    if (!s->ev0) {
        HIP_TRY(hipEventCreate(&s->ev0));
        HIP_TRY(hipEventCreate(&s->ev1));
    }
    int rc = ensure_ring(s);
    if (rc) return rc;
    const KClose cl = close_of(s);
    hipError_t e = hipSuccess;
    HIP_TRY(hipEventRecord(s->ev0, stream));
    // every launch reads slot 0 (no step pending) and recomputes the same step;
    // what it writes (slot 1, the ring's first slot, accumulator sets 0 and 1)
    // is scratch until the next run
    for (int k = 0; k < nlaunch && e == hipSuccess; ++k)
        e = step_launch(s, cl, c.parity, 0, 0, stream);
    HIP_TRY(e);
    HIP_TRY(hipEventRecord(s->ev1, stream));
    HIP_TRY(hipMemsetAsync(s->d_acc, 0, ACC_BYTES, stream));
    HIP_TRY(hipEventSynchronize(s->ev1));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, s->ev0, s->ev1));
    *avg_ms = ms / nlaunch;
    c.t_end = t_end;
    c.dt_max = dtm;
    c.step_limit = lim;
    HIP_TRY(hipMemcpyAsync(s->d_ctl, s->h_ctl, sizeof(Ctl), hipMemcpyHostToDevice, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    return HEXSV_OK;
}

// Time per step of the launches that run() would issue with the current tile: on-chip launches
// of ring_len steps and their folds where the raster takes those, else time_kernel's.  The
// launches take the same steps from the current state each time and none is committed, so the
// state is untouched afterwards; if one was given up, single launches are timed.
static int time_run(hexsv_sim *s, int nlaunch, double *ms_step, hipStream_t st) {
    ResPlan plan;
    if (!resident_plan(s, &plan)) return hexsv_sim_time_kernel(s, nlaunch, ms_step, st);
    int rc = ensure_ring(s);
    if (rc == HEXSV_OK) rc = ensure_resident(s, plan, st);
    if (rc == HEXSV_ENOMEM) return hexsv_sim_time_kernel(s, nlaunch, ms_step, st);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    Ctl &c = *s->h_ctl;
    const Ctl c0 = c;
    c.t_end = INFINITY;
    c.step_limit = c.steps + s->ring_len;
    HIP_TRY(hipMemcpyAsync(s->d_ctl, s->h_ctl, sizeof(Ctl), hipMemcpyHostToDevice, st));
    if (!s->ev0) {
        HIP_TRY(hipEventCreate(&s->ev0));
        HIP_TRY(hipEventCreate(&s->ev1));
    }
    const int reps = (nlaunch + s->ring_len - 1) / s->ring_len;
    HIP_TRY(hipEventRecord(s->ev0, st));
    for (int k = 0; k < reps; ++k) HIP_TRY(resident_issue(s, plan, false, true, st));
    HIP_TRY(hipEventRecord(s->ev1, st));
    // the launches' proposed control block and marks: did every workgroup reach the end?
    std::vector<uint32_t> done(plan.nwg);
    HIP_TRY(hipMemcpyAsync(done.data(), s->res.done, sizeof(uint32_t) * plan.nwg,
                           hipMemcpyDeviceToHost, st));
    HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl + 1, sizeof(Ctl), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    const int steps = c.open;
    const uint32_t last = s->res_tag - (uint32_t)s->ring_len - 1;
    bool all = steps == s->ring_len;
    for (uint32_t d : done) all = all && d == last;
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, s->ev0, s->ev1));
    c = c0;
    HIP_TRY(hipMemcpyAsync(s->d_ctl, s->h_ctl, sizeof(Ctl), hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (!all) return hexsv_sim_time_kernel(s, nlaunch, ms_step, st);
    *ms_step = ms / ((double)reps * steps);
    return HEXSV_OK;
}

static int set_tile(hexsv_sim *s, int v) {
    s->tile = v;
    tile_grid(v, s->grid->kg.nq, s->grid->kg.nr, &s->ntq, &s->ntiles);
    s->nwg = s->ntiles;
    drop_graph(s);
    return HEXSV_OK;
}

extern "C" int hexsv_sim_autotune(hexsv_sim *s, int32_t nlaunch, const char *cache_path,
                                  int32_t *best_tile, double *best_ms, hipStream_t stream) {
    if (!s || nlaunch < 1) return fail(HEXSV_EINVAL, "autotune: bad argument");
    if (!s->state_set) return fail(HEXSV_ESTATE, "autotune: set the state first (it is left unchanged)");
    int best = -1;
    double bms = INFINITY;
    std::vector<double> times(NUM_TILES, INFINITY);
    for (int v = 0; v < NUM_TILES; ++v) {
        set_tile(s, v);
        double ms = 0.0;
        int rc = time_run(s, 2, &ms, stream);  // warm-up
        if (rc == HEXSV_OK) rc = time_run(s, nlaunch, &ms, stream);
        if (rc != HEXSV_OK) return rc;
        times[v] = ms;
        if (ms < bms) {
            bms = ms;
            best = v;
        }
    }
    set_tile(s, best);
    if (best_tile) *best_tile = best;
    if (best_ms) *best_ms = bms;
    if (cache_path && *cache_path) {
        int rc = tune_cache_store(cache_path, "step", s->prec, s->grid->n, best, bms, times.data(),
                                  NUM_TILES);
        if (rc) return rc;
    }
    return HEXSV_OK;
}

// ------------------------------------------------ autotuning without a caller's workload

// The tuner's own workload on an nq x nr raster: a planar 5 % slope (downhill towards
// r = 0, whose side drains), theta 0.8, the paper's plant coefficient, under a uniform
// 5 cm sheet moving downslope at 0.2 m/s: every cell wet, the arithmetic of a flowing
// catchment.  Device FP64 arrays in one allocation of 6 n values: z, theta, alpha_p,
// h, v1, v2.
static int tune_workload(int nq, int nr, double a, double **out) {
    const int64_t n = (int64_t)nq * nr;
    std::vector<double> host(6 * (size_t)n);
    for (int64_t i = 0; i < n; ++i) {
        const int r = (int)(i / nq);
        host[i] = 0.05 * 1.5 * a * r;   // z over the row centres y = 1.5 a r
        host[n + i] = 0.8;              // theta
        host[2 * n + i] = 73.39;        // alpha_p
        host[3 * n + i] = 0.05;         // h
        host[4 * n + i] = 0.0;          // v1
        host[5 * n + i] = -0.2;         // v2
    }
    double *d = nullptr;
    hipError_t e = hipMalloc(&d, sizeof(double) * 6 * (size_t)n);
    if (e != hipSuccess) return fail(HEXSV_ENOMEM, "autotune: %s", hipGetErrorString(e));
    e = hipMemcpy(d, host.data(), sizeof(double) * 6 * (size_t)n, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(d);
        return fail(HEXSV_EHIP, "autotune: %s", hipGetErrorString(e));
    }
    *out = d;
    return HEXSV_OK;
}

extern "C" int hexsv_autotune(const char *cache_path, int32_t kernel, int32_t precision,
                              int64_t cells_hint, int32_t *best_tile, double *best_ms,
                              hipStream_t stream) {
    if (!cache_path || !*cache_path) return fail(HEXSV_EINVAL, "autotune: no cache path");
    if (kernel != HEXSV_TUNE_STEP && kernel != HEXSV_TUNE_ENSEMBLE)
        return fail(HEXSV_EINVAL, "autotune: kernel %d is not HEXSV_TUNE_STEP or _ENSEMBLE", kernel);
    if (precision != HEXSV_FP64 && precision != HEXSV_FP32)
        return fail(HEXSV_EINVAL, "autotune: precision %d", precision);
    if (cells_hint < 64 || cells_hint > ((int64_t)1 << 30))
        return fail(HEXSV_EINVAL, "autotune: cells_hint %lld outside [64, 2^30]", (long long)cells_hint);
    const int nscen = kernel == HEXSV_TUNE_STEP ? 1 : 8;
    const int side = (int)ceil(sqrt((double)cells_hint / nscen));
    const double a = 1.0;
    hexsv_grid_desc gd;
    memset(&gd, 0, sizeof gd);
    gd.nq = side;
    gd.nr = side;
    gd.edge = a;
    gd.side_bc[HEXSV_S] = HEXSV_OUTFLOW;
    gd.side_bc[HEXSV_E] = gd.side_bc[HEXSV_N] = gd.side_bc[HEXSV_W] = HEXSV_WALL;
    gd.mask_bc = HEXSV_WALL;
    hexsv_grid *grid = nullptr;
    int rc = hexsv_grid_create(&gd, &grid);
    if (rc) return rc;
    double *f = nullptr;
    rc = tune_workload(side, side, a, &f);
    if (rc) {
        hexsv_grid_destroy(grid);
        return rc;
    }
    const int64_t n = (int64_t)side * side;
    hexsv_params p;
    memset(&p, 0, sizeof p);
    p.g = 9.81;
    p.cfl = 0.5;
    p.dt_max = 1.0;
    p.precision = precision;
    p.tile = -1;
    if (kernel == HEXSV_TUNE_STEP) {
        hexsv_sim *sim = nullptr;
        rc = hexsv_sim_create(grid, &p, &sim);
        if (!rc) rc = hexsv_sim_set_fields(sim, f, f + n, f + 2 * n, nullptr, 0.00709, stream);
        if (!rc) rc = hexsv_sim_set_state(sim, 0.0, f + 3 * n, f + 4 * n, f + 5 * n, stream);
        if (!rc) rc = hexsv_sim_autotune(sim, 30, cache_path, best_tile, best_ms, stream);
        hexsv_sim_destroy(sim);
    } else {
        std::vector<const hexsv_grid *> grids(nscen, grid);
        hexsv_ensemble *ens = nullptr;
        p.ensemble_mode = HEXSV_ENS_AUTO;
        rc = hexsv_ensemble_create(nscen, grids.data(), &p, &ens);
        const hexsv_rain rain{0, 50.0 / 3.6e6, 0.0, INFINITY};
        for (int sc = 0; sc < nscen && !rc; ++sc)
            rc = hexsv_ensemble_set_scenario(ens, sc, f, f + n, f + 2 * n, 0.00709, &rain, 0.0,
                                             f + 3 * n, f + 4 * n, f + 5 * n, stream);
        if (!rc) rc = hexsv_ensemble_autotune(ens, 10, cache_path, best_tile, best_ms, stream);
        hexsv_ensemble_destroy(ens);
    }
    (void)hipStreamSynchronize(stream);
    (void)hipFree(f);
    hexsv_grid_destroy(grid);
    return rc;
}

extern "C" int hexsv_sim_get_books(hexsv_sim *s, hexsv_books *out, hipStream_t stream) {
    if (!s || !out) return fail(HEXSV_EINVAL, "get_books: null argument");
    if (!s->state_set) return fail(HEXSV_ESTATE, "get_books: no state set");
    HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    const Ctl &c = *s->h_ctl;
    out->t = c.t;
    out->initial = c.initial;
    out->stored = c.stored;
    out->rain = c.rain;
    out->outflow = c.outflow;
    out->clamp = c.clamp;
    // water supplied: initial, rain and any net inflow through Dirichlet edges
    double ref = c.initial + c.rain + (c.outflow < 0.0 ? -c.outflow : 0.0);
    if (ref < 1e-300) ref = 1e-300;
    out->residual = fabs(c.stored - (c.initial + c.rain - c.outflow + c.clamp)) / ref;
    out->steps = c.steps;
    out->dt_min = c.dt_min;
    out->dt_max_seen = c.dt_max_seen;
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_books(hexsv_sim *s, const hexsv_books *b, hipStream_t stream) {
    if (!s || !b) return fail(HEXSV_EINVAL, "set_books: null argument");
    if (!s->state_set) return fail(HEXSV_ESTATE, "set_books: call set_state first");
    if (!isfinite(b->t) || b->steps < 0) return fail(HEXSV_EDOMAIN, "set_books: bad time or step count");
    HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    Ctl &c = *s->h_ctl;
    c.t = b->t;
    c.t_end = b->t;
    c.initial = b->initial;
    c.rain = b->rain;
    c.outflow = b->outflow;
    c.clamp = b->clamp;
    c.steps = b->steps;
    c.step_limit = b->steps;
    c.dt_min = b->dt_min;
    c.dt_max_seen = b->dt_max_seen;
    HIP_TRY(hipMemcpyAsync(s->d_ctl, s->h_ctl, sizeof(Ctl), hipMemcpyHostToDevice, stream));
    HIP_TRY(s->prec == HEXSV_FP64 ? prime<double>(s, 0, stream) : prime<float>(s, 0, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    return HEXSV_OK;
}

// ------------------------------------------------------------ surrogate

// Records of a window's predicted state: one per workgroup of the apply kernel
// (WIN_PARTS) or per conv tile of the last-layer kernel, whichever runs.
static int win_part_count(const hexsv_sim *s) {
    return std::max(WIN_PARTS, nn::conv_tiles(s->grid->kg.nq, s->grid->kg.nr, 1));
}

// Scratch of the windows (probe state) and their control record.
static int window_buffers(hexsv_sim *s) {
    if (!s->d_sw) {
        HIP_TRY(hipMalloc(&s->d_sw, sizeof(SurWin)));
        HIP_TRY(hipHostMalloc(&s->h_sw, sizeof(SurWin), hipHostMallocDefault));
        // the predicted state's records, then one per probe tile
        HIP_TRY(hipMalloc(&s->d_op, sizeof(Part) * ((size_t)win_part_count(s) + win_probe_tiles(
                                                                   s->grid->kg.nq, s->grid->kg.nr))));
        HIP_TRY(hipMalloc(&s->d_scr, s->esz * 3 * (size_t)s->grid->n));
        HIP_TRY(hipMalloc(&s->d_slope, sizeof(float2) * (size_t)s->grid->n));
    }
    return HEXSV_OK;
}

template <typename T>
static int window_slope(hexsv_sim *s, hipStream_t st) {
    if (!s->slope_ok) {
        HIP_TRY(launch_win_slope<T>(dom_of<T>(s), s->grid->kg, s->grid->edge, s->d_slope, st));
        s->slope_ok = true;
    }
    return HEXSV_OK;
}

static void window_record(hexsv_sim *s, double t_stop, double window, int32_t k, double tol,
                          int project) {
    SurWin &w = *s->h_sw;
    memset(&w, 0, sizeof w);
    w.t_stop = t_stop;
    w.window = window;
    w.tol = tol;
    w.k = k;
    w.project = project ? 1 : 0;
    w.perr_cell = -1;
    w.c0 = -1.0;
}

static FeatScale feat_scale(const float *sc) { return FeatScale{sc[0], sc[1], sc[2], sc[5], sc[3], sc[4]}; }

template <typename T>
static int window_features(hexsv_sim *s, hexsv_surrogate *sur, double window, int32_t k,
                           float *d_features, hipStream_t st) {
    int rc = window_buffers(s);
    if (rc) return rc;
    float sc[8];
    rc = hexsv_surrogate_get_scales(sur, sc, 8);
    if (rc) return rc;
    rc = window_slope<T>(s, st);
    if (rc) return rc;
    window_record(s, INFINITY, window, k, 0.0, 0);
    HIP_TRY(hipMemcpyAsync(s->d_sw, s->h_sw, sizeof(SurWin), hipMemcpyHostToDevice, st));
    const KDom<T> d = dom_of<T>(s);
    HIP_TRY(launch_win_reset(s->d_sw, st));
    HIP_TRY(launch_win_probe<T>(d, s->grid->kg, s->kc, s->rn, s->d_ctl, s->d_sw, (T *)s->d_scr,
                                s->p.dt_max, s->d_slope, feat_scale(sc), 2, d_features,
                                s->d_op + win_part_count(s), st));
    return HEXSV_OK;
}

extern "C" int hexsv_sim_surrogate_features(hexsv_sim *s, hexsv_surrogate *sur, double window,
                                            int32_t k, float *d_features, hipStream_t stream) {
    if (sur && k <= 0) k = hexsv_surrogate_steps(sur);  // the surrogate's own window length
    if (!s || !sur || !d_features || !(window > 0.0) || !isfinite(window) || k < 1)
        return fail(HEXSV_EINVAL, "surrogate_features: bad argument");
    if (!s->state_set) return fail(HEXSV_ESTATE, "surrogate_features: call set_state first");
    if (s->grid->n_dirichlet)
        return fail(HEXSV_EUNSUPPORTED, "surrogate_features: windows are not built for Dirichlet cells");
    if (s->kc.visc || s->kc.f_inf > 0.0 || s->as_field)  // the probe step runs the plain scheme
        return fail(HEXSV_EUNSUPPORTED,
                    "surrogate_features: windows are not built for the viscous flux, infiltration "
                    "or a soil field");
    return s->prec == HEXSV_FP64 ? window_features<double>(s, sur, window, k, d_features, stream)
                                 : window_features<float>(s, sur, window, k, d_features, stream);
}

// Windows chained in one graph launch (a refused window stops the rest of
// its chain, whose kernels then return at once: dead windows, each still a few
// launches).  Graphs are captured for the chain lengths below.  After a refusal
// the next chain is as long as the run of kept windows before it plus one
// (refusals tend to recur at that period, so the chain ends where the next
// refusal is expected, and a run of refusals tries one window at a time); a
// chain kept whole is followed by one at least twice as long (fewer host round
// trips).
constexpr int N_CHAINS = 6;
static const int WIN_CHAINS[N_CHAINS] = {1, 2, 3, 4, 8, 16};
static int chain_at_most(int n) {  // the longest captured chain of at most n windows
    int j = 0;
    while (j + 1 < N_CHAINS && WIN_CHAINS[j + 1] <= n) ++j;
    return j;
}
static int chain_at_least(int n) {  // the shortest captured chain of at least n windows
    int j = 0;
    while (j + 1 < N_CHAINS && WIN_CHAINS[j] < n) ++j;
    return j;
}
// Most plain steps one refused window may take before the run reports a stall.
static const int64_t FALLBACK_STEP_LIMIT = 1 << 20;

// One window: probe step (which starts the window and forms the network's
// features with the start state's outflow rate), network, predicted state (with
// its sums and outflow rate), gate, and the optional projection.
template <typename T>
static int window_body(hexsv_sim *s, hexsv_surrogate *sur, void *x0, const float *out,
                       const float *sc, hipStream_t st) {
    const KDom<T> d = dom_of<T>(s);
    const KGrid &g = s->grid->kg;
    const double l = s->grid->edge;
    T *scr = (T *)s->d_scr;
    const double dt_max = s->p.dt_max;
    Part *part = s->d_op, *op0 = s->d_op + win_part_count(s);
    const int n_op0 = win_probe_tiles(g.nq, g.nr);
    HIP_TRY(launch_win_probe<T>(d, g, s->kc, s->rn, s->d_ctl, s->d_sw, scr, dt_max, s->d_slope,
                                feat_scale(sc), 1, x0, op0, st));
    // the hidden layers, then the last layer with the predicted state as its epilogue;
    // a fused forward runs whole and the predicted state follows from its output
    SurLast last;
    int rc = sur_forward_hidden(sur, s->grid, st, &s->d_sw->live, &last);
    int n_part = WIN_PARTS;
    if (rc == HEXSV_OK) {
        HIP_TRY(launch_win_last<T>(last.x, last.wm, last.bias, last.cm, d, g, l, s->kc, s->d_ctl,
                                   s->d_sw, scr, dt_max, sc[3], sc[4], 1e-6, part, st));
        n_part = nn::conv_tiles(g.nq, g.nr, 1);
    } else if (rc == HEXSV_EUNSUPPORTED) {
        rc = sur_forward_x0(sur, s->grid, st, &s->d_sw->live);
        if (rc) return rc;
        HIP_TRY(launch_win_apply<T>(d, g, l, s->kc, s->d_ctl, s->d_sw, scr, dt_max, out,
                                    nn::OUT_STRIDE, sc[3], sc[4], 1e-6, part, st));
    } else {
        return rc;
    }
    HIP_TRY(launch_win_gate(s->d_ctl, s->d_sw, part, n_part, op0, n_op0, s->kc, st));
    return HEXSV_OK;
}

template <typename T>
static int window_chain(hexsv_sim *s, hexsv_surrogate *sur, int nwin, void *x0, const float *out,
                        const float *sc, hipStream_t st) {
    HIP_TRY(launch_win_reset(s->d_sw, st));
    for (int w = 0; w < nwin; ++w) {
        int rc = window_body<T>(s, sur, x0, out, sc, st);
        if (rc) return rc;
    }
    // the projection of the chain's last accepted window (the windows read it scaled)
    HIP_TRY(launch_win_scale<T>(dom_of<T>(s), s->grid->n, s->d_ctl, s->d_sw, st));
    return HEXSV_OK;
}

template <typename T>
static int capture_windows(hexsv_sim *s, hexsv_surrogate *sur, void *x0, const float *out,
                           const float *sc, uint64_t gen) {
    drop_win_graph(s);
    for (int j = 0; j < N_CHAINS; ++j) {
        HIP_TRY(hipStreamBeginCapture(s->cap, hipStreamCaptureModeThreadLocal));
        int rc = window_chain<T>(s, sur, WIN_CHAINS[j], x0, out, sc, s->cap);
        hipGraph_t g = nullptr;
        hipError_t e2 = hipStreamEndCapture(s->cap, &g);
        if (rc || e2 != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            return rc ? rc
                      : fail(HEXSV_EHIP, "window graph capture failed: %s", hipGetErrorString(e2));
        }
        s->wgraph[j] = g;
        HIP_TRY(hipGraphInstantiate(&s->wexec[j], g, nullptr, nullptr, 0));
    }
    s->w_sur = sur;
    s->w_gen = gen;
    return HEXSV_OK;
}

template <typename T>
static int surrogate_windows(hexsv_sim *s, hexsv_surrogate *sur, double t_end, double window,
                             int32_t k, double tol, int project, int64_t *n_acc, int64_t *n_fb,
                             hipStream_t st) {
    int rc = window_buffers(s);
    if (rc) return rc;
    float sc[8];
    rc = hexsv_surrogate_get_scales(sur, sc, 8);
    if (rc) return rc;
    void *x0 = nullptr;
    const float *out = nullptr;
    uint64_t gen = 0;
    rc = sur_window_bind(sur, s->grid->kg.nq, s->grid->kg.nr, &x0, &out, &gen);
    if (rc) return rc;
    rc = window_slope<T>(s, st);
    if (rc) return rc;
    // the scales are kernel arguments of the graph: rebuild when they change
    static_assert(sizeof(sc) == 8 * sizeof(float), "scales");
    bool same = s->wexec[N_CHAINS - 1] && s->w_sur == sur && s->w_gen == gen;
    for (int j = 0; j < 8 && same; ++j) same = s->w_scales[j] == sc[j];
    if (!same) {
        rc = capture_windows<T>(s, sur, x0, out, sc, gen);
        if (rc) return rc;
        for (int j = 0; j < 8; ++j) s->w_scales[j] = sc[j];
    }
    window_record(s, t_end, window, k, tol, project);
    const SurWin &w = *s->h_sw;
    HIP_TRY(hipMemcpyAsync(s->d_sw, s->h_sw, sizeof(SurWin), hipMemcpyHostToDevice, st));
    Ctl &c = *s->h_ctl;
    HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    int level = chain_at_most(2);  // index into WIN_CHAINS
    int streak = 0;                // windows refused since the last kept one
    int run = 0;                   // windows kept since the last refusal
    for (;;) {  // c is current here
        if (c.err) return fail(HEXSV_ENUMERIC, "run_surrogate: non-finite value at cell %d", c.err_cell);
        const double t0 = c.t;
        if (t0 >= t_end) break;
        // whole windows left, formed exactly as the device forms them
        const int want = WIN_CHAINS[level];
        int left = 0;
        for (double t = t0; left < want && t + window <= t_end; t += window) ++left;
        if (left == 0) {  // last partial span: the plain solver
            rc = sim_run(s, t_end, 0, true, true, st);
            if (rc) return rc;
            *n_fb += 1;
            break;
        }
        if (left == want) {
            HIP_TRY(hipGraphLaunch(s->wexec[level], st));
        } else {
            rc = window_chain<T>(s, sur, left, x0, out, sc, st);
            if (rc) return rc;
        }
        HIP_TRY(hipMemcpyAsync(s->h_sw, s->d_sw, sizeof(SurWin), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipMemcpyAsync(s->h_ctl, s->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        *n_acc += w.accepted;
        s->w_stats[0] += w.accepted;
        if (w.rejected) s->w_stats[w.why == 1 ? 1 : (w.why == 2 ? 2 : 3)] += 1;
        if (w.accepted) streak = 0;
        run += (int)w.accepted;
        if (w.rejected) {  // the refused window's span, by the plain solver from its start
            level = chain_at_most(run + 1);
            run = 0;
            if (c.err) continue;
            ++streak;
            // the refused span, then the back-off spans; each span ends where a window would
            int spans = 1;
            if (streak >= 2) spans += std::min(1 << std::min(streak - 1, 30), s->w_backoff);
            for (int j = 0; j < spans; ++j) {
                const double target = c.t + window;
                if (j > 0 && (c.err || target > t_end)) break;
                rc = sim_run(s, target, FALLBACK_STEP_LIMIT, true, true, st);
                if (rc) return rc;
                if (!(c.t >= target))
                    return fail(HEXSV_ENUMERIC,
                                "run_surrogate: the solver stalled at t=%g before %g", c.t, target);
                *n_fb += 1;
            }
            // the solver's state is the new reference wave speed of the windows that follow
            static const double fresh = -1.0;
            HIP_TRY(hipMemcpyAsync((char *)s->d_sw + offsetof(SurWin, c0), &fresh, sizeof fresh,
                                   hipMemcpyHostToDevice, st));
        } else {
            level = chain_at_least(2 * left);
        }
    }
    return HEXSV_OK;
}

extern "C" int hexsv_sim_set_surrogate_backoff(hexsv_sim *s, int32_t max_spans) {
    if (!s || max_spans < 0) return fail(HEXSV_EINVAL, "set_surrogate_backoff: bad argument");
    s->w_backoff = max_spans;
    return HEXSV_OK;
}

extern "C" int hexsv_sim_window_kernels(const hexsv_sim *s) {
    if (!s) return fail(HEXSV_EINVAL, "window_kernels: null sim");
    size_t n = 0;
    if (s->wgraph[0]) HIP_TRY(hipGraphGetNodes(s->wgraph[0], nullptr, &n));
    return (int)n;
}

extern "C" int hexsv_sim_surrogate_stats(const hexsv_sim *s, int64_t *counts) {
    if (!s || !counts) return fail(HEXSV_EINVAL, "surrogate_stats: null argument");
    for (int j = 0; j < 4; ++j) counts[j] = s->w_stats[j];
    return HEXSV_OK;
}

extern "C" int hexsv_sim_run_surrogate(hexsv_sim *s, hexsv_surrogate *sur, double t_end,
                                       double window, int32_t k, double residual_tol,
                                       int32_t project, int64_t *n_accepted, int64_t *n_fallback,
                                       hipStream_t st) {
    if (sur && k <= 0) k = hexsv_surrogate_steps(sur);  // the surrogate's own window length
    if (!s || !sur || !(window > 0.0) || !isfinite(window) || k < 1 || !(residual_tol >= 0.0))
        return fail(HEXSV_EINVAL, "run_surrogate: bad argument");
    if (!s->state_set) return fail(HEXSV_ESTATE, "run_surrogate: call set_state first");
    if (s->kc.visc)
        return fail(HEXSV_EUNSUPPORTED, "run_surrogate: windows are not built for the viscous flux");
    if (s->grid->n_dirichlet)
        return fail(HEXSV_EUNSUPPORTED, "run_surrogate: windows are not built for Dirichlet or flux cells");
    if (s->kc.f_inf > 0.0 || s->as_field)
        return fail(HEXSV_EUNSUPPORTED,
                    "run_surrogate: windows are not built for infiltration or a soil field");
    int64_t a = 0, f = 0;
    const int rc =
        s->prec == HEXSV_FP64
            ? surrogate_windows<double>(s, sur, t_end, window, k, residual_tol, project, &a, &f, st)
            : surrogate_windows<float>(s, sur, t_end, window, k, residual_tol, project, &a, &f, st);
    if (n_accepted) *n_accepted = a;
    if (n_fallback) *n_fallback = f;
    return rc;
}
