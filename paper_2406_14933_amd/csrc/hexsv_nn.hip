// hexsv_nn.hip — kernels of the learned hex-convolution surrogate: BF16 MFMA
// forward and gradient hex convolutions with FP32 accumulation (the tile's
// staging and MFMA mapping are in hexsv_conv.h), the one-launch 4-layer forward,
// the L1 loss, Adam, and the weight-layout preparation.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "hexsv_conv.h"
#include "hexsv_device.h"
#include "hexsv_nn.h"

namespace hexsv {
namespace nn {

// ---------------------------------------------------------------- conv

// out[i][co] for the tile; EPI selects the epilogue:
//   EPI_RELU:  bf16 out = max(acc + b, 0)           (hidden layers, forward)
//   EPI_LIN:   f32 out[i][co < cout_real] = acc + b  (last layer, forward)
template <int CIN, int COUT, int EPI>
__global__ __launch_bounds__(NT) void k_hexconv(const __bf16 *__restrict__ x,
                                                const __bf16 *__restrict__ wm,
                                                const float *__restrict__ bias, void *out, int nq,
                                                int nr, int ntiles_total, int cout_real,
                                                const int32_t *live, ConvMask cm) {
    constexpr int CH = CIN / 8;
    constexpr int MB = COUT / 16;                 // output-channel blocks
    __shared__ uint4 lds[NSLOT * CH];
    __shared__ uint8_t fl[NSLOT];
    const int ntq = (nq + TQ - 1) / TQ, ntr = (nr + TR - 1) / TR;
    // XCD-banded tile order: every layer gives a tile to the same XCD, so the
    // activations a layer writes are mostly read back from that XCD's L2
    const int tile = xcd_tile(blockIdx.x, gridDim.x, ntiles_total, 0);
    if (tile < 0) return;
    if (live && !*live) return;  // a surrogate window that does not run
    int b, q0, r0;
    tile_of(tile, ntq, ntr, b, q0, r0);
    const int64_t soff = (int64_t)b * nq * nr;
    stage_act<CIN>(lds, fl, x, nq, nr, soff, q0, r0, cm);
    __syncthreads();
    const bool masked = cm.active != nullptr;

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;  // wave w: tile row w
    const int g = lane >> 4, l16 = lane & 15;
    f32x4 acc[MB][4];
    conv_acc<CIN, COUT>(lds, fl, masked, wm, acc);
    // epilogue: lane holds channels co = m*16 + 4g + j of cell n*16 + l16
    const int r = r0 + w;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int q = q0 + n * 16 + l16;
        if (q >= nq || r >= nr) continue;
        const int64_t i = soff + (int64_t)r * nq + q;
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const int co = m * 16 + 4 * g;
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = acc[m][n][j] + bias[co + j];
            if constexpr (EPI == EPI_LIN) {
                float *o = reinterpret_cast<float *>(out) + i * OUT_STRIDE;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (co + j < cout_real) o[co + j] = v[j];
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = v[j] > 0.f ? v[j] : 0.f;
                __bf16 *o = reinterpret_cast<__bf16 *>(out) + i * COUT + co;
                typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                bf16x4 pk;
#pragma unroll
                for (int j = 0; j < 4; ++j) pk[j] = (__bf16)v[j];
                *reinterpret_cast<bf16x4 *>(o) = pk;
            }
        }
    }
}

// ------------------------------------------------------- fused 4-layer forward
//
// The whole 4-layer network (16 -> 32 -> 32 -> 32 -> 16 channels) in one kernel: a workgroup
// sweeps a strip of columns row by row with the four layers two rows apart, so a hidden row
// lives in LDS for one step and never leaves the CU.  The layer chain moves 540 bytes a cell,
// most of them hidden activations, against the 56 this reads and writes; on 16 x 512 x 512
// samples it takes 609 us, this 273 us (its MFMAs run at 0.9 PFLOP/s, where an 8192^3 library
// product reaches 1.2 on the card).
//
// All layers share a frame of 64 columns (four MFMA columns of 16 cells); layer l's outermost
// l columns lack a neighbour, so 58 columns come out, and 6 of 64 are computed twice (10 % of
// the MFMA work; the 16 x 16 tiles with a 4-cell margin this replaces spent 46 %).  Sixteen
// waves: four per layer, one MFMA column each, so every SIMD holds one wave of each layer and
// has 43 MFMAs a row.  Weights and the operands that a layer's rows share stay in registers for
// the whole strip.  A row is a chain of short phases (LDS reads, seven dependent MFMAs,
// epilogue, barrier): four waves per SIMD hide each other's (370 us with two, 475 us with two
// workgroups of eight waves that read every operand from LDS).
//
// Each layer's arithmetic is k_hexconv's: the same MFMA, the same K order, bias, ReLU and bf16
// rounding, so the output equals the chain's bit for bit.  Positions outside the raster are
// zero for the taps, as the chain stages them.  MASK: a tap t >= 1 is zero unless the cell and
// the neighbour are both in the domain (flags staged with the input); without a mask only
// positions outside the raster (after periodic wraps) are cut, by storing them as zeros.
namespace r4 {
constexpr int FW = 64;             // frame columns
constexpr int OW = FW - 6;         // output columns
constexpr int LW = FW + 2;         // staged columns (one pad or halo column on each side)
constexpr int ICH = 4;             // input rows loaded at a time
constexpr int IRING = 12;          // input rows staged
constexpr int FRING = 32;          // flag rows staged (layer 3 is 6 rows behind layer 0)
constexpr int NTH = 1024;
constexpr int EXTRA = 9;           // steps of a strip beyond its output rows
constexpr int DQ[7] = {0, 1, 0, -1, -1, 0, 1};
constexpr int DR[7] = {0, 0, 1, 1, 0, -1, -1};
}  // namespace r4

// Element offset of 8-channel chunk `ch` of staged column c: a rotation of the chunks by column
// keeps the 16 cells of an MFMA column on distinct LDS banks without padding (32 channels: four
// chunks of 16 bytes, 16 channels: two).
__device__ inline int act_at(int c, int ch) { return c * 32 + ((ch ^ ((c >> 2) & 3)) << 3); }
__device__ inline int in_at(int c, int ch) { return c * 16 + ((ch ^ ((c >> 3) & 1)) << 3); }

// One MFMA column's operands of the 3 rows around an output row, one set per dq (-1, 0, +1):
// lane (g, l16) holds channels 8 g .. 8 g + 7 of its cell's neighbour.  Rows take turns: with
// the newest (above the output row) in slot j, the middle one is in j + 2 and the oldest in
// j + 1 (mod 3), so that no row is moved; with a domain mask, whose predicates take the registers
// that three copies of a step need, slot 0 is the newest and rows are moved.
struct Taps {
    bf16x8 r[3][3];
    int in[3];  // MASK: bit dq + 1, the cell is in the domain
};

// A new row into slot j; staged column c + 1 is frame column c.
template <bool MASK>
__device__ inline void taps_push(Taps &t, int j, const __bf16 *row, int c, int g,
                                 const uint8_t *frow) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
        t.r[j][d] = *reinterpret_cast<const bf16x8 *>(row + act_at(c + d, g));
    if constexpr (MASK) t.in[j] = frow[c] | frow[c + 1] << 1 | frow[c + 2] << 2;
}
// The newest row becomes the middle one, with slot 0 free.
__device__ inline void taps_move(Taps &t) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        t.r[1][d] = t.r[2][d];
        t.r[2][d] = t.r[0][d];
    }
    t.in[1] = t.in[2];
    t.in[2] = t.in[0];
}
// MASK: the operand of a tap t >= 1 is zero unless both cells are in the domain.
template <bool MASK>
__device__ inline bf16x8 tap_of(const Taps &t, int j, int tap) {
    using namespace r4;
    const int mid = (j + 2) % 3, k = DR[tap] > 0 ? j : DR[tap] == 0 ? mid : (j + 1) % 3;
    bf16x8 v = t.r[k][1 + DQ[tap]];
    if constexpr (MASK)
        if (tap > 0 && !((t.in[mid] >> 1) & (t.in[k] >> (1 + DQ[tap])) & 1)) v = bf16x8{};
    return v;
}

// Output channel of row i of MFMA block m (of two): a lane's eight accumulators, rows 4 g .. 4 g
// + 3 of both blocks, are channels 8 g .. 8 g + 7, one 16-byte chunk of its cell.
__device__ inline int row_channel(int m, int i) { return 8 * (i >> 2) + 4 * m + (i & 3); }

// The eight hidden activations of lane group g's cell into its staged row; zeros unless keep.
__device__ inline uint4 put_act(__bf16 *row, int c, int g, const f32x4 (&acc)[2],
                                const float (&b)[8], bool keep) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        const float v0 = acc[j / 4][j % 4] + b[j], v1 = acc[j / 4][j % 4 + 1] + b[j + 1];
        const bf16x2 pk = {(__bf16)(v0 > 0.f ? v0 : 0.f), (__bf16)(v1 > 0.f ? v1 : 0.f)};
        w[j / 2] = keep ? __builtin_bit_cast(uint32_t, pk) : 0u;
    }
    const uint4 v = make_uint4(w[0], w[1], w[2], w[3]);
    *reinterpret_cast<uint4 *>(row + act_at(c + 1, g)) = v;
    return v;
}

// F32IN: x holds the FP32 features (FEATURES per cell), else the packed bf16 input.
// w4: write the fourth float of each output too (zero).  KEEP: the packed input and the hidden
// activations go to memory too, as the chain leaves them for the gradient.
template <bool MASK, bool F32IN, bool KEEP>
__global__ __launch_bounds__(r4::NTH) void k_hexnet4(const void *__restrict__ x, Net4 nw,
                                                        float *__restrict__ out, int nq, int nr,
                                                        int batch, int rh, int nseg, int w4,
                                                        const int32_t *live, ConvMask cm,
                                                        Net4Keep keep) {
    using namespace r4;
    __shared__ __align__(16) __bf16 sin[IRING][LW * 16];
    __shared__ __align__(16) __bf16 act[3][2][LW * 32];
    __shared__ uint8_t fl[MASK ? FRING : 1][LW + 2];
    if (live && !*live) return;  // a surrogate window that does not run
    const int nstrip = (nq + OW - 1) / OW;
    const int wgs = nstrip * nseg * batch;
    const int id = xcd_tile(blockIdx.x, gridDim.x, wgs, 0);
    if (id < 0) return;
    const int b = id / (nstrip * nseg), rem = id - b * nstrip * nseg;
    const int strip = rem / nseg, seg = rem - strip * nseg;
    const int Q0 = strip * OW - 3;  // raster column of frame column 0
    const int R0 = seg * rh, R1 = R0 + rh < nr ? R0 + rh : nr;
    if (R0 >= nr) return;
    const int64_t soff = (int64_t)b * nq * nr;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane >> 4, l16 = lane & 15;
    // staged rows start as zeros: pad channels and columns are never written
    for (int i = tid; i < IRING * LW * 16 / 8; i += NTH)
        reinterpret_cast<uint4 *>(&sin[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = tid; i < 3 * 2 * LW * 32 / 8; i += NTH)
        reinterpret_cast<uint4 *>(&act[0][0][0])[i] = make_uint4(0u, 0u, 0u, 0u);

    // input rows: staged row v is raster row R0 - 4 + v, staged column c raster column Q0 - 1 + c;
    // thread p of 256 owns the same elements of every row
    constexpr int EL = F32IN ? (LW * FEATURES + 255) / 256 : 1;
    const int p = tid & 255;
    int eq[EL], eo[EL];  // raster column (-1: none) and offset in the staged row
    int ec[EL];          // element of the source cell
#pragma unroll
    for (int i = 0; i < EL; ++i) {
        const int e = p + 256 * i;
        const int c = F32IN ? e / FEATURES : e / 2, ch = F32IN ? e - c * FEATURES : e - c * 2;
        int q = Q0 - 1 + c;
        if (cm.perq) q = ((q % nq) + nq) % nq;
        const bool ok = c < LW && q >= 0 && q < nq;
        eq[i] = ok ? q : -1;
        ec[i] = ch;
        eo[i] = F32IN ? in_at(c, ch >> 3) + (ch & 7) : in_at(c, ch);
    }
    const bool fthread = MASK && p < LW;  // stages the flag of column p
    int fq = Q0 - 1 + p;
    if (MASK && cm.perq) fq = ((fq % nq) + nq) % nq;
    float vf[F32IN ? ICH : 1][EL];
    uint4 vb[F32IN ? 1 : ICH];
    uint8_t vfl[ICH];
    auto load_rows = [&](int v0) {
#pragma unroll
        for (int k = 0; k < ICH; ++k) {
            int r = R0 - 4 + v0 + k;
            if (cm.perr) r = ((r % nr) + nr) % nr;
            const bool rok = r >= 0 && r < nr;
            if constexpr (F32IN) {
#pragma unroll
                for (int i = 0; i < EL; ++i)
                    vf[k][i] = rok && eq[i] >= 0
                                   ? reinterpret_cast<const float *>(x)[(soff + (int64_t)r * nq + eq[i]) * FEATURES + ec[i]]
                                   : 0.f;
            } else {
                vb[k] = rok && eq[0] >= 0
                            ? reinterpret_cast<const uint4 *>(x)[(soff + (int64_t)r * nq + eq[0]) * 2 + ec[0]]
                            : make_uint4(0u, 0u, 0u, 0u);
            }
            vfl[k] = MASK && fthread && rok && fq >= 0 && fq < nq
                         ? (uint8_t)(cm.active[(int64_t)r * nq + fq] != 0)
                         : (uint8_t)0;
        }
    };
    auto store_rows = [&](int v0) {
#pragma unroll
        for (int k = 0; k < ICH; ++k) {
            __bf16 *row = sin[(v0 + k) % IRING];
            if constexpr (F32IN) {
#pragma unroll
                for (int i = 0; i < EL; ++i)
                    if (p + 256 * i < LW * FEATURES) row[eo[i]] = (__bf16)vf[k][i];
            } else {
                if (p < 2 * LW) *reinterpret_cast<uint4 *>(row + eo[0]) = vb[k];
            }
            if constexpr (MASK)
                if (fthread) fl[(v0 + k) % FRING][p] = vfl[k];
        }
    };
    // is frame column c a raster column? (rows are tested as they come)
    auto inside_q = [&](int c) { return cm.perq || (Q0 + c >= 0 && Q0 + c < nq); };
    auto inside_r = [&](int r) { return cm.perr || (r >= 0 && r < nr); };

    // every wave: one MFMA column (frame columns 16 n .. 16 n + 15) of one layer
    const int steps = (R1 - R0) + EXTRA;
    constexpr int UN = MASK ? 1 : 3;  // steps per loop turn (see Taps)
    const int n = wave & 3, c = n * 16 + l16;
    const bool qok = inside_q(c);
    // this workgroup's output columns; its output rows are R0 to R1 - 1 (KEEP: of every layer)
    const bool own_q = c >= 3 && c < 3 + OW && Q0 + c < nq;
    const auto own_r = [&](int r) { return r >= R0 && r < R1; };
    const auto cell_at = [&](int r) { return soff + (int64_t)r * nq + Q0 + c; };
    if (wave >= 8) load_rows(wave >= 12 ? ICH : 0);  // the first rows, one latency for all
    __syncthreads();
    if (wave >= 12) {
        // ---- layer 0, and the input
        bf16x8 w[4][2];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int tap = 2 * ks + g / 2;
                w[ks][m] = tap < 7 ? *reinterpret_cast<const bf16x8 *>(
                                         nw.wm[0] + (tap * 32 + row_channel(m, l16)) * 16 + (g % 2) * 8)
                                   : bf16x8{};
            }
        float bb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) bb[j] = nw.bias[0][8 * g + j];
        store_rows(ICH);
        // this lane's tap of K step ks is 2 ks or 2 ks + 1; its cell in a staged row
        const bool second = g >= 2;
        int slot[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            slot[ks] = in_at(c + 1 + (second ? DQ[ks < 3 ? 2 * ks + 1 : 6] : DQ[2 * ks]), g % 2);
        // operands of step u, from staged input rows u, u + 1, u + 2
        bf16x8 v[4];
        auto operands = [&](int u) {
            int ro[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) ro[k] = (u + k) % IRING * (LW * 16);
            bool in = true;
            if constexpr (MASK) in = fl[(u + 1) % FRING][c + 1] != 0;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int ta = 2 * ks, tb = ks < 3 ? 2 * ks + 1 : 6;
                v[ks] = *reinterpret_cast<const bf16x8 *>(
                    &sin[0][0] + (second ? ro[1 + DR[tb]] : ro[1 + DR[ta]]) + slot[ks]);
                if constexpr (MASK) {
                    const int dr = second ? DR[tb] : DR[ta], dq = second ? DQ[tb] : DQ[ta];
                    const bool cut =
                        (ks > 0 || second) && !(in && fl[(u + 1 + dr) % FRING][c + 1 + dq]);
                    if (cut) v[ks] = bf16x8{};
                }
            }
        };
        __syncthreads();
        operands(0);
        for (int u = 0; u < steps; ++u) {
            if (u % ICH == 0) load_rows(u + 2 * ICH);
            // raster row R0 - 3 + u (the eighth tap does not exist: its weights are zero)
            f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
            const int r = R0 - 3 + u;
            const bool mine = KEEP && own_q && own_r(r);
            if (mine && !second)  // the cell itself: tap 0 of the first K step
                *reinterpret_cast<bf16x8 *>(keep.x0 + cell_at(r) * FEATURES_PAD + g * 8) = v[0];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 x8 = ks == 3 && second ? bf16x8{} : v[ks];
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][m], x8, acc[m], 0, 0, 0);
            }
            operands(u + 1);  // staged two rows ahead at least
            const bool ok = MASK || (qok && inside_r(r));
            const uint4 a = put_act(act[0][u & 1], c, g, acc, bb, ok);
            if (mine) *reinterpret_cast<uint4 *>(keep.act[0] + cell_at(r) * 32 + 8 * g) = a;
            if (u % ICH == ICH - 1) store_rows(u - (ICH - 1) + 2 * ICH);
            __syncthreads();
        }
    } else if (wave >= 8) {
        // ---- layer 3
        bf16x8 w[7];
#pragma unroll
        for (int t = 0; t < 7; ++t)
            w[t] = *reinterpret_cast<const bf16x8 *>(nw.wm[3] + (t * 16 + l16) * 32 + g * 8);
        float bb[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) bb[j] = nw.bias[3][4 * g + j];
        store_rows(0);
        Taps tp{};
        const bool qout = g == 0 && own_q;
        float *o = out + (soff + (int64_t)(R0 - 9) * nq + Q0 + c) * OUT_STRIDE;
        const int64_t pitch = (int64_t)nq * OUT_STRIDE;
        __syncthreads();
        for (int u0 = 0; u0 < steps; u0 += UN)
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int u = u0 + j;
                if (u >= steps) break;
                if (MASK) taps_move(tp);
                // raster row R0 - 9 + u; layer 2's row above it is the newest
                taps_push<MASK>(tp, j, act[2][(u + 1) & 1], c, g,
                                fl[MASK ? (u + FRING - 4) % FRING : 0]);
                __builtin_amdgcn_sched_barrier(0);  // the reads first: they wait longest
                f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int t = 0; t < 7; ++t)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t], tap_of<MASK>(tp, j, t), acc, 0, 0, 0);
                if (qout && u >= 9) {
                    if (w4) {
                        *reinterpret_cast<float4 *>(o) =
                            make_float4(acc[0] + bb[0], acc[1] + bb[1], acc[2] + bb[2], 0.f);
                    } else {
#pragma unroll
                        for (int k = 0; k < 3; ++k) o[k] = acc[k] + bb[k];
                    }
                }
                o += pitch;
                __syncthreads();
            }
    } else {
        // ---- layer 1 (waves 0 to 3) or 2
        const int l = 1 + (wave >> 2);
        __bf16 *const kept = KEEP ? (l == 1 ? keep.act[1] : keep.act[2]) : nullptr;
        bf16x8 w[7][2];
#pragma unroll
        for (int t = 0; t < 7; ++t)
#pragma unroll
            for (int m = 0; m < 2; ++m)
                w[t][m] = *reinterpret_cast<const bf16x8 *>(
                    nw.wm[l] + (t * 32 + row_channel(m, l16)) * 32 + g * 8);
        float bb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) bb[j] = nw.bias[l][8 * g + j];
        Taps tp{};
        __syncthreads();
        for (int u0 = 0; u0 < steps; u0 += UN)
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int u = u0 + j;
                if (u >= steps) break;
                if (MASK) taps_move(tp);
                // raster row R0 - 3 + u - 2 l; the row above it, of layer l - 1, is the newest
                taps_push<MASK>(tp, j, act[l - 1][(u + 1) & 1], c, g,
                                fl[MASK ? (u + FRING + 2 - 2 * l) % FRING : 0]);
                __builtin_amdgcn_sched_barrier(0);
                f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int t = 0; t < 7; ++t) {
                    const bf16x8 v = tap_of<MASK>(tp, j, t);
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][m], v, acc[m], 0, 0, 0);
                }
                const int r = R0 - 3 + u - 2 * l;
                const bool ok = MASK || (qok && inside_r(r));
                const uint4 a = put_act(act[l][u & 1], c, g, acc, bb, ok);
                if (KEEP && own_q && own_r(r))
                    *reinterpret_cast<uint4 *>(kept + cell_at(r) * 32 + 8 * g) = a;
                __syncthreads();
            }
    }
}

// ---------------------------------------------- the same network, tile by tile
//
// For many small samples, and narrow rasters with a domain mask, where a sweep's margins and
// start cost more than its rows: the whole network for a 16 x 16 tile of output cells in one
// workgroup of four waves, two on a CU.  The packed input of the tile and a 4-cell margin (24 x
// 24 positions) are staged once; layer l is evaluated on the tile grown by 3 - l cells on each
// side (46 % of the MFMA work is margin) and its activations stay in LDS for layer l + 1.  25 us
// for every 512 tiles, whatever they hold.  4096 samples of 16 x 16 cells: 245 us against 375 of
// the sweep and 304 of the layer chain; 512 masked ones 51 against 94 and 84; 8 masked ones of 3
// x 1000 51 against 83 and 73.
//
// Each layer's arithmetic is k_hexconv's, so the output equals the chain's bit for bit.  fl[p] is
// 1 where staged position p holds a cell of the domain (wrapped through periodic sides); a tap
// t >= 1 reads its neighbour only when the centre and the neighbour both are, which also zeroes
// every position outside the raster, as the chain's zero staging does.
namespace f4 {
constexpr int OT = 16;        // output tile edge
constexpr int WI = OT + 8;    // staged input frame edge (margin 4)
constexpr int NG = 4;         // 16-cell column groups per wave pass
}

// One layer over a WO x WO frame.  taps_all: every staged position of the tile is
// a domain cell (an interior tile of an unmasked raster), so no tap is cut.
// SSTR: 16-byte chunks between consecutive source cells; DSTR: bf16 values
// between consecutive destination cells (hidden activations are padded from 64
// to 80 bytes per cell, so that the 16 cells of an MFMA column fall on distinct
// LDS banks when gathered and when written).
template <int CIN, int COUT, int EPI, int WO, int SSTR, int DSTR>
__device__ inline void net_layer(const uint4 *src, uint4 *dst, const uint8_t *fl,
                                 const __bf16 *__restrict__ wm, const float *__restrict__ bias,
                                 float *__restrict__ out, int nq, int nr, int64_t soff, int q0,
                                 int r0, bool taps_all) {
    using namespace f4;
    constexpr int CH = CIN / 8;            // 16-byte chunks per source cell
    constexpr int MB = COUT / 16;
    constexpr int TPK = 32 / CIN;
    constexpr int KSTEPS = (7 + TPK - 1) / TPK;
    constexpr int WS = WO + 2;             // source frame edge
    constexpr int OI = (WI - WO) / 2;      // this frame's origin in the staged frame
    constexpr int NCELL = WO * WO;
    constexpr int NGRP = (NCELL + 15) / 16;
    constexpr int NCHUNK = (NGRP + NG - 1) / NG;
    constexpr int OFF_S[7] = {0, 1, WS, WS - 1, -1, -WS, -WS + 1};
    constexpr int OFF_I[7] = {0, 1, WI, WI - 1, -1, -WI, -WI + 1};
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int g = lane >> 4, l16 = lane & 15;
    // this lane's weight fragments for every K step, loaded once per layer
    bf16x8 av[KSTEPS][MB];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        const int tap = ks * TPK + g / CH;
        const int c0 = (g % CH) * 8;
#pragma unroll
        for (int m = 0; m < MB; ++m)
            av[ks][m] = tap < 7 ? *reinterpret_cast<const bf16x8 *>(
                                      wm + ((int64_t)(tap * COUT + m * 16 + l16)) * CIN + c0)
                                : bf16x8{};
    }
    for (int chunk = w; chunk < NCHUNK; chunk += 4) {
        f32x4 acc[MB][NG];
        int sslot[NG], islot[NG], cell[NG];
#pragma unroll
        for (int n = 0; n < NG; ++n) {
#pragma unroll
            for (int m = 0; m < MB; ++m) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
            int c = (chunk * NG + n) * 16 + l16;
            cell[n] = c;
            c = c < NCELL ? c : NCELL - 1;  // lanes past the frame compute a copy, never stored
            const int b = c / WO, a = c - b * WO;
            sslot[n] = (b + 1) * WS + (a + 1);
            islot[n] = (b + OI) * WI + (a + OI);
        }
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            const int tap = ks * TPK + g / CH;
            const int c0 = (g % CH) * 8;
#pragma unroll
            for (int n = 0; n < NG; ++n) {
                if ((chunk * NG + n) >= NGRP) break;  // uniform over the wave
                bf16x8 bv = bf16x8{};
                if (tap < 7) {
                    uint4 raw = src[(sslot[n] + OFF_S[tap]) * SSTR + c0 / 8];
                    if (!taps_all && tap > 0 && !(fl[islot[n]] & fl[islot[n] + OFF_I[tap]]))
                        raw = make_uint4(0u, 0u, 0u, 0u);
                    bv = *reinterpret_cast<const bf16x8 *>(&raw);
                }
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[ks][m], bv, acc[m][n], 0, 0, 0);
            }
        }
        // epilogue: lane holds channels co = m*16 + 4g + j of cell[n]
#pragma unroll
        for (int n = 0; n < NG; ++n) {
            const int c = cell[n];
            if ((chunk * NG + n) >= NGRP || c >= NCELL) continue;
            const int b = c / WO, a = c - b * WO;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const int co = m * 16 + 4 * g;
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = acc[m][n][j] + bias[co + j];
                if constexpr (EPI == EPI_LIN) {
                    const int q = q0 + a, r = r0 + b;
                    if (q < nq && r < nr) {
                        float *o = out + (soff + (int64_t)r * nq + q) * OUT_STRIDE;
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (co + j < 3) o[co + j] = v[j];
                    }
                } else {
                    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                    bf16x4 pk;
#pragma unroll
                    for (int j = 0; j < 4; ++j) pk[j] = (__bf16)(v[j] > 0.f ? v[j] : 0.f);
                    *reinterpret_cast<bf16x4 *>(reinterpret_cast<__bf16 *>(dst) + c * DSTR + co) = pk;
                }
            }
        }
    }
}

__global__ __launch_bounds__(NT) void k_hexnet4_tile(const __bf16 *__restrict__ x, Net4 nw,
                                                     float *__restrict__ out, int nq, int nr,
                                                     int ntiles_total, const int32_t *live,
                                                     ConvMask cm) {
    using namespace f4;
    constexpr int W0 = OT + 6, W1 = OT + 4;
    constexpr int AS = 5;  // 16-byte chunks per cell of hidden activations (32 channels + pad)
    __shared__ uint4 bufA[W0 * W0 * AS];  // layer 0 and layer 2 activations
    __shared__ uint4 bufB[W1 * W1 * AS];  // the staged input (16 channels), then layer 1
    __shared__ uint8_t fl[WI * WI];
    static_assert(WI * WI * 2 <= W1 * W1 * AS, "staged input fits the layer-1 buffer");
    const int ntq = (nq + OT - 1) / OT, ntr = (nr + OT - 1) / OT;
    const int tile = xcd_tile(blockIdx.x, gridDim.x, ntiles_total, 0);
    if (tile < 0) return;
    if (live && !*live) return;  // a surrogate window that does not run
    const int per = ntq * ntr;
    const int bs = tile / per, lt = tile - bs * per;
    const int tr = lt / ntq;
    const int q0 = (lt - tr * ntq) * OT, r0 = tr * OT;
    const int64_t soff = (int64_t)bs * nq * nr;
    // stage the 24 x 24 input frame: two 16-byte chunks per position, loads first
    constexpr int NE = WI * WI * 2;
    constexpr int ITERS = (NE + NT - 1) / NT;
    uint4 v[ITERS];
    uint8_t a[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int e = threadIdx.x + it * NT;
        const int p = e >> 1, ch = e & 1;
        const int pb = p / WI, pa = p - pb * WI;
        int q = q0 - 4 + pa, r = r0 - 4 + pb;
        if (cm.perq) q = ((q % nq) + nq) % nq;
        if (cm.perr) r = ((r % nr) + nr) % nr;
        v[it] = make_uint4(0u, 0u, 0u, 0u);
        a[it] = 0;
        if (e < NE && q >= 0 && q < nq && r >= 0 && r < nr) {
            const int64_t i = soff + (int64_t)r * nq + q;
            v[it] = reinterpret_cast<const uint4 *>(x + i * FEATURES_PAD)[ch];
            a[it] = cm.active ? (uint8_t)(cm.active[(int64_t)r * nq + q] != 0) : (uint8_t)1;
        }
    }
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int e = threadIdx.x + it * NT;
        if (e < NE) {
            bufB[e] = v[it];
            if ((e & 1) == 0) fl[e >> 1] = a[it];
        }
    }
    __syncthreads();
    // the staged frame lies inside an unmasked raster: no tap is cut
    const bool all = !cm.active && q0 >= 4 && q0 + OT + 4 <= nq && r0 >= 4 && r0 + OT + 4 <= nr;
    net_layer<16, 32, EPI_RELU, OT + 6, 2, 8 * AS>(bufB, bufA, fl, nw.wm[0], nw.bias[0], nullptr,
                                                   nq, nr, soff, q0, r0, all);
    __syncthreads();
    net_layer<32, 32, EPI_RELU, OT + 4, AS, 8 * AS>(bufA, bufB, fl, nw.wm[1], nw.bias[1], nullptr,
                                                    nq, nr, soff, q0, r0, all);
    __syncthreads();
    net_layer<32, 32, EPI_RELU, OT + 2, AS, 8 * AS>(bufB, bufA, fl, nw.wm[2], nw.bias[2], nullptr,
                                                    nq, nr, soff, q0, r0, all);
    __syncthreads();
    net_layer<32, 16, EPI_LIN, OT, AS, 0>(bufA, nullptr, fl, nw.wm[3], nw.bias[3], out, nq, nr,
                                          soff, q0, r0, all);
}

// ------------------------------------------------------------ weight grad

// A 16-channel column of 8 consecutive cells: the transposing LDS read returns, to
// lane i of each group of 16, column i of the 4 x 16 block whose rows the group's
// lanes address (lane i: row i / 4, columns 4 (i % 4)...), so two reads give the 8
// cells of an MFMA operand whose K runs over cells from channels-last data.
__device__ inline bf16x8 read_cells8(const __bf16 *p, int cell_stride) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
    union {
        s16x4 h[2];
        bf16x8 v;
    } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * cell_stride));
    return u.v;
}

// Partial dW[t][co][ci] = sum_cells dy[cell][co] x[nbr_t(cell)][ci] and
// db[co] = sum_cells dy[cell][co], in FP32, of the tiles this workgroup sweeps.
// A = dy^T (16 channels x 32 cells), B = x_t (32 cells x 16 channels); wave w takes
// row w of each 64 x 4 tile for all seven taps, so a dy operand serves all of them,
// and keeps the sums in registers over its tiles.
//
// Bound by the reads of x and dy (cache resident at the usual mini-batches) and by
// the records the reduction has to read back: one per workgroup, at most WGRAD_WGS,
// instead of one per tile.  Operands come from channels-last LDS rows through
// transposing reads (8 two-byte gathers per operand before); rows are padded by 16
// bytes per cell against bank conflicts.  The next tile's loads are in flight during
// the arithmetic.  2 x 512 x 512 samples, 32 -> 32 channels: 27 us against 48 us.
//
// DX (every layer but the first): the data gradient too, dx = (W^T stencil of dy) where
// x > 0, from the same staged tiles: dy is staged with its halo, x's own cells are the ReLU's
// mask.  Four more waves do it, one row each, with conv_acc's MFMAs in its order, so a SIMD
// holds one wave of each gradient and one workgroup fills a CU (half the records).  As a
// launch of its own it read dy and x again: 39 us against 50 for 32 -> 32 channels, 33
// against 39 for the last layer, and the reduction 9.5 against 14.7.  One set of four waves
// that did both spilled 184 registers (128 us).
template <bool DX>
constexpr int WG_NT = DX ? 512 : 256;
template <int CIN, int COUT, bool DX>
__global__ __launch_bounds__(WG_NT<DX>, 2) void k_hexconv_wgrad(const __bf16 *__restrict__ x,
                                                         const __bf16 *__restrict__ dy,
                                                         float *__restrict__ part,
                                                         const __bf16 *__restrict__ wt,
                                                         __bf16 *__restrict__ dx, int nq, int nr,
                                                         int ntiles_total, ConvMask cm) {
    constexpr int NTH = WG_NT<DX>;
    constexpr int CH = CIN / 8, DCH = COUT / 8;
    constexpr int MB = COUT / 16, NB = CIN / 16;
    constexpr int PSZ = 7 * COUT * CIN + COUT;
    constexpr int XS = CIN + 8, DS = COUT + 8;  // padded bf16 per staged cell
    constexpr int DN = DX ? NSLOT : TQ * TR;    // staged cells of dy
    constexpr int XB = NSLOT * XS * 2, DB = DN * DS * 2;
    constexpr int BYTES = XB + DB > PSZ * 4 ? XB + DB : PSZ * 4;
    __shared__ __align__(16) unsigned char smem[BYTES];
    __shared__ uint8_t fl[NSLOT];
    __bf16 *sx = reinterpret_cast<__bf16 *>(smem);
    __bf16 *sdy = reinterpret_cast<__bf16 *>(smem + XB);
    float *red = reinterpret_cast<float *>(smem);  // the waves' sums, after the last tile
    const int ntq = (nq + TQ - 1) / TQ, ntr = (nr + TR - 1) / TR;
    const bool masked = cm.active != nullptr;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, l16 = lane & 15;
    const int w = wave & 3;  // row of the tile

    constexpr int XIT = (NSLOT * CH + NTH - 1) / NTH, DIT = (DN * DCH + NTH - 1) / NTH;
    uint4 xv[XIT], dv[DIT];
    uint8_t av[XIT];
    auto load = [&](int tile) {
        int b, q0, r0;
        tile_of(tile, ntq, ntr, b, q0, r0);
        const int64_t soff = (int64_t)b * nq * nr;
#pragma unroll
        for (int it = 0; it < XIT; ++it) {
            const int e = threadIdx.x + it * NTH;
            const int s = e / CH, ch = e - s * CH;
            const int lr = s / SW, lq = s - lr * SW;
            int q = q0 + lq - 1, r = r0 + lr - 1;
            if (cm.perq) q = q < 0 ? q + nq : (q >= nq ? q - nq : q);
            if (cm.perr) r = r < 0 ? r + nr : (r >= nr ? r - nr : r);
            xv[it] = make_uint4(0u, 0u, 0u, 0u);
            av[it] = 0;
            if (e < NSLOT * CH && q >= 0 && q < nq && r >= 0 && r < nr) {
                xv[it] = reinterpret_cast<const uint4 *>(x + (soff + (int64_t)r * nq + q) * CIN)[ch];
                if (masked && ch == 0) av[it] = cm.active[(int64_t)r * nq + q] != 0;
            }
        }
#pragma unroll
        for (int it = 0; it < DIT; ++it) {  // dy of the tile's cells, zero outside the raster
            const int e = threadIdx.x + it * NTH;
            const int c = e / DCH, ch = e - c * DCH;
            int q, r;
            if constexpr (DX) {
                q = q0 + c % SW - 1;
                r = r0 + c / SW - 1;
                if (cm.perq) q = q < 0 ? q + nq : (q >= nq ? q - nq : q);
                if (cm.perr) r = r < 0 ? r + nr : (r >= nr ? r - nr : r);
            } else {
                q = q0 + c % TQ;
                r = r0 + c / TQ;
            }
            dv[it] = make_uint4(0u, 0u, 0u, 0u);
            if (e < DN * DCH && q >= 0 && q < nq && r >= 0 && r < nr)
                dv[it] = reinterpret_cast<const uint4 *>(dy + (soff + (int64_t)r * nq + q) * COUT)[ch];
        }
    };

    auto stage = [&]() {
#pragma unroll
        for (int it = 0; it < XIT; ++it) {
            const int e = threadIdx.x + it * NTH;
            if (e < NSLOT * CH) {
                const int s = e / CH, ch = e - s * CH;
                *reinterpret_cast<uint4 *>(sx + s * XS + ch * 8) = xv[it];
                if (masked && ch == 0) fl[s] = av[it];
            }
        }
#pragma unroll
        for (int it = 0; it < DIT; ++it) {
            const int e = threadIdx.x + it * NTH;
            if (e < DN * DCH) {
                const int c = e / DCH, ch = e - c * DCH;
                *reinterpret_cast<uint4 *>(sdy + c * DS + ch * 8) = dv[it];
            }
        }
    };
    // the tiles in turn, the next one's loads in flight: wait until the last one's operands
    // have been read, stage, then do(tile's place)
    auto sweep = [&](auto &&work) {
        int tile = xcd_tile(blockIdx.x, gridDim.x, ntiles_total, 0);
        if (tile >= 0) load(tile);
        for (int k = 0; tile >= 0; ++k) {
            __syncthreads();
            stage();
            int b, q0, r0;
            tile_of(tile, ntq, ntr, b, q0, r0);
            tile = xcd_tile(blockIdx.x, gridDim.x, ntiles_total, k + 1);
            if (tile >= 0) load(tile);
            __syncthreads();
            work(b, q0, r0);
        }
    };

    if (DX && wave >= 4) {
        // ---- data gradient, as conv_acc does it, over dy with the transposed stencil
        sweep([&](int b, int q0, int r0) {
            constexpr int TPK = 32 / COUT, KSTEPS = (7 + TPK - 1) / TPK;
            const int64_t soff = (int64_t)b * nq * nr;
            f32x4 da[NB][4];
#pragma unroll
            for (int m = 0; m < NB; ++m)
#pragma unroll
                for (int n = 0; n < 4; ++n) da[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                const int tap = ks * TPK + g / DCH, c0 = (g % DCH) * 8;
                bf16x8 a[NB];
#pragma unroll
                for (int m = 0; m < NB; ++m)
                    a[m] = tap < 7 ? *reinterpret_cast<const bf16x8 *>(
                                         wt + (tap * CIN + m * 16 + l16) * COUT + c0)
                                   : bf16x8{};
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    const int s = (w + 1) * SW + n * 16 + l16 + 1;
                    bf16x8 bv = bf16x8{};
                    if (tap < 7) {
                        bv = *reinterpret_cast<const bf16x8 *>(sdy + (s + OFFS[tap]) * DS + c0);
                        if (masked && tap > 0 && !(fl[s] & fl[s + OFFS[tap]])) bv = bf16x8{};
                    }
#pragma unroll
                    for (int m = 0; m < NB; ++m)
                        da[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], bv, da[m][n], 0, 0, 0);
                }
            }
            const int r = r0 + w;
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const int q = q0 + n * 16 + l16, s = (w + 1) * SW + n * 16 + l16 + 1;
                if (q >= nq || r >= nr) continue;
#pragma unroll
                for (int m = 0; m < NB; ++m) {
                    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                    const int co = m * 16 + 4 * g;
                    const bf16x4 own = *reinterpret_cast<const bf16x4 *>(sx + s * XS + co);
                    bf16x4 pk;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        pk[j] = (float)own[j] > 0.f ? (__bf16)da[m][n][j] : (__bf16)0.f;
                    *reinterpret_cast<bf16x4 *>(dx + (soff + (int64_t)r * nq + q) * CIN + co) = pk;
                }
            }
        });
        for (int v = 0; v < 4; ++v) __syncthreads();  // the other waves' reduction
    } else {
        // ---- weight gradient
        f32x4 acc[7][MB][NB], accb[MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            accb[m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 7; ++t)
#pragma unroll
                for (int n = 0; n < NB; ++n) acc[t][m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        bf16x8 ones;
#pragma unroll
        for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.f;

        sweep([&](int, int q0, int r0) {
            // dy staged with periodic wraps: positions of the tile past the raster's end hold
            // other cells', which the weights must not see
            const bool cut = DX && (cm.perq || cm.perr) && (q0 + TQ > nq || r0 + TR > nr);
#pragma unroll
            for (int ks = 0; ks < TQ / 32; ++ks) {
                const int c0 = ks * 32 + 8 * g;                 // first of this lane's 8 cells
                const int sc = (w + 1) * SW + (c0 + 1);         // its staged slot
                const int row = l16 >> 2, col = (l16 & 3) * 4;  // what this lane addresses
                bf16x8 a[MB];
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    a[m] = read_cells8(sdy + ((DX ? sc : w * TQ + c0) + row) * DS + m * 16 + col, DS);
                if (cut) {
#pragma unroll
                    for (int m = 0; m < MB; ++m)
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (q0 + c0 + j >= nq || r0 + w >= nr) a[m][j] = (__bf16)0.f;
                }
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], ones, accb[m], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < 7; ++t) {
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        bf16x8 bv = read_cells8(sx + (sc + OFFS[t] + row) * XS + n * 16 + col, XS);
                        if (masked && t > 0) {
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                if (!(fl[sc + j] & fl[sc + OFFS[t] + j])) bv[j] = (__bf16)0.f;
                        }
#pragma unroll
                        for (int m = 0; m < MB; ++m)
                            acc[t][m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], bv, acc[t][m][n], 0, 0, 0);
                    }
                }
            }
        });
        // the four waves' sums in wave order: a lane holds dW rows co = m*16 + 4g + j,
        // column ci = n*16 + l16
        for (int v = 0; v < 4; ++v) {
            __syncthreads();
            if (w != v) continue;
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int co = m * 16 + 4 * g + j;
#pragma unroll
                    for (int t = 0; t < 7; ++t)
#pragma unroll
                        for (int n = 0; n < NB; ++n) {
                            float *o = red + (t * COUT + co) * CIN + n * 16 + l16;
                            *o = v == 0 ? acc[t][m][n][j] : *o + acc[t][m][n][j];
                        }
                    if (l16 == 0) {
                        float *o = red + 7 * COUT * CIN + co;
                        *o = v == 0 ? accb[m][j] : *o + accb[m][j];
                    }
                }
        }
    }
    __syncthreads();
    float *P = part + (int64_t)blockIdx.x * PSZ;
    for (int e = threadIdx.x; e < PSZ; e += NTH) P[e] = red[e];
}

// Sum the workgroups' partials of every layer in a fixed order (deterministic) and
// scatter them into the flat parameter-gradient layout W[o][c][t] (o < cout, c < cin),
// b[o].  16 threads share an element, each adding every 16th record with eight loads
// in flight, then a tree over the 16: one launch for all layers, 15 us at 512
// records of 4 layers (10 with half the records of three), where one thread per element
// over 2048 records took 635 us a layer (its loads one behind the other).
constexpr int RED_GRP = 16, RED_EL = 256 / RED_GRP;
__global__ __launch_bounds__(256) void k_wgrad_reduce(WgradTable tab,
                                                      float *__restrict__ grad) {
    int l = 0;
    while (l + 1 < tab.layers && (int)blockIdx.x >= tab.y[l + 1].block0) ++l;
    const WgradLayer y = tab.y[l];
    const int psz = 7 * y.coutp * y.cinp + y.coutp, nrec = y.nrec;
    const int el = threadIdx.x % RED_EL, grp = threadIdx.x / RED_EL;
    const int src = ((int)blockIdx.x - y.block0) * RED_EL + el;
    float s = 0.f;
    if (src < psz) {
        const float *p = y.part + src;
        for (int k = grp; k < nrec; k += RED_GRP * 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int r = k + u * RED_GRP;
                v[u] = r < nrec ? p[(int64_t)r * psz] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    }
    __shared__ float red[RED_GRP][RED_EL];
    red[grp][el] = s;
    __syncthreads();
    if (grp != 0 || src >= psz) return;
#pragma unroll
    for (int o = RED_GRP / 2; o > 0; o >>= 1)
#pragma unroll
        for (int k = 0; k < o; ++k) red[k][el] += red[k + o][el];
    const float tot = red[0][el];
    if (src >= 7 * y.coutp * y.cinp) {
        const int o = src - 7 * y.coutp * y.cinp;
        if (o < y.cout) grad[y.off + (int64_t)y.cout * y.cin * 7 + o] = tot;
        return;
    }
    const int t = src / (y.coutp * y.cinp), rem = src - t * y.coutp * y.cinp;
    const int o = rem / y.cinp, c = rem - o * y.cinp;
    if (o < y.cout && c < y.cin) grad[y.off + ((int64_t)o * y.cin + c) * 7 + t] = tot;
}

// ------------------------------------------------------------ parameters

// From the flat FP32 parameters of one layer (W[o][c][t], b[o]) build the
// bf16 MFMA weights: forward wm[t][co][ci] = W[co][ci][t]; data gradient
// wt[t][ci][co] = W[co][ci][opp(t)] (the transposed, mirrored stencil).
// Padded channels are zero.
__global__ void k_prepare_weights(const float *__restrict__ p, int cin, int cout, int cinp,
                                  int coutp, __bf16 *__restrict__ wm, __bf16 *__restrict__ wt,
                                  float *__restrict__ bias) {
    const int n = 7 * coutp * cinp;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const int t = e / (coutp * cinp), rem = e - t * coutp * cinp;
        const int co = rem / cinp, ci = rem - co * cinp;
        const float v = (co < cout && ci < cin) ? p[(co * cin + ci) * 7 + t] : 0.f;
        wm[e] = (__bf16)v;
        // wt is [t][ci][co] with cinp/coutp swapped roles
        const float vt = (co < cout && ci < cin) ? p[(co * cin + ci) * 7 + OPP[t]] : 0.f;
        wt[(t * cinp + ci) * coutp + co] = (__bf16)vt;
    }
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < coutp; e += gridDim.x * blockDim.x)
        bias[e] = e < cout ? p[cout * cin * 7 + e] : 0.f;
}

__global__ void k_adam(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

// ------------------------------------------------------------ loss, pack

// L1 loss of pred (OUT_STRIDE floats per cell, 3 used) against target (3 per
// cell): per-workgroup FP64 partial sums and dy = sign(diff)/count as bf16
// in the 16-channel layout of the last layer.
__global__ __launch_bounds__(256) void k_l1_loss(const float *__restrict__ pred,
                                                 const float *__restrict__ target, int64_t ncell,
                                                 double inv_count, __bf16 *__restrict__ dy,
                                                 double *__restrict__ part) {
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ncell;
         i += (int64_t)gridDim.x * blockDim.x) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        bf16x4 d0 = bf16x4{}, d1 = bf16x4{}, d2 = bf16x4{}, d3 = bf16x4{};
        for (int c = 0; c < 3; ++c) {
            const float df = pred[i * OUT_STRIDE + c] - target[i * 3 + c];
            s += fabs((double)df);
            const float gs = df > 0.f ? (float)inv_count : (df < 0.f ? -(float)inv_count : 0.f);
            d0[c] = (__bf16)gs;
        }
        bf16x4 *o = reinterpret_cast<bf16x4 *>(dy + i * 16);
        o[0] = d0;
        o[1] = d1;
        o[2] = d2;
        o[3] = d3;
    }
    __shared__ double red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// FP32 features -> the packed bf16 input (FEATURES_PAD channels, the last ones zero).
__global__ void k_pack_features(const float *__restrict__ f, int64_t ncell,
                                __bf16 *__restrict__ x) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ncell;
         i += (int64_t)gridDim.x * blockDim.x) {
        bf16x8 v[FEATURES_PAD / 8];
#pragma unroll
        for (int c = 0; c < FEATURES_PAD; ++c)
            v[c / 8][c % 8] = c < FEATURES ? (__bf16)f[i * FEATURES + c] : (__bf16)0.f;
#pragma unroll
        for (int u = 0; u < FEATURES_PAD / 8; ++u)
            reinterpret_cast<bf16x8 *>(x + i * FEATURES_PAD)[u] = v[u];
    }
}

// ------------------------------------------------------------- launchers

static int blocks_for(int64_t n, int per = 256) {
    const int64_t b = (n + per - 1) / per;
    return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

int conv_tiles(int nq, int nr, int batch) {
    return ((nq + TQ - 1) / TQ) * ((nr + TR - 1) / TR) * batch;
}

hipError_t launch_conv(int cinp, int coutp, int epi, const __bf16 *x, const __bf16 *wm,
                       const float *bias, void *out, int nq, int nr, int batch, int cout_real,
                       const ConvMask &cm, hipStream_t st, const int32_t *live) {
    const int nt = conv_tiles(nq, nr, batch);
#define HEXSV_CONV(CI, CO, E)                                                                   \
    if (cinp == CI && coutp == CO && epi == E) {                                                \
        hipLaunchKernelGGL((k_hexconv<CI, CO, E>), dim3(nt), dim3(NT), 0, st, x, wm, bias, out, \
                           nq, nr, nt, cout_real, live, cm);                                    \
        return hipGetLastError();                                                               \
    }
    HEXSV_CONV(16, 32, EPI_RELU)
    HEXSV_CONV(32, 32, EPI_RELU)
    HEXSV_CONV(32, 16, EPI_LIN)
#undef HEXSV_CONV
    return hipErrorInvalidValue;
}

// Segments of the rows: the split that costs the fewest rounds of steps, with one
// workgroup per CU at a time and a strip's start (weights, first input rows) as six steps.
static int net4_segments(int nq, int nr, int batch) {
    const int64_t strips = (int64_t)((nq + r4::OW - 1) / r4::OW) * batch;
    int best = 1;
    int64_t cost = INT64_MAX;
    const int64_t least = (strips + 255) / 256;
    for (int64_t rounds = least; rounds < least + 12; ++rounds) {
        const int64_t most = rounds * 256 / strips;  // segments that these rounds hold
        const int s = (int)(most < nr ? most : nr);
        const int rh = (nr + s - 1) / s;
        const int64_t c = rounds * (rh + r4::EXTRA + 6);
        if (c < cost) {
            cost = c;
            best = (nr + rh - 1) / rh;
        }
    }
    return best;
}

// The fastest way through the network for these samples: the layer chain, the sweep or the
// tiles.  Estimates in us, from all three measured over 1 to 20000 samples of 1 x 1 to 1000 x
// 1000 cells: the sweep by its rounds of steps (it recomputes nine rows of a segment and six
// columns of a strip, and fills a CU with one strip of one sample), dearer with a domain mask;
// the chain by its tiles beyond those of one round and by its cells; the tiles by rounds of 512.
// The pick was within 8 % of the best of the three everywhere.  Sweep / chain / tiles: forward
// 16 x 512 x 512 273 / 609 / 868, 512 x 8 x 8 53 / 49 / 49, 512 x 16 x 16 65 / 73 / 51, 4096 x 8
// x 8 286 / 166 / 227; masked 64 x 64 x 64 90 / 76 / 82, 64 x 58 x 58 63 / 71 / 73.  In a window
// the chain's last layer forms the predicted state as well, worth 6 us (masked 512 x 512 84 / 73
// us a window, 2048 x 1024 373 / 453).  A gradient's forward keeps its activations: no tiles,
// and with a mask no sweep (1 x 512 x 512 275 / 255, no size measured where it was faster).
Net4Route net4_route(int nq, int nr, int batch, bool masked, Net4Use use, bool chain_too) {
    const double cells = (double)batch * nq * nr;
    const double never = 1e30;
    const int64_t count = (int64_t)((nq + f4::OT - 1LL) / f4::OT) * ((nr + f4::OT - 1LL) / f4::OT) * batch;
    double tiles = 21.0 + (masked ? 1 : 0) + 25.0 * (double)((count + 511) / 512) + 2e-5 * cells;
    if (use == NET4_KEEP || count > 1 << 23) tiles = never;  // (a launch holds 2^32 threads)
    double sweep = never;
    if (nq <= 1 << 26 && !(masked && use == NET4_KEEP)) {
        const int64_t strips = (int64_t)((nq + r4::OW - 1) / r4::OW) * batch;
        const int nseg = net4_segments(nq, nr, batch), rh = (nr + nseg - 1) / nseg;
        const double rounds = (double)((strips * nseg + 255) / 256);
        sweep = masked ? 20 + 1.3 * rounds * (rh + 11) + 4.8e-5 * cells
                       : 18 + 0.72 * rounds * (rh + 15) + 1e-5 * cells;
    }
    const double more = fmax(0.0, (double)((nq + TQ - 1LL) / TQ) * (double)((nr + TR - 1LL) / TR) * batch - 512);
    double chain = masked ? 42 + 0.0177 * more + 1e-4 * cells : 38 + 0.0133 * more + 9e-5 * cells;
    if (use == NET4_WINDOW) chain -= 6;
    if (!chain_too && fmin(sweep, tiles) < never) chain = never;
    if (chain < sweep && chain < tiles) return NET4_CHAIN;
    return sweep <= tiles ? NET4_SWEEP : NET4_TILES;
}

hipError_t launch_net4_tiles(const __bf16 *x, const Net4 &nw, float *out, int nq, int nr, int batch,
                             const ConvMask &cm, hipStream_t st, const int32_t *live) {
    const int64_t nt = (int64_t)((nq + f4::OT - 1LL) / f4::OT) * ((nr + f4::OT - 1LL) / f4::OT) * batch;
    if (nt > 1 << 23) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_hexnet4_tile, dim3((unsigned)nt), dim3(NT), 0, st, x, nw, out, nq, nr, (int)nt,
                       live, cm);
    return hipGetLastError();
}

hipError_t launch_net4(const void *x, bool f32in, const Net4 &nw, float *out, bool w4, int nq,
                       int nr, int batch, const ConvMask &cm, hipStream_t st,
                       const int32_t *live, const Net4Keep *keep) {
    // a launch holds fewer than 2^32 threads: many small samples go in several
    const int64_t strips = (nq + r4::OW - 1) / r4::OW;
    const int64_t most = (int64_t(1) << 21) / strips;
    if (most < 1) return hipErrorInvalidValue;
    if (batch > most) {
        const int64_t cells = (int64_t)nq * nr, step = cells * (f32in ? FEATURES * 4 : 32);
        for (int64_t b = 0; b < batch; b += most) {
            const int n = (int)(batch - b < most ? batch - b : most);
            Net4Keep k = keep ? *keep : Net4Keep{};
            if (keep) {
                k.x0 += b * cells * FEATURES_PAD;
                for (int l = 0; l < 3; ++l) k.act[l] += b * cells * 32;
            }
            const hipError_t err = launch_net4((const char *)x + b * step, f32in, nw,
                                               out + b * cells * OUT_STRIDE, w4, nq, nr, n, cm, st,
                                               live, keep ? &k : nullptr);
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }
    const int nseg = net4_segments(nq, nr, batch), rh = (nr + nseg - 1) / nseg;
    const int64_t wgs = strips * nseg * batch;
    if (keep && (!f32in || cm.active)) return hipErrorInvalidValue;
#define HEXSV_NET4(M, F, K)                                                                    \
    hipLaunchKernelGGL((k_hexnet4<M, F, K>), dim3((unsigned)wgs), dim3(r4::NTH), 0, st, x, nw,  \
                       out, nq, nr, batch, rh, nseg, w4 ? 1 : 0, live, cm,                      \
                       keep ? *keep : Net4Keep{})
    if (cm.active) {
        if (f32in) HEXSV_NET4(true, true, false);
        else HEXSV_NET4(true, false, false);
    } else {
        if (keep) HEXSV_NET4(false, true, true);
        else if (f32in) HEXSV_NET4(false, true, false);
        else HEXSV_NET4(false, false, false);
    }
#undef HEXSV_NET4
    return hipGetLastError();
}

int wgrad_records(int nq, int nr, int batch, bool dx) {
    const int nt = conv_tiles(nq, nr, batch), most = dx ? WGRAD_WGS / 2 : WGRAD_WGS;
    return nt < most ? nt : most;
}

hipError_t launch_wgrad(int cinp, int coutp, const __bf16 *x, const __bf16 *dy, float *part,
                        const __bf16 *wt, __bf16 *dx, int nq, int nr, int batch,
                        const ConvMask &cm, hipStream_t st) {
    if ((cinp == 32) != (dx != nullptr)) return hipErrorInvalidValue;
    const int nt = conv_tiles(nq, nr, batch), nwg = wgrad_records(nq, nr, batch, dx != nullptr);
#define HEXSV_WG(CI, CO)                                                                       \
    if (cinp == CI && coutp == CO) {                                                           \
        hipLaunchKernelGGL((k_hexconv_wgrad<CI, CO, CI == 32>), dim3(nwg), dim3(WG_NT<CI == 32>), 0, \
                           st, x, dy, part, wt, dx, nq, nr, nt, cm);                                   \
        return hipGetLastError();                                                              \
    }
    HEXSV_WG(16, 32)
    HEXSV_WG(32, 32)
    HEXSV_WG(32, 16)
#undef HEXSV_WG
    return hipErrorInvalidValue;
}

hipError_t launch_wgrad_reduce(WgradTable tab, float *grad, hipStream_t st) {
    int blocks = 0;
    for (int l = 0; l < tab.layers; ++l) {
        tab.y[l].block0 = blocks;
        blocks += (7 * tab.y[l].coutp * tab.y[l].cinp + tab.y[l].coutp + RED_EL - 1) / RED_EL;
    }
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks), dim3(256), 0, st, tab, grad);
    return hipGetLastError();
}

hipError_t launch_prepare_weights(const float *p, int cin, int cout, int cinp, int coutp,
                                  __bf16 *wm, __bf16 *wt, float *bias, hipStream_t st) {
    hipLaunchKernelGGL(k_prepare_weights, dim3(blocks_for(7 * cinp * coutp)), dim3(256), 0, st, p,
                       cin, cout, cinp, coutp, wm, wt, bias);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, float *m, float *v, const float *g, int64_t n, float lr,
                       int step, hipStream_t st) {
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(256), 0, st, p, m, v, g, n, lr, b1, b2,
                       1e-8f, c1, c2);
    return hipGetLastError();
}

hipError_t launch_l1_loss(const float *pred, const float *target, int64_t ncell, double inv_count,
                          __bf16 *dy, double *part, int nparts, hipStream_t st) {
    hipLaunchKernelGGL(k_l1_loss, dim3(nparts), dim3(256), 0, st, pred, target, ncell, inv_count,
                       dy, part);
    return hipGetLastError();
}

hipError_t launch_pack_features(const float *f, int64_t ncell, __bf16 *x, hipStream_t st) {
    hipLaunchKernelGGL(k_pack_features, dim3(blocks_for(ncell)), dim3(256), 0, st, f, ncell, x);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace hexsv
