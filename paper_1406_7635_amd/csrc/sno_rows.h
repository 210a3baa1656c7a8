// sno_rows.h -- device passes of the spectral neural operator that work on
// whole grid rows, shared by inference (kernels_sno.hip, BF16 weights) and
// training (kernels_sno_train.hip, FP32 weights, a batch of samples).
//
// Per row (sample b, row y) all the work along x is small matrix products over
// tiles of 32 pixels, done on the matrix cores in FP32
// (v_mfma_f32_32x32x2_f32: operands and accumulators FP32):
//   pointwise part   z[o][x] = sum_c W[o][c] h[c][x] + b[o]
//                              + sum_k g[o][k] E[k][x]      K = 32 + 1 + 32
//   kept modes       line[k][o] = sum_x E[k][x] h'[o][x]    K = pixels
//   weight gradient  dW[o][c] = sum_x dz[o][x] h[c][x]      K = pixels
// with E[2 kx + {0, 1}][x] the real and imaginary part of
// exp(-2 pi i kx x / nx) and g[o][2 kx + {0, 1}] those of the row's inverse y
// transform, formed at the start of the row from the mixed modes.
//
// What bounds it, and why this split: one pass per layer reads and writes each
// activation once (forward: h in, h' and GELU' out; backward: dz, GELU', h in,
// the next dz out), so the training passes are bound by those bytes.  With a
// kernel per product (x transform, GELU backward with its weight sums on the
// vector units, pointwise part) every activation was read two or three times
// and the sums over pixels took 0.83 ms a layer.  256 x 256, batch 16: loss and
// gradient 7.4 -> 1.55 ms; one 256 x 256 prediction 244 -> 90 us.
//
// Operand layout of the instruction (wave of 64, h = lane / 32, l = lane % 32):
// A[m = l][k = h], B[k = h][n = l], result register i = D[m = drow(i, h)][n = l].
// The pointwise product has x along the lanes, so rows are loaded and stored
// coalesced; a product over pixels needs the channel along the lanes, so a tile
// is turned through LDS (pitch 33: no two lanes of a half share a bank), and
// then both halves' registers i are the pixels drow(i, h): no further shuffle.
#pragma once

#include <hip/hip_runtime.h>

#include "sno_internal.h"

namespace mm {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ inline f32x16 mfma32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ inline f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}
// result row of register i in lane half h
__device__ constexpr int drow(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

__device__ inline float wval(float w) { return w; }
__device__ inline float wval(uint16_t w) { return __uint_as_float((unsigned int)w << 16); }  // BF16

// Loads and stores of a row's channels through a raw buffer resource: uniform
// base, a 32-bit byte offset per lane, and the channel's offset in a scalar
// register (one address register for all sixteen channels of a lane; one
// sample's channels stay below 32 x 512 x 512 x 4 bytes).
__device__ inline __amdgpu_buffer_rsrc_t row_buffer(const float* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, (int)0xffffffffu, 0x00020000);
}
__device__ inline float ldr(__amdgpu_buffer_rsrc_t r, int lane_off, int chan_off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_off, chan_off, 0));
}
__device__ inline void str(__amdgpu_buffer_rsrc_t r, int lane_off, int chan_off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, lane_off, chan_off, 0);
}

constexpr int NMODE = SNO_KY * SNO_KX;      // kept modes
constexpr int ROW_WAVES = 8;                // waves of a row-pass workgroup
constexpr int ROW_NTH = 64 * ROW_WAVES;
constexpr int TPITCH = 33;                  // LDS pitch of 32-wide tiles
constexpr int GPITCH = 36;                  // LDS pitch of the g rows (16-byte aligned)
constexpr int KLAYER = SNO_C * SNO_C + SNO_C;   // dW, db
constexpr int KPROJ = 3 * SNO_C + 3;            // dQ, dq
constexpr int KLIFT = 3 * SNO_C + SNO_C;        // dP, dp
// Pixels of an FP32 weight sum before it goes to FP64 (a wave takes up to 64 of
// a row).  Equal terms, where the rounding adds up, 512 x 512, batch 128 (8192
// pixels a wave): 1.2e-4 of a component in one FP32 chain, 7e-6 in these; 256 x
// 256, batch 16 (256 pixels a wave, one flush): 1548 us before, 1557 us.
constexpr int SUM_PIXELS = 256;

// The passes.  ROW_LIFT: h0 = P m + p.  ROW_LAYER: one layer, h' = GELU(z).
// ROW_OUT: the last layer with the projection y = scale (Q h' + q).
// ROW_BOUT: dh = Q^T dy, dy = s_b (y - t), then the last layer's dz = dh GELU',
// its dW, db, and dQ, dq.  ROW_BLAYER: dh = W^T dz + inverse of the modes, then
// dz, dW, db of the layer below.  ROW_BLIFT: the same dh, then dP, dp.
enum RowMode { ROW_LIFT, ROW_LAYER, ROW_OUT, ROW_BOUT, ROW_BLAYER, ROW_BLIFT };

template <class WT>
struct RowArgs {
    int nx, ny, n, rows;          // rows = batch ny
    int wshift;                   // log2 of the waves that share a row
    const float* src;             // h (forward) or dz (backward) [b][32][n]; ROW_LIFT: m [b][3][n]
    float* dst;                   // h' or the next dz [b][32][n] (null: not kept)
    float* gd;                    // GELU' of this layer, written (forward, null: not kept)
    const float* gd_in;           // GELU' of the layer whose dz is formed
    const float* hprev;           // input of the layer whose dW is formed [b][32][n]; ROW_BLIFT: m
    const float2* modes;          // mixed modes of this row pass's inverse transform [b][32][256]
    float* line;                  // kept modes along x of the result [b][y][32][32] (re, im interleaved)
    const float4* ex;             // E[x][k], x < nx rounded up to 32 (k_sno_ex)
    const float2* twy;            // exp(-2 pi i m / ny)
    const WT* w;                  // W [32][32] or P [32][3]
    const WT* wb;                 // b or p [32]
    const WT* q;                  // Q [3][32]
    const WT* qb;                 // q [3]
    float out_scale;
    float* y;                     // prediction [b][3][n] (written by ROW_OUT, read by ROW_BOUT)
    const float* t;               // target
    const float* sb;              // per-sample loss scale
    double* part;                 // weight sums of the workgroup [gridDim.x][K]
};

// Waves that share a row: a wave per 32-pixel tile, up to the workgroup's 8, and
// more (some then without a tile) where the rows would not give each of the 256 CUs
// a workgroup: the rows of a workgroup form their g one after the other.  One
// prediction with a wave per tile and with this rule: 32 x 16 157, 69 us; 64 x 64 113,
// 70 us; 64 x 512 134, 108 us.
inline int row_wave_shift(int nx, long long rows) {
    const int tiles = (nx + 31) / 32;
    int s = 0;
    while ((1 << s) < tiles && s < 3) ++s;
    while (s < 3 && rows < 256LL * (ROW_WAVES >> s)) ++s;
    return s;
}
inline size_t row_lds(int nx, int wshift) {
    const int nxp = (nx + 31) / 32 * 32;
    return ((size_t)nxp * TPITCH + (size_t)ROW_WAVES * 32 * TPITCH + 3) / 4 * 4 * sizeof(float) +
           (size_t)((ROW_WAVES >> wshift) + 1) * SNO_C * GPITCH * sizeof(float);
}
// Workgroups: up to two for each of the 256 CUs (the tables in LDS and the
// weights in registers are then set up once for all rows of a workgroup).
inline unsigned row_blocks(long long rows, int wshift) {
    const long long groups = (rows + (ROW_WAVES >> wshift) - 1) / (ROW_WAVES >> wshift);
    return (unsigned)(groups < 512 ? groups : 512);
}

__device__ inline float phi_cdf(float z) { return 0.5f * (1.f + erff(z * 0.70710678118654752f)); }

// LDS written by some lanes of a wave and read by others of the same wave
__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v[i] at (row drow(i, h), pixel l) -> v[i] at (row l, pixel drow(i, h))
__device__ inline void turn(float (&v)[16], float* tr, int l, int h) {
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 16; ++i) tr[drow(i, h) * TPITCH + l] = v[i];
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = tr[l * TPITCH + drow(i, h)];
}

template <int MODE, class WT>
__global__ void __launch_bounds__(ROW_NTH) __attribute__((amdgpu_waves_per_eu(4)))
k_sno_row(const RowArgs<WT> a) {
    constexpr bool LAYER = MODE == ROW_LAYER || MODE == ROW_OUT;
    constexpr bool BACK = MODE == ROW_BOUT || MODE == ROW_BLAYER || MODE == ROW_BLIFT;
    constexpr bool INV = LAYER || MODE == ROW_BLAYER || MODE == ROW_BLIFT;  // has the inverse transform
    constexpr bool FWDX = MODE != ROW_OUT && MODE != ROW_BLIFT;             // has the transform of the result
    constexpr bool WGRAD = BACK;
    constexpr int C = SNO_C;
    extern __shared__ float rl[];
    const int nx = a.nx, ny = a.ny, n = a.n;
    const int nt = (nx + 31) / 32, nxp = 32 * nt;
    const int tid = threadIdx.x, lane = tid & 63, l = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ws = a.wshift, wpr = 1 << ws, rg = ROW_WAVES >> ws;
    float* E = rl;                                  // E[x][k], pitch 33
    float* trs = rl + nxp * TPITCH;                 // a 32 x 33 tile per wave
    float* tr = trs + wave * 32 * TPITCH;
    float* gs = rl + ((nxp + ROW_WAVES * 32) * TPITCH + 3) / 4 * 4;  // g[row of the group][o][k]

    // A operands of the pointwise product, k = 16 h + s: W[o][c] forward,
    // W[o][c]^T backward, in LDS like g (in registers they would cost the
    // second workgroup of a CU)
    float* wl = gs + rg * C * GPITCH;
    {
        // every load of the tables before the first LDS write: one round trip
        float4 e[512 * 8 / ROW_NTH];
#pragma unroll
        for (int u = 0; u < 512 * 8 / ROW_NTH; ++u)
            if (tid + u * ROW_NTH < nxp * 8) e[u] = a.ex[tid + u * ROW_NTH];
        float w2[C * C / ROW_NTH];
        if constexpr (INV) {
#pragma unroll
            for (int u = 0; u < C * C / ROW_NTH; ++u) w2[u] = wval(a.w[tid + u * ROW_NTH]);
        }
#pragma unroll
        for (int u = 0; u < 512 * 8 / ROW_NTH; ++u) {
            const int i = tid + u * ROW_NTH;
            if (i >= nxp * 8) continue;
            float* p = E + (i >> 3) * TPITCH + 4 * (i & 7);
            p[0] = e[u].x;
            p[1] = e[u].y;
            p[2] = e[u].z;
            p[3] = e[u].w;
        }
        if constexpr (INV) {
#pragma unroll
            for (int u = 0; u < C * C / ROW_NTH; ++u) {
                const int i = tid + u * ROW_NTH, o = i >> 5, c = i & 31;
                wl[(LAYER ? o : c) * GPITCH + (LAYER ? c : o)] = w2[u];
            }
        }
    }
    float wa[2];
    float wbias = 0.f;
    if constexpr (INV) {
        if (LAYER && h == 0) wbias = wval(a.wb[l]);
    } else if constexpr (MODE == ROW_LIFT) {
        wa[0] = wval(a.w[3 * l + h]);
        wa[1] = h == 0 ? wval(a.w[3 * l + 2]) : wval(a.wb[l]);
    } else {
        wa[0] = wval(a.q[h * C + l]);
        wa[1] = h == 0 ? wval(a.q[2 * C + l]) : 0.f;
    }
    float qa[16];  // A operand of the projection: Q[j][o], o = drow(s, h)
    float qb[3] = {0.f, 0.f, 0.f};
    if constexpr (MODE == ROW_OUT) {
#pragma unroll
        for (int s = 0; s < 16; ++s) qa[s] = l < 3 ? wval(a.q[l * C + drow(s, h)]) : 0.f;
#pragma unroll
        for (int j = 0; j < 3; ++j) qb[j] = wval(a.qb[j]);
    }
    f32x16 dw = zero16(), dq = zero16();
    float db = 0.f, dyq[2] = {0.f, 0.f};

    const int groups = (a.rows + rg - 1) / rg;
    // row groups until the weight sums leave the FP32 accumulators
    const int period = SUM_PIXELS / (32 * ((nt + wpr - 1) >> ws));
    int held = 0;
    bool first = true;
    for (int grp = blockIdx.x; grp < groups; grp += gridDim.x) {
        const int row = grp * rg + (wave >> ws);
        const int row_b = row < a.rows ? row / ny : 0, row_y = row < a.rows ? row - row_b * ny : 0;
        const long long base = (long long)row_b * C * n, base3 = (long long)row_b * 3 * n;
        const float* src = MODE == ROW_LIFT ? a.src + base3 : a.src + base;
        const auto rsrc = row_buffer(src);
        const int n4 = 4 * n;
        // channels 16 h + s of a tile (past the row: those of x = 0, masked by the caller)
        auto load_tile = [&](int tile, float (&v)[16]) {
            const int x = 32 * tile + l;
            const int off = (16 * h * n + row_y * nx + (x < nx ? x : 0)) * 4;
#pragma unroll
            for (int s = 0; s < 16; ++s) v[s] = ldr(rsrc, off, s * n4);
        };
        float hv[16];
        if constexpr (INV) {
            // g of the group's rows: inverse y transform of the mixed modes,
            // sum_j Gh[o][j][kx] exp(+2 pi i (j - 8) y / ny), thread (o, kx)
            const int o = tid >> 4, kx = tid & 15;
            const float sc = LAYER ? (kx == 0 ? 1.f : 2.f) / ((float)nx * (float)ny) : 1.f;
            for (int rr = 0; rr < rg; ++rr) {
                const int r = grp * rg + rr;
                if (r >= a.rows) break;
                const int b = r / ny, y = r - b * ny;
                const float2* g = a.modes + ((long long)b * C + o) * NMODE + kx;
                float2 v[SNO_KY];
#pragma unroll
                for (int j = 0; j < SNO_KY; ++j) v[j] = g[j * SNO_KX];
                // the first tile, on its way while g is formed (behind the
                // modes: loads return in order)
                if (rr == 0) load_tile(wave & (wpr - 1), hv);
                int e = (8 * y) % ny;
                e = e ? ny - e : 0;  // -8 y mod ny
                float re = 0.f, im = 0.f;
#pragma unroll
                for (int j = 0; j < SNO_KY; ++j) {
                    const float2 w = a.twy[e];  // exp(-2 pi i (j - 8) y / ny), conjugated here
                    re += v[j].x * w.x + v[j].y * w.y;
                    im += v[j].y * w.x - v[j].x * w.y;
                    e += y;
                    if (e >= ny) e -= ny;
                }
                gs[(rr * C + o) * GPITCH + 2 * kx] = sc * re;
                gs[(rr * C + o) * GPITCH + 2 * kx + 1] = sc * im;
            }
        }
        __syncthreads();  // g (and, the first time, E) is complete
        f32x16 ld = zero16();  // transform of the row's result: D[k][o]
        if (row < a.rows) {
            const auto rdst = row_buffer(a.dst + base), rgd = row_buffer(a.gd + base),
                       rgi = row_buffer(a.gd_in + base), rhp = row_buffer(a.hprev + base);
            const float* gr = gs + ((wave >> ws) * C + l) * GPITCH + 16 * h;
            const float* wr = wl + l * GPITCH + 16 * h;
            const float sb = MODE == ROW_BOUT ? a.sb[row_b] : 0.f;
            for (int tile = wave & (wpr - 1); tile < nt; tile += wpr) {
                const int x = 32 * tile + l;
                const bool in = x < nx;
                const int px = row_y * nx + (in ? x : 0);
                const int p4 = (4 * h * n + px) * 4;  // channels drow(i, h)
                f32x16 d = zero16();
                float dy[2];
                if constexpr (INV) {
                    if (tile >= wpr) load_tile(tile, hv);
#pragma unroll
                    for (int s = 0; s < 16; ++s) hv[s] = in ? hv[s] : 0.f;
                    if (LAYER) d = mfma32(wbias, h == 0 ? 1.f : 0.f, d);
#pragma unroll
                    for (int s = 0; s < 16; s += 4) {
                        const float4 g4 = *reinterpret_cast<const float4*>(gr + s);
                        const float* e = E + x * TPITCH + 16 * h + s;
                        d = mfma32(g4.x, e[0], d);
                        d = mfma32(g4.y, e[1], d);
                        d = mfma32(g4.z, e[2], d);
                        d = mfma32(g4.w, e[3], d);
                    }
#pragma unroll
                    for (int s = 0; s < 16; s += 4) {
                        const float4 w4 = *reinterpret_cast<const float4*>(wr + s);
                        d = mfma32(w4.x, hv[s], d);
                        d = mfma32(w4.y, hv[s + 1], d);
                        d = mfma32(w4.z, hv[s + 2], d);
                        d = mfma32(w4.w, hv[s + 3], d);
                    }
                } else if constexpr (MODE == ROW_LIFT) {
                    const float m0 = in ? src[h * n + px] : 0.f, m1 = h == 0 ? (in ? src[2 * n + px] : 0.f) : 1.f;
                    d = mfma32(wa[0], m0, d);
                    d = mfma32(wa[1], m1, d);
                } else {
                    dy[0] = in ? sb * (a.y[base3 + h * n + px] - a.t[base3 + h * n + px]) : 0.f;
                    dy[1] = in && h == 0 ? sb * (a.y[base3 + 2 * n + px] - a.t[base3 + 2 * n + px]) : 0.f;
                    d = mfma32(wa[0], dy[0], d);
                    d = mfma32(wa[1], dy[1], d);
                    dyq[0] += dy[0];
                    dyq[1] += dy[1];
                }
                // the result: v[i] = channel drow(i, h) at pixel x
                float v[16];
                if constexpr (LAYER) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float z = d[i], cdf = phi_cdf(z);
                        v[i] = z * cdf;
                        if (a.gd && in)
                            str(rgd, p4, drow(i, 0) * n4, cdf + z * 0.39894228040143268f * expf(-0.5f * z * z));
                        if (i & 1) __builtin_amdgcn_sched_barrier(0);  // two error functions in flight, not sixteen
                    }
                } else if constexpr (MODE == ROW_BOUT || MODE == ROW_BLAYER) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = d[i] * ldr(rgi, p4, drow(i, 0) * n4);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = d[i];
                }
                if (MODE != ROW_BLIFT && a.dst && in) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) str(rdst, p4, drow(i, 0) * n4, v[i]);
                }
                if constexpr (MODE == ROW_OUT) {
                    f32x16 o = zero16();
#pragma unroll
                    for (int i = 0; i < 16; ++i) o = mfma32(qa[i], v[i], o);
                    if (in && h == 0) {
#pragma unroll
                        for (int j = 0; j < 3; ++j) a.y[base3 + j * n + px] = a.out_scale * (o[j] + qb[j]);
                    }
                }
                if constexpr (MODE != ROW_OUT) {
                    // no pixel past the row enters a sum over pixels
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = in ? v[i] : 0.f;
                    turn(v, tr, l, h);  // channel l at pixels drow(i, h)
                }
                if constexpr (FWDX) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) ld = mfma32(E[(32 * tile + drow(i, h)) * TPITCH + l], v[i], ld);
                }
                if constexpr (MODE == ROW_BOUT || MODE == ROW_BLAYER) {
                    float hp[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float u = ldr(rhp, p4, drow(i, 0) * n4);
                        hp[i] = in ? u : 0.f;
                    }
                    turn(hp, tr, l, h);
#pragma unroll
                    for (int i = 0; i < 16; ++i) dw = mfma32(v[i], hp[i], dw);
                }
                if constexpr (MODE == ROW_BOUT) {
                    // dQ: the layer's output h4 (src) against dy
                    float hq[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float u = ldr(rsrc, p4, drow(i, 0) * n4);
                        hq[i] = in ? u : 0.f;
                    }
                    turn(hq, tr, l, h);
                    wave_lds_fence();
                    tr[h * TPITCH + l] = dy[0];
                    if (h == 0) tr[2 * TPITCH + l] = dy[1];
                    wave_lds_fence();
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        dq = mfma32(l < 3 ? tr[(l < 3 ? l : 0) * TPITCH + drow(i, h)] : 0.f, hq[i], dq);
                }
                if constexpr (MODE == ROW_BLIFT) {
                    // dP, dp: columns m_x, m_y, m_z, 1
                    const float* m = a.hprev + base3;
                    const float m0 = in ? m[h * n + px] : 0.f, m2 = in && h == 0 ? m[2 * n + px] : 0.f;
                    wave_lds_fence();
                    tr[h * TPITCH + l] = m0;
                    if (h == 0) tr[2 * TPITCH + l] = m2;
                    wave_lds_fence();
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float mj = l < 3 ? tr[(l < 3 ? l : 0) * TPITCH + drow(i, h)] : (l == 3 ? 1.f : 0.f);
                        dw = mfma32(v[i], mj, dw);
                    }
                }
            }
        }
        if constexpr (FWDX) {
            if (WGRAD) db += ld[0];  // k = 0 (lanes h = 0): the plain sum over the row
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < 16; ++i) tr[l * TPITCH + drow(i, h)] = ld[i];
        }
        __syncthreads();
        if constexpr (FWDX) {
            for (int e = tid; e < rg * 1024; e += ROW_NTH) {
                const int rr = e >> 10, ok = e & 1023;
                const int r = grp * rg + rr;
                if (r >= a.rows) break;
                const float* p = trs + (rr << ws) * 32 * TPITCH + (ok >> 5) * TPITCH + (ok & 31);
                float s = p[0];
                for (int w = 1; w < wpr; ++w) s += p[w * 32 * TPITCH];
                a.line[(long long)r * 1024 + ok] = s;
            }
        }
        if constexpr (WGRAD) {
            if (++held < period && grp + (int)gridDim.x < groups) continue;
            // the weight sums of these row groups, the workgroup's waves one
            // after the other, onto its FP64 partials (an element always by the
            // same thread)
            constexpr int K = MODE == ROW_BLIFT ? KLIFT : (MODE == ROW_BOUT ? KLAYER + KPROJ : KLAYER);
            double* part = a.part + (long long)blockIdx.x * K;
            auto add = [&](int k, int e) {  // element e of the waves' tiles to partial k
                double s = trs[e];
                for (int w = 1; w < ROW_WAVES; ++w) s += trs[w * 32 * TPITCH + e];
                part[k] = first ? s : part[k] + s;
            };
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 16; ++i) tr[drow(i, h) * TPITCH + l] = dw[i];
            __syncthreads();
            if constexpr (MODE == ROW_BLIFT) {
                for (int e = tid; e < KLIFT; e += ROW_NTH) {
                    const int c = e < 3 * C ? e / 3 : e - 3 * C, j = e < 3 * C ? e - 3 * c : 3;
                    add(e, c * TPITCH + j);
                }
            } else {
                for (int e = tid; e < C * C; e += ROW_NTH) add(e, (e >> 5) * TPITCH + (e & 31));
                __syncthreads();
                if (h == 0) tr[l] = db;
                if constexpr (MODE == ROW_BOUT) {
                    if (h == 0) {
#pragma unroll
                        for (int j = 0; j < 3; ++j) tr[(1 + j) * TPITCH + l] = dq[j];
                    }
                    // dq_j: sum of dy_j over the lanes (half 0: x, half 1: y; half 0 again: z)
                    float s0 = dyq[0], s1 = dyq[1];
                    for (int off = 16; off > 0; off >>= 1) {
                        s0 += __shfl_xor(s0, off, 64);
                        s1 += __shfl_xor(s1, off, 64);
                    }
                    if (l == 0) {
                        tr[4 * TPITCH + h] = s0;
                        if (h == 0) tr[4 * TPITCH + 2] = s1;
                    }
                }
                __syncthreads();
                for (int e = C * C + tid; e < K; e += ROW_NTH) {
                    const int k = e - C * C;  // db, then dQ, then dq: rows of 32
                    add(e, (k >> 5) * TPITCH + (k & 31));
                }
            }
            dw = zero16();
            dq = zero16();
            db = dyq[0] = dyq[1] = 0.f;
            held = 0;
            first = false;
        }
    }
}

// Hh[q][j][kx] = sum_y line[b][y][c][kx] exp(-2 pi i (j - 8) y / ny), times
// w_kx / (nx ny) if `scaled`, q = (b, c): one product P[jc][kc] = sum_y
// Ey[jc][y] line[y][kc] over the real and imaginary parts (32 x 32, K = ny),
// the rows dealt over the waves, then combined.  A workgroup per q; its time is
// one pass over the rows' latency, not the 16 MB it reads (a thread per mode
// walking ny rows in turn took 16 us at batch 16 and 14 us for one sample).
__global__ void __launch_bounds__(ROW_NTH) k_sno_dfty(int nx, int ny, const float2* __restrict__ twy,
                                                      const float* __restrict__ line, float2* __restrict__ Hh,
                                                      int scaled) {
    __shared__ float2 tw[512];
    __shared__ float red[ROW_WAVES * 32 * TPITCH];
    const int q = blockIdx.x, b = q / SNO_C, c = q - b * SNO_C;
    const int tid = threadIdx.x, lane = tid & 63, l = lane & 31, h = lane >> 5, wave = tid >> 6;
    for (int i = tid; i < ny; i += ROW_NTH) tw[i] = twy[i];
    __syncthreads();
    const int ky = (l >> 1) - SNO_KY / 2;
    const int step = ky >= 0 ? ky : ky + ny;
    const float* src = line + ((long long)b * ny * SNO_C + c) * 32 + l;
    f32x16 acc = zero16();
    constexpr int BATCH = 16;  // rows in flight per lane
    for (int y0 = 2 * wave; y0 < ny; y0 += 2 * ROW_WAVES * BATCH) {
        float v[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int y = y0 + 2 * ROW_WAVES * u + h;
            v[u] = y < ny ? src[y * SNO_C * 32] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int y = y0 + 2 * ROW_WAVES * u + h;
            const float2 w = tw[y < ny ? (step * y) % ny : 0];
            acc = mfma32(y < ny ? ((l & 1) ? w.y : w.x) : 0.f, v[u], acc);
        }
    }
    float* tr = red + wave * 32 * TPITCH;
#pragma unroll
    for (int i = 0; i < 16; ++i) tr[drow(i, h) * TPITCH + l] = acc[i];
    __syncthreads();
    if (tid >= NMODE) return;
    const int j = tid >> 4, kx = tid & 15;
    float p[2][2] = {};
    for (int w = 0; w < ROW_WAVES; ++w)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int k = 0; k < 2; ++k) p[u][k] += red[w * 32 * TPITCH + (2 * j + u) * TPITCH + 2 * kx + k];
    const float s = scaled ? (kx == 0 ? 1.f : 2.f) / ((float)nx * (float)ny) : 1.f;
    Hh[(long long)q * NMODE + tid] = make_float2(s * (p[0][0] - p[1][1]), s * (p[0][1] + p[1][0]));
}

template <int MODE, class WT>
inline hipError_t row_launch(const RowArgs<WT>& a, hipStream_t s) {
    hipLaunchKernelGGL((k_sno_row<MODE, WT>), dim3(row_blocks(a.rows, a.wshift)), dim3(ROW_NTH),
                       row_lds(a.nx, a.wshift), s, a);
    return hipGetLastError();
}
template <int MODE, class WT>
inline hipError_t row_configure(int nx) {
    return hipFuncSetAttribute((const void*)k_sno_row<MODE, WT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)row_lds(nx, row_wave_shift(nx, 1LL << 40)));
}

}  // namespace

}  // namespace mm
