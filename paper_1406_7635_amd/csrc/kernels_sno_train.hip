// kernels_sno_train.hip -- training of the spectral neural operator that can
// stand in for the magnetostatic convolution: batched forward pass that keeps
// the activations, backward pass, Adam.
//
// The network is the one of kernels_sno.hip (lift 3 -> 32 channels, four
// layers of kept-mode transform -> per-mode complex 32 x 32 mixing -> inverse
// plus a pointwise 32 x 32 branch and exact-erf GELU, projection 32 -> 3),
// here with FP32 weights (the master copy; inference rounds them to BF16) and
// a batch of B samples.  Loss: the mean over the batch of the relative L2
// error ||y - t|| / ||t|| of each sample.
//
// Backward of one layer, z = g + W h + b, h' = GELU(z), g = inverse(R . H),
// H(k) = sum_r h(r) exp(-i k.r) over the kept modes, with the complex
// gradient convention Xbar = dL/dRe X + i dL/dIm X:
//   dz      = dh' GELU'(z),  GELU'(z) = Phi(z) + z phi(z)
//   dW      = sum dz h^T,  db = sum dz,  dh = W^T dz + (spectral part)
//   Gbar(k) = (w_kx / N) sum_r dz(r) exp(-i k.r)     (the forward transform of dz)
//   Rbar(k) = sum_b Gbar(k) conj(H(k))^T,  Hbar(k) = R(k)^H Gbar(k)
//   dh(r)  += Re sum_k Hbar(k) exp(+i k.r)           (inverse without w_kx / N)
// with w_0 = 1 and w_kx = 2 otherwise, N = nx ny.
//
// Layouts: fields [B][channels][ny][nx] (x fastest), kept modes
// [B][C][ky + 8][kx], weights in the flat order of include/mm.h.  Everything
// along x, and the sums over pixels (dW, db, dQ, dq, dP, dp), is done by the row
// passes of sno_rows.h; the sums go through per-workgroup partials reduced by a
// second kernel, so results do not depend on scheduling.
#include <hip/hip_runtime.h>
#include <math.h>

#include "sno_rows.h"

namespace mm {

namespace {

constexpr int C = SNO_C;
constexpr int NM = NMODE;

// Gh[b][o][k] = sum_c R[k][o][c] Hh[b][c][k]: workgroup (mode, sample), thread o.
__global__ void __launch_bounds__(C) k_tr_mix(const SnoTrainArgs a, int layer, const float2* __restrict__ Hh,
                                              float2* __restrict__ Gh) {
    __shared__ float2 hm[C];
    const int mode = blockIdx.x, b = blockIdx.y;
    const int o = threadIdx.x;
    hm[o] = Hh[((long long)b * C + o) * NM + mode];
    __syncthreads();
    const float* r = a.w + SNO_OFF_R(layer) + ((long long)mode * C + o) * C * 2;
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll 8
    for (int c = 0; c < C; ++c) {
        const float wr = r[2 * c], wi = r[2 * c + 1];
        const float2 v = hm[c];
        acc.x += wr * v.x - wi * v.y;
        acc.y += wr * v.y + wi * v.x;
    }
    Gh[((long long)b * C + o) * NM + mode] = acc;
}

// Hbar[b][c][k] = sum_o conj(R[k][o][c]) Gbar[b][o][k]: workgroup (mode,
// sample), thread c.
__global__ void __launch_bounds__(C) k_tr_hbar(const SnoTrainArgs a, int layer, const float2* __restrict__ Gb,
                                               float2* __restrict__ Hb) {
    __shared__ float2 gm[C];
    const int mode = blockIdx.x, b = blockIdx.y;
    const int c = threadIdx.x;
    gm[c] = Gb[((long long)b * C + c) * NM + mode];
    __syncthreads();
    const float* r = a.w + SNO_OFF_R(layer) + (long long)mode * C * C * 2;
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll 8
    for (int o = 0; o < C; ++o) {
        const float wr = r[(o * C + c) * 2], wi = r[(o * C + c) * 2 + 1];
        const float2 v = gm[o];
        acc.x += wr * v.x + wi * v.y;  // conj(w) v
        acc.y += wr * v.y - wi * v.x;
    }
    Hb[((long long)b * C + c) * NM + mode] = acc;
}

// Rbar[k][o][c] = sum_b Gbar[b][o][k] conj(H[b][c][k]) into the gradient:
// workgroup per mode, thread (o, c).
__global__ void __launch_bounds__(C * C) k_tr_rgrad(const SnoTrainArgs a, int layer, const float2* __restrict__ Gb,
                                                    const float2* __restrict__ H) {
    const int mode = blockIdx.x;
    const int o = threadIdx.x / C, c = threadIdx.x % C;
    float2 acc = make_float2(0.f, 0.f);
    for (int b = 0; b < a.batch; ++b) {
        const float2 g = Gb[((long long)b * C + o) * NM + mode];
        const float2 h = H[((long long)b * C + c) * NM + mode];
        acc.x += g.x * h.x + g.y * h.y;  // g conj(h)
        acc.y += g.y * h.x - g.x * h.y;
    }
    float* out = a.g + SNO_OFF_R(layer) + (((long long)mode * C + o) * C + c) * 2;
    out[0] = acc.x;
    out[1] = acc.y;
}

// per (sample, chunk): sum (y - t)^2 and sum t^2 in FP64
constexpr int LOSS_CHUNKS = 64;
__global__ void __launch_bounds__(256) k_tr_loss_part(const SnoTrainArgs a, const float* __restrict__ y,
                                                      const float* __restrict__ t, double* __restrict__ part) {
    __shared__ double red[2][4];
    const int b = blockIdx.y, ch = blockIdx.x;
    const long long len = 3LL * a.n;
    const long long per = (len + LOSS_CHUNKS - 1) / LOSS_CHUNKS;
    const long long i0 = ch * per, i1 = i0 + per < len ? i0 + per : len;
    const float* yb = y + (long long)b * len;
    const float* tb = t + (long long)b * len;
    double dd = 0.0, tt = 0.0;
    for (long long i = i0 + threadIdx.x; i < i1; i += 256) {
        const double d = (double)yb[i] - (double)tb[i];
        dd += d * d;
        tt += (double)tb[i] * (double)tb[i];
    }
    for (int off = 32; off > 0; off >>= 1) {
        dd += __shfl_xor(dd, off, 64);
        tt += __shfl_xor(tt, off, 64);
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        red[0][wv] = dd;
        red[1][wv] = tt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[((long long)b * LOSS_CHUNKS + ch) * 2] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        part[((long long)b * LOSS_CHUNKS + ch) * 2 + 1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
}

// scale[b] = 1 / (||d_b|| ||t_b|| B) (0 when d_b = 0 or t_b = 0), loss = mean
// ||d_b|| / ||t_b||: one wave, a lane per chunk of the sample
__global__ void __launch_bounds__(LOSS_CHUNKS) k_tr_loss_final(const SnoTrainArgs a, const double* __restrict__ part,
                                                               float* __restrict__ scale,
                                                               double* __restrict__ loss) {
    static_assert(LOSS_CHUNKS == 64, "a lane per chunk");
    double l = 0.0;
#pragma unroll 4
    for (int b = 0; b < a.batch; ++b) {
        double dd = part[((long long)b * LOSS_CHUNKS + threadIdx.x) * 2];
        double tt = part[((long long)b * LOSS_CHUNKS + threadIdx.x) * 2 + 1];
        for (int off = 32; off > 0; off >>= 1) {
            dd += __shfl_xor(dd, off, 64);
            tt += __shfl_xor(tt, off, 64);
        }
        const double nd = sqrt(dd), nt = sqrt(tt);
        if (threadIdx.x == 0) scale[b] = (nd > 0.0 && nt > 0.0) ? (float)(1.0 / (nd * nt * a.batch)) : 0.f;
        l += nt > 0.0 ? nd / nt : 0.0;
    }
    if (threadIdx.x == 0) *loss = l / a.batch;
}

// out[k] = sum_r part[r][k] (FP64), k < K: a workgroup takes 32
// columns, 32 threads each (a thread per column walking all rows took 0.18 ms)
__global__ void __launch_bounds__(1024) k_tr_reduce(const double* __restrict__ part, int nrows, int K,
                                                    float* __restrict__ out) {
    __shared__ double red[32][33];
    const int k = blockIdx.x * 32 + (threadIdx.x & 31), r0 = threadIdx.x >> 5;
    double s = 0.0;
    if (k < K) {
#pragma unroll 4
        for (int r = r0; r < nrows; r += 32) s += part[(long long)r * K + k];
    }
    red[r0][threadIdx.x & 31] = s;
    __syncthreads();
    if (r0 != 0 || k >= K) return;
    double t = 0.0;
    for (int i = 0; i < 32; ++i) t += red[i][threadIdx.x];
    out[k] = (float)t;
}

// Adam (Kingma and Ba): m1 <- b1 m1 + (1 - b1) g, m2 <- b2 m2 + (1 - b2) g^2,
// w <- w - lr (m1 / c1) / (sqrt(m2 / c2) + eps), c = 1 - beta^t
__global__ void __launch_bounds__(256) k_tr_adam(float* __restrict__ w, const float* __restrict__ g,
                                                 float* __restrict__ m1, float* __restrict__ m2, long long n,
                                                 float lr, float b1, float b2, float eps, float c1, float c2) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float v = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = v;
    w[i] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
}

unsigned nblk(long long n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

hipError_t configure_sno_train(int nx) {
    hipError_t e = row_configure<ROW_LIFT, float>(nx);
    if (e == hipSuccess) e = row_configure<ROW_LAYER, float>(nx);
    if (e == hipSuccess) e = row_configure<ROW_OUT, float>(nx);
    if (e == hipSuccess) e = row_configure<ROW_BOUT, float>(nx);
    if (e == hipSuccess) e = row_configure<ROW_BLAYER, float>(nx);
    if (e == hipSuccess) e = row_configure<ROW_BLIFT, float>(nx);
    return e;
}

size_t sno_train_part(int nx, int ny, int batch) {
    const long long rows = (long long)batch * ny;
    return (size_t)row_blocks(rows, row_wave_shift(nx, rows)) * (KLAYER + KPROJ);
}

// forward pass with the activations kept, loss, backward pass into a.g
hipError_t sno_train_grad(const SnoTrainArgs& a, const SnoTrainBufs& s, const float* m, const float* t,
                          hipStream_t st) {
    const int nq = a.batch * C;
    RowArgs<float> r{};
    r.nx = a.nx;
    r.ny = a.ny;
    r.n = a.n;
    r.rows = a.batch * a.ny;
    r.wshift = row_wave_shift(a.nx, r.rows);
    r.line = s.line;
    r.ex = a.ex;
    r.twy = a.twy;
    r.q = a.w + SNO_OFF_Q;
    r.qb = a.w + SNO_OFF_QB;
    r.out_scale = 1.f;
    r.y = s.y;
    r.t = t;
    r.sb = s.scale;
    r.part = s.part;
    const int blocks = (int)row_blocks(r.rows, r.wshift);
    auto reduce = [&](int K, float* out) {
        hipLaunchKernelGGL(k_tr_reduce, dim3(nblk(K, 32)), dim3(1024), 0, st, s.part, blocks, K, out);
    };
    // forward
    r.src = m;
    r.dst = s.h[0];
    r.w = a.w + SNO_OFF_P;
    r.wb = a.w + SNO_OFF_PB;
    hipError_t e = row_launch<ROW_LIFT>(r, st);
    r.modes = s.modes;
    for (int l = 0; l < SNO_LAYERS && e == hipSuccess; ++l) {
        hipLaunchKernelGGL(k_sno_dfty, dim3(nq), dim3(ROW_NTH), 0, st, a.nx, a.ny, a.twy, s.line, s.H[l], 0);
        hipLaunchKernelGGL(k_tr_mix, dim3(NM, a.batch), dim3(C), 0, st, a, l, s.H[l], s.modes);
        r.src = s.h[l];
        r.dst = s.h[l + 1];
        r.gd = s.gd[l];
        r.w = a.w + SNO_OFF_W(l);
        r.wb = a.w + SNO_OFF_B(l);
        e = l == SNO_LAYERS - 1 ? row_launch<ROW_OUT>(r, st) : row_launch<ROW_LAYER>(r, st);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tr_loss_part, dim3(LOSS_CHUNKS, a.batch), dim3(256), 0, st, a, s.y, t, s.lpart);
    hipLaunchKernelGGL(k_tr_loss_final, dim3(1), dim3(LOSS_CHUNKS), 0, st, a, s.lpart, s.scale, s.loss);
    // backward: the last layer's dz with dW, db, dQ, dq (contiguous in the flat weights)
    float* dz = s.dz[0];
    float* dzn = s.dz[1];
    r.src = s.h[SNO_LAYERS];
    r.dst = dz;
    r.gd_in = s.gd[SNO_LAYERS - 1];
    r.hprev = s.h[SNO_LAYERS - 1];
    e = row_launch<ROW_BOUT>(r, st);
    reduce(KLAYER + KPROJ, a.g + SNO_OFF_W(SNO_LAYERS - 1));
    r.modes = s.modes2;
    for (int l = SNO_LAYERS - 1; l >= 0 && e == hipSuccess; --l) {
        hipLaunchKernelGGL(k_sno_dfty, dim3(nq), dim3(ROW_NTH), 0, st, a.nx, a.ny, a.twy, s.line, s.modes, 1);
        hipLaunchKernelGGL(k_tr_rgrad, dim3(NM), dim3(C * C), 0, st, a, l, s.modes, s.H[l]);
        hipLaunchKernelGGL(k_tr_hbar, dim3(NM, a.batch), dim3(C), 0, st, a, l, s.modes, s.modes2);
        r.src = dz;
        r.dst = dzn;
        r.w = a.w + SNO_OFF_W(l);
        if (l > 0) {
            r.gd_in = s.gd[l - 1];
            r.hprev = s.h[l - 1];
            e = row_launch<ROW_BLAYER>(r, st);
            reduce(KLAYER, a.g + SNO_OFF_W(l - 1));
        } else {
            r.hprev = m;
            e = row_launch<ROW_BLIFT>(r, st);
            reduce(KLIFT, a.g + SNO_OFF_P);
        }
        float* tmp = dz;
        dz = dzn;
        dzn = tmp;
    }
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

hipError_t sno_train_adam(float* w, const float* g, float* m1, float* m2, long long n, float lr, float b1, float b2,
                          float eps, long long step, hipStream_t st) {
    const float c1 = (float)(1.0 - pow((double)b1, (double)step));
    const float c2 = (float)(1.0 - pow((double)b2, (double)step));
    hipLaunchKernelGGL(k_tr_adam, dim3(nblk(n, 256)), dim3(256), 0, st, w, g, m1, m2, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace mm
