// kernels_sno.hip -- forward pass of the spectral neural operator that can
// stand in for the magnetostatic convolution at the inner Runge-Kutta stages.
//
// The network (32 channels, kept modes kx = 0..15, ky = -8..7, four layers):
//   lift      h_c = sum_j P[c][j] m_j + p[c]
//   layer     hhat_c(k) = sum_{x,y} h_c(x, y) exp(-2 pi i (kx x/nx + ky y/ny))
//             ghat_o(k) = sum_c R[ky + 8][kx][o][c] hhat_c(k)
//             g_o = Re sum_k w_kx ghat_o(k) exp(+2 pi i (...)) / (nx ny), w_0 = 1, else 2
//             h_o <- GELU(g_o + sum_c W[o][c] h_c + b[o])   (exact erf form)
//   project   B_j = scale (sum_c Q[j][c] h_c + q[j])
// Weights are stored as BF16 and widened to FP32; all arithmetic and
// accumulation is FP32.  Activations are FP32 [32][ny][nx].
//
// Launches: the lift, then per layer the y transform of the kept columns, the
// mode mixing, and one pass over the rows (inverse transform, pointwise branch,
// GELU and the x transform of the result; the last layer's also projects).
// The row passes and the y transform are in sno_rows.h.
#include <hip/hip_runtime.h>

#include "sno_rows.h"

namespace mm {

namespace {

// exp(-2 pi i m / n), m < n, evaluated in FP64 and rounded once
__global__ void k_sno_twiddles(float2* tw, int n) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m < n) {
        double s, c;
        sincospi(-2.0 * (double)m / (double)n, &s, &c);
        tw[m] = make_float2((float)c, (float)s);
    }
}

// E[x][2 kx + {0, 1}] = re, im of exp(-2 pi i kx x / nx), 0 for x >= nx, from the
// table of exp(-2 pi i m / nx)
__global__ void __launch_bounds__(256) k_sno_ex(const float2* __restrict__ twx, int nx, float* __restrict__ ex) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int x = i >> 4, kx = i & 15;
    if (x >= (nx + 31) / 32 * 32) return;
    const float2 w = x < nx ? twx[(kx * x) % nx] : make_float2(0.f, 0.f);
    ex[2 * i] = w.x;
    ex[2 * i + 1] = w.y;
}

// Ghat[o][j][kx] = sum_c R[j][kx][o][c] Hhat[c][j][kx]: a workgroup per mode,
// thread o.
__global__ void __launch_bounds__(SNO_C) k_sno_mix(const SnoArgs a, const uint16_t* __restrict__ R,
                                                   const float2* __restrict__ Hh, float2* __restrict__ Gh) {
    __shared__ float2 hm[SNO_C];
    const int mode = blockIdx.x;  // j * 16 + kx
    const int o = threadIdx.x;
    hm[o] = Hh[(long long)o * SNO_KY * SNO_KX + mode];
    __syncthreads();
    const uint16_t* r = R + ((long long)mode * SNO_C + o) * SNO_C * 2;
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll 8
    for (int c = 0; c < SNO_C; ++c) {
        const float2 w = make_float2(wval(r[2 * c]), wval(r[2 * c + 1]));
        const float2 v = hm[c];
        acc.x += w.x * v.x - w.y * v.y;
        acc.y += w.x * v.y + w.y * v.x;
    }
    Gh[(long long)o * SNO_KY * SNO_KX + mode] = acc;
}

}  // namespace

hipError_t sno_twiddles(float2* tw, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_sno_twiddles, dim3((n + 255) / 256), dim3(256), 0, s, tw, n);
    return hipGetLastError();
}

hipError_t sno_ex(const float2* twx, int nx, float4* ex, hipStream_t s) {
    hipLaunchKernelGGL(k_sno_ex, dim3((unsigned)(sno_ex_floats(nx) / 2 + 255) / 256), dim3(256), 0, s, twx, nx,
                       reinterpret_cast<float*>(ex));
    return hipGetLastError();
}

hipError_t sno_forward(const SnoArgs& a, const float* m, float* out, hipStream_t s) {
    RowArgs<uint16_t> r{};
    r.nx = a.nx;
    r.ny = a.ny;
    r.n = a.n;
    r.rows = a.ny;
    r.wshift = row_wave_shift(a.nx, r.rows);
    r.line = a.line;
    r.ex = a.ex;
    r.twy = a.twy;
    r.src = m;
    r.dst = a.h0;
    r.w = a.lift;
    r.wb = a.lift_b;
    hipError_t e = row_launch<ROW_LIFT>(r, s);
    r.modes = a.Gh;
    r.q = a.proj;
    r.qb = a.proj_b;
    r.out_scale = a.scale;
    r.y = out;
    float* h = a.h0;
    float* hn = a.h1;
    for (int l = 0; l < SNO_LAYERS && e == hipSuccess; ++l) {
        hipLaunchKernelGGL(k_sno_dfty, dim3(SNO_C), dim3(ROW_NTH), 0, s, a.nx, a.ny, a.twy, a.line, a.Hh, 0);
        hipLaunchKernelGGL(k_sno_mix, dim3(NMODE), dim3(SNO_C), 0, s, a, a.spec[l], a.Hh, a.Gh);
        r.src = h;
        r.w = a.pw[l];
        r.wb = a.pw_b[l];
        const bool last = l == SNO_LAYERS - 1;
        r.dst = last ? nullptr : hn;
        e = last ? row_launch<ROW_OUT>(r, s) : row_launch<ROW_LAYER>(r, s);
        float* t = h;
        h = hn;
        hn = t;
    }
    return e;
}

hipError_t configure_sno(int nx) {
    hipError_t e = row_configure<ROW_LIFT, uint16_t>(nx);
    if (e == hipSuccess) e = row_configure<ROW_LAYER, uint16_t>(nx);
    if (e == hipSuccess) e = row_configure<ROW_OUT, uint16_t>(nx);
    return e;
}

}  // namespace mm
