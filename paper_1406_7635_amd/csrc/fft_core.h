// fft_core.h -- register-resident FP32 FFT building blocks for gfx950.
//
// Power-of-two transforms in Stockham (autosort) form: stage (R, L) reads
// inputs j + r P/R, multiplies them by w^(r k) with w = exp(-+2 pi i/(L R)) and
// k = j mod L, does an R-point DFT and writes the outputs to (j - k) R + k + r L.
// Forward uses exp(-2 pi i n k / P), inverse exp(+...), both unnormalised.
// Each thread keeps its points in registers; LDS is only the exchange medium
// between stages.
#pragma once

#include <hip/hip_runtime.h>

namespace mm {

// No implicit contraction in this file: where a product and a sum fuse is
// written out, so every instance of a transform (tile shapes, components per
// thread, single grids and ensembles) rounds alike.  That holds for the operators
// below wherever they are used: a sum of products of a caller takes cfma and
// crow3, or it rounds twice a term.
#pragma clang fp contract(off)

struct alignas(8) cf {
    float x, y;
};

__host__ __device__ inline cf mkc(float x, float y) { cf r; r.x = x; r.y = y; return r; }
__host__ __device__ inline cf operator+(cf a, cf b) { return mkc(a.x + b.x, a.y + b.y); }
__host__ __device__ inline cf operator-(cf a, cf b) { return mkc(a.x - b.x, a.y - b.y); }
__host__ __device__ inline cf operator*(float s, cf a) { return mkc(s * a.x, s * a.y); }
__host__ __device__ inline cf cmul(cf a, cf b) {
    return mkc(__builtin_fmaf(-a.y, b.y, a.x * b.x), __builtin_fmaf(a.y, b.x, a.x * b.y));
}
// a + s b with a real s, and k0 a + k1 b + k2 c with real k
__host__ __device__ inline cf cfma(float s, cf b, cf a) {
    return mkc(__builtin_fmaf(s, b.x, a.x), __builtin_fmaf(s, b.y, a.y));
}
__host__ __device__ inline cf crow3(float k0, cf a, float k1, cf b, float k2, cf c) {
    return cfma(k2, c, cfma(k1, b, k0 * a));
}
__host__ __device__ inline cf cconj(cf a) { return mkc(a.x, -a.y); }

// Complex load and store through a raw buffer resource: uniform base in
// scalar registers, 32-bit byte offset per lane (no 64-bit address
// arithmetic); the third resource word is the gfx9 family's untyped format.
// Device code only (declared in both compilation passes, as device code
// that the host pass parses refers to them).
__device__ inline __amdgpu_buffer_rsrc_t cf_buffer(const cf* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<cf*>(base), (short)0, (int)0xffffffffu, 0x00020000);
}
__device__ inline cf ld_cf(const cf* base, unsigned int byte_off) {
    return __builtin_bit_cast(cf, __builtin_amdgcn_raw_buffer_load_b64(cf_buffer(base), (int)byte_off, 0, 0));
}
__device__ inline void st_cf(cf* base, unsigned int byte_off, cf v) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), cf_buffer(base), (int)byte_off, 0, 0);
}

// Two adjacent complex values.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ inline f32x4 ld_cf2(const cf* base, unsigned int byte_off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(cf_buffer(base), (int)byte_off, 0, 0));
}
__device__ inline void st_cf2(cf* base, unsigned int byte_off, f32x4 v) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), cf_buffer(base), (int)byte_off, 0, 0);
}

// multiply by exp(+-i pi/2): forward (INV=false) by -i, inverse by +i
template <bool INV>
__host__ __device__ inline cf rot90(cf a) {
    return INV ? mkc(-a.y, a.x) : mkc(a.y, -a.x);
}

constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }
constexpr int ilog2_floor(int n) { return n <= 1 ? 0 : 1 + ilog2_floor(n / 2); }
__host__ __device__ inline int ilog2_rt(int n) {
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

// LDS position of sequence element i outside the transforms (staging,
// separation, crop): three spare elements after every 32, so contiguous wave
// accesses meet at most one spare run; being additive over 32-aligned
// offsets, the per-register offsets fold into the instructions' immediate
// offsets.  The exchanges inside a transform use their own padding
// (RegFft::xpad), at most one spare per 8 elements.
__host__ __device__ constexpr int lds_pad(int i) { return i + 3 * (i >> 5); }
__host__ __device__ constexpr int seq_len(int P) { return P + (P >> 3); }

// R-point DFTs in registers -------------------------------------------------
template <int R, bool INV>
struct Dft;

template <bool INV>
struct Dft<1, INV> {
    __host__ __device__ static void run(cf*) {}
};

template <bool INV>
struct Dft<2, INV> {
    __host__ __device__ static void run(cf* v) {
        cf a = v[0], b = v[1];
        v[0] = a + b;
        v[1] = a - b;
    }
};

template <bool INV>
struct Dft<4, INV> {
    __host__ __device__ static void run(cf* v) {
        cf a0 = v[0] + v[2], a1 = v[0] - v[2];
        cf a2 = v[1] + v[3], a3 = rot90<INV>(v[1] - v[3]);
        v[0] = a0 + a2;
        v[2] = a0 - a2;
        v[1] = a1 + a3;
        v[3] = a1 - a3;
    }
};

template <bool INV>
struct Dft<8, INV> {
    __host__ __device__ static void run(cf* v) {
        const float h = 0.70710678118654752f;  // 1/sqrt(2)
        cf e[4] = {v[0], v[2], v[4], v[6]};
        cf o[4] = {v[1], v[3], v[5], v[7]};
        Dft<4, INV>::run(e);
        Dft<4, INV>::run(o);
        // v[k], v[k + 4] = e[k] +- w8^k o[k] with w8 = exp(-+ i pi/4); the factor
        // 1/sqrt(2) of k = 1, 3 goes into fused multiply-adds
        const cf o2 = rot90<INV>(o[2]);
        const cf p1 = INV ? mkc(o[1].x - o[1].y, o[1].x + o[1].y) : mkc(o[1].x + o[1].y, o[1].y - o[1].x);
        const cf p3 = INV ? mkc(-(o[3].x + o[3].y), o[3].x - o[3].y) : mkc(o[3].y - o[3].x, -(o[3].x + o[3].y));
        v[0] = e[0] + o[0];
        v[4] = e[0] - o[0];
        v[1] = cfma(h, p1, e[1]);
        v[5] = cfma(-h, p1, e[1]);
        v[2] = e[2] + o2;
        v[6] = e[2] - o2;
        v[3] = cfma(h, p3, e[3]);
        v[7] = cfma(-h, p3, e[3]);
    }
};

template <bool INV>
struct Dft<16, INV> {
    // 16 = 4 x 4: DFT-4 over n1 for each n2, twiddle w16^(n2 k1), DFT-4 over n2
    __host__ __device__ static void run(cf* v) {
        const float c1 = 0.92387953251128676f, s1 = 0.38268343236508977f, h = 0.70710678118654752f;
        const float cs[10][2] = {{1.f, 0.f}, {c1, s1}, {h, h}, {s1, c1}, {0.f, 1.f},
                                 {-s1, c1}, {-h, h}, {-c1, s1}, {-1.f, 0.f}, {-c1, -s1}};
        cf a[4][4];
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) {
            cf t[4] = {v[n2], v[n2 + 4], v[n2 + 8], v[n2 + 12]};
            Dft<4, INV>::run(t);
#pragma unroll
            for (int k1 = 0; k1 < 4; ++k1) {
                const int m = n2 * k1;
                const cf w = mkc(cs[m][0], INV ? cs[m][1] : -cs[m][1]);
                a[n2][k1] = (m == 0) ? t[k1] : cmul(t[k1], w);
            }
        }
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            cf t[4] = {a[0][k1], a[1][k1], a[2][k1], a[3][k1]};
            Dft<4, INV>::run(t);
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = t[k2];
        }
    }
};

// exp(-+2 pi i m / 16) x for a compile-time m (after unrolling): the
// multiplications by 0 and +-1 are spelled out, since the compiler may not
// drop them itself (signed zeros)
template <bool INV>
__host__ __device__ inline cf twist16(cf x, int m) {
    const float c1 = 0.92387953251128676f, s1 = 0.38268343236508977f, h = 0.70710678118654752f;
    m &= 15;
    if (m == 0) return x;
    if (m == 4) return rot90<INV>(x);
    if (m == 8) return mkc(-x.x, -x.y);
    if (m == 12) return rot90<!INV>(x);
    const float cs[16][2] = {{1.f, 0.f}, {c1, s1}, {h, h}, {s1, c1}, {0.f, 1.f}, {-s1, c1}, {-h, h}, {-c1, s1},
                             {-1.f, 0.f}, {-c1, -s1}, {-h, -h}, {-s1, -c1}, {0.f, -1.f}, {s1, -c1}, {h, -h}, {c1, -s1}};
    const float wr = cs[m][0], wi = INV ? cs[m][1] : -cs[m][1];
    if ((m & 3) == 2) {  // +-h (1 +- i): two products instead of four
        const float hr = wr, hi = wi;  // |hr| = |hi| = h
        return (hr == hi) ? mkc(hr * (x.x - x.y), hr * (x.x + x.y)) : mkc(hr * (x.x + x.y), hr * (x.y - x.x));
    }
    return cmul(x, mkc(wr, wi));
}

// R-point DFT of a sequence whose upper R/2 inputs are zero (zero padding):
// the even outputs are the R/2-point DFT of the inputs, the odd outputs that
// of the inputs twisted by w_R^n.  Inputs in v[0..R/2), outputs in v[0..R).
template <int R, bool INV>
struct DftHalf {
    __host__ __device__ static void run(cf* v) {
        constexpr int H = R / 2;
        cf y[H], z[H];
#pragma unroll
        for (int n = 0; n < H; ++n) {
            y[n] = v[n];
            z[n] = twist16<INV>(v[n], n * (16 / R));
        }
        Dft<H, INV>::run(y);
        Dft<H, INV>::run(z);
#pragma unroll
        for (int j = 0; j < H; ++j) {
            v[2 * j] = y[j];
            v[2 * j + 1] = z[j];
        }
    }
};

// Radix-2 step (a, b) -> (a + w b, a - w b) in six fused multiply-adds: the
// difference is 2 a - (a + w b).
__host__ __device__ inline void bfly_fma(cf a, cf b, cf w, cf& p, cf& m) {
    p = mkc(__builtin_fmaf(-w.y, b.y, __builtin_fmaf(w.x, b.x, a.x)),
            __builtin_fmaf(w.y, b.x, __builtin_fmaf(w.x, b.y, a.y)));
    m = mkc(__builtin_fmaf(2.f, a.x, -p.x), __builtin_fmaf(2.f, a.y, -p.y));
}

// R-point DFT of inputs twisted by w^r (the twiddle of a Stockham stage),
// X[j] = sum_r w^r v[r] w_R^(r j): decimation in time with the twist folded
// into the radix-2 multipliers, X[j], X[j + R/2] = E[j] +- (w w_R^j) O[j], E and
// O the twisted DFTs (w^2) of the even and odd inputs.  wt: the multipliers
// w w_R^j for j < max(R/4, 1) (the next R/4 are a quarter turn further), then
// those of R/2 with w^2, and so on.
// Why: the passes spend about half their time issuing vector instructions.  A
// radix-8 stage takes 72 of them here plus 4 for the multipliers; twisting the
// seven inputs first (28), the plain butterflies (about 64) and the products
// that form the other four powers (16) took 108.  1024^2 film, one attempt:
// 408 -> 397 us; 150 x 90 x 37 field: 152 -> 149 us; error against 64 bits
// unchanged (B_demag 2.5e-7 -> 2.4e-7).
template <int R, bool INV>
struct TwDft {
    __host__ __device__ static void run(cf* v, const cf* wt) {
        constexpr int H = R / 2, Q = R / 4;
        cf e[H], o[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            e[i] = v[2 * i];
            o[i] = v[2 * i + 1];
        }
        TwDft<H, INV>::run(e, wt + Q);
        TwDft<H, INV>::run(o, wt + Q);
#pragma unroll
        for (int j = 0; j < H; ++j) bfly_fma(e[j], o[j], j < Q ? wt[j] : rot90<INV>(wt[j - Q]), v[j], v[j + H]);
    }
};
template <bool INV>
struct TwDft<2, INV> {
    __host__ __device__ static void run(cf* v, const cf* wt) { bfly_fma(v[0], v[1], wt[0], v[0], v[1]); }
};
template <bool INV>
struct TwDft<1, INV> {
    __host__ __device__ static void run(cf*, const cf*) {}
};

// ---------------------------------------------------------------------------
// Barrier of the threads that exchange through one LDS sequence.  A group of at
// most 64 threads with consecutive indices lies in one wave, whose LDS accesses
// complete in order: a fence for the compiler is enough, and the waves of a
// workgroup are free to drift apart (their loads, butterflies and stores then
// overlap; with workgroup barriers they ran in step).  64^2 film: 139 -> 134 us
// an attempt; 32 x 32 x 4 RK4 step: 90.6 -> 86.6 us; 96-member ensemble, two
// attempts: 2.02 -> 1.96 ms.  Lengths from 1024 on (128 threads a sequence and
// more) keep the workgroup barrier.
template <bool WAVE>
__device__ inline void group_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// Register-resident transform.  A group of TPF threads owns NF sequences of
// length P; thread t keeps PPT = P/TPF points of each in registers, in
// natural order v[f][m] = x[t + TPF m] on entry and X[t + TPF m] on exit.
// Stage 0 has radix R0 (the remainder of log2 P modulo log2 PPT, else PPT) and
// runs on the loaded registers; every later stage has radix PPT and gets its
// inputs through one LDS exchange (write the previous stage's outputs at their
// Stockham positions, barrier, read j + r TPF).  The NF sequences go through a
// single LDS sequence one after the other, so a group needs seq_len(P)
// elements of LDS.  The exchange halves are separate __host__ __device__
// functions so a host program can emulate a group without a GPU.
// HIN: the inputs x[n], n >= P/2, are zero (zero padding) and the registers
// holding them are ignored; stage 0 then runs the half-input butterflies.
template <int P, int TPF, int NF, bool INV, bool HIN = false>
struct RegFft {
    static constexpr int PPT = P / TPF;
    static constexpr int LP = ilog2(P);
    static constexpr int LA = ilog2(PPT);
    static constexpr int REM = LA == 0 ? 0 : LP % LA;
    static constexpr int R0 = LA == 0 ? 1 : (REM ? (1 << REM) : PPT);
    static constexpr int NS = LA == 0 ? 0 : (REM ? 1 : 0) + LP / LA;
    static constexpr int SEQ = seq_len(P);

    // span of stage s (product of the radices before it)
    __host__ __device__ static int span(int s) { return s == 0 ? 1 : R0 << (LA * (s - 1)); }

    // natural order -> stage-0 order, then the stage-0 butterflies (no twiddles).
    // Input r of butterfly u is x[t + TPF u + r P/R0], zero for r >= R0/2 under HIN.
    __host__ __device__ static void stage0(cf (&v)[NF][PPT]) {
        constexpr bool HALF = HIN && R0 >= 2;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            cf w[PPT];
#pragma unroll
            for (int u = 0; u < PPT / R0; ++u)
#pragma unroll
                for (int r = 0; r < R0; ++r) w[u * R0 + r] = v[f][u + r * (PPT / R0)];
#pragma unroll
            for (int u = 0; u < PPT / R0; ++u) {
                if constexpr (HALF)
                    DftHalf<R0, INV>::run(w + u * R0);
                else
                    Dft<R0, INV>::run(w + u * R0);
            }
#pragma unroll
            for (int i = 0; i < PPT; ++i) v[f][i] = w[i];
        }
    }

    // The multipliers of thread t in stage s >= 1, in the order TwDft takes
    // them: for R = PPT, PPT/2, ... 2 the first quarter (at least one) of
    // w^(k PPT/R) w_R^j.  The powers w^(2^i k) come from the table
    // (exp(-2 pi i m / PT) rounded once), the others are one constant rotation
    // of them away.
    __host__ __device__ static void twiddles(int s, int t, const cf* __restrict__ tw, int twshift, cf (&wt)[PPT]) {
        const int L = span(s);
        int k = t & (L - 1);
#ifdef __HIP_DEVICE_COMPILE__
        asm volatile("" : "+v"(k));  // keep the table loads at their stage (short live ranges)
#endif
        const int sh = twshift - ilog2_rt(L * PPT);
        int o = 0;
#pragma unroll
        for (int r = PPT; r >= 2; r >>= 1) {
            const int m = ((PPT / r) * k) << sh;
#ifdef __HIP_DEVICE_COMPILE__
            const cf w = ld_cf(tw, (unsigned int)m * 8u);
#else
            const cf w = tw[m];
#endif
            const cf b = INV ? cconj(w) : w;
            const int q = r >= 4 ? r / 4 : 1;
#pragma unroll
            for (int j = 0; j < q; ++j) wt[o + j] = twist16<INV>(b, j * (16 / r));
            o += q;
        }
    }

    // LDS position of element i in the exchange whose writes have radix RP
    // and span lp (the exchange that feeds a stage).  Each wave writes its 16-lane
    // groups (8 bytes a lane, 128 bytes a group) so that no two lanes share a
    // bank: span 1 writes lanes RP elements apart, which one spare per 16
    // elements spreads over all banks; spans 2 ... 8 write runs of lp elements
    // RP lp apart, which lp spares per RP lp elements stagger; from span 16 on the
    // runs are contiguous and need none.  Every form is additive over the
    // thread's register offsets (r lp, r TPF for TPF a multiple of 8 lp), so
    // they fold into immediate offsets, and stays below P + P/8.
    __host__ __device__ static int xpad(int rp, int lp, int i) {
        if (lp == 1) return i + (i >> 4);
        if (lp < 16) {
            const int sh = ilog2_rt(rp * lp), sl = ilog2_rt(lp);
            return i + ((i >> sh) << sl);
        }
        return i;
    }
    // radix and span of the writes of the exchange that feeds stage s (>= 1)
    __host__ __device__ static int xrp(int s) { return s == 1 ? R0 : PPT; }
    __host__ __device__ static int xlp(int s) { return s == 1 ? 1 : span(s - 1); }

    // write the outputs of stage s-1 of sequence f at their positions
    template <int RP>
    __host__ __device__ static void write_r(int lp, const cf (&v)[NF][PPT], int f, cf* buf, int t) {
#pragma unroll
        for (int uu = 0; uu < PPT / RP; ++uu) {
            const int j = t + TPF * uu;
            const int k = j & (lp - 1);
            const int base = (j - k) * RP + k;
#pragma unroll
            for (int r = 0; r < RP; ++r) buf[xpad(RP, lp, base + r * lp)] = v[f][uu * RP + r];
        }
    }
    __host__ __device__ static void write(int s, const cf (&v)[NF][PPT], int f, cf* buf, int t) {
        if (s == 1)
            write_r<R0>(1, v, f, buf, t);
        else
            write_r<PPT>(span(s - 1), v, f, buf, t);
    }

    // read the inputs of stage s (>= 1) for sequence f
    __host__ __device__ static void read(int s, cf (&v)[NF][PPT], int f, const cf* buf, int t) {
        const int rp = xrp(s), lp = xlp(s);
#pragma unroll
        for (int r = 0; r < PPT; ++r) v[f][r] = buf[xpad(rp, lp, t + r * TPF)];
    }
    // twiddled butterfly of stage s (>= 1) for sequence f
    __host__ __device__ static void compute(cf (&v)[NF][PPT], int f, const cf (&wt)[PPT]) {
        TwDft<PPT, INV>::run(v[f], wt);
    }
    __host__ __device__ static void read_compute(int s, cf (&v)[NF][PPT], int f, const cf* buf, int t,
                                                 const cf (&wt)[PPT]) {
        read(s, v, f, buf, t);
        compute(v, f, wt);
    }

    // stage order of the last stage -> natural order
    __host__ __device__ static void finish(cf (&v)[NF][PPT]) {
        constexpr int RL = NS == 1 ? R0 : PPT;
        if (RL == 1) return;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            cf w[PPT];
#pragma unroll
            for (int u = 0; u < PPT / RL; ++u)
#pragma unroll
                for (int r = 0; r < RL; ++r) w[u + r * (PPT / RL)] = v[f][u * RL + r];
#pragma unroll
            for (int i = 0; i < PPT; ++i) v[f][i] = w[i];
        }
    }

    // CONTIG: the threads of a group have consecutive indices (group_sync).
    // The group's LDS sequence must be free of other waves' accesses on entry.
    // With NF > 1 the butterfly of sequence f - 1 runs between the LDS writes
    // of sequence f and the barrier that publishes them, so it covers their
    // latency and the wait at the barrier.
    static constexpr bool IN_WAVE = TPF <= 64;
    template <bool CONTIG = true>
    __device__ static void run(cf (&v)[NF][PPT], cf* buf, const cf* __restrict__ tw, int twshift, int t) {
        if (NS == 0) return;
        stage0(v);
#pragma unroll
        for (int s = 1; s < NS; ++s) {
            cf wt[PPT];
            twiddles(s, t, tw, twshift, wt);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                group_sync<CONTIG && IN_WAVE>();
                if (s == 1)
                    write_r<R0>(1, v, f, buf, t);
                else
                    write_r<PPT>(span(s - 1), v, f, buf, t);
                if (f > 0) compute(v, f - 1, wt);
                group_sync<CONTIG && IN_WAVE>();
                read(s, v, f, buf, t);
            }
            compute(v, NF - 1, wt);
        }
        finish(v);
    }
};

#pragma clang fp contract(fast)

}  // namespace mm
