// OaAConv: the method the paper compares the split convolution against
// (Section 2 and Fig. 1; its operation counts are eqs. 11-12).  The image is
// cut into patches of the filter's size, T = K; each is zero-padded to
// L = 2K - 1 points per side and transformed, multiplied by the filter
// spectra per bin and summed over input channels (the shared contraction
// kernel), inverse-transformed, and the L x L results of neighbouring
// patches are overlap-added.  Here it is the library's overlap-add pipeline
// run at T = K, with the odd transform sizes L = 5, 9, 13 (K = 3, 5, 7) that
// this file adds.
//
// One thread owns one (channel, patch): at these sizes a patch's whole 2-D
// transform fits in registers, and the lanes of a wave hold consecutive
// patches, so every spectrum slot is written (forward) or read (inverse) as
// one contiguous run across the wave.  The transforms are direct sums with
// compile-time twiddles that use the structure of the data:
//   forward: only K x K of the L x L inputs are nonzero, and the input is
//     real, so only columns k2 in [0, (L-1)/2] are formed
//     (S(k1, L-k2) = conj S(L-k1, k2));
//   inverse: the output is real; column k2 = 0 and the pairs k2, L-k2
//     combine into real parts (y = C_0 + 2 Re sum_{k2=1}^{(L-1)/2} ...).
// The inverse's 1/L^2 is folded into the filter spectra, as for even L.
// Of each L x L result only one entry's output pixel is reached by no other
// patch (T - 2P = 1 per side).  oaa_inverse_strip_kernel adds the results up
// in LDS; for images too wide for its strips oaa_inverse_kernel writes them
// to the aux buffer and the seam pass sums the 1-4 contributions of every
// pixel.
#include <type_traits>

#include "fftsplit_internal.hpp"
#include "fft_regs.hpp"
#include "launch_util.hpp"

namespace fftsplit {

// cos and sin of 2 pi k / L for the odd sizes (twiddles.inc), k reduced
// mod L; k is a compile-time constant after unrolling.
template <int L>
__device__ __forceinline__ float odd_cos(int k) {
    k %= L;
    if constexpr (L == 5) return kTw5CosF[k];
    else if constexpr (L == 9) return kTw9CosF[k];
    else return kTw13CosF[k];
}
template <int L>
__device__ __forceinline__ float odd_sin(int k) {
    k %= L;
    if constexpr (L == 5) return kTw5SinF[k];
    else if constexpr (L == 9) return kTw9SinF[k];
    else return kTw13SinF[k];
}

template <int L>
__global__ __launch_bounds__(256) void oaa_forward_kernel(const float* __restrict__ x, float2* __restrict__ xs,
                                                          int cin, int h, int w, int th, int tw, int nt, int ntp) {
    constexpr int K = (L + 1) / 2, T = K, H = L / 2, F = stored_bins(L);
    const int c = blockIdx.y;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= ntp) return;
    float2* dst = xs + spec_offset(c, 0, t, F, ntp);
    const size_t bstride = size_t(kChanBlock) * ntp;   // between the slots of one channel
    if (t >= nt) {   // padding patches: zero spectra
#pragma unroll
        for (int f = 0; f < F; ++f) dst[f * bstride] = make_float2(0.f, 0.f);
        return;
    }
    const int b = t % tw;
    const int rest = t / tw;
    const int a = rest % th;
    const int img = rest / th;
    const int rows = min(T, h - a * T), cols = min(T, w - b * T);
    const float* src = x + ((size_t(img) * cin + c) * h + a * T) * w + b * T;
    float v[K][K];
#pragma unroll
    for (int m = 0; m < K; ++m)
#pragma unroll
        for (int q = 0; q < K; ++q) v[m][q] = (m < rows && q < cols) ? src[m * w + q] : 0.f;

    // rows: R[m][k2] = sum_q v[m][q] exp(-2 pi i q k2 / L), k2 in [0, H]
    float2 R[K][H + 1];
#pragma unroll
    for (int m = 0; m < K; ++m) {
#pragma unroll
        for (int k2 = 0; k2 <= H; ++k2) {
            float re = 0.f, im = 0.f;
#pragma unroll
            for (int q = 0; q < K; ++q) {
                re = fmaf(v[m][q], odd_cos<L>(q * k2), re);
                im = fmaf(-v[m][q], odd_sin<L>(q * k2), im);
            }
            R[m][k2] = make_float2(re, im);
        }
    }
    // columns: S(k1, k2) = sum_m R[m][k2] exp(-2 pi i m k1 / L)
    auto bin = [&](int k1, int k2) {
        float re = 0.f, im = 0.f;
#pragma unroll
        for (int m = 0; m < K; ++m) {
            const float cs = odd_cos<L>(m * k1), sn = odd_sin<L>(m * k1);
            re = fmaf(R[m][k2].x, cs, fmaf(R[m][k2].y, sn, re));
            im = fmaf(R[m][k2].y, cs, fmaf(-R[m][k2].x, sn, im));
        }
        return make_float2(re, im);
    };
#pragma unroll
    for (int k2 = 1; k2 <= H; ++k2)
#pragma unroll
        for (int k1 = 0; k1 < L; ++k1) dst[bin_mid(L, k1, k2) * bstride] = bin(k1, k2);
#pragma unroll
    for (int k1 = 0; k1 <= H; ++k1) dst[bin_odd_col0(L, k1) * bstride] = bin(k1, 0);
}

// One patch's L x L result from its F stored bins, all in registers: the
// columns k2 = 0 (Hermitian, real results) and 1..H, then each row m.  Both
// passes form the outputs m and L - m (q and L - q) from one even and one
// odd sum over the sums and differences of the inputs k and L - k: at L = 9
// about 800 vector operations instead of the 2000 of a sum per output.
template <int L>
__device__ __forceinline__ void oaa_inverse_patch(const float2 (&Y)[stored_bins(L)], float (&o)[L][L]) {
    constexpr int H = L / 2;
    float c0[L];
    float2 C[H][L];
    {
        const float y00 = Y[bin_odd_col0(L, 0)].x;
        c0[0] = y00;
#pragma unroll
        for (int k = 1; k <= H; ++k) c0[0] = fmaf(2.f, Y[bin_odd_col0(L, k)].x, c0[0]);
#pragma unroll
        for (int m = 1; m <= H; ++m) {
            float even = y00, odd = 0.f;
#pragma unroll
            for (int k = 1; k <= H; ++k) {
                even = fmaf(2.f * Y[bin_odd_col0(L, k)].x, odd_cos<L>(m * k), even);
                odd = fmaf(-2.f * Y[bin_odd_col0(L, k)].y, odd_sin<L>(m * k), odd);
            }
            c0[m] = even + odd;
            c0[L - m] = even - odd;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k2 = 1; k2 <= H; ++k2) {
        float2 s[H + 1], d[H + 1];
        s[0] = Y[bin_mid(L, 0, k2)];
        float2 sum = s[0];
#pragma unroll
        for (int k = 1; k <= H; ++k) {
            const float2 u = Y[bin_mid(L, k, k2)], v = Y[bin_mid(L, L - k, k2)];
            s[k] = make_float2(u.x + v.x, u.y + v.y);
            d[k] = make_float2(u.x - v.x, u.y - v.y);
            sum.x += s[k].x;
            sum.y += s[k].y;
        }
        C[k2 - 1][0] = sum;
#pragma unroll
        for (int m = 1; m <= H; ++m) {
            float2 even = s[0], odd = make_float2(0.f, 0.f);
#pragma unroll
            for (int k = 1; k <= H; ++k) {
                even.x = fmaf(s[k].x, odd_cos<L>(m * k), even.x);
                even.y = fmaf(s[k].y, odd_cos<L>(m * k), even.y);
                odd.x = fmaf(d[k].x, odd_sin<L>(m * k), odd.x);
                odd.y = fmaf(d[k].y, odd_sin<L>(m * k), odd.y);
            }
            C[k2 - 1][m] = make_float2(even.x - odd.y, even.y + odd.x);
            C[k2 - 1][L - m] = make_float2(even.x + odd.y, even.y - odd.x);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int m = 0; m < L; ++m) {
        float sum = c0[m];
#pragma unroll
        for (int k2 = 1; k2 <= H; ++k2) sum = fmaf(2.f, C[k2 - 1][m].x, sum);
        o[m][0] = sum;
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            float even = c0[m], odd = 0.f;
#pragma unroll
            for (int k2 = 1; k2 <= H; ++k2) {
                even = fmaf(2.f * C[k2 - 1][m].x, odd_cos<L>(q * k2), even);
                odd = fmaf(-2.f * C[k2 - 1][m].y, odd_sin<L>(q * k2), odd);
            }
            o[m][q] = even + odd;
            o[m][L - q] = even - odd;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The inverse through memory, for images wider than the strips below take:
// each patch's result goes to its aux slot and the seam pass adds them up.
template <int L>
__global__ __launch_bounds__(256) void oaa_inverse_kernel(const float2* __restrict__ ys,
                                                          const float* __restrict__ bias, float* __restrict__ y,
                                                          float* __restrict__ aux, int cout, int h, int w, int th,
                                                          int tw, int nt, int ntp, int relu) {
    constexpr int K = (L + 1) / 2, T = K, P = K / 2, F = stored_bins(L), G = patch_group(L);
    const int co = blockIdx.y;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= nt) return;
    const float2* src = ys + yspec_offset(co, 0, t, F, G, ntp / G);
    float2 Y[F];
#pragma unroll
    for (int f = 0; f < F; ++f) Y[f] = src[f * G];
    const int b = t % tw;
    const int rest = t / tw;
    const int a = rest % th;
    const int img = rest / th;
    float* slot = aux + (size_t(co) * ntp + t) * seam_entries(L, 1);
    float o[L][L];
    oaa_inverse_patch<L>(Y, o);
#pragma unroll
    for (int m = 0; m < L; ++m)
#pragma unroll
        for (int q = 0; q < L; ++q) {
            if (m == 0 && q == 0) {
                // the one pixel only this patch reaches: (aT + P, bT + P)
                const int r = a * T + P, cc = b * T + P;
                if (r < h && cc < w) {
                    float v = o[0][0] + (bias ? bias[co] : 0.f);
                    if (relu) v = vmax(v, 0.f);
                    y[((size_t(img) * cout + co) * h + r) * w + cc] = v;
                }
            } else {
                slot[seam_entry(m, q, L, 1)] = o[m][q];
            }
        }
}

// The inverse with the overlap-add in LDS.  A workgroup owns R patch rows of
// one plane (image, output channel), or `ni` whole planes of one channel
// where planes are small, and sums in an LDS plane of their pixels with a
// border of P on each side.  It transforms the owned patches and the patch
// rows just above and below, whose results reach P rows into its own.  Of a
// patch's L x L entries, entry (m', q') (index minus L where above L/2)
// belongs at pixel (aT + P + m', bT + P + q'): |m'|, |q'| <= P is the
// patch's own T x T tile, the rest reaches P into a neighbour's from either
// side, and as 2P < T the entries that come from one direction never meet.
// So the adds run in four passes with a barrier after each -- own tiles,
// from the left and right, from above and below, from the corners -- with no
// atomics, in an order that is the same in every run.
//
// Bound: memory (8 F bytes read per patch, the output written once).  Before,
// every entry but one went to the aux buffer and a second kernel read it
// back: 16x256x56^2 K = 5 (2304 patches, L = 9) 131 + 77 us, this kernel 52
// us (244 MB, 4.7 TB/s); 32x64x224^2 -> 64 K = 3 865 + 615 against 346 us,
// 32x512x14^2 K = 3 25 + 47 against 14 us, 1x64x224^2 K = 3 20 + 17 against
// 13 us, 8x64x56^2 K = 7 20 + 10 against 17 us.
template <int L>
__global__ __launch_bounds__(256) void oaa_inverse_strip_kernel(const float2* __restrict__ ys,
                                                                const float* __restrict__ bias,
                                                                float* __restrict__ y, int n, int cout, int h, int w,
                                                                int th, int tw, int ntp, int relu, int R, int strips,
                                                                int ni, int passes) {
    constexpr int K = (L + 1) / 2, T = K, P = K / 2, F = stored_bins(L), G = patch_group(L);
    extern __shared__ float plane[];
    const int nimg = (n + ni - 1) / ni;
    const int co = blockIdx.x / (nimg * strips);
    const int rem = blockIdx.x - co * (nimg * strips);
    const int img0 = (rem / strips) * ni, a0 = (rem % strips) * R;
    const int images = min(ni, n - img0), a1 = min(th, a0 + R);
    // patches [t0, t1): rows a0 - 1 .. a1 of one image, or whole images
    const int t0 = (img0 * th + max(a0 - 1, 0)) * tw;
    const int t1 = ((img0 + images - 1) * th + min(a1 + 1, th)) * tw;
    const int pitch = (tw * T + 2 * P) | 1, size = (R * T + 2 * P) * pitch;   // of one image's part
    const int nthreads = blockDim.x;
    for (int i = threadIdx.x; i < images * size; i += nthreads) plane[i] = 0.f;
    __syncthreads();

    for (int pass = 0; pass < passes; ++pass) {
        const int t = t0 + pass * nthreads + int(threadIdx.x);
        const bool live = t < t1;
        const int tt = live ? t : t1 - 1;
        const float2* src = ys + yspec_offset(co, 0, tt, F, G, ntp / G);
        float2 Y[F];
#pragma unroll
        for (int f = 0; f < F; ++f) Y[f] = src[f * G];
        float o[L][L];
        oaa_inverse_patch<L>(Y, o);
        // all results formed here: left to the conditional adds below, the
        // compiler keeps the sums they come from as well (189 registers
        // instead of 119 at L = 9)
#pragma unroll
        for (int m = 0; m < L; ++m)
#pragma unroll
            for (int q = 0; q < L; ++q) asm volatile("" : "+v"(o[m][q]));
        const int b = tt % tw;
        const int rest = tt / tw;
        const int a = rest % th;
        const int img = rest / th;
        const bool own = live && a >= a0 && a < a1;
        const bool up = live && a >= a0, down = live && a < a1;   // its entries above (below) its tile are in the strip
        // entry (m', q') at base[m' * pitch + q']
        float* base = plane + (img - img0) * size + ((a - a0) * T + 2 * P) * pitch + b * T + 2 * P;
        auto add = [&](auto mlo, auto mhi, auto qlo, auto qhi) __attribute__((always_inline)) {
            constexpr int M0 = decltype(mlo)::value, M1 = decltype(mhi)::value;
            constexpr int Q0 = decltype(qlo)::value, Q1 = decltype(qhi)::value;
            float v[M1 - M0 + 1][Q1 - Q0 + 1];
#pragma unroll
            for (int m = M0; m <= M1; ++m)
#pragma unroll
                for (int q = Q0; q <= Q1; ++q) v[m - M0][q - Q0] = base[m * pitch + q];
#pragma unroll
            for (int m = M0; m <= M1; ++m)
#pragma unroll
                for (int q = Q0; q <= Q1; ++q)
                    base[m * pitch + q] = v[m - M0][q - Q0] + o[m < 0 ? m + L : m][q < 0 ? q + L : q];
        };
        using std::integral_constant;
        constexpr integral_constant<int, -2 * P> lo0;
        constexpr integral_constant<int, -P - 1> lo1;
        constexpr integral_constant<int, -P> mid0;
        constexpr integral_constant<int, P> mid1;
        constexpr integral_constant<int, P + 1> hi0;
        constexpr integral_constant<int, 2 * P> hi1;
        if (own) add(mid0, mid1, mid0, mid1);
        __syncthreads();
        if (own) {
            add(mid0, mid1, lo0, lo1);
            add(mid0, mid1, hi0, hi1);
        }
        __syncthreads();
        if (up) add(lo0, lo1, mid0, mid1);
        if (down) add(hi0, hi1, mid0, mid1);
        __syncthreads();
        if (up) {
            add(lo0, lo1, lo0, lo1);
            add(lo0, lo1, hi0, hi1);
        }
        if (down) {
            add(hi0, hi1, lo0, lo1);
            add(hi0, hi1, hi0, hi1);
        }
        __syncthreads();
    }

    // The owned rows of an image are one contiguous run of the output.
    const float bv = bias ? bias[co] : 0.f;
    const int r0 = a0 * T, rows = min(h, a1 * T) - r0;
    for (int i = 0; i < images; ++i) {
        const float* from = plane + i * size + P * pitch + P;
        float* to = y + ((size_t(img0 + i) * cout + co) * h + r0) * w;
        if (w % 4 == 0) {
            const BufRsrc rout = make_rsrc(to, unsigned(rows) * unsigned(w) * 4u);
            const int w4 = w / 4;
            for (int e = threadIdx.x; e < rows * w4; e += nthreads) {
                const int r = e / w4, c = 4 * (e - r * w4);
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    v[j] = from[r * pitch + c + j] + bv;
                    if (relu) v[j] = vmax(v[j], 0.f);
                }
                buf_store_f32x4(make_float4(v[0], v[1], v[2], v[3]), rout, unsigned(e) * 16u, 0);
            }
        } else {
            for (int e = threadIdx.x; e < rows * w; e += nthreads) {
                const int r = e / w, c = e - r * w;
                float v = from[r * pitch + c] + bv;
                if (relu) v = vmax(v, 0.f);
                to[e] = v;
            }
        }
    }
}

template <int L>
static hipError_t launch_oaa_forward_L(const fftsplit_plan_s& p, const float* x, float2* xs, hipStream_t s,
                                       const LaunchEvents& ev) {
    const dim3 grid(unsigned((p.ntp + 255) / 256), unsigned(p.prob.cin));
    return launch_kernel(oaa_forward_kernel<L>, grid, dim3(256), 0, s, ev.start, ev.stop, x, xs, p.prob.cin,
                         p.prob.h, p.prob.w, p.th, p.tw, p.nt, p.ntp);
}

template <int L>
static hipError_t launch_oaa_inverse_L(const fftsplit_plan_s& p, const float2* ys, const float* bias, float* y,
                                       float* aux, hipStream_t s, const LaunchEvents& ev) {
    const OaaStrips& st = p.oaa_strips;
    if (st.blocks)
        return launch_kernel(oaa_inverse_strip_kernel<L>, dim3(unsigned(st.blocks)), dim3(unsigned(st.threads)),
                             unsigned(st.lds), s, ev.start, ev.stop, ys, bias, y, p.prob.n, p.prob.cout, p.prob.h,
                             p.prob.w, p.th, p.tw, p.ntp, int(p.relu), st.R, st.strips, st.ni, st.passes);
    const dim3 grid(unsigned((p.nt + 255) / 256), unsigned(p.prob.cout));
    hipError_t e = launch_kernel(oaa_inverse_kernel<L>, grid, dim3(256), 0, s, ev.start, nullptr, ys, bias, y, aux,
                                 p.prob.cout, p.prob.h, p.prob.w, p.th, p.tw, p.nt, p.ntp, int(p.relu));
    if (e != hipSuccess) return e;
    return launch_seam(p, aux, bias, y, s, ev.stop);
}

hipError_t launch_oaa_forward(const fftsplit_plan_s& p, const float* x, float2* xs, hipStream_t s,
                              const LaunchEvents& ev) {
    if (!p.oaa || p.T != p.prob.k) return hipErrorInvalidValue;
    switch (p.L) {
        case 5: return launch_oaa_forward_L<5>(p, x, xs, s, ev);
        case 9: return launch_oaa_forward_L<9>(p, x, xs, s, ev);
        case 13: return launch_oaa_forward_L<13>(p, x, xs, s, ev);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_oaa_inverse(const fftsplit_plan_s& p, const float2* ys, const float* bias, float* y, float* aux,
                              hipStream_t s, const LaunchEvents& ev) {
    if (!p.oaa || p.T != p.prob.k || !aux) return hipErrorInvalidValue;
    switch (p.L) {
        case 5: return launch_oaa_inverse_L<5>(p, ys, bias, y, aux, s, ev);
        case 9: return launch_oaa_inverse_L<9>(p, ys, bias, y, aux, s, ev);
        case 13: return launch_oaa_inverse_L<13>(p, ys, bias, y, aux, s, ev);
    }
    return hipErrorInvalidValue;
}

}  // namespace fftsplit
