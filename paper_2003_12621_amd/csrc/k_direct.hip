// Direct spatial cross-correlation on the fp32 matrix cores: the spatial
// convolution the paper compares the split method against (Section 2,
// eq. 1; Section 4, Table 1 and Fig. 4).
//
//     y[n][co][p] = b[co] + sum_{ci, u, v} w[co][ci][u][v] * x[n][ci][py + u - P][px + v - P]
//
// as an implicit GEMM: rows = output channels, columns = output pixels
// (flattened over image, row, column), reduction over (u, v, ci).  The
// filters are rearranged once per layer into Wd[u][v][ci16][coutp]
// (direct_weights_kernel), so that a stage of 16 input channels of one tap
// (u, v) is a contiguous 16 x 64 block; the input operand of a stage is
// gathered from x with the tap's shift, zero outside the image.
//
// Workgroup tile: 64 output channels x 64 pixels, 4 waves of 32 x 32, one
// v_mfma_f32_32x32x2_f32 per two input channels (operand layout as in the
// contraction kernel).  Stages are double-buffered through registers and
// LDS: the next stage's loads are in flight while the current one is
// multiplied.  Bias and ReLU are applied in the epilogue.
#include "bf16_split.hpp"
#include "fftsplit_internal.hpp"
#include "launch_util.hpp"

namespace fftsplit {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kDirBM = 64, kDirBN = 64, kDirKC = 16;

// w [cout][cin][k][k] -> Wd[k*k][cin16][coutp], zero for padded channels.
__global__ __launch_bounds__(256) void direct_weights_kernel(const float* __restrict__ w, float* __restrict__ wd,
                                                             int cin, int cout, int cin16, int coutp, int kk) {
    const size_t total = size_t(kk) * cin16 * coutp;
    const size_t idx = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int co = int(idx % coutp);
    const size_t rest = idx / coutp;
    const int ci = int(rest % cin16);
    const int uv = int(rest / cin16);
    wd[idx] = (co < cout && ci < cin) ? w[(size_t(co) * cin + ci) * kk + uv] : 0.f;
}

__global__ __launch_bounds__(256) void direct_kernel(const float* __restrict__ x, const float* __restrict__ wd,
                                                     const float* __restrict__ bias, float* __restrict__ y, int n,
                                                     int cin, int h, int w, int cout, int coutp, int k, int relu,
                                                     unsigned x_bytes, int nbco, int npix) {
    constexpr int BM = kDirBM, BN = kDirBN, KC = kDirKC, NT = 256;
    __shared__ float lds[2][KC * (BM + BN)];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int cbk = lb % nbco;
    const int pbk = lb / nbco;
    const int co0 = cbk * BM;
    const int p0 = pbk * BN;
    const int P = k / 2;
    const int hw = h * w;
    const int cin16 = (cin + KC - 1) / KC * KC;
    const int nchunk = cin16 / KC;
    const int nstage = k * k * nchunk;

    // B loads: thread -> (row kr = tid / 16, 4 consecutive pixels at 4 * (tid % 16))
    const int kr = tid >> 4;
    const int pj = (tid & 15) * 4;
    int pimg[4], py[4], px[4];
    bool pok[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int p = p0 + pj + e;
        pok[e] = p < npix;
        const int pp = pok[e] ? p : 0;
        pimg[e] = pp / hw;
        const int r = pp - pimg[e] * hw;
        py[e] = r / w;
        px[e] = r - py[e] * w;
    }
    const BufRsrc rxs = make_rsrc(x, x_bytes);
    // A loads: thread -> (row tid / 16, 4 consecutive channels at 4 * (tid % 16))
    const float* wsrc = wd + co0 + (tid & 15) * 4;

    float4 areg;
    float breg[4];
    auto load_stage = [&](int s) {
        const int uv = s / nchunk;
        const int c0 = (s - uv * nchunk) * KC;
        const int u = uv / k, v = uv - u * k;
        areg = *reinterpret_cast<const float4*>(wsrc + (size_t(uv) * cin16 + c0 + kr) * coutp);
        const int ci = c0 + kr;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int yy = py[e] + u - P, xx = px[e] + v - P;
            const bool ok = pok[e] && ci < cin && unsigned(yy) < unsigned(h) && unsigned(xx) < unsigned(w);
            const unsigned off = ok ? unsigned(((pimg[e] * cin + ci) * h + yy) * w + xx) * 4u : kOutOfRange;
            breg[e] = buf_load_f32(rxs, off, 0);
        }
    };
    auto store_stage = [&](int buf) {
        *reinterpret_cast<float4*>(&lds[buf][kr * BM + (tid & 15) * 4]) = areg;
        *reinterpret_cast<float4*>(&lds[buf][KC * BM + kr * BN + pj]) =
            make_float4(breg[0], breg[1], breg[2], breg[3]);
    };

    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const int krow = lane >> 5;
    const int col = lane & 31;

    load_stage(0);
    store_stage(0);
    __syncthreads();
    for (int s = 0; s < nstage; ++s) {
        const int buf = s & 1;
        if (s + 1 < nstage) load_stage(s + 1);
        const float* sa = &lds[buf][krow * BM + wm * 32 + col];
        const float* sb = &lds[buf][KC * BM + krow * BN + wn * 32 + col];
        float a[KC / 2], b[KC / 2];
#pragma unroll
        for (int kp = 0; kp < KC / 2; ++kp) {
            a[kp] = sa[2 * kp * BM];
            b[kp] = sb[2 * kp * BN];
        }
#pragma unroll
        for (int kp = 0; kp < KC / 2; ++kp) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[kp], b[kp], acc, 0, 0, 0);
        if (s + 1 < nstage) store_stage(buf ^ 1);
        __syncthreads();
    }

    // epilogue: D[i][j], register r: i = 8 (r / 4) + 4 krow + r % 4, j = col
    const int p = p0 + wn * 32 + col;
    if (p < npix) {
        const int img = p / hw;
        const int rem = p - img * hw;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int co = co0 + wm * 32 + 8 * (r >> 2) + 4 * krow + (r & 3);
            if (co < cout) {
                float v = acc[r] + (bias ? bias[co] : 0.f);
                if (relu) v = vmax(v, 0.f);
                y[(size_t(img) * cout + co) * hw + rem] = v;
            }
        }
    }
}

// The same convolution on the bf16 matrix instruction (bf16_split.hpp), for
// filters up to 13 x 13: an fp32 result from six part products per product.
// A workgroup owns NW * 64 output channels x 64 pixels (a th x tw block of
// one image), a wave 64 x 64.  Per group of 32 input channels the block's
// pixels and their halo are split once into LDS, part by part and octet of
// channels by octet ([part][octet][pixel], 16 bytes: the B operand of a
// reduction step of 32 channels, 16 lanes of neighbouring pixels reading
// neighbouring 16 bytes), and all K * K taps read them there at shifted
// addresses.  The filter operand (channels 8 quad + 0..7 of rows 4 col + 0..3:
// eight 16-byte loads of the re-laid filters, one tap ahead) is split in
// registers: 208 vector instructions against 96 matrix instructions of 16
// cycles, which two waves per SIMD overlap.  Pixels and filters are scaled
// before they are split (bf16_split.hpp), and a wave whose sums are not all
// finite computes its block again on the fp32 instruction, in direct_kernel's
// order.
// Bound: the matrix cores (clock 2.0 GHz under them) and the vector work
// beside them.  16x256x56^2 -> 256, K = 5: 1761 us on the fp32 instruction,
// 973 us here (169 TFLOP/s of the convolution's operations; 955 without the
// scale); 8x128x112^2 K = 3 324 -> 209 us, 32x512x28^2 1264 -> 728 us.  Error
// against float64 1.0e-6 -> 2.8e-7 on the first: each tap's 32 channels are
// summed from zero and added in fp32 (with the running sum in the matrix unit it
// was 1.2e-6, 5 % faster).
template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void direct_split_kernel(
    const float* __restrict__ x, const float* __restrict__ wd, const float* __restrict__ bias, float* __restrict__ y,
    int cin, int h, int w, int cout, int coutp, int k, int relu, unsigned x_bytes, int nbco, int tiles_h, int tiles_w,
    int ltw, unsigned y_bytes) {
    constexpr int NT = 64 * NW;
    extern __shared__ float4 lds_raw[];
    u32x4* const lds = reinterpret_cast<u32x4*>(lds_raw);   // [part][octet][pixel]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int quad = lane >> 4, col = lane & 15;

    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int pbk = __builtin_amdgcn_readfirstlane(lb / nbco);
    const int co0 = (__builtin_amdgcn_readfirstlane(lb) - pbk * nbco) * NT + wave * 64;
    const int img = __builtin_amdgcn_readfirstlane(pbk / (tiles_h * tiles_w));
    const int tile = pbk - img * tiles_h * tiles_w;
    const int trow = __builtin_amdgcn_readfirstlane(tile / tiles_w);
    const int tw = 1 << ltw, th = 64 >> ltw;
    const int r0 = trow * th, c0 = (tile - trow * tiles_w) * tw;

    const int P = k / 2, hw = h * w;
    const int pitch = tw + 2 * P, npx = (th + 2 * P) * pitch;
    const int cin16 = (cin + kDirKC - 1) / kDirKC * kDirKC;
    const BufRsrc rx = make_rsrc(x, x_bytes);

    floatx4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[i][n] = floatx4{0.f, 0.f, 0.f, 0.f};

    // LDS index of this lane's pixel of column block n, at tap (0, 0)
    int pb[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int p = 16 * n + col;
        pb[n] = (p >> ltw) * pitch + (p & (tw - 1)) + quad * npx;
    }
    const int part = 4 * npx;

    // this lane's filter rows: channels c + 8 quad + 0..7 of a tap.  In a last
    // group of 16 channels the upper quads, whose pixels are zero, read the
    // lower ones' rows.
    float4 av[8];
    auto load_a = [&](int uv, int c) __attribute__((always_inline)) {
        const int q = c + 32 <= cin16 ? quad : quad & 1;
        const float* src = wd + (size_t(uv) * cin16 + c) * coutp + co0 + unsigned(8 * q) * unsigned(coutp) + 4 * col;
#pragma unroll
        for (int j = 0; j < 8; ++j) av[j] = *reinterpret_cast<const float4*>(src + size_t(j) * coutp);
    };

    for (int c = 0; c < cin16; c += 32) {
        load_a(0, c);
        __syncthreads();   // the pixels of the group before are no longer read
        for (int e = tid; e < 4 * npx; e += NT) {
            const int oct = e / npx, px = e - oct * npx;
            const int hr = px / pitch;
            const int yy = r0 + hr - P, xx = c0 + (px - hr * pitch) - P;
            const bool ok = unsigned(yy) < unsigned(h) && unsigned(xx) < unsigned(w);
            const int ch = c + 8 * oct;
            const unsigned off = unsigned((img * cin + ch) * hw + yy * w + xx) * 4u;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j] = buf_load_f32(rx, ok && ch + j < cin ? off + unsigned(j * hw) * 4u : kOutOfRange, 0);
            u32x4 s[3];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                unsigned p[3];
                split3(v[2 * d] * kSplitScale, v[2 * d + 1] * kSplitScale, p);
#pragma unroll
                for (int q = 0; q < 3; ++q) s[q][d] = p[q];
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) lds[q * part + e] = s[q];
        }
        __syncthreads();
        int u = 0, v = 0;
        for (int uv = 0; uv < k * k; ++uv) {
            u32x4 a[3][4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const float* e0 = &av[2 * d].x;
                const float* e1 = &av[2 * d + 1].x;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    unsigned p[3];
                    split3(e0[i] * kSplitScale, e1[i] * kSplitScale, p);
#pragma unroll
                    for (int q = 0; q < 3; ++q) a[q][i][d] = p[q];
                }
            }
            if (uv + 1 < k * k) load_a(uv + 1, c);
            const u32x4* src = lds + (u * pitch + v);
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                u32x4 b[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) b[q] = src[q * part + pb[n]];
                // the tap's 32 channels from zero, then one fp32 addition: the
                // matrix unit's rounding of a running sum is coarser than that
                floatx4 t[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) t[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[i] = mfma_bf16(a[kSplitA[q]][i], b[kSplitB[q]], t[i]);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i][n] += t[i];
            }
            if (++v == k) {
                v = 0;
                ++u;
            }
        }
    }

    const BufRsrc ry = make_rsrc(y, y_bytes);
    // byte offset of pixel p (0..63) of the block in channel 0, or out of range
    auto pixel = [&](int p) __attribute__((always_inline)) {
        const int yy = r0 + (p >> ltw), xx = c0 + (p & (tw - 1));
        return yy < h && xx < w ? unsigned(img * cout * hw + yy * w + xx) * 4u : kOutOfRange;
    };
    auto store = [&](float v, int co, unsigned px) __attribute__((always_inline)) {
        v += bias && co < cout ? bias[co] : 0.f;
        if (relu) v = vmax(v, 0.f);
        buf_store_f32(v, ry, co < cout && px != kOutOfRange ? px + unsigned(co * hw) * 4u : kOutOfRange, 0);
    };
    if (all_finite(acc)) {
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const unsigned px = pixel(16 * n + col);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) store(acc[i][n][r] * kSplitUnscale, co0 + 4 * (4 * quad + r) + i, px);
        }
        return;
    }
    const int krow = lane >> 5, l32 = lane & 31;
    for (int blk = 0; blk < 4; ++blk) {
        const int cb = co0 + (blk >> 1) * 32, p = (blk & 1) * 32 + l32;
        const int yy = r0 + (p >> ltw), xx = c0 + (p & (tw - 1));
        floatx16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        for (int uv = 0; uv < k * k; ++uv) {
            const int ry0 = yy + uv / k - P, rx0 = xx + uv % k - P;
            const bool ok = unsigned(ry0) < unsigned(h) && unsigned(rx0) < unsigned(w);
            for (int c = krow; c < cin16; c += 2) {
                const float a = wd[(size_t(uv) * cin16 + c) * coutp + cb + l32];
                const float b = buf_load_f32(rx, ok && c < cin ? unsigned(((img * cin + c) * h + ry0) * w + rx0) * 4u : kOutOfRange, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, s, 0, 0, 0);
            }
        }
        const unsigned px = pixel(p);
#pragma unroll
        for (int r = 0; r < 16; ++r) store(s[r], cb + 8 * (r >> 2) + 4 * krow + (r & 3), px);
    }
}

size_t direct_wspec_bytes(const fftsplit_plan_s& p) {
    return size_t(p.prob.k) * p.prob.k * round_up_block(p.prob.cin) * p.coutp * 4;
}

hipError_t launch_direct_weights(const fftsplit_plan_s& p, const float* w, float* wd, hipStream_t s) {
    const int kk = p.prob.k * p.prob.k;
    const size_t total = size_t(kk) * round_up_block(p.prob.cin) * p.coutp;
    const unsigned blocks = unsigned((total + 255) / 256);
    hipLaunchKernelGGL(direct_weights_kernel, dim3(blocks), dim3(256), 0, s, w, wd, p.prob.cin, p.prob.cout,
                       round_up_block(p.prob.cin), p.coutp, kk);
    return hipGetLastError();
}

template <int NW>
static hipError_t launch_direct_split(const fftsplit_plan_s& p, const float* x, const float* wd, const float* bias,
                                      float* y, hipStream_t s, const LaunchEvents& ev, int ltw, int lds) {
    auto kern = direct_split_kernel<NW>;
    // the most that the plan's rule takes, not this filter's: plans of other
    // filters may launch at the same time
    const hipError_t attr = allow_dynamic_lds(kern, lds > 64 * 1024 ? 80 * 1024 : lds);
    if (attr != hipSuccess) return attr;
    const int tw = 1 << ltw, th = 64 >> ltw;
    const int tiles_h = (p.prob.h + th - 1) / th, tiles_w = (p.prob.w + tw - 1) / tw;
    const int nbco = p.coutp / (64 * NW);
    const size_t hw = size_t(p.prob.h) * p.prob.w;
    const size_t nb = size_t(p.prob.n) * tiles_h * tiles_w * nbco;
    return launch_kernel(kern, dim3(unsigned(nb)), dim3(64 * NW), unsigned(lds), s, ev.start, ev.stop, x, wd, bias, y,
                         p.prob.cin, p.prob.h, p.prob.w, p.prob.cout, p.coutp, p.prob.k, int(p.relu),
                         unsigned(p.prob.n * p.prob.cin * hw * 4), nbco, tiles_h, tiles_w, ltw,
                         unsigned(p.prob.n * p.prob.cout * hw * 4));
}

hipError_t launch_direct(const fftsplit_plan_s& p, const float* x, const float* wd, const float* bias, float* y,
                         hipStream_t s, const LaunchEvents& ev) {
    const int npix = p.prob.n * p.prob.h * p.prob.w;
    if (p.dir_ltw) {
        const int halo = p.prob.k / 2 * 2;
        const int lds = 3 * 64 * ((64 >> p.dir_ltw) + halo) * ((1 << p.dir_ltw) + halo);
        if (p.coutp % 256 == 0) return launch_direct_split<4>(p, x, wd, bias, y, s, ev, p.dir_ltw, lds);
        if (p.coutp % 128 == 0) return launch_direct_split<2>(p, x, wd, bias, y, s, ev, p.dir_ltw, lds);
        return launch_direct_split<1>(p, x, wd, bias, y, s, ev, p.dir_ltw, lds);
    }
    const int nbco = p.coutp / kDirBM;
    const int nbp = (npix + kDirBN - 1) / kDirBN;
    const unsigned x_bytes = unsigned(size_t(p.prob.n) * p.prob.cin * p.prob.h * p.prob.w * 4);
    return launch_kernel(direct_kernel, dim3(unsigned(nbco) * unsigned(nbp)), dim3(256), 0, s, ev.start, ev.stop, x,
                         wd, bias, y, p.prob.n, p.prob.cin, p.prob.h, p.prob.w, p.prob.cout, p.coutp, p.prob.k,
                         int(p.relu), x_bytes, nbco, npix);
}

}  // namespace fftsplit
