// Per-frequency-bin channel contraction on the bf16 matrix instruction with
// fp32 results (the same product, layouts and grid order as contract_kernel in
// k_contract.hip): for every stored bin f,
//     Y[f][co][t] = sum_ci W[f][ci][co] * X[f][ci][t]        (complex).
//
// Each fp32 operand is split exactly into three bf16 parts and a product
// takes six part products (bf16_split.hpp), so a channel block's 16 products
// are six matrix instructions.  Their rounding of the running sum is coarser
// than a vector addition's: with that sum as their addend throughout, the
// error against float64 was up to 30 % above the fp32 kernel's on a network's
// activations (positive, correlated; below it on others).  In the last 3/8 of
// the channels, where the sum is large, a block is therefore summed from zero
// and then added in fp32.  Error over the layers of a VGG-16 stack at batch 1, 4
// and 32, against the fp32 kernel's: 0.39-0.81 of it (0.67-0.96 with (re, im)
// pairs along the reduction, see below, and then 0.36-0.70 with every block from
// zero, 4-8 % slower).  Operands are scaled by a power of two, so
// that no part underflows, and a wave whose sums are not all finite computes its
// tile again on the fp32 instruction, with contract_kernel's products and order
// (bf16_split.hpp): infinities and NaN come out as there.
//
// The complex product is real along the matrix instruction's reduction, where a
// lane's four channels c are four dwords, each a pair of channels:
//     filter operand            (Wr01, Wr23, Wi01, Wi23)
//     patch operand for Re Y    (Xr01, Xr23, -Xi01, -Xi23)
//     patch operand for Im Y    (Xi01, Xi23, Xr01, Xr23),
// so the patch parts are converted once and only negated (one bit operation a
// pair) for Re Y, whose operand overlaps the other one's registers.  A reduction
// step of v_mfma_f32_16x16x32_bf16 is 16 input channels, one channel block.
// Operand layout (64 lanes, lane l):
//     A[i][k]: i = l % 16, k = 8 (l / 16) + 0..7     (channels 4 (l / 16) + 0..3)
//     B[k][j]: j = l % 16, likewise
//     D[i][j], register r: i = 4 (l / 16) + r, j = l % 16.
// Rows and columns go to lanes in neighbouring pairs (row 32 p + 2 (l % 16)
// + e is element l % 16 of block 2 p + e), so one 16-byte LDS read serves two
// blocks and an output row is written in 16-byte pairs of patches.
//
// A workgroup tile is BM channels x BN patches of one bin, wave tiles of
// 16 TM x 16 TN; channel blocks are loaded one ahead straight into LDS as
// fp32 and split after the LDS read.  At 64 x 64 a wave issues 440 vector
// instructions of splits, 64 of them for the scale (and 128 additions where a
// block is summed from zero), beside 192 matrix instructions of 16 cycles per
// channel block; two waves per SIMD overlap them in part.  (With (re, im) dwords
// the patch parts were converted twice, 96 of 192 conversions: 32x512x28^2 187
// us, in channel pairs 176; 16x256x56^2 K=5 105, 100.)  With KG > 1, KG wave
// groups take the channel blocks in turn and add their sums through LDS: more
// waves on a compute unit that has one workgroup (small grids, where a wave's
// chain of LDS read, split and product is what takes the time).
//
// What bounds it (MI355X): the matrix cores, whose clock falls to 2.0 GHz
// under it (2.4 under the fp32 kernel; a loop of the instruction alone
// reaches 1745 TFLOP/s at 32x32x16 and 2040 at 16x16x32, hence that shape),
// then the vector work and, with few patches, HBM.  Against the fp32 kernel,
// whole launches in us (algorithmic rate at 8 flops per complex product; one
// run, other boxes are up to 10 % slower):
//     32x256x56^2, 512 patches            214 -> 158  (161 -> 217 TFLOP/s)
//     32x512x28^2, 128 patches            207 -> 160
//     32x128x112^2, 2048 patches          228 -> 162
//     16x256x56^2 K=5, 64 patches         112 ->  93  (4.3 TB/s)
//     32x64x224^2, 8192 patches           254 -> 206  (5.2 TB/s)
//     1x512x28^2 at L = 8, 25 patches      36 ->  25
// Tried without gain: the vector work interleaved with the matrix
// instructions by the scheduler instead of two waves overlapping, two and three
// stages ahead, and a priority for one of a compute unit's two workgroups.
#include "bf16_split.hpp"
#include "fftsplit_internal.hpp"
#include "launch_util.hpp"

#include <type_traits>

namespace fftsplit {

// Waits until no vector memory instruction and no LDS read is outstanding, then
// passes the workgroup's barrier.  One block, so that nothing the wave reads
// from LDS before it can still be in flight after it.
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 16 bytes per lane from uniform base + lane offset straight into LDS: lane
// l writes LDS bytes [lds + 16 l, lds + 16 l + 16).  Inline assembly because
// for the builtin the compiler waits for every outstanding load before each
// LDS read; the caller waits (s_waitcnt vmcnt) before the barrier that
// publishes a buffer.  The wait states cover a base that a vector
// instruction wrote just before (five before a memory instruction reads it)
// and the M0 write (one).
template <bool NT>
__device__ __forceinline__ void split_dma16(uint64_t base, unsigned voff, const void* lds_wave_base) {
    const unsigned m0 = __builtin_amdgcn_readfirstlane(unsigned(reinterpret_cast<uintptr_t>(lds_wave_base)));
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base), "s"(m0)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(m0)
                     : "memory", "m0");
}

// The lane's number, computed anew: what only the rare paths and the epilogue
// need of it is not held in registers through the loop.
__device__ __forceinline__ int fresh_lane() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// A 64-bit address that is the same in every lane, in scalar registers.
// (readfirstlane returns a signed int: through unsigned, or the low word's
// sign would overwrite the high word)
__device__ __forceinline__ uint64_t uniform_address(const void* p) {
    const uint64_t a = reinterpret_cast<uintptr_t>(p);
    const unsigned lo = unsigned(__builtin_amdgcn_readfirstlane(int(unsigned(a))));
    const unsigned hi = unsigned(__builtin_amdgcn_readfirstlane(int(unsigned(a >> 32))));
    return uint64_t(lo) | uint64_t(hi) << 32;
}

template <int BM, int BN, int TM, int TN>
struct SplitShape {
    static constexpr int KC = kChanBlock;   // a stage is one channel block = one reduction step
    static constexpr int WM = BM / (16 * TM), WN = BN / (16 * TN);   // waves
    static constexpr int NT = 64 * WM * WN;
    static constexpr int WE = KC * BM, XE = KC * BN;           // stage elements (complex)
    static constexpr int WL = WE / 2 / NT, XL = XE / 2 / NT;   // 16-byte loads per thread and stage
    static constexpr int STAGE = WE + XE;
    static constexpr int WROWS = NT / (BM / 2), XROWS = NT / (BN / 2);   // rows per load
    static_assert(TM % 2 == 0 && TN % 2 == 0, "row and column pairs");
    static_assert(WL * NT * 2 == WE && XL * NT * 2 == XE, "loads divide evenly");
    static_assert(NT % (BM / 2) == 0 && NT % (BN / 2) == 0, "whole rows per load");
};

template <int BM, int BN, int TM, int TN, int KG, bool WS, bool XS>
__global__ __launch_bounds__((KG * SplitShape<BM, BN, TM, TN>::NT), 2) void contract_split_kernel(
    const float2* __restrict__ xs, const float2* __restrict__ ws, float2* __restrict__ ys, int cin, int coutp, int ntp,
    int nt, int nbco, int nbt, int nbins, int ygroup, int npacked) {
    using S = SplitShape<BM, BN, TM, TN>;
    constexpr int KC = S::KC;
    constexpr int NT = S::NT;             // threads of a group
    extern __shared__ float4 lds_raw[];   // two stage buffers for each group

    const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(int(threadIdx.x) / NT);
    const int tid = int(threadIdx.x) - group * NT;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / S::WN, wn = wave % S::WN;
    const int quad = lane >> 4, col = lane & 15;

    // (bin, patch block, channel block), channel blocks fastest, the bins
    // dealt to the XCDs in turn (as contract_kernel)
    const int per_bin = nbco * nbt;
    int lb;
    if (int(gridDim.x) % (kNumXcd * per_bin) == 0) {
        const int x = int(blockIdx.x) % kNumXcd, j = int(blockIdx.x) / kNumXcd;
        lb = ((j / per_bin) * kNumXcd + x) * per_bin + j % per_bin;
    } else {
        lb = xcd_logical_block(blockIdx.x, gridDim.x);
    }
    const int rest = lb / nbco;
    const int co0 = (lb - rest * nbco) * BM;
    const int f = rest / nbt;
    const int t0 = (rest - f * nbt) * BN;

    // this lane's 16 bytes of a load: row tid / (B / 2) of the rows it covers
    const unsigned wrow = unsigned(coutp) * 8u, xrow = unsigned(ntp) * 8u;
    const unsigned wvoff = unsigned(tid / (BM / 2)) * wrow + unsigned(tid % (BM / 2)) * 16u;
    const unsigned xvoff = unsigned(tid / (BN / 2)) * xrow + unsigned(tid % (BN / 2)) * 16u;
    const uint64_t wbase = uniform_address(ws + size_t(f) * cin * coutp + co0);
    const uint64_t xbase = uniform_address(xs + spec_offset(0, f, t0, nbins, ntp));
    const uint64_t xblock = uint64_t(unsigned(nbins)) * xrow;   // bytes from a channel block to the next, per channel

    float2* const lds = reinterpret_cast<float2*>(lds_raw) + group * (2 * S::STAGE);
    // Channel block s into `stage`.  In a partial last one the missing rows
    // are read from the last row (in range); the filter's are zeroed before
    // they are used (below), so that what the patch rows hold does not count.
    auto dma_stage = [&](int s, float2* stage) __attribute__((always_inline)) {
        uint4* sw = reinterpret_cast<uint4*>(stage) + wave * 64;
        uint4* sx = reinterpret_cast<uint4*>(stage + S::WE) + wave * 64;
        const int k0 = s * KC, last = cin - 1 - k0;
        const uint64_t wb = wbase + uint64_t(unsigned(k0)) * wrow, xb = xbase + uint64_t(unsigned(k0)) * xblock;
        if (last >= KC - 1) {
#pragma unroll
            for (int i = 0; i < S::WL; ++i) split_dma16<WS>(wb + uint64_t(i * S::WROWS) * wrow, wvoff, sw + i * NT);
#pragma unroll
            for (int i = 0; i < S::XL; ++i) split_dma16<XS>(xb + uint64_t(i * S::XROWS) * xrow, xvoff, sx + i * NT);
        } else {
            const int tid = 64 * wave + fresh_lane();
#pragma unroll
            for (int i = 0; i < S::WL; ++i) {
                const int c = i * S::WROWS + tid / (BM / 2);
                split_dma16<WS>(wb, wvoff + unsigned(min(c, last) - tid / (BM / 2)) * wrow, sw + i * NT);
            }
#pragma unroll
            for (int i = 0; i < S::XL; ++i) {
                const int c = i * S::XROWS + tid / (BN / 2);
                split_dma16<XS>(xb, xvoff + unsigned(min(c, last) - tid / (BN / 2)) * xrow, sx + i * NT);
            }
        }
    };

    // One stage (16 channels = one reduction step).  Lane (quad, col) holds
    // channels 4 quad + 0..3 of rows (columns) 32 p + 2 col + 0, 1 of the
    // wave's tile, one 16-byte LDS read per channel and pair; the filter
    // parts of the whole tile stay in registers, the patch parts are made a
    // column block at a time.
    auto multiply = [&](const float2* stage, floatx4 (&accR)[TM][TN], floatx4 (&accI)[TM][TN], auto packed, auto fresh) __attribute__((always_inline)) {
        const float2* sw = stage + (4 * quad) * BM + wm * (16 * TM) + 2 * col;
        const float2* sx = stage + S::WE + (4 * quad) * BN + wn * (16 * TN) + 2 * col;
        u32x4 a[3][TM];
#pragma unroll
        for (int p = 0; p < TM / 2; ++p)
#pragma unroll
            for (int c = 0; c < 4; c += 2) {
                const float4 u = *reinterpret_cast<const float4*>(sw + c * BM + 32 * p);
                const float4 v = *reinterpret_cast<const float4*>(sw + (c + 1) * BM + 32 * p);
                unsigned re[2][3], im[2][3];
                split3(u.x * kSplitScale, v.x * kSplitScale, re[0]);
                split3(u.y * kSplitScale, v.y * kSplitScale, im[0]);
                split3(u.z * kSplitScale, v.z * kSplitScale, re[1]);
                split3(u.w * kSplitScale, v.w * kSplitScale, im[1]);
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        a[q][2 * p + e][c / 2] = re[e][q];
                        a[q][2 * p + e][2 + c / 2] = im[e][q];
                    }
            }
#pragma unroll
        for (int p = 0; p < TN / 2; ++p) {
            float4 v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = *reinterpret_cast<const float4*>(sx + c * BN + 32 * p);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int j = 2 * p + e;
                // (im, re, -im) of both channel pairs; in a slot of two real
                // bins (0, re, 0) and (0, im)
                u32x8 x[3];
                u32x4 br[3], bi[3];
#pragma unroll
                for (int c = 0; c < 4; c += 2) {
                    unsigned re[3], im[3];
                    split3((e ? v[c].z : v[c].x) * kSplitScale, (e ? v[c + 1].z : v[c + 1].x) * kSplitScale, re);
                    split3((e ? v[c].w : v[c].y) * kSplitScale, (e ? v[c + 1].w : v[c + 1].y) * kSplitScale, im);
                    constexpr bool two_real = decltype(packed)::value;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        x[q][c / 2] = two_real ? 0u : im[q];
                        x[q][2 + c / 2] = re[q];
                        x[q][4 + c / 2] = two_real ? 0u : im[q] ^ 0x80008000u;
                        x[q][6 + c / 2] = im[q];
                    }
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    bi[q] = decltype(packed)::value ? __builtin_shufflevector(x[q], x[q], 0, 1, 6, 7)
                                                    : __builtin_shufflevector(x[q], x[q], 0, 1, 2, 3);
                    br[q] = __builtin_shufflevector(x[q], x[q], 2, 3, 4, 5);
                }
                // Smallest part products first; `fresh`: the block's sum from
                // zero, then one fp32 addition.
                auto add = [&](const u32x4 (&b)[3], floatx4 (&acc)[TM][TN]) __attribute__((always_inline)) {
                    constexpr bool F = decltype(fresh)::value;
                    floatx4 t[TM];
#pragma unroll
                    for (int i = 0; i < TM; ++i) t[i] = F ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[i][j];
#pragma unroll
                    for (int q = 0; q < 6; ++q)
#pragma unroll
                        for (int i = 0; i < TM; ++i) t[i] = mfma_bf16(a[kSplitA[q]][i], b[kSplitB[q]], t[i]);
#pragma unroll
                    for (int i = 0; i < TM; ++i) acc[i][j] = F ? acc[i][j] + t[i] : t[i];
                };
                add(br, accR);
                add(bi, accI);
            }
        }
    };

    // (a block of padding patches only has zero spectra: no stages)
    const int nstage = t0 < nt ? (cin + KC - 1) / KC : 0;
    // The group's stage of iteration it (channel block it * KG + group).
    auto buffer = [&](int it) __attribute__((always_inline)) { return lds + (it & 1) * S::STAGE; };
    auto load_stage = [&](int it) __attribute__((always_inline)) {
        const int s = it * KG + group;
        if (s < nstage) dma_stage(s, buffer(it));
    };
    // Stores the wave's sums and tells whether they are finite (bf16_split.hpp).
    auto run = [&](auto packed) __attribute__((always_inline)) {
        floatx4 accR[TM][TN], accI[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) accR[i][j][r] = accI[i][j][r] = 0.f;

        load_stage(0);
        const int nit = (nstage + KG - 1) / KG;
        auto iterations = [&](int it, int end, auto fresh) __attribute__((always_inline)) {
            for (; it < end; ++it) {
                // past the wait and the barrier this iteration's stage is
                // there, and every wave has finished with the buffer of the
                // iteration before, which the next one's stage then fills
                const int s = it * KG + group;
                wait_and_barrier();
                load_stage(it + 1);
                float2* const cur = buffer(it);
                if (it == nit - 1 && cin % KC != 0) {
                    // the partial block's missing filter rows (only its own
                    // group's; the barrier is everyone's)
                    const int last = cin - 1 - s * KC, tid = 64 * wave + fresh_lane();
#pragma unroll
                    for (int i = 0; i < S::WL; ++i)
                        if (i * S::WROWS + tid / (BM / 2) > last)
                            reinterpret_cast<uint4*>(cur)[i * NT + tid] = make_uint4(0, 0, 0, 0);
                    __syncthreads();
                }
                if (KG == 1 || s < nstage) multiply(cur, accR, accI, packed, fresh);
            }
        };
        // The first 5/8 of the channels are added by the matrix instructions
        // themselves, the rest from zero (see above): a step's error grows
        // with the sum, so that part holds about half of the squared error.
        // Wave groups' sums are short enough without.
        const int direct = KG > 1 ? nit : nit * 5 / 8;
        iterations(0, direct, std::false_type{});
        if constexpr (KG == 1) iterations(direct, nit, std::true_type{});
        if constexpr (KG > 1) {
            // the groups' partial sums, through LDS to the first group
            constexpr int NA = 2 * TM * TN;
            const int tid = 64 * wave + fresh_lane();
            floatx4* part = reinterpret_cast<floatx4*>(lds_raw) + tid;
            __syncthreads();
            if (group > 0) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        part[((group - 1) * NA + 2 * (i * TN + j)) * NT] = accR[i][j];
                        part[((group - 1) * NA + 2 * (i * TN + j) + 1) * NT] = accI[i][j];
                    }
            }
            __syncthreads();
            if (group > 0) return true;
#pragma unroll
            for (int g = 0; g < KG - 1; ++g)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        accR[i][j] += part[(g * NA + 2 * (i * TN + j)) * NT];
                        accI[i][j] += part[(g * NA + 2 * (i * TN + j) + 1) * NT];
                    }
        }

        const int lane = fresh_lane(), quad = lane >> 4, col = lane & 15;
        // Output spectra (patch-group-major): D register r of lane (quad,
        // col) is row 4 quad + r, column col of its 16 x 16 block, so a lane
        // holds pairs of neighbouring patches: 16-byte stores, 16 lanes a row.
        const unsigned cs8 = unsigned(nbins) * unsigned(ntp) * 8u;   // next channel
        const BufRsrc ry = make_rsrc(ys + size_t(co0) * nbins * ntp, unsigned(size_t(coutp - co0) * cs8));
        const unsigned row8 = unsigned(wm * (16 * TM) + 8 * quad) * cs8;
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
            const int t = t0 + wn * (16 * TN) + 16 * j + 2 * col;
            const unsigned voff = row8 + unsigned(yspec_offset(0, f, t, nbins, ygroup, ntp / ygroup)) * 8u;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    buf_store_f32x4(make_float4(accR[i][j][r] * kSplitUnscale, accI[i][j][r] * kSplitUnscale,
                                                accR[i][j + 1][r] * kSplitUnscale, accI[i][j + 1][r] * kSplitUnscale), ry,
                                    voff, unsigned(32 * (i / 2) + 2 * r + i % 2) * cs8);
        }
        return all_finite(accR) && all_finite(accI);
    };
    // one loop for each kind of bin (a branch inside the loop would merge the
    // accumulators of its two sides by copies)
    const bool two_real = f >= nbins - npacked;
    if (two_real ? run(std::true_type{}) : run(std::false_type{})) return;

    // The wave's tile again on the fp32 instruction, operands from memory: the
    // products and the order of contract_kernel with three real products.  It
    // takes the place of what was stored.
    __builtin_amdgcn_s_waitcnt(0);
    const int krow = fresh_lane() >> 5, l32 = fresh_lane() & 31;
    for (int blk = 0; blk < (TM / 2) * (TN / 2); ++blk) {
        const int co = co0 + wm * (16 * TM) + blk / (TN / 2) * 32, t = t0 + wn * (16 * TN) + blk % (TN / 2) * 32;
        floatx16 p1, p2, p3;
#pragma unroll
        for (int r = 0; r < 16; ++r) p1[r] = p2[r] = p3[r] = 0.f;
#pragma unroll 1
        for (int c0 = 0; c0 < cin; c0 += 2) {
            const int c = c0 + krow;
            float2 a = make_float2(0.f, 0.f), b = a;
            if (c < cin) {
                a = ws[(size_t(f) * cin + c) * coutp + co + l32];
                b = xs[spec_offset(c, f, t + l32, nbins, ntp)];
            }
            p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, p1, 0, 0, 0);
            p2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, p2, 0, 0, 0);
            p3 = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x + a.y, b.x + b.y, p3, 0, 0, 0);
        }
        float2* dst = ys + yspec_offset(co + 4 * krow, f, t + l32, nbins, ygroup, ntp / ygroup);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            dst[size_t(8 * (r >> 2) + (r & 3)) * nbins * ntp] =
                two_real ? make_float2(p1[r], p2[r]) : make_float2(p1[r] - p2[r], p3[r] - p1[r] - p2[r]);
    }
}

template <SplitTile TILE, int TM, int TN>
static hipError_t launch_split_v(const fftsplit_plan_s& p, const float2* xs, const float2* ws, float2* ys,
                                 hipStream_t s, const LaunchEvents& ev) {
    constexpr SplitTileShape V = kSplitTileShapes[TILE];
    constexpr int BM = V.bm, BN = V.bn, KG = V.groups;
    using S = SplitShape<BM, BN, TM, TN>;
    constexpr int lds = KG * 2 * S::STAGE * 8;
    static_assert(lds <= 160 * 1024 && (KG - 1) * 2 * TM * TN * S::NT * 16 <= lds, "fits the LDS");
    if (p.coutp % BM != 0 || p.ntp % BN != 0) return hipErrorInvalidValue;
    const int nbco = p.coutp / BM, nbt = p.ntp / BN;
    // Patch spectra that one workgroup reads are streamed past the caches, and
    // filter spectra that at most two read, or one on tiles of up to 64 x 64:
    // streamed, the second of those two workgroups often fetches the block
    // from memory again, which costs more than keeping it where such tiles
    // leave the compute units waiting for loads.  Whole layers in us, streamed
    // and kept at two readers: 4x512x28^2 T = 6 69.7, 67.3; 2x300x40^2 T = 6
    // 46.8, 44.9; 1x300x40^2 K=5 T = 4 45.9, 44.1; 7x30x50^2 -> 512 54.4,
    // 53.7; on larger tiles 16x256x56^2 T = 14 136.4, 137.7; 64x512x28^2 410,
    // 416; 2x256x112^2 77.7, 78.7.  (blocks of padding patches read nothing)
    const int readers = (p.nt + BN - 1) / BN;
    const bool w_stream = readers <= (BM * BN <= 64 * 64 ? 1 : 2);
    auto kern = w_stream ? (nbco == 1 ? contract_split_kernel<BM, BN, TM, TN, KG, true, true>
                                      : contract_split_kernel<BM, BN, TM, TN, KG, true, false>)
                         : (nbco == 1 ? contract_split_kernel<BM, BN, TM, TN, KG, false, true>
                                      : contract_split_kernel<BM, BN, TM, TN, KG, false, false>);
    const hipError_t attr = allow_dynamic_lds(kern, lds);
    if (attr != hipSuccess) return attr;
    const size_t nb = size_t(nbco) * nbt * p.bins;
    return launch_kernel(kern, dim3(unsigned(nb)), dim3(KG * S::NT), lds, s, ev.start, ev.stop, xs, ws, ys, p.prob.cin,
                         p.coutp, p.ntp, p.nt, nbco, nbt, p.bins, patch_group(p.L), packed_slots(p.L));
}

hipError_t launch_contract_split(const fftsplit_plan_s& p, const float2* xs, const float2* ws, float2* ys,
                                 hipStream_t s, const LaunchEvents& ev) {
    switch (p.con_split) {
        case kSplit128x128: return launch_split_v<kSplit128x128, 4, 4>(p, xs, ws, ys, s, ev);
        case kSplit256x64: return launch_split_v<kSplit256x64, 4, 4>(p, xs, ws, ys, s, ev);
        case kSplit64x256: return launch_split_v<kSplit64x256, 4, 4>(p, xs, ws, ys, s, ev);
        case kSplit128x64: return launch_split_v<kSplit128x64, 4, 2>(p, xs, ws, ys, s, ev);
        case kSplit64x64: return launch_split_v<kSplit64x64, 2, 2>(p, xs, ws, ys, s, ev);
        case kSplit64x64g2: return launch_split_v<kSplit64x64g2, 2, 2>(p, xs, ws, ys, s, ev);
        case kSplit64x32g2: return launch_split_v<kSplit64x32g2, 2, 2>(p, xs, ws, ys, s, ev);
        case kSplit64x32g4: return launch_split_v<kSplit64x32g4, 2, 2>(p, xs, ws, ys, s, ev);
        case kSplitNone: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace fftsplit
