// First convolution (8x8, stride 4, uint8 NCHW input) of the fp32 path, straight from the image.
//
// The im2col view repeats every input byte in four output windows.  A workgroup loads its image rows with 16-byte
// loads, converts them ONCE and keeps them in LDS as bf16 in the same (c, y, x) order.  The MFMA A fragment of an
// output position (oy, ox) and k-group (c, ky) is then the 16 bytes at img[c][4*oy + ky][4*ox .. 4*ox + 7],
// i.e. one base address per fragment plus compile-time offsets; the weights (COUT x 256) stay in
// registers for the lifetime of the workgroup.  An image row is 84 elements = 42 words: the rows of
// consecutive output rows continue each other's bank sequence, no padding is needed.
//
// It runs on the bf16 matrix cores without giving up fp32 accuracy.
// A byte (0..255) is exact in bf16, and an fp32 weight is exactly the sum of three bf16 numbers
// (its 24 significand bits cut into 8 + 8 + 8 by truncation: w = hi + mid + lo, every residual
// exact).  Every product byte x part is exact in fp32, so three bf16 MFMAs accumulate, in fp32,
// exactly the terms of the fp32 dot product; only the order of the fp32 additions differs from
// the fp32 MFMA path.  16 k per 32-cycle instruction x 3 parts against 2 k per 64-cycle fp32
// instruction: 5.3 times fewer matrix-core cycles, and no im2col gather.
// A workgroup takes one band of HO / PARTS output rows of one sample: its 4 x (4 BR + 4) image
// rows are four contiguous pieces of global memory.  The weights arrive as their three bf16 parts in
// fragment order (WeightSplits: the optimiser writes them with every update), 16 bytes per lane and k-step.
#pragma once
#include "gemm_bf16.hip.h"

namespace paac {

template <class G, int PARTS>
__global__ __launch_bounds__(256, 1) void conv1_exact_kernel(const uint8_t* __restrict__ x, const bf16_t* __restrict__ Wp,
                                                          const float* __restrict__ bias, float* __restrict__ out, int ns,
                                                          float scale) {
    static_assert(G::CIN == 4 && G::H == 84 && G::W == 84 && G::KS == 8 && G::ST == 4 && G::COUT <= 32, "first layer");
    static_assert(G::HO % PARTS == 0, "bands of whole output rows");
    constexpr int SAMPLE = G::CIN * G::H * G::W, PLANE = G::H * G::W;
    constexpr int BR = G::HO / PARTS, IR = 4 * BR + 4;            // output rows per band, image rows it reads
    constexpr int CPC = IR * G::W / 16, CHUNKS = 4 * CPC, IT = (CHUNKS + 255) / 256;   // 16-byte chunks per channel piece
    constexpr int ROWS = BR * G::WO, FRAGS = (ROWS + 31) / 32;
    static_assert((IR * G::W) % 16 == 0 && (G::ST * G::W * BR) % 16 == 0 && PLANE % 16 == 0, "whole 16-byte chunks");
    __shared__ __attribute__((aligned(16))) bf16_t img[4 * IR * G::W];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fidx = lane & 31, kg = lane >> 5;
    const int items = ns * PARTS;

    uint4 pre[IT];
    auto prefetch = [&](int p) __attribute__((always_inline)) {
        const size_t base = (size_t)(p / PARTS) * SAMPLE + (size_t)(p % PARTS) * (BR * G::ST * G::W);
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int ch = tid + i * 256;
            const bool ok = ch < CHUNKS;
            const int cc = ok ? ch : 0;
            pre[i] = *reinterpret_cast<const uint4*>(x + base + (size_t)(cc / CPC) * PLANE + (size_t)(cc % CPC) * 16);
        }
    };
    int p = blockIdx.x;
    if (p >= items) return;
    prefetch(p);

    // weights of output channel fidx, this lane's eight k of each of the sixteen k-steps, as three bf16 parts
    bf16x8 bh[16], bm[16], bl[16];
#pragma unroll
    for (int kt = 0; kt < 16; ++kt) {
        const bf16_t* w = Wp + (kt * 64 + lane) * 8;                // one contiguous KB per wave; channels COUT..31 are zero
        bh[kt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(w));
        bm[kt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(w + 8192));
        bl[kt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(w + 2 * 8192));
    }
    const float bias_r = fidx < G::COUT ? bias[fidx] : 0.f;

    for (; p < items; p += gridDim.x) {
#pragma unroll
        for (int i = 0; i < IT; ++i) {                                // bytes -> bf16, same linear order
            const int ch = tid + i * 256;
            if (ch < CHUNKS) {
                uint4* dst = reinterpret_cast<uint4*>(img + ch * 16);
                dst[0] = u8x8_to_bf16(make_uint2(pre[i].x, pre[i].y));
                dst[1] = u8x8_to_bf16(make_uint2(pre[i].z, pre[i].w));
            }
        }
        __syncthreads();
        if (p + (int)gridDim.x < items) prefetch(p + gridDim.x);     // in flight during the MFMA phase
        const size_t orow0 = (size_t)(p / PARTS) * (G::HO * G::WO) + (size_t)(p % PARTS) * ROWS;
        for (int f = wave; f < FRAGS; f += 4) {
            const int r = min(f * 32 + fidx, ROWS - 1);               // rows past the band: a valid address, never stored
            const int oy = r / G::WO, ox = r % G::WO;
            const bf16_t* a0 = img + (oy * G::ST + kg) * G::W + ox * G::ST;
            f32x16 acc;
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[q] = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const uint2* ap = reinterpret_cast<const uint2*>(a0 + c * (IR * G::W) + ks * 2 * G::W);   // 8-byte aligned
                    const uint2 lo = ap[0], hi = ap[1];
                    const bf16x8 a = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bl[c * 4 + ks], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bm[c * 4 + ks], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bh[c * 4 + ks], acc, 0, 0, 0);
                }
            if (fidx < G::COUT) {
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int lr = f * 32 + Mma<32>::row(q, lane);
                    if (lr < ROWS) out[(orow0 + lr) * G::COUT + fidx] = fmaxf(acc[q] * scale + bias_r, 0.f);
                }
            }
        }
        __syncthreads();                                              // the image is rewritten next
    }
}

template <class G, int PARTS>
inline void launch_conv1_exact_p(hipStream_t s, int cus, const uint8_t* x, const bf16_t* Wk, const float* bias, float* out, int ns) {
    launch_k((conv1_exact_kernel<G, PARTS>), dim3(std::min(ns * PARTS, 2 * cus)), dim3(256), s, x, Wk, bias, out, ns, 1.0f / 255.0f);
}

template <class G>
inline hipError_t launch_conv1_exact(hipStream_t s, const uint8_t* x, const bf16_t* Wk, const float* bias, float* out, int ns) {
    if (ns <= 0) return hipErrorInvalidValue;
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    }
    // one workgroup per compute unit (its registers allow no more): split samples into bands while
    // that still gives every workgroup a compute unit of its own
    if (ns * 2 <= cus) launch_conv1_exact_p<G, 2>(s, cus, x, Wk, bias, out, ns);
    else launch_conv1_exact_p<G, 1>(s, cus, x, Wk, bias, out, ns);
    return hipGetLastError();
}

}  // namespace paac
