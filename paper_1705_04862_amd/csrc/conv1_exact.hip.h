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
// A workgroup takes bands of HO / PARTS output rows of one sample: the band's 4 x (4 BR + 4) image
// rows are four contiguous pieces of global memory.  The weights arrive as their three bf16 parts in
// fragment order (WeightSplits: the optimiser writes them with every update), 16 bytes per lane and k-step.
// Bound: the MFMAs (6100 cycles per sample and SIMD).  Waves 0 .. 3 do nothing else: the weights are operand A, so that
// a lane holds COUT / 2 neighbouring channels of one position and stores them 16 bytes at a time; waves 4 .. 7 load and
// convert the next band into the other of two images meanwhile.  One wave per SIMD that loaded, converted, multiplied
// and stored (4 bytes at a time) in turn took 7.6 us per sample: 1536 samples of arch_nature 45.5 -> 38 us, 2560 of arch_nips 84 -> 46.
#pragma once
#include "gemm_bf16.hip.h"

namespace paac {

// Operand A of the first layer's 32 x 32 MFMAs: row r is this channel, so that the register groups g < COUT / 8 of lane half h
// are channels h COUT / 2 + 4 g .. + 3 (rows past the channels: zero weights)
template <int COUT> __device__ __forceinline__ int conv1_exact_channel(int r) {
    constexpr int NG = COUT / 8;
    const int g = r >> 3, h = (r >> 2) & 1;
    return g < NG ? h * (COUT / 2) + g * 4 + (r & 3) : COUT + h * (16 - COUT / 2) + (g - NG) * 4 + (r & 3);
}

template <class G, int PARTS>
__global__ __launch_bounds__(512, 2) void conv1_exact_kernel(const uint8_t* __restrict__ x, const bf16_t* __restrict__ Wp,
                                                          const float* __restrict__ bias, float* __restrict__ out, int ns,
                                                          float scale) {
    static_assert(G::CIN == 4 && G::H == 84 && G::W == 84 && G::KS == 8 && G::ST == 4 && (G::COUT == 16 || G::COUT == 32), "first layer");
    static_assert(G::HO % PARTS == 0, "bands of whole output rows");
    constexpr int SAMPLE = G::CIN * G::H * G::W, PLANE = G::H * G::W;
    constexpr int BR = G::HO / PARTS, IR = 4 * BR + 4;            // output rows per band, image rows it reads
    constexpr int CPC = IR * G::W / 16, CHUNKS = 4 * CPC, IT = (CHUNKS + 255) / 256;   // 16-byte chunks per channel piece
    constexpr int ROWS = BR * G::WO, FRAGS = (ROWS + 31) / 32, FPW = (FRAGS + 3) / 4, NG = G::COUT / 8;
    static_assert((IR * G::W) % 16 == 0 && (G::ST * G::W * BR) % 16 == 0 && PLANE % 16 == 0, "whole 16-byte chunks");
    constexpr int IMG = 4 * IR * G::W;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    bf16_t* const img = reinterpret_cast<bf16_t*>(lds_raw);       // two of them
    u32x4* const w_low = reinterpret_cast<u32x4*>(lds_raw + 2 * IMG * 2);         // the weights' third part, [k-step][lane]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p0 = blockIdx.x, step = gridDim.x, items = ns * PARTS;
    if (p0 >= items) return;
    const int count = (items - p0 + step - 1) / step;             // bands of this workgroup; both roles pass count + 1 barriers

    if (wave >= 4) {
        const int tid = threadIdx.x - 256;
        uint4 pre[IT];
        auto request = [&](int n) __attribute__((always_inline)) {        // past the end: the last band again, not used
            const int p = p0 + min(n, count - 1) * step;
            const size_t base = (size_t)(p / PARTS) * SAMPLE + (size_t)(p % PARTS) * (BR * G::ST * G::W);
#pragma unroll
            for (int i = 0; i < IT; ++i) {                                // threads past the last chunk repeat it
                const int cc = min(tid + i * 256, CHUNKS - 1);
                pre[i] = *reinterpret_cast<const uint4*>(x + base + (size_t)(cc / CPC) * PLANE + (size_t)(cc % CPC) * 16);
            }
        };
        auto deposit = [&](int n) __attribute__((always_inline)) {        // bytes -> bf16, same linear order
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                uint4* dst = reinterpret_cast<uint4*>(img + (n & 1) * IMG + min(tid + i * 256, CHUNKS - 1) * 16);
                dst[0] = u8x8_to_bf16(make_uint2(pre[i].x, pre[i].y));
                dst[1] = u8x8_to_bf16(make_uint2(pre[i].z, pre[i].w));
            }
        };
        request(0);
        deposit(0);
        request(1);
        __syncthreads();
        for (int n = 0; n < count; ++n) {
            if (n + 1 < count) { deposit(n + 1); request(n + 2); }
            __syncthreads();
        }
        return;
    }
    const int fidx = lane & 31, half = lane >> 5, ch = half * (G::COUT / 2);
    // two of the weights' parts in registers; with the third in them too, nothing would be left for the accumulators
    bf16x8 w[2][16];
    const bf16_t* const wp = Wp + ((lane & 32) + conv1_exact_channel<G::COUT>(fidx)) * 8;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
        w_low[(wave * 4 + kt) * 64 + lane] = *reinterpret_cast<const u32x4*>(wp + 2 * 8192 + (wave * 4 + kt) * 512);
#pragma unroll
    for (int kt = 0; kt < 16; ++kt)
#pragma unroll
        for (int q = 0; q < 2; ++q) w[q][kt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(wp + q * 8192 + kt * 512));
    float4 bias_r[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) bias_r[g] = *reinterpret_cast<const float4*>(bias + ch + g * 4);
    int a_off[FPW];
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
        const int r = min((wave + 4 * j) * 32 + fidx, ROWS - 1);          // positions past the band: a valid address, never stored
        a_off[j] = ((r / G::WO) * G::ST + half) * G::W + (r % G::WO) * G::ST;
    }
    __syncthreads();
    for (int n = 0; n < count; ++n) {
        const int p = p0 + n * step;
        const bf16_t* const src = img + (n & 1) * IMG;
        float* const dst = out + ((size_t)(p / PARTS) * (G::HO * G::WO) + (size_t)(p % PARTS) * ROWS) * G::COUT + ch;
        // two fragments at a time
#pragma unroll
        for (int j0 = 0; j0 < FPW; j0 += 2) {
            constexpr int LAST = FPW - 1;
            if ((wave + 4 * j0) * 32 < ROWS) {
                f32x16 acc[2];
                bf16x8 a[2][2];
                u32x4 wl[2];
                const bool two = j0 + 1 <= LAST && (wave + 4 * (j0 + 1)) * 32 < ROWS;
                auto load = [&](int kt, int e) __attribute__((always_inline)) {
                    const uint2* ap = reinterpret_cast<const uint2*>(src + a_off[j0 + e <= LAST ? j0 + e : LAST] + (kt >> 2) * (IR * G::W) + (kt & 3) * 2 * G::W);   // 8-byte aligned
                    const uint2 lo = ap[0], hi = ap[1];
                    a[kt & 1][e] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
                };
                auto multiply = [&](auto NF) __attribute__((always_inline)) {
                    constexpr int nf = decltype(NF)::value;
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt) {
                        wl[kt] = w_low[kt * 64 + lane];
#pragma unroll
                        for (int e = 0; e < nf; ++e) load(kt, e);
                    }
#pragma unroll
                    for (int e = 0; e < nf; ++e)
#pragma unroll
                        for (int q = 0; q < 16; ++q) acc[e][q] = 0.f;
#pragma unroll
                    for (int kt = 0; kt < 16; ++kt) {
#pragma unroll
                        for (int q = 2; q >= 0; --q)
#pragma unroll
                            for (int e = 0; e < nf; ++e) acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q == 2 ? __builtin_bit_cast(bf16x8, wl[kt & 1]) : w[q & 1][kt], a[kt & 1][e], acc[e], 0, 0, 0);
                        if (kt + 2 < 16) {
                            wl[kt & 1] = w_low[(kt + 2) * 64 + lane];
#pragma unroll
                            for (int e = 0; e < nf; ++e) load(kt + 2, e);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int e = 0; e < nf; ++e) {
                        const int r = (wave + 4 * (j0 + e)) * 32 + fidx;
                        if (r < ROWS) {
#pragma unroll
                            for (int g = 0; g < NG; ++g)
                                *reinterpret_cast<float4*>(dst + (unsigned)(r * G::COUT + 4 * g)) =
                                    make_float4(fmaxf(acc[e][4 * g] * scale + bias_r[g].x, 0.f), fmaxf(acc[e][4 * g + 1] * scale + bias_r[g].y, 0.f),
                                                fmaxf(acc[e][4 * g + 2] * scale + bias_r[g].z, 0.f), fmaxf(acc[e][4 * g + 3] * scale + bias_r[g].w, 0.f));
                        }
                    }
                };
                if (two) multiply(std::integral_constant<int, 2>());
                else multiply(std::integral_constant<int, 1>());
            }
        }
        __syncthreads();                                                  // the next band's image is complete, this one free
    }
}

template <class G, int PARTS>
inline hipError_t launch_conv1_exact_p(hipStream_t s, const uint8_t* x, const bf16_t* Wk, const float* bias, float* out, int ns) {
    constexpr int LDS = 2 * 4 * (4 * G::HO / PARTS + 4) * G::W * 2 + 16 * 1024;
    static const hipError_t ready = hipFuncSetAttribute(reinterpret_cast<const void*>(conv1_exact_kernel<G, PARTS>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, LDS);        // more than the default
    if (ready != hipSuccess) return ready;
    launch_k_lds((conv1_exact_kernel<G, PARTS>), dim3(std::min(ns * PARTS, device_cus())), dim3(512), LDS, s, x, Wk, bias, out, ns, 1.0f / 255.0f);
    return hipGetLastError();
}

template <class G>
inline hipError_t launch_conv1_exact(hipStream_t s, const uint8_t* x, const bf16_t* Wk, const float* bias, float* out, int ns) {
    if (ns <= 0) return hipErrorInvalidValue;
    // half a sample per workgroup while that still gives every workgroup a compute unit of its own
    return ns * 2 <= device_cus() ? launch_conv1_exact_p<G, 2>(s, x, Wk, bias, out, ns) : launch_conv1_exact_p<G, 1>(s, x, Wk, bias, out, ns);
}

}  // namespace paac
