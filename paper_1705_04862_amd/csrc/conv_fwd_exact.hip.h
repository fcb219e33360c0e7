// Forward pass of the convolutions of the fp32 path, one sample per workgroup from LDS, on the bf16
// matrix cores with exact operands.
//
// An fp32 number is the sum of three bf16 numbers (its 24 significand bits cut 8 + 8 + 8 by
// truncation); the product of two bf16 numbers is exact in fp32.  a*w = sum over the nine part
// products; the six of order >= 2^-16 are accumulated (the three left out are of relative size
// 2^-24 and below, the rounding level of an fp32 product), each one MFMA of four times the depth and
// twice the rate of the fp32 instruction.  The weights arrive already split, in the order in which
// the lanes read their B fragments (WeightSplits); the activations are split once, when a sample is
// written into LDS as three images.
//
// Position-major images with the channels contiguous, de-interleaved by the parity of x for the stride-2 layer, pitch an odd
// multiple of 16 bytes; waves = (32-wide block of output channels) x (share of the k-steps), weights
// in registers, k-shares added through LDS.  The weights are operand A of the MFMAs, their rows in an order
// that gives a lane neighbouring channels of one position: sums are exchanged, split, written to LDS and
// stored 16 bytes at a time.  (With positions as rows every value was handled on its own, and results went
// through an LDS image of their own: all layers of 192 samples 30.7 -> 25.6 us, second layer of 1536 samples
// 56 -> 50 us, third 39 -> 34 us.)
//
// Two kernels: conv_fwd_exact_kernel runs one layer (2 or 3) over any number of samples, a workgroup
// keeping its weights for all its samples; trunk_fwd_exact_kernel runs all convolutions of one sample
// in one workgroup (the first layer as in conv1_exact_kernel), for batches of at most one sample per
// compute unit: a layer's output is split into the next layer's LDS images directly, and is written to
// global memory only for the backward pass.
// Bound: MFMAs for 22000 of the 45000 cycles of a sample that has its workgroup to itself; the rest are the
// phases around them (image and weights from memory, conversion, splitting, exchange), which one wave per SIMD
// cannot overlap with them.
#pragma once
#include "conv1_exact.hip.h"

namespace paac {

// two fp32 numbers -> their three bf16 parts, packed (a in the low half)
__device__ __forceinline__ void split3_pair(float a, float b, unsigned& hi, unsigned& mid, unsigned& lo) {
    const unsigned ah = __float_as_uint(a) & 0xffff0000u, bh = __float_as_uint(b) & 0xffff0000u;
    const float a1 = a - __uint_as_float(ah), b1 = b - __uint_as_float(bh);
    const unsigned am = __float_as_uint(a1) & 0xffff0000u, bm = __float_as_uint(b1) & 0xffff0000u;
    const float a2 = a1 - __uint_as_float(am), b2 = b1 - __uint_as_float(bm);
    hi = (ah >> 16) | bh;
    mid = (am >> 16) | bm;
    lo = __builtin_amdgcn_perm(__float_as_uint(b2), __float_as_uint(a2), 0x07060302u);
}

// Shape constants and the phases of one layer (2 or 3) for the 256 threads of a workgroup.
template <class G> struct ExactConv {
    static_assert((G::ST == 1 || G::ST == 2) && G::CIN % 16 == 0 && G::COUT % 32 == 0 && G::COUT <= 64, "layer shape");
    static_assert(G::ST == 1 || G::W % 2 == 0, "x parity planes");
    static constexpr int CIN = G::CIN, COUT = G::COUT, KS = G::KS, ST = G::ST;
    static constexpr int PI = CIN + 8;                        // position pitch of the bf16 input images
    static constexpr int NB = COUT / 32, KW = 4 / NB, GPO = 4 / KW;        // column blocks, k-shares, register groups finished per wave
    static constexpr int CSI = CIN / 16, KSTEPS = KS * KS * CSI, KPW = KSTEPS / KW;
    static_assert(KSTEPS % KW == 0, "equal k-shares");
    static constexpr int ROWS = G::HO * G::WO, FRAGS = (ROWS + 31) / 32;
    static constexpr int IN_POS = G::H * G::W, PLANE = IN_POS * PI;
    static constexpr int WPLANE = NB * 32 * G::KK;            // elements of one part of the weights
    static constexpr int IN_BYTES = 3 * PLANE * 2;
    // k-shares reach the wave that finishes them through LDS: with two, the other's; with four, all (see give)
    static constexpr int SLOTS = KW == 2 ? 1 : KW, RED_BYTES = NB * KW * SLOTS * FRAGS * GPO * 64 * 16;
    static constexpr int NCH = 4 * GPO;                       // neighbouring channels a lane finishes
    static constexpr int IN_CH = IN_POS * CIN / 4, IN_IT = (IN_CH + 255) / 256;       // 4-channel chunks of a sample
    static_assert(IN_BYTES % 16 == 0 && (PLANE * 2) % 16 == 0 && RED_BYTES % 16 == 0, "16-byte aligned images");

    // LDS position of input (y, x)
    static __device__ __forceinline__ constexpr int ipos(int y, int x) {
        return ST == 2 ? (y * 2 + (x & 1)) * (G::W / 2) + (x >> 1) : y * G::W + x;
    }
    // offset of k-step ks = (ky, kx, channel group) relative to a row's base
    static __device__ __forceinline__ constexpr int koff(int ks) {
        const int tap = ks / CSI, cs = ks % CSI, ky = tap / KS, kx = tap % KS;
        return ipos(ky, kx) * PI + cs * 16;
    }

    // Channel (of a block of 32) in row r of operand A: the GPO register groups from j GPO on are finished by wave
    // (kg + j) mod KW, the wave's own are the first; a lane's channels follow each other.
    static __device__ __forceinline__ int channel(int r, int kg) {
        const int g = r >> 3, h = (r >> 2) & 1;
        return (kg + g / GPO) % KW * (8 * GPO) + h * (4 * GPO) + g % GPO * 4 + (r & 3);
    }
    // the three parts of k-step i of this wave's share
    static __device__ __forceinline__ void load_weights_step(const bf16_t* __restrict__ Wp, int nb, int kg, int lane, int i, bf16x8 (&bw)[3][KPW]) {
        const int row = (lane & 32) + channel(lane & 31, kg);
#pragma unroll
        for (int p = 0; p < 3; ++p)
            bw[p][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(
                Wp + (size_t)p * WPLANE + ((size_t)(nb * KSTEPS + kg * KPW + i) * 64 + row) * 8));
    }
    // all of this wave's share, requested in the order of use
    static __device__ __forceinline__ void load_weights(const bf16_t* __restrict__ Wp, int nb, int kg, int lane, bf16x8 (&bw)[3][KPW]) {
#pragma unroll
        for (int i = 0; i < KPW; ++i) load_weights_step(Wp, nb, kg, lane, i, bw);
    }

    static __device__ __forceinline__ void row_offsets(int lane, int (&a_off)[FRAGS]) {
        const int m = lane & 31, half = lane >> 5;
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) {
            const int r = min(f * 32 + m, ROWS - 1);          // rows past the map: a valid position, never stored
            a_off[f] = ipos((r / G::WO) * ST, (r % G::WO) * ST) * PI + half * 8;
        }
    }

    // four channels from ch on of one position -> their place in the three images
    static __device__ __forceinline__ void split_store(float4 v, int pos, int ch, bf16_t* img) {
        uint2 hi, mid, lo;
        split3_pair(v.x, v.y, hi.x, mid.x, lo.x);
        split3_pair(v.z, v.w, hi.y, mid.y, lo.y);
        bf16_t* at = img + ipos(pos / G::W, pos % G::W) * PI + ch;
        *reinterpret_cast<uint2*>(at) = hi;
        *reinterpret_cast<uint2*>(at + PLANE) = mid;
        *reinterpret_cast<uint2*>(at + 2 * PLANE) = lo;
    }

    // acc += this wave's k-steps of (images) x (weights); the fragments of step i + 1 are read while
    // those of i are multiplied
    // `between(i)` runs after the MFMAs of step i have been issued (requests for later phases go there:
    // the matrix pipe is busy for hundreds of cycles, the memory instructions issue in its shadow).
    struct Nothing { __device__ __forceinline__ void operator()(int) const {} };
    template <class F = Nothing>
    static __device__ __forceinline__ void mfma(const bf16_t* img, const int (&a_off)[FRAGS], int kg, const bf16x8 (&bw)[3][KPW],
                                                f32x16 (&acc)[FRAGS], F&& between = F()) {
        u32x4 a_cur[3][FRAGS], a_nxt[3][FRAGS];
        const int k0 = koff(kg * KPW);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int f = 0; f < FRAGS; ++f) a_cur[p][f] = *reinterpret_cast<const u32x4*>(img + p * PLANE + a_off[f] + k0);
#pragma unroll
        for (int i = 0; i < KPW; ++i) {
            if (i + 1 < KPW) {
                const int kn = koff(kg * KPW + i + 1);
#pragma unroll
                for (int p = 0; p < 3; ++p)
#pragma unroll
                    for (int f = 0; f < FRAGS; ++f) a_nxt[p][f] = *reinterpret_cast<const u32x4*>(img + p * PLANE + a_off[f] + kn);
            }
            __builtin_amdgcn_sched_barrier(0);
            // smallest products first; consecutive MFMAs write different accumulators
            auto mul = [&](int pa, int pw) __attribute__((always_inline)) {
#pragma unroll
                for (int f = 0; f < FRAGS; ++f)
                    acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw[pw][i], __builtin_bit_cast(bf16x8, a_cur[pa][f]), acc[f], 0, 0, 0);
            };
            mul(2, 0); mul(0, 2); mul(1, 1); mul(1, 0); mul(0, 1); mul(0, 0);
            __builtin_amdgcn_sched_barrier(0);
            between(i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int f = 0; f < FRAGS; ++f) a_cur[p][f] = a_nxt[p][f];
        }
    }

    // Exchange of the k-shares of a column block: slots [block][finishing wave][SLOTS][FRAGS][GPO][64 lanes] of 16 bytes.
    // A sum starts with one share and takes the others in the order of the waves.  Of two shares either
    // order is the same sum, and the finishing wave's own stays in its registers; of four, the first is that of wave
    // (position / 8) mod 4, and all pass through LDS.
    static __device__ __forceinline__ void give(const f32x16 (&acc)[FRAGS], float* red, int nb, int kg, int lane) {
        float4* const slots = reinterpret_cast<float4*>(red) + lane;
#pragma unroll
        for (int j = KW == 2 ? 1 : 0; j < KW; ++j) {
            float4* const at = slots + ((nb * KW + (kg + j) % KW) * SLOTS + (KW == 2 ? 0 : kg)) * (FRAGS * GPO * 64);
#pragma unroll
            for (int f = 0; f < FRAGS; ++f)
#pragma unroll
                for (int gi = 0; gi < GPO; ++gi) {
                    const int q = 4 * (j * GPO + gi);
                    at[(f * GPO + gi) * 64] = make_float4(acc[f][q], acc[f][q + 1], acc[f][q + 2], acc[f][q + 3]);
                }
        }
    }
    // first channel a lane finishes (of the whole layer)
    static __device__ __forceinline__ int first_channel(int nb, int kg, int lane) { return nb * 32 + kg * (8 * GPO) + (lane >> 5) * (4 * GPO); }
    // sum, bias, ReLU: emit(position, first_channel + 4 gi, four channels)
    template <class F>
    static __device__ __forceinline__ void take(const f32x16 (&acc)[FRAGS], const float* red, int nb, int kg, int lane, const float4 (&bias)[GPO], F&& emit) {
        const float4* const slots = reinterpret_cast<const float4*>(red) + lane + (nb * KW + kg) * SLOTS * (FRAGS * GPO * 64);
        const int first = (lane & 31) >> 3;
        int src[SLOTS];
        src[0] = 0;
        if constexpr (KW == 4) {
            src[0] = first; src[1] = first == 0 ? 1 : 0; src[2] = first <= 1 ? 2 : 1; src[3] = first <= 2 ? 3 : 2;
        }
        float4 u[FRAGS][GPO][SLOTS];
#pragma unroll
        for (int f = 0; f < FRAGS; ++f)
#pragma unroll
            for (int gi = 0; gi < GPO; ++gi)
#pragma unroll
                for (int j = 0; j < SLOTS; ++j) u[f][gi][j] = slots[((src[j] * FRAGS + f) * GPO + gi) * 64];
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) {
            const int r = f * 32 + (lane & 31);
#pragma unroll
            for (int gi = 0; gi < GPO; ++gi) {
                float4 v = u[f][gi][0];
                if (KW == 2) { v.x += acc[f][4 * gi]; v.y += acc[f][4 * gi + 1]; v.z += acc[f][4 * gi + 2]; v.w += acc[f][4 * gi + 3]; }
#pragma unroll
                for (int j = 1; j < SLOTS; ++j) { v.x += u[f][gi][j].x; v.y += u[f][gi][j].y; v.z += u[f][gi][j].z; v.w += u[f][gi][j].w; }
                v = make_float4(fmaxf(v.x + bias[gi].x, 0.f), fmaxf(v.y + bias[gi].y, 0.f), fmaxf(v.z + bias[gi].z, 0.f), fmaxf(v.w + bias[gi].w, 0.f));
                if (r < ROWS) emit(r, gi, v);
            }
        }
    }
};

// ---------------------------------------------------------------------------------------------
// One layer, any number of samples.
template <class G>
__global__ __launch_bounds__(256, 1) void conv_fwd_exact_kernel(const float* __restrict__ in, const bf16_t* __restrict__ Wp,
                                                                const float* __restrict__ bias, float* __restrict__ out, int ns) {
    typedef ExactConv<G> S;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    bf16_t* const img = reinterpret_cast<bf16_t*>(lds_raw);                   // [3 parts][PLANE]
    float* const red = reinterpret_cast<float*>(lds_raw + S::IN_BYTES);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = wave % S::NB, kg = wave / S::NB;

    int a_off[S::FRAGS];
    S::row_offsets(lane, a_off);

    float4 pin[S::IN_IT];
    auto prefetch_in = [&](int smp) __attribute__((always_inline)) {
        const float* base = in + (size_t)smp * (S::IN_POS * S::CIN);
#pragma unroll
        for (int i = 0; i < S::IN_IT; ++i) pin[i] = *reinterpret_cast<const float4*>(base + (size_t)min(tid + i * 256, S::IN_CH - 1) * 4);
    };
    int s = blockIdx.x;
    if (s >= ns) return;
    prefetch_in(s);
    __builtin_amdgcn_sched_barrier(0);                 // keep the sample's loads ahead of the weights'
    // the weights arrive while the sample is split and written to LDS
    bf16x8 bw[3][S::KPW];
    S::load_weights(Wp, nb, kg, lane, bw);
    const int ch0 = S::first_channel(nb, kg, lane);
    float4 bias_r[S::GPO];
#pragma unroll
    for (int gi = 0; gi < S::GPO; ++gi) bias_r[gi] = *reinterpret_cast<const float4*>(bias + ch0 + gi * 4);

    for (; s < ns; s += gridDim.x) {
        // (threads past the last chunk repeat it: a load that is used under a condition only would be
        // moved behind the weights' loads, and the split would wait for those as well)
#pragma unroll
        for (int i = 0; i < S::IN_IT; ++i) {
            const int ch = min(tid + i * 256, S::IN_CH - 1);
            S::split_store(pin[i], ch / (S::CIN / 4), ch % (S::CIN / 4) * 4, img);
        }
        __syncthreads();
        if (s + (int)gridDim.x < ns) prefetch_in(s + gridDim.x);

        f32x16 acc[S::FRAGS];
#pragma unroll
        for (int f = 0; f < S::FRAGS; ++f)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[f][q] = 0.f;
        S::mfma(img, a_off, kg, bw, acc);
        S::give(acc, red, nb, kg, lane);
        __syncthreads();                               // the shares are complete, the input image has been read
        float* const dst = out + (size_t)s * (S::ROWS * S::COUT);
        S::take(acc, red, nb, kg, lane, bias_r, [&](int r, int gi, float4 v) __attribute__((always_inline)) {
            *reinterpret_cast<float4*>(dst + (unsigned)(r * S::COUT + ch0 + gi * 4)) = v;
        });
    }
}

template <class G>
inline hipError_t launch_conv_fwd_exact(hipStream_t s, const float* in, const bf16_t* Wp, const float* bias, float* out, int ns) {
    if (ns <= 0) return hipErrorInvalidValue;
    constexpr int LDS = ExactConv<G>::IN_BYTES + ExactConv<G>::RED_BYTES;
    static_assert(LDS <= 160 * 1024, "fits the LDS of a compute unit");
    static bool ready = false;
    if (!ready) {                       // more LDS than a kernel gets by default
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_fwd_exact_kernel<G>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        ready = true;
    }
    launch_k_lds((conv_fwd_exact_kernel<G>), dim3(std::min(ns, device_cus())), dim3(256), LDS, s, in, Wp, bias, out, ns);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// All convolutions of one sample in one workgroup.  G3 = NoLayer: two layers.
struct NoLayer {};
template <class G1, class G2, class G3> struct TrunkShape {
    static constexpr bool L3 = !std::is_same<G3, NoLayer>::value;
    typedef ExactConv<G2> S2;
    typedef ExactConv<std::conditional_t<L3, G3, G2>> S3;
    static constexpr int IMG1 = G1::CIN * G1::H * G1::W * 2;                  // the byte image as bf16
    // region A: layer 2's input images, then layer 3's.  Region B: the first layer's image, then the k-share sums.
    static constexpr int A_BYTES = L3 && S3::IN_BYTES > S2::IN_BYTES ? S3::IN_BYTES : S2::IN_BYTES;
    static constexpr int RED = L3 && S3::RED_BYTES > S2::RED_BYTES ? S3::RED_BYTES : S2::RED_BYTES;
    static constexpr int B_BYTES = IMG1 > RED ? IMG1 : RED;
    static constexpr int LDS = A_BYTES + B_BYTES;
    static_assert(A_BYTES % 16 == 0 && IMG1 % 16 == 0, "16-byte aligned regions");
    static_assert(LDS <= 160 * 1024, "fits the LDS of a compute unit");
    static_assert(G1::HO == G2::H && G1::WO == G2::W && G1::COUT == G2::CIN && (G1::COUT == 16 || G1::COUT == 32), "layer 1 feeds layer 2");
};

template <class G1, class G2, class G3>
__global__ __launch_bounds__(256, 1) void trunk_fwd_exact_kernel(const uint8_t* __restrict__ x, const bf16_t* __restrict__ W1p,
                                                                 const float* __restrict__ b1, float* __restrict__ out1,
                                                                 const bf16_t* __restrict__ W2p, const float* __restrict__ b2, float* __restrict__ out2,
                                                                 const bf16_t* __restrict__ W3p, const float* __restrict__ b3, float* __restrict__ out3,
                                                                 int ns, float scale) {
    typedef TrunkShape<G1, G2, G3> T;
    typedef typename T::S2 S2;
    typedef typename T::S3 S3;
    static_assert(G1::CIN == 4 && G1::H == 84 && G1::W == 84 && G1::KS == 8 && G1::ST == 4 && G1::COUT <= 32, "first layer");
    constexpr int PLANE1 = G1::H * G1::W, SAMPLE = 4 * PLANE1;
    constexpr int CHUNKS = SAMPLE / 16, IT = (CHUNKS + 255) / 256;
    constexpr int ROWS1 = G1::HO * G1::WO, FRAGS1 = (ROWS1 + 31) / 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    bf16_t* const img2 = reinterpret_cast<bf16_t*>(lds_raw);
    bf16_t* const img3 = reinterpret_cast<bf16_t*>(lds_raw);
    bf16_t* const img1 = reinterpret_cast<bf16_t*>(lds_raw + T::A_BYTES);
    float* const red = reinterpret_cast<float*>(lds_raw + T::A_BYTES);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fidx = lane & 31, half = lane >> 5;
    const int s = blockIdx.x;
    if (s >= ns) return;

    // ---- requests: the sample, the biases, then the first layer's first weights
    const int nb2 = wave % S2::NB, kg2 = wave / S2::NB, ch2 = S2::first_channel(nb2, kg2, lane);
    const int nb3 = wave % S3::NB, kg3 = wave / S3::NB, ch3 = S3::first_channel(nb3, kg3, lane);
    uint4 pre[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) pre[i] = *reinterpret_cast<const uint4*>(x + (size_t)s * SAMPLE + (size_t)min(tid + i * 256, CHUNKS - 1) * 16);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int NG1 = G1::COUT / 8;                  // register groups with channels
    const int row1 = (lane & 32) + conv1_exact_channel<G1::COUT>(fidx), ch1 = half * (G1::COUT / 2);
    bf16x8 w1[3][16];
    auto load_w1 = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 3; ++p) w1[p][kt] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(W1p + p * 8192 + (kt * 64 + row1) * 8));
    };
    // (not all of them: a wave that requests 48 KB at once is still issuing when its part of the image has arrived)
    constexpr int AHEAD1 = 5;
#pragma unroll
    for (int kt = 0; kt < AHEAD1; ++kt) load_w1(kt);
    float4 bias1[NG1], bias2[S2::GPO], bias3[S3::GPO];
#pragma unroll
    for (int g = 0; g < NG1; ++g) bias1[g] = *reinterpret_cast<const float4*>(b1 + ch1 + g * 4);
#pragma unroll
    for (int g = 0; g < S2::GPO; ++g) bias2[g] = *reinterpret_cast<const float4*>(b2 + ch2 + g * 4);
    if constexpr (T::L3) {
#pragma unroll
        for (int g = 0; g < S3::GPO; ++g) bias3[g] = *reinterpret_cast<const float4*>(b3 + ch3 + g * 4);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- first layer: bytes -> bf16 in the same linear order
    // (threads past the last chunk repeat it: a load that is used under a condition only would be
    // moved behind the weights' loads, and the conversion would wait for those as well)
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        uint4* dst = reinterpret_cast<uint4*>(img1 + min(tid + i * 256, CHUNKS - 1) * 16);
        dst[0] = u8x8_to_bf16(make_uint2(pre[i].x, pre[i].y));
        dst[1] = u8x8_to_bf16(make_uint2(pre[i].z, pre[i].w));
    }
    __syncthreads();
    // Fragments wave, wave + 4, .. of the 32-position fragments, all at once (k-steps outside, fragments
    // inside: four independent accumulators per weight fragment; a fragment index past the map repeats
    // the last position and is not stored).  The weights of later k-steps and of the second layer are requested on
    // the way, some after each k-step: in the shadow of the MFMAs, and before the stores of this
    // layer's epilogue, so that waiting for them never waits for a store.
    constexpr int FPW = (FRAGS1 + 3) / 4;
    const bf16_t* a0[FPW];
    f32x16 acc1[FPW];
#pragma unroll
    for (int j = 0; j < FPW; ++j) {
        const int r = min((wave + 4 * j) * 32 + fidx, ROWS1 - 1);
        a0[j] = img1 + ((r / G1::WO) * G1::ST + half) * G1::W + (r % G1::WO) * G1::ST;
#pragma unroll
        for (int q = 0; q < 16; ++q) acc1[j][q] = 0.f;
    }
    bf16x8 w2[3][S2::KPW];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 a[FPW];
#pragma unroll
            for (int j = 0; j < FPW; ++j) {
                const uint2* ap = reinterpret_cast<const uint2*>(a0[j] + c * PLANE1 + ks * 2 * G1::W);   // 8-byte aligned
                const uint2 lo = ap[0], hi = ap[1];
                a[j] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
            }
#pragma unroll
            for (int p = 2; p >= 0; --p)
#pragma unroll
                for (int j = 0; j < FPW; ++j) acc1[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[p][c * 4 + ks], a[j], acc1[j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (c * 4 + ks + AHEAD1 < 16) load_w1(c * 4 + ks + AHEAD1);
#pragma unroll
            for (int i = (c * 4 + ks) * S2::KPW / 16; i < (c * 4 + ks + 1) * S2::KPW / 16; ++i)
                S2::load_weights_step(W2p, nb2, kg2, lane, i, w2);
            __builtin_amdgcn_sched_barrier(0);
        }
    // bias + ReLU, split into layer 2's images; the backward pass reads the output from global memory
    {
        float* const o1 = out1 + (size_t)s * (ROWS1 * G1::COUT) + ch1;
#pragma unroll
        for (int j = 0; j < FPW; ++j) {
            const int r = (wave + 4 * j) * 32 + fidx;
            if (r < ROWS1) {
                bf16_t* const at = img2 + S2::ipos(r / G1::WO, r % G1::WO) * S2::PI + ch1;
#pragma unroll
                for (int g = 0; g < NG1; g += 2) {
                    u32x4 part[3];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int q = 4 * (g + e);
                        const float4 b = bias1[g + e];
                        const float4 v = make_float4(fmaxf(acc1[j][q] * scale + b.x, 0.f), fmaxf(acc1[j][q + 1] * scale + b.y, 0.f),
                                                     fmaxf(acc1[j][q + 2] * scale + b.z, 0.f), fmaxf(acc1[j][q + 3] * scale + b.w, 0.f));
                        unsigned hi, mid, lo;
                        split3_pair(v.x, v.y, hi, mid, lo);
                        part[0][2 * e] = hi; part[1][2 * e] = mid; part[2][2 * e] = lo;
                        split3_pair(v.z, v.w, hi, mid, lo);
                        part[0][2 * e + 1] = hi; part[1][2 * e + 1] = mid; part[2][2 * e + 1] = lo;
                        if (out1) *reinterpret_cast<float4*>(o1 + (unsigned)(r * G1::COUT + q)) = v;
                    }
#pragma unroll
                    for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(at + p * S2::PLANE + 4 * g) = part[p];
                }
            }
        }
    }
    __syncthreads();                                   // layer 2's images are complete, the first image is free

    // ---- second layer
    int a_off2[S2::FRAGS];
    S2::row_offsets(lane, a_off2);
    f32x16 acc2[S2::FRAGS];
#pragma unroll
    for (int f = 0; f < S2::FRAGS; ++f)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc2[f][q] = 0.f;
    // the third layer's weights are requested k-step by k-step while the second layer multiplies
    // (its own weights' registers become free at the same rate)
    bf16x8 w3[3][S3::KPW];
    S2::mfma(img2, a_off2, kg2, w2, acc2, [&](int i) __attribute__((always_inline)) {
        if constexpr (T::L3) {
#pragma unroll
            for (int j = 0; j < S3::KPW; ++j)
                if (j * S2::KPW / S3::KPW == i) S3::load_weights_step(W3p, nb3, kg3, lane, j, w3);
        }
    });
    __builtin_amdgcn_sched_barrier(0);
    S2::give(acc2, red, nb2, kg2, lane);
    __syncthreads();                                   // the shares are complete, layer 2's images have been read
    float* const o2 = out2 + (size_t)s * (S2::ROWS * S2::COUT);
    S2::take(acc2, red, nb2, kg2, lane, bias2, [&](int r, int gi, float4 v) __attribute__((always_inline)) {
        if (!T::L3 || out2) *reinterpret_cast<float4*>(o2 + (unsigned)(r * S2::COUT + ch2 + gi * 4)) = v;
        if constexpr (T::L3) S3::split_store(v, r, ch2 + gi * 4, img3);
    });
    if constexpr (T::L3) {
        static_assert(G2::HO == G3::H && G2::WO == G3::W && G2::COUT == G3::CIN && G3::ST == 1, "layer 2 feeds layer 3");
        __syncthreads();                               // layer 3's images are complete
        int a_off3[S3::FRAGS];
        S3::row_offsets(lane, a_off3);
        f32x16 acc3[S3::FRAGS];
#pragma unroll
        for (int f = 0; f < S3::FRAGS; ++f)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc3[f][q] = 0.f;
        S3::mfma(img3, a_off3, kg3, w3, acc3);
        S3::give(acc3, red, nb3, kg3, lane);
        __syncthreads();
        float* const o3 = out3 + (size_t)s * (S3::ROWS * S3::COUT);
        S3::take(acc3, red, nb3, kg3, lane, bias3, [&](int r, int gi, float4 v) __attribute__((always_inline)) {
            *reinterpret_cast<float4*>(o3 + (unsigned)(r * S3::COUT + ch3 + gi * 4)) = v;
        });
    }
}

// ns <= compute units (one workgroup per sample, no loop over samples)
template <class G1, class G2, class G3>
inline hipError_t launch_trunk_fwd_exact(hipStream_t s, const uint8_t* x, const bf16_t* W1p, const float* b1, float* out1,
                                         const bf16_t* W2p, const float* b2, float* out2,
                                         const bf16_t* W3p, const float* b3, float* out3, int ns) {
    if (ns <= 0 || ns > device_cus()) return hipErrorInvalidValue;
    constexpr int LDS = TrunkShape<G1, G2, G3>::LDS;
    static bool ready = false;
    if (!ready) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(trunk_fwd_exact_kernel<G1, G2, G3>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        ready = true;
    }
    launch_k_lds((trunk_fwd_exact_kernel<G1, G2, G3>), dim3(ns), dim3(256), LDS, s, x, W1p, b1, out1, W2p, b2, out2, W3p, b3, out3, ns,
                 1.0f / 255.0f);
    return hipGetLastError();
}

}  // namespace paac
