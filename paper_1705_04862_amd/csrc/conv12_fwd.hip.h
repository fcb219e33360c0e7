// First and second convolution of the fp32 path in one launch, for batches of a few dozen samples.
//
// At that size neither layer has work for more than a microsecond or two; a launch of each costs its latencies
// (the boundary between two launches alone is 2.5 us).  A workgroup takes a band of BR output rows of the
// second layer of one sample (and COUT2 / CG of its channels): the 2 BR + 2 rows of the first layer that
// the band reads are computed here, from the 8 BR + 12 image rows below them, and stay in LDS.  Neighbouring
// bands compute two rows of the first layer each for themselves; its bf16 MFMAs are cheap next to a launch.
// One action selection, two launches before -> this one: arch_nips n_e = 1 13.2 -> 11.3 us, n_e = 32 15.7 -> 13.4;
// arch_nature n_e = 1 20.2 -> 17.7, n_e = 32 25.6 -> 22.3, n_e = 64 34.5 -> 28.3.
//
// First layer: exact bf16 parts (see conv1_exact_kernel); wave w takes input channel w & 3 for every other
// fragment of 32 positions, with the weights as operand A, so that a lane holds four channels of one position.
// The four channels' sums meet in LDS and are added in a fixed order.
// Second layer: fp32 MFMAs, wave w takes an eighth of the k range (two of the 4 x 4 taps) for all of the band's
// positions and channels; a lane's weights are CT neighbouring channels of one k, one load.  The eight
// sums are added in ascending order.
// Bound, in bands of three rows of arch_nature and halves of the channels (14000 cycles): a third are the fp32
// MFMAs of the second layer, a fifth the way of image and weights from memory, the rest the first layer's
// MFMAs and the LDS writes of its sums (64 bytes per cycle), a chain of short phases with a barrier after each.
#pragma once
#include "gemm_bf16.hip.h"

namespace paac {

template <class G1, class G2, int BR_, int CG_> struct Conv12Shape {
    static_assert(G1::CIN == 4 && G1::H == 84 && G1::W == 84 && G1::KS == 8 && G1::ST == 4 && G1::COUT <= 32, "first layer");
    static_assert(G2::H == G1::HO && G2::W == G1::WO && G2::CIN == G1::COUT && G2::KS == 4 && G2::ST == 2, "second layer");
    static constexpr int BR = BR_, CG = CG_, BANDS = G2::HO / BR;
    static_assert(G2::HO % BR == 0, "bands of whole output rows");
    static constexpr int R1 = 2 * BR + 2, IR = 4 * R1 + 4;                // rows of the first layer, image rows
    static constexpr int CPC = IR * G1::W / 16, CHUNKS = 4 * CPC, IT = (CHUNKS + 511) / 512;
    static_assert((IR * G1::W) % 16 == 0 && (8 * BR * G1::W) % 16 == 0 && G1::H * G1::W % 16 == 0, "whole 16-byte chunks");
    static constexpr int P1 = R1 * G1::WO, F1 = (P1 + 31) / 32, FPW = (F1 + 1) / 2;
    static constexpr int C1 = G1::COUT, PITCH = C1 + 4;                   // floats per position
    static constexpr int HALF = G1::WO / 2 * PITCH + (96 - G1::WO / 2 * PITCH % 64) % 64;     // one row's columns of one parity: 32 mod 64 floats
    static constexpr int PLANE = R1 * 2 * HALF;
    static constexpr int P2 = BR * G2::WO, F2 = (P2 + 15) / 16;
    static constexpr int COLS = G2::COUT / CG, CT = COLS / 16;            // output channels of a workgroup, per lane
    static_assert(CT == 1 || CT == 2 || CT == 4, "a lane loads 4, 8 or 16 bytes of weights");
    static constexpr int KG = G2::KK / 8 / 16;                            // groups of 16 k per wave
    static_assert(G2::KK % 128 == 0 && KG * 16 == 2 * C1, "a wave takes two taps");
    static constexpr int PITCH2 = COLS + 4, PLANE2 = F2 * 16 * PITCH2;
    // byte image as bf16 | four planes of channel sums; the first becomes the layer's output, the other three
    // are free after that and take the eight planes of the second layer's sums, with what lies behind them
    static constexpr int IMG_BYTES = 4 * IR * G1::W * 2;
    static constexpr int SUM_FLOATS = 3 * PLANE > 8 * PLANE2 ? 3 * PLANE : 8 * PLANE2;
    static constexpr int LDS = IMG_BYTES + (PLANE + SUM_FLOATS) * 4;
    static_assert(LDS <= 160 * 1024 && IMG_BYTES % 16 == 0, "fits the LDS of a compute unit");
    // float index of a position of the band's first-layer rows.  Columns of one parity together: the second layer
    // reads every other column, and the pitches give sixteen lanes sixteen different groups of four banks there as
    // well as where the sums are written
    static __device__ __forceinline__ constexpr int at(int y, int x) { return (y * 2 + (x & 1)) * HALF + (x >> 1) * PITCH; }
};

template <class G1, class G2, int BR, int CG>
__global__ __launch_bounds__(512, BR == 1 ? 4 : 2) void conv12_fwd_kernel(const uint8_t* __restrict__ x, const bf16_t* __restrict__ W1p,
                                                            const float* __restrict__ b1, float* __restrict__ out1,
                                                            const float* __restrict__ W2, const float* __restrict__ b2,
                                                            float* __restrict__ out2, int ns, float scale, int ten_bands) {
    typedef Conv12Shape<G1, G2, BR, CG> S;
    typedef Mma<16> MM;
    typedef float vct __attribute__((ext_vector_type(S::CT == 1 ? 2 : S::CT)));     // (CT == 1 uses element 0)
    constexpr int PLANE_IN = G1::H * G1::W, SAMPLE = 4 * PLANE_IN;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    bf16_t* const img = reinterpret_cast<bf16_t*>(lds_raw);
    float* const act = reinterpret_cast<float*>(lds_raw + S::IMG_BYTES);
    float* const sums = act + S::PLANE;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int id = blockIdx.x;
    const int cg = id % CG, band = id / CG % S::BANDS, s = id / (CG * S::BANDS);
    if (s >= ns) return;

    // ---- requests: image rows, first layer's weights, second layer's weights, biases
    const uint8_t* const xb = x + (size_t)s * SAMPLE + (size_t)band * (8 * BR * G1::W);
    uint4 pre[S::IT];
#pragma unroll
    for (int i = 0; i < S::IT; ++i) {                   // threads past the last chunk repeat it
        const int cc = min(tid + i * 512, S::CHUNKS - 1);
        pre[i] = *reinterpret_cast<const uint4*>(xb + (size_t)(cc / S::CPC) * PLANE_IN + (size_t)(cc % S::CPC) * 16);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int c_in = wave & 3;
    bf16x8 w1[3][4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            w1[q][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(W1p + q * 8192 + ((c_in * 4 + ks) * 64 + lane) * 8));
    __builtin_amdgcn_sched_barrier(0);
    constexpr int Q1 = S::C1 / 4;                       // float4 per position of layer 1
    const float4 bias1 = *reinterpret_cast<const float4*>(b1 + tid % Q1 * 4);
    constexpr int Q2 = S::COLS / 4;
    const float4 bias2 = *reinterpret_cast<const float4*>(b2 + cg * S::COLS + tid % Q2 * 4);
    static_assert(512 % Q1 == 0 && 512 % Q2 == 0, "a thread keeps its channels");
    __builtin_amdgcn_sched_barrier(0);

    // ---- while they are under way: where this thread reads and writes in the phases below
    const int pidx = lane & 31, half = lane >> 5, f0 = wave >> 2;
    int a1_off[S::FPW], s1_off[S::FPW];
#pragma unroll
    for (int f = 0; f < S::FPW; ++f) {
        const int r = min((f0 + 2 * f) * 32 + pidx, S::P1 - 1);           // positions past the band: a valid address, not written
        a1_off[f] = c_in * (S::IR * G1::W) + ((r / G1::WO) * 4 + half) * G1::W + (r % G1::WO) * 4;
        s1_off[f] = c_in * S::PLANE + S::at(r / G1::WO, r % G1::WO) + 4 * half;
    }
    constexpr int ITEMS1 = S::P1 * Q1, ITI1 = (ITEMS1 + 511) / 512;
    int p1_off[ITI1][4];
    bool own1[ITI1];
    {
        const bool store = out1 != nullptr && cg == 0;
        const int own_rows = !store ? 0 : band == S::BANDS - 1 ? S::R1 : 2 * BR;
#pragma unroll
        for (int it = 0; it < ITI1; ++it) {
            const int p = min(tid + it * 512, ITEMS1 - 1) / Q1, y = p / G1::WO, xx = p % G1::WO;
            // which channel comes first depends on the position in bands of two (or five) rows
            const int gy = band * (2 * BR) + y;
            const int lr = ten_bands ? (gy & 1) * G1::WO + xx : (gy % 5) * G1::WO + xx;
            const int first = ten_bands ? (lr < 16 ? 0 : lr < 32 ? 2 : 1) : lr >> 5;
            const int base = S::at(y, xx) + tid % Q1 * 4;
            p1_off[it][0] = base + first * S::PLANE;
            p1_off[it][1] = base + (first == 0 ? S::PLANE : 0);
            p1_off[it][2] = base + (first <= 1 ? 2 : 1) * S::PLANE;
            p1_off[it][3] = base + (first <= 2 ? 3 : 2) * S::PLANE;
            own1[it] = y < own_rows;
        }
    }
    const int fidx = lane & 15, fk = lane >> 4;
    int a2_off[S::F2];
#pragma unroll
    for (int f = 0; f < S::F2; ++f) {                   // this wave's taps are (ky, kx) = (wave / 2, wave % 2 * 2) and (ky, kx + 1)
        const int r = min(f * 16 + fidx, S::P2 - 1);
        a2_off[f] = S::at(2 * (r / G2::WO) + (wave >> 1), 2 * (r % G2::WO) + (wave & 1) * 2) + 4 * fk;
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- first layer
#pragma unroll
    for (int i = 0; i < S::IT; ++i) {
        uint4* dst = reinterpret_cast<uint4*>(img + min(tid + i * 512, S::CHUNKS - 1) * 16);
        dst[0] = u8x8_to_bf16(make_uint2(pre[i].x, pre[i].y));
        dst[1] = u8x8_to_bf16(make_uint2(pre[i].z, pre[i].w));
    }
    __syncthreads();
    const int col = cg * S::COLS + fidx * S::CT;        // this lane's first output channel of layer 2
    const float* const w2_base = W2 + (size_t)(wave * (S::KG * 16) + 4 * fk) * G2::COUT + col;
    vct w2[S::KG][4];
    // waves 4 .. 7 have the odd fragments, one fewer where their number is odd
    auto first_layer = [&](auto NF) __attribute__((always_inline)) {
        constexpr int nf = decltype(NF)::value;
        f32x16 acc[nf];
        bf16x8 a[2][nf];
        auto load_a = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < nf; ++f) {
                const uint2* ap = reinterpret_cast<const uint2*>(img + a1_off[f] + ks * 2 * G1::W);   // 8-byte aligned
                const uint2 lo = ap[0], hi = ap[1];
                a[ks & 1][f] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
            }
        };
        load_a(0);
#pragma unroll
        for (int f = 0; f < nf; ++f)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[f][q] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) load_a(ks + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 2; q >= 0; --q)
#pragma unroll
                for (int f = 0; f < nf; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[q][ks], a[ks & 1][f], acc[f], 0, 0, 0);
            // the second layer's weights, a part per k-step: requested all at once they held up the first MFMAs
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < S::KG; ++j) {
                const float* q = w2_base + (size_t)((ks * S::KG + j) / 4 * 16 + (ks * S::KG + j) % 4) * G2::COUT;
                if constexpr (S::CT == 1) w2[(ks * S::KG + j) / 4][(ks * S::KG + j) % 4][0] = *q;
                else w2[(ks * S::KG + j) / 4][(ks * S::KG + j) % 4] = *reinterpret_cast<const vct*>(q);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // register q of a lane: channel (q / 4) 8 + 4 half + q % 4 of position pidx
#pragma unroll
        for (int f = 0; f < nf; ++f)
            if ((f0 + 2 * f) * 32 + pidx < S::P1) {
#pragma unroll
                for (int g = 0; g < S::C1 / 8; ++g)
                    *reinterpret_cast<float4*>(act + s1_off[f] + 8 * g) = make_float4(acc[f][4 * g], acc[f][4 * g + 1], acc[f][4 * g + 2], acc[f][4 * g + 3]);
            }
    };
    if (f0 == 0) first_layer(std::integral_constant<int, S::FPW>());
    else first_layer(std::integral_constant<int, S::F1 / 2>());
    __syncthreads();
    // the first layer's output replaces the sums of input channel 0; rows that belong to this band (the last band
    // takes what is left) also go to global memory, where the backward pass reads them
    {
        float* const o1 = out1 + ((size_t)s * G1::HO + band * (2 * BR)) * (G1::WO * S::C1);
#pragma unroll
        for (int it = 0; it < ITI1; ++it) {
            const int e = tid + it * 512;
            if (e < ITEMS1) {
                float4 v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = *reinterpret_cast<const float4*>(act + p1_off[it][c]);
                const float4 r = make_float4(fmaxf((((v[0].x + v[1].x) + v[2].x) + v[3].x) * scale + bias1.x, 0.f),
                                             fmaxf((((v[0].y + v[1].y) + v[2].y) + v[3].y) * scale + bias1.y, 0.f),
                                             fmaxf((((v[0].z + v[1].z) + v[2].z) + v[3].z) * scale + bias1.z, 0.f),
                                             fmaxf((((v[0].w + v[1].w) + v[2].w) + v[3].w) * scale + bias1.w, 0.f));
                // the sums of input channel 0 are the first or the second addend
                *reinterpret_cast<float4*>(act + min(p1_off[it][0], p1_off[it][1])) = r;
                if (own1[it]) *reinterpret_cast<float4*>(o1 + (size_t)e * 4) = r;
            }
        }
    }
    __syncthreads();

    // ---- second layer
    {
        typename MM::Acc acc[S::F2][S::CT][2];
#pragma unroll
        for (int f = 0; f < S::F2; ++f)
#pragma unroll
            for (int t = 0; t < S::CT; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[f][t][h][r] = 0.f;
#pragma unroll
        for (int i = 0; i < S::KG; ++i) {
            float4 a[S::F2];
#pragma unroll
            for (int f = 0; f < S::F2; ++f)
                a[f] = *reinterpret_cast<const float4*>(act + a2_off[f] + (i * 16 / S::C1) * S::HALF + i * 16 % S::C1);
            auto mul = [&](int h, int j) __attribute__((always_inline)) {
#pragma unroll
                for (int f = 0; f < S::F2; ++f)
#pragma unroll
                    for (int t = 0; t < S::CT; ++t)
                        acc[f][t][h] = MM::mma(j == 0 ? a[f].x : j == 1 ? a[f].y : j == 2 ? a[f].z : a[f].w, w2[i][j][t], acc[f][t][h]);
            };
            mul(0, 0); mul(1, 1); mul(0, 2); mul(1, 3);
        }
        // accumulator register r: position f 16 + 4 fk + r, channel fidx CT + t
        float* const dst = sums + wave * S::PLANE2 + fidx * S::CT;
#pragma unroll
        for (int f = 0; f < S::F2; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vct v;
#pragma unroll
                for (int t = 0; t < S::CT; ++t) v[t] = acc[f][t][0][r] + acc[f][t][1][r];
                float* const q = dst + (f * 16 + 4 * fk + r) * S::PITCH2;
                if constexpr (S::CT == 1) *q = v[0];
                else *reinterpret_cast<vct*>(q) = v;
            }
    }
    __syncthreads();
    {
        constexpr int ITEMS = S::P2 * Q2, ITI = (ITEMS + 511) / 512;
        float* const o2 = out2 + ((size_t)s * (G2::HO * G2::WO) + band * S::P2) * G2::COUT + cg * S::COLS;
#pragma unroll
        for (int it = 0; it < ITI; ++it) {
            const int e = tid + it * 512;
            if (e < ITEMS) {
                const int p = e / Q2, c4 = e % Q2;
                const float* const q = sums + p * S::PITCH2 + c4 * 4;
                float4 v = *reinterpret_cast<const float4*>(q);
#pragma unroll
                for (int w = 1; w < 8; ++w) {
                    const float4 u = *reinterpret_cast<const float4*>(q + w * S::PLANE2);
                    v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
                }
                *reinterpret_cast<float4*>(o2 + (size_t)p * G2::COUT + c4 * 4) =
                    make_float4(fmaxf(v.x + bias2.x, 0.f), fmaxf(v.y + bias2.y, 0.f), fmaxf(v.z + bias2.z, 0.f), fmaxf(v.w + bias2.w, 0.f));
            }
        }
    }
}

template <class G1, class G2, int BR, int CG>
inline hipError_t launch_conv12_fwd_t(hipStream_t s, const uint8_t* x, const bf16_t* W1p, const float* b1, float* out1,
                                      const float* W2, const float* b2, float* out2, int ns) {
    typedef Conv12Shape<G1, G2, BR, CG> S;
    static const hipError_t ready = hipFuncSetAttribute(reinterpret_cast<const void*>(conv12_fwd_kernel<G1, G2, BR, CG>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);   // more than the default
    if (ready != hipSuccess) return ready;
    launch_k_lds((conv12_fwd_kernel<G1, G2, BR, CG>), dim3(ns * S::BANDS * CG), dim3(512), S::LDS, s, x, W1p, b1, out1, W2, b2, out2, ns,
                 1.0f / 255.0f, (int)(ns * 10 <= 2 * device_cus()));
    return hipGetLastError();
}

// The finest split whose workgroups all find a compute unit of their own: a second one on a unit has to wait
// for the first (registers and LDS hold one, except in bands of one row), and the launch takes twice as long
// (arch_nature, 42 -> 43 samples in halves of the channels: 9.2 -> 15 us, undivided 11 us).  Bands of one row compute the
// first layer 1.8 times over, bands of three 1.2 times.
template <class G1, class G2>
inline hipError_t launch_conv12_fwd(hipStream_t s, const uint8_t* x, const bf16_t* W1p, const float* b1, float* out1,
                                    const float* W2, const float* b2, float* out2, int ns) {
    if (ns <= 0 || ns > kConv12MaxSamples) return hipErrorInvalidValue;
    const int bands = G2::HO, cus = device_cus();
    if constexpr (G2::COUT == 64) {
        if (ns * bands * 4 <= cus) return launch_conv12_fwd_t<G1, G2, 1, 4>(s, x, W1p, b1, out1, W2, b2, out2, ns);
        if (ns * bands * 2 <= cus) return launch_conv12_fwd_t<G1, G2, 1, 2>(s, x, W1p, b1, out1, W2, b2, out2, ns);
        if (ns * (bands / 3) * 4 <= cus) return launch_conv12_fwd_t<G1, G2, 3, 4>(s, x, W1p, b1, out1, W2, b2, out2, ns);
    } else {
        if (ns * bands * 2 <= cus) return launch_conv12_fwd_t<G1, G2, 1, 2>(s, x, W1p, b1, out1, W2, b2, out2, ns);
        if (ns * bands <= cus) return launch_conv12_fwd_t<G1, G2, 1, 1>(s, x, W1p, b1, out1, W2, b2, out2, ns);
    }
    if (ns * (bands / 3) * 2 <= cus) return launch_conv12_fwd_t<G1, G2, 3, 2>(s, x, W1p, b1, out1, W2, b2, out2, ns);
    return launch_conv12_fwd_t<G1, G2, 3, 1>(s, x, W1p, b1, out1, W2, b2, out2, ns);
}

}  // namespace paac
