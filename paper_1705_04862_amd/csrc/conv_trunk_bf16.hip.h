// All convolutions of the bf16 path in one launch: a workgroup takes whole samples, and a layer's output goes to
// the next layer through LDS (to global memory only where the backward pass reads it).
//
// As launches of their own the layers move every activation twice: 106 KB of traffic per sample and train step of
// arch_nature against 70 here, 100 per selection against 34, and a launch boundary (2.5 us) between them.
// All convolutions, launches of their own -> one launch: arch_nature, selection n_e = 256 19.1 -> 11.3 us, n_e = 1024
// 43 -> 27.8; train step of 1536 states 50 -> 34 us, of 21504 states 495 -> 397 (its traffic alone takes 310 at the
// rate of a large copy); arch_nips, selection n_e = 256 12.3 -> 8 us, train step of 21504 states 304 -> 180.
//
// Roles.  One wave per SIMD runs the first layer of sample n + 1 (FIRST), the other the layers behind it for
// sample n (REST): the matrix pipe of a SIMD is shared, and while one of the two converts, exchanges sums, packs
// or waits at a barrier the other multiplies.  The first layer's output image is double-buffered between them.
// Every wave keeps its weights in registers for all samples.
//   FIRST: the sample's bytes (requested two samples ahead) -> bf16 in LDS in their own order; 16x16x32 MFMAs,
//     weights as operand A, the eight k of a lane are an eight-element piece of an image row.  Fragments of 16
//     positions: 400 positions are 25 of them, without remainder.
//   REST: 32x32x16 MFMAs on position-major images with the channels contiguous (second layer: columns of one parity
//     together; pitches that let sixteen lanes read sixteen different bank groups, also across the end of an output
//     row), the four waves are (32 output channels) x (share of the k-steps); the shares are added through LDS,
//     each wave finishing its part of the channels.
// Rows of operand A are output channels in an order that gives a lane neighbouring channels of one position:
// results are packed, written to LDS and stored 8 or 16 bytes at a time.
// Bound per sample of arch_nature, of about 8000 cycles: 4500 of MFMA per SIMD, 5000 of LDS traffic (a fragment from
// LDS feeds 32 cycles of MFMA in every layer), 4500 of vector instructions (5.4 cycles each for a wave alone, 4.5
// for two on a SIMD; conversion of the bytes, packing, sums), spread over four phases between barriers.
// Converting the bytes on their way from LDS to the MFMA instead (half the LDS traffic of the image) takes 12
// instructions per fragment and was slower: 8600 cycles per sample, arch_nips 252 us instead of 194.
#pragma once
#include "gemm_bf16.hip.h"

namespace paac {

// One layer behind the first, for the four REST waves.
template <class G> struct TrunkLayer {
    static_assert((G::ST == 1 || (G::ST == 2 && G::W % 2 == 0 && G::H % 2 == 0)) && G::CIN % 16 == 0 && G::COUT % 32 == 0 && G::COUT <= 64, "layer shape");
    static constexpr int PI = G::CIN + 8;                                  // position pitch: an odd multiple of 16 bytes
    static constexpr int NB = G::COUT / 32, KW = 4 / NB, GPO = 4 / KW;     // column blocks, k-shares, register groups finished per wave
    static constexpr int CSI = G::CIN / 16, KSTEPS = G::KS * G::KS * CSI, KPW = KSTEPS / KW;
    static_assert(KSTEPS % KW == 0, "equal k-shares");
    static constexpr int COUT = G::COUT, ROWS = G::HO * G::WO, FRAGS = (ROWS + 31) / 32;
    static constexpr int RP = G::ST == 1 ? bank_continuing_pitch(G::W * PI, G::WO, PI / 8) : bank_continuing_pitch(2 * G::W * PI, G::WO, PI / 8);
    static constexpr int IMG = (G::ST == 1 ? G::H : G::H / 2) * RP;        // elements of the input image
    static constexpr int SLOTS = KW == 2 ? 1 : KW;                         // shares that reach a finishing wave through LDS (see give)
    static constexpr int RED = NB * KW * SLOTS * FRAGS * GPO * 64 * 16;    // bytes of the exchange
    static constexpr int NCH = 4 * GPO;                                    // neighbouring channels a lane finishes
    typedef unsigned Out __attribute__((ext_vector_type(NCH / 2)));

    static __device__ __forceinline__ constexpr int at(int y, int x) {
        return G::ST == 2 ? (y >> 1) * RP + (((y & 1) * 2 + (x & 1)) * (G::W / 2) + (x >> 1)) * PI : y * RP + x * PI;
    }
    static __device__ __forceinline__ constexpr int koff(int ks) {         // k-step ks = (ky, kx, channel group)
        const int tap = ks / CSI;
        return at(tap / G::KS, tap % G::KS) + ks % CSI * 16;
    }
    // Share kg is the k-steps from kg KPW on.  Where that is whole rows of taps its LDS offsets are those of share 0 plus
    // a constant; else (third layer: four and a half taps) a step's offset depends on the share.
    static_assert(KW <= 2 || CSI == 1, "steps of shares that are not whole rows: two shares");
    static constexpr bool ROWS_OF_TAPS = KPW % (G::KS * CSI) == 0 && (G::ST == 1 || KW == 4 || KPW / (G::KS * CSI) % 2 == 0);
    static __device__ __forceinline__ int share_off(int kg, int i) {       // what step i of share kg has more than step i of share 0
        return kg == 0 ? 0 : kg == 1 ? koff(KPW + i) - koff(i) : kg == 2 ? koff(2 * KPW + i) - koff(i) : koff(3 * KPW + i) - koff(i);
    }
    // Channel (of a block of 32) in row r of operand A: the GPO register groups from j GPO on are finished by wave
    // (kg + j) mod KW, the wave's own are the first; a lane's channels follow each other
    static __device__ __forceinline__ int channel(int r, int kg) {
        const int g = r >> 3, h = (r >> 2) & 1;
        return (kg + g / GPO) % KW * (8 * GPO) + h * (4 * GPO) + g % GPO * 4 + (r & 3);
    }

    int lane, kg, first_ch;           // k-share of the wave; first channel this lane finishes
    int a_off[FRAGS];
    bf16x8 w[KPW];
    const float* bias;                // LDS
    float4 *give_at[KW], *take_at;    // this lane's 16 bytes of the exchange's slots: j-th other wave, own

    __device__ __forceinline__ void init(const bf16_t* __restrict__ Wt, int img_off, const float* bias_lds, float* red, int wave, int lane_) {
        lane = lane_; kg = wave / NB;
        const int nb = wave % NB, m = lane & 31, half = lane >> 5;
#pragma unroll
        for (int i = 0; i < KPW; ++i)                                      // weights as [k / 8][channel][8]
            w[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(
                Wt + ((size_t)((kg * KPW + i) * 2 + half) * G::COUT + nb * 32 + channel(m, kg)) * 8));
        first_ch = nb * 32 + kg * (8 * GPO) + half * (4 * GPO);
        bias = bias_lds + first_ch;
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) {
            const int r = min(f * 32 + m, ROWS - 1);                       // positions past the map: a valid one, never stored
            a_off[f] = at(r / G::WO * G::ST, r % G::WO * G::ST) + half * 8 + img_off + (ROWS_OF_TAPS ? share_off(kg, 0) : 0);
        }
        float4* const slots = reinterpret_cast<float4*>(red) + lane;       // [block][finishing wave][SLOTS][FRAGS][GPO][64]
#pragma unroll
        for (int j = 0; j < KW; ++j) give_at[j] = slots + ((nb * KW + (kg + j) % KW) * SLOTS + (KW == 2 ? 0 : kg)) * (FRAGS * GPO * 64);
        take_at = slots + (nb * KW + kg) * SLOTS * (FRAGS * GPO * 64);
    }

    // A fragment's registers are loaded again as soon as its MFMA has been issued, for two k-steps later: the
    // way from LDS is longer than the MFMAs of one step.
    __device__ __forceinline__ void multiply(const bf16_t* img, f32x16 (&acc)[FRAGS]) const {
        u32x4 a[2][FRAGS];
        int at_f[FRAGS];
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) at_f[f] = a_off[f];
        auto load = [&](int i, int f) __attribute__((always_inline)) {     // (in ascending order of i)
            if (!ROWS_OF_TAPS && (i == 0 || koff(KPW + i) - koff(i) != koff(KPW + i - 1) - koff(i - 1))) at_f[f] = a_off[f] + share_off(kg, i);
            a[i & 1][f] = *reinterpret_cast<const u32x4*>(img + at_f[f] + koff(i));
        };
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int f = 0; f < FRAGS; ++f) load(i, f);
#pragma unroll
        for (int f = 0; f < FRAGS; ++f)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[f][q] = 0.f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < KPW; ++i)
#pragma unroll
            for (int f = 0; f < FRAGS; ++f) {
                acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[i], __builtin_bit_cast(bf16x8, a[i & 1][f]), acc[f], 0, 0, 0);
                if (i + 2 < KPW) load(i + 2, f);
                __builtin_amdgcn_sched_barrier(0);
            }
    }

    // Shares are added in the order of the waves.  Of two, either order is the same sum, and the finishing wave's own
    // stays in its registers; of four, it passes through LDS with the others.
    __device__ __forceinline__ void give(const f32x16 (&acc)[FRAGS]) const {
#pragma unroll
        for (int j = KW == 2 ? 1 : 0; j < KW; ++j)
#pragma unroll
            for (int f = 0; f < FRAGS; ++f)
#pragma unroll
                for (int gi = 0; gi < GPO; ++gi) {
                    const int q = 4 * (j * GPO + gi);
                    give_at[j][(f * GPO + gi) * 64] = make_float4(acc[f][q], acc[f][q + 1], acc[f][q + 2], acc[f][q + 3]);
                }
    }
    // sum, bias, ReLU, bf16: emit(position, packed channels first_ch ..)
    template <class F> __device__ __forceinline__ void take(const f32x16 (&acc)[FRAGS], F&& emit) const {
        int m = lane & 31;
        asm volatile("" : "+v"(m));        // what emit derives from the position is computed here, not kept in registers from sample to sample
        float4 u[FRAGS][GPO][SLOTS], b[GPO];
#pragma unroll
        for (int gi = 0; gi < GPO; ++gi) b[gi] = *reinterpret_cast<const float4*>(bias + gi * 4);
#pragma unroll
        for (int f = 0; f < FRAGS; ++f)
#pragma unroll
            for (int gi = 0; gi < GPO; ++gi)
#pragma unroll
                for (int j = 0; j < SLOTS; ++j) u[f][gi][j] = take_at[((j * FRAGS + f) * GPO + gi) * 64];
#pragma unroll
        for (int f = 0; f < FRAGS; ++f) {
            Out o;
#pragma unroll
            for (int gi = 0; gi < GPO; ++gi) {
                float4 v = u[f][gi][0];
                if (KW == 2) { v.x += acc[f][4 * gi]; v.y += acc[f][4 * gi + 1]; v.z += acc[f][4 * gi + 2]; v.w += acc[f][4 * gi + 3]; }
#pragma unroll
                for (int j = 1; j < SLOTS; ++j) { v.x += u[f][gi][j].x; v.y += u[f][gi][j].y; v.z += u[f][gi][j].z; v.w += u[f][gi][j].w; }
                o[gi * 2] = pack2(fmaxf(v.x + b[gi].x, 0.f), fmaxf(v.y + b[gi].y, 0.f));
                o[gi * 2 + 1] = pack2(fmaxf(v.z + b[gi].z, 0.f), fmaxf(v.w + b[gi].w, 0.f));
            }
            const int r = f * 32 + m;
            if (r < ROWS) emit(r, o);
        }
    }
};

// G3 = NoThirdLayer: two layers.
struct NoThirdLayer {};
template <class G1, class G2, class G3> struct TrunkB {
    static_assert(G1::CIN == 4 && G1::H == 84 && G1::W == 84 && G1::KS == 8 && G1::ST == 4 && (G1::COUT == 16 || G1::COUT == 32), "first layer");
    static_assert(G2::H == G1::HO && G2::W == G1::WO && G2::CIN == G1::COUT, "layer 1 feeds layer 2");
    static constexpr bool L3 = !std::is_same<G3, NoThirdLayer>::value;
    typedef TrunkLayer<G2> T2;
    typedef TrunkLayer<std::conditional_t<L3, G3, G2>> T3;
    static constexpr int SAMPLE = 4 * G1::H * G1::W, CHUNKS = SAMPLE / 16, IT = (CHUNKS + 255) / 256;
    static constexpr int NCB = G1::COUT / 16, POS = G1::HO * G1::WO;
    static_assert(G1::HO == 20 && G1::WO == 20 && SAMPLE % 16 == 0, "five groups of four columns, five rows apart; whole chunks");
    static constexpr int IMG1 = SAMPLE * 2, IMG2 = T2::IMG * 2, IMG3 = L3 ? T3::IMG * 2 : 0;
    static constexpr int RED = L3 && T3::RED > T2::RED ? T3::RED : T2::RED;
    static constexpr int BIAS = (G2::COUT + (L3 ? G2::COUT : 0)) * 4;       // of the layers behind the first
    static constexpr int LDS = IMG1 + 2 * IMG2 + IMG3 + RED + BIAS;
    static_assert(IMG1 % 16 == 0 && IMG2 % 16 == 0 && IMG3 % 16 == 0 && LDS <= 160 * 1024, "fits the LDS of a compute unit");
};

template <class G1, class G2, class G3>
__global__ __launch_bounds__(512, 2) void conv_trunk_bf16_kernel(const uint8_t* __restrict__ x, const bf16_t* __restrict__ W1, const float* __restrict__ b1,
                                                                 bf16_t* __restrict__ out1, const bf16_t* __restrict__ W2, const float* __restrict__ b2,
                                                                 bf16_t* __restrict__ out2, const bf16_t* __restrict__ W3, const float* __restrict__ b3,
                                                                 bf16_t* __restrict__ out3, int ns, float scale) {
    typedef TrunkB<G1, G2, G3> S;
    typedef typename S::T2 T2;
    typedef typename S::T3 T3;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    bf16_t* const img1 = reinterpret_cast<bf16_t*>(lds_raw);
    bf16_t* const img2 = reinterpret_cast<bf16_t*>(lds_raw + S::IMG1);                        // two of them
    bf16_t* const img3 = reinterpret_cast<bf16_t*>(lds_raw + S::IMG1 + 2 * S::IMG2);
    float* const red = reinterpret_cast<float*>(lds_raw + S::IMG1 + 2 * S::IMG2 + S::IMG3);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s0 = blockIdx.x, step = gridDim.x;
    if (s0 >= ns) return;
    const int count = (ns - s0 + step - 1) / step;        // samples of this workgroup; both roles pass every barrier of count + 1 turns

    if (wave < 4) {
        // ---- FIRST
        const int tid = threadIdx.x, p16 = lane & 15, g4 = lane >> 4;
        u32x4 pre[S::IT];
        auto request = [&](int n) __attribute__((always_inline)) {        // past the end: the last sample again, not used
            const uint8_t* base = x + (size_t)(s0 + min(n, count - 1) * step) * S::SAMPLE;
#pragma unroll
            for (int i = 0; i < S::IT; ++i) pre[i] = *reinterpret_cast<const u32x4*>(base + (size_t)min(tid + i * 256, S::CHUNKS - 1) * 16);
        };
        auto deposit = [&](auto I0_, auto I1_) __attribute__((always_inline)) {          // threads past the last chunk repeat it
#pragma unroll
            for (int i = decltype(I0_)::value; i < decltype(I1_)::value; ++i) {
                uint4* d = reinterpret_cast<uint4*>(img1 + min(tid + i * 256, S::CHUNKS - 1) * 16);
                d[0] = u8x8_to_bf16(make_uint2(pre[i].x, pre[i].y));
                d[1] = u8x8_to_bf16(make_uint2(pre[i].z, pre[i].w));
            }
        };
        typedef std::integral_constant<int, 0> I0; typedef std::integral_constant<int, 3> I3; typedef std::integral_constant<int, 4> I4;
        typedef std::integral_constant<int, S::IT> All;
        // chunks of the first three channels only
        constexpr int EARLY = 3 * G1::H * G1::W / 16 / 256;
        typedef std::integral_constant<int, EARLY> Early;
        request(0);
        __builtin_amdgcn_sched_barrier(0);
        // row m of block cb: channel NCB 4 (m / 4) + 4 cb + m % 4, so a lane's registers are 4 NCB neighbouring channels
        bf16x8 w[8][S::NCB];
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int cb = 0; cb < S::NCB; ++cb)
                w[t][cb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(
                    W1 + ((size_t)(t * 4 + g4) * 32 + (p16 >> 2) * (4 * S::NCB) + cb * 4 + (p16 & 3)) * 8));
        const int ch = g4 * (4 * S::NCB);
        float bias[4 * S::NCB];
#pragma unroll
        for (int i = 0; i < 4 * S::NCB; ++i) bias[i] = b1[ch + i];
        // A fragment: the positions of four columns (4 group + p16 % 4) and four rows (r + 5 (p16 / 4)).  The values under
        // kernel rows 4 .. 7 of row r are those under kernel rows 0 .. 3 of row r + 1: a chain of fragments r0, r0 + 1, ..
        // reads every value once.  Each wave takes a chain of five in its own column group and a part of the fifth
        // group: wave 0 two fragments, the others one.
        const int r_last = wave == 0 ? 0 : wave + 1;
        auto column = [&](int group) { return group * 4 + (p16 & 3); };
        const int a_own = (20 * (p16 >> 2) + g4) * G1::W + column(wave) * 4;
        const int a_last = (20 * (p16 >> 2) + 4 * r_last + g4) * G1::W + column(4) * 4;
        // One channel after the other: its image is free for the next sample while the others are still worked on.
        constexpr int AHEAD = 4, STEPS = 8;                                // steps between a read from LDS and its use; steps per channel
        bf16x8 a[AHEAD], a_third;
        f32x4 acc[7][S::NCB];                                              // own chain, fifth group
        auto read = [&](int off) __attribute__((always_inline)) {
            const uint2* ap = reinterpret_cast<const uint2*>(img1 + off);  // 8-byte aligned
            const uint2 lo = ap[0], hi = ap[1];
            return __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
        };
        // step i: row block i % 8 of the own chain, or i % 8 - 6 of the fifth group's, in channel i / 8
        auto load = [&](int i) __attribute__((always_inline)) {
            const int c = i / STEPS, k = i % STEPS;
            a[i % AHEAD] = read((k < 6 ? a_own + k * (4 * G1::W) : a_last + (k - 6) * (4 * G1::W)) + c * (G1::H * G1::W));
        };
        auto mma = [&](f32x4 (&v)[S::NCB], int c, int odd, bf16x8 x) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < S::NCB; ++cb)
                v[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[2 * c + odd][cb], x, c == 0 && !odd ? f32x4{0.f, 0.f, 0.f, 0.f} : v[cb], 0, 0, 0);
        };
        auto channels = [&](auto C0_, auto C1_) __attribute__((always_inline)) {
            constexpr int C0 = decltype(C0_)::value, C1 = decltype(C1_)::value;
            if constexpr (C0 == 0) {
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) load(i);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = C0 * STEPS; i < C1 * STEPS; ++i) {
                const int c = i / STEPS, k = i % STEPS;
                const bf16x8 x = a[i % AHEAD];
                if (k < 5) mma(acc[k], c, 0, x);
                if (k > 0 && k < 6) mma(acc[k - 1], c, 1, x);
                if (k == 6) mma(acc[5], c, 0, x);
                if (k == 7) mma(acc[5], c, 1, x);
                if (i + AHEAD < 4 * STEPS) load(i + AHEAD);
                if (k == 4 && wave == 0) a_third = read(a_last + 2 * (4 * G1::W) + c * (G1::H * G1::W));
                if (k == 7 && wave == 0) { mma(acc[6], c, 0, x); mma(acc[6], c, 1, a_third); }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto emit = [&](const f32x4 (&v)[S::NCB], int r, int group, int n) __attribute__((always_inline)) {
            typedef unsigned Out __attribute__((ext_vector_type(2 * S::NCB)));
            Out o;
#pragma unroll
            for (int cb = 0; cb < S::NCB; ++cb)
#pragma unroll
                for (int q = 0; q < 4; q += 2)
                    o[cb * 2 + q / 2] = pack2(fmaxf(v[cb][q] * scale + bias[cb * 4 + q], 0.f), fmaxf(v[cb][q + 1] * scale + bias[cb * 4 + q + 1], 0.f));
            const int oy = r + 5 * (p16 >> 2), ox = column(group);
            *reinterpret_cast<Out*>(img2 + (n & 1) * T2::IMG + T2::at(oy, ox) + ch) = o;
            if (out1) *reinterpret_cast<Out*>(out1 + (size_t)(s0 + n * step) * (S::POS * G1::COUT) + (unsigned)((oy * G1::WO + ox) * G1::COUT + ch)) = o;
        };
        deposit(I0(), All());
        request(1);
        __syncthreads();                                                   // the first sample's bytes are in place
        for (int n = 0; n <= count; ++n) {
            const bool work = n < count;
            const bool more = n + 1 < count;
            // beside the other role's phases: second layer | its sums | third layer | its sums
            if constexpr (S::L3) {
                if (work) channels(I0(), I3());
                __syncthreads();                                           // three channels of the byte image are free
                if (work) channels(I3(), I4());
            } else if (work) channels(I0(), I4());
            if constexpr (!S::L3) __syncthreads();                         // all of it is free
            if (work) {
#pragma unroll
                for (int r = 0; r < 3; ++r) emit(acc[r], r, wave, n);
            }
            if constexpr (S::L3) __syncthreads();                          // all of it is free
            if (work) { emit(acc[3], 3, wave, n); emit(acc[4], 4, wave, n); emit(acc[5], r_last, 4, n); }
            if (work && wave == 0) emit(acc[6], r_last + 1, 4, n);
            if (more) deposit(I0(), Early());
            if constexpr (S::L3) __syncthreads();
            if (more) {
                deposit(Early(), All());
                request(n + 2);
            }
            __syncthreads();                                               // the output image and the next bytes are complete
        }
    } else {
        // ---- REST
        float* const bias = red + S::RED / 4;
        const int tid = threadIdx.x - 256;
        if (tid < G2::COUT) bias[tid] = b2[tid];                           // (the first barrier is long before they are read)
        if constexpr (S::L3) { if (tid < G3::COUT) bias[G2::COUT + tid] = b3[tid]; }
        int off3 = (S::IMG1 + 2 * S::IMG2) / 2;                       // a register: the instructions' offsets end before the third image
        asm volatile("" : "+s"(off3));
        T2 l2;
        l2.init(W2, 0, bias, red, wave - 4, lane);
        T3 l3;
        if constexpr (S::L3) l3.init(W3, off3, bias + G2::COUT, red, wave - 4, lane);
        __syncthreads();
        for (int n = 0; n <= count; ++n) {                                 // sample n - 1
            const bool work = n > 0;
            // (uniform base, 32-bit offset per lane: 64-bit addresses would take registers that the weights need)
            bf16_t* const o2 = out2 + (size_t)(s0 + (n - 1) * step) * (T2::ROWS * G2::COUT);
            bf16_t* const o3 = S::L3 ? out3 + (size_t)(s0 + (n - 1) * step) * (T3::ROWS * T3::COUT) : nullptr;
            f32x16 acc2[T2::FRAGS];
            if (work) {
                l2.multiply(img2 + ((n - 1) & 1) * T2::IMG, acc2);
                l2.give(acc2);
            }
            __syncthreads();
            if (work)
                l2.take(acc2, [&](int r, typename T2::Out o) __attribute__((always_inline)) {
                    if constexpr (S::L3) *reinterpret_cast<typename T2::Out*>(img3 + T3::at(r / G2::WO, r % G2::WO) + l2.first_ch) = o;
                    if (!S::L3 || out2) *reinterpret_cast<typename T2::Out*>(o2 + (unsigned)(r * G2::COUT + l2.first_ch)) = o;
                });
            __syncthreads();
            if constexpr (S::L3) {
                f32x16 acc3[T3::FRAGS];
                if (work) {
                    l3.multiply(reinterpret_cast<const bf16_t*>(lds_raw), acc3);
                    l3.give(acc3);
                }
                __syncthreads();
                if (work)
                    l3.take(acc3, [&](int r, typename T3::Out o) __attribute__((always_inline)) {
                        *reinterpret_cast<typename T3::Out*>(o3 + (unsigned)(r * G3::COUT + l3.first_ch)) = o;
                    });
                __syncthreads();
            }
        }
    }
}

// out1 (and, with three layers, out2) may be null: only the last layer's output is then written.
template <class G1, class G2, class G3>
inline hipError_t launch_conv_trunk_bf16(hipStream_t s, const uint8_t* x, const bf16_t* const* w, const float* const* b, bf16_t* const* out, int ns) {
    if (ns <= 0) return hipErrorInvalidValue;
    typedef TrunkB<G1, G2, G3> S;
    static const hipError_t ready = hipFuncSetAttribute(reinterpret_cast<const void*>(conv_trunk_bf16_kernel<G1, G2, G3>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);      // more than the default
    if (ready != hipSuccess) return ready;
    launch_k_lds((conv_trunk_bf16_kernel<G1, G2, G3>), dim3(std::min(ns, device_cus())), dim3(512), S::LDS, s, x, w[0], b[0], out[0], w[1], b[1], out[1],
                 S::L3 ? w[2] : nullptr, S::L3 ? b[2] : nullptr, S::L3 ? out[2] : nullptr, ns, 1.0f / 255.0f);
    return hipGetLastError();
}

}  // namespace paac
