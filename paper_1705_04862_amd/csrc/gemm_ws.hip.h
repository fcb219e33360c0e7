// Tiled fp32 GEMM on the fp32 matrix cores (v_mfma_f32_32x32x2f32) with wave roles: the backward pass of layers
// 2.. and of the fully connected layer of the fp32 path, and its fully connected forward pass from 65 rows on.
//
//   C[m][n] = sum_k A(m,k) * B(k,n)
//
// An fp32 MFMA holds the matrix pipe for 64 cycles, so these contractions are bound by it as soon as nothing else
// holds it up.  With four waves that load, write LDS and multiply in turn the pipe was busy 55-60 % of the time
// (64 x 64 tile: 1 750 cycles per 32-deep k tile for 1 024 cycles of MFMA): a wave issues in order, so address
// arithmetic, LDS writes, the barrier and the first fragments' LDS latency all stand between its MFMAs.  A
// workgroup is therefore eight waves with two roles, one of each on a SIMD: waves 4-7 load and write k tile
// g + 1 while waves 0-3 read the fragments of tile g and issue its MFMAs; two LDS buffers, one barrier per k
// tile.  The multiplying waves pass that barrier with the last fragments of their tile already in registers
// and request the next tile's first ones behind it, so the pipe does not drain there.  Two workgroups share a
// compute unit, one's multiplication covers the other's first loads and stores (persistent workgroups that walk over
// output tiles, loading the next one while the last is stored, were measured and are no faster).
//
// The additions of an output element run in the order that its tile says (TileW): ascending 32- or 64-deep k
// tiles, MFMA step 4 g + j of a wave taking k = 8 g + j and 8 g + 4 + j of its part of the tile, even and odd
// steps in separate accumulators where a wave has one fragment.  Tiles that agree in that give the same bits.
//
// LDS: an operand contiguous along k in memory (kContig) is kept row-major, [row][BK + 4] floats: 16-byte writes and
// 16-byte fragment reads of four k (the odd pitch in 16-byte words puts sixteen rows into sixteen bank groups); one
// contiguous along m / n is kept k-major, [k][rows + 4], written 16 bytes and read 4 bytes at a time.
// The fragments are multiplied as (B, A), which leaves the transposed tile in the accumulators: a lane
// holds one row m and groups of four consecutive n, so results leave as 16-byte stores and the address of
// a row is computed once per lane.
#pragma once
#include "gemm_bf16.hip.h"

namespace paac {

// BM x BN x BK tile; the four multiplying waves are WM along m, WN along n, WK along the k of a tile (their sums are added
// in wave order through LDS at the end); KACC accumulators per fragment, MFMA steps dealt to them in turn.
template <int BM_, int BN_, int BK_, int WM_, int WN_, int WK_, int KACC_>
struct TileW {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, WK = WK_, KACC = KACC_;
    static constexpr int TM = BM / (WM * 32), TN = BN / (WN * 32);
    static constexpr int NG = BK / WK / 8;                  // groups of four MFMA steps (8 k) of a wave per tile
    static constexpr int MFMA_PER_K = TM * TN * BK / 2 / WK; // MFMAs of a wave per k tile
    static_assert(WM * WN * WK == 4 && TM * WM * 32 == BM && TN * WN * 32 == BN, "four waves of whole fragments");
    static_assert(NG * WK * 8 == BK && NG % 2 == 0, "groups alternate between two register slots");
    static_assert(KACC == 1 || KACC == 2, "one accumulator, or even and odd steps apart");
};
constexpr int kWsStages = 2;        // k tiles of loads in flight behind the one in LDS (three and four: no faster, more registers)
constexpr int kWsPerCu = 2;         // workgroups on a compute unit

// ---------------------------------------------------------------------------------------------- operands
// Loads are raw buffer loads: 32-bit byte offsets against a descriptor of the tensor (all are below 4 GiB),
// and an offset past its end reads zeros, which is what a tap outside the map and the reduction indices
// behind the last one should give.
//   base(), bytes()                          the tensor
// kContig:   unsigned prep(row, dk, z, Pos&)   per-thread offset (row, and dk inside the k tile); rows past the end
//                                          are clamped to a valid one (their results are not stored)
//            Uni uni(kb)                   wave-uniform part, kb = first k of the tile
//            unsigned off(voff, Pos, Uni)  per-thread offset of this tile, soff(Uni) its uniform rest
//   kSpan: consecutive k that the uniform part holds for, a multiple of 32 (0: all of them); with a longer k tile a
//   thread takes the part of its own 32 k.  K is a multiple of BK
// !kContig:  unsigned prep(col, z), unsigned entry(r) (offset of reduction index r; past the end: past the tensor)
//   kTab: entry() needs divisions; the kernel keeps the entries of the coming k tiles in an LDS table
struct WsNoPos {};
constexpr unsigned kOutside = 0xffffff00u;     // past the end of every tensor

struct WsDenseRows {             // element (row, k) = data[row*ld + k]
    static constexpr bool kContig = true, kTab = false;
    static constexpr int kSpan = 0;
    const float* data; int rows, ld;
    __device__ __forceinline__ const float* base() const { return data; }
    __device__ __forceinline__ unsigned bytes() const { return (unsigned)rows * (unsigned)ld * 4u; }
    typedef WsNoPos Pos;
    struct Uni { unsigned s; };
    __device__ __forceinline__ unsigned prep(int row, int dk, int, Pos&) const { return ((unsigned)min(row, rows - 1) * (unsigned)ld + dk) * 4u; }
    __device__ __forceinline__ Uni uni(int kb) const { return Uni{(unsigned)kb * 4u}; }
    __device__ __forceinline__ unsigned off(unsigned v, const Pos&, const Uni&) const { return v; }
    __device__ __forceinline__ unsigned soff(const Uni& u) const { return u.s; }
};

// im2col rows of a float NHWC activation, k = (ky, kx, c): contiguous over a kernel row
template <class G> struct WsConvRows {
    static constexpr bool kContig = true, kTab = false;
    static constexpr int kSpan = G::KS * G::CIN;
    const float* x; int ns;
    __device__ __forceinline__ const float* base() const { return x; }
    __device__ __forceinline__ unsigned bytes() const { return (unsigned)ns * (G::H * G::W * G::CIN * 4u); }
    typedef WsNoPos Pos;
    struct Uni { unsigned s; };
    __device__ __forceinline__ unsigned prep(int row, int dk, int, Pos&) const {
        const unsigned q = (unsigned)min(row, ns * (G::HO * G::WO) - 1), n = q / (G::HO * G::WO), r = q % (G::HO * G::WO), oy = r / G::WO, ox = r % G::WO;
        return (((n * G::H + oy * G::ST) * G::W + ox * G::ST) * G::CIN + dk) * 4u;
    }
    __device__ __forceinline__ Uni uni(int kb) const {
        const unsigned ky = (unsigned)kb / (G::KS * G::CIN), rem = (unsigned)kb % (G::KS * G::CIN);
        return Uni{(unsigned)(ky * (G::W * G::CIN) + rem) * 4u};
    }
    __device__ __forceinline__ unsigned off(unsigned v, const Pos&, const Uni&) const { return v; }
    __device__ __forceinline__ unsigned soff(const Uni& u) const { return u.s; }
};

// Data gradient, gather form.  Row = (n, yy, xx); k = (ty, tx, co); value = dY[n][yy - ty][xx - tx][co] where
// that output position exists, else 0.
template <class G> struct WsDgradRows {
    static constexpr bool kContig = true, kTab = false;
    static constexpr int kSpan = G::COUT;
    const float* dy; int ns;
    __device__ __forceinline__ const float* base() const { return dy; }
    __device__ __forceinline__ unsigned bytes() const { return (unsigned)ns * (G::HO * G::WO * G::COUT * 4u); }
    struct Pos { int yy, xx; };
    struct Uni { unsigned add; int ty, tx; };
    __device__ __forceinline__ unsigned prep(int row, int dk, int, Pos& p) const {
        const unsigned q = (unsigned)min(row, ns * (G::HC * G::WC) - 1), n = q / (G::HC * G::WC), r = q % (G::HC * G::WC);
        p.yy = r / G::WC; p.xx = r % G::WC;
        return (((n * G::HO + p.yy) * G::WO + p.xx) * G::COUT + dk) * 4u;
    }
    __device__ __forceinline__ Uni uni(int kb) const {
        const int tap = (unsigned)kb / G::COUT, co = (unsigned)kb % G::COUT;
        Uni u; u.ty = (unsigned)tap / G::TAPS; u.tx = (unsigned)tap % G::TAPS;
        u.add = (unsigned)(co - (u.ty * G::WO + u.tx) * G::COUT) * 4u;      // may be below zero: added modulo 2^32
        return u;
    }
    __device__ __forceinline__ unsigned off(unsigned v, const Pos& p, const Uni& u) const {
        const bool ok = (unsigned)(p.yy - u.ty) < (unsigned)G::HO && (unsigned)(p.xx - u.tx) < (unsigned)G::WO;
        return ok ? v + u.add : kOutside;
    }
    __device__ __forceinline__ unsigned soff(const Uni&) const { return 0u; }
};

// Weights seen by the data gradient, all ST*ST parity classes as columns: B(k = (ty,tx,co), n = (z,ci)) =
// W[(ky,kx,ci)][co] with ky = py + ST*ty, kx = px + ST*tx for class z = py*ST + px.
template <class G> struct WsDgradWeights {
    static constexpr bool kContig = true, kTab = false;
    static constexpr int kSpan = G::COUT;
    const float* w;
    __device__ __forceinline__ const float* base() const { return w; }
    __device__ __forceinline__ unsigned bytes() const { return G::KK * G::COUT * 4u; }
    typedef WsNoPos Pos;
    struct Uni { unsigned s; };
    __device__ __forceinline__ unsigned prep(int col, int dk, int, Pos&) const {
        const unsigned q = (unsigned)min(col, G::ST * G::ST * G::CIN - 1), z = q / G::CIN, ci = q % G::CIN, py = z / G::ST, px = z % G::ST;
        return (((py * G::KS + px) * G::CIN + ci) * G::COUT + dk) * 4u;
    }
    __device__ __forceinline__ Uni uni(int kb) const {
        const unsigned tap = (unsigned)kb / G::COUT, co = (unsigned)kb % G::COUT, ty = tap / G::TAPS, tx = tap % G::TAPS;
        return Uni{(unsigned)((ty * G::ST * G::KS + tx * G::ST) * (G::CIN * G::COUT) + co) * 4u};
    }
    __device__ __forceinline__ unsigned off(unsigned v, const Pos&, const Uni&) const { return v; }
    __device__ __forceinline__ unsigned soff(const Uni& u) const { return u.s; }
};

struct WsDenseCols {             // element (k, col) = data[k*ld + col], k < rows
    static constexpr bool kContig = false, kTab = false;
    static constexpr int kSpan = 0;
    const float* data; int rows, cols, ld;
    __device__ __forceinline__ const float* base() const { return data; }
    __device__ __forceinline__ unsigned bytes() const { return (unsigned)rows * (unsigned)ld * 4u; }
    typedef WsNoPos Pos;
    __device__ __forceinline__ unsigned prep(int col, int) const { return (unsigned)min(col, cols - 4) * 4u; }
    __device__ __forceinline__ unsigned entry(int r) const { return (unsigned)r * (unsigned)ld * 4u; }
};

// Weight gradient of the later conv layers: A(m = (ky,kx,c), k = output position) from NHWC input.
template <class G> struct WsConvCols {
    static constexpr bool kContig = false, kTab = true;
    static constexpr int kSpan = 0;
    const float* x; int ns;
    __device__ __forceinline__ const float* base() const { return x; }
    __device__ __forceinline__ unsigned bytes() const { return (unsigned)ns * (G::H * G::W * G::CIN * 4u); }
    typedef WsNoPos Pos;
    __device__ __forceinline__ unsigned prep(int col, int) const {
        col = min(col, G::KK - 4);
        const int ky = col / (G::KS * G::CIN), rem = col % (G::KS * G::CIN);
        return (unsigned)(ky * (G::W * G::CIN) + rem) * 4u;
    }
    __device__ __forceinline__ unsigned entry(int row) const {
        const unsigned q = row, n = q / (G::HO * G::WO), r = q % (G::HO * G::WO), oy = r / G::WO, ox = r % G::WO;
        return ((n * G::H + oy * G::ST) * G::W + ox * G::ST) * (G::CIN * 4u);
    }
};

// ---------------------------------------------------------------------------------------------- epilogues
// out[row_off(row, z) + col_off(8-column group) + column in the group] (element offsets); N is a multiple of 8
template <bool COLSUM> struct WsPartial {      // out[z][row][col] = v ; optional column sums of B
    static constexpr bool kMask = false, kColSum = COLSUM;
    float* out; unsigned z_stride; int ldo; float* colsum; int colsum_stride;
    __device__ __forceinline__ unsigned row_off(int row, int z) const { return (unsigned)z * z_stride + (unsigned)row * (unsigned)ldo; }
    __device__ __forceinline__ unsigned col_off(int col) const { return (unsigned)col; }
    __device__ __forceinline__ float* dst() const { return out; }
    __device__ __forceinline__ const float* mask() const { return nullptr; }
    __device__ __forceinline__ void store_colsum(int col, float v, int z) const { colsum[(size_t)z * colsum_stride + col] = v; }
};
struct WsDenseMask {                           // out[row][col] = act[row][col] > 0 ? v : 0
    static constexpr bool kMask = true, kColSum = false;
    float* out; const float* act; int ld;
    __device__ __forceinline__ unsigned row_off(int row, int) const { return (unsigned)row * (unsigned)ld; }
    __device__ __forceinline__ unsigned col_off(int col) const { return (unsigned)col; }
    __device__ __forceinline__ float* dst() const { return out; }
    __device__ __forceinline__ const float* mask() const { return act; }
};
template <class G> struct WsDgradMask {        // columns n = (z, ci) of all parity classes back to NHWC, times ReLU'
    static constexpr bool kMask = true, kColSum = false;
    static_assert(G::CIN % 8 == 0, "eight columns stay in one class");
    float* dx; const float* act;
    __device__ __forceinline__ unsigned row_off(int row, int) const {
        const unsigned q = row, n = q / (G::HC * G::WC), r = q % (G::HC * G::WC), yy = r / G::WC, xx = r % G::WC;
        return ((n * G::H + yy * G::ST) * G::W + xx * G::ST) * G::CIN;
    }
    __device__ __forceinline__ unsigned col_off(int col) const {
        const int z = col / G::CIN, ci = col % G::CIN;
        return (unsigned)(((z / G::ST) * G::W + z % G::ST) * G::CIN + ci);
    }
    __device__ __forceinline__ float* dst() const { return dx; }
    __device__ __forceinline__ const float* mask() const { return act; }
};

// ---------------------------------------------------------------------------------------------- kernel body
// A GEMM with its launch shape, as a value.  Items are (output tile, k-split), tiles fastest.
template <class T_, class AL_, class BL_, class EP_> struct GemmWs {
    typedef T_ T; typedef AL_ AL; typedef BL_ BL; typedef EP_ EP;
    AL al; BL bl; EP ep;
    int M, N, K, z_count, k_per_split;
    __host__ __device__ int m_tiles() const { return (M + T::BM - 1) / T::BM; }
    __host__ __device__ int tiles() const { return m_tiles() * ((N + T::BN - 1) / T::BN); }
    __host__ __device__ int items() const { return tiles() * z_count; }
    int item_mfmas() const { return ((k_per_split > 0 ? k_per_split : K) + T::BK - 1) / T::BK * T::MFMA_PER_K; }      // of a wave
    // operands contiguous along k are read in whole k tiles, the others run into the zeros behind the tensor
    bool valid() const {
        return M > 0 && N > 0 && N % 8 == 0 && K > 0 && z_count > 0 && k_per_split % T::BK == 0 && (!(AL::kContig || BL::kContig) || K % T::BK == 0) &&
               (z_count == 1 || (k_per_split > 0 && (z_count - 1) * (long)k_per_split < K));
    }
};
template <class T, class AL, class BL, class EP>
inline GemmWs<T, AL, BL, EP> gemm_ws(const AL& al, const BL& bl, const EP& ep, int M, int N, int K, int z, int k_per) {
    return GemmWs<T, AL, BL, EP>{al, bl, ep, M, N, K, z, k_per};
}

template <class C> struct WsSmem {
    typedef typename C::T T;
    static constexpr int LDA = C::AL::kContig ? T::BK + 4 : T::BM + 4, LDB = C::BL::kContig ? T::BK + 4 : T::BN + 4;      // floats
    static constexpr int A_BUF = C::AL::kContig ? T::BM * LDA : T::BK * LDA, B_BUF = C::BL::kContig ? T::BN * LDB : T::BK * LDB;
    static constexpr int BUF = A_BUF + B_BUF;
    static constexpr int TAB_SLOTS = kWsStages + 1;    // table slots: k tile j lives in slot j % TAB_SLOTS
    static constexpr int TAB = C::AL::kTab ? TAB_SLOTS * T::BK : 0;
    static constexpr int BYTES = (2 * BUF + TAB) * 4;
    static_assert(BYTES * kWsPerCu <= 160 * 1024, "fits the LDS of a compute unit");
    static_assert((T::WK - 1) * T::WM * T::WN * T::TM * T::TN * 1024 <= 2 * BUF, "the k-waves' sums reuse the tile buffers");
};

// Item `idx` of call c; 512 threads.
template <class C>
__device__ __forceinline__ void gemm_ws_run(const C& c, int idx, float* smem) {
    typedef typename C::T T; typedef typename C::AL AL; typedef typename C::BL BL; typedef typename C::EP EP;
    typedef WsSmem<C> L;
    constexpr int BM = T::BM, BN = T::BN, BK = T::BK, TM = T::TM, TN = T::TN, S = kWsStages;
    static_assert(!AL::kTab || !AL::kContig, "tables are for operands contiguous along m");
    static_assert(!BL::kTab, "operand B has no table");
    static_assert(AL::kSpan % 32 == 0 && BL::kSpan % 32 == 0, "uniform offsets hold for 32 k");
    constexpr bool A_PER_LANE = AL::kSpan % BK != 0, B_PER_LANE = BL::kSpan % BK != 0;

    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m_tiles = c.m_tiles(), tiles = c.tiles();
    const int z = (unsigned)idx / (unsigned)tiles, tile = idx - z * tiles, nt = (unsigned)tile / (unsigned)m_tiles;
    const int m0 = (tile - nt * m_tiles) * BM, n0 = nt * BN;
    const int k_begin = c.k_per_split > 0 ? z * c.k_per_split : 0;
    const int k_end = c.k_per_split > 0 ? min(c.K, k_begin + c.k_per_split) : c.K;
    const int nk = (unsigned)(k_end - k_begin + BK - 1) / BK;

    if (wave >= 4) {
        // ======================= waves 4-7: global memory -> registers -> LDS =======================
        const int tid = (int)threadIdx.x - 256;
        // staging units of 16 bytes: four k of one row, or four columns at one k; lanes along the contiguous side
        constexpr int A_U = BM * BK / 4, B_U = BN * BK / 4, A_IT = A_U / 256, B_IT = B_U / 256;
        static_assert(A_U % 256 == 0 && B_U % 256 == 0, "whole rounds of the 256 threads");
        const __amdgpu_buffer_rsrc_t a_res = __builtin_amdgcn_make_buffer_rsrc((void*)c.al.base(), 0, c.al.bytes(), 0x00027000);
        const __amdgpu_buffer_rsrc_t b_res = __builtin_amdgcn_make_buffer_rsrc((void*)c.bl.base(), 0, c.bl.bytes(), 0x00027000);
        auto fetch = [](__amdgpu_buffer_rsrc_t res, unsigned voff, unsigned soff) __attribute__((always_inline)) {
            return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(res, voff, soff, 0));
        };
        unsigned a_off[A_IT], b_off[B_IT];
        typename AL::Pos a_pos[A_IT];
        typename BL::Pos b_pos[B_IT];
        int a_lds[A_IT], b_lds[B_IT], a_k[A_IT], b_k[B_IT];
#pragma unroll
        for (int i = 0; i < A_IT; ++i) {
            const int f = tid + i * 256;
            if constexpr (AL::kContig) {
                const int row = f / (BK / 4); a_k[i] = f % (BK / 4) * 4; a_lds[i] = row * L::LDA + a_k[i];
                a_off[i] = c.al.prep(m0 + row, A_PER_LANE ? a_k[i] & 31 : a_k[i], z, a_pos[i]);
            } else {
                const int m = f % (BM / 4) * 4; a_k[i] = f / (BM / 4); a_lds[i] = a_k[i] * L::LDA + m;
                a_off[i] = c.al.prep(m0 + m, z) + (AL::kTab ? 0u : c.al.entry(a_k[i]));
            }
        }
#pragma unroll
        for (int i = 0; i < B_IT; ++i) {
            const int f = tid + i * 256;
            if constexpr (BL::kContig) {
                const int row = f / (BK / 4); b_k[i] = f % (BK / 4) * 4; b_lds[i] = L::A_BUF + row * L::LDB + b_k[i];
                b_off[i] = c.bl.prep(n0 + row, B_PER_LANE ? b_k[i] & 31 : b_k[i], z, b_pos[i]);
            } else {
                const int n = f % (BN / 4) * 4; b_k[i] = f / (BN / 4); b_lds[i] = L::A_BUF + b_k[i] * L::LDB + n;
                b_off[i] = c.bl.prep(n0 + n, z) + c.bl.entry(b_k[i]);
            }
        }
        int* const ktab = reinterpret_cast<int*>(smem + 2 * L::BUF);
        auto fill_tab = [&](int kt, int slot) __attribute__((always_inline)) {      // tiles past the end: past the tensor or unused
            if constexpr (AL::kTab) { if (tid < BK) ktab[slot * BK + tid] = (int)c.al.entry(min(k_begin + kt * BK, k_end) + tid); }
        };
        f32x4 areg[S][A_IT], breg[S][B_IT];
        // the scheduling barriers keep the order of the stages' loads: a wait for one stage must not cover the next one's
        auto gload = [&](int kt, int slot, auto stage) __attribute__((always_inline)) {
            constexpr int G = decltype(stage)::value;
            const int kb = k_begin + min(kt, nk - 1) * BK;       // tiles past the end: the last one again, never stored
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < A_IT; ++i) {
                if constexpr (AL::kContig) {
                    const typename AL::Uni u = c.al.uni(A_PER_LANE ? kb + (a_k[i] & ~31) : kb);
                    if constexpr (A_PER_LANE) areg[G][i] = fetch(a_res, c.al.off(a_off[i], a_pos[i], u) + c.al.soff(u), 0);
                    else areg[G][i] = fetch(a_res, c.al.off(a_off[i], a_pos[i], u), c.al.soff(u));
                } else if constexpr (AL::kTab) areg[G][i] = fetch(a_res, a_off[i] + (unsigned)ktab[slot * BK + a_k[i]], 0);
                else areg[G][i] = fetch(a_res, a_off[i] + c.al.entry(kb), 0);
            }
#pragma unroll
            for (int i = 0; i < B_IT; ++i) {
                if constexpr (BL::kContig) {
                    const typename BL::Uni u = c.bl.uni(B_PER_LANE ? kb + (b_k[i] & ~31) : kb);
                    if constexpr (B_PER_LANE) breg[G][i] = fetch(b_res, c.bl.off(b_off[i], b_pos[i], u) + c.bl.soff(u), 0);
                    else breg[G][i] = fetch(b_res, c.bl.off(b_off[i], b_pos[i], u), c.bl.soff(u));
                } else breg[G][i] = fetch(b_res, b_off[i] + c.bl.entry(kb), 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (AL::kTab) {
#pragma unroll
            for (int g = 0; g <= S; ++g) fill_tab(g, g);
            __syncthreads();                           // the multiplying waves take part
        }
        gload(0, 0, std::integral_constant<int, 0>());
        gload(1, 1, std::integral_constant<int, 1>());
        float csum = 0.f;                              // EP::kColSum: sum of column tid of B, k ascending
        int slot = S;                                  // table slot of tile kt + S
        auto step = [&](int kt, auto stage) __attribute__((always_inline)) {
            constexpr int G = decltype(stage)::value;
            float* const buf = smem + (kt & 1) * L::BUF;
#pragma unroll
            for (int i = 0; i < A_IT; ++i) *reinterpret_cast<f32x4*>(buf + a_lds[i]) = areg[G][i];
#pragma unroll
            for (int i = 0; i < B_IT; ++i) *reinterpret_cast<f32x4*>(buf + b_lds[i]) = breg[G][i];
            gload(kt + S, slot, stage);
            slot = slot + 1 == L::TAB_SLOTS ? 0 : slot + 1;
            fill_tab(kt + S + 1, slot);                // read by the next step, behind this step's barrier
            __syncthreads();                           // tile kt is in LDS; tile kt - 1 has been read
            if constexpr (EP::kColSum) {               // the first waves add, k ascending
                static_assert(!BL::kContig && BN <= 256 && (BN % 64 == 0 || BN == 32), "one thread per column");
                if (m0 == 0 && (wave - 4) * 64 < BN) {
                    const float* const bs = buf + L::A_BUF + tid;
                    float v[BK];
#pragma unroll
                    for (int k = 0; k < BK; ++k) v[k] = bs[k * L::LDB];       // 32 columns: the upper half wave reads the pad and the next row, unused
#pragma unroll
                    for (int k = 0; k < BK; ++k) csum += v[k];
                }
            }
        };
        // whole rounds of S steps without an exit inside (a path on which a stage is not loaded again would make the
        // loop's waits drain the other stage), the remainder behind the loop
        int kt = 0;
        for (int r = nk / S; r > 0; --r, kt += S) {
            step(kt, std::integral_constant<int, 0>());
            step(kt + 1, std::integral_constant<int, 1>());
        }
        if (kt < nk) step(kt, std::integral_constant<int, 0>());
        if constexpr (EP::kColSum) {
            if (m0 == 0 && tid < BN && n0 + tid < c.N) c.ep.store_colsum(n0 + tid, csum, z);
        }
        __syncthreads();                               // the multiplying waves' barrier behind the last tile
        if constexpr (T::WK > 1) __syncthreads();      // and the one between their sums
        return;
    }

    // ======================= waves 0-3: fragments from LDS, MFMA, results =======================
    const int wm = wave % T::WM, wn = wave / T::WM % T::WN, wk = wave / (T::WM * T::WN);
    const int fidx = lane & 31, half = lane >> 5;
    constexpr int NG = T::NG, KACC = T::KACC;
    const int k_lane = wk * NG * 8 + 4 * half;
    const int a_rd = AL::kContig ? (wm * TM * 32 + fidx) * L::LDA + k_lane : k_lane * L::LDA + wm * TM * 32 + fidx;
    const int b_rd = L::A_BUF + (BL::kContig ? (wn * TN * 32 + fidx) * L::LDB + k_lane : k_lane * L::LDB + wn * TN * 32 + fidx);
    f32x4 a[2][TM], b[2][TN];
    auto read_group = [&](int buf, auto GRP) __attribute__((always_inline)) {      // the four MFMA steps of group GRP -> register slot GRP % 2
        constexpr int g = decltype(GRP)::value, sl = g & 1;
        const float* const base = smem + buf * L::BUF;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if constexpr (AL::kContig) a[sl][i] = *reinterpret_cast<const f32x4*>(base + a_rd + i * 32 * L::LDA + g * 8);
            else
#pragma unroll
                for (int j = 0; j < 4; ++j) a[sl][i][j] = base[a_rd + (g * 8 + j) * L::LDA + i * 32];
        }
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            if constexpr (BL::kContig) b[sl][i] = *reinterpret_cast<const f32x4*>(base + b_rd + i * 32 * L::LDB + g * 8);
            else
#pragma unroll
                for (int j = 0; j < 4; ++j) b[sl][i][j] = base[b_rd + (g * 8 + j) * L::LDB + i * 32];
        }
    };
    f32x16 acc[KACC][TM][TN];
    auto mul_group = [&](auto GRP) __attribute__((always_inline)) {
        constexpr int sl = decltype(GRP)::value & 1;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < TN; ++q)
                    acc[j % KACC][i][q] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[sl][q][j], a[sl][i][j], acc[j % KACC][i][q], 0, 0, 0);
    };
    // Byte offset of accumulator registers 4 g .. 4 g + 3 of fragment (i, j): C[row fidx][column 8 g + 4 half + e].  A
    // group of eight columns is wave-uniform, its part is computed on the scalar unit; past the edges: clamped.
    auto out_at = [&](int i, int j, int g) __attribute__((always_inline)) {
        const int row = m0 + wm * (TM * 32) + i * 32 + fidx, col = n0 + wn * (TN * 32) + j * 32 + g * 8;
        return (c.ep.row_off(min(row, c.M - 1), z) + half * 4 + c.ep.col_off(min(col, c.N - 8))) * 4u;
    };
#pragma unroll
    for (int q = 0; q < KACC; ++q)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[q][i][j][r] = 0.f;
    // the ReLU mask of the tile is requested now and used behind the k loop
    f32x4 mask[EP::kMask ? TM : 1][TN][4];
    if constexpr (EP::kMask) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) mask[i][j][g] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(c.ep.mask()) + out_at(i, j, g));
    }
    constexpr std::integral_constant<int, 0> G0;
    if constexpr (AL::kTab) __syncthreads();
    __syncthreads();                                   // tile 0 is in LDS
    read_group(0, G0);
    for (int kt = 0; kt < nk; ++kt) {
        [&]<int... GR>(std::integer_sequence<int, GR...>) __attribute__((always_inline)) {
            ([&] {
                constexpr int g = GR;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (g + 1 < NG) read_group(kt & 1, std::integral_constant<int, g + 1>());
                else {
                    __syncthreads();                   // this tile is in registers; the next one is in LDS
                    read_group((kt + 1) & 1, G0);      // behind the last tile: old data that nobody uses
                }
                __builtin_amdgcn_sched_barrier(0);
                mul_group(std::integral_constant<int, g>());
            }(), ...);
        }(std::make_integer_sequence<int, NG>());
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (KACC == 2) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[0][i][j] += acc[1][i][j];
    }
    if constexpr (T::WK > 1) {                         // every k tile has been read: the sums go through the tile buffers
        constexpr int F = TM * TN * 4;                 // groups of four registers
        const int wmn = wave % (T::WM * T::WN);
        float* const red = smem + lane * 4;
        if (wk > 0) {
#pragma unroll
            for (int f = 0; f < F; ++f) {
                const f32x16& v = acc[0][f / 4 / TN][f / 4 % TN];
                *reinterpret_cast<f32x4*>(red + (((wk - 1) * (T::WM * T::WN) + wmn) * F + f) * 256) = f32x4{v[f % 4 * 4], v[f % 4 * 4 + 1], v[f % 4 * 4 + 2], v[f % 4 * 4 + 3]};
            }
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int q = 0; q < T::WK - 1; ++q)
#pragma unroll
            for (int f = 0; f < F; ++f) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(red + ((q * (T::WM * T::WN) + wmn) * F + f) * 256);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[0][f / 4 / TN][f / 4 % TN][f % 4 * 4 + e] += v[e];
            }
    }
    auto store_tile = [&](auto FULL) __attribute__((always_inline)) {
        constexpr bool full = decltype(FULL)::value;   // no row or column past the edges: no test per store
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const bool rok = full || m0 + wm * (TM * 32) + i * 32 + fidx < c.M;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = acc[0][i][j][4 * g + e];
                        if constexpr (EP::kMask) v[e] = mask[i][j][g][e] > 0.f ? v[e] : 0.f;
                    }
                    if (full || (rok && n0 + wn * (TN * 32) + j * 32 + g * 8 < c.N))
                        *reinterpret_cast<f32x4*>(reinterpret_cast<char*>(c.ep.dst()) + out_at(i, j, g)) = v;
                }
        }
    };
    if (m0 + BM <= c.M && n0 + BN <= c.N) store_tile(std::integral_constant<bool, true>());
    else store_tile(std::integral_constant<bool, false>());
}

template <class C>
__global__ __launch_bounds__(512, 2 * kWsPerCu) void gemm_ws_kernel(const C c) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    gemm_ws_run(c, xcd_order(blockIdx.x, gridDim.x), lds_f);
}

// Two independent GEMMs in one grid: the first n1 workgroups run the items of `a`, the rest those of `b`.
template <class C1, class C2>
__global__ __launch_bounds__(512, 2 * kWsPerCu) void gemm_ws_pair_kernel(const C1 a, const C2 b, int n1) {
    extern __shared__ __attribute__((aligned(16))) float lds_f[];
    if ((int)blockIdx.x < n1) gemm_ws_run(a, xcd_order(blockIdx.x, n1), lds_f);
    else gemm_ws_run(b, xcd_order(blockIdx.x - n1, gridDim.x - n1), lds_f);
}

// more LDS than a kernel gets by default
template <class K> inline hipError_t allow_lds(K kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <class C>
inline hipError_t launch_gemm_ws(hipStream_t s, const C& c) {
    if (!c.valid()) return hipErrorInvalidValue;
    constexpr int LDS = WsSmem<C>::BYTES;
    static const hipError_t ready = allow_lds(gemm_ws_kernel<C>, LDS);
    if (ready != hipSuccess) return ready;
    launch_k_lds((gemm_ws_kernel<C>), dim3(c.items()), dim3(512), LDS, s, c);
    return hipGetLastError();
}

template <class C1, class C2>
inline hipError_t launch_gemm_ws_first(hipStream_t s, const C1& a, const C2& b) {
    constexpr int LDS = WsSmem<C1>::BYTES > WsSmem<C2>::BYTES ? WsSmem<C1>::BYTES : WsSmem<C2>::BYTES;
    static const hipError_t ready = allow_lds(gemm_ws_pair_kernel<C1, C2>, LDS);
    if (ready != hipSuccess) return ready;
    launch_k_lds((gemm_ws_pair_kernel<C1, C2>), dim3(a.items() + b.items()), dim3(512), LDS, s, a, b, a.items());
    return hipGetLastError();
}
// The one whose items take longer is started first: the shorter ones fill the places that become free (1280 samples:
// fully connected layer 101 -> 77 us, second layer 211 -> 164).
template <class C1, class C2>
inline hipError_t launch_gemm_ws_pair(hipStream_t s, const C1& a, const C2& b) {
    if (!a.valid() || !b.valid()) return hipErrorInvalidValue;
    return a.item_mfmas() >= b.item_mfmas() ? launch_gemm_ws_first(s, a, b) : launch_gemm_ws_first(s, b, a);
}

}  // namespace paac
