// Forward pass of the dense layers of the fp32 path on the fp32 matrix cores, for the batches that are too small
// for the exact-operand kernels: convolution and the hidden fully connected layer, for the two networks of the paper's
// Experiments section (arch_nips: 16@8x8/4, 32@4x4/2, fc 256; arch_nature: 32@8x8/4, 64@4x4/2,
// 64@3x3/1, fc 512; input 4x84x84, no padding).
#include "gemm_core.hip.h"
#include "gemm_reg16.hip.h"
#include "internal.h"

namespace paac {

typedef ConvGeom<16, 20, 20, 4, 2, 32> NipsC2;
typedef ConvGeom<32, 20, 20, 4, 2, 64> NatC2;
typedef ConvGeom<64, 9, 9, 3, 1, 64> NatC3;

// tile shapes: BM, BN, BK, waves along m / n / k, MFMA edge, register prefetch stages
typedef Tile<128, 32, 32, 4, 1, 1, 32, 3> T128x32;
typedef Tile<32, 32, 64, 1, 1, 4, 32, 4> T32x32;
typedef Tile<64, 64, 32, 2, 2, 1, 32, 3> T64x64;
typedef Tile<32, 64, 64, 1, 2, 2, 32, 4> T32x64;
// eight wavefronts: the k-steps of a tile are split four ways, so a wave's chain of 64-cycle fp32
// MFMAs is half as long as in the four-wave tile of the same shape, without doubling the number of
// workgroups the dispatcher has to start (the batch-of-32 launches are bound by exactly these two).
// Measured at n_e = 32: first layer 10.3 -> 9.2 us; a 32x64 eight-wave tile for the 64-wide layers
// (half the workgroups of the 32x32 tile) was slower, 8.2 -> 9.7 us, and is not used.
typedef Tile<64, 32, 64, 2, 1, 4, 32, 4> T64x32w8;
// big / middle / small tile per output width
template <int N> struct TileForN;
template <> struct TileForN<32> { typedef T128x32 big; typedef T64x32w8 mid; typedef T32x32 small; };
template <> struct TileForN<64> { typedef T64x64 big; typedef T32x64 mid; typedef T32x32 small; };

// Workgroups are dispatched at a finite rate (on the order of 100 per microsecond), so a launch of
// thousands of small workgroups is bound by dispatch: take the largest tile that still gives about
// one workgroup per compute unit (256 of them).
static const int kMinWgs = 192;
template <class TBig, class TMid, class TSmall, class AL, class BL, class EP>
static hipError_t launch_auto(hipStream_t s, const AL& al, const BL& bl, const EP& ep, int M, int N, int K, int z) {
    auto wgs = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn) * z; };
    if (wgs(TBig::BM, TBig::BN) >= kMinWgs) return launch_gemm<TBig>(s, al, bl, ep, M, N, K, z, 0);
    if (wgs(TMid::BM, TMid::BN) >= kMinWgs) return launch_gemm<TMid>(s, al, bl, ep, M, N, K, z, 0);
    if (wgs(TSmall::BM, TSmall::BN) < kMinWgs) {
        return launch_gemm_reg16(s, al, bl, ep, M, N, K, z, 0);
    }
    return launch_gemm<TSmall>(s, al, bl, ep, M, N, K, z, 0);
}

NetDesc make_net(int arch, int n_actions) {
    NetDesc n{};
    n.arch = arch;
    n.n_actions = n_actions;
    auto set = [](ConvDesc& c, int cin, int h, int w, int ks, int st, int cout) {
        c.cin = cin; c.h = h; c.w = w; c.ks = ks; c.st = st; c.cout = cout;
        c.ho = (h - ks) / st + 1; c.wo = (w - ks) / st + 1; c.kk = ks * ks * cin;
    };
    if (arch == 0) {
        n.n_conv = 2;
        set(n.conv[0], 4, 84, 84, 8, 4, 16);
        set(n.conv[1], 16, 20, 20, 4, 2, 32);
        n.fc = 256;
    } else {
        n.n_conv = 3;
        set(n.conv[0], 4, 84, 84, 8, 4, 32);
        set(n.conv[1], 32, 20, 20, 4, 2, 64);
        set(n.conv[2], 64, 9, 9, 3, 1, 64);
        n.fc = 512;
    }
    const ConvDesc& l = n.conv[n.n_conv - 1];
    n.flat = l.ho * l.wo * l.cout;
    return n;
}

Split plan_split(int k_total, int tiles, int granule, int target_wgs) {
    int n = target_wgs / (tiles > 0 ? tiles : 1);
    if (n < 1) n = 1;
    int k_per = (k_total + n - 1) / n;
    k_per = (k_per + granule - 1) / granule * granule;
    if (k_per < granule) k_per = granule;
    Split s;
    s.k_per = k_per;
    s.n = (k_total + k_per - 1) / k_per;
    if (s.n < 1) s.n = 1;
    return s;
}

// ---------------------------------------------------------------------------------- forward
template <class G>
static hipError_t conv_fwd_f32(hipStream_t s, const void* in, const float* W, const float* b, float* out, int ns) {
    typedef TileForN<G::COUT> TS;
    const int M = ns * G::HO * G::WO;
    ConvNHWCRowsK<G> al{(const float*)in, M};
    DenseKCols bl{W, G::COUT, G::COUT};
    EpiBiasRelu ep{out, b, G::COUT};
    // third layer, up to 64 samples: the register-only kernel on 16x32 tiles (49 rows per sample, 392 tiles of 16x16 at
    // n_e = 32: 6.0 -> 5.55 us per select call against 16x16; on 16x64 8.1 us)
    if (ns <= 64 && G::ST == 1) return launch_gemm_reg16<2>(s, al, bl, ep, M, G::COUT, G::KK, 1, 0);
    return launch_auto<typename TS::big, typename TS::mid, typename TS::small>(s, al, bl, ep, M, G::COUT, G::KK, 1);
}

// layers 1.. of the fp32 path (the first layer runs in conv1_fwd_exact, up to kConv12MaxSamples samples the first two in conv12_fwd)
hipError_t conv_fwd(hipStream_t s, int arch, int layer, const void* in, const float* W, const float* b,
                    float* out, int ns) {
    if (arch == 0) {
        if (layer == 1) return conv_fwd_f32<NipsC2>(s, in, W, b, out, ns);
    } else {
        if (layer == 1) return conv_fwd_f32<NatC2>(s, in, W, b, out, ns);
        if (layer == 2) return conv_fwd_f32<NatC3>(s, in, W, b, out, ns);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------------- fully connected
static void fc_dims(int arch, int& flat, int& fc) {
    if (arch == 0) { flat = 2592; fc = 256; } else { flat = 3136; fc = 512; }
}
// up to 48 rows: 16x16 tiles and about 512 workgroups (fewer, longer k-splits than with wider tiles:
// fewer partial sums for the heads kernel to add; arch_nips select: fc 4.5 -> 4.2 us, heads 5.4 -> 4.6 us)
static bool fc_small(int ns) { return ns <= 48; }
// 49 to 64 rows: 32x32 tiles, four times the tiles of the 64x64 ones and so a quarter of the k-splits, each
// of which is a partial sum for the heads kernel to add (n_e = 64: heads 5.8 -> 4.65 us per select call, the
// GEMM unchanged, step +1.5 %)
static bool fc_mid(int ns) { return ns <= 64; }
Split fc_fwd_plan(int arch, int ns) {
    int flat, fc; fc_dims(arch, flat, fc);
    if (fc_small(ns)) return plan_split(flat, ((ns + 15) / 16) * (fc / 16), 32, 512);
    if (fc_mid(ns)) return plan_split(flat, ((ns + 31) / 32) * (fc / 32), 32, 256);
    return plan_split(flat, ((ns + 63) / 64) * (fc / 64), 32, 256);
}

hipError_t fc_fwd(hipStream_t s, int arch, const float* x, const float* W, float* partial, int ns, Split sp) {
    int flat, fc; fc_dims(arch, flat, fc);
    DenseRowsK al{x, ns, flat};
    DenseKCols bl{W, fc, fc};
    EpiPartial<false> ep{partial, (size_t)ns * fc, fc, nullptr, 0};
    if (fc_small(ns)) return launch_gemm_reg16(s, al, bl, ep, ns, fc, flat, sp.n, sp.k_per);
    if (fc_mid(ns)) return launch_gemm<T32x32>(s, al, bl, ep, ns, fc, flat, sp.n, sp.k_per);
    return fc_fwd_ws(s, arch, x, W, partial, ns, sp);
}

}  // namespace paac
