// Backward pass of layers 2.. and of the fully connected layer of the fp32 path, and its fully connected forward pass
// from 65 rows on, on the wave-specialised fp32 GEMM (gemm_ws.hip.h): tiles by size.
#include "gemm_ws.hip.h"
#include "internal.h"

namespace paac {

typedef ConvGeom<16, 20, 20, 4, 2, 32> NipsC2;
typedef ConvGeom<32, 20, 20, 4, 2, 64> NatC2;
typedef ConvGeom<64, 9, 9, 3, 1, 64> NatC3;

typedef TileW<64, 128, 32, 2, 2, 1, 1> W64x128;
typedef TileW<64, 64, 32, 2, 2, 1, 2> W64x64;
// a quarter and a half of the 64 x 64 tile, for launches that would leave compute units idle: 64-deep k tiles whose k
// the waves divide, so that a workgroup's chain of MFMAs shrinks with its tile
typedef TileW<32, 64, 64, 1, 2, 2, 2> W32x64;
typedef TileW<64, 32, 64, 2, 1, 2, 2> W64x32;
typedef TileW<32, 32, 64, 1, 1, 4, 2> W32x32;

// about one workgroup per compute unit: the largest tile that still gives so many
constexpr int kMinWgs = 192;

// The data gradient and the weight gradient of a layer both start from dY and are independent of each other (the chain
// conv3 -> conv2 of data gradients is the critical path of the backward pass, the weight gradients ride along).
template <class TD, class TW, class G>
static hipError_t conv_bwd_tiles(hipStream_t s, const float* act_in, const float* dy, const float* W, float* dx, float* pw, float* pb, int ns, Split sp) {
    const int M = ns * G::HC * G::WC, R = ns * G::HO * G::WO;
    const auto d = gemm_ws<TD>(WsDgradRows<G>{dy, ns}, WsDgradWeights<G>{W}, WsDgradMask<G>{dx, act_in}, M, G::ST * G::ST * G::CIN, G::KD, 1, 0);
    const auto w = gemm_ws<TW>(WsConvCols<G>{act_in, ns}, WsDenseCols{dy, R, G::COUT, G::COUT},
                               WsPartial<true>{pw, (unsigned)(G::KK * G::COUT), G::COUT, pb, G::COUT}, G::KK, G::COUT, R, sp.n, sp.k_per);
    return launch_gemm_ws_pair(s, d, w);
}
template <class G>
static hipError_t conv_bwd_t(hipStream_t s, const float* act_in, const float* dy, const float* W, float* dx, float* pw, float* pb, int ns, Split sp) {
    typedef std::conditional_t<G::COUT == 64, W64x64, W64x32> TW;
    // 64 x 128: all parity classes of a 64-row block of positions gather the same dY rows once
    constexpr int NA = G::ST * G::ST * G::CIN;
    const int M = ns * G::HC * G::WC;
    auto wgs = [&](int bm, int z) { return (M + bm - 1) / bm * z; };
    if constexpr (NA == 128) { if (wgs(64, 1) >= kMinWgs) return conv_bwd_tiles<W64x128, TW, G>(s, act_in, dy, W, dx, pw, pb, ns, sp); }
    if (NA == 64 ? wgs(64, 1) >= kMinWgs : wgs(32, 1) >= kMinWgs) return conv_bwd_tiles<W64x64, TW, G>(s, act_in, dy, W, dx, pw, pb, ns, sp);
    if constexpr (G::ST == 1) {
        if (wgs(32, 1) >= kMinWgs) return conv_bwd_tiles<W32x64, TW, G>(s, act_in, dy, W, dx, pw, pb, ns, sp);
    } else {
        if (NA == 64 && wgs(32, 1) >= kMinWgs) return conv_bwd_tiles<W32x64, TW, G>(s, act_in, dy, W, dx, pw, pb, ns, sp);
        if (wgs(128, 4) >= kMinWgs) return conv_bwd_tiles<W64x64, TW, G>(s, act_in, dy, W, dx, pw, pb, ns, sp);
        if (wgs(64, 4) >= kMinWgs) return conv_bwd_tiles<W32x64, TW, G>(s, act_in, dy, W, dx, pw, pb, ns, sp);
    }
    return conv_bwd_tiles<W32x32, TW, G>(s, act_in, dy, W, dx, pw, pb, ns, sp);
}
hipError_t conv_bwd(hipStream_t s, int arch, int layer, const float* act_in, const float* dy, const float* W, float* dx,
                    float* pw, float* pb, int ns, Split sp) {
    if (arch == 0 && layer == 1) return conv_bwd_t<NipsC2>(s, act_in, dy, W, dx, pw, pb, ns, sp);
    if (arch == 1 && layer == 1) return conv_bwd_t<NatC2>(s, act_in, dy, W, dx, pw, pb, ns, sp);
    if (arch == 1 && layer == 2) return conv_bwd_t<NatC3>(s, act_in, dy, W, dx, pw, pb, ns, sp);
    return hipErrorInvalidValue;
}
template <class G, class T> static int tiles_of() { return ((G::KK + T::BM - 1) / T::BM) * ((G::COUT + T::BN - 1) / T::BN); }
int conv_wgrad_tiles(int arch, int layer) {
    if (arch == 0) return tiles_of<NipsC2, W64x32>();
    return layer == 1 ? tiles_of<NatC2, W64x64>() : tiles_of<NatC3, W64x64>();
}

// ---------------------------------------------------------------------------------- fully connected
static void fc_dims(int arch, int& flat, int& fc) {
    if (arch == 0) { flat = 2592; fc = 256; } else { flat = 3136; fc = 512; }
}
template <class TD, class TW>
static hipError_t fc_bwd_tiles(hipStream_t s, int arch, const float* x, const float* dh, const float* W, float* dx, float* pw, float* pb, int ns) {
    int flat, fc; fc_dims(arch, flat, fc);
    const auto d = gemm_ws<TD>(WsDenseRows{dh, ns, fc}, WsDenseRows{W, flat, fc}, WsDenseMask{dx, x, flat}, ns, flat, fc, 1, 0);
    // not split: its reduction dimension is the batch, and its output alone has enough tiles
    const auto w = gemm_ws<TW>(WsDenseCols{x, ns, flat, flat}, WsDenseCols{dh, ns, fc, fc}, WsPartial<true>{pw, (unsigned)(flat * fc), fc, pb, fc}, flat, fc, ns, 1, 0);
    return launch_gemm_ws_pair(s, d, w);
}
hipError_t fc_bwd(hipStream_t s, int arch, const float* x, const float* dh, const float* W, float* dx, float* pw, float* pb, int ns) {
    int flat, fc; fc_dims(arch, flat, fc);
    const bool wide = arch == 1 && ns >= 128 && ns <= 384;      // half as many workgroups where a tile's reduction is a handful of k tiles
    if ((ns + 63) / 64 * (flat / 64) >= kMinWgs) {
        if (wide) return fc_bwd_tiles<W64x64, W64x128>(s, arch, x, dh, W, dx, pw, pb, ns);
        return fc_bwd_tiles<W64x64, W64x64>(s, arch, x, dh, W, dx, pw, pb, ns);
    }
    if (wide) return fc_bwd_tiles<W32x64, W64x128>(s, arch, x, dh, W, dx, pw, pb, ns);
    return fc_bwd_tiles<W32x64, W64x64>(s, arch, x, dh, W, dx, pw, pb, ns);
}

// forward from 65 rows on: partial[split][ns][fc] = x . W
hipError_t fc_fwd_ws(hipStream_t s, int arch, const float* x, const float* W, float* partial, int ns, Split sp) {
    int flat, fc; fc_dims(arch, flat, fc);
    return launch_gemm_ws(s, gemm_ws<W64x64>(WsDenseRows{x, ns, flat}, WsDenseCols{W, flat, fc, fc}, WsPartial<false>{partial, (unsigned)(ns * fc), fc, nullptr, 0},
                                             ns, fc, flat, sp.n, sp.k_per));
}

}  // namespace paac
