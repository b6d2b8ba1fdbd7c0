// Binary convolution layers without a materialised im2col matrix, and max pooling on bits.
//
// bnn_conv_xnor / bnn_conv_bn_sign_pack: a kh x kw binary convolution (3 x 3 in the paper's
// nets, Sec. 3.3) as the XnorDotProduct of Alg. 4 over receptive fields that the GEMM's tile
// loader gathers straight from the packed NHWC input (taps outside the image are +1: zero
// padding through Eq. (1)).  The kernels: fused layers, 3 x 3 ones first of all, in equal strips of pixels, filters resident
// (conv_strip.hip); the LDS-patch kernel (conv_patch.hip) wherever the
// input patch of a tile fits; else the conv modes of the matrix-engine
// GEMMs (xnor_gemm_mfma.hip, xnor_gemm_mfma_shortk.hip); launch_conv_mfma chooses.
//
// bnn_conv_pool_bn_sign_pack: the same layer with the paper's 2 x 2 max pooling between the
// convolution and BatchNorm + Sign, in one launch (strips and the LDS-patch kernel), on tiles of whole image rows.
// bnn_conv_pool_windows_bn_sign_pack: on any even map whose patch fits.  bnn_conv_pool_form: which of the two, or
// neither, is the fastest form of a layer.
//
// bnn_maxpool_bits: the paper's ConvNets pool the integer pre-activations before BatchNorm and
// Sign.  Sign(BatchNorm(.)) is monotone per channel - non-decreasing where the folded flip bit
// is 0, non-increasing where it is 1 - so Sign(BN(max over the window)) is the OR of the
// window's output bits where flip = 0 and their AND where flip = 1: pooling can run after the
// fused layer, on packed bits, 32 channels per operation.
#include "bnn_internal.h"
#include "gemm_staging.h"

namespace bnn {

bool mfma_path_supports(int64_t K);
int launch_conv_mfma(const uint32_t* in, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc, int64_t M,
                     int64_t N, int64_t K, ConvArgs cv, void* stream);
int launch_conv_mfma_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                           BnSignArgs bn, ConvArgs cv, void* stream);
int launch_conv_patch_pool_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                                 BnSignArgs bn, ConvArgs cv, bool any_map, ConvUse use, void* stream);
// Vector-ALU form for receptive fields beyond the matrix engine's exact range (valu_fallbacks.hip).
int launch_conv_xnor_valu(const uint32_t* in, const uint32_t* Wb, int64_t ldw, int32_t* S, int64_t lds, int64_t M,
                          int64_t N, int64_t K, ConvArgs cv, bool fused, BnSignArgs bn, void* stream);

// Validates a convolution and fills the geometry.  M = B*Ho*Wo, K = kh*kw*Cin.
static int conv_geometry(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t Cin, const uint32_t* Wb,
                         int64_t ldw, int64_t Cout, int kh, int kw, int stride, int pad, ConvArgs& cv,
                         int64_t& M, int64_t& K) {
    if (B < 0 || H < 1 || W < 1 || Cin < 1 || Cout < 0 || kh < 1 || kw < 1 || stride < 1 || pad < 0)
        return BNN_ERR_INVALID_ARG;
    if (B > kMaxDim || H > 32767 || W > 32767 || Cin > kMaxDim || Cout > kMaxDim) return BNN_ERR_INVALID_ARG;
    if (H + 2 * int64_t(pad) < kh || W + 2 * int64_t(pad) < kw) return BNN_ERR_INVALID_ARG;
    const int64_t Ho = (H + 2 * int64_t(pad) - kh) / stride + 1;
    const int64_t Wo = (W + 2 * int64_t(pad) - kw) / stride + 1;
    // The tile loaders carry an output pixel as (oy << 16) | ox and form input coordinates in 32 bits.
    if (pad > 32767 || Ho > 32767 || Wo > 32767) return BNN_ERR_UNSUPPORTED;
    K = int64_t(kh) * kw * Cin;
    M = B * Ho * Wo;
    if (K > kMaxK || M > kMaxDim - 1024) return BNN_ERR_INVALID_ARG;      // row indices run up to one tile past M
    if (ldw < ceil_div(K, 32)) return BNN_ERR_INVALID_ARG;
    if (B > 0 && Cout > 0 && (!in || !Wb)) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(in, 4) || !aligned_to(Wb, 4)) return BNN_ERR_ALIGNMENT;
    // Whole channel words only.  With Cin % 128 == 0 the tile loaders move 16-byte groups of 4 channel
    // words; other multiples of 32 are taken word by word, by the LDS-patch kernel alone (same-size
    // stride-1 layers; launch_conv_mfma refuses the rest).  The input is addressed with 32-bit word offsets.
    if (Cin % 32 != 0) return BNN_ERR_UNSUPPORTED;
    if (Cin % 128 == 0 && !aligned_to(in, 16)) return BNN_ERR_UNSUPPORTED;
    if (B * H * W * (Cin / 32) > (int64_t(1) << 32) - 1) return BNN_ERR_UNSUPPORTED;
    cv.H = int(H); cv.W = int(W); cv.Cw = int(Cin / 32);
    cv.kh = kh; cv.kw = kw; cv.stride = stride; cv.pad = pad;
    cv.Ho = int(Ho); cv.Wo = int(Wo);
    return BNN_OK;
}

// One thread per VW words of an output pixel (4-byte aligned); TWO: 2 x 2 windows, whose four loads are in flight together.
// 128 images of 28 x 28 x 256, 2 x 2: 3.3 us with one word per thread, its window in a loop and its place from three 64-bit
// divisions, 2.4 this way (an empty launch takes about 2).
template <int VW, bool TWO>
__global__ __launch_bounds__(256) void maxpool_units_kernel(const uint32_t* __restrict__ in, int H, int W, int Cw, int ph,
                                                            int pw, int stride, int Hp, int Wp, FastDiv by_units,
                                                            FastDiv by_wp, FastDiv by_hp,
                                                            const uint32_t* __restrict__ flip_bits,
                                                            uint32_t* __restrict__ out, int n_units) {
    typedef uint32_t unit_t __attribute__((ext_vector_type(VW), aligned(4)));
    const int64_t at = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (at >= n_units) return;
    const int u = int(at), units = Cw / VW;
    const int pix = by_units(u), cu = (u - pix * units) * VW;
    const int row = by_wp(pix), px = pix - row * Wp;
    const int b = by_hp(row), py = row - b * Hp;
    const uint32_t* p = in + ((int64_t(b) * H + int64_t(py) * stride) * W + int64_t(px) * stride) * Cw + cu;
    const int64_t down = int64_t(W) * Cw;
    unit_t any, all;
    if (TWO) {
        const unit_t v00 = *reinterpret_cast<const unit_t*>(p), v01 = *reinterpret_cast<const unit_t*>(p + Cw);
        const unit_t v10 = *reinterpret_cast<const unit_t*>(p + down), v11 = *reinterpret_cast<const unit_t*>(p + down + Cw);
        any = v00 | v01 | v10 | v11;
        all = v00 & v01 & v10 & v11;
    } else {
        any = all = *reinterpret_cast<const unit_t*>(p);
        for (int dy = 0; dy < ph; ++dy)
            for (int dx = 0; dx < pw; ++dx) {
                const unit_t v = *reinterpret_cast<const unit_t*>(p + dy * down + int64_t(dx) * Cw);
                any |= v;
                all &= v;
            }
    }
    unit_t flip;
#pragma unroll
    for (int e = 0; e < VW; ++e) flip[e] = flip_bits ? flip_bits[cu + e] : 0u;
    *reinterpret_cast<unit_t*>(out + int64_t(u) * VW) = (any & ~flip) | (all & flip);
}

// The same for outputs of 2^31 words and more.
__global__ __launch_bounds__(256) void maxpool_bits_kernel(const uint32_t* __restrict__ in, int H, int W,
                                                           int Cw, int ph, int pw, int stride, int Hp, int Wp,
                                                           const uint32_t* __restrict__ flip_bits,
                                                           uint32_t* __restrict__ out, int64_t n_words) {
    for (int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; u < n_words;
         u += int64_t(gridDim.x) * blockDim.x) {
        const int cw = int(u % Cw);
        int64_t t = u / Cw;
        const int px = int(t % Wp);
        t /= Wp;
        const int py = int(t % Hp);
        const int64_t b = t / Hp;
        uint32_t any = 0u, all = ~0u;
        for (int dy = 0; dy < ph; ++dy)
            for (int dx = 0; dx < pw; ++dx) {
                const uint32_t v = in[((b * H + py * stride + dy) * W + px * stride + dx) * Cw + cw];
                any |= v;
                all &= v;
            }
        const uint32_t flip = flip_bits ? flip_bits[cw] : 0u;
        out[u] = (any & ~flip) | (all & flip);
    }
}

}  // namespace bnn

extern "C" int bnn_conv_xnor(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t Cin, const uint32_t* Wb,
                             int64_t ldw, int64_t Cout, int kh, int kw, int stride, int pad, int32_t* S,
                             int64_t lds, void* stream) {
    using namespace bnn;
    ConvArgs cv;
    int64_t M, K;
    const int st = conv_geometry(in, B, H, W, Cin, Wb, ldw, Cout, kh, kw, stride, pad, cv, M, K);
    if (st != BNN_OK) return st;
    if (lds < Cout) return BNN_ERR_INVALID_ARG;
    if (M == 0 || Cout == 0) return BNN_OK;
    if (!S) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(S, 4)) return BNN_ERR_ALIGNMENT;
    if (!mfma_path_supports(K)) return launch_conv_xnor_valu(in, Wb, ldw, S, lds, M, Cout, K, cv, false, BnSignArgs{}, stream);
    return launch_conv_mfma(in, Wb, ldw, S, lds, M, Cout, K, cv, stream);
}

extern "C" int bnn_conv_bn_sign_pack(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t Cin,
                                     const uint32_t* Wb, int64_t ldw, int64_t Cout, int kh, int kw, int stride,
                                     int pad, const int32_t* thr, const uint32_t* flip_bits, uint32_t* out,
                                     int64_t ld_out, void* stream) {
    using namespace bnn;
    ConvArgs cv;
    int64_t M, K;
    const int st = conv_geometry(in, B, H, W, Cin, Wb, ldw, Cout, kh, kw, stride, pad, cv, M, K);
    if (st != BNN_OK) return st;
    if (ld_out < ceil_div(Cout, 32)) return BNN_ERR_INVALID_ARG;
    if (M == 0 || Cout == 0) return BNN_OK;
    if (!thr || !flip_bits || !out) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(thr, 4) || !aligned_to(flip_bits, 4) || !aligned_to(out, 4)) return BNN_ERR_ALIGNMENT;
    if (!mfma_path_supports(K))
        return launch_conv_xnor_valu(in, Wb, ldw, nullptr, 0, M, Cout, K, cv, true, BnSignArgs{thr, flip_bits, out, ld_out},
                                     stream);
    return launch_conv_mfma_fused(in, Wb, ldw, M, Cout, K, BnSignArgs{thr, flip_bits, out, ld_out}, cv, stream);
}

static int conv_pool(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t Cin, const uint32_t* Wb, int64_t ldw,
                     int64_t Cout, int kh, int kw, int stride, int pad, int pool, const int32_t* thr,
                     const uint32_t* flip_bits, uint32_t* out, int64_t ld_out, bool any_map, void* stream) {
    using namespace bnn;
    ConvArgs cv;
    int64_t M, K;
    const int st = conv_geometry(in, B, H, W, Cin, Wb, ldw, Cout, kh, kw, stride, pad, cv, M, K);
    if (st != BNN_OK) return st;
    if (pool < 1 || ld_out < ceil_div(Cout, 32)) return BNN_ERR_INVALID_ARG;
    if (pool != 2 || !mfma_path_supports(K)) return BNN_ERR_UNSUPPORTED;
    if (M == 0 || Cout == 0) return BNN_OK;
    if (!thr || !flip_bits || !out) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(thr, 4) || !aligned_to(flip_bits, 4) || !aligned_to(out, 4)) return BNN_ERR_ALIGNMENT;
    return launch_conv_patch_pool_fused(in, Wb, ldw, M, Cout, K, BnSignArgs{thr, flip_bits, out, ld_out}, cv, any_map,
                                        ConvUse::faster, stream);
}

extern "C" int bnn_conv_pool_bn_sign_pack(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t Cin,
                                          const uint32_t* Wb, int64_t ldw, int64_t Cout, int kh, int kw, int stride,
                                          int pad, int pool, const int32_t* thr, const uint32_t* flip_bits,
                                          uint32_t* out, int64_t ld_out, void* stream) {
    return conv_pool(in, B, H, W, Cin, Wb, ldw, Cout, kh, kw, stride, pad, pool, thr, flip_bits, out, ld_out, false, stream);
}

extern "C" int bnn_conv_pool_windows_bn_sign_pack(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t Cin,
                                                  const uint32_t* Wb, int64_t ldw, int64_t Cout, int kh, int kw,
                                                  int stride, int pad, int pool, const int32_t* thr,
                                                  const uint32_t* flip_bits, uint32_t* out, int64_t ld_out, void* stream) {
    return conv_pool(in, B, H, W, Cin, Wb, ldw, Cout, kh, kw, stride, pad, pool, thr, flip_bits, out, ld_out, true, stream);
}

extern "C" int bnn_conv_pool_form(int64_t B, int64_t H, int64_t W, int64_t Cin, int64_t Cout, int kh, int kw, int stride, int pad,
                                  int pool) {
    using namespace bnn;
    // Buffers of any alignment and filters of any length that the calls can ask for: nothing is read.
    const uint32_t* const aligned = reinterpret_cast<const uint32_t*>(uintptr_t(256));
    const int64_t ldw = ceil_div(kMaxK, 128) * 4;
    ConvArgs cv;
    int64_t M, K;
    if (conv_geometry(aligned, B, H, W, Cin, aligned, ldw, Cout, kh, kw, stride, pad, cv, M, K) != BNN_OK) return BNN_POOL_APART;
    if (pool != 2 || !mfma_path_supports(K) || M == 0 || Cout == 0) return BNN_POOL_APART;
    auto takes = [&](bool any_map) {
        return launch_conv_patch_pool_fused(aligned, aligned, ldw, M, Cout, K, BnSignArgs{}, cv, any_map, ConvUse::ask, nullptr) == BNN_OK;
    };
    return takes(false) ? BNN_POOL_IN_CONV : takes(true) ? BNN_POOL_WINDOWS : BNN_POOL_APART;
}

extern "C" int bnn_maxpool_bits(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t C, int ph, int pw,
                                int stride, const uint32_t* flip_bits, uint32_t* out, void* stream) {
    using namespace bnn;
    if (B < 0 || H < 1 || W < 1 || C < 1 || ph < 1 || pw < 1 || stride < 1) return BNN_ERR_INVALID_ARG;
    if (B > kMaxDim || H > kMaxDim || W > kMaxDim || C > kMaxDim || H < ph || W < pw) return BNN_ERR_INVALID_ARG;
    if (B == 0) return BNN_OK;
    if (!in || !out) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(in, 4) || !aligned_to(out, 4) || !aligned_to(flip_bits, 4)) return BNN_ERR_ALIGNMENT;
    const int64_t Hp = (H - ph) / stride + 1, Wp = (W - pw) / stride + 1;
    const int64_t Cw = ceil_div(C, 32);
    const int64_t n_words = B * Hp * Wp * Cw;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (n_words <= kMaxDim) {
        // Four words a thread for 2 x 2 windows, and for others where the loads and not the wait for them count: the windows are
        // walked load by load, longer the wider the loads (64 of 14 x 14 x 512, 7 x 7 6.7 us a word at a time, 7.8 four; 2000 of
        // 6 x 6 x 128, 6 x 6 4.7 and 6.8; 256 of 28 x 28 x 256, 3 x 3 at stride 2 3.6 and 3.5, at stride 1 4.9 and 3.9).
        const bool two = ph == 2 && pw == 2;
        const int vw = Cw % 4 == 0 && (two || n_words >= 1 << 18) ? 4 : 1;
        const int64_t n_units = n_words / vw;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(unsigned(ceil_div(n_units, 256))), dim3(256), 0, s, in, int(H), int(W), int(Cw), ph,
                               pw, stride, int(Hp), int(Wp), fast_div(Cw / vw), fast_div(Wp), fast_div(Hp), flip_bits, out,
                               int(n_units));
        };
        if (vw == 4 && two) launch(maxpool_units_kernel<4, true>);
        else if (vw == 4) launch(maxpool_units_kernel<4, false>);
        else if (two) launch(maxpool_units_kernel<1, true>);
        else launch(maxpool_units_kernel<1, false>);
        return check_launch();
    }
    int64_t blocks = ceil_div(n_words, 256);
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(maxpool_bits_kernel, dim3(unsigned(blocks)), dim3(256), 0, s,
                       in, int(H), int(W), int(Cw), ph, pw, stride, int(Hp), int(Wp), flip_bits, out, n_words);
    return check_launch();
}
