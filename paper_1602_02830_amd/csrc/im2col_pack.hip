// bnn_conv_im2col_pack: lowers a binary kh x kw convolution (3 x 3 in the
// paper's nets, Sec. 3.3) to the XNOR-popcount matrix product.
//
// Row m = (b*Ho + oy)*Wo + ox of the output is the receptive field of output
// pixel (b, oy, ox): K = kh*kw*Cin bits, bit (ky*kw + kx)*Cin + ci.  Taps
// outside the image are +1 (bit 1): zero padding seen through Eq. (1).
//
// HBM-bound on the write side: (kh*kw*Cin)/8 bytes written per output pixel;
// reads mostly hit cache (each input pixel is used kh*kw times).
//   units   - Cin % 32 == 0: copies of 4, 2 or 1 words (Cin a multiple of 128, 64 or 32).  A thread
//             keeps one unit of the receptive field (its tap and channel words, fixed for the
//             kernel's life) and walks over the batch's output pixels by carries, so the copy loop
//             has no division; the threads of a pass write whole consecutive output rows.
//   words   - the same a word at a time, for batches of 2^31 pixels and more.
//   bits    - any Cin: an output word gathers bit runs from up to 32 taps.
#include "bnn_internal.h"
#include "gemm_staging.h"

namespace bnn {

struct ConvGeom {
    int B, H, W, Cin, Cw;        // Cw = words per input pixel
    int kh, kw, stride, pad;
    int Ho, Wo;
    int64_t M;                   // B*Ho*Wo
    int Kbits;                   // kh*kw*Cin
    int Kwords;                  // ceil(Kbits/32)
};

__global__ __launch_bounds__(256) void im2col_words_kernel(const uint32_t* __restrict__ in, ConvGeom g,
                                                           uint32_t* __restrict__ out, int64_t ld_out,
                                                           int64_t n_units) {
    const int words_per_row = g.kh * g.kw * g.Cw;
    for (int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; u < n_units;
         u += int64_t(gridDim.x) * blockDim.x) {
        const int64_t m = u / words_per_row;
        const int r = int(u - m * words_per_row);
        const int tap = r / g.Cw;
        const int cu = r - tap * g.Cw;
        const int ky = tap / g.kw, kx = tap - ky * g.kw;
        const int ox = int(m % g.Wo);
        const int64_t t = m / g.Wo;
        const int oy = int(t % g.Ho);
        const int64_t b = t / g.Ho;
        const int y = oy * g.stride + ky - g.pad;
        const int x = ox * g.stride + kx - g.pad;
        const bool inside = y >= 0 && y < g.H && x >= 0 && x < g.W;
        out[m * ld_out + r] = inside ? in[((b * g.H + y) * g.W + x) * g.Cw + cu] : ~0u;
    }
}

// Units of VW words, 4-byte aligned (one load and one store each).  A pass is P pixels, per_pass threads each.
struct UnitCopy {
    FastDiv by_pass, by_chunks, by_tap, by_kw, by_Wo, by_Ho;
    int units, per_pass, P, chunks, pixels_per_block;
    int step_b, step_y, step_x;                          // P pixels further, before the carries
};

template <int VW>
__global__ __launch_bounds__(256) void im2col_units_kernel(const uint32_t* __restrict__ in, ConvGeom g,
                                                           uint32_t* __restrict__ out, int64_t ld_out, UnitCopy c) {
    typedef uint32_t unit_t __attribute__((ext_vector_type(VW), aligned(4)));
    const int pixel_chunk = c.by_chunks(int(blockIdx.x)), chunk = int(blockIdx.x) - pixel_chunk * c.chunks;
    const int p = c.by_pass(int(threadIdx.x)), r = chunk * 256 + int(threadIdx.x) - p * c.per_pass;
    if (p >= c.P || r >= c.units) return;                // 256 % units leftover threads
    const int tap = c.by_tap(r), cu = r - tap * (g.Cw / VW);
    const int ky = c.by_kw(tap), kx = tap - ky * g.kw;
    const int first = pixel_chunk * c.pixels_per_block;
    const int M = int(g.M), q_end = min(first + c.pixels_per_block, M);
    int q = first + p;
    const int row = c.by_Wo(q);
    int b = c.by_Ho(row), ox = q - row * g.Wo, oy = row - b * g.Ho;
    const uint32_t* src = in + cu * VW;
    uint32_t* dst = out + q * ld_out + r * VW;
    const int64_t dst_step = c.P * ld_out;
    for (; q < q_end; q += c.P) {
        const int y = oy * g.stride + ky - g.pad;
        const int x = ox * g.stride + kx - g.pad;
        unit_t v;
#pragma unroll
        for (int e = 0; e < VW; ++e) v[e] = ~0u;
        if (y >= 0 && y < g.H && x >= 0 && x < g.W)
            v = *reinterpret_cast<const unit_t*>(src + ((b * g.H + y) * g.W + x) * g.Cw);
        *reinterpret_cast<unit_t*>(dst) = v;
        dst += dst_step;
        ox += c.step_x;
        oy += c.step_y;
        b += c.step_b;
        if (ox >= g.Wo) {
            ox -= g.Wo;
            ++oy;
        }
        if (oy >= g.Ho) {
            oy -= g.Ho;
            ++b;
        }
    }
}

// `len` (1..32) bits of a pixel's channel vector starting at channel ci.
__device__ inline uint32_t channel_bits(const uint32_t* __restrict__ px, int ci, int len) {
    const int w = ci >> 5, s = ci & 31;
    uint32_t v = px[w] >> s;
    if (s + len > 32) v |= px[w + 1] << (32 - s);
    return len == 32 ? v : (v & ((1u << len) - 1u));
}

__global__ __launch_bounds__(256) void im2col_bits_kernel(const uint32_t* __restrict__ in, ConvGeom g,
                                                          uint32_t* __restrict__ out, int64_t ld_out,
                                                          int64_t n_units) {
    for (int64_t u = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; u < n_units;
         u += int64_t(gridDim.x) * blockDim.x) {
        const int64_t m = u / g.Kwords;
        const int j = int(u - m * g.Kwords);
        const int ox = int(m % g.Wo);
        const int64_t t = m / g.Wo;
        const int oy = int(t % g.Ho);
        const int64_t b = t / g.Ho;
        const int k_end = min(32 * j + 32, g.Kbits);
        uint32_t word = 0u;
        int k = 32 * j;
        while (k < k_end) {
            const int tap = k / g.Cin;
            const int ci = k - tap * g.Cin;
            const int len = min(g.Cin - ci, k_end - k);
            const int ky = tap / g.kw, kx = tap - ky * g.kw;
            const int y = oy * g.stride + ky - g.pad;
            const int x = ox * g.stride + kx - g.pad;
            uint32_t bits = len == 32 ? ~0u : ((1u << len) - 1u);
            if (y >= 0 && y < g.H && x >= 0 && x < g.W)
                bits = channel_bits(in + ((b * g.H + y) * g.W + x) * g.Cw, ci, len);
            word |= bits << (k - 32 * j);
            k += len;
        }
        out[m * ld_out + j] = word;
    }
}

}  // namespace bnn

extern "C" int bnn_conv_im2col_pack(const uint32_t* in, int64_t B, int64_t H, int64_t W, int64_t Cin,
                                    int kh, int kw, int stride, int pad, uint32_t* out, int64_t ld_out,
                                    void* stream) {
    using namespace bnn;
    if (B < 0 || H < 1 || W < 1 || Cin < 1 || kh < 1 || kw < 1 || stride < 1 || pad < 0)
        return BNN_ERR_INVALID_ARG;
    if (B > kMaxDim || H > kMaxDim || W > kMaxDim || Cin > kMaxDim) return BNN_ERR_INVALID_ARG;
    if (H + 2 * int64_t(pad) < kh || W + 2 * int64_t(pad) < kw) return BNN_ERR_INVALID_ARG;
    const int64_t Ho = (H + 2 * int64_t(pad) - kh) / stride + 1;
    const int64_t Wo = (W + 2 * int64_t(pad) - kw) / stride + 1;
    const int64_t kbits = int64_t(kh) * kw * Cin;
    if (kbits > kMaxK || Ho > kMaxDim || Wo > kMaxDim) return BNN_ERR_INVALID_ARG;
    const int64_t kwords = ceil_div(kbits, 32);
    if (ld_out < kwords) return BNN_ERR_INVALID_ARG;
    if (B == 0) return BNN_OK;
    if (!in || !out) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(in, 4) || !aligned_to(out, 4)) return BNN_ERR_ALIGNMENT;

    ConvGeom g;
    g.B = int(B); g.H = int(H); g.W = int(W); g.Cin = int(Cin); g.Cw = int(ceil_div(Cin, 32));
    g.kh = kh; g.kw = kw; g.stride = stride; g.pad = pad;
    g.Ho = int(Ho); g.Wo = int(Wo);
    g.M = B * Ho * Wo;
    g.Kbits = int(kbits); g.Kwords = int(kwords);

    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t max_blocks = 256 * 64;
    auto blocks_for = [&](int64_t units) {
        int64_t b = ceil_div(units, 256);
        return unsigned(b > max_blocks ? max_blocks : b);
    };
    if (Cin % 32 == 0) {
        // 64 channels of 30 x 30 images, batch 100: 10.1 us word by word, with six 64-bit divisions for each; 4.9 in units
        // of two words.  128 channels of 32 x 32, batch 256: 10.2 with the images one by one in the grid and 64-bit places,
        // 9.7 now (75 MB written); 14 x 14 x 96, batch 100: 4.7 -> 3.5.
        const int vw = g.Cw % 4 == 0 ? 4 : g.Cw % 2 == 0 ? 2 : 1;
        // Pixels per workgroup: eight passes, and fewer until there are enough workgroups to fill the chip.
        UnitCopy c;
        c.units = int(kwords / vw);
        c.per_pass = c.units < 256 ? c.units : 256;
        c.P = 256 / c.per_pass;
        c.chunks = int(ceil_div(c.units, 256));
        c.pixels_per_block = c.P * 8;
        while (c.pixels_per_block > c.P && ceil_div(g.M, c.pixels_per_block) * c.chunks < 2048) c.pixels_per_block -= c.P;
        const int64_t blocks = ceil_div(g.M, c.pixels_per_block) * c.chunks;
        // 32-bit places and indexes: everything but batches of more than 2^31 pixels or input words.
        if (g.M <= kMaxDim - 4096 && B * H * W <= kMaxDim / g.Cw && blocks <= kMaxDim / 256) {
            const int64_t n_pix = Ho * Wo;
            c.step_b = int(c.P / n_pix);
            c.step_y = int(c.P % n_pix / Wo);
            c.step_x = int(c.P % n_pix % Wo);
            c.by_pass = fast_div(c.per_pass);
            c.by_chunks = fast_div(c.chunks);
            c.by_tap = fast_div(g.Cw / vw);
            c.by_kw = fast_div(kw);
            c.by_Wo = fast_div(Wo);
            c.by_Ho = fast_div(Ho);
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(256), 0, s, in, g, out, ld_out, c);
            };
            if (vw == 4) launch(im2col_units_kernel<4>);
            else if (vw == 2) launch(im2col_units_kernel<2>);
            else launch(im2col_units_kernel<1>);
        } else {
            const int64_t units = g.M * kwords;
            hipLaunchKernelGGL(im2col_words_kernel, dim3(blocks_for(units)), dim3(256), 0, s, in, g, out, ld_out, units);
        }
    } else {
        const int64_t units = g.M * kwords;
        hipLaunchKernelGGL(im2col_bits_kernel, dim3(blocks_for(units)), dim3(256), 0, s, in, g, out, ld_out,
                           units);
    }
    return bnn::check_launch();
}
