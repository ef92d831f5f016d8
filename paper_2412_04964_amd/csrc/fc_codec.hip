// fc_codec.hip -- launchers of the stand-alone quantize and dequantize kernels.
#include "fc_device.hpp"
#include "fc_launch.hpp"

namespace fc {

// 4-bit codes, volumes of many rounds of wavefronts: with all that fit more reads wait in the memory system than it serves
// well (see fc_sim.hip), and the launch limits the wavefronts per compute unit, 16 in the quantizer (20 where its workgroups have four), 24 in
// the dequantizer, from 36 * 2^20 elements on.  us, without and with so many, hidden 8192, group 128: quantize 32 M elements 15.49 / 15.42, 40 M 18.83 / 18.46, 64 M
// 28.8 / 27.8, 128 M 55.8 / 53.2 (with 14 wavefronts 52.8, but 32 M 15.56; with 12 55.1); symmetric 128 M 55.5 / 53.7; group 1024 64 M 28.6 / 28.0;
// dequantize 24 M 11.18 / 11.22, 40 M 18.52 / 18.47, 48 M 21.7 / 21.0, 64 M 28.5 / 27.3, 128 M 55.2 / 51.6 (with 20 52.0); symmetric 128 M 57.8 /
// 52.6.  8-bit codes write half as much as they read, and no limit gains anything.
static bool limits_wavefronts(int bits, int64_t n_elems) { return bits == 4 && n_elems >= (int64_t)36 << 20; }

template <int BITS, int LPG>
static hipError_t launch_q(int codec, hipStream_t stream, const uint16_t *x, int64_t n_elems, int lpg,
                     int group_shift, uint8_t *c, float *scales, float *zeros)
{
    constexpr int BT = quantize_block_threads(BITS, LPG);
    const int64_t tile = (int64_t)BT * lane_elems(BITS);
    const dim3 grid((unsigned)((n_elems + tile - 1) / tile)), block(BT);
    const size_t pad = limits_wavefronts(BITS, n_elems) ? lds_to_limit(BT == 128 ? 8 : 5, BT * lane_elems(BITS) * 2) : 0;
    if (codec == CODEC_ASYM)
        return launch_kernel_lds(k_quantize<BITS, LPG, kAsym>, grid, block, pad, stream, x, n_elems, lpg, group_shift, c, scales, zeros);
    else if (codec == CODEC_SYM)
        return launch_kernel_lds(k_quantize<BITS, LPG, kSym>, grid, block, pad, stream, x, n_elems, lpg, group_shift, c, scales, nullptr);
    else if (codec == CODEC_ASYMH)
        return launch_kernel_lds(k_quantize<BITS, LPG, kAsymH>, grid, block, pad, stream, x, n_elems, lpg, group_shift, c, scales, nullptr);
    else if constexpr (BITS == 8)
        return launch_kernel_lds(k_quantize<8, LPG, kFp8>, grid, block, pad, stream, x, n_elems, lpg, group_shift, c, scales, nullptr);
    return hipErrorInvalidValue;
}

template <int BITS>
static hipError_t launch_q_bits(int codec, hipStream_t stream, const uint16_t *x, int64_t n_elems, int group,
                          uint8_t *c, float *scales, float *zeros)
{
    const int lpg = group / lane_elems(BITS), sh = log2_int(group);
    switch (lpg) {
    case 1: return launch_q<BITS, 1>(codec, stream, x, n_elems, lpg, sh, c, scales, zeros);
    case 2: return launch_q<BITS, 2>(codec, stream, x, n_elems, lpg, sh, c, scales, zeros);
    case 4: return launch_q<BITS, 4>(codec, stream, x, n_elems, lpg, sh, c, scales, zeros);
    case 8: return launch_q<BITS, 8>(codec, stream, x, n_elems, lpg, sh, c, scales, zeros);
    default: return launch_q<BITS, 0>(codec, stream, x, n_elems, lpg, sh, c, scales, zeros);
    }
}

hipError_t launch_quantize(int bits, int codec, const void *x_f16, int64_t n_elems, int group,
                           void *codes, float *scales, float *zeros, hipStream_t stream)
{
    if (codec == CODEC_FP8 && bits != 8) return hipErrorInvalidValue;
    if (is_wide_group(bits, group))
        return launch_quantize_wide(bits, codec, x_f16, n_elems, group, codes, scales, zeros, stream);
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint8_t *c = static_cast<uint8_t *>(codes);
    if (bits == 4) return launch_q_bits<4>(codec, stream, x, n_elems, group, c, scales, zeros);
    return launch_q_bits<8>(codec, stream, x, n_elems, group, c, scales, zeros);
}

hipError_t launch_dequantize(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                             int64_t n_elems, int group, void *y_f16, hipStream_t stream)
{
    const uint8_t *c = static_cast<const uint8_t *>(codes);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    const int sh = log2_int(group);
    const int64_t tile = block_elems(bits);
    const dim3 grid((unsigned)((n_elems + tile - 1) / tile)), block(kBlockThreads);
    const size_t pad = limits_wavefronts(bits, n_elems) ? lds_to_limit(6, (size_t)tile * 2) : 0;
    if (codec == CODEC_FP8) {
        if (bits != 8) return hipErrorInvalidValue;
        return launch_kernel_lds(k_dequantize<8, kFp8>, grid, block, pad, stream, c, scales, nullptr, n_elems, sh, y);
    } else if (codec == CODEC_ASYMH) {
        if (bits == 4)
            return launch_kernel_lds(k_dequantize<4, kAsymH>, grid, block, pad, stream, c, scales, nullptr, n_elems, sh, y);
        else
            return launch_kernel_lds(k_dequantize<8, kAsymH>, grid, block, pad, stream, c, scales, nullptr, n_elems, sh, y);
    } else if (bits == 4 && codec == CODEC_ASYM)
        return launch_kernel_lds(k_dequantize<4, kAsym>, grid, block, pad, stream, c, scales, zeros, n_elems, sh, y);
    else if (bits == 4)
        return launch_kernel_lds(k_dequantize<4, kSym>, grid, block, pad, stream, c, scales, nullptr, n_elems, sh, y);
    else if (codec == CODEC_ASYM)
        return launch_kernel_lds(k_dequantize<8, kAsym>, grid, block, pad, stream, c, scales, zeros, n_elems, sh, y);
    else
        return launch_kernel_lds(k_dequantize<8, kSym>, grid, block, pad, stream, c, scales, nullptr, n_elems, sh, y);
}

}  // namespace fc
