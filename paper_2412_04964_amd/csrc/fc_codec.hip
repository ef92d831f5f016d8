// fc_codec.hip -- launchers of the stand-alone quantize and dequantize kernels.
#include "fc_device.hpp"
#include "fc_launch.hpp"

namespace fc {

// Dequantizer, 4-bit codes, volumes of many rounds of wavefronts: with all that fit more accesses wait in the memory system than it serves
// well (see fc_sim.hip), and the launch limits the wavefronts per compute unit to 24, from 36 * 2^20 elements on.  us, without and with
// so many, hidden 8192, group 128: 24 M elements 11.18 / 11.22, 40 M 18.52 / 18.47, 48 M 21.7 / 21.0, 64 M 28.5 / 27.3, 128 M 55.2 / 51.6 (with
// 20 52.0); symmetric 128 M 57.8 / 52.6.  8-bit codes write half as much as they read, and no limit gains anything.
static bool limits_wavefronts(int bits, int64_t n_elems) { return bits == 4 && n_elems >= (int64_t)36 << 20; }

// Elements per lane and threads per workgroup of the quantizer.  A wavefront waits for all that it reads before it computes, so the
// finer its tile the earlier arithmetic and stores begin, and the more evenly the memory system is asked; a wider tile has fewer reductions
// and metadata per element, which counts where a group spans 16 lanes or more.  us by elements (2^20), hidden 8192, 16 elements per lane in
// workgroups of 64 / 128 / 256 threads, and 32 elements in workgroups of 128:
//   4-bit codes, group 32      1: 2.69 2.77 2.73 2.89   4: 3.89 3.89 3.86 4.01   8: 5.81 5.77 5.80 5.86   12: 7.49 7.76 7.86 7.75   24: 12.2 12.5 12.7 13.0
//                group 128  1/4: 2.13 2.24 2.30 2.42    6: 4.83 4.71 4.79 4.82   8: 5.70 5.60 5.68 5.70   10: 6.48 6.75 6.85 6.43   32: 15.4 15.2 15.4 15.8
//                          128: 52.6 52.9 53.9 53.6 (with fewer wavefronts per compute unit than fit: 53.8 with 24, 58 with 20)
//   16 elements in workgroups of 64, and 32 in workgroups of 256 (of 128 for group 256):
//                group 256    6: 4.93 4.79   16: 8.99 8.89   24: 12.10 12.22   32: 15.36 15.67   128: 52.4 53.5
//                group 1024   6: 4.97 4.85   16: 8.92 8.98   24: 11.98 12.25   32: 15.08 15.67   128: 51.3 54.0
//   8-bit codes have 16 elements in any case; workgroups of 64 and of 256: group 32  1/4: 2.10 2.17   1: 2.70 2.77   4: 4.29 4.10   16: 10.37 10.40;
//                group 128  1/4: 2.12 2.20   2: 3.06 3.09   3: 3.55 3.49   32: 18.1 17.7;   group 256  1: 2.84 2.80
constexpr int64_t kOneRound = (int64_t)8 << 20;          // elements that 256 compute units of 32 wavefronts hold, at 16 per lane
struct QuantizeForm {
    int epl, threads;
};
static QuantizeForm quantize_form(int bits, int64_t n_elems, int group)
{
    if (bits == 8) return {16, group <= 128 && n_elems <= (int64_t)5 << 19 ? 64 : 256};
    if (group <= 128) return {16, n_elems > (int64_t)3 << 20 && n_elems <= kOneRound ? 128 : 64};
    if (group <= 1024 && n_elems >= 3 * kOneRound) return {16, 64};
    return {32, group == 256 ? 128 : 256};
}

template <int BITS, int EPL, int BT, int LPG>
static hipError_t launch_q(int codec, hipStream_t stream, const uint16_t *x, int64_t n_elems, int group,
                           uint8_t *c, float *scales, float *zeros)
{
    constexpr int64_t tile = (int64_t)BT * EPL;
    const dim3 grid((unsigned)((n_elems + tile - 1) / tile)), block(BT);
    const int lpg = group / EPL, sh = log2_int(group);
    if (codec == CODEC_ASYM)
        return launch_kernel(k_quantize<BITS, LPG, kAsym, EPL, BT>, grid, block, stream, x, n_elems, lpg, sh, c, scales, zeros);
    else if (codec == CODEC_SYM)
        return launch_kernel(k_quantize<BITS, LPG, kSym, EPL, BT>, grid, block, stream, x, n_elems, lpg, sh, c, scales, nullptr);
    else if (codec == CODEC_ASYMH)
        return launch_kernel(k_quantize<BITS, LPG, kAsymH, EPL, BT>, grid, block, stream, x, n_elems, lpg, sh, c, scales, nullptr);
    else if constexpr (BITS == 8)
        return launch_kernel(k_quantize<8, LPG, kFp8, EPL, BT>, grid, block, stream, x, n_elems, lpg, sh, c, scales, nullptr);
    return hipErrorInvalidValue;
}

// groups of 32, 64 and 128, lanes per group known to the compiler
template <int BITS, int BT>
static hipError_t launch_q_narrow(int codec, hipStream_t stream, const uint16_t *x, int64_t n_elems, int group,
                                  uint8_t *c, float *scales, float *zeros)
{
    switch (group) {
    case 32: return launch_q<BITS, 16, BT, 2>(codec, stream, x, n_elems, group, c, scales, zeros);
    case 64: return launch_q<BITS, 16, BT, 4>(codec, stream, x, n_elems, group, c, scales, zeros);
    case 128: return launch_q<BITS, 16, BT, 8>(codec, stream, x, n_elems, group, c, scales, zeros);
    default: return hipErrorInvalidValue;
    }
}

template <int BITS>
static hipError_t launch_q_bits(int codec, hipStream_t stream, const uint16_t *x, int64_t n_elems, int group,
                                uint8_t *c, float *scales, float *zeros)
{
    const QuantizeForm f = quantize_form(BITS, n_elems, group);
    if (group <= 128) {
        if (f.threads == 64) return launch_q_narrow<BITS, 64>(codec, stream, x, n_elems, group, c, scales, zeros);
        return launch_q_narrow<BITS, BITS == 4 ? 128 : 256>(codec, stream, x, n_elems, group, c, scales, zeros);
    }
    if constexpr (BITS == 4) {
        if (f.epl == 16) return launch_q<4, 16, 64, 0>(codec, stream, x, n_elems, group, c, scales, zeros);
        if (group == 256) return launch_q<4, 32, 128, 8>(codec, stream, x, n_elems, group, c, scales, zeros);
    }
    return launch_q<BITS, lane_elems(BITS), 256, 0>(codec, stream, x, n_elems, group, c, scales, zeros);
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

// 4-bit codes: up to one round of wavefronts 16 elements per lane, for the reason given at quantize_form; above it 32 elements, whose
// loads and stores are twice as wide.  us by elements (2^20), hidden 8192, 32 / 16 elements: group 32  1/4: 2.11 / 1.92   2: 2.76 / 2.67   6: 4.16 / 4.00
// 8: 4.91 / 4.79   12: 6.41 / 6.96   32: 15.4 / 16.2;   group 128  1/4: 2.11 / 1.92   1: 2.39 / 2.22   6: 4.09 / 3.92   8: 4.79 / 4.65   12: 6.03 / 6.90.
// Workgroups of 64 or 128 threads: from -2 to +25 %.  8-bit codes with 8 elements per lane: 1/4 M 1.94 / 1.87, 2 M 2.77 / 2.88, 8 M 5.28 / 6.58.
template <int BITS, int EPL>
static hipError_t launch_dq(int codec, hipStream_t stream, const uint8_t *c, const float *scales, const float *zeros, int64_t n_elems,
                            int group_shift, uint16_t *y)
{
    constexpr int64_t tile = (int64_t)kBlockThreads * EPL;
    const dim3 grid((unsigned)((n_elems + tile - 1) / tile)), block(kBlockThreads);
    const size_t pad = limits_wavefronts(BITS, n_elems) ? lds_to_limit(6, (size_t)tile * 2) : 0;
    if (codec == CODEC_ASYM)
        return launch_kernel_lds(k_dequantize<BITS, kAsym, EPL>, grid, block, pad, stream, c, scales, zeros, n_elems, group_shift, y);
    if (codec == CODEC_SYM)
        return launch_kernel_lds(k_dequantize<BITS, kSym, EPL>, grid, block, pad, stream, c, scales, nullptr, n_elems, group_shift, y);
    if (codec == CODEC_ASYMH)
        return launch_kernel_lds(k_dequantize<BITS, kAsymH, EPL>, grid, block, pad, stream, c, scales, nullptr, n_elems, group_shift, y);
    if constexpr (BITS == 8)
        return launch_kernel_lds(k_dequantize<8, kFp8, EPL>, grid, block, pad, stream, c, scales, nullptr, n_elems, group_shift, y);
    return hipErrorInvalidValue;
}

hipError_t launch_dequantize(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                             int64_t n_elems, int group, void *y_f16, hipStream_t stream)
{
    const uint8_t *c = static_cast<const uint8_t *>(codes);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    const int sh = log2_int(group);
    if (bits == 8) return launch_dq<8, 16>(codec, stream, c, scales, zeros, n_elems, sh, y);
    if (n_elems <= kOneRound) return launch_dq<4, 16>(codec, stream, c, scales, zeros, n_elems, sh, y);
    return launch_dq<4, 32>(codec, stream, c, scales, zeros, n_elems, sh, y);
}

}  // namespace fc
