// fc_codec.hip -- launchers of the stand-alone quantize and dequantize kernels.
#include "fc_device.hpp"
#include "fc_fused_small.hpp"
#include "fc_launch.hpp"

namespace fc {

// Dequantizer, 4-bit codes, volumes of many rounds of wavefronts: with all that fit more accesses wait in the memory system than it serves
// well (see fc_sim.hip), and the launch limits the wavefronts per compute unit to 24, from 48 * 2^20 elements on.  us, without and with
// so many, hidden 8192, group 128: 24 M elements 11.18 / 11.22, 48 M 21.7 / 21.0, 64 M 29.4 / 28.4, 128 M 55.2 / 51.6 (with 20 52.0);
// symmetric 40 M 16.9 / 17.7 (over 700 MB of buffers 19.2 / 19.2), 64 M 29.4 / 28.4, 128 M 57.8 / 52.6.  8-bit codes write half as much as
// they read, and no limit gains anything.
static bool limits_wavefronts(int bits, int64_t n_elems) { return bits == 4 && n_elems >= (int64_t)48 << 20; }

// Elements per lane and threads per workgroup of the quantizer for 4-bit codes, past quantize_small_applies.  A wavefront waits for
// all that it reads before it computes, so the finer its tile the earlier arithmetic and stores begin, and the more evenly the memory
// system is asked; a wider tile has fewer reductions and metadata per element, which counts where a group spans 16 lanes or more.
// Replayed graphs over two or three buffer sets / over 700 MB of them, us by elements (2^20), hidden 8192:
//   groups of up to 128, 32 elements per lane in workgroups of 128; 16 in workgroups of 64 / 256 (128 threads lie between)
//     asymmetric, group 128   4.5: 3.24, 3.55 / 3.28   6: 3.72, 4.20 / 3.60   8: 4.72, 4.96 / 4.64   10: 5.81, 5.91 / 6.13
//       16: 8.31, 8.65 / 8.61   40: 19.5, 19.1 / 19.2   64: 30.2, 29.1 / 29.1;   700 MB  6: 3.93, 4.28 / 3.82   10: 6.54, 6.62 / 6.85
//       24: 12.8, 12.4 / 12.6   64: 30.2, 29.2 / 29.5
//     symmetric, group 32     4.5: 3.13, 3.41 / 3.09   8: 4.69, 4.83 / 4.56   10: 5.75, 5.70 / 6.03   24: 11.3, 10.9 / 11.2
//   groups of 256 to 1024, 32 elements / 16 in workgroups of 64
//     asymmetric, group 256   24: 11.2 / 11.9   32: 15.3 / 15.7   36: 17.9 / 17.5   64: 29.9 / 29.1;   700 MB  24: 12.6 / 12.4   40: 19.8 / 19.3
//     group 1024              32: 14.7 / 15.1   36: 17.3 / 17.1   64: 29.8 / 28.1
constexpr int64_t kOneRound = (int64_t)8 << 20;          // elements that 256 compute units of 32 wavefronts hold, at 16 per lane
struct QuantizeForm {
    int epl, threads;
};
static QuantizeForm quantize_form(int64_t n_elems, int group)
{
    if (n_elems / 16 >= (int64_t)1 << 32) return {32, 256};             // more threads than the runtime launches
    if (group <= 128) return {16, n_elems <= kOneRound ? 256 : 64};
    if (group <= 1024 && n_elems >= (int64_t)36 << 20) return {16, 64};
    return {32, group == 256 ? 128 : 256};
}

// Few elements: 8 per lane, loaded straight into registers instead of through LDS, since a lane's 16 bytes are one access.  SPANS, a
// group of more than 512 is a workgroup, its wavefronts exchange minimum and maximum with one barrier.  The limits by how the two sides
// cross; the quantizers without a zero-point have less to compute per lane and cross earlier.  us by elements (2^20), hidden 8192, the
// other forms / this one:
//   4-bit codes, group 128: asymmetric  1/8: 2.09 / 2.03   1: 2.72 / 2.31   2.5: 2.61 / 2.38   3: 2.64 / 2.57   4: 2.76 / 2.85   4.5: 3.24 / 3.20
//     5: 3.44 / 3.48, over 700 MB  3: 3.03 / 2.71   4: 3.14 / 3.09   5: 3.54 / 3.70;   symmetric  4: 2.69 / 2.67, 700 MB 2.98 / 2.93
//     binary16 metadata  3.5: 2.68 / 2.73, 700 MB -3 to -5 %   4: 2.77 / 2.93
//   group 256, 512: 2.5: 2.60 / 2.57   3.5: 2.63 / 2.91;   group 1024: symmetric, 700 MB  1.5: +3 %   2.5: +7 %
//   group 8192: asymmetric  1: 3.35 / 2.72   3: 4.33 / 3.84;   symmetric  2: -7 %   2.5: +4 %
//   8-bit codes, group 32: 1/2: 2.53 / 2.28   1: 2.72 / 2.35;   group 256: asymmetric  1.5: 3.00 / 2.71, symmetric +3 %
//   group 1024: 1: 2.89 / 2.55   1.25: +2 to +5 %   1.5: +6 to +9 %;   group 4096: 1/4: 2.54 / 2.21   2: 3.59 / 3.24   3: 4.03 / 4.36
static bool quantize_small_applies(int codec, int bits, int64_t n_elems, int group)
{
    const bool zero_point = codec == CODEC_ASYM || codec == CODEC_ASYMH;
    int halves;                                                          // of 2^20 elements
    if (bits == 4)
        halves = group <= 128 ? (zero_point ? 7 : 8) : group <= 512 ? 5 : group == 1024 ? 3 : zero_point ? 6 : group == 2048 ? 3 : 4;
    else
        halves = group >= 2048 ? 4 : zero_point && group <= 512 ? 3 : 2;
    return group <= 8192 && n_elems <= halves * ((int64_t)1 << 19);
}
template <int BITS, int CODEC, bool SPANS>
__global__ __launch_bounds__(SPANS ? 1024 : kBlockThreads) void k_quantize_small(const uint16_t *__restrict__ x, int64_t n_elems, int lpg, int group_shift,
                                                         uint8_t *__restrict__ codes, float *__restrict__ scales, float *__restrict__ zeros)
{
    constexpr int E = 8;
    __shared__ float slot[SPANS ? 16 : 1][2];
    const int64_t e = (SPANS ? (int64_t)blockIdx.x << group_shift : (int64_t)blockIdx.x * (kBlockThreads * E)) + threadIdx.x * E;
    const bool live = SPANS || e < n_elems;
    const u32x4 raw = *reinterpret_cast<const u32x4 *>(x + (live ? e : 0));
    float v[E];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const h2 p = as_h2(raw[k]);
        v[2 * k] = (float)p.x;
        v[2 * k + 1] = (float)p.y;
    }
    float mn, mx, s, inv, zf = 0.0f;
    u32 word[BITS / 4];
    lane_minmax(v, mn, mx);
    if constexpr (SPANS) span_minmax(mn, mx, (u32)lpg >> 6, slot);
    else group_minmax<0>(mn, mx, lpg);
    if constexpr (CODEC == kFp8) {
        group_params_absmax<448>(fmaxf(fabsf(mn), fabsf(mx)), s, inv);
        pack_lane_fp8<E>(v, inv, word);
    } else if constexpr (CODEC == kSym) {
        group_params_sym<BITS>(fmaxf(fabsf(mn), fabsf(mx)), s, inv);
        pack_lane_sym<BITS, E>(v, inv, word);
    } else {
        group_params<BITS, CODEC == kAsymH>(mn, mx, s, inv, zf);
        pack_lane<BITS, E>(v, inv, zf, mx, word);
    }
    if (!live) return;
    uint8_t *to = codes + e * BITS / 8;
    if constexpr (BITS == 4) *reinterpret_cast<u32 *>(to) = word[0];
    else *reinterpret_cast<u32x2 *>(to) = u32x2{word[0], word[1]};
    if ((threadIdx.x & (u32)(lpg - 1)) == 0) {
        const int64_t gi = e >> group_shift;
        scales[gi] = CODEC == kAsymH ? __builtin_bit_cast(float, pack_meta(s, zf)) : s;
        if constexpr (CODEC == kAsym) zeros[gi] = zf;
    }
}

template <int BITS, bool SPANS>
static hipError_t launch_q_small(int codec, hipStream_t stream, const uint16_t *x, int64_t n_elems, int group, uint8_t *c, float *scales,
                                 float *zeros)
{
    const dim3 block(SPANS ? group / 8 : kBlockThreads), grid((unsigned)((n_elems + block.x * 8 - 1) / (block.x * 8)));
    const int lpg = group / 8, sh = log2_int(group);
    switch (codec) {
    case CODEC_ASYM: return launch_kernel(k_quantize_small<BITS, kAsym, SPANS>, grid, block, stream, x, n_elems, lpg, sh, c, scales, zeros);
    case CODEC_SYM: return launch_kernel(k_quantize_small<BITS, kSym, SPANS>, grid, block, stream, x, n_elems, lpg, sh, c, scales, nullptr);
    case CODEC_ASYMH: return launch_kernel(k_quantize_small<BITS, kAsymH, SPANS>, grid, block, stream, x, n_elems, lpg, sh, c, scales, nullptr);
    case CODEC_FP8:
        if constexpr (BITS == 8) return launch_kernel(k_quantize_small<8, kFp8, SPANS>, grid, block, stream, x, n_elems, lpg, sh, c, scales, nullptr);
        [[fallthrough]];
    default: return hipErrorInvalidValue;
    }
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
    if (quantize_small_applies(codec, BITS, n_elems, group))
        return group > 512 ? launch_q_small<BITS, true>(codec, stream, x, n_elems, group, c, scales, zeros)
                           : launch_q_small<BITS, false>(codec, stream, x, n_elems, group, c, scales, zeros);
    if (is_wide_group(BITS, group)) return launch_quantize_wide(BITS, codec, x, n_elems, group, c, scales, zeros, stream);
    if constexpr (BITS == 4) {
        const QuantizeForm f = quantize_form(n_elems, group);
        if (group <= 128 && f.epl == 16)
            return f.threads == 64 ? launch_q_narrow<4, 64>(codec, stream, x, n_elems, group, c, scales, zeros)
                                   : launch_q_narrow<4, 256>(codec, stream, x, n_elems, group, c, scales, zeros);
        if (f.epl == 16) return launch_q<4, 16, 64, 0>(codec, stream, x, n_elems, group, c, scales, zeros);
        if (f.threads == 128) return launch_q<4, 32, 128, 8>(codec, stream, x, n_elems, group, c, scales, zeros);
    } else if (group <= 128) {
        return launch_q_narrow<8, 256>(codec, stream, x, n_elems, group, c, scales, zeros);
    }
    return launch_q<BITS, lane_elems(BITS), 256, 0>(codec, stream, x, n_elems, group, c, scales, zeros);
}

hipError_t launch_quantize(int bits, int codec, const void *x_f16, int64_t n_elems, int group,
                           void *codes, float *scales, float *zeros, hipStream_t stream)
{
    if (codec == CODEC_FP8 && bits != 8) return hipErrorInvalidValue;
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint8_t *c = static_cast<uint8_t *>(codes);
    if (bits == 4) return launch_q_bits<4>(codec, stream, x, n_elems, group, c, scales, zeros);
    return launch_q_bits<8>(codec, stream, x, n_elems, group, c, scales, zeros);
}

// 4-bit codes: up to one round of wavefronts 16 elements per lane, for the reason given at quantize_form; above it 32 elements, whose
// loads and stores are twice as wide.  Without zero-points to load the wide tile catches up sooner where the buffers are not cached, hence
// another limit.  us by elements (2^20), hidden 8192, group 128, 32 / 16 elements (over 700 MB of buffers): asymmetric  1/4: 2.11 / 1.92
// 1: 2.39 / 2.22   6: 3.52 / 3.46 (4.11 / 3.94)   8: 4.09 / 4.10 (4.76 / 4.67)   12: 6.03 / 6.90;   symmetric  4: 2.80 / 2.85 (3.19 / 3.01)   5: 3.10 / 3.05
// (3.47 / 3.46)   6: 3.37 / 3.33 (3.76 / 3.94)   8: 3.95 / 3.92 (4.36 / 5.08);   binary16 metadata  8: 4.08 / 3.95 (4.42 / 4.67).  Workgroups of 64 or
// 128 threads: from -2 to +25 %.  8-bit codes with 8 elements per lane: 1/4 M 1.94 / 1.87, 2 M 2.77 / 2.88, 8 M 5.28 / 6.58.
static bool dequantize_narrow_applies(int codec, int64_t n_elems) { return n_elems <= (codec == CODEC_ASYM ? kOneRound : kOneRound * 5 / 8); }
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
    if (dequantize_narrow_applies(codec, n_elems)) return launch_dq<4, 16>(codec, stream, c, scales, zeros, n_elems, sh, y);
    return launch_dq<4, 32>(codec, stream, c, scales, zeros, n_elems, sh, y);
}

}  // namespace fc
