// fc_fused.hip -- instantiations of the fused Dequantize-ReduceSum-Quantize
// kernel for one (FC_BITS_IN, FC_BITS_OUT) pair and every fan-in 1..8.
// Compiled once per pair (the build defines the two macros).
#include "fc_device.hpp"
#include "fc_fused_small.hpp"
#include "fc_launch.hpp"

#if !defined(FC_BITS_IN) || !defined(FC_BITS_OUT)
#error "define FC_BITS_IN and FC_BITS_OUT (4 or 8)"
#endif

#define FC_CAT3(a, b, c) a##b##_##c
#define FC_NAME(in, out) FC_CAT3(launch_fused_, in, out)

namespace fc {

template <int NSRC, int LPG>
static hipError_t launch_nl(const FusedArgs &a, hipStream_t stream)
{
    constexpr int BT = fused_block_threads(LPG);
    const int64_t tile = (int64_t)BT * lane_elems(FC_BITS_IN);
    const int64_t blocks = (a.n_elems + tile - 1) / tile;
#if FC_BITS_IN == 8 && FC_BITS_OUT == 8
    if (a.codec == CODEC_FP8) {
        return launch_kernel(k_dequant_reduce_requant_sym<8, 8, NSRC, LPG, true>, dim3((unsigned)blocks), dim3(BT), stream,
                static_cast<const uint8_t *>(a.codes_in), a.codes_stride, a.scales_in, a.meta_stride,
                a.n_elems, log2_int(a.group),
                static_cast<uint8_t *>(a.codes_out), a.scales_out);
    }
#endif
    if (a.codec == CODEC_SYM) {
        return launch_kernel(k_dequant_reduce_requant_sym<FC_BITS_IN, FC_BITS_OUT, NSRC, LPG>, dim3((unsigned)blocks), dim3(BT), stream,
                static_cast<const uint8_t *>(a.codes_in), a.codes_stride, a.scales_in, a.meta_stride,
                a.n_elems, log2_int(a.group),
                static_cast<uint8_t *>(a.codes_out), a.scales_out);
    }
    // Where fc_fused_small.hpp is not taken, at most one workgroup per compute unit: the shorter chain of instructions
    // (hidden 8192, 8 to 128 tokens, us under graph replay, accumulate_nibbles / accumulate_fast: g = 1024, INT4 N = 4
    // 3.29 / 3.14 at 8 tokens, 3.38 / 3.23 at 128, but 3.69 / 3.91 at 160, where a second workgroup comes in; N = 3 4 -> 8 bit
    // 3.27 / 3.11 at 128, compact metadata N = 4 3.38 / 3.14; g = 8192 3.59 / 3.47 at 256 tokens, 3.99 / 4.14 at 384).
    // The same for two or three sources coded again at 8 bit, volumes that the memory-side cache holds, groups of 8 lanes and more
    // (replayed graphs over four buffer sets, us, accumulate_nibbles / accumulate_fast: g = 256, N = 2 6 M elements 4.87 / 4.84,
    // 8 M 5.12 / 5.00, 16 M 10.67 / 9.67, 28 M 16.08 / 14.02, 32 M 16.82 / 15.31; N = 3 8 M 6.19 / 5.76, 12 M 9.87 / 9.19, 20 M
    // 14.08 / 12.91, 32 M 21.73 / 17.90; g = 1024 the same; over 1.2 GB of buffers both are equal up to
    // 40 M, 64 M 23.5 / 25.2, 28.6 / 29.6.  g = 128, N = 2 8 M 5.08 / 5.52, 24 M 13.2 / 14.5; N = 4 16 M 12.46 / 12.79).
    constexpr bool kAloneOnUnit = FC_BITS_IN == 4 && ((NSRC <= 2 && LPG >= 32) || (NSRC <= 4 && LPG == 256));
    constexpr bool kCached = FC_BITS_IN == 4 && FC_BITS_OUT == 8 && (NSRC == 2 || NSRC == 3) && LPG >= 8;
    if constexpr (kAloneOnUnit || kCached) {
        constexpr int kComputeUnits = 256;
        constexpr int64_t k1M = (int64_t)1 << 20;
        const bool alone = kAloneOnUnit && blocks <= kComputeUnits;
        const bool cached = kCached && a.n_elems > 6 * k1M && a.n_elems <= 32 * k1M;
        if ((alone || cached) && a.codec == CODEC_ASYM)
            return launch_kernel(k_dequant_reduce_requant<FC_BITS_IN, FC_BITS_OUT, NSRC, LPG, false, BT, 0, true>, dim3((unsigned)blocks), dim3(BT), stream,
                    static_cast<const uint8_t *>(a.codes_in), a.codes_stride, a.scales_in, a.zeros_in,
                    a.meta_stride, a.n_elems, log2_int(a.group),
                    static_cast<uint8_t *>(a.codes_out), a.scales_out, a.zeros_out);
        if constexpr (kAloneOnUnit)
            if (alone && a.codec == CODEC_ASYMH)
                return launch_kernel(k_dequant_reduce_requant<FC_BITS_IN, FC_BITS_OUT, NSRC, LPG, true, BT, 0, true>, dim3((unsigned)blocks), dim3(BT), stream,
                        static_cast<const uint8_t *>(a.codes_in), a.codes_stride, a.scales_in, nullptr,
                        a.meta_stride, a.n_elems, log2_int(a.group),
                        static_cast<uint8_t *>(a.codes_out), a.scales_out, nullptr);
    }
    if (a.codec == CODEC_ASYMH) {
        return launch_kernel(k_dequant_reduce_requant<FC_BITS_IN, FC_BITS_OUT, NSRC, LPG, true>, dim3((unsigned)blocks), dim3(BT), stream,
                static_cast<const uint8_t *>(a.codes_in), a.codes_stride, a.scales_in, nullptr,
                a.meta_stride, a.n_elems, log2_int(a.group),
                static_cast<uint8_t *>(a.codes_out), a.scales_out, nullptr);
    }
    if (a.codec != CODEC_ASYM) return hipErrorInvalidValue;
    return launch_kernel(k_dequant_reduce_requant<FC_BITS_IN, FC_BITS_OUT, NSRC, LPG>, dim3((unsigned)blocks), dim3(BT), stream,
            static_cast<const uint8_t *>(a.codes_in), a.codes_stride, a.scales_in, a.zeros_in,
            a.meta_stride, a.n_elems, log2_int(a.group),
            static_cast<uint8_t *>(a.codes_out), a.scales_out, a.zeros_out);
}

template <int CODEC, int NSRC, int BT>
static hipError_t launch_small_bt(const FusedArgs &a, int64_t blocks, int threads, int lane_elems, hipStream_t stream)
{
    return launch_kernel(k_fused_small<CODEC, FC_BITS_IN, FC_BITS_OUT, NSRC, BT>, dim3((unsigned)blocks), dim3(threads), stream,
            static_cast<const uint8_t *>(a.codes_in), a.codes_stride, a.scales_in, a.zeros_in,
            a.meta_stride, a.n_elems, log2_int(a.group), a.group / lane_elems,
            static_cast<uint8_t *>(a.codes_out), a.scales_out, a.zeros_out);
}

template <int CODEC, int NSRC>
static hipError_t launch_small(const FusedArgs &a, hipStream_t stream)
{
    if (a.group > fused_small_wave_elems(FC_BITS_IN))
        return launch_small_bt<CODEC, NSRC, 0>(a, a.n_elems / a.group, a.group / 8, 8, stream);
    const int64_t wave_elems = fused_small_wave_elems(FC_BITS_IN), waves = (a.n_elems + wave_elems - 1) / wave_elems;
    const int lane_elems = fused_small_lane_elems(FC_BITS_IN);
    if (waves <= kFusedSmallAlone) return launch_small_bt<CODEC, NSRC, 64>(a, waves, 64, lane_elems, stream);
    return launch_small_bt<CODEC, NSRC, kBlockThreads>(a, (waves + kBlockWaves - 1) / kBlockWaves, kBlockThreads, lane_elems, stream);
}

// one instantiation per group width in lanes: 1 ... 128 lanes in 128-thread workgroups, 256 lanes in
// 256-thread workgroups (wider groups go to fc_wide.hip before this point)
template <int NSRC>
static hipError_t launch_n(const FusedArgs &a, hipStream_t stream)
{
    // launch-bound volumes: one code word per lane and source
    if (fused_small_applies(a.codec, FC_BITS_IN, FC_BITS_OUT, NSRC, a.n_elems, a.group)) {
        switch (a.codec) {
        case CODEC_ASYM: return launch_small<kAsym, NSRC>(a, stream);
        case CODEC_SYM: return launch_small<kSym, NSRC>(a, stream);
        case CODEC_ASYMH: return launch_small<kAsymH, NSRC>(a, stream);
#if FC_BITS_IN == 8 && FC_BITS_OUT == 8
        case CODEC_FP8: return launch_small<kFp8, NSRC>(a, stream);
#endif
        default: return hipErrorInvalidValue;
        }
    }
    switch (a.group / lane_elems(FC_BITS_IN)) {
    case 1: return launch_nl<NSRC, 1>(a, stream);
    case 2: return launch_nl<NSRC, 2>(a, stream);
    case 4: return launch_nl<NSRC, 4>(a, stream);
    case 8: return launch_nl<NSRC, 8>(a, stream);
    case 16: return launch_nl<NSRC, 16>(a, stream);
    case 32: return launch_nl<NSRC, 32>(a, stream);
    case 64: return launch_nl<NSRC, 64>(a, stream);
    case 128: return launch_nl<NSRC, 128>(a, stream);
    case 256: return launch_nl<NSRC, 256>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t FC_NAME(FC_BITS_IN, FC_BITS_OUT)(const FusedArgs &a, hipStream_t stream)
{
    switch (a.n_src) {
    case 1: return launch_n<1>(a, stream);
    case 2: return launch_n<2>(a, stream);
    case 3: return launch_n<3>(a, stream);
    case 4: return launch_n<4>(a, stream);
    case 5: return launch_n<5>(a, stream);
    case 6: return launch_n<6>(a, stream);
    case 7: return launch_n<7>(a, stream);
    case 8: return launch_n<8>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fc
