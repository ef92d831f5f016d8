// fc_launch.hpp -- host-side launch functions implemented by the .hip units.
// Internal to the library; the public interface is include/fc.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>
#include <utility>

namespace fc {

// Launch `kernel` and return the status of THIS launch.  (The <<< >>> syntax reports failures only
// through the thread's last-error slot, which hipGetLastError would also clear of errors that other
// code left there, and a stale one would be taken for a failure of a launch that succeeded.)
template <typename... P, size_t... I>
inline hipError_t launch_kernel_impl(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                                     std::tuple<P...> &args, std::index_sequence<I...>)
{
    void *ptrs[] = {static_cast<void *>(&std::get<I>(args))...};
    return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, ptrs, lds, stream);
}

// lds: bytes of LDS that a workgroup holds beyond what the kernel declares (see lds_to_limit)
template <typename... P, typename... A>
inline hipError_t launch_kernel_lds(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, A... a)
{
    static_assert(sizeof...(P) == sizeof...(A), "one argument per kernel parameter");
    std::tuple<P...> args{static_cast<P>(a)...};
    return launch_kernel_impl(kernel, grid, block, lds, stream, args, std::index_sequence_for<P...>{});
}

template <typename... P, typename... A>
inline hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t stream, A... a)
{
    return launch_kernel_lds(kernel, grid, block, 0, stream, a...);
}

// LDS to ask for at the launch of a kernel that declares `own` bytes, so that a compute unit (160 KB) holds at most `groups`
// workgroups of it; 0 for no limit.  The kernel does not touch it.  A launch decides by its volume how many workgroups
// share a compute unit, which a bound on registers in the kernel's own code could not.  The middle between what
// `groups` and one more of them would leave each, so that the granularity of LDS allocation does not matter.
inline size_t lds_to_limit(int groups, size_t own)
{
    constexpr size_t kUnitLds = 160 * 1024;
    if (groups <= 0) return 0;
    const size_t each = (kUnitLds / (size_t)groups + kUnitLds / (size_t)(groups + 1)) / 2;
    return each > own ? each - own : 0;
}

// Quantizer: 0 = asymmetric (Eq. 1-2), 1 = symmetric (Eq. 3-4), 2 = FP8 E4M3 (8 bit only),
// 3 = asymmetric with binary16 metadata (one 32-bit word per group, passed where the other
// codecs pass `scales`); the values match kAsym / kSym / kFp8 / kAsymH of the device code.
// Only codec 0 uses the zero-point arrays.
enum { CODEC_ASYM = 0, CODEC_SYM = 1, CODEC_FP8 = 2, CODEC_ASYMH = 3 };

// n_elems = tokens*hidden (a multiple of `group`, which is a power of two in
// [32, 16384]).  All pointers are device pointers.
hipError_t launch_quantize(int bits, int codec, const void *x_f16, int64_t n_elems, int group,
                           void *codes, float *scales, float *zeros, hipStream_t stream);

hipError_t launch_dequantize(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                             int64_t n_elems, int group, void *y_f16, hipStream_t stream);

struct FusedArgs {
    int codec;
    const void *codes_in;
    int64_t codes_stride;
    const float *scales_in;
    const float *zeros_in;
    int64_t meta_stride;
    int n_src;
    int64_t n_elems;
    int group;
    void *codes_out;
    float *scales_out;
    float *zeros_out;
};

// one translation unit per (bits_in, bits_out) pair
hipError_t launch_fused_4_4(const FusedArgs &a, hipStream_t stream);
hipError_t launch_fused_4_8(const FusedArgs &a, hipStream_t stream);
hipError_t launch_fused_8_4(const FusedArgs &a, hipStream_t stream);
hipError_t launch_fused_8_8(const FusedArgs &a, hipStream_t stream);

// fc_wide.hip holds one-group-per-workgroup kernels for coarse groups.  The
// stand-alone quantizer uses them for every group wider than one wavefront (64
// lanes x 128 bits of codes); the fused kernel reduces across the wavefronts of
// its workgroup itself and hands over only groups wider than its 256-lane tile.
inline bool is_wide_group(int bits, int group) { return group * bits / 128 > 64; }
inline bool exceeds_tile(int bits, int group) { return group * bits / 128 > 256; }

hipError_t launch_quantize_wide(int bits, int codec, const void *x_f16, int64_t n_elems, int group,
                                void *codes, float *scales, float *zeros, hipStream_t stream);
hipError_t launch_fused_wide(int bits_in, int bits_out, const FusedArgs &a, hipStream_t stream);

// Hadamard rotation fused into the quantizer / dequantizer (fc_rot.hip), applied to every aligned block of
// rotation_block(hidden) elements, which must be 1024, 2048, 4096 or 8192.
inline int rotation_block(int64_t hidden) { return (int)(hidden & -hidden); }     // largest power of two dividing hidden
hipError_t launch_quantize_rot(int bits, int codec, const void *x_f16, int64_t tokens, int hidden, int group,
                               void *codes, float *scales, float *zeros, hipStream_t stream);
hipError_t launch_dequantize_rot(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                                 int64_t tokens, int hidden, int group, void *y_f16, hipStream_t stream);

// fc_rot_fine.hip: the same for launch-bound volumes.
hipError_t launch_quantize_rot_fine(int bits, int codec, const void *x_f16, int64_t n_elems, int log_b, int group,
                                    void *codes, float *scales, float *zeros, hipStream_t stream);
hipError_t launch_dequantize_rot_fine(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                                      int64_t n_elems, int log_b, int group, void *y_f16, hipStream_t stream);

// the last two steps of the rotated all-reduce in one, from the first step's codes to the result
hipError_t launch_reduce_rot_fine(int codec, int bits_rs, int bits_ag, const void *codes, int64_t codes_stride, const float *scales,
                                  const float *zeros, int64_t meta_stride, int n_src, int64_t n_elems, int log_b, int group, void *y_f16,
                                  hipStream_t stream);

// the whole rotated all-reduce, where that is the fastest form of it
bool allreduce_rot_fine_applies(int log_b, int n_src, int64_t n_elems);
// whether the one-launch form has all sources of a block, or a round of them, in one workgroup
bool allreduce_rot_at_once(int log_b, int n_src, int64_t n_elems);
hipError_t launch_allreduce_rot_fine(int codec, int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems, int log_b, int group,
                                     void *y_f16, hipStream_t stream);

// fc_rot_rows.hip: the same for volumes between those and a full chip, blocks of 1024, 2048 and 4096 (2^log_b); at 4 bit in blocks of
// 1024 only, the quantizer in blocks of 4096 for FP8 only.
hipError_t launch_quantize_rot_rows(int bits, int codec, const void *x_f16, int64_t n_elems, int log_b, int group,
                                    void *codes, float *scales, float *zeros, hipStream_t stream);
hipError_t launch_dequantize_rot_rows(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                                      int64_t n_elems, int log_b, int group, void *y_f16, hipStream_t stream);
// fc_rot_sim.hip: the whole rotated all-reduce in one launch, every group and fan-in.
hipError_t launch_allreduce_rot(int codec, int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t tokens,
                                int hidden, int group, void *y_f16, hipStream_t stream);

// fc_small.hip: the whole all-reduce in one launch, for launch-bound volumes: at most kSmallAllreduceMaxElems elements
// per partial (of seven partials 6/7 of that) and groups of at most 512 elements.
constexpr int64_t kSmallAllreduceMaxElems = (int64_t)1 << 20;
bool allreduce_small_applies(int n_src, int64_t n_elems, int group);
hipError_t launch_allreduce_small(int codec, int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems,
                                  int group, void *y_f16, hipStream_t stream);

// fc_sim.hip (one translation unit per quantizer): the same in one launch for volumes that memory bandwidth bounds
// (the N binary16 partials are read once, the binary16 result is written once, nothing else touches memory);
// groups of at most 1024 elements, every quantizer.  fc_sim_wide.hip: the same for groups of 1024 to 16384.
constexpr int kFusedAllreduceMaxGroup = 1024;         // one wavefront's 64 lanes x 16 elements
constexpr int kFusedAllreduceTileElems = 2048;        // one workgroup
#define FC_DECLARE_SIM(name)                                                                                       \
    hipError_t launch_allreduce_fused_##name(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems, \
                                             int group, void *y_f16, hipStream_t stream);                          \
    hipError_t launch_allreduce_wide_##name(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems, \
                                            int group, void *y_f16, hipStream_t stream);
FC_DECLARE_SIM(asym) FC_DECLARE_SIM(sym) FC_DECLARE_SIM(fp8) FC_DECLARE_SIM(cmeta)
#undef FC_DECLARE_SIM
// Groups of 1024 fit both kernels: a wavefront of fc_sim.hip, or a workgroup of one wavefront of fc_sim_wide.hip, which works out Eq. 1 of all
// sources in one evaluation and has all of them in flight.  That is the shorter chain for small volumes and fewer instructions per
// element for the asymmetric quantizers; with six sources and more of 2 M elements it has too much in flight, and the max|x| of the others costs
// the first kernel less.  us, fc_sim / fc_sim_wide, hidden 8192: INT4 N = 2 64 tokens 3.40 / 3.01, 400 5.61 / 5.29, 1000 10.11 / 10.50,
// 2500 22.7 / 21.4, 8192 65.5 / 62.6; N = 4 8 tokens 3.99 / 3.14, 160 5.33 / 4.90, 400 8.13 / 7.82, 1000 15.9 / 15.7, 2500 36.9 / 35.1, 8192 105.7 /
// 103.0; N = 8 8 tokens 5.75 / 4.19, 160 7.98 / 7.01, 260 9.90 / 9.81, 400 12.1 / 13.2; symmetric INT8 N = 2 400 tokens 4.96 / 5.29, N = 4
// 8 tokens 3.66 / 2.99, 160 4.98 / 4.58, 400 7.63 / 7.72, 8192 103.5 / 103.6; FP8 N = 8 160 tokens 7.57 / 7.11, 400 11.8 / 13.3.  One source has nothing
// to share: symmetric INT8 1 M 2.57 / 2.58, 1.25 M 2.53 / 2.67, FP8 1.5 M 2.72 / 2.86.
inline bool allreduce_wide_applies(int codec, int n_src, int64_t n_elems, int group)
{
    constexpr int64_t k1M = (int64_t)1 << 20;
    if (group != kFusedAllreduceMaxGroup) return group > kFusedAllreduceMaxGroup;
    const bool asym = codec == CODEC_ASYM || codec == CODEC_ASYMH;
    if (n_elems <= (n_src == 1 ? 2 : 3) * k1M / 2) return true;
    return asym && n_src <= 4 && (n_elems <= 4 * k1M || n_elems >= 12 * k1M);
}
inline hipError_t launch_allreduce_fused(int codec, int bits_rs, int bits_ag, const void *x_f16, int n_src,
                                         int64_t n_elems, int group, void *y_f16, hipStream_t stream)
{
    // volumes of up to 2^36 elements: at most 2^25 workgroups of either form
    const bool wide = allreduce_wide_applies(codec, n_src, n_elems, group);
#define FC_SIM_CASE(CODEC, name)                                                                                     \
    case CODEC:                                                                                                      \
        return (wide ? launch_allreduce_wide_##name : launch_allreduce_fused_##name)(bits_rs, bits_ag, x_f16, n_src, \
                                                                                     n_elems, group, y_f16, stream);
    switch (codec) {
        FC_SIM_CASE(CODEC_ASYM, asym) FC_SIM_CASE(CODEC_SYM, sym) FC_SIM_CASE(CODEC_FP8, fp8)
        FC_SIM_CASE(CODEC_ASYMH, cmeta)
    default: return hipErrorInvalidValue;
    }
#undef FC_SIM_CASE
}

inline int log2_int(int v)
{
    int s = 0;
    while ((1 << s) < v) ++s;
    return s;
}

}  // namespace fc
