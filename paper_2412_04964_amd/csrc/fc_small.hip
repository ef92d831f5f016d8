// fc_small.hip -- Algorithm 1 in ONE launch for volumes that launching, not memory, bounds.
//
// The paper's own design is a single fused kernel around its exchanges (Section 3.2.3, "Kernel Design"); on one
// device with identity exchanges the counterpart is a kernel that takes the N binary16 partials and writes the
// binary16 result, with both quantizations happening in registers.  Every rounding of the three-kernel path is
// kept: FinegrainedQuantize of each partial (Eq. 1-2) gives codes q_j, scale s_j and zero-point z_j of the group;
// the sum is acc = fma(q_j - z_j, s_j, acc) in source order from +0; FinegrainedQuantize of acc with the second
// bit-width; Dequantize to binary16.  Codes never leave the lane, and the result is bit-identical to
// fc_quantize x N -> fc_dequant_reduce_requant -> fc_dequantize while a decode-sized all-reduce costs one launch
// instead of three.
//
// Decomposition: a lane owns 8 consecutive elements (one 128-bit access of binary16), a wavefront 512; a group of
// g <= 512 elements is g/8 adjacent lanes, reduced with DPP / cross-lane steps.  A workgroup of NSRC wavefronts
// owns one 512-element tile of the result: wavefront j quantizes that tile of partial j (the expensive, independent
// part: min / max, Eq. 1, Eq. 2) and leaves q - z and the scale in LDS; after one barrier wavefront 0 runs the
// sequential fp32 FMA chain over the sources, requantizes, dequantizes and stores.  For a decode-sized volume a
// wavefront's work is a chain of dependent instructions with nothing to overlap it, so spreading the NSRC
// quantizations over wavefronts is what shortens the launch (N = 8: 7.4 -> about 4 us).
#include "fc_device.hpp"
#include "fc_launch.hpp"

namespace fc {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSmallLaneElems = 8;
constexpr int kSmallWaveElems = 64 * kSmallLaneElems;

// FinegrainedQuantize of the lane's values and the inverse of Eq. 2 without its scale: d = q - z (the signed code, the value
// of the E4M3 byte).  +0 is added to a signed code: the stored integer has no -0.  Asymmetric codes are not formed as integers:
// clamp(t + z) - z is a median of three on t where t and z are integers of few bits (HALF: the values were binary16), and the
// literal fp32 operations otherwise; fc_sim.hip has the reasons.  us under graph replay, codes as integers / so, INT4, group 128,
// hidden 8192: N = 2 64 tokens 2.92 / 2.79, 115 tokens 3.52 / 3.25; N = 4 3.49 / 3.26, 4.30 / 3.96; N = 8 32 tokens 3.52 / 3.33,
// 64 tokens 4.51 / 4.09, 115 tokens 6.69 / 6.05.
template <int CODEC, int BITS, bool HALF>
__device__ __forceinline__ void small_codes(const float (&v)[kSmallLaneElems], int lpg, float &s, float (&d)[kSmallLaneElems])
{
    constexpr int E = kSmallLaneElems;
    float inv;
    if constexpr (is_asym(CODEC)) {
        float mn, mx, zf;
        lane_minmax(v, mn, mx);
        group_minmax<0>(mn, mx, lpg);
        group_params<BITS, CODEC == kAsymH>(mn, mx, s, inv, zf);
        constexpr float qmax = (float)((1 << BITS) - 1);
        const float d_lo = 0.0f - zf, d_hi = qmax - zf;
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const float t = rintf(v[i] * inv);
            d[i] = HALF ? __builtin_amdgcn_fmed3f(t, d_lo, d_hi) : __builtin_amdgcn_fmed3f(t + zf, 0.0f, qmax) - zf;
        }
    } else {
        const float amax = group_max<0>(lane_absmax(v), lpg);
        if constexpr (CODEC == kFp8) {
            group_params_absmax<448>(amax, s, inv);
            u32 word[E / 4];
            pack_lane_fp8<E>(v, inv, word);
#pragma unroll
            for (int k = 0; k < E / 4; ++k) {
                const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)word[k], false);
                const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)word[k], true);
                d[4 * k + 0] = lo.x;
                d[4 * k + 1] = lo.y;
                d[4 * k + 2] = hi.x;
                d[4 * k + 3] = hi.y;
            }
        } else {
            group_params_sym<BITS>(amax, s, inv);
#pragma unroll
            for (int i = 0; i < E; ++i) d[i] = rintf(v[i] * inv) + 0.0f;
        }
    }
}

template <int CODEC, int BITS_RS, int BITS_AG, int NSRC>
__global__ __launch_bounds__(64 * NSRC) void k_allreduce_small(const uint16_t *__restrict__ x, int64_t n_elems, int lpg,
                                                              uint16_t *__restrict__ y)
{
    constexpr int E = kSmallLaneElems;
    // per source: q - z of the tile's 512 elements as fp32 (exact small integers, or the literal fp32 difference
    // for extreme zero-points) and the scale of each lane's group
    __shared__ __attribute__((aligned(16))) float diff[NSRC][64][E];
    __shared__ float scale[NSRC][64];

    const u32 lane = threadIdx.x & 63u, j = threadIdx.x >> 6;            // wavefront j <-> source j
    const int64_t e_tile = (int64_t)blockIdx.x * kSmallWaveElems;
    const int64_t left = (n_elems - e_tile) * 2;                         // bytes from the tile to the end of a partial

    {
        const rsrc_t rx = make_rsrc(x + (int64_t)j * n_elems + e_tile, left);
        const u32x4 raw = __builtin_amdgcn_raw_buffer_load_b128(rx, lane * 16, 0, kStreamLoadPolicy);
        float v[E];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const h2 p = as_h2(raw[k]);
            v[2 * k] = (float)p.x;
            v[2 * k + 1] = (float)p.y;
        }
        float s, d[E];
        small_codes<CODEC, BITS_RS, true>(v, lpg, s, d);
        if constexpr (NSRC > 1) {
            f32x4 *mine = reinterpret_cast<f32x4 *>(&diff[j][lane][0]);
            mine[0] = f32x4{d[0], d[1], d[2], d[3]};
            mine[1] = f32x4{d[4], d[5], d[6], d[7]};
            scale[j][lane] = s;
            __syncthreads();
            if (j != 0) return;
        }

        float acc[E];
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = 0.0f;
        if constexpr (NSRC > 1) {
#pragma unroll
            for (int k = 0; k < NSRC; ++k) {                                               // ReduceSum, source order
                const f32x4 lo = *reinterpret_cast<const f32x4 *>(&diff[k][lane][0]);
                const f32x4 hi = *reinterpret_cast<const f32x4 *>(&diff[k][lane][4]);
                const float sk = scale[k][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[i] = fmaf(lo[i], sk, acc[i]);
                    acc[4 + i] = fmaf(hi[i], sk, acc[4 + i]);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i) acc[i] = fmaf(d[i], s, acc[i]);
        }

        float s2, d2[E];
        small_codes<CODEC, BITS_AG, false>(acc, lpg, s2, d2);
        u32x4 out;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            h2 p;
            p.x = (_Float16)(d2[2 * k] * s2);
            p.y = (_Float16)(d2[2 * k + 1] * s2);
            out[k] = as_u32(p);
        }
        const rsrc_t ry = make_rsrc(y + e_tile, left);
        __builtin_amdgcn_raw_buffer_store_b128(out, ry, lane * 16, 0, kStreamStorePolicy);
    }
}

template <int CODEC, int BITS_RS, int BITS_AG, int NSRC>
static hipError_t launch_small_one(const uint16_t *x, int64_t n_elems, int group, uint16_t *y, hipStream_t stream)
{
    return launch_kernel(k_allreduce_small<CODEC, BITS_RS, BITS_AG, NSRC>,
                         dim3((unsigned)((n_elems + kSmallWaveElems - 1) / kSmallWaveElems)), dim3(64 * NSRC), stream, x,
                         n_elems, group / kSmallLaneElems, y);
}

template <int CODEC, int BITS_RS, int BITS_AG>
static hipError_t launch_small_bits(const uint16_t *x, int n_src, int64_t n_elems, int group, uint16_t *y, hipStream_t stream)
{
    switch (n_src) {
    case 1: return launch_small_one<CODEC, BITS_RS, BITS_AG, 1>(x, n_elems, group, y, stream);
    case 2: return launch_small_one<CODEC, BITS_RS, BITS_AG, 2>(x, n_elems, group, y, stream);
    case 3: return launch_small_one<CODEC, BITS_RS, BITS_AG, 3>(x, n_elems, group, y, stream);
    case 4: return launch_small_one<CODEC, BITS_RS, BITS_AG, 4>(x, n_elems, group, y, stream);
    case 5: return launch_small_one<CODEC, BITS_RS, BITS_AG, 5>(x, n_elems, group, y, stream);
    case 6: return launch_small_one<CODEC, BITS_RS, BITS_AG, 6>(x, n_elems, group, y, stream);
    case 7: return launch_small_one<CODEC, BITS_RS, BITS_AG, 7>(x, n_elems, group, y, stream);
    case 8: return launch_small_one<CODEC, BITS_RS, BITS_AG, 8>(x, n_elems, group, y, stream);
    default: return hipErrorInvalidValue;
    }
}

template <int CODEC>
static hipError_t launch_small_codec(int bits_rs, int bits_ag, const uint16_t *x, int n_src, int64_t n_elems, int group,
                                     uint16_t *y, hipStream_t stream)
{
    if constexpr (CODEC == kFp8) {
        return launch_small_bits<kFp8, 8, 8>(x, n_src, n_elems, group, y, stream);
    } else {
        if (bits_rs == 4)
            return bits_ag == 4 ? launch_small_bits<CODEC, 4, 4>(x, n_src, n_elems, group, y, stream)
                                : launch_small_bits<CODEC, 4, 8>(x, n_src, n_elems, group, y, stream);
        return bits_ag == 4 ? launch_small_bits<CODEC, 8, 4>(x, n_src, n_elems, group, y, stream)
                            : launch_small_bits<CODEC, 8, 8>(x, n_src, n_elems, group, y, stream);
    }
}

// Where the two forms cross (hidden 8192, g = 128, us per launch under graph replay, this one / bulk; asymmetric, symmetric, compact metadata
// INT4, FP8):
//   N = 2   128 tokens (the limit) 2.80 / 3.03, 2.60 / 2.66, 2.81 / 3.04, 2.61 / 2.84; 160 tokens 3.13 / 3.07, 2.89 / 2.73, 3.23 / 3.17, 2.93 / 2.96
//   N = 4   128 tokens 3.46 / 3.94, 3.07 / 3.38, 3.48 / 3.90, 3.14 / 3.84; 160 tokens 4.13 / 4.35, 3.85 / 3.80, 4.18 / 4.35, 3.85 / 4.29; 192 tokens 4.73 /
//           4.45, 4.40 / 3.92, 4.76 / 4.51, 4.41 / 4.36
//   N = 6   128 tokens 4.88 / 5.29, 4.53 / 4.49, 4.98 / 5.33, 4.55 / 5.19; 160 tokens 5.76 / 5.55, 5.39 / 4.74, 5.85 / 5.58, 5.39 / 5.38
//   N = 7   96 tokens 4.84 / 5.60, 4.53 / 4.74, 4.88 / 5.53, 4.54 / 5.51; 115 tokens 5.73 / 5.80, 5.34 / 4.97, 5.77 / 5.79, 5.36 / 5.71; 128 tokens 6.13 /
//           5.85, 5.76 / 4.99, 6.16 / 5.86, 5.77 / 5.77: seven wavefronts leave one of a workgroup's SIMDs half empty
//   N = 8   64 tokens 3.40 / 4.96, 3.09 / 4.57, 3.54 / 4.77, 3.12 / 4.86; 128 tokens 5.92 / 6.33, 5.55 / 5.45, 6.00 / 6.32, 5.59 / 6.23; 160 tokens
//           6.74 / 6.48, 6.29 / 5.62, 6.88 / 6.45, 6.34 / 6.41
// They cross between 128 and 192 tokens, 128 and 160 for most: at most 2^20 elements per partial for all of them, 1 to 2 % too many for six and eight
// sources of symmetric codes, and of seven partials at most 6 * 2^20 altogether.
bool allreduce_small_applies(int n_src, int64_t n_elems, int group)
{
    return group <= kSmallWaveElems && n_elems <= kSmallAllreduceMaxElems &&
           (n_src != 7 || n_src * n_elems <= 6 * kSmallAllreduceMaxElems);
}

hipError_t launch_allreduce_small(int codec, int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems,
                                  int group, void *y_f16, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    switch (codec) {
    case CODEC_ASYM: return launch_small_codec<kAsym>(bits_rs, bits_ag, x, n_src, n_elems, group, y, stream);
    case CODEC_SYM: return launch_small_codec<kSym>(bits_rs, bits_ag, x, n_src, n_elems, group, y, stream);
    case CODEC_FP8: return launch_small_codec<kFp8>(bits_rs, bits_ag, x, n_src, n_elems, group, y, stream);
    case CODEC_ASYMH: return launch_small_codec<kAsymH>(bits_rs, bits_ag, x, n_src, n_elems, group, y, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fc
