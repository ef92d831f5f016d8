// fc_fused_small.hpp -- Dequantize x NSRC, ReduceSum, FinegrainedQuantize for volumes that launching bounds.
//
// A decode-sized volume (N = 8 partials of 8 x 8192 codes) is 64 wavefront tiles of the bulk kernel: a quarter of
// the compute units get one wavefront each, and that wavefront walks through 16 or 32 elements per lane and
// source as one chain of dependent instructions.  Here a lane owns ONE 32-bit word of codes per source (4
// elements at 8 bit, 8 at 4 bit), so the same volume spreads over four times as many single-wavefront workgroups
// and every chain is a quarter as long; all loads (codes, scales, zero-points of every source) are issued before
// the first use.  The arithmetic is the literal form of the contract in include/fc.h, the same that the bulk
// kernel's general path evaluates: d = (float)q - z, acc = fma(d, s, acc) in source order from +0, then Eq. 1-2 (the
// quantizer's own equations) on the sums.  Groups span g / E adjacent lanes (at most the wavefront: g <= 256 at 8 bit, 512 at 4 bit).
#pragma once

#include "fc_device.hpp"
#include "fc_launch.hpp"

namespace fc {

constexpr int fused_small_lane_elems(int bits_in) { return 32 / bits_in; }
constexpr int fused_small_wave_elems(int bits_in) { return 64 * fused_small_lane_elems(bits_in); }
// Up to this many wavefronts (eight per compute unit of the part) the asymmetric quantizer's launch is latency-bound and this kernel wins
// (decode shape, N = 8 at 8 bit: 2.63 -> 2.14 us per launch under graph replay; the two forms cross between 2048
// and 4096 wavefronts).  The other quantizers the same way (N = 8, hidden 8192, g = 128, bulk -> this one): symmetric 4 bit
// 3.46 -> 2.29 us at 8 tokens, 3.79 -> 2.77 at 64, 3.95 -> 3.35 at 128 (the limit); compact metadata 3.64 -> 2.36, 3.88 -> 2.90,
// 4.06 -> 3.71; FP8 2.67 -> 2.18 at 8 tokens, 3.16 -> 2.99 at 64 (its limit).
constexpr int kFusedSmallMaxWaves = 2048;

// The other quantizers' bulk kernels read less metadata.  With few sources, and groups of 32 lanes and more to reduce here, they are
// the faster ones from fewer wavefronts on (hidden 2048, g = 256, 2048 wavefronts, bulk / this one: 8 -> 8 bit, N = 2, symmetric
// 2.37 / 2.57 us, FP8 2.32 / 2.58, compact metadata 2.50 / 2.72; N = 4 2.72 / 2.83 with compact metadata; N = 2 at 4 bit
// 2.53 / 2.72, 2.74 / 2.89; but g = 32, 8 -> 8 bit, N = 3, compact metadata 2.74 / 2.59).  The forms cross at about 448
// wavefronts per source at 8 bit and twice that at 4 bit.  A volume of at most three workgroups of the bulk kernel starts sooner
// there than as 24 of these (8 bit, one row of 4096, N = 1, FP8 2.24 / 2.40 us, symmetric 2.23 / 2.39; N = 3 2.27 / 2.37; compact
// metadata N = 2 2.37 / 2.34; 6144: FP8 N = 3 2.28 / 2.39; 7168: 2.41 / 2.41); from four sources on its chain is too long.
constexpr int kFusedSmallWavesPerSource = 448;
constexpr int kFusedSmallMinWaves = 24;

inline bool fused_small_applies(int codec, int bits_in, int n_src, int64_t n_elems, int group)
{
    const int64_t waves = (n_elems + fused_small_wave_elems(bits_in) - 1) / fused_small_wave_elems(bits_in);
    if (group > fused_small_wave_elems(bits_in) || waves > kFusedSmallMaxWaves) return false;
    if (codec != CODEC_ASYM && bits_in == 8 && n_src <= (codec == CODEC_ASYMH ? 1 : 3) && waves <= kFusedSmallMinWaves) return false;
    if (codec == CODEC_ASYM || group < 32 * fused_small_lane_elems(bits_in)) return true;
    return waves <= n_src * kFusedSmallWavesPerSource * (8 / bits_in);
}

// Codes of the lane as numbers, before the scale: q - z, the signed code, or the value of the E4M3 byte
template <int CODEC, int BITS>
__device__ __forceinline__ void small_decode(u32 w, float z, float (&d)[32 / BITS])
{
    constexpr int E = 32 / BITS;
    if constexpr (CODEC == kFp8) {
        const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false), hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
        d[0] = lo.x;
        d[1] = lo.y;
        d[2] = hi.x;
        d[3] = hi.y;
    } else {
#pragma unroll
        for (int i = 0; i < E; ++i) {
            if constexpr (CODEC == kSym)
                d[i] = (float)((int)(w << (32 - BITS * (i + 1))) >> (32 - BITS));
            else
                d[i] = (float)((w >> (BITS * i)) & ((1u << BITS) - 1u)) - z;
        }
    }
}

template <int CODEC, int BITS_IN, int BITS_OUT, int NSRC>
__global__ __launch_bounds__(64) void k_fused_small(
    const uint8_t *__restrict__ codes_in, int64_t codes_stride,
    const float *__restrict__ scales_in, const float *__restrict__ zeros_in, int64_t meta_stride,
    int64_t n_elems, int group_shift, int lpg,
    uint8_t *__restrict__ codes_out, float *__restrict__ scales_out, float *__restrict__ zeros_out)
{
    constexpr int E = fused_small_lane_elems(BITS_IN);
    constexpr int kOutBytes = E * BITS_OUT / 8;                 // 2, 4 or 8 code bytes per lane
    const u32 lane = threadIdx.x;
    const int64_t e_wave = (int64_t)blockIdx.x * (64 * E);
    const int64_t e_lane = e_wave + (int64_t)lane * E;
    const bool live = e_lane < n_elems;                         // (the volume is a multiple of the group, hence of E)
    const int64_t n_groups = n_elems >> group_shift;
    const int64_t g_mine = e_lane >> group_shift;
    const int64_t gi = g_mine < n_groups ? g_mine : n_groups - 1;   // lanes beyond the end stay inside the arrays

    u32 w[NSRC];
    float s[NSRC], z[NSRC];
#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        const rsrc_t rc = make_rsrc(codes_in + (int64_t)j * codes_stride + e_wave * BITS_IN / 8,
                                    (n_elems - e_wave) * BITS_IN / 8);
        w[j] = __builtin_amdgcn_raw_buffer_load_b32(rc, lane * 4, 0, 0);
        s[j] = scales_in[(int64_t)j * meta_stride + gi];
        z[j] = CODEC == kAsym ? zeros_in[(int64_t)j * meta_stride + gi] : 0.0f;
    }

    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        if constexpr (CODEC == kAsymH) unpack_meta(__builtin_bit_cast(u32, s[j]), s[j], z[j]);
        float d[E];
        small_decode<CODEC, BITS_IN>(w[j], z[j], d);
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = fmaf(d[i], s[j], acc[i]);
    }

    float s2, inv, zf = 0.0f;
    uint64_t packed = 0;
    if constexpr (is_asym(CODEC)) {
        float mn, mx;
        lane_minmax(acc, mn, mx);
        group_minmax<0>(mn, mx, lpg);
        group_params<BITS_OUT, CODEC == kAsymH>(mn, mx, s2, inv, zf);
#pragma unroll
        for (int i = 0; i < E; ++i) packed |= (uint64_t)encode<BITS_OUT>(acc[i], inv, zf) << (BITS_OUT * i);
    } else {
        const float amax = group_max<0>(lane_absmax(acc), lpg);
        if constexpr (CODEC == kFp8) {
            group_params_absmax<448>(amax, s2, inv);
            u32 word[1];
            pack_lane_fp8<4>(acc, inv, word);
            packed = word[0];
        } else {
            group_params_sym<BITS_OUT>(amax, s2, inv);          // neither clamp of Eq. 4 can act (see pack_lane_sym)
#pragma unroll
            for (int i = 0; i < E; ++i)
                packed |= (uint64_t)((u32)(int)rintf(acc[i] * inv) & ((1u << BITS_OUT) - 1u)) << (BITS_OUT * i);
        }
    }

    const rsrc_t ro = make_rsrc(codes_out + e_wave * BITS_OUT / 8, (n_elems - e_wave) * BITS_OUT / 8);
    if constexpr (kOutBytes == 8)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{(u32)packed, (u32)(packed >> 32)}, ro, lane * 8, 0, 0);
    else if constexpr (kOutBytes == 4)
        __builtin_amdgcn_raw_buffer_store_b32((u32)packed, ro, lane * 4, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)packed, ro, lane * 2, 0, 0);
    if (live && (lane & (u32)(lpg - 1)) == 0) {
        scales_out[g_mine] = CODEC == kAsymH ? __builtin_bit_cast(float, pack_meta(s2, zf)) : s2;
        if constexpr (CODEC == kAsym) zeros_out[g_mine] = zf;
    }
}

}  // namespace fc
