// fc_fused_small.hpp -- Dequantize x NSRC, ReduceSum, FinegrainedQuantize for volumes that launching bounds.
//
// A decode-sized volume (N = 8 partials of 8 x 8192 codes) is 64 wavefront tiles of the bulk kernel: a quarter of
// the compute units get one wavefront each, and that wavefront walks through 16 or 32 elements per lane and
// source as one chain of dependent instructions.  Here a lane owns ONE 32-bit word of codes per source (4
// elements at 8 bit, 8 at 4 bit), so the same volume spreads over four times as many single-wavefront workgroups
// and every chain is a quarter as long; all loads (codes, scales, zero-points of every source) are issued before
// the first use.  The arithmetic is the literal form of the contract in include/fc.h, the same that the bulk
// kernel's general path evaluates: d = (float)q - z, acc = fma(d, s, acc) in source order from +0, then Eq. 1-2 (the
// quantizer's own equations) on the sums.  Groups span g / E adjacent lanes; those that are wider than a wavefront (256 elements at 8 bit, 512
// at 4 bit) have a workgroup each.
#pragma once

#include "fc_device.hpp"
#include "fc_launch.hpp"

namespace fc {

constexpr int fused_small_lane_elems(int bits_in) { return 32 / bits_in; }
constexpr int fused_small_wave_elems(int bits_in) { return 64 * fused_small_lane_elems(bits_in); }
// Up to how many wavefronts of this kernel, in units of 1024 (one per SIMD of the part), a launch takes it rather than the
// bulk kernel, whose wavefronts hold four times the elements: past that many the bulk kernel's shorter instruction stream per element
// counts more than the number of wavefronts.  Eight bits out of four take longer to form than to move, and the bulk kernel has fewer
// instructions for them: with few sources it crosses earlier there (us, bulk / this one: asymmetric, N = 2, group 32  1.75 M
// elements 2.89 / 2.86, 2.5 M 2.88 / 3.24, group 256  2 M 3.08 / 3.08, 2.5 M 3.05 / 3.32;  N = 4, group 128  2 M 3.38 / 3.21, 2.5 M 3.42 / 3.54;  compact metadata,
// group 256, N = 2  1.5 M 2.98 / 2.74, 2 M 2.93 / 3.14;  N = 4  1.5 M 3.41 / 3.00, 2 M 3.42 / 3.53).  Time against the bulk kernel's, per cent, replayed graphs, hidden 4096, at 1024 x 1.5, 2, 3, 4, 5,
// 6, 7 wavefronts (us at 3072: asymmetric 4 -> 4 bit, N = 4, group 128 3.88 / 3.07):
//   16 lanes to a group (128 elements at 4 bit, 64 at 8 bit)
//     asymmetric 4 -> 4 bit  N = 2 -23 -19 -19 -13 -12 -8 -3; N = 4 -26 -23 -21 -16 -14 -11 -5; N = 8 -25 -21 -29 -19 -12 -6 -2
//       4 -> 8 bit  N = 1 -13 -10 -3 +4 +4 +11; N = 2 -20 -13 -15 -8 -5 -2 +5; N = 4 -25 -21 -18 -12 -8 -2 +7; N = 8 -24 -19 -26 -13 -11 -2 +3
//     symmetric 4 -> 4 bit  N = 2 -13 -10 -20 -16 -14 -11 -6; N = 8 -28 -24 -31 -24 -19 -12 -6
//     compact metadata 4 -> 4 bit  N = 2 -18 -19 -17 -9 -5 +1 +6; N = 8 -18 -13 -20 -9 -1 +8 +13
//     8 -> 8 bit, asymmetric  N = 2 -17 -17 -20 -17 -19 -16 -14; N = 4 -17 -15 -18 -15 -13 -11 -8; N = 8 -21 -17 -21 -15 -7 +1; symmetric N = 4 -15 -14 -21 -18 -16
//       -15 -12; FP8 N = 1 -2 -1 -5 -6 -5 -3 +1; N = 4 -13 -12 -16 -14 -12 -12 -10; compact metadata N = 4 -13 -11 -16 -11 -10 -4 -1
//   64 lanes (512 and 256 elements), the same order
//     asymmetric 4 -> 4 bit  N = 2 -16 -8 -12 -6 -3 +1 +6; N = 8 -20 -16 -22 -12 -10 -4 +6; 4 -> 8 bit  N = 4 -20 -19 -14 -4 +0 +4 +10
//     symmetric 4 -> 4 bit  N = 4 -19 -16 -24 -18 -13 -11 -6; compact metadata  N = 4 -18 -16 -12 -4 +2 +5 +15
//     8 -> 8 bit, asymmetric  N = 4 -12 -9 -13 -7 -4 -2 -1; N = 8 -14 -10 -13 -8 -3 +7; compact metadata  N = 4 -7 -4 -10 -5 -3 +5 +7; FP8 N = 1 +0 +1 +0 -4 -1 +2
// Workgroups of 256 threads start faster than four of 64 (N = 8 4 -> 4 bit 1.5 M elements 4.29 / 3.64 us, N = 4 1/4 M 2.35 / 2.14, 2 M 3.69 / 3.27), except
// that a wavefront has a compute unit to itself in the smallest launches (N = 8 10 K elements 2.22 / 2.30): 64 threads up to kFusedSmallAlone wavefronts.
// The number is a constant of the kernel: as an argument it costs 0.04 us, read from the launch's description 0.15 (1/4 M 2.70 / 2.53).
constexpr int kFusedSmallAlone = 256;
inline int fused_small_limit(int codec, int bits_in, int bits_out, int n_src, bool wide)
{
    if (n_src == 1) return bits_in == 8 ? 3 : 2;
    if (bits_in == 8) return wide ? 5 : 6;
    const int widens = bits_out == 8 && n_src <= 4 ? 1 : 0;
    return codec == CODEC_SYM ? 6 : (codec == CODEC_ASYMH ? 4 : 5) - widens;
}

// The other quantizers' bulk kernels read less metadata.  With few sources at 8 bit, a volume of at most three workgroups of the bulk kernel starts sooner
// there (one to three sources, 16 to 24 wavefronts: symmetric and FP8 N = 1 and 2 3 to 5 per cent, FP8 N = 3 3, compact metadata N = 1 4); from four sources on
// its chain is too long.
constexpr int kFusedSmallMinWaves = 24;

// Groups of several wavefronts (SPANS below): 8 elements per lane and one barrier, against 16 or 32 per lane in the bulk kernel, and against one
// workgroup that walks through the sources of a group of 8192 at 8 bit.  us by elements (2^20), hidden 8192, bulk / this one:
//   4 -> 4 bit, group 1024: N = 2  1/4: 2.59 / 2.31   1/2: 2.60 / 2.44   1: 2.69 / 2.64, symmetric 2.40 / 2.54;   N = 3  1/2: 2.87 / 2.56   2: 3.66 / 3.49   2.5: 3.87 /
//     4.01;   N = 4  1/64: 2.84 / 2.36   1: 3.26 / 3.07   2: 3.90 / 3.79   3: 4.35 / 4.52;   N = 8  1/4: 3.73 / 2.87   1: 4.01 / 3.55   2: 5.28 / 4.74   3: 5.92 / 6.11;
//     compact metadata N = 4  1/2: 3.01 / 2.71   1.5: 3.83 / 3.84   2: 3.89 / 3.93, 4 -> 8 bit, group 2048, N = 8  1.5: 5.24 / 4.86   2: 5.33 / 5.69
//   group 4096: N = 4  1/2: 3.05 / 2.79   2: 4.08 / 3.80;   N = 8  1: 4.06 / 3.56.   group 8192: N = 4  1/4: 3.19 / 3.19   1: 3.42 / 3.53
//   8 -> 8 bit, group 512: N = 8  1/4: 3.24 / 2.92   1/2: 3.36 / 3.20   1.5: 4.92 / 5.32;   N = 2  1/8: 2.33 / 2.23;   group 1024: N = 8  1/4: 3.21 / 2.99   1/2: 3.32 /
//     3.47;   N = 2, symmetric, group 512  1/16: 2.06 / 2.08, 1024 2.09 / 2.18, 2048 -3 %;   N = 4  1/64: 2.53 / 2.28   1/2: 2.84 / 2.98, FP8 1/4: 2.25 / 2.30;   group 4096: N = 4  1/4: 2.77 / 2.78
//   group 8192: N = 1  2: 3.38 / 3.28   2.5: 3.82 / 3.87;   N = 2  1: 3.68 / 3.18   3.5: 4.89 / 4.67   4: 5.04 / 5.16;   N = 4  1: 4.60 / 3.57   3.5: 6.81 / 6.72   4: 7.12 / 6.99   5: 7.98 /
//     8.64;   N = 8  1: 6.79 / 4.33   3.5: 9.69 / 9.51   5: 11.33 / 12.10;   FP8 N = 4  1: 3.82 / 3.22   3.5: 5.79 / 5.63   4: 6.10 / 6.35;   N = 8  2: 6.29 / 5.80   2.5: 7.30 / 7.55
inline bool fused_spans_applies(int codec, int bits_in, int n_src, int64_t n_elems, int group)
{
    constexpr int64_t k1M = (int64_t)1 << 20;
    if (bits_in == 4) return group <= 4096 && n_elems <= (n_src <= 2 ? k1M * 3 / 4 : codec == CODEC_ASYMH ? k1M * 3 / 2 : 2 * k1M);
    if (group == 8192) return n_elems <= (n_src == 1 || (codec == CODEC_FP8 && n_src >= 6) ? 4 : 7) * (k1M / 2);
    if (codec != CODEC_ASYM && n_src == 2 && group == 1024) return false;
    return group <= 2048 && n_elems <= (n_src >= 5 ? k1M / 4 : n_src >= 2 ? k1M / 8 : 0);
}

inline bool fused_small_applies(int codec, int bits_in, int bits_out, int n_src, int64_t n_elems, int group)
{
    const int64_t waves = (n_elems + fused_small_wave_elems(bits_in) - 1) / fused_small_wave_elems(bits_in);
    if (group > fused_small_wave_elems(bits_in)) return fused_spans_applies(codec, bits_in, n_src, n_elems, group);
    const bool wide = group >= 32 * fused_small_lane_elems(bits_in);
    if (waves > fused_small_limit(codec, bits_in, bits_out, n_src, wide) * 1024) return false;
    if (codec != CODEC_ASYM && bits_in == 8 && n_src <= (codec == CODEC_ASYMH ? 1 : 3) && waves <= kFusedSmallMinWaves) return false;
    return true;
}

// Codes of the lane as numbers, before the scale: q - z, the signed code, or the value of the E4M3 byte
template <int CODEC, int BITS>
__device__ __forceinline__ void small_decode(u32 w, float z, float *d)
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

// min and max of a group that is the whole workgroup, up to 16 wavefronts (identical in all lanes): in the wavefront, then every lane takes
// one wavefront's pair
__device__ __forceinline__ void span_minmax(float &mn, float &mx, u32 n_waves, float (*slot)[2])
{
    group_minmax<0>(mn, mx, 64);
    const u32 lane = threadIdx.x & 63u;
    if (lane == 0) {
        slot[threadIdx.x >> 6][0] = mn;
        slot[threadIdx.x >> 6][1] = mx;
    }
    lds_barrier();
    mn = slot[lane & (n_waves - 1u)][0];
    mx = slot[lane & (n_waves - 1u)][1];
    group_minmax<0>(mn, mx, (int)n_waves);
}

// BT: threads per workgroup, or 0 (SPANS): a group takes several wavefronts, which are the workgroup; 8 elements per lane
template <int CODEC, int BITS_IN, int BITS_OUT, int NSRC, int BT>
__global__ __launch_bounds__(BT == 0 ? 1024 : BT) void k_fused_small(
    const uint8_t *__restrict__ codes_in, int64_t codes_stride,
    const float *__restrict__ scales_in, const float *__restrict__ zeros_in, int64_t meta_stride,
    int64_t n_elems, int group_shift, int lpg,
    uint8_t *__restrict__ codes_out, float *__restrict__ scales_out, float *__restrict__ zeros_out)
{
    constexpr bool SPANS = BT == 0;
    constexpr int E = SPANS ? 8 : fused_small_lane_elems(BITS_IN);
    constexpr int W = E * BITS_IN / 32;                         // code words per lane and source
    constexpr int kOutBytes = E * BITS_OUT / 8;                 // 2, 4 or 8 code bytes per lane
    __shared__ float slot[SPANS ? 16 : 1][2];
    const u32 lane = threadIdx.x;                               // of the workgroup
    const int64_t e_wave = SPANS ? (int64_t)blockIdx.x << group_shift : (int64_t)blockIdx.x * (BT * E);
    const int64_t e_lane = e_wave + (int64_t)lane * E;
    const bool live = e_lane < n_elems;                         // (the volume is a multiple of the group, hence of E)
    const int64_t n_groups = n_elems >> group_shift;
    const int64_t g_mine = e_lane >> group_shift;
    const int64_t gi = g_mine < n_groups ? g_mine : n_groups - 1;   // lanes beyond the end stay inside the arrays

    u32 w[NSRC][W];
    float s[NSRC], z[NSRC];
#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        const rsrc_t rc = make_rsrc(codes_in + (int64_t)j * codes_stride + e_wave * BITS_IN / 8,
                                    (n_elems - e_wave) * BITS_IN / 8);
        if constexpr (W == 1) {
            w[j][0] = __builtin_amdgcn_raw_buffer_load_b32(rc, lane * 4, 0, 0);
        } else {
            const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(rc, lane * 8, 0, 0);
            w[j][0] = a[0];
            w[j][1] = a[1];
        }
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
#pragma unroll
        for (int k = 0; k < W; ++k) small_decode<CODEC, BITS_IN>(w[j][k], z[j], d + k * (E / W));
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = fmaf(d[i], s[j], acc[i]);
    }

    float s2, inv, zf = 0.0f;
    uint64_t packed = 0;
    if constexpr (is_asym(CODEC)) {
        float mn, mx;
        lane_minmax(acc, mn, mx);
        if constexpr (SPANS) span_minmax(mn, mx, (u32)lpg >> 6, slot);
        else group_minmax<0>(mn, mx, lpg);
        group_params<BITS_OUT, CODEC == kAsymH>(mn, mx, s2, inv, zf);
#pragma unroll
        for (int i = 0; i < E; ++i) packed |= (uint64_t)encode<BITS_OUT>(acc[i], inv, zf) << (BITS_OUT * i);
    } else {
        float amax = lane_absmax(acc);
        if constexpr (SPANS) {
            float lo = -amax;
            span_minmax(lo, amax, (u32)lpg >> 6, slot);
        } else {
            amax = group_max<0>(amax, lpg);
        }
        if constexpr (CODEC == kFp8) {
            group_params_absmax<448>(amax, s2, inv);
            u32 word[E / 4];
            pack_lane_fp8<E>(acc, inv, word);
            packed = word[0];
            if constexpr (E == 8) packed |= (uint64_t)word[1] << 32;
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
