// fc_rot_fine.hip -- the rotated quantizer and dequantizer for launch-bound volumes: 8 elements per lane.
//
// The same arithmetic as fc_rot.hip (butterflies in the order of the spans, so bit-identical), split finer: a wavefront there
// works through 2048 elements as one chain of dependent instructions, here through 512.  A lane holds 8 consecutive elements (bits 0-2 in
// registers, 3-8 in the lanes), a workgroup one block; the bits of the wavefronts go through LDS, two at a time.
//
// What bounds it: latency, of the launch (1.6 us), of one load, of the chain of some 250 instructions and of one barrier or two; past one
// wavefront per SIMD (2^19 elements) the instructions themselves, of which there are more per element than in the other forms.  us per launch
// under graph replay, group 128, the other forms (fc_rot.hip, fc_rot_rows.hip) / this one (rot_fine_applies says where it is taken):
//   quantize, INT4, blocks of 1024: 10 K elements 3.07 / 2.34; 1/2 M 3.25 / 2.74; 1 M 3.09 / 2.60; 1.25 M 3.20 / 3.01; 1.5 M 3.32 / 3.38, group 1024 3.54 / 3.87
//     2048: 3.02 / 2.46; 1 M 3.11 / 2.77; 1.5 M 3.53 / 3.23; 2 M 3.58 / 3.70.   4096: 3.21 / 2.76; 1 M 3.34 / 2.96; 1.25 M 3.74 / 3.75; 2 M 3.67 / 3.79
//     8192, group 64: 3.43 / 3.61; 1 M 4.27 / 4.35.   One group per block of 4096, symmetric: 3.29 / 2.95
//   INT8, blocks of 1024: 2.79 / 2.36; 1 M 3.05 / 2.61; 1.5 M 3.21 / 3.40.   2048: 1 M 3.07 / 2.90; 1.25 M 3.15 / 3.17; 2 M 3.47 / 3.71.   FP8, 1024: 2.77 / 2.33; 2048: 1 M 2.88 /
//     2.63; 2 M 3.36 / 3.53.   8192: one group per block 1 M 4.03 / 4.35; 2 M 4.17 / 4.64, groups of up to 128  -2 to +3 %
//   dequantize, INT4, blocks of 1024: 2.77 / 2.20; 1/2 M 2.89 / 2.49; 1 M 3.09 / 2.82; 1.5 M 3.27 / 3.50.   2048: 3.04 / 2.22; 1 M 3.11 / 2.92; 2 M 3.97 /
//     3.72; 2.5 M 3.85 / 4.20.   4096: 3.09 / 2.45; 1 M 3.46 / 2.97; 2 M 4.26 / 3.90.   8192, group 64: 3.39 / 3.16; 1 M 3.75 / 3.72; 2 M 4.09 / 4.19
//   INT8, blocks of 1024: 2.51 / 2.19; 1 M 3.07 / 2.95; 2 M 3.75 / 3.77.   FP8, 4096: 2.66 / 2.43; 1 M 3.25 / 3.18; 2 M 3.97 / 4.08
// The frames of fc_rot.hip save an instruction per value and stage between lanes: equal up to 1 M elements, 2 M 3.83 for 3.92.
#include "fc_rot_wave.hpp"
#include "fc_fused_small.hpp"
#include "fc_launch.hpp"

namespace fc {

constexpr int fine_waves(int lb) { return 1 << (lb - 9); }
// an exchange holds 32 bytes of every lane; blocks of 4096 and 8192 take two in turn
constexpr int fine_exchanges(int lb) { return lb > 11 ? 2 : 1; }

// Stages 7 and 8: lanes 16 and 32 apart.  After the swap of a value with itself a holds what the lower lanes have, b the upper ones'
template <int LANE_BIT>
__device__ __forceinline__ void fine_swap_stage(float (&v)[8], float s)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        u32 a = __builtin_bit_cast(u32, v[i]), b = a;
        swap_lane_bit<LANE_BIT>(a, b);
        v[i] = fmaf(__builtin_bit_cast(float, b), s, __builtin_bit_cast(float, a));
    }
}

__device__ __forceinline__ void fine_put(const float (&v)[8], uint8_t *at)
{
    *reinterpret_cast<u32x4 *>(at) = u32x4{__builtin_bit_cast(u32, v[0]), __builtin_bit_cast(u32, v[1]), __builtin_bit_cast(u32, v[2]),
                                           __builtin_bit_cast(u32, v[3])};
    *reinterpret_cast<u32x4 *>(at + 1024) = u32x4{__builtin_bit_cast(u32, v[4]), __builtin_bit_cast(u32, v[5]), __builtin_bit_cast(u32, v[6]),
                                                  __builtin_bit_cast(u32, v[7])};
}
__device__ __forceinline__ void fine_get(const uint8_t *at, float (&v)[8])
{
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(at + k * 1024);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32 w = a[i];            // (a bit_cast applied to the vector element itself reads element 0)
            v[4 * k + i] = __builtin_bit_cast(float, w);
        }
    }
}

// Stages of wavefront bits B0 and (NB = 2) B0 + 1: every wavefront forms its own results from the values of two or four
template <int B0, int NB>
__device__ __forceinline__ void fine_wave_stages(float (&v)[8], uint8_t *lds, u32 wave, u32 lane)
{
    const float s0 = (wave >> B0) & 1u ? -1.0f : 1.0f;
    fine_put(v, lds + wave * 2048 + lane * 16);
    lds_barrier();
    float a[8];
    fine_get(lds + (wave ^ (1u << B0)) * 2048 + lane * 16, a);
    if constexpr (NB == 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = fmaf(v[i], s0, a[i]);
    } else {
        const float s1 = (wave >> (B0 + 1)) & 1u ? -1.0f : 1.0f;
        float b[8], c[8];
        fine_get(lds + (wave ^ (2u << B0)) * 2048 + lane * 16, b);
        fine_get(lds + (wave ^ (3u << B0)) * 2048 + lane * 16, c);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = fmaf(fmaf(v[i], s0, a[i]), s1, fmaf(b[i], s0, c[i]));
    }
}

// Stages S0 ... LB-1 of the transform of the block.  Every stage multiplies by +1 or -1 and adds, so zeros have the contract's signs
// (the frames of fc_rot.hip would need its literal form besides)
template <int LB, int S0>
__device__ __forceinline__ void fine_transform(float (&v)[8], const RotLane &L, uint8_t *lds, u32 wave)
{
    if constexpr (S0 == 0) rot_register_stage<1>(v);
    rot_register_stage<2>(v);
    rot_register_stage<4>(v);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(v[i], L.s[0], dpp_read<kDppQuadXor1>(v[i]));
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(v[i], L.s[1], dpp_read<kDppQuadXor2>(v[i]));
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(v[i], L.s[2], dpp_read<kDppRowHalfMirror>(v[i]));
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(v[i], L.s[3], dpp_read<kDppRowRor8>(v[i]));
    fine_swap_stage<4>(v, L.s[4]);
    fine_swap_stage<5>(v, L.lane & 32u ? -1.0f : 1.0f);
    if constexpr (LB == 10) fine_wave_stages<0, 1>(v, lds, wave, L.lane);
    else fine_wave_stages<0, 2>(v, lds, wave, L.lane);
    if constexpr (LB == 12) fine_wave_stages<2, 1>(v, lds + fine_waves(LB) * 2048, wave, L.lane);
    if constexpr (LB == 13) fine_wave_stages<2, 2>(v, lds + fine_waves(LB) * 2048, wave, L.lane);
}

// Rotate a block and quantize it.  lpg: lanes per group
template <int BITS, int CODEC, int LB>
__global__ __launch_bounds__(64 * fine_waves(LB)) void k_quantize_rot_fine(
    const uint16_t *__restrict__ x, int lpg, int group_shift, uint8_t *__restrict__ codes, float *__restrict__ scales,
    float *__restrict__ zeros)
{
    constexpr bool FP8 = CODEC == kFp8;
    __shared__ __attribute__((aligned(16))) uint8_t lds[fine_exchanges(LB) * fine_waves(LB) * 2048];
    __shared__ float slot[fine_waves(LB)][2];
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const int64_t e0 = (int64_t)blockIdx.x << LB;
    const RotLane L = rot_lane<true>(lane);
    const u32 at = wave * 64 + L.pos;                                  // of the lane's 8 elements
    const u32x4 raw = *reinterpret_cast<const u32x4 *>(x + e0 + at * 8);
    float v[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) first_stage(raw[i], v[2 * i], v[2 * i + 1]);
    fine_transform<LB, 1>(v, L, lds, wave);

    // the forward scaling goes into the group's min and max and its reciprocal (see k_quantize_rot)
    constexpr float fwd = 1.0f / (float)(1 << ((LB + 1) / 2));
    float mn, mx, s, inv, zf = 0.0f;
    lane_minmax(v, mn, mx);
    group_minmax<0>(mn, mx, lpg);
    if (lpg > 64) cross_wave_minmax(mn, mx, slot, wave, lane, (u32)lpg >> 6);

    u32 word[BITS / 4];
    const float mn_s = mn * fwd, mx_s = mx * fwd;
    if constexpr (FP8) {
        group_params_absmax<448>(fmaxf(fabsf(mn_s), fabsf(mx_s)), s, inv);
        pack_lane_fp8<8>(v, inv * fwd, word);
    } else if constexpr (CODEC == kSym) {
        group_params_sym<BITS>(fmaxf(fabsf(mn_s), fabsf(mx_s)), s, inv);
        pack_lane_sym<BITS, 8>(v, inv * fwd, word);
    } else {
        group_params<BITS>(mn_s, mx_s, s, inv, zf);
        pack_lane<BITS, 8>(v, inv * fwd, zf, mx, word);
    }
    uint8_t *to = codes + (e0 + at * 8) * BITS / 8;
    if constexpr (BITS == 4) *reinterpret_cast<u32 *>(to) = word[0];
    else *reinterpret_cast<u32x2 *>(to) = u32x2{word[0], word[1]};
    if ((tid & (u32)(lpg - 1)) == 0) {
        const int64_t gi = (e0 + tid * 8) >> group_shift;
        scales[gi] = s;
        if constexpr (CODEC == kAsym) zeros[gi] = zf;
    }
}

// Dequantize a block and rotate it back
template <int BITS, int CODEC, int LB>
__global__ __launch_bounds__(64 * fine_waves(LB)) void k_dequantize_rot_fine(
    const uint8_t *__restrict__ codes, const float *__restrict__ scales, const float *__restrict__ zeros, int group_shift,
    uint16_t *__restrict__ y)
{
    constexpr int W = BITS / 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[fine_exchanges(LB) * fine_waves(LB) * 2048];
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const int64_t e0 = (int64_t)blockIdx.x << LB;
    const RotLane L = rot_lane<true>(lane);
    const u32 at = wave * 64 + L.pos;
    const int64_t gi = (e0 + tid * 8) >> group_shift;
    const float s = scales[gi];
    u32 w[W];
    const uint8_t *from = codes + (e0 + at * 8) * BITS / 8;
    if constexpr (BITS == 4) w[0] = *reinterpret_cast<const u32 *>(from);
    else {
        const u32x2 a = *reinterpret_cast<const u32x2 *>(from);
        w[0] = a[0];
        w[1] = a[1];
    }
    float v[8];
    if constexpr (CODEC == kFp8) {
        decode_fp8(w, v);
    } else if constexpr (CODEC == kSym) {
#pragma unroll
        for (int i = 0; i < W; ++i) w[i] = to_offset_binary<BITS>(w[i]);
        codes_minus_zero_fast<BITS>(w, sym_zero_const<BITS>(), v);
    } else {
        codes_minus_zero_general<BITS>(w, zeros[gi], v);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] *= s;
    fine_transform<LB, 0>(v, L, lds, wave);

    constexpr float back = 1.0f / (float)(1 << (LB / 2));              // 2^-floor(n/2), n = LB
    u32x4 out;
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = round_pair(v[2 * i] * back, v[2 * i + 1] * back);
    *reinterpret_cast<u32x4 *>(y + e0 + at * 8) = out;
}

// The values' codes before the scale, literally, and the scale of their group: minimum and maximum times f, Eq. 1-2 (3-4, E4M3), q - z.  All wavefronts of the
// workgroup call it, each block with slots of its own
template <int CODEC>
__device__ __forceinline__ void fine_codes(float (&v)[8], float f, int lpg, float (*slot)[2], u32 wave, u32 lane, float qmax, float rcp, float &s)
{
    float mn, mx, inv, zf = 0.0f;
    lane_minmax(v, mn, mx);
    group_minmax<0>(mn, mx, lpg);
    if (lpg > 64) cross_wave_minmax(mn, mx, slot, wave, lane, (u32)lpg >> 6);
    mn *= f;
    mx *= f;
    if constexpr (CODEC == kAsym) group_params_levels<false>(mn, mx, qmax, rcp, s, inv, zf);
    else group_params_absmax_levels(fmaxf(fabsf(mn), fabsf(mx)), qmax, rcp, s, inv);
    inv *= f;
    if constexpr (CODEC == kFp8) {
        u32 word[2];
        pack_lane_fp8<8>(v, inv, word);
        decode_fp8(word, v);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float t = rintf(v[i] * inv);
            v[i] = CODEC == kAsym ? __builtin_amdgcn_fmed3f(t + zf, 0.0f, qmax) - zf : t + 0.0f;   // a stored code has no -0
        }
    }
}

// scaled, rotated back and rounded
template <int LB>
__device__ __forceinline__ u32x4 fine_back(float (&v)[8], float s, const RotLane &L, uint8_t *lds, u32 wave)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] *= s;
    fine_transform<LB, 0>(v, L, lds, wave);
    constexpr float back = 1.0f / (float)(1 << (LB / 2));              // 2^-floor(n/2), n = LB
    u32x4 out;
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = round_pair(v[2 * i] * back, v[2 * i + 1] * back);
    return out;
}

// The last two steps of the rotated all-reduce on one block: dequantize the sources' codes, sum, quantize, dequantize, rotate back.
// One launch and one way through memory less than fc_dequant_reduce_requant and fc_dequantize_rot, term by term the same: all-reduces in steps
// became 1.1 to 1.9 us shorter by it.  All loads of all sources come first.  qmax and
// rcp: highest code of the second quantization and its reciprocal
template <int BITS, int CODEC, int LB>
__global__ __launch_bounds__(64 * fine_waves(LB)) void k_reduce_rot_fine(
    const uint8_t *__restrict__ codes, int64_t codes_stride, const float *__restrict__ scales, const float *__restrict__ zeros,
    int64_t meta_stride, int n_src, int lpg, int group_shift, float qmax, float rcp, uint16_t *__restrict__ y)
{
    constexpr int W = BITS / 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[fine_exchanges(LB) * fine_waves(LB) * 2048];
    __shared__ float slot[fine_waves(LB)][2];
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const int64_t e0 = (int64_t)blockIdx.x << LB;
    const RotLane L = rot_lane<true>(lane);
    const u32 at = wave * 64 + L.pos;
    const int64_t gi = (e0 + tid * 8) >> group_shift;
    const uint8_t *from = codes + (e0 + at * 8) * BITS / 8;

    u32 w[8][W];
    float s[8], z[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < n_src) {
            if constexpr (BITS == 4) {
                w[j][0] = *reinterpret_cast<const u32 *>(from + j * codes_stride);
            } else {
                const u32x2 a = *reinterpret_cast<const u32x2 *>(from + j * codes_stride);
                w[j][0] = a[0];
                w[j][1] = a[1];
            }
            s[j] = scales[j * meta_stride + gi];
            if constexpr (CODEC == kAsym) z[j] = zeros[j * meta_stride + gi];
            else z[j] = 0.0f;
        }
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < n_src) {
            float d[8];
#pragma unroll
            for (int k = 0; k < W; ++k) small_decode<CODEC, BITS>(w[j][k], z[j], d + k * (8 / W));
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fmaf(d[i], s[j], v[i]);
        }

    float s2;
    fine_codes<CODEC>(v, 1.0f, lpg, slot, wave, lane, qmax, rcp, s2);
    *reinterpret_cast<u32x4 *>(y + e0 + at * 8) = fine_back<LB>(v, s2, L, lds, wave);
}

// The whole rotated all-reduce of a block in one workgroup, 8 elements per lane: a part of the workgroup per source (see SPREAD in
// fc_rot_sim.hip), n_src <= 16 / fine_waves(LB).  LDS: two areas of 2 KB per wavefront, for the exchanges and (the second one) the handing over
template <int CODEC, int LB>
__global__ __launch_bounds__(1024) void k_allreduce_rot_fine(const uint16_t *__restrict__ x, int64_t n_elems, int n_src, int lpg, float q_rs,
                                                            float rcp_rs, float q_ag, float rcp_ag, uint16_t *__restrict__ y)
{
    constexpr int kWaves = fine_waves(LB);
    constexpr u32 kArea = kWaves * 2048;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ float slots[16][2], scale[16][64];
    const u32 lane = threadIdx.x & 63u;
    const u32 wave_all = (u32)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const u32 wave = wave_all % (u32)kWaves, part = wave_all / (u32)kWaves;
    uint8_t *mine = lds + part * (2 * kArea);
    float (*slot)[2] = slots + part * kWaves;
    const RotLane L = rot_lane<true>(lane);
    const int64_t e = ((int64_t)blockIdx.x << LB) + (wave * 64 + L.pos) * 8;
    constexpr float fwd = 1.0f / (float)(1 << ((LB + 1) / 2));          // 2^-ceil(n/2), n = LB

    const u32x4 raw = *reinterpret_cast<const u32x4 *>(x + (int64_t)part * n_elems + e);
    float v[8], s;
#pragma unroll
    for (int i = 0; i < 4; ++i) first_stage(raw[i], v[2 * i], v[2 * i + 1]);
    fine_transform<LB, 1>(v, L, mine, wave);
    fine_codes<CODEC>(v, fwd, lpg, slot, wave, lane, q_rs, rcp_rs, s);
    if constexpr (LB == 12) lds_barrier();                             // every wavefront has taken the second exchange
    if (part != 0) {
        fine_put(v, mine + kArea + wave * 2048 + lane * 16);
        scale[wave_all][lane] = s;
    }
    lds_barrier();
    if (part != 0) return;                                             // a barrier waits for the wavefronts that are left
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = fmaf(v[i], s, 0.0f);
    for (int k = 1; k < n_src; ++k) {                                  // ReduceSum, source order
        fine_get(lds + k * (2 * kArea) + kArea + wave * 2048 + lane * 16, v);
        s = scale[k * kWaves + wave][lane];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = fmaf(v[i], s, acc[i]);
    }
    fine_codes<CODEC>(acc, 1.0f, lpg, slot, wave, lane, q_ag, rcp_ag, s);
    *reinterpret_cast<u32x4 *>(y + e) = fine_back<LB>(acc, s, L, mine, wave);
}

namespace {

template <int BITS, int CODEC, int LB>
hipError_t quantize_one(const uint16_t *x, int64_t n_elems, int group, uint8_t *c, float *scales, float *zeros, hipStream_t stream)
{
    return launch_kernel(k_quantize_rot_fine<BITS, CODEC, LB>, dim3((unsigned)(n_elems >> LB)), dim3(64 * fine_waves(LB)), stream, x,
                         group / 8, log2_int(group), c, scales, zeros);
}

template <int BITS, int CODEC, int LB>
hipError_t dequantize_one(const uint8_t *c, const float *scales, const float *zeros, int64_t n_elems, int group, uint16_t *y,
                          hipStream_t stream)
{
    return launch_kernel(k_dequantize_rot_fine<BITS, CODEC, LB>, dim3((unsigned)(n_elems >> LB)), dim3(64 * fine_waves(LB)), stream, c,
                         scales, zeros, log2_int(group), y);
}

template <int BITS, int CODEC>
hipError_t quantize_block(int log_b, const uint16_t *x, int64_t n_elems, int group, uint8_t *c, float *scales, float *zeros,
                          hipStream_t stream)
{
    switch (log_b) {
    case 10: return quantize_one<BITS, CODEC, 10>(x, n_elems, group, c, scales, zeros, stream);
    case 11: return quantize_one<BITS, CODEC, 11>(x, n_elems, group, c, scales, zeros, stream);
    case 12: return quantize_one<BITS, CODEC, 12>(x, n_elems, group, c, scales, zeros, stream);
    default: return hipErrorInvalidValue;  // 8192: the form of fc_rot.hip at every volume
    }
}

template <int BITS, int CODEC>
hipError_t dequantize_block(int log_b, const uint8_t *c, const float *scales, const float *zeros, int64_t n_elems, int group,
                            uint16_t *y, hipStream_t stream)
{
    switch (log_b) {
    case 10: return dequantize_one<BITS, CODEC, 10>(c, scales, zeros, n_elems, group, y, stream);
    case 11: return dequantize_one<BITS, CODEC, 11>(c, scales, zeros, n_elems, group, y, stream);
    case 12: return dequantize_one<BITS, CODEC, 12>(c, scales, zeros, n_elems, group, y, stream);
    case 13: return dequantize_one<BITS, CODEC, 13>(c, scales, zeros, n_elems, group, y, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_quantize_rot_fine(int bits, int codec, const void *x_f16, int64_t n_elems, int log_b, int group, void *codes,
                                    float *scales, float *zeros, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint8_t *c = static_cast<uint8_t *>(codes);
    if (codec == CODEC_FP8)
        return bits == 8 ? quantize_block<8, kFp8>(log_b, x, n_elems, group, c, scales, nullptr, stream) : hipErrorInvalidValue;
    if (bits == 4)
        return codec == CODEC_ASYM ? quantize_block<4, kAsym>(log_b, x, n_elems, group, c, scales, zeros, stream)
                                   : quantize_block<4, kSym>(log_b, x, n_elems, group, c, scales, nullptr, stream);
    return codec == CODEC_ASYM ? quantize_block<8, kAsym>(log_b, x, n_elems, group, c, scales, zeros, stream)
                               : quantize_block<8, kSym>(log_b, x, n_elems, group, c, scales, nullptr, stream);
}

hipError_t launch_dequantize_rot_fine(int bits, int codec, const void *codes, const float *scales, const float *zeros, int64_t n_elems,
                                      int log_b, int group, void *y_f16, hipStream_t stream)
{
    const uint8_t *c = static_cast<const uint8_t *>(codes);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    if (codec == CODEC_FP8)
        return bits == 8 ? dequantize_block<8, kFp8>(log_b, c, scales, nullptr, n_elems, group, y, stream) : hipErrorInvalidValue;
    if (bits == 4)
        return codec == CODEC_ASYM ? dequantize_block<4, kAsym>(log_b, c, scales, zeros, n_elems, group, y, stream)
                                   : dequantize_block<4, kSym>(log_b, c, scales, nullptr, n_elems, group, y, stream);
    return codec == CODEC_ASYM ? dequantize_block<8, kAsym>(log_b, c, scales, zeros, n_elems, group, y, stream)
                               : dequantize_block<8, kSym>(log_b, c, scales, nullptr, n_elems, group, y, stream);
}

template <int BITS, int CODEC, int LB>
static hipError_t reduce_one(const uint8_t *c, int64_t codes_stride, const float *scales, const float *zeros, int64_t meta_stride, int n_src,
                             int bits_ag, int64_t n_elems, int group, uint16_t *y, hipStream_t stream)
{
    const float q = CODEC == kFp8 ? 448.0f : (float)((1 << (CODEC == kSym ? bits_ag - 1 : bits_ag)) - 1);
    return launch_kernel(k_reduce_rot_fine<BITS, CODEC, LB>, dim3((unsigned)(n_elems >> LB)), dim3(64 * fine_waves(LB)), stream, c,
                         codes_stride, scales, zeros, meta_stride, n_src, group / 8, log2_int(group), q, 1.0f / q, y);
}

hipError_t launch_reduce_rot_fine(int codec, int bits_rs, int bits_ag, const void *codes, int64_t codes_stride, const float *scales,
                                  const float *zeros, int64_t meta_stride, int n_src, int64_t n_elems, int log_b, int group, void *y_f16,
                                  hipStream_t stream)
{
    const uint8_t *c = static_cast<const uint8_t *>(codes);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    const auto by_block = [&](auto width, auto quantizer) {
        constexpr int BITS = decltype(width)::value, CODEC = decltype(quantizer)::value;
        switch (log_b) {
        case 10: return reduce_one<BITS, CODEC, 10>(c, codes_stride, scales, zeros, meta_stride, n_src, bits_ag, n_elems, group, y, stream);
        case 11: return reduce_one<BITS, CODEC, 11>(c, codes_stride, scales, zeros, meta_stride, n_src, bits_ag, n_elems, group, y, stream);
        case 12: return reduce_one<BITS, CODEC, 12>(c, codes_stride, scales, zeros, meta_stride, n_src, bits_ag, n_elems, group, y, stream);
        case 13: return reduce_one<BITS, CODEC, 13>(c, codes_stride, scales, zeros, meta_stride, n_src, bits_ag, n_elems, group, y, stream);
        default: return hipErrorInvalidValue;
        }
    };
    using Four = std::integral_constant<int, 4>;
    using Eight = std::integral_constant<int, 8>;
    using Asym = std::integral_constant<int, kAsym>;
    using Sym = std::integral_constant<int, kSym>;
    switch (codec) {
    case CODEC_ASYM: return bits_rs == 4 ? by_block(Four{}, Asym{}) : by_block(Eight{}, Asym{});
    case CODEC_SYM: return bits_rs == 4 ? by_block(Four{}, Sym{}) : by_block(Eight{}, Sym{});
    case CODEC_FP8: return by_block(Eight{}, std::integral_constant<int, kFp8>{});
    default: return hipErrorInvalidValue;
    }
}

// All sources at once in a workgroup, and at most 2^21 elements of all sources together (four wavefronts per SIMD), 3 * 2^19 in blocks of 1024; a
// single source, which no other hides, up to 5 * 2^18 in blocks of 1024 and 3 * 2^19 in blocks of 2048.  us by elements (2^20) of a partial, the
// form of fc_rot_sim.hip / this one, group 128 unless said: INT4, block 1024, N = 1  1: 4.5 / 4.0   1.25: 5.3 / 4.8   1.38: 5.3 / 5.6   2: 5.3 / 5.8, group 1024  1.25: 5.4 / 5.2
// 1.38: 5.4 / 6.1   2: 5.5 / 6.6;   N = 2  1/8: 4.67 / 3.28   3/4: 5.6 / 4.7   1: 5.7 / 5.7, group 1024  3/4: 5.6 / 5.3   1: 5.7 / 6.4;   group 1024, N = 4  1/4: 5.34 / 4.50   1/2: 5.63 / 5.70;   block 2048,
// N = 1  1/8: 4.45 / 3.33   1.5: 5.7 / 5.1   1.75: 5.7 / 6.0;   N = 2  1/8: 4.94 / 3.77   1: 6.39 / 5.43   1.5: 6.71 / 6.91;   N = 3  1/8: 5.09 / 4.18   3/4: 6.45 / 6.31   1.5: 7.63 /
// 9.59;   block 4096, N = 1  1/8: 5.01 / 4.19   2: 6.83 / 6.74;   N = 2  1/8: 5.78 / 5.29   1: 6.46 / 6.08   2: 8.65 / 8.96;   FP8, N = 2, block 2048  1/8: 5.46 / 3.70   1: 6.59 / 5.33;   block
// 4096  1/8: 6.17 / 5.22;   symmetric INT8, groups of the block, N = 3, block 2048  1/8: 4.79 / 4.85.  Three sources in blocks of 4096 would take two rounds: 1/8: 6.65 / 7.80.
bool allreduce_rot_fine_applies(int log_b, int n_src, int64_t n_elems)
{
    if (log_b > 12 || n_src > 16 / fine_waves(log_b)) return false;
    const int quarters = log_b == 10 ? (n_src == 1 ? 5 : 6) : log_b == 11 && n_src == 1 ? 6 : 8;      // of 2^20 elements
    return n_src * n_elems <= quarters * ((int64_t)1 << 18);
}

template <int CODEC, int LB>
static hipError_t allreduce_one(const uint16_t *x, int n_src, int64_t n_elems, int group, int bits_rs, int bits_ag, uint16_t *y,
                                hipStream_t stream)
{
    const auto top = [](int bits) { return CODEC == kFp8 ? 448.0f : (float)((1 << (CODEC == kSym ? bits - 1 : bits)) - 1); };
    constexpr int kWaves = fine_waves(LB);
    if (n_src > 16 / kWaves) return hipErrorInvalidValue;
    return launch_kernel_lds(k_allreduce_rot_fine<CODEC, LB>, dim3((unsigned)(n_elems >> LB)), dim3(64 * kWaves * n_src),
                             (size_t)(n_src * kWaves * 4096), stream, x, n_elems, n_src, group / 8, top(bits_rs), 1.0f / top(bits_rs),
                             top(bits_ag), 1.0f / top(bits_ag), y);
}

hipError_t launch_allreduce_rot_fine(int codec, int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems, int log_b, int group,
                                     void *y_f16, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    const auto by_block = [&](auto c) {
        constexpr int CODEC = decltype(c)::value;
        switch (log_b) {
        case 10: return allreduce_one<CODEC, 10>(x, n_src, n_elems, group, bits_rs, bits_ag, y, stream);
        case 11: return allreduce_one<CODEC, 11>(x, n_src, n_elems, group, bits_rs, bits_ag, y, stream);
        case 12: return allreduce_one<CODEC, 12>(x, n_src, n_elems, group, bits_rs, bits_ag, y, stream);
        default: return hipErrorInvalidValue;
        }
    };
    switch (codec) {
    case CODEC_ASYM: return by_block(std::integral_constant<int, kAsym>{});
    case CODEC_SYM: return by_block(std::integral_constant<int, kSym>{});
    case CODEC_FP8: return by_block(std::integral_constant<int, kFp8>{});
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fc
