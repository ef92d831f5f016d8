// fc_rot_sim.hip -- Algorithm 1 with the rotation around it, in ONE launch: every partial is read once, rotated,
// quantized and dequantized into the sum; the sum is quantized, dequantized and rotated back; the result is written
// once.  2 N + 2 bytes per element; nothing else goes through HBM.  Bit-identical to fc_quantize_rot x N ->
// fc_dequant_reduce_requant -> fc_dequantize_rot.
//
// What bounds it: vector instructions, (N + 1) log2 B of them per element for the butterflies alone, and which of them can issue side
// by side (rot_priority in fc_rot_wave.hpp).  4 partials, group 128, us: 8192 x 8192 INT4 161, x 4096 79.5, x 5120 84, FP8 4096 x 8192 97.5.
// 8192 x 8192 INT4 with the first stage at the ordinary priority 166, all of it 181; with element bits 9 and 10 brought into registers by
// permlane swaps as well 187.  Five wavefronts per SIMD instead of four: slower.
// The transform and its layout are those of fc_rot_wave.hpp; the partials are taken in source order in a loop, the next one's loads in
// flight while one is coded.  The sum stays in the frame of the rotated values (see there): rounding is symmetric, so the quantizer
// works on a negated value as on the value, and the inverse transform undoes the frame.
//
// Exactness of the short form of the codes, taken when every zero-point of the wavefront is below 2048 in magnitude
// and no rounding passes the top code: t = rint(x * inv) and z are then small integers, the lower clamp cannot act
// (x >= min), so q - z = t.  Otherwise the codes are formed literally.  Zeros may come out with either sign in the
// short form and across frames; for the integer quantizers the sum and the result of the contract never hold -0 (every
// dequantized value is q - z = +0 times a positive scale, and sums of +0 are +0), and the last multiply-add, which
// adds +0, makes every zero of the result +0.
#include "fc_rot_wave.hpp"
#include "fc_launch.hpp"

namespace fc {

struct RotLevels {           // of one quantization: qmax and 1 / qmax (2^bits - 1, 2^(bits-1) - 1, or 448)
    float q, c;
};

// scale, scaled reciprocal, zero-point and (asymmetric) maximum of the lane's group
template <int CODEC, int LB, bool SWAPS>
__device__ __forceinline__ void rot_params(const float (&v)[4][8], const RotLane &L, int group_shift, u32 wave, float (*slot)[kRotSlots][2],
                                           RotLevels lv, float fwd, float &mx, float &s, float &inv, float &zf)
{
    zf = mx = 0.0f;
    if constexpr (CODEC == kAsym) {
        float mn;
        rot_group_minmax<LB, SWAPS>(v, L, group_shift, wave, slot, mn, mx);
        group_params_levels<false>(mn * fwd, mx * fwd, lv.q, lv.c, s, inv, zf);
    } else {
        group_params_absmax_levels(rot_group_absmax<LB, SWAPS>(v, L, group_shift, wave, slot) * fwd, lv.q, lv.c, s, inv);
    }
    inv *= fwd;
}

// Literal form of d = q - z for piece P
template <int P>
__device__ __forceinline__ void rot_literal_codes(float (&v)[4][8], float frame, float inv, float zf, float qmax)
{
    const float inv_p = of_piece<P>(inv) * frame, z_p = of_piece<P>(zf), z_f = z_p * frame;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float u = rintf(v[P][i] * inv_p) + z_p;
        v[P][i] = fmaf(__builtin_amdgcn_fmed3f(u, 0.0f, qmax), frame, -z_f);           // (code - z) * frame, rounded alike
    }
}

// Short form of d for piece P (or its E4M3 code)
template <bool FP8, int P>
__device__ __forceinline__ void rot_short_codes(float (&v)[4][8], float inv)
{
    const float inv_p = of_piece<P>(inv);
    if constexpr (FP8) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int w = __builtin_amdgcn_cvt_pk_fp8_f32(v[P][4 * h] * inv_p, v[P][4 * h + 1] * inv_p, 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(v[P][4 * h + 2] * inv_p, v[P][4 * h + 3] * inv_p, w, true);
            const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8(w, false), b = __builtin_amdgcn_cvt_pk_f32_fp8(w, true);
            v[P][4 * h] = a.x;
            v[P][4 * h + 1] = a.y;
            v[P][4 * h + 2] = b.x;
            v[P][4 * h + 3] = b.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[P][i] = rintf(v[P][i] * inv_p);
    }
}

// Every value becomes its dequantized code before the scale, in the lane's frame.  Where the short form does not hold
// the literal differences are formed first; they are integers, so the short form with reciprocal 1 leaves them alone
// (a one-sided branch: two alternatives cost 24 registers more).
template <int CODEC>
__device__ __forceinline__ void rot_codes(float (&v)[4][8], const RotLane &L, float mx, float inv, float zf, RotLevels lv)
{
    if constexpr (CODEC == kAsym) {
        if (__builtin_amdgcn_ballot_w64(!(fabsf(zf) < 2048.0f) || rintf(mx * inv) > lv.q - zf) != 0) {
            rot_literal_codes<0>(v, L.frame, inv, zf, lv.q);
            rot_literal_codes<1>(v, L.frame, inv, zf, lv.q);
            rot_literal_codes<2>(v, L.frame, inv, zf, lv.q);
            rot_literal_codes<3>(v, L.frame, inv, zf, lv.q);
            inv = 1.0f;
        }
    }
    rot_short_codes<CODEC == kFp8, 0>(v, inv);
    rot_short_codes<CODEC == kFp8, 1>(v, inv);
    rot_short_codes<CODEC == kFp8, 2>(v, inv);
    rot_short_codes<CODEC == kFp8, 3>(v, inv);
}

template <int P>
__device__ __forceinline__ void rot_accumulate(const float (&d)[4][8], float s, float (&acc)[4][8])
{
    const float s_p = of_piece<P>(s);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[P][i] = fmaf(d[P][i], s_p, acc[P][i]);
}

template <int P>
__device__ __forceinline__ void rot_scale(float (&d)[4][8], float s)
{
    const float s_p = of_piece<P>(s);
#pragma unroll
    for (int i = 0; i < 8; ++i) d[P][i] *= s_p;
}

// The lane number, for what is derived from it after the first loads: left to itself the compiler derives it all before
// them, 30 instructions and 0.07 us of every launch (not with KEPT: the form for one wavefront per SIMD in blocks of 8192 is 0.03 us
// faster without it).
template <bool KEPT>
__device__ __forceinline__ u32 after_loads(u32 lane)
{
    if constexpr (!KEPT) asm volatile("" : "+v"(lane) : : "memory");
    return lane;
}

// SPREAD: a wavefront's dequantized codes and scales, from the part that has a source to the one that sums.  Runs of 1 KB; the lanes keep their places.
constexpr int kRotHandBytes = 8 * 1024 + 256;
constexpr int rot_part_bytes(int lb) { return rot_block_waves(lb) * (kRotHandBytes + kRotSlots * 8); }
// Sources that a workgroup of SPREAD works on at once: 1024 threads at most, and rot_part_bytes each in 160 KB
__host__ __device__ constexpr int rot_parts(int lb, int n_src)
{
    const int most = lb == 13 ? 4 : 8;
    return n_src < most ? n_src : most;
}
__device__ __forceinline__ void rot_hand_over(const float (&d)[4][8], float s, uint8_t *to, u32 lane)
{
#pragma unroll
    for (int k = 0; k < 8; ++k)
        *reinterpret_cast<u32x4 *>(to + k * 1024 + lane * 16) =
            u32x4{__builtin_bit_cast(u32, d[k / 2][4 * (k & 1)]), __builtin_bit_cast(u32, d[k / 2][4 * (k & 1) + 1]),
                  __builtin_bit_cast(u32, d[k / 2][4 * (k & 1) + 2]), __builtin_bit_cast(u32, d[k / 2][4 * (k & 1) + 3])};
    *reinterpret_cast<float *>(to + 8 * 1024 + lane * 4) = s;
}
__device__ __forceinline__ void rot_take_over(const uint8_t *from, u32 lane, float (&d)[4][8], float &s)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const u32x4 a = *reinterpret_cast<const u32x4 *>(from + k * 1024 + lane * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32 w = a[i];            // (a bit_cast applied to the vector element itself reads element 0)
            d[k / 2][4 * (k & 1) + i] = __builtin_bit_cast(float, w);
        }
    }
    s = *reinterpret_cast<const float *>(from + 8 * 1024 + lane * 4);
}

// ALONE: no wavefront shares its SIMD (launches of at most one workgroup per compute unit), so nothing is raised above another, and blocks
// of 8192 take the layout with the shorter chain (rot_swaps_apply).  us, the other form / this, two partials one after the other, group 128: INT4 one
// token of 8192 7.41 / 7.25, 200 tokens 8.95 / 8.86, sym INT8 7.24 / 7.03, 8.74 / 8.66, FP8 8.40 / 8.32.  Past the limit it loses at once.
// SPREAD: the form for volumes that leave the chip idle.  One source after the other is a chain of 1.1 to 2 us each; here the workgroup
// has several times the wavefronts of a block, each such part works on a source of its own, and the first one sums what the others hand over
// through LDS, in source order as ever, and goes on alone.  For rot_spread_applies.
template <int CODEC, bool ALONE, int LB, bool SPREAD>
__device__ __forceinline__ void allreduce_rot(const uint16_t *__restrict__ x, int64_t n_elems, int n_src, int group_shift, RotLevels rs,
                                              RotLevels ag, uint16_t *__restrict__ y)
{
    constexpr bool FP8 = CODEC == kFp8, SWAPS = FP8 || ALONE;           // see rot_swaps_apply
    constexpr RotOrder kOrder = ALONE ? kFlat : LB >= 12 ? kPinned : kRaised;
    constexpr int kWaves = SPREAD ? rot_block_waves(LB) : rot_group_waves(LB);
    constexpr int kTile = 2048 * kWaves;
    constexpr int kChunk = (512 * 1024) / (kTile * 2);                  // 512 KB of every partial per XCD and run
    extern __shared__ __attribute__((aligned(16))) uint8_t parts[];     // SPREAD: rot_part_bytes for every source of a round
    __shared__ __attribute__((aligned(16))) uint8_t own[SPREAD ? 16 : rot_exchange_bytes(LB, 1)];
    __shared__ float own_mm[SPREAD ? 1 : kWaves][kRotSlots][2];

    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave_all = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const u32 wave = SPREAD ? wave_all % (u32)kWaves : wave_all;        // of the block
    const u32 part = SPREAD ? wave_all / (u32)kWaves : 0u;
    const int n_parts = SPREAD ? rot_parts(LB, n_src) : 1;
    uint8_t *pieces = SPREAD ? parts + part * rot_part_bytes(LB) : own;
    float (*mm)[kRotSlots][2] = SPREAD ? reinterpret_cast<float (*)[kRotSlots][2]>(pieces + kWaves * kRotHandBytes) : own_mm;
    const u32 tile = xcd_tile<kChunk>((u32)((n_elems + kTile - 1) / kTile));
    const int64_t e_tile = (int64_t)tile * kTile;
    const int64_t e_begin = rot_begin<LB>(e_tile, wave);
    const int64_t left = (n_elems - e_begin) * 2;                      // bytes from there to the end of a partial

    u32x4 raw[4];
    const u32 lane_at = rot_lane_offset(kRotLoaded, rot_lane<FP8>(lane)) * 2;
    auto fetch = [&](int j) {
        u32 in_at = lane_at;
        asm volatile("" : "+v"(in_at));                                // the pieces' addresses stay out of the loop's registers
        const rsrc_t rx = make_rsrc(x + (int64_t)j * n_elems + e_begin, left);
#pragma unroll
        for (u32 p = 0; p < 4; ++p) {
            const RotAt at = rot_at<LB>(in_at, kRotLoaded, wave, p, 16);
            raw[p] = __builtin_amdgcn_raw_buffer_load_b128(rx, at.vec, at.scalar, kStreamLoadPolicy);
        }
    };
    constexpr float fwd = 1.0f / (float)(1 << ((LB + 1) / 2));          // 2^-ceil(n/2), n = LB
    constexpr float back = 1.0f / (float)(1 << (LB / 2));               // 2^-floor(n/2)

    fetch((int)part);                                                  // n_parts <= n_src
    const RotLane L = rot_lane<FP8, rot_forward_framed(LB, SWAPS)>(after_loads<ALONE && LB == 13>(lane));
    float acc[4][8];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[p][i] = 0.0f;

    int j = 0;
    do {                                                               // n_src >= 1; a loop that may be skipped has its loads moved behind the test
        float v[4][8];
        // All pieces at once, in any order: 256 tokens of 8192 13.66 us, piece by piece 13.85, four of 30 x 2048 8.93 / 9.15; the same for large
        // volumes, except FP8 in short blocks (4 x 8192 x 5120 104.7 / 102.5).
        if constexpr (FP8 && LB < 12) {
#pragma unroll
            for (int p = 0; p < 4; ++p)
                rot_first_stages<1>(v[p], [&] {
#pragma unroll
                    for (int i = 0; i < 4; ++i) first_stage(raw[p][i], v[p][2 * i], v[p][2 * i + 1]);
                });
        } else {
            if constexpr (!ALONE) __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int i = 0; i < 4; ++i) first_stage(raw[p][i], v[p][2 * i], v[p][2 * i + 1]);
            if constexpr (!ALONE) __builtin_amdgcn_s_setprio(0);
            rot_register_stage<2>(v);
            rot_register_stage<4>(v);
        }
        if ((LB >= 12 || SPREAD) && j > 0) lds_barrier();              // every wavefront has taken the last exchange
        rot_forward<LB, SWAPS, FP8, 1, kOrder>(v, L, pieces, wave);
        float mx, s, inv, zf;
        int shift = group_shift;
        // its comparisons stay scalar and in the loop: hoisted, they come back through vector registers (us, before / so: two partials of one token of 4096 6.59 / 6.44,
        // of 100 x 8192 8.29 / 8.18, eight of 4096 x 6144 105.8 / 103.8, four of 8192 x 8192 1 % at most)
        asm volatile("" : "+s"(shift));
        rot_params<CODEC, LB, SWAPS>(v, L, shift, wave, mm, rs, fwd, mx, s, inv, zf);
        if constexpr (SPREAD) {
            const int next = j + n_parts + (int)part;                  // a part without a source repeats the last one; nothing takes it
            if (j + n_parts < n_src) fetch(next < n_src ? next : n_src - 1);
        } else {
            if (j + 1 < n_src) fetch(j + 1);
        }
        rot_codes<CODEC>(v, L, mx, inv, zf, rs);
        if (!SPREAD || part == 0) {
            rot_accumulate<0>(v, s, acc);
            rot_accumulate<1>(v, s, acc);
            rot_accumulate<2>(v, s, acc);
            rot_accumulate<3>(v, s, acc);
        }
        if constexpr (SPREAD) {
            if (LB >= 12) lds_barrier();                               // every wavefront has taken the exchange
            if (part != 0) rot_hand_over(v, s, pieces + wave * kRotHandBytes, lane);
            lds_barrier();
            if (part == 0)
                for (int k = 1; k < n_parts && j + k < n_src; ++k) {
                    rot_take_over(parts + k * rot_part_bytes(LB) + wave * kRotHandBytes, lane, v, s);
                    rot_accumulate<0>(v, s, acc);
                    rot_accumulate<1>(v, s, acc);
                    rot_accumulate<2>(v, s, acc);
                    rot_accumulate<3>(v, s, acc);
                }
        }
        j += n_parts;
    } while (j < n_src);
    if (SPREAD && part != 0) return;                                   // a barrier waits for the wavefronts that are left

    float mx, s, inv, zf;
    if (LB >= 12) lds_barrier();
    rot_params<CODEC, LB, SWAPS>(acc, L, group_shift, wave, mm, ag, 1.0f, mx, s, inv, zf);
    rot_codes<CODEC>(acc, L, mx, inv, zf, ag);
    rot_scale<0>(acc, s);
    rot_scale<1>(acc, s);
    rot_scale<2>(acc, s);
    rot_scale<3>(acc, s);
    RotLane M = L;                         // nothing derived from it for the rest is held in registers over the loop, of which ALONE has enough
    if constexpr (!ALONE) asm volatile("" : "+v"(M.lane), "+v"(M.pos));
    const float frame = rot_inverse_back<LB, SWAPS, FP8, 1, kOrder>(acc, M, pieces, wave);

    const rsrc_t ry = make_rsrc(y + e_begin, left);
    const float scale = back * frame;
    u32x4 out[4];
#pragma unroll
    for (u32 p = 0; p < 4; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = acc[p][2 * i], b = acc[p][2 * i + 1];
            out[p][i] = FP8 ? round_pair(a * scale, b * scale) : round_pair(fmaf(a, scale, 0.0f), fmaf(b, scale, 0.0f));
        }
    if constexpr (LB == 12 || (LB == 13 && !SWAPS)) {
        // the values' binary16 image goes through LDS, so that every store of a wavefront is one run of 1 KB.  16-byte units;
        // the low four bits of a unit's number are xor-ed with its element bits 9 and on, which vary along a row of lanes
        // and else lie in the same banks (LB = 12: the fourth that varies is 5, unit bit 2).
        auto banks = [](u32 h) -> u32 { return LB == 13 ? h : (h & 3u) | ((h & 4u) << 1); };
        lds_barrier();                                                 // every wavefront has taken the exchange
        const u32 high = M.pos & (LB == 13 ? 15u : 7u);
        const u32 low = (M.lane >> 4) + (LB == 13 ? wave * 4 : ((M.pos >> 1) & 4u) + wave * 8);
        uint8_t *mine = pieces + high * 1024 + ((low ^ banks(high)) * 16);
#pragma unroll
        for (u32 p = 0; p < 4; ++p) *reinterpret_cast<u32x4 *>(mine + p * 256) = out[p];
        lds_barrier();
#pragma unroll
        for (u32 k = 0; k < 4; ++k) {
            const u32 run = k * kWaves + wave;                         // of 64 units
            store_b128_at(*reinterpret_cast<const u32x4 *>(pieces + run * 1024 + ((M.lane ^ banks(run)) * 16)), ry,
                          M.lane * 16 + k * (kWaves * 1024), wave * 1024);
        }
    } else {
        constexpr RotMap done = rot_back_map(LB, SWAPS);
        const u32 out_at = rot_lane_offset(done, M) * 2;
#pragma unroll
        for (u32 p = 0; p < 4; ++p) {
            const RotAt at = rot_at<LB>(out_at, done, wave, p, 16);
            store_b128_at(out[p], ry, at.vec, at.scalar);
        }
    }
}

template <int CODEC, bool ALONE, int LB>
__global__ __launch_bounds__(64 * rot_group_waves(LB)) __attribute__((amdgpu_waves_per_eu(4))) void k_allreduce_rot(
    const uint16_t *__restrict__ x, int64_t n_elems, int n_src, int group_shift, RotLevels rs, RotLevels ag,
    uint16_t *__restrict__ y)
{
    allreduce_rot<CODEC, ALONE, LB, false>(x, n_elems, n_src, group_shift, rs, ag, y);
}

template <int CODEC, int LB>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_allreduce_rot_spread(
    const uint16_t *__restrict__ x, int64_t n_elems, int n_src, int group_shift, RotLevels rs, RotLevels ag,
    uint16_t *__restrict__ y)
{
    allreduce_rot<CODEC, true, LB, true>(x, n_elems, n_src, group_shift, rs, ag, y);
}

namespace {

RotLevels levels(int codec, int bits)
{
    const float q = codec == CODEC_FP8 ? 448.0f : (float)((1 << (codec == CODEC_SYM ? bits - 1 : bits)) - 1);
    return RotLevels{q, 1.0f / q};
}

// Up to 2^21 elements, and no more than one round of workgroups (16 wavefronts of 128 registers per compute unit), where neither the steps of
// rot_steps_apply nor the finer form (allreduce_rot_fine_applies) go first.  us under graph replay by elements (2^20), one source after the other / side by side, group 128:
//   INT4, block 2048: N = 2  1/4: 6.49 / 5.28   1: 6.80 / 6.40   2: 8.74 / 7.78   3: 9.00 / 9.59;   N = 3  1/4: 7.88 / 5.31   1: 8.41 / 6.69
//     2: 10.20 / 8.94   3: 10.47 / 10.89;   N = 5  1.5: 13.53 / 11.64   2 (two rounds): 13.70 / 14.35;   block 1024, group 1024, N = 4
//     1/4: 9.36 / 5.33   1: 9.86 / 7.01   2: 11.17 / 9.36   2.25: 11.20 / 11.32
//   INT4, block 4096: N = 2  1/4: 7.14 / 5.80   1: 7.56 / 6.46   2: 9.24 / 8.62   3: 9.76 / 11.02;   N = 3  1/4: 8.67 / 6.87   2: 10.85 / 10.65
//   INT4, block 8192: N = 2  1/4: 7.63 / 7.05   2: 9.00 / 8.39   2.25: 9.32 / 10.03 (INT8);   N = 3  1/4: 9.81 / 8.53   2: 11.07 / 9.71;   N = 4  1: 12.46 /
//     10.09   2: 13.17 / 10.98;   N = 5, whose second round has one source  1.25: 14.4 / 15.3   2: 14.9 / 15.5;   N = 7  1.5: 19.48 / 15.80;   N = 8  2: 21.82 / 16.91
//   FP8, N = 2: block 2048  1/4: 7.01 / 5.52   2: 9.45 / 8.03;   block 4096  1/4: 7.71 / 6.18   2: 10.58 / 9.43;   block 8192  1/4: 8.35 / 7.57   2: 9.90 / 9.02
//   A single source: 5.03 / 5.09, 5.57 / 5.61.
inline bool rot_spread_applies(int lb, int n_src, int64_t n_elems)
{
    if (n_src < 2 || n_elems > (int64_t)1 << 21 || (lb == 13 && n_src == 5)) return false;
    const int waves = rot_block_waves(lb), at_once = 256 * (16 / (waves * rot_parts(lb, n_src)));
    return n_elems <= (int64_t)at_once * waves * 2048;
}

template <int CODEC, int LB>
hipError_t launch_spread(const uint16_t *x, int n_src, int64_t n_elems, int group, RotLevels rs, RotLevels ag, uint16_t *y,
                         hipStream_t stream)
{
    constexpr int kWaves = rot_block_waves(LB), kTile = 2048 * kWaves;
    const int parts = rot_parts(LB, n_src);
    return launch_kernel_lds(k_allreduce_rot_spread<CODEC, LB>, dim3((unsigned)((n_elems + kTile - 1) / kTile)),
                             dim3(64 * kWaves * parts), (size_t)rot_part_bytes(LB) * parts, stream, x, n_elems, n_src,
                             log2_int(group), rs, ag, y);
}

template <int CODEC, int LB>
hipError_t launch_one(const uint16_t *x, int n_src, int64_t n_elems, int group, RotLevels rs, RotLevels ag, uint16_t *y,
                      hipStream_t stream)
{
    constexpr int kTile = 2048 * rot_group_waves(LB);
    if (rot_spread_applies(LB, n_src, n_elems)) return launch_spread<CODEC, LB>(x, n_src, n_elems, group, rs, ag, y, stream);
    const dim3 grid((unsigned)((n_elems + kTile - 1) / kTile)), block(64 * rot_group_waves(LB));
    if constexpr (LB == 13)                // see k_allreduce_rot; one and five sources, the others go side by side
        if (n_elems <= 256 * (int64_t)kTile)
            return launch_kernel(k_allreduce_rot<CODEC, true, LB>, grid, block, stream, x, n_elems, n_src, log2_int(group), rs, ag, y);
    return launch_kernel(k_allreduce_rot<CODEC, false, LB>, grid, block, stream, x, n_elems, n_src, log2_int(group), rs, ag, y);
}

template <int CODEC>
hipError_t launch_codec(int log_b, const uint16_t *x, int n_src, int64_t n_elems, int group, RotLevels rs, RotLevels ag,
                        uint16_t *y, hipStream_t stream)
{
    switch (log_b) {
    case 10: return launch_one<CODEC, 10>(x, n_src, n_elems, group, rs, ag, y, stream);
    case 11: return launch_one<CODEC, 11>(x, n_src, n_elems, group, rs, ag, y, stream);
    case 12: return launch_one<CODEC, 12>(x, n_src, n_elems, group, rs, ag, y, stream);
    case 13: return launch_one<CODEC, 13>(x, n_src, n_elems, group, rs, ag, y, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_allreduce_rot(int codec, int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t tokens,
                                int hidden, int group, void *y_f16, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    const int lb = log2_int(rotation_block(hidden));
    const int64_t n = tokens * hidden;
    const RotLevels rs = levels(codec, bits_rs), ag = levels(codec, bits_ag);
    if (allreduce_rot_fine_applies(lb, n_src, n))
        return launch_allreduce_rot_fine(codec, bits_rs, bits_ag, x, n_src, n, lb, group, y, stream);
    switch (codec) {
    case CODEC_ASYM: return launch_codec<kAsym>(lb, x, n_src, n, group, rs, ag, y, stream);
    case CODEC_SYM: return launch_codec<kSym>(lb, x, n_src, n, group, rs, ag, y, stream);
    case CODEC_FP8: return launch_codec<kFp8>(lb, x, n_src, n, group, rs, ag, y, stream);
    default: return hipErrorInvalidValue;
    }
}

bool allreduce_rot_at_once(int log_b, int n_src, int64_t n_elems)
{
    return allreduce_rot_fine_applies(log_b, n_src, n_elems) || rot_spread_applies(log_b, n_src, n_elems);
}

}  // namespace fc
