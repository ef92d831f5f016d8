// fc_rot.hip -- Hadamard rotation fused into the first quantization and the
// last dequantization of the all-reduce (paper Section 4, rotation-based
// quantization: the transform QuaRot applies before quantizing activations).
//
// Arithmetic contract (must match include/fc.h): the natural-order
// Walsh-Hadamard transform over every aligned block of B = 2^n elements of a
// token's row, B the largest power of two dividing hidden (the whole row when
// hidden is a power of two; five blocks of 1024 for hidden 5120), evaluated in
// fp32 as n butterfly stages with spans 1, 2, 4, ... in that order, each
// butterfly (a, b) -> (a + b, a - b); forward scaling 2^-ceil(n/2), inverse
// scaling 2^-floor(n/2).  A butterfly's result does not depend on which thread
// computes it, so any assignment of butterflies to threads that keeps the stage
// order is bit-identical.
//
// The transform is the one of fc_rot_wave.hpp: 32 values per lane, in registers throughout; a workgroup of two
// wavefronts (blocks of 1024 and 2048, which need no LDS) or of one block (4096, 8192).  Blocks and quantization
// groups never cross block boundaries, so the tensor is handled as a flat sequence of tiles; the last tile of a
// tensor of 1024- or 2048-element blocks may be a partial one (loads beyond the end give zeros, stores are dropped).
//
// What bounds them: vector instructions and which of them issue side by side (rot_priority in fc_rot_wave.hpp) in blocks of 4096 and 8192; in
// the dequantizer of blocks of 1024 more the wait for memory, since a wavefront loads, transforms, stores and ends.  Rotate + quantize /
// dequantize + rotate, group 128, us by card (launches of one kernel in a row, four to seven cards): 8192 x 8192 INT4 35-39 / 37-39, INT8
// 37-40 / 39-41, FP8 42-45 / 41-43; 5461 x 12288 (blocks of 4096) INT4 34-38 / 36-38, INT8 36-40 / 38-40, FP8 40-43 / 40-42; 10922 x 6144 (2048)
// INT4 33-37 / 32-35, INT8 35-40 / 35-38, FP8 38-41 / 38-40; 8192 x 5120 (1024) INT4 21-24 / 20-21, INT8 24-26 / 22-23, FP8 23-29 / 23-24.
// Without priorities over the instructions that issue alone, and with element bits 9 and 10 by swaps: 8192 x 8192 41-46 / 40-42, 43-47 / 41-44,
// 45-48 / 44-46; 8192 x 5120 22-24 (rows in LDS) / 22-23, 24-27 / 24-25, 25-29 / 25-27.  Launch-bound volumes run in fc_rot_fine.hip and
// fc_rot_rows.hip where these are faster.
// Measured and not taken: 32 consecutive elements per lane and a 16 x 16 exchange with other lanes through 5 KB of LDS (40.3 us for blocks
// of 8192, when this form took 43.0, but 23.8 for 1024 and 23.0 / 48 in the dequantizer, whose register needs it does not fit); all stages
// between lanes by permlane swaps; persistent workgroups that load the next tile while they transform the current one (4, 5, 6, 12
// wavefronts per SIMD: 24.3, 23.6, 25.8, 22.5 us against 21.6, quantize 8192 x 5120; dequantize no gain); fewer wavefronts per
// SIMD by holding LDS (3 to 7: no gain).
#include "fc_rot_wave.hpp"
#include "fc_launch.hpp"

namespace fc {

constexpr int kRounds = 2;       // of an exchange between wavefronts: 16 KB instead of 32 for a block of 8192

template <int P>
__device__ __forceinline__ u32 of_piece_bits(u32 v)
{
    return __builtin_bit_cast(u32, of_piece<P>(__builtin_bit_cast(float, v)));
}

// Code words of piece P.  `inv` (with the forward scaling in it) and `fix` belong to piece lane & 3 of the lane.
// The values are in the lane's frame: rounding is symmetric, so the frame goes into the reciprocal.
template <int BITS, int CODEC, int P>
__device__ __forceinline__ void rot_pack(const float (&v)[4][8], const RotLane &L, float inv, u32 fix,
                                         u32 (&word)[4][BITS / 4])
{
    const float inv_p = of_piece<P>(inv) * L.frame;
    if constexpr (CODEC == kFp8)
        pack_lane_fp8<8>(v[P], inv_p, word[P]);
    else if constexpr (CODEC == kSym)
        pack_lane_sym<BITS, 8>(v[P], inv_p, word[P]);
    else
        pack_digits<BITS, 8, false>(v[P], inv_p, 0.0f, of_piece_bits<P>(fix), word[P]);
}

template <int BITS, int P>
__device__ __forceinline__ void rot_pack_literal(const float (&v)[4][8], const RotLane &L, float inv, float zf,
                                                 u32 (&word)[4][BITS / 4])
{
    const float inv_p = of_piece<P>(inv) * L.frame, z_p = of_piece<P>(zf);
#pragma unroll
    for (int w = 0; w < BITS / 4; ++w) {
        u32 acc = 0;
#pragma unroll
        for (int i = 0; i < 32 / BITS; ++i) acc |= encode<BITS>(v[P][32 / BITS * w + i], inv_p, z_p) << (BITS * i);
        word[P][w] = acc;
    }
}

// A wavefront runs at raised priority until its loads are issued: among seven others in the middle of their transforms it would
// take eight times as long to get there.  us, without / with: quantize INT4 8192 x 8192 37.7 / 35.1, x 5120 21.0 / 20.6, INT8 x 4096
// 20.8 / 20.0, x 2048 10.9 / 10.1; dequantize 37.5 / 35.9, 20.9 / 19.3, 20.7 / 19.9, 9.6 / 9.4, FP8 4096 x 8192 21.7 / 21.1; no change up to 1024 x
// 8192, nor for the all-reduce, whose wavefronts live longer.  Raised again for the last instructions: no gain.
__device__ __forceinline__ void rot_to_loads() { __builtin_amdgcn_s_setprio(3); }
__device__ __forceinline__ void rot_loads_issued() { asm volatile("s_setprio 0" ::: "memory"); }

// Whether a quantizer's wavefronts run at raised priority until their loads are issued and over the first stage.  Not in blocks of 1024 with
// integer codes where there are more wavefronts than the chip holds at once (8 per SIMD, 2^24 elements): cards differ there.  us,
// raised / not, on two cards, and the rows in LDS: 8192 x 5120 INT4 20.6, 25.2 / 22.2, 22.6, 24.2, INT8 24.4, 28.1 / 23.5, 23.9, 25.6; 4000 x 5120
// -, 14.5 / -, 13.3, 13.2; below the limit both cards gain (2000 x 5120 7.00 / 7.50).  FP8 in blocks of 1024, without any priority -> so, launches
// of one kernel in a row on two cards: 3481 x 5120 13.6 -> 14.4, 14.1 -> 14.8, but 8192 x 5120 26.3 -> 25.2, 27.7 -> 28.2 and the three steps of
// a rank of four 31.0 -> 28.4, 60.5 -> 56.0.  INT8 in wider blocks gains in a row on every card (8192 x 8192 43-47 -> 37-40; the three
// steps 101 -> 91, with this limit for it too 94); where two builds take turns every few milliseconds it loses on some (8192 x 6144 32.2 ->
// 36.0), which no program does.
template <int LB, bool FP8>
__device__ __forceinline__ bool rot_raised(int64_t n_elems)
{
    return LB != 10 || FP8 || n_elems <= (int64_t)8 * 1024 * 2048;
}

// Rotate block by block and quantize (FinegrainedQuantize of Algorithm 1 on the rotated values).
// n_elems: elements of the whole tensor, a multiple of 2^LB.
template <int BITS, int CODEC, bool SWAPS, int LB>
__global__ __launch_bounds__(64 * rot_group_waves(LB)) void k_quantize_rot(
    const uint16_t *__restrict__ x, int64_t n_elems, int group_shift, uint8_t *__restrict__ codes,
    float *__restrict__ scales, float *__restrict__ zeros)
{
    constexpr bool FP8 = CODEC == kFp8;
    constexpr int kWaves = rot_group_waves(LB);
    constexpr int kTile = 2048 * kWaves;
    __shared__ __attribute__((aligned(16))) uint8_t pieces[rot_exchange_bytes(LB, kRounds)];
    __shared__ float mm[kWaves][kRotSlots][2];

    const bool raised = rot_raised<LB, FP8>(n_elems);
    if (raised) rot_to_loads();
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const RotLane L = rot_lane<FP8, rot_forward_framed(LB, SWAPS)>(lane);
    const int64_t e_tile = (int64_t)blockIdx.x * kTile;
    const int64_t e_begin = rot_begin<LB>(e_tile, wave);
    const int64_t left = n_elems - e_begin;

    u32x4 raw[4];
    const rsrc_t rx = make_rsrc(x + e_begin, left * 2);
    const u32 in_at = rot_lane_offset(kRotLoaded, L) * 2;
#pragma unroll
    for (u32 p = 0; p < 4; ++p) {
        const RotAt at = rot_at<LB>(in_at, kRotLoaded, wave, p, 16);
        raw[p] = __builtin_amdgcn_raw_buffer_load_b128(rx, at.vec, at.scalar, kStreamLoadPolicy);
    }
    if (raised) rot_loads_issued();
    float v[4][8];
    if constexpr (FP8) {
        // Nothing that waits for one of the loads moves up between them (with the other codes rot_first_stages sees to that): in blocks of
        // 8192 the compiler put the first widening, and the wait for its load, ahead of the last load.  us, without / with:
        // 128 tokens 4.62 / 4.22, 256 4.93 / 4.55, 8 3.64 / 3.60.
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i) first_stage(raw[p][i], v[p][2 * i], v[p][2 * i + 1]);
        rot_register_stage<2>(v);
        rot_register_stage<4>(v);
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p)
            rot_first_stages<1>(v[p], [&] {
#pragma unroll
                for (int i = 0; i < 4; ++i) first_stage(raw[p][i], v[p][2 * i], v[p][2 * i + 1]);
            }, raised);
    }
    rot_forward<LB, SWAPS, FP8, kRounds, kRaised>(v, L, pieces, wave);

    // Forward scaling fwd = 2^-ceil(n/2), n = LB.  It is a power of two and nothing here is near the ends of
    // the fp32 range (the transformed values are multiples of 2^-24 below 2^30), so scaling commutes
    // with every rounding: instead of scaling all values, the group's min and max are scaled (which
    // gives the scale, reciprocal and zero-point of the scaled values exactly) and the codes are formed
    // from the unscaled values with the reciprocal times fwd, the same real product and hence the
    // same rounded one.
    constexpr float fwd = 1.0f / (float)(1 << ((LB + 1) / 2));
    float mn, mx = 0.0f, s, inv, zf = 0.0f;
    if constexpr (CODEC == kAsym) {
        rot_group_minmax<LB, SWAPS>(v, L, group_shift, wave, mm, mn, mx);
        group_params<BITS>(mn * fwd, mx * fwd, s, inv, zf);
    } else {
        const float amax = rot_group_absmax<LB, SWAPS>(v, L, group_shift, wave, mm) * fwd;
        if constexpr (FP8) group_params_absmax<448>(amax, s, inv);
        else group_params_sym<BITS>(amax, s, inv);
    }
    inv *= fwd;

    // the packed form needs zero-points below 2048 in magnitude and no rounding past the top code (see pack_lane);
    // both hold for every group of the wavefront or its codes are formed literally
    u32 word[4][BITS / 4];
    bool literal = false;
    u32 fix = 0;
    if constexpr (CODEC == kAsym) {
        constexpr float qmax = (float)((1 << BITS) - 1);
        literal = __builtin_amdgcn_ballot_w64(!(fabsf(zf) < 2048.0f) || rintf(mx * inv) > qmax - zf) != 0;
        fix = digit_fix<BITS>(zf);
    }
    if (literal) {
        if constexpr (CODEC == kAsym) {
            rot_pack_literal<BITS, 0>(v, L, inv, zf, word);
            rot_pack_literal<BITS, 1>(v, L, inv, zf, word);
            rot_pack_literal<BITS, 2>(v, L, inv, zf, word);
            rot_pack_literal<BITS, 3>(v, L, inv, zf, word);
        }
    } else {
        rot_pack<BITS, CODEC, 0>(v, L, inv, fix, word);
        rot_pack<BITS, CODEC, 1>(v, L, inv, fix, word);
        rot_pack<BITS, CODEC, 2>(v, L, inv, fix, word);
        rot_pack<BITS, CODEC, 3>(v, L, inv, fix, word);
    }

    // Blocks of 1024 and 2048: bits 7 and 8 go to lane bits 4 and 5, so that a store covers runs of 512 elements.  The others store runs
    // of 128 (a pass through LDS for runs of a whole block: 38.8 us instead of 38.4, 8192 x 8192 INT4).
    constexpr RotMap done = rot_forward_map(LB, SWAPS);
    constexpr RotMap out = LB >= 12 ? done : RotMap{7, 8, done.l4 == 7 ? done.p0 : done.l4, done.l5 == 8 ? done.p1 : done.l5, done.w0, done.w1};
    if constexpr (out.l4 != done.l4) rot_swap_words<4>(word);
    if constexpr (out.l5 != done.l5) rot_swap_words<5>(word);
    const rsrc_t rc = make_rsrc(codes + e_begin * BITS / 8, left * BITS / 8);
    const u32 lane_at = rot_lane_offset(out, L) * BITS / 8;
#pragma unroll
    for (u32 p = 0; p < 4; ++p) {
        const RotAt at = rot_at<LB>(lane_at, out, wave, p, BITS);
        if constexpr (BITS == 4)
            __builtin_amdgcn_raw_buffer_store_b32(word[p][0], rc, at.vec, at.scalar, kStreamStorePolicy);
        else
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{word[p][0], word[p][1]}, rc, at.vec, at.scalar, kStreamStorePolicy);
    }
    // the lane whose quad begins the group in its piece stores the group's metadata
    const u32 e_quad = rot_quad_offset(done, L, wave);
    if ((e_quad & ((1u << group_shift) - 1u)) == 0) {
        const int64_t g_tile = e_tile >> group_shift, n_groups = n_elems >> group_shift;
        const u32 gi = (e_quad >> group_shift) * 4u;
        store_f32(make_rsrc(scales + g_tile, (n_groups - g_tile) * 4), gi, s);
        if constexpr (CODEC == kAsym) store_f32(make_rsrc(zeros + g_tile, (n_groups - g_tile) * 4), gi, zf);
    }
}

// v[P] = (q - z) * s for the codes of piece P, in the lane's frame (EXACT: frame +1 and the literal operations).
// s and z (z: as pack_zero_const gives it, EXACT: the bits of the number) belong to piece lane & 3 of the lane.
template <int BITS, int CODEC, int P, bool EXACT>
__device__ __forceinline__ void rot_unpack(const u32 (&word)[4][BITS / 4], float s, u32 z, float frame, float (&v)[4][8])
{
    float s_p = of_piece<P>(s);
    if constexpr (CODEC == kFp8) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)word[P][k], false);
            const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)word[P][k], true);
            v[P][4 * k + 0] = lo.x * s_p;
            v[P][4 * k + 1] = lo.y * s_p;
            v[P][4 * k + 2] = hi.x * s_p;
            v[P][4 * k + 3] = hi.y * s_p;
        }
    } else if constexpr (EXACT) {
        const float z_p = CODEC == kSym ? (float)(1 << (BITS - 1)) : __builtin_bit_cast(float, of_piece_bits<P>(z));
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            constexpr int per_word = 32 / BITS;
            const u32 w = CODEC == kSym ? to_offset_binary<BITS>(word[P][i / per_word]) : word[P][i / per_word];
            v[P][i] = ((float)((w >> (BITS * (i % per_word))) & ((1u << BITS) - 1u)) - z_p) * s_p;
        }
    } else {
        s_p *= frame;
        const ZeroConst c = CODEC == kSym ? sym_zero_const<BITS>() : unpack_zero_const(of_piece_bits<P>(z));
#pragma unroll
        for (int k = 0; k < BITS / 4; ++k) {
            const u32 w = CODEC == kSym ? to_offset_binary<BITS>(word[P][k]) : word[P][k];
            if constexpr (BITS == 4) {
                h2 d[4];
                nibbles_minus_zero(w, c, d);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[P][i] = fmaf((float)d[i].x, s_p, 0.0f);
                    v[P][4 + i] = fmaf((float)d[i].y, s_p, 0.0f);
                }
            } else {
                h2 d[2];
                bytes_minus_zero(w, c, d);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    v[P][4 * k + i] = fmaf((float)d[i].x, s_p, 0.0f);
                    v[P][4 * k + 2 + i] = fmaf((float)d[i].y, s_p, 0.0f);
                }
            }
        }
    }
}

// ... and its stages 0-2 of the inverse transform
template <int BITS, int CODEC, int P, bool EXACT>
__device__ __forceinline__ void rot_unpack_stages(const u32 (&word)[4][BITS / 4], float s, u32 z, float frame, float (&v)[4][8])
{
    rot_first_stages<0>(v[P], [&] { rot_unpack<BITS, CODEC, P, EXACT>(word, s, z, frame, v); });
}

// Dequantize, rotate back block by block and round to binary16 (last step of Algorithm 1).
//
// Zeros: stages 3-6 lose the sign of a zero in the signed frame.  Where every zero-point of the wavefront is an
// integer in reach of the short form and every scale is a normal positive number, no value of the contract is ever -0
// (q - z = +0 times a positive scale; no product underflows; +0 + +0, a - a and a + -a are +0), so turning every zero
// of the result into +0 restores it.  Otherwise the wavefront evaluates the literal operations in frame +1.  FP8
// always does.  Wavefronts of one block tell each other with the exchange which form they took, so that a zero of
// either sign meets only exact ones.
template <int BITS, int CODEC, int LB>
__global__ __launch_bounds__(64 * rot_group_waves(LB)) void k_dequantize_rot(
    const uint8_t *__restrict__ codes, const float *__restrict__ scales, const float *__restrict__ zeros,
    int64_t n_elems, int group_shift, uint16_t *__restrict__ y)
{
    constexpr bool FP8 = CODEC == kFp8;
    constexpr int kWaves = rot_group_waves(LB);
    constexpr int kTile = 2048 * kWaves;
    __shared__ __attribute__((aligned(16))) uint8_t pieces[rot_exchange_bytes(LB, kRounds)];
    __shared__ u32 exact_wave[kWaves];

    rot_to_loads();
    const u32 tid = threadIdx.x, lane = tid & 63u;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const RotLane L = rot_lane<FP8>(lane);
    const int64_t e_tile = (int64_t)blockIdx.x * kTile;
    const int64_t e_begin = rot_begin<LB>(e_tile, wave);
    const int64_t left = n_elems - e_begin;
    const int64_t g_tile = e_tile >> group_shift, n_groups = n_elems >> group_shift;

    const u32 gi = (rot_quad_offset(kRotLoaded, L, wave) >> group_shift) * 4u;
    const rsrc_t rs = make_rsrc(scales + g_tile, (n_groups - g_tile) * 4);
    const rsrc_t rc = make_rsrc(codes + e_begin * BITS / 8, left * BITS / 8);
    const float s = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, gi, 0, 0));
    float zf = 0.0f;
    if constexpr (CODEC == kAsym) {
        const rsrc_t rz = make_rsrc(zeros + g_tile, (n_groups - g_tile) * 4);
        zf = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rz, gi, 0, 0));
    }
    u32 word[4][BITS / 4];
    const u32 lane_at = rot_lane_offset(kRotNatural, L) * BITS / 8;
#pragma unroll
    for (u32 p = 0; p < 4; ++p) {
        const RotAt at = rot_at<LB>(lane_at, kRotNatural, wave, p, BITS);
        if constexpr (BITS == 4) {
            word[p][0] = __builtin_amdgcn_raw_buffer_load_b32(rc, at.vec, at.scalar, kStreamLoadPolicy);
        } else {
            const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(rc, at.vec, at.scalar, kStreamLoadPolicy);
            word[p][0] = a[0];
            word[p][1] = a[1];
        }
    }
    rot_loads_issued();
    rot_swap_words<4>(word);               // kRotNatural -> kRotLoaded
    rot_swap_words<5>(word);

    float v[4][8];
    bool exact = true;
    if constexpr (!FP8)
        exact = (__builtin_amdgcn_ballot_w64(!(s >= FLT_MIN)) | (CODEC == kAsym ? zero_is_slow_mask(zf) : 0)) != 0;
    if (exact) {
        const u32 z = __builtin_bit_cast(u32, zf);
        rot_unpack_stages<BITS, CODEC, 0, true>(word, s, z, 1.0f, v);
        rot_unpack_stages<BITS, CODEC, 1, true>(word, s, z, 1.0f, v);
        rot_unpack_stages<BITS, CODEC, 2, true>(word, s, z, 1.0f, v);
        rot_unpack_stages<BITS, CODEC, 3, true>(word, s, z, 1.0f, v);
        rot_row_stages<true, true, kRaised, !FP8>(v, L);
    } else if constexpr (!FP8) {
        const u32 z = CODEC == kAsym ? pack_zero_const(zf) : 0;
        rot_unpack_stages<BITS, CODEC, 0, false>(word, s, z, L.frame, v);
        rot_unpack_stages<BITS, CODEC, 1, false>(word, s, z, L.frame, v);
        rot_unpack_stages<BITS, CODEC, 2, false>(word, s, z, L.frame, v);
        rot_unpack_stages<BITS, CODEC, 3, false>(word, s, z, L.frame, v);
        rot_row_stages<false, true, kRaised>(v, L);
    }
    if constexpr (!FP8 && LB >= 12)
        if (lane == 0) exact_wave[wave] = exact;
    rot_inverse_rest<LB, kRounds>(v, L, pieces, wave, [&] {
        if constexpr (!FP8 && LB >= 12) {
            u32 n_exact = 0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) n_exact += (u32)__builtin_amdgcn_readfirstlane((int)exact_wave[w]);
            exact = n_exact != 0;
            if (n_exact != 0 && n_exact != (u32)kWaves) {
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (exact_wave[LB == 13 ? p : p >> 1] == 0)            // the piece's sender took the short form
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[p][i] += 0.0f;
            }
        }
    });

    constexpr float back = 1.0f / (float)(1 << (LB / 2));               // 2^-floor(n/2), n = LB
    const float plus_zero = exact ? -0.0f : 0.0f;                       // t + -0 is t, t + +0 has no negative zero
    const rsrc_t ry = make_rsrc(y + e_begin, left * 2);
    const u32 out_at = rot_lane_offset(rot_inverse_map(LB), L) * 2;
#pragma unroll
    for (u32 p = 0; p < 4; ++p) {
        u32x4 out;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            out[i] = round_pair(fmaf(v[p][2 * i], back, plus_zero), fmaf(v[p][2 * i + 1], back, plus_zero));
        const RotAt at = rot_at<LB>(out_at, rot_inverse_map(LB), wave, p, 16);
        store_b128_at(out, ry, at.vec, at.scalar);
    }
}

// ---------------------------------------------------------------------------
// launchers: block = largest power of two dividing hidden, in {1024, 2048, 4096, 8192};
// group a power of two in [32, block]
// ---------------------------------------------------------------------------
namespace {

template <int LB>
dim3 rot_grid(int64_t n_elems)
{
    constexpr int64_t kTile = 2048 * rot_group_waves(LB);
    return dim3((unsigned)((n_elems + kTile - 1) / kTile));
}

template <int BITS, int CODEC, int LB>
hipError_t quantize_rot_one(const uint16_t *x, int64_t n_elems, int group, uint8_t *c, float *scales,
                            float *zeros, hipStream_t stream)
{
    const dim3 grid = rot_grid<LB>(n_elems), block(64 * rot_group_waves(LB));
    const int sh = log2_int(group);
    if constexpr (LB == 13 && CODEC != kFp8)
        if (!rot_swaps_apply(n_elems))
            return launch_kernel(k_quantize_rot<BITS, CODEC, false, LB>, grid, block, stream, x, n_elems, sh, c, scales, zeros);
    return launch_kernel(k_quantize_rot<BITS, CODEC, true, LB>, grid, block, stream, x, n_elems, sh, c, scales, zeros);
}

template <int BITS, int CODEC>
hipError_t quantize_rot_h(int log_b, const uint16_t *x, int64_t n_elems, int group, uint8_t *c, float *scales,
                          float *zeros, hipStream_t stream)
{
    switch (log_b) {
    case 10: return quantize_rot_one<BITS, CODEC, 10>(x, n_elems, group, c, scales, zeros, stream);
    case 11: return quantize_rot_one<BITS, CODEC, 11>(x, n_elems, group, c, scales, zeros, stream);
    case 12: return quantize_rot_one<BITS, CODEC, 12>(x, n_elems, group, c, scales, zeros, stream);
    case 13: return quantize_rot_one<BITS, CODEC, 13>(x, n_elems, group, c, scales, zeros, stream);
    default: return hipErrorInvalidValue;
    }
}

template <int BITS, int CODEC, int LB>
hipError_t dequantize_rot_one(const uint8_t *c, const float *scales, const float *zeros, int64_t n_elems,
                              int group, uint16_t *y, hipStream_t stream)
{
    return launch_kernel(k_dequantize_rot<BITS, CODEC, LB>, rot_grid<LB>(n_elems), dim3(64 * rot_group_waves(LB)),
                         stream, c, scales, zeros, n_elems, log2_int(group), y);
}

template <int BITS, int CODEC>
hipError_t dequantize_rot_h(int log_b, const uint8_t *c, const float *scales, const float *zeros,
                            int64_t n_elems, int group, uint16_t *y, hipStream_t stream)
{
    switch (log_b) {
    case 10: return dequantize_rot_one<BITS, CODEC, 10>(c, scales, zeros, n_elems, group, y, stream);
    case 11: return dequantize_rot_one<BITS, CODEC, 11>(c, scales, zeros, n_elems, group, y, stream);
    case 12: return dequantize_rot_one<BITS, CODEC, 12>(c, scales, zeros, n_elems, group, y, stream);
    case 13: return dequantize_rot_one<BITS, CODEC, 13>(c, scales, zeros, n_elems, group, y, stream);
    default: return hipErrorInvalidValue;
    }
}

// Whether the form of fc_rot_fine.hip is the fastest one (both headers have all sides' times): the quantizer up to 5 * 2^18 elements in
// blocks of 1024, 2^20 in those of 2048 and 4096, 3 * 2^19 at 4 bit in blocks of 2048; the dequantizer up to 2^20, at 4 bit in blocks
// of 2048 and 4096 up to 2^21.  The row form comes next, then the one here.
bool rot_fine_applies(bool quantize, int bits, int log_b, int64_t n_elems)
{
    constexpr int64_t k1M = (int64_t)1 << 20;
    if (quantize) return log_b <= 12 && n_elems <= (log_b == 10 ? 5 : log_b == 11 && bits == 4 ? 6 : 4) * (k1M / 4);
    return n_elems <= (bits == 4 && (log_b == 11 || log_b == 12) ? 2 : 1) * k1M;
}

// Whether the form of fc_rot_rows.hip is the faster one (its header has both sides' times) where that of fc_rot_fine.hip is not taken.  At 8 bit
// a wavefront here has twice the work of one there, and FP8's stages cost most in a chain that nothing covers, so its limits lie between 2^21
// and 2^22 elements; at 4 bit a wavefront has 2048 elements in both forms.  Just past the third wavefront per SIMD, 5 to 6 * 2^20 elements,
// the row form wins once more in two cases (rows / registers, 5.5 M: 4-bit dequantizer, blocks of 1024 4.90 / 5.12; FP8 quantizer, 2048
// 6.19 / 6.50; 6.5 M 5.44 / 5.22, 6.91 / 6.88).
bool rot_rows_apply(bool quantize, int codec, int bits, int log_b, int64_t n_elems)
{
    // up to so many times 2^19 elements, blocks of 1024, 2048, 4096: 4 bit, 8 bit, FP8
    static constexpr unsigned char kQuantize[3][3] = {{4, 0, 0}, {4, 4, 0}, {6, 8, 8}}, kDequantize[3][3] = {{4, 0, 0}, {4, 4, 6}, {5, 6, 8}};
    constexpr int64_t k1M = (int64_t)1 << 20;
    const bool fp8 = codec == CODEC_FP8;
    if (log_b > 12) return false;
    if (n_elems <= (quantize ? kQuantize : kDequantize)[fp8 ? 2 : bits == 8][log_b - 10] * (k1M / 2)) return true;
    return (quantize ? fp8 && log_b == 11 : bits == 4 && log_b == 10) && n_elems > 5 * k1M && n_elems <= 6 * k1M;
}

}  // namespace

hipError_t launch_quantize_rot(int bits, int codec, const void *x_f16, int64_t tokens, int hidden, int group,
                               void *codes, float *scales, float *zeros, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint8_t *c = static_cast<uint8_t *>(codes);
    const int lb = log2_int(rotation_block(hidden));
    const int64_t n = tokens * hidden;
    if (rot_fine_applies(true, bits, lb, n))
        return launch_quantize_rot_fine(bits, codec, x_f16, n, lb, group, codes, scales, zeros, stream);
    if (rot_rows_apply(true, codec, bits, lb, n))
        return launch_quantize_rot_rows(bits, codec, x_f16, n, lb, group, codes, scales, zeros, stream);
    if (codec == CODEC_FP8)
        return bits == 8 ? quantize_rot_h<8, kFp8>(lb, x, n, group, c, scales, nullptr, stream)
                         : hipErrorInvalidValue;
    if (bits == 4)
        return codec == CODEC_ASYM ? quantize_rot_h<4, kAsym>(lb, x, n, group, c, scales, zeros, stream)
                                   : quantize_rot_h<4, kSym>(lb, x, n, group, c, scales, nullptr, stream);
    return codec == CODEC_ASYM ? quantize_rot_h<8, kAsym>(lb, x, n, group, c, scales, zeros, stream)
                               : quantize_rot_h<8, kSym>(lb, x, n, group, c, scales, nullptr, stream);
}

hipError_t launch_dequantize_rot(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                                 int64_t tokens, int hidden, int group, void *y_f16, hipStream_t stream)
{
    const uint8_t *c = static_cast<const uint8_t *>(codes);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    const int lb = log2_int(rotation_block(hidden));
    const int64_t n = tokens * hidden;
    if (rot_fine_applies(false, bits, lb, n))
        return launch_dequantize_rot_fine(bits, codec, codes, scales, zeros, n, lb, group, y_f16, stream);
    if (rot_rows_apply(false, codec, bits, lb, n))
        return launch_dequantize_rot_rows(bits, codec, codes, scales, zeros, n, lb, group, y_f16, stream);
    if (codec == CODEC_FP8)
        return bits == 8 ? dequantize_rot_h<8, kFp8>(lb, c, scales, nullptr, n, group, y, stream)
                         : hipErrorInvalidValue;
    if (bits == 4)
        return codec == CODEC_ASYM ? dequantize_rot_h<4, kAsym>(lb, c, scales, zeros, n, group, y, stream)
                                   : dequantize_rot_h<4, kSym>(lb, c, scales, nullptr, n, group, y, stream);
    return codec == CODEC_ASYM ? dequantize_rot_h<8, kAsym>(lb, c, scales, zeros, n, group, y, stream)
                               : dequantize_rot_h<8, kSym>(lb, c, scales, nullptr, n, group, y, stream);
}

}  // namespace fc
