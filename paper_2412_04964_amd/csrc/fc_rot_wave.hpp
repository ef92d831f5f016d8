// fc_rot_wave.hpp -- the Walsh-Hadamard transform of the rotation kernels, held in registers.
//
// A wavefront owns 2048 elements, 32 per lane: v[p][i], p = 0..3, i = 0..7.  Element bits 0-2 are i.  The other bits lie in the lane's
// place in its row of 16 (a permutation of the lanes inside every 8, below), in lane bits 4 and 5, in the two bits of p and in the
// wavefront number, and move as the stages pass (RotMap): where a stage runs between registers its bit lies in p.  Values are loaded
// and stored in runs of at least 256 bytes, a 16-byte access per lane and piece, with no staging through LDS.  Stages run in the
// order of the bits; costs are SIMD cycles per value, as measured where nothing else limits (v_add_f32, v_sub_f32, v_fmac_f32:
// 2; anything with a DPP operand: 4, and see rot_priority; v_permlane16/32_swap: 8 for two values; ds_swizzle 2 and ds_bpermute 6 LDS
// cycles for the whole compute unit):
//   0-2    between registers: 2.
//   3-6    between lanes of a row of 16, ONE instruction per value: v_fmac_f32 with a DPP operand, y = dpp(y) * sgn + y: 4.
//          DPP offers lane ^ 1, ^ 2, ^ 7 (half-row mirror) and ^ 8 (rotation by 8) but not ^ 4; these four masks are
//          independent, so bits 3-6 are laid over them: pos(lane) = lane ^ (lane & 4 ? 3 : 0) and bit 3..6 flips when
//          the lane is xor-ed with 1, 2, 7, 8.  The accumulating operand cannot be negated, so the lane with the bit
//          set computes (b - a) instead of a - b: it carries the value negated from then on (its "frame" is -1).  A
//          rounded difference negates exactly, later stages between lanes of one frame are unaffected, and the
//          inverse transform, run on values in this frame with the opposite signs, undoes it.  The one thing that
//          is lost is the sign of a zero.
//   7, 8   between pieces: 2.  Values are loaded with these bits in p.
//   blocks of 1024 and 2048 (a wavefront, or half of one):
//   9      in lane bit 4: the partner's value comes through the LDS crossbar (ds_swizzle: no LDS memory), then one
//          v_fmac_f32: 2.
//   10     changes places with bit 8 (v_permlane32_swap, then between pieces): 6.
//   blocks of 4096 and 8192: all values go through LDS once (rot_exchange), where wavefronts exchange pieces and lanes
//          change places: 9, of blocks of 8192 also 10, comes into the row of 16 (DPP: 4), the last two bits into p (2); what
//          took their places, 5 to 8, needs no more stages.  The form `swaps` of blocks of 8192 brings 9 and 10 into p by swaps
//          (6 each) and only 11 and 12 through LDS.
// FP8 codes keep the sign of zero, so that quantizer's lanes compute a - b itself in the stages inside a row (a DPP move and a
// v_fma_f32 in 3 and 4, the crossbar as in stage 9 in 5 and 6 and, blocks of 4096, 9) and every frame is +1.  The crossbar for 5 and 6
// of the other quantizers as well: 2 % faster for blocks of 1024, 3 % slower in the all-reduce.
#pragma once

#include "fc_device.hpp"

namespace fc {

struct RotLane {
    u32 lane, pos;           // pos: place of the lane's 8 elements in the wavefront's 64
    float s[5];              // +1 / -1 by bits 0..4 of pos
    float frame;             // the frame after the DPP stages, the product of their s (1 for FP8)
};

// FRAMED: bits of pos, and lane bits 4 and 5, that hold element bits whose stage was a DPP one
template <bool FP8, u32 FRAMED = 15u>
__device__ __forceinline__ RotLane rot_lane(u32 lane)
{
    RotLane L;
    L.lane = lane;
    L.pos = lane ^ ((lane & 4u) ? 3u : 0u);
#pragma unroll
    for (int b = 0; b < 5; ++b) L.s[b] = (L.pos >> b) & 1u ? -1.0f : 1.0f;
    L.frame = FP8 ? 1.0f : ((__popc(L.pos & FRAMED) & 1) ? -1.0f : 1.0f);
    return L;
}

// Which element bit lies in lane bits 4 and 5, in the two piece bits, in the wavefront number and in bits 0-3 of pos
struct RotMap {
    int l4, l5, p0, p1, w0, w1;
    int r0 = 3, r1 = 4, r2 = 5, r3 = 6;
};
constexpr RotMap kRotLoaded = {9, 10, 7, 8, 11, 12};                 // as values are loaded and the transforms begin
constexpr RotMap kRotNatural = {7, 8, 9, 10, 11, 12};                // as codes are loaded (see rot_words_loaded)
// A block of 8192 has two forms, `swaps` or not (rot_swaps_apply); the other blocks have one.
constexpr RotMap rot_forward_map(int lb, bool swaps)                 // after the forward transform
{
    return lb == 10 ? RotMap{9, 10, 7, 8, 11, 12} : lb == 11 ? RotMap{9, 8, 7, 10, 11, 12}
         : lb == 12 ? RotMap{5, 6, 10, 11, 8, 12, 3, 4, 9, 7}
         : swaps ? RotMap{7, 8, 11, 12, 9, 10} : RotMap{5, 6, 11, 12, 7, 8, 3, 4, 9, 10};
}
constexpr RotMap rot_back_map(int lb, bool swaps)                    // after the inverse transform that follows a forward one
{
    return lb == 12 ? RotMap{3, 4, 7, 8, 6, 12, 9, 10, 11, 5}
         : lb == 13 ? (swaps ? RotMap{11, 10, 9, 12, 7, 8} : RotMap{3, 4, 7, 8, 5, 6, 9, 10, 11, 12})
         : rot_forward_map(lb, swaps);
}
constexpr u32 rot_forward_framed(int lb, bool swaps)                 // see rot_lane
{
    return lb == 12 ? 55u : lb == 13 && !swaps ? 63u : 15u;
}
// element offsets in the workgroup's tile: of the lane (without the bits of pos that `keep` leaves out), and of a piece
__device__ __forceinline__ u32 rot_lane_offset(const RotMap m, const RotLane &L, u32 keep = 15u)
{
    const u32 r = L.pos & keep;
    const u32 row = m.r0 == 3 && m.r2 == 5 ? r * 8u
                  : ((r & 1u) << m.r0) + (((r >> 1) & 1u) << m.r1) + (((r >> 2) & 1u) << m.r2) + ((r >> 3) << m.r3);
    return row + (((L.lane >> 4) & 1u) << m.l4) + ((L.lane >> 5) << m.l5);
}
__device__ __forceinline__ u32 rot_piece_offset(const RotMap m, u32 wave, u32 p)
{
    return ((p & 1u) << m.p0) + ((p >> 1) << m.p1) + ((wave & 1u) << m.w0) + ((wave >> 1) << m.w1);
}
// Where an access to a piece lies.  The range check of a buffer access compares the vector and the immediate offset with the
// size of the resource; what it does where the scalar offset alone passes that size is not documented.  Blocks of 4096
// and 8192 are whole tiles: nothing passes the end, and the piece may go into the scalar offset.  Blocks of 1024 and 2048 lie
// two wavefronts to a tile, of which the last may hold fewer: there a wavefront's resource begins at its own 2048 elements
// (rot_begin; size 0 where these lie past the end), the scalar offset is 0 and the piece goes into the immediate offset.
constexpr bool rot_whole_tiles(int lb) { return lb >= 12; }
template <int LB>
__device__ __forceinline__ int64_t rot_begin(int64_t e_tile, u32 wave)
{
    return rot_whole_tiles(LB) ? e_tile : e_tile + (int64_t)wave * 2048;
}
struct RotAt {
    u32 vec, scalar;         // byte offsets
};
// `lane_at`: rot_lane_offset(m, L) in bytes
template <int LB>
__device__ __forceinline__ RotAt rot_at(u32 lane_at, const RotMap m, u32 wave, u32 p, u32 bits)
{
    if (rot_whole_tiles(LB)) return RotAt{lane_at, rot_piece_offset(m, wave, p) * bits / 8};
    return RotAt{lane_at + rot_piece_offset(m, 0, p) * bits / 8, 0};
}
// Element where the quad of lanes of this lane begins in piece lane & 3.  Scale and zero-point of that piece's 32 elements
// are this lane's to load, or to derive and store.
__device__ __forceinline__ u32 rot_quad_offset(const RotMap m, const RotLane &L, u32 wave)
{
    return rot_lane_offset(m, L, 12u) + rot_piece_offset(m, wave, L.lane & 3u);
}

// Stages of the element bits in bits FIRST ... FIRST + COUNT - 1 of pos, v[0..7] = dpp(v) * s + v each, INV: with -s.  s_nop: two
// wait states between the write of a register and its DPP read; behind the first stage the other seven values lie between.  With an
// s_nop before every stage: all-reduce of two of one token of 8192 7.20 / 7.15 us, of 12 x 2048 6.06 / 5.96; no change where wavefronts share a SIMD.
#define FC_FMAC_DPP8(ctrl, s)                                                                                        \
    "v_fmac_f32_dpp %0, %0, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                           \
    "v_fmac_f32_dpp %1, %1, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                           \
    "v_fmac_f32_dpp %2, %2, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                           \
    "v_fmac_f32_dpp %3, %3, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                           \
    "v_fmac_f32_dpp %4, %4, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                           \
    "v_fmac_f32_dpp %5, %5, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                           \
    "v_fmac_f32_dpp %6, %6, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                           \
    "v_fmac_f32_dpp %7, %7, " s " " ctrl " row_mask:0xf bank_mask:0xf\n\t"
#define FC_BIT0 "quad_perm:[1,0,3,2]"
#define FC_BIT1 "quad_perm:[2,3,0,1]"
#define FC_BIT2 "row_half_mirror"
#define FC_BIT3 "row_ror:8"
#define FC_ROW_VALUES                                                                                                \
    "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7])

template <int FIRST, int COUNT, bool INV>
__device__ __forceinline__ void fmac_dpp8(float (&v)[8], const float (&s)[5])
{
    constexpr int kForm = FIRST * 100 + COUNT * 10 + INV;
    static_assert(kForm == 40 || kForm == 41 || kForm == 11 || kForm == 21 || kForm == 120 || kForm == 210 || kForm == 220, "as the transforms need them");
    if constexpr (kForm == 40)
        asm("s_nop 1\n\t" FC_FMAC_DPP8(FC_BIT0, "%8") FC_FMAC_DPP8(FC_BIT1, "%9") FC_FMAC_DPP8(FC_BIT2, "%10") FC_FMAC_DPP8(FC_BIT3, "%11")
            : FC_ROW_VALUES : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]));
    if constexpr (kForm == 41)
        asm("s_nop 1\n\t" FC_FMAC_DPP8(FC_BIT0, "-%8") FC_FMAC_DPP8(FC_BIT1, "-%9") FC_FMAC_DPP8(FC_BIT2, "-%10") FC_FMAC_DPP8(FC_BIT3, "-%11")
            : FC_ROW_VALUES : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]));
    if constexpr (kForm == 11) asm("s_nop 1\n\t" FC_FMAC_DPP8(FC_BIT0, "-%8") : FC_ROW_VALUES : "v"(s[0]));
    if constexpr (kForm == 21) asm("s_nop 1\n\t" FC_FMAC_DPP8(FC_BIT0, "-%8") FC_FMAC_DPP8(FC_BIT1, "-%9") : FC_ROW_VALUES : "v"(s[0]), "v"(s[1]));
    if constexpr (kForm == 120) asm("s_nop 1\n\t" FC_FMAC_DPP8(FC_BIT1, "%8") FC_FMAC_DPP8(FC_BIT2, "%9") : FC_ROW_VALUES : "v"(s[1]), "v"(s[2]));
    if constexpr (kForm == 210) asm("s_nop 1\n\t" FC_FMAC_DPP8(FC_BIT2, "%8") : FC_ROW_VALUES : "v"(s[2]));
    if constexpr (kForm == 220) asm("s_nop 1\n\t" FC_FMAC_DPP8(FC_BIT2, "%8") FC_FMAC_DPP8(FC_BIT3, "%9") : FC_ROW_VALUES : "v"(s[2]), "v"(s[3]));
}
#undef FC_FMAC_DPP8
#undef FC_BIT0
#undef FC_BIT1
#undef FC_BIT2
#undef FC_BIT3
#undef FC_ROW_VALUES

template <int MASK>
__device__ __forceinline__ float crossbar(float v)                      // the value of lane ^ MASK, MASK < 32
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), (MASK << 10) | 0x1F));
}

// the stage of the element bit that flips with lane ^ MASK, with its sign s
template <int MASK>
__device__ __forceinline__ void rot_crossbar_stage(float (&v)[4][8], float s)
{
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) v[p][i] = fmaf(v[p][i], s, crossbar<MASK>(v[p][i]));
}

// Two wavefronts' additions, multiplications, FMAs and logical operations run side by side on a SIMD, 2 cycles each in the mean;
// an instruction with a DPP operand (also SDWA, v_permlane*, packed binary16, v_fma_mix, v_cvt_pk_f16_f32) has it to itself for 4
// cycles, and wavefronts at random places of the transform that issue some keep the others' additions from pairing: a stream of three
// additions to one DPP instruction takes 4.0 cycles per instruction, without DPP 2.1.  Stretches of DPP instructions therefore run at a
// raised wave priority: they go through at their own rate, and the additions of all wavefronts meet afterwards.  us, without /
// with: all-reduce, 4 x 8192 x 8192, INT4, group 128 181 / 166, 4 x 8192 x 5120 96 / 90; quantize 8192 x 8192 INT4 43.3 / 38.6; the
// other way round (additions first) 184 and 43.6.
// kPinned: nothing moves across (the all-reduce in blocks of 8192 is 2 % faster for it, in blocks of 1024 and 2048 1 % slower, the single
// transforms as fast or 2 % slower).  kFlat: no priorities, for a wavefront that has its SIMD to itself (see ALONE in fc_rot_sim.hip).
enum RotOrder { kRaised, kPinned, kFlat };
template <int PRIORITY, RotOrder ORDER>
__device__ __forceinline__ void rot_priority(float (&v)[4][8])
{
    if constexpr (ORDER == kFlat) return;
    if constexpr (ORDER == kPinned) {
#pragma unroll
        for (int p = 0; p < 4; ++p) pin_values(v[p]);
    }
    __builtin_amdgcn_s_setprio(PRIORITY);
    if constexpr (ORDER == kPinned) {
#pragma unroll
        for (int p = 0; p < 4; ++p) pin_values(v[p]);
    }
}

// The stages of the element bits in bits FIRST ... FIRST + COUNT - 1 of pos.  INV: the values come in the frame of the forward transform
// and leave without these bits' share of it.  FP8: no frames; the partner's value is moved, then one v_fma_f32.
template <int FIRST, int COUNT, bool FP8, bool INV>
__device__ __forceinline__ void rot_row_some(float (&v)[4][8], const RotLane &L)
{
    constexpr int kCtrl[4] = {kDppQuadXor1, kDppQuadXor2, kDppRowHalfMirror, kDppRowRor8};
    if constexpr (FP8) {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int i = 0; i < 8; ++i) v[p][i] = fmaf(v[p][i], L.s[FIRST], dpp_read<kCtrl[FIRST]>(v[p][i]));
        if constexpr (COUNT > 1) rot_row_some<FIRST + 1, COUNT - 1, FP8, INV>(v, L);
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) fmac_dpp8<FIRST, COUNT, INV>(v[p], L.s);
    }
}

// stages 3-6.  INV: the values come in the frame of the forward transform and leave in frame +1.  RARE: piece after piece, with few registers
// (left to itself the compiler has so many results of the crossbar in flight that the kernel gets 72 to 80 registers, where 64 let
// eight wavefronts onto a SIMD: dequantize INT8 8192 x 2048 11.0 / 9.5 us).
template <bool FP8, bool INV, RotOrder ORDER, bool RARE = false>
__device__ __forceinline__ void rot_row_stages(float (&v)[4][8], const RotLane &L)
{
    rot_priority<1, ORDER>(v);
    if constexpr (FP8) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[p][i] = fmaf(v[p][i], L.s[0], dpp_read<kDppQuadXor1>(v[p][i]));
#pragma unroll
            for (int i = 0; i < 8; ++i) v[p][i] = fmaf(v[p][i], L.s[1], dpp_read<kDppQuadXor2>(v[p][i]));
        }
        if constexpr (RARE) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
#pragma unroll
                for (int i = 0; i < 8; ++i) v[p][i] = fmaf(v[p][i], L.s[2], crossbar<7>(v[p][i]));
#pragma unroll
                for (int i = 0; i < 8; ++i) v[p][i] = fmaf(v[p][i], L.s[3], crossbar<8>(v[p][i]));
                pin_values(v[p]);
            }
        } else {
            rot_crossbar_stage<7>(v, L.s[2]);
            rot_crossbar_stage<8>(v, L.s[3]);
        }
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            fmac_dpp8<0, 4, INV>(v[p], L.s);
        }
    }
    rot_priority<0, ORDER>(v);
}

// a and b exchange what lane bit LANE_BIT = 1 of a and = 0 of b hold
template <int LANE_BIT>
__device__ __forceinline__ void swap_lane_bit(u32 &a, u32 &b)
{
    static_assert(LANE_BIT == 4 || LANE_BIT == 5, "rows of 16 lanes, halves of 32");
    const u32x2 r = LANE_BIT == 4 ? __builtin_amdgcn_permlane16_swap(a, b, false, false)
                                  : __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// The bits of lane bit 4 and piece bit 0 (lane bit 5 and piece bit 1) change places.  A swap needs wait states behind the
// vector instruction that wrote its operands; the compiler sees to that unless this was written in assembly: then
// settle_pieces comes first.  ALONE: at raised priority (see rot_priority), for FP8, whose transforms swap most: quantize 4096 x 8192
// 24.2 / 23.8 us, 1024 x 8192 8.7 / 8.2, all-reduce of four 4096 x 8192 103.8 / 100.3; with integer codes no gain to 1 % slower.
template <int LANE_BIT, bool ALONE = false, RotOrder ORDER = kPinned>
__device__ __forceinline__ void rot_swap(float (&v)[4][8])
{
    constexpr RotOrder kOrder = ALONE && ORDER != kFlat ? kPinned : kFlat;
    rot_priority<1, kOrder>(v);
    constexpr int P = LANE_BIT == 4 ? 1 : 2;
#pragma unroll
    for (int p = 0; p < 4; ++p)
        if (!(p & P))
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                u32 a = __builtin_bit_cast(u32, v[p][i]), b = __builtin_bit_cast(u32, v[p | P][i]);
                swap_lane_bit<LANE_BIT>(a, b);
                v[p][i] = __builtin_bit_cast(float, a);
                v[p | P][i] = __builtin_bit_cast(float, b);
            }
    rot_priority<0, kOrder>(v);
}

// the same on packed words: W per piece and lane
template <int LANE_BIT, int W>
__device__ __forceinline__ void rot_swap_words(u32 (&word)[4][W])
{
    constexpr int P = LANE_BIT == 4 ? 1 : 2;
#pragma unroll
    for (int p = 0; p < 4; ++p)
        if (!(p & P))
#pragma unroll
            for (int k = 0; k < W; ++k) swap_lane_bit<LANE_BIT>(word[p][k], word[p | P][k]);
}

__device__ __forceinline__ void settle_pieces(float (&v)[4][8])
{
#pragma unroll
    for (int p = 0; p < 4; ++p)
        asm("s_nop 1" : "+v"(v[p][0]), "+v"(v[p][1]), "+v"(v[p][2]), "+v"(v[p][3]), "+v"(v[p][4]), "+v"(v[p][5]),
                        "+v"(v[p][6]), "+v"(v[p][7]));
}

// First stage (span 1) on a pair of binary16 inputs held in one word: (lo + hi, lo - hi) in fp32.  Widening a
// binary16 number is exact, so a mixed-precision multiply-add lo * 1 +- hi rounds the same real sum once, as the
// conversion followed by an fp32 add does: one instruction per output instead of a conversion and an add.
__device__ __forceinline__ void first_stage(u32 pair, float &sum, float &diff)
{
    asm("v_fma_mix_f32 %0, %1, 1.0, %1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(sum) : "v"(pair));
    asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(diff) : "v"(pair));
}

// one stage between the registers of a piece (span 1, 2, 4)
template <int SPAN>
__device__ __forceinline__ void rot_register_stage(float (&v)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (!(i & SPAN)) {
            const float a = v[i], b = v[i | SPAN];
            v[i] = a + b;
            v[i | SPAN] = a - b;
        }
}
template <int SPAN>
__device__ __forceinline__ void rot_register_stage(float (&v)[4][8])
{
#pragma unroll
    for (int p = 0; p < 4; ++p) rot_register_stage<SPAN>(v[p]);
}

// Stages 0-2 of a piece, whose values `form` forms from what was loaded by instructions that issue alone (v_fma_mix_f32, v_cvt_pk_f32_fp8),
// hence at raised priority (see rot_priority; `raised`: rot_raised in fc_rot.hip); FIRST: the first of the three that it leaves to do.  us, without / with: quantize INT4
// (group 128) 8192 x 8192 37.9 / 35.9, x 5120 20.8 / 19.7, INT8 x 4096 20.2 / 19.4; dequantize INT4 37.9 / 36.0, 20.8 / 19.6, FP8
// 4096 x 8192 22.0 / 21.2; all-reduce of four INT4 x 8192 164.3 / 160.7, x 5120 87.9 / 84.0, FP8 4096 x 8192 102.0 / 97.5.  Not in FP8's
// quantizer (24.2 / 25.9).  Where a launch has a wavefront per SIMD or less there is nobody to give way to, and the order costs up to 1 %;
// all four pieces before the next stages are as fast for large volumes and cost the single transforms 2 % there.
template <int FIRST, typename F>
__device__ __forceinline__ void rot_first_stages(float (&v)[8], F form, bool raised = true)
{
    if (raised) __builtin_amdgcn_s_setprio(1);
    form();
    pin_values(v);
    __builtin_amdgcn_s_setprio(0);
    pin_values(v);
    if constexpr (FIRST == 0) rot_register_stage<1>(v);
    rot_register_stage<2>(v);
    rot_register_stage<4>(v);
}

// one stage between pieces (P = 1, 2).  FLIPPED: the second value of a pair comes negated, in the frame of a DPP stage of this
// bit, which the stage of the inverse transform undoes.
template <int P, bool FLIPPED = false>
__device__ __forceinline__ void rot_piece_stage(float (&v)[4][8])
{
#pragma unroll
    for (int p = 0; p < 4; ++p)
        if (!(p & P))
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = v[p][i], b = v[p | P][i];
                v[p][i] = FLIPPED ? a - b : a + b;
                v[p | P][i] = FLIPPED ? a + b : a - b;
            }
}

// Wavefronts per block of 2^LB elements, and per workgroup (blocks of at most one wavefront go two wavefronts to a
// workgroup; these never meet)
constexpr int rot_block_waves(int lb) { return lb <= 11 ? 1 : 1 << (lb - 11); }
constexpr int rot_group_waves(int lb) { return lb <= 11 ? 2 : 1 << (lb - 11); }
// bytes of LDS through which the wavefronts of a block exchange pieces, in one or two rounds
constexpr int rot_exchange_bytes(int lb, int rounds) { return lb <= 11 ? 16 : rot_block_waves(lb) * 4 * 2048 / rounds; }

// Piece bits change places with wavefront bits; an involution.  LB = 13: the two piece bits with the two wavefront
// bits.  LB = 12: the upper piece bit with the one wavefront bit.  Pieces lie in LDS by receiving wavefront, then by
// sending wavefront, so that one address register serves all writes and one all reads.  The piece that stays goes
// through LDS as well: sorting it out costs a branch per piece and nothing is gained (LDS is not what bounds these
// kernels).  The caller sees to it that the previous readers of `lds` are done.
// Two rounds of half the values each halve the LDS, for kernels that it keeps from filling the SIMDs with wavefronts.
//
// The lanes may change places as well, and for LB = 12 the lower piece bit with a lane bit: a lane writes its 16 bytes of a 1 KB
// run at `out_lane` (odd pieces: at out_lane ^ out_odd), and takes those at `in_lane`, of odd pieces at
// (in_lane ^ in_odd) + in_step.
struct RotPlaces {
    u32 out_lane, out_odd, in_lane, in_odd, in_step;
};
template <int LB, int ROUNDS>
__device__ __forceinline__ void rot_exchange(float (&v)[4][8], uint8_t *lds, u32 wave, const RotPlaces at_lane)
{
    static_assert(LB == 12 || LB == 13, "blocks of several wavefronts");
    static_assert(ROUNDS == 1 || ROUNDS == 2, "all of a lane's 32 bytes per piece, or half of them");
    constexpr u32 kPiece = 2048 / ROUNDS, kPerSender = LB == 13 ? kPiece : 2 * kPiece, kPerReceiver = 4 * kPiece;
    uint8_t *out = lds + wave * kPerSender;
    const uint8_t *in = lds + wave * kPerReceiver;
#pragma unroll
    for (u32 r = 0; r < (u32)ROUNDS; ++r) {
        if (r > 0) lds_barrier();
#pragma unroll
        for (u32 p = 0; p < 4; ++p)
#pragma unroll
            for (u32 k = 0; k < 2 / ROUNDS; ++k) {
                const u32 h = r + k;
                const u32 at = (LB == 13 ? p * kPerReceiver : (p >> 1) * kPerReceiver + (p & 1u) * kPiece) + k * 1024;
                *reinterpret_cast<u32x4 *>(out + (p & 1u ? at_lane.out_lane ^ at_lane.out_odd : at_lane.out_lane) + at) =
                    u32x4{__builtin_bit_cast(u32, v[p][4 * h]), __builtin_bit_cast(u32, v[p][4 * h + 1]),
                          __builtin_bit_cast(u32, v[p][4 * h + 2]), __builtin_bit_cast(u32, v[p][4 * h + 3])};
            }
        lds_barrier();
#pragma unroll
        for (u32 p = 0; p < 4; ++p)
#pragma unroll
            for (u32 k = 0; k < 2 / ROUNDS; ++k) {
                const u32 h = r + k;
                const u32 at = (LB == 13 ? p * kPiece : (p >> 1) * kPerSender) + (p & 1u) * at_lane.in_step + k * 1024;
                const u32x4 a = *reinterpret_cast<const u32x4 *>(in + (p & 1u ? at_lane.in_lane ^ at_lane.in_odd : at_lane.in_lane) + at);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u32 w = a[i];    // (a bit_cast applied to the vector element itself reads element 0)
                    v[p][4 * h + i] = __builtin_bit_cast(float, w);
                }
            }
    }
}
// every lane keeps its place, every piece its lower bit
template <int LB, int ROUNDS>
__device__ __forceinline__ RotPlaces rot_same_places(u32 lane)
{
    return RotPlaces{lane * 16, 0, lane * 16, 0, LB == 13 ? 0u : 2048u / ROUNDS};
}

// The places of the exchanges of the forward and of the back transform, where a lane takes over from the one that holds its
// element bits, wherever they lie.  Element bits of pos 0-3 / lane 4 5 / pieces:
//   LB = 13  forward  3 4 5 6 / 9 10 / 7 8   -> 3 4 9 10 / 5 6 / 11 12      back  3 4 9 10 / 11 12 / 5 6 -> 9 10 11 12 / 3 4 / 7 8
//   LB = 12  forward  3 4 5 6 / 9 10 / 7 8   -> 3 4 9 7 / 5 6 / 10 11       back  3 4 9 7 / 10 11 / 5 6  -> 9 10 11 5 / 3 4 / 7 8
// The xor terms keep the 16 lanes of a row in different banks on both sides.
template <int LB, int ROUNDS, bool BACK>
__device__ __forceinline__ RotPlaces rot_places(const RotLane &L)
{
    constexpr u32 kPiece = 2048 / ROUNDS;
    auto out = [](u32 lane) -> u32 {
        return (lane * 16u) ^ (BACK ? ((lane >> 4) & 3u) << 4 : ((lane >> 4) & (LB == 13 ? 3u : 1u)) << 6);
    };
    auto lane_of = [](u32 pos, u32 rows) -> u32 { return (pos ^ ((pos & 4u) ? 3u : 0u)) | (rows << 4); };
    const u32 rows = (L.lane >> 4) & 3u, r = L.pos & 15u, r3 = r >> 3;
    if constexpr (LB == 13) {
        const u32 from = BACK ? lane_of(rows | ((r & 3u) << 2), r >> 2) : lane_of((r & 3u) | (rows << 2), r >> 2);
        return RotPlaces{out(L.lane), 0, out(from), 0, 0};
    } else if constexpr (BACK) {
        const u32 from = lane_of(rows | ((r & 1u) << 2), (r >> 1) & 3u);
        return RotPlaces{out(L.lane), 128, (out(from) ^ (r3 << 7)) + r3 * kPiece, 128, 0};
    } else {
        const u32 from = lane_of((r & 3u) | (rows << 2), (r >> 2) & 1u);
        return RotPlaces{out(L.lane), 128, (out(from) ^ (r3 << 7)) + r3 * kPiece, 0, 512};
    }
}

// Stages 3 ... LB-1 of the forward transform (0-2: rot_first_stages): kRotLoaded -> rot_forward_map
template <int LB, bool SWAPS, bool FP8, int ROUNDS, RotOrder ORDER>
__device__ __forceinline__ void rot_forward(float (&v)[4][8], const RotLane &L, uint8_t *lds, u32 wave)
{
    rot_row_stages<FP8, false, ORDER>(v, L);
    rot_piece_stage<1>(v);
    rot_piece_stage<2>(v);
    if constexpr (LB == 13 && SWAPS) {
        rot_swap<4, FP8, ORDER>(v);
        rot_piece_stage<1>(v);
        rot_swap<5, FP8, ORDER>(v);
        rot_piece_stage<2>(v);
        rot_exchange<LB, ROUNDS>(v, lds, wave, rot_same_places<LB, ROUNDS>(L.lane));
        rot_piece_stage<1>(v);
        rot_piece_stage<2>(v);
    } else if constexpr (LB >= 12) {
        rot_exchange<LB, ROUNDS>(v, lds, wave, rot_places<LB, ROUNDS, false>(L));
        if constexpr (FP8) {
            rot_crossbar_stage<7>(v, L.s[2]);
            static_assert(LB == 12 || !FP8, "blocks of 8192: the other form");
        } else {                           // through the crossbar instead: all-reduce 166 -> 179 us
            rot_priority<1, ORDER>(v);
            rot_row_some<2, LB == 13 ? 2 : 1, false, false>(v, L);
            rot_priority<0, ORDER>(v);
        }
        rot_piece_stage<1>(v);
        rot_piece_stage<2>(v);
    } else {
        rot_crossbar_stage<16>(v, L.s[4]);
        if constexpr (LB == 11) {
            rot_swap<5, FP8, ORDER>(v);
            rot_piece_stage<2>(v);
        }
    }
}

// Inverse transform: stages 0-6 on values in the frame of the forward transform, which they leave (FP8: frame +1)
template <bool FP8, RotOrder ORDER>
__device__ __forceinline__ void rot_inverse_row(float (&v)[4][8], const RotLane &L)
{
    rot_register_stage<1>(v);
    rot_register_stage<2>(v);
    rot_register_stage<4>(v);
    rot_row_stages<FP8, true, ORDER>(v, L);
}

// ... and the remaining ones, on values that come from memory: kRotLoaded -> rot_forward_map.  `exchanged` is called between the
// exchange and the stages after it.
template <int LB, int ROUNDS, typename F>
__device__ __forceinline__ void rot_inverse_rest(float (&v)[4][8], const RotLane &L, uint8_t *lds, u32 wave, F exchanged)
{
    rot_piece_stage<1>(v);
    rot_piece_stage<2>(v);
    rot_crossbar_stage<16>(v, L.s[4]);
    if constexpr (LB >= 11) {
        rot_swap<5>(v);
        rot_piece_stage<2>(v);
    }
    if constexpr (LB >= 12) {
        rot_exchange<LB, ROUNDS>(v, lds, wave, rot_same_places<LB, ROUNDS>(L.lane));
        exchanged();
        if constexpr (LB == 13) rot_piece_stage<1>(v);
        rot_piece_stage<2>(v);
    }
}
constexpr RotMap rot_inverse_map(int lb)
{
    return lb == 13 ? RotMap{9, 8, 11, 12, 7, 10} : lb == 12 ? RotMap{9, 8, 7, 11, 10, 12} : rot_forward_map(lb, true);
}

// The inverse transform of values that a forward transform has left, in its frame: rot_forward_map -> rot_back_map.
// Returns the frame of the results.
template <int LB, bool SWAPS, bool FP8, int ROUNDS, RotOrder ORDER>
__device__ __forceinline__ float rot_inverse_back(float (&v)[4][8], const RotLane &L, uint8_t *lds, u32 wave)
{
    if constexpr (LB == 13 && SWAPS) {
        rot_inverse_row<FP8, ORDER>(v, L);
        if constexpr (!FP8) settle_pieces(v);
        rot_swap<4, FP8, ORDER>(v);                    // l4 l5 p0 p1 w0 w1 = 11  8  7 12  9 10
        rot_piece_stage<1>(v);
        rot_swap<5, FP8, ORDER>(v);                    //                     11 12  7  8  9 10
        rot_piece_stage<2>(v);
        rot_exchange<LB, ROUNDS>(v, lds, wave, rot_same_places<LB, ROUNDS>(L.lane));       //     11 12  9 10  7  8
        rot_piece_stage<1>(v);
        rot_piece_stage<2>(v);
        rot_crossbar_stage<16>(v, L.s[4]);
        rot_swap<5, FP8, ORDER>(v);                    //                     11 10  9 12  7  8
        rot_piece_stage<2>(v);
        return 1.0f;
    } else if constexpr (LB >= 12) {
        rot_register_stage<1>(v);
        rot_register_stage<2>(v);
        rot_register_stage<4>(v);
        rot_priority<1, ORDER>(v);
        rot_row_some<0, 2, FP8, true>(v, L);
        if constexpr (!FP8) settle_pieces(v);
        rot_swap<4, FP8, ORDER>(v);                    // 5 into piece bit 0
        rot_priority<0, ORDER>(v);
        rot_piece_stage<1, !FP8>(v);
        rot_swap<5, FP8, ORDER>(v);                    // 6 into piece bit 1
        rot_piece_stage<2, !FP8>(v);
        rot_exchange<LB, ROUNDS>(v, lds, wave, rot_places<LB, ROUNDS, true>(L));
        rot_piece_stage<1>(v);
        rot_piece_stage<2>(v);
        // 9 ... LB-1 in the row: 9 (and 10 of blocks of 8192) was a DPP stage of the forward transform
        rot_priority<1, ORDER>(v);
        if constexpr (LB == 13) {
            rot_row_some<0, 2, FP8, true>(v, L);
            rot_row_some<2, 2, FP8, false>(v, L);
        } else {
            rot_row_some<0, 1, FP8, true>(v, L);
            rot_row_some<1, 2, FP8, false>(v, L);
        }
        rot_priority<0, ORDER>(v);
        return FP8 ? 1.0f : LB == 13 ? L.s[2] * L.s[3] : L.s[1] * L.s[2];
    } else {
        rot_inverse_row<FP8, ORDER>(v, L);
        rot_piece_stage<1>(v);
        if constexpr (LB == 11) rot_swap<5, FP8, ORDER>(v);            //  9 10  7  8
        rot_piece_stage<2>(v);
        rot_crossbar_stage<16>(v, L.s[4]);
        if constexpr (LB == 11) {
            rot_swap<5, FP8, ORDER>(v);                                //  9  8  7 10
            rot_piece_stage<2>(v);
        }
        return 1.0f;
    }
}

// Quantizer, blocks of 8192, integer codes, the two forms of the transform: `swaps` has fewer instructions that issue alone, the other form
// fewer in all (and lays a group of 256 elements across wavefronts).  us, swaps / exchange: INT4, group 128 4.14 / 4.21 (128 tokens), 4.44 / 4.50
// (256), 5.23 / 5.00 (320), 7.96 / 7.52 (1024), 42 / 38 (8192); sym, group 1024 4.49 / 4.50 (256), 5.25 / 5.05, 7.88 / 7.51.  Hence by the
// volume, at one workgroup per compute unit.  FP8 always swaps: its stages in a row cost a move and a multiply-add or a pass
// through the crossbar.  The all-reduce: ALONE in fc_rot_sim.hip.
inline bool rot_swaps_apply(int64_t n_elems) { return n_elems <= ((int64_t)256 << 13); }

// ---------------------------------------------------------------------------
// min / max of the groups.  Each lane first has one (min, max) pair per piece; a transposing reduction over bits 3
// and 4 leaves ONE pair per lane, that of piece lane & 3, so that Eq. 1 is evaluated once per lane for all four
// pieces.  Pairs are in the lane's frame; a partner across a frame boundary has min and max exchanged and negated,
// which the DPP instruction's operand modifier does.
// ---------------------------------------------------------------------------
template <int CTRL_BIT>
__device__ __forceinline__ void minmax_step(float &mn, float &mx, float other_mn, float other_mx)
{
    static_assert(CTRL_BIT == 3 || CTRL_BIT == 4, "inside a quad of lanes");
    float a, b;
#define FC_MINMAX_DPP(ctrl)                                                                                            \
    asm("s_nop 1\n\tv_min_f32_dpp %0, -%3, %4 " ctrl " row_mask:0xf bank_mask:0xf\n\t"                                \
        "v_max_f32_dpp %1, -%2, %5 " ctrl " row_mask:0xf bank_mask:0xf"                                                \
        : "=&v"(a), "=v"(b) : "v"(other_mn), "v"(other_mx), "v"(mn), "v"(mx))
    if constexpr (CTRL_BIT == 3) FC_MINMAX_DPP("quad_perm:[1,0,3,2]");
    if constexpr (CTRL_BIT == 4) FC_MINMAX_DPP("quad_perm:[2,3,0,1]");
#undef FC_MINMAX_DPP
    mn = a;
    mx = b;
}

// One instruction each; the compiler's own would first canonicalize the inputs.
__device__ __forceinline__ void minmax_with(float &mn, float &mx, float other_mn, float other_mx)
{
    asm("v_min_f32 %0, %0, %1" : "+v"(mn) : "v"(other_mn));
    asm("v_max_f32 %0, %0, %1" : "+v"(mx) : "v"(other_mx));
}

// with the pair of lane ^ 16 (LANE_BIT = 4) or lane ^ 32
template <int LANE_BIT>
__device__ __forceinline__ void minmax_across(float &mn, float &mx)
{
    u32 a = __builtin_bit_cast(u32, mn), b = a, c = __builtin_bit_cast(u32, mx), d = c;
    asm("s_nop 1" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));     // see rot_swap
    swap_lane_bit<LANE_BIT>(a, b);
    swap_lane_bit<LANE_BIT>(c, d);
    mn = __builtin_bit_cast(float, a);
    mx = __builtin_bit_cast(float, c);
    minmax_with(mn, mx, __builtin_bit_cast(float, b), __builtin_bit_cast(float, d));
}

template <int CTRL>
__device__ __forceinline__ void minmax_dpp(float &mn, float &mx)
{
    mn = dpp_min<CTRL>(mn);
    mx = dpp_max<CTRL>(mx);
}

// min and max of the group that piece lane & 3 of the lane belongs to (identical in all its lanes, frame +1).  LDS slots
// `slot` carry the pairs of groups that span wavefronts; the caller has a barrier between two uses of them.
constexpr int kRotSlots = 16;              // pairs per wavefront: those of the lanes of its first row
template <int LB, bool SWAPS>
__device__ __forceinline__ void rot_group_minmax(const float (&v)[4][8], const RotLane &L, int group_shift, u32 wave,
                                                 float (*slot)[kRotSlots][2], float &mn_out, float &mx_out)
{
    float mn[4], mx[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) lane_minmax(v[p], mn[p], mx[p]);
    const bool b3 = (L.lane & 1u) != 0, b4 = (L.lane & 2u) != 0;
    float n2[2], x2[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        n2[h] = b3 ? mn[2 * h + 1] : mn[2 * h];
        x2[h] = b3 ? mx[2 * h + 1] : mx[2 * h];
        minmax_step<3>(n2[h], x2[h], b3 ? mn[2 * h] : mn[2 * h + 1], b3 ? mx[2 * h] : mx[2 * h + 1]);
    }
    float n = b4 ? n2[1] : n2[0], x = b4 ? x2[1] : x2[0];
    minmax_step<4>(n, x, b4 ? n2[0] : n2[1], b4 ? x2[0] : x2[1]);
    const float t = L.frame < 0.0f ? -x : n;
    x = L.frame < 0.0f ? -n : x;
    n = t;
    // the other element bits, where the forward transform left them; partners hold the same piece (lane & 3) throughout,
    // piece bits flip with lane bits 0 and 1
    constexpr RotMap m = rot_forward_map(LB, SWAPS);
    if constexpr (m.r2 == 5) {
        if (group_shift > 6) {             // the other three quads of the row
            minmax_dpp<kDppRowRor4>(n, x);
            minmax_dpp<kDppRowRor8>(n, x);
        } else if (group_shift > 5) {      // lane ^ 4, as lane ^ 3 ^ 7
            float n3, x3;
            asm("s_nop 1\n\tv_mov_b32_dpp %2, %0 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %3, %1 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                "v_min_f32_dpp %0, %2, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_max_f32_dpp %1, %3, %1 row_half_mirror row_mask:0xf bank_mask:0xf"
                : "+v"(n), "+v"(x), "=&v"(n3), "=&v"(x3));
        }
    }
    if (group_shift > m.l4) minmax_across<4>(n, x);
    if (group_shift > m.l5) minmax_across<5>(n, x);
    if constexpr (m.r2 != 5) {
        if (group_shift > m.r2) minmax_with(n, x, crossbar<4>(n), crossbar<4>(x));
        if (group_shift > m.r3) minmax_dpp<kDppRowRor8>(n, x);
    }
    if (group_shift > m.p0) minmax_dpp<kDppQuadXor1>(n, x);
    if (group_shift > m.p1) minmax_dpp<kDppQuadXor2>(n, x);
    if constexpr (LB >= 12) {
        if (group_shift > m.w0) {
            if (L.lane < (u32)kRotSlots) {
                slot[wave][L.lane][0] = n;
                slot[wave][L.lane][1] = x;
            }
            lds_barrier();
            const u32 at = L.lane & (kRotSlots - 1u);
            minmax_with(n, x, slot[wave ^ 1u][at][0], slot[wave ^ 1u][at][1]);
            if (LB == 13 && group_shift > m.w1) {
                minmax_with(n, x, slot[wave ^ 2u][at][0], slot[wave ^ 2u][at][1]);
                minmax_with(n, x, slot[wave ^ 3u][at][0], slot[wave ^ 3u][at][1]);
            }
        }
    }
    mn_out = n;
    mx_out = x;
}

// max|x| in place of the pair, for the symmetric and the FP8 quantizer: no frames, half of the instructions.  us, from the pair / this: all-reduce
// of four 8192 x 8192 sym INT8 162.1 / 155.3, x 5120 INT4 87.4 / 82.5, x 4096 83.6 / 79.1, FP8 103.3 / 99.8; of two of one token of 8192
// 6.89 / 6.69, of 12 x 2048 5.90 / 5.53; quantize 8192 x 8192 sym INT4 36.7 / 34.8, FP8 43.3 / 42.5.
template <int CTRL_BIT>
__device__ __forceinline__ float absmax_step(float own, float other)
{
    static_assert(CTRL_BIT == 3 || CTRL_BIT == 4, "inside a quad of lanes");
    float r;
    if constexpr (CTRL_BIT == 3)
        asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(other), "v"(own));
    else
        asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(other), "v"(own));
    return r;
}

__device__ __forceinline__ float max_with(float a, float b)
{
    asm("v_max_f32 %0, %0, %1" : "+v"(a) : "v"(b));
    return a;
}

template <int LANE_BIT>
__device__ __forceinline__ float max_across(float m)
{
    u32 a = __builtin_bit_cast(u32, m), b = a;
    asm("s_nop 1" : "+v"(a), "+v"(b));                       // see rot_swap
    swap_lane_bit<LANE_BIT>(a, b);
    return max_with(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}

template <int LB, bool SWAPS>
__device__ __forceinline__ float rot_group_absmax(const float (&v)[4][8], const RotLane &L, int group_shift, u32 wave,
                                                  float (*slot)[kRotSlots][2])
{
    float a[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) a[p] = lane_absmax(v[p]);
    const bool b3 = (L.lane & 1u) != 0, b4 = (L.lane & 2u) != 0;
    float h[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
        h[k] = absmax_step<3>(b3 ? a[2 * k + 1] : a[2 * k], b3 ? a[2 * k] : a[2 * k + 1]);
    float m = absmax_step<4>(b4 ? h[1] : h[0], b4 ? h[0] : h[1]);
    constexpr RotMap at = rot_forward_map(LB, SWAPS);
    if constexpr (at.r2 == 5) {
        if (group_shift > 6) {
            m = dpp_max<kDppRowRor4>(m);
            m = dpp_max<kDppRowRor8>(m);
        } else if (group_shift > 5) {
            m = max_with(m, crossbar<4>(m));
        }
    }
    if (group_shift > at.l4) m = max_across<4>(m);
    if (group_shift > at.l5) m = max_across<5>(m);
    if constexpr (at.r2 != 5) {
        if (group_shift > at.r2) m = max_with(m, crossbar<4>(m));
        if (group_shift > at.r3) m = dpp_max<kDppRowRor8>(m);
    }
    if (group_shift > at.p0) m = dpp_max<kDppQuadXor1>(m);
    if (group_shift > at.p1) m = dpp_max<kDppQuadXor2>(m);
    if constexpr (LB >= 12) {
        if (group_shift > at.w0) {
            if (L.lane < (u32)kRotSlots) slot[wave][L.lane][0] = m;
            lds_barrier();
            const u32 k = L.lane & (kRotSlots - 1u);
            m = max_with(m, slot[wave ^ 1u][k][0]);
            if (LB == 13 && group_shift > at.w1) m = max_with(max_with(m, slot[wave ^ 2u][k][0]), slot[wave ^ 3u][k][0]);
        }
    }
    return m;
}

// the value that the lanes with lane & 3 == P of the quad hold, in all lanes
template <int P>
__device__ __forceinline__ float of_piece(float v)
{
    float r = dpp_read<P * 0x55>(v);
    asm("" : "+v"(r));                     // else the DPP operand is folded into every multiplication (4 cycles instead of 2)
    return r;
}

}  // namespace fc
