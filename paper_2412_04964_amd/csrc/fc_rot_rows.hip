// fc_rot_rows.hip -- the rotated quantizer and dequantizer between the launch-bound volumes of fc_rot_fine.hip and those that fill the chip:
// the row in LDS.
//
// The same arithmetic as fc_rot.hip (butterflies in the order of the spans, so bit-identical), split the other way: a lane
// holds one 128-bit word of codes, 32 elements at 4 bit and 16 at 8 bit, as in the plain kernels, transforms these, and then the row lies
// in LDS and each phase gives every lane the values that differ in the next four or five index bits, with a barrier
// between phases.  More LDS traffic than the register form of fc_rot.hip, which wins once the chip is full, but shorter
// chains of dependent instructions: a wavefront of that form works through 2048 elements, here 1024 at 8 bit.
//
// What bounds it: latency of one wavefront.  us per launch under graph replay, this / register form, group 128
// (rot_rows_apply says where each is taken):
//   quantize, this / register form / the form of fc_rot_fine.hip, blocks of 1024: 4 bit, group 128  1.25 M 3.20 / 3.56 / 3.01, 1.5 M 3.32 / 3.59 / 3.38, group 1024  1.5 M
//     3.54 / 3.77 / 3.87, 2 M 3.83 / 3.96 / 3.91; 8 bit, group 128  1.5 M 3.21 / 3.56 / 3.40, 2 M 3.46 / 3.62 / 3.55; 2048: 8 bit, group 128  1 M 3.07 / 3.20 / 2.90, 1.5 M
//     3.18 / 3.52 / 3.22, 2 M 3.47 / 3.59 / 3.71, 2.5 M 3.83 / 3.79.
//   quantize FP8, blocks of 1024: 3 M 4.67 / 4.79; 4 M 5.22 / 5.11; 2048: 3 M 4.70 / 4.99; 4 M 5.25 / 5.33; 5 M 5.89 / 5.83; 4096: 3 M
//     5.02 / 5.39; 4 M 5.67 / 5.79; 5 M 6.30 / 6.20.
//   dequantize, blocks of 1024: 8 bit 1 M elements 3.08 / 3.20; 2 M 3.62 / 3.85; 2.5 M 3.95 / 3.93; 8 M 7.23 / 5.78; FP8 1 M 2.98 / 3.47;
//     3 M 4.21 / 4.19; 4 M 4.81 / 4.37; 4 bit 1 M 3.08 / 3.06; 2 M 3.50 / 3.69; 2.5 M 3.95 / 3.74; 8 M 6.05 / 5.57; 16 M 11.01 / 9.94.
//   2048: 8 bit 2 M 3.65 / 3.94; 3 M 4.39 / 4.11; FP8 3 M 4.24 / 4.28; 4 M 4.81 / 4.48.
//   4096: 8 bit 2 M 3.89 / 4.43; 3 M 4.53 / 4.75; 4 M 5.17 / 5.01; FP8 3 M 4.46 / 4.82; 4 M 5.10 / 5.11; 5 M 5.69 / 5.49.
//   Blocks of 8192: the register form.
#include "fc_rot_wave.hpp"
#include "fc_launch.hpp"

namespace fc {

constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v / 2); }

// Butterfly stages S0 ... NB-1 over the low NB bits of the register index, spans 2^S0, 2^(S0+1), ...
template <int R, int NB, int S0 = 0>
__device__ __forceinline__ void butterflies(float (&x)[R])
{
#pragma unroll
    for (int s = S0; s < NB; ++s)
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (!(q & (1 << s))) {
                const float a = x[q], b = x[q | (1 << s)];
                x[q] = a + b;
                x[q | (1 << s)] = a - b;
            }
}

// word position of element e in the padded LDS row: 4 extra words per lane segment of 2^LE elements
template <int LE>
__device__ __forceinline__ constexpr u32 padded(u32 e)
{
    return e + 4u * (e >> LE);
}

// One LDS phase: stages over index bits [B0, B0 + NB).  Thread `tid` of T = 2^LT
// threads holds the R values whose index has register bits q_lo at [B0, B0+NB)
// and whose remaining bits are u = q_hi * T + tid; the position of the values is
// unchanged, so there is no hazard inside a phase.
template <int B0, int NB, int R, int LT, int LE>
__device__ __forceinline__ void lds_phase(float *row, u32 tid)
{
    const u32 et = ((tid >> B0) << (B0 + NB)) | (tid & ((1u << B0) - 1u));
    float *base = row + padded<LE>(et);
    auto at = [](int q) constexpr -> u32 {
        const u32 q_lo = (u32)q & ((1u << NB) - 1u), u = ((u32)q >> NB) << LT;
        const u32 e = ((u >> B0) << (B0 + NB)) | (q_lo << B0) | (u & ((1u << B0) - 1u));
        return e + 4u * (e >> LE);         // disjoint bit fields: padded(et | e) == padded(et) + padded(e)
    };
    float x[R];
#pragma unroll
    for (int q = 0; q < R; ++q) x[q] = base[at(q)];
    butterflies<R, NB>(x);
#pragma unroll
    for (int q = 0; q < R; ++q) base[at(q)] = x[q];
}

// Remaining stages for index bits [B0, END), R registers per thread, in phases of up to log2(R) bits.
template <int B0, int END, int R, int LT, int LE>
__device__ __forceinline__ void lds_phases(float *row, u32 tid)
{
    if constexpr (B0 < END) {
        constexpr int NB = (END - B0) < ilog2(R) ? (END - B0) : ilog2(R);
        lds_phase<B0, NB, R, LT, LE>(row, tid);
        __syncthreads();
        lds_phases<B0 + NB, END, R, LT, LE>(row, tid);
    }
}

// Shape of the workgroup for a code width and a row of 2^LOGH elements: one 128-bit word of codes per lane.
template <int BITS, int LOGH>
struct RowShape {
    static constexpr int EPL = lane_elems(BITS);
    static constexpr int LE = ilog2(EPL);
    static constexpr int H = 1 << LOGH;
    static constexpr int T = H / EPL;
    static constexpr int LT = ilog2(T);
    static constexpr int ROW_WORDS = H + 4 * (H / EPL);
    static constexpr int kPieces = EPL * 2 / 16;                       // 1 KB runs of binary16 values per wavefront
    static constexpr int kImgBytes = (T / 64) * kPieces * 1024;
    // the binary16 image of the row and the padded fp32 row of the transform share their LDS
    static constexpr int kLdsBytes = kImgBytes > ROW_WORDS * 4 ? kImgBytes : ROW_WORDS * 4;
    static_assert(T >= 64 && T <= kBlockThreads, "rows of 2048 and 4096 elements");
};

// In-place transform of every aligned block of 2^LB elements of the row held as v[i] = element tid*EPL + i.
// With S0 = 1 the caller has already applied the first stage (span 1).
template <int BITS, int LOGH, int LB, int S0, int NE>
__device__ __forceinline__ void hadamard_row(float (&v)[NE], float *row, u32 tid)
{
    using S = RowShape<BITS, LOGH>;
    static_assert(NE == S::EPL, "row held as v[EPL]");
    static_assert(LB <= LOGH && LB > S::LE, "blocks of at least two lanes, at most the row");
    butterflies<S::EPL, S::LE, S0>(v);
    u32x4 *mine = reinterpret_cast<u32x4 *>(row + padded<S::LE>(tid * S::EPL));
#pragma unroll
    for (int k = 0; k < S::EPL / 4; ++k)
        mine[k] = u32x4{__builtin_bit_cast(u32, v[4 * k]), __builtin_bit_cast(u32, v[4 * k + 1]),
                        __builtin_bit_cast(u32, v[4 * k + 2]), __builtin_bit_cast(u32, v[4 * k + 3])};
    __syncthreads();
    lds_phases<S::LE, LB, S::EPL, S::LT, S::LE>(row, tid);     // ends with a barrier
#pragma unroll
    for (int k = 0; k < S::EPL / 4; ++k) {
        const u32x4 a = mine[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32 w = a[i];            // (a bit_cast applied to the vector element itself reads element 0)
            v[4 * k + i] = __builtin_bit_cast(float, w);
        }
    }
}

// Rotate one row block by block and quantize it (FinegrainedQuantize of Algorithm 1 on the rotated values).
// n_elems: elements of the whole tensor (a multiple of 2^LB; the last row may be a partial one when LB < LOGH:
// lanes beyond the end read zeros and have their stores dropped or skipped).
template <int BITS, int CODEC, int LOGH, int LB>
__global__ __launch_bounds__((RowShape<BITS, LOGH>::T)) void k_quantize_rot_rows(
    const uint16_t *__restrict__ x, int64_t n_elems, int lpg, int group_shift, uint8_t *__restrict__ codes,
    float *__restrict__ scales, float *__restrict__ zeros)
{
    using S = RowShape<BITS, LOGH>;
    constexpr int EPL = S::EPL, kPieces = S::kPieces;
    __shared__ __attribute__((aligned(16))) uint8_t lds[S::kLdsBytes];
    __shared__ float slot[kBlockWaves][2];
    uint8_t (*img)[kPieces * 1024] = reinterpret_cast<uint8_t (*)[kPieces * 1024]>(lds);
    float *row = reinterpret_cast<float *>(lds);

    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const int64_t e0 = (int64_t)blockIdx.x << LOGH;
    const int64_t here = (n_elems - e0) < (int64_t)S::H ? (n_elems - e0) : (int64_t)S::H;      // elements of this row
    const rsrc_t rx = make_rsrc(x + e0, here * 2);
    const rsrc_t rc = make_rsrc(codes + e0 * BITS / 8, here * BITS / 8);

#pragma unroll
    for (int k = 0; k < kPieces; ++k)
        dma_piece(rx, wave * 64 * EPL * 2 + k * 1024 + lane * 16, &img[wave][k * 1024]);
    wait_vmem_outstanding(0);

    float v[EPL];
    const u32x4 *mine = reinterpret_cast<const u32x4 *>(&img[wave][lane * (EPL * 2)]);
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const u32x4 a = mine[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) first_stage(a[i], v[8 * k + 2 * i], v[8 * k + 2 * i + 1]);
    }
    __syncthreads();                                   // the image is read; its LDS becomes the row

    hadamard_row<BITS, LOGH, LB, 1>(v, row, tid);
    // the forward scaling goes into the group's min and max and its reciprocal (see k_quantize_rot)
    constexpr float fwd = 1.0f / (float)(1 << ((LB + 1) / 2));
    float mn, mx, s, inv, zf = 0.0f;
    lane_minmax(v, mn, mx);
    group_minmax<0>(mn, mx, lpg);
    if (lpg > 64) cross_wave_minmax(mn, mx, slot, wave, lane, (u32)lpg >> 6);

    u32 word[4];
    const float mn_s = mn * fwd, mx_s = mx * fwd;
    if constexpr (CODEC == kFp8) {
        group_params_absmax<448>(fmaxf(fabsf(mn_s), fabsf(mx_s)), s, inv);
        pack_lane_fp8<EPL>(v, inv * fwd, word);
    } else if constexpr (CODEC == kSym) {
        group_params_sym<BITS>(fmaxf(fabsf(mn_s), fabsf(mx_s)), s, inv);
        pack_lane_sym<BITS, EPL>(v, inv * fwd, word);
    } else {
        group_params<BITS>(mn_s, mx_s, s, inv, zf);
        pack_lane<BITS, EPL>(v, inv * fwd, zf, mx, word);
    }
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{word[0], word[1], word[2], word[3]}, rc, tid * 16, 0, kStreamStorePolicy);
    if ((tid & (u32)(lpg - 1)) == 0 && (int64_t)(tid * EPL) < here) {
        const int64_t gi = (e0 >> group_shift) + ((tid * EPL) >> group_shift);
        scales[gi] = s;
        if constexpr (CODEC == kAsym) zeros[gi] = zf;
    }
}

// Dequantize one row, rotate it back block by block and round to binary16 (last step of Algorithm 1).
template <int BITS, int CODEC, int LOGH, int LB>
__global__ __launch_bounds__((RowShape<BITS, LOGH>::T)) void k_dequantize_rot_rows(
    const uint8_t *__restrict__ codes, const float *__restrict__ scales, const float *__restrict__ zeros,
    int64_t n_elems, int group_shift, uint16_t *__restrict__ y)
{
    using S = RowShape<BITS, LOGH>;
    constexpr int EPL = S::EPL, kPieces = S::kPieces;
    __shared__ __attribute__((aligned(16))) uint8_t lds[S::kLdsBytes];
    uint8_t (*img)[kPieces * 1024] = reinterpret_cast<uint8_t (*)[kPieces * 1024]>(lds);
    float *row = reinterpret_cast<float *>(lds);

    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const int64_t e0 = (int64_t)blockIdx.x << LOGH;
    const int64_t here = (n_elems - e0) < (int64_t)S::H ? (n_elems - e0) : (int64_t)S::H;      // elements of this row
    const int64_t g_last = (n_elems >> group_shift) - 1;
    const rsrc_t rc = make_rsrc(codes + e0 * BITS / 8, here * BITS / 8);
    const rsrc_t ry = make_rsrc(y + e0, here * 2);

    float v[EPL];
    int64_t gi = (e0 >> group_shift) + ((tid * EPL) >> group_shift);
    gi = gi < g_last ? gi : g_last;                        // lanes beyond a partial last row stay inside the arrays
    const float s = scales[gi];
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rc, tid * 16, 0, kStreamLoadPolicy);
    if constexpr (CODEC == kFp8) {
        const u32 w[4] = {a[0], a[1], a[2], a[3]};
        decode_fp8(w, v);
#pragma unroll
        for (int i = 0; i < EPL; ++i) v[i] *= s;
    } else if constexpr (CODEC == kSym) {
        const u32 w[4] = {to_offset_binary<BITS>(a[0]), to_offset_binary<BITS>(a[1]),
                          to_offset_binary<BITS>(a[2]), to_offset_binary<BITS>(a[3])};
        scaled_differences_fast<BITS>(w, sym_zero_const<BITS>(), s, v);
    } else {
        const float zf = zeros[gi];
        const u32 w[4] = {a[0], a[1], a[2], a[3]};
        if (__builtin_amdgcn_ballot_w64(!zero_is_fast(zf)) == 0) {
            scaled_differences_fast<BITS>(w, unpack_zero_const(pack_zero_const(zf)), s, v);
        } else {
            codes_minus_zero_general<BITS>(w, zf, v);
#pragma unroll
            for (int i = 0; i < EPL; ++i) v[i] *= s;
        }
    }

    hadamard_row<BITS, LOGH, LB, 0>(v, row, tid);
    __syncthreads();                                   // the row is read; its LDS becomes the output image
    constexpr float back = 1.0f / (float)(1 << (LB / 2));              // 2^-floor(n/2), n = LB

    u32x4 *mine = reinterpret_cast<u32x4 *>(&img[wave][lane * (EPL * 2)]);
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        u32x4 out;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h2 h;
            h.x = (_Float16)(v[8 * k + 2 * i] * back);
            h.y = (_Float16)(v[8 * k + 2 * i + 1] * back);
            out[i] = as_u32(h);
        }
        mine[k] = out;
    }
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
        const u32x4 o = *reinterpret_cast<const u32x4 *>(&img[wave][k * 1024 + lane * 16]);
        __builtin_amdgcn_raw_buffer_store_b128(o, ry, wave * 64 * EPL * 2 + k * 1024 + lane * 16, 0, kStreamStorePolicy);
    }
}

namespace {

template <int BITS, int CODEC, int LOGH, int LB>
hipError_t quantize_one(const uint16_t *x, int64_t n_elems, int group, uint8_t *c, float *scales, float *zeros,
                        hipStream_t stream)
{
    const unsigned grid = (unsigned)((n_elems + ((int64_t)1 << LOGH) - 1) >> LOGH);
    return launch_kernel(k_quantize_rot_rows<BITS, CODEC, LOGH, LB>, dim3(grid), dim3(RowShape<BITS, LOGH>::T), stream, x,
                         n_elems, group / lane_elems(BITS), log2_int(group), c, scales, zeros);
}

template <int BITS, int CODEC, int LOGH, int LB>
hipError_t dequantize_one(const uint8_t *c, const float *scales, const float *zeros, int64_t n_elems, int group,
                          uint16_t *y, hipStream_t stream)
{
    const unsigned grid = (unsigned)((n_elems + ((int64_t)1 << LOGH) - 1) >> LOGH);
    return launch_kernel(k_dequantize_rot_rows<BITS, CODEC, LOGH, LB>, dim3(grid), dim3(RowShape<BITS, LOGH>::T), stream, c,
                         scales, zeros, n_elems, log2_int(group), y);
}

// blocks of 1024 go two to a row
template <int BITS, int CODEC>
hipError_t quantize_block(int log_b, const uint16_t *x, int64_t n_elems, int group, uint8_t *c, float *scales,
                          float *zeros, hipStream_t stream)
{
    if (log_b == 10) return quantize_one<BITS, CODEC, 11, 10>(x, n_elems, group, c, scales, zeros, stream);
    if constexpr (BITS == 8)               // at 4 bit the other forms
        if (log_b == 11) return quantize_one<BITS, CODEC, 11, 11>(x, n_elems, group, c, scales, zeros, stream);
    if constexpr (CODEC == kFp8)
        if (log_b == 12) return quantize_one<BITS, CODEC, 12, 12>(x, n_elems, group, c, scales, zeros, stream);
    return hipErrorInvalidValue;
}

template <int BITS, int CODEC>
hipError_t dequantize_block(int log_b, const uint8_t *c, const float *scales, const float *zeros, int64_t n_elems,
                            int group, uint16_t *y, hipStream_t stream)
{
    if (log_b == 10) return dequantize_one<BITS, CODEC, 11, 10>(c, scales, zeros, n_elems, group, y, stream);
    if constexpr (BITS == 8) {             // at 4 bit the other forms
        if (log_b == 11) return dequantize_one<BITS, CODEC, 11, 11>(c, scales, zeros, n_elems, group, y, stream);
        if (log_b == 12) return dequantize_one<BITS, CODEC, 12, 12>(c, scales, zeros, n_elems, group, y, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_quantize_rot_rows(int bits, int codec, const void *x_f16, int64_t n_elems, int log_b, int group,
                                    void *codes, float *scales, float *zeros, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint8_t *c = static_cast<uint8_t *>(codes);
    if (codec == CODEC_FP8)
        return bits == 8 ? quantize_block<8, kFp8>(log_b, x, n_elems, group, c, scales, nullptr, stream)
                         : hipErrorInvalidValue;
    if (bits == 4)
        return codec == CODEC_ASYM ? quantize_block<4, kAsym>(log_b, x, n_elems, group, c, scales, zeros, stream)
                                   : quantize_block<4, kSym>(log_b, x, n_elems, group, c, scales, nullptr, stream);
    return codec == CODEC_ASYM ? quantize_block<8, kAsym>(log_b, x, n_elems, group, c, scales, zeros, stream)
                               : quantize_block<8, kSym>(log_b, x, n_elems, group, c, scales, nullptr, stream);
}

hipError_t launch_dequantize_rot_rows(int bits, int codec, const void *codes, const float *scales, const float *zeros,
                                      int64_t n_elems, int log_b, int group, void *y_f16, hipStream_t stream)
{
    const uint8_t *c = static_cast<const uint8_t *>(codes);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    if (codec == CODEC_FP8)
        return bits == 8 ? dequantize_block<8, kFp8>(log_b, c, scales, nullptr, n_elems, group, y, stream)
                         : hipErrorInvalidValue;
    if (bits == 4)
        return codec == CODEC_ASYM ? dequantize_block<4, kAsym>(log_b, c, scales, zeros, n_elems, group, y, stream)
                                   : dequantize_block<4, kSym>(log_b, c, scales, nullptr, n_elems, group, y, stream);
    return codec == CODEC_ASYM ? dequantize_block<8, kAsym>(log_b, c, scales, zeros, n_elems, group, y, stream)
                               : dequantize_block<8, kSym>(log_b, c, scales, nullptr, n_elems, group, y, stream);
}

}  // namespace fc
