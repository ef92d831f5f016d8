// fc_sim_wide.hip -- Algorithm 1 in ONE launch for groups wider than a wavefront's tile of fc_sim.hip, 2048 to 16384
// elements, the coarse end of the paper's block-size study, up to one group per token (Section 3.2.1); and for groups of one such tile
// where it is the faster form (allreduce_wide_applies).
//
// What bounds it: HBM, 2 N + 2 bytes per output element as in fc_sim.hip; the arithmetic is the same, term by term
// (see the exactness notes there), so the result is bit-identical to fc_quantize x N -> fc_dequant_reduce_requant ->
// fc_dequantize.
//
// Decomposition: one workgroup of group / 16 threads (1 to 16 wavefronts) owns one group.  Because every lane belongs
// to the same group it does not matter which of the group's elements a lane holds: a lane takes two pieces of 8
// elements, each one coalesced 128-bit access, straight into registers and back, and nothing is staged in LDS.  All N
// partials of the group stay in registers (8 N words per lane) between their min / max and their codes, so the
// workgroup meets at two barriers, one for the N first quantizations together and one for the second, instead of one
// per partial.  After the first barrier lane l works out scale, reciprocal and zero-point of source l / 8 (one
// evaluation of Eq. 1 per wavefront for all N sources), and they are broadcast by v_readlane.
//
// Large volumes run with a limited number of workgroups per compute unit (wide_workgroups_per_unit): with all that fit,
// more reads wait in the memory system than it serves well (see fc_sim.hip).
//
// Measured, 4 partials of 8192 x 8192, INT4: groups of 2048 101 us a call (6.6 TB/s on 10 bytes per element; without the limit
// 115), of 4096 102 (110), one group per token 102 (112), against 168 us for the three kernels, whose codes and
// metadata travel through HBM.
#include "fc_device.hpp"
#include "fc_launch.hpp"

namespace fc {

constexpr int kSimWideMaxThreads = 1024;                               // groups of 16384
constexpr int kSimWideMaxWaves = kSimWideMaxThreads / 64;

// min and max over the wavefront, valid in lane 63 only
__device__ __forceinline__ void wave_minmax_last(float &mn, float &mx)
{
    group_minmax<16>(mn, mx, 16);
    mn = rows_reduce<true, true>(mn);
    mx = rows_reduce<false, true>(mx);
}

__device__ __forceinline__ float from_lane(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

template <int CODEC, int BITS_RS, int BITS_AG, int NSRC>
__global__ __launch_bounds__(kSimWideMaxThreads) void k_allreduce_wide(const uint16_t *__restrict__ x, int64_t n_elems,
                                                                      int group_shift, uint16_t *__restrict__ y)
{
    constexpr int E = 16;
    constexpr bool HM = CODEC == kAsymH;
    static_assert(CODEC != kFp8 || (BITS_RS == 8 && BITS_AG == 8), "E4M3 codes are bytes");
    static_assert(NSRC >= 1 && NSRC <= 8, "eight lanes per source in the parameter step");
    __shared__ float slot[NSRC + 1][kSimWideMaxWaves][2];

    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u32 waves = 1u << (group_shift - 10);                        // 64 lanes x 16 elements each
    const u32 piece = 1u << group_shift;                               // bytes of one of the two pieces of the group
    const u32 tile = xcd_tile<16>((u32)(n_elems >> group_shift));
    const int64_t e0 = (int64_t)tile << group_shift;

    u32x4 raw[NSRC][2];
#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        const rsrc_t rx = make_rsrc(x + (int64_t)j * n_elems + e0, (int64_t)piece * 2);
        raw[j][0] = __builtin_amdgcn_raw_buffer_load_b128(rx, tid * 16, 0, kStreamLoadPolicy);
        raw[j][1] = __builtin_amdgcn_raw_buffer_load_b128(rx, tid * 16, piece, kStreamLoadPolicy);
    }

#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        h2 lo = as_h2(raw[j][0][0]), hi = lo;
#pragma unroll
        for (int k = 1; k < 8; ++k) {
            const h2 p = as_h2(raw[j][k >> 2][k & 3]);
            lo = pk_min(lo, p);
            hi = pk_max(hi, p);
        }
        float mn = fminf((float)lo.x, (float)lo.y), mx = fmaxf((float)hi.x, (float)hi.y);
        wave_minmax_last(mn, mx);
        if (lane == 63u) {
            slot[j][wave][0] = mn;
            slot[j][wave][1] = mx;
        }
    }
    __syncthreads();

    // first quantization of source lane / 8 (surplus lanes repeat the last source): its wavefronts' minima and maxima
    // are spread over the eight lanes, two per lane for sixteen wavefronts
    float s_l, inv_l, zf_l = 0.0f;
    {
        const u32 src = (lane >> 3) < (u32)NSRC ? (lane >> 3) : (u32)(NSRC - 1);
        const u32 w0 = (lane & 7u) & (waves - 1u), w1 = ((lane & 7u) + 8u) & (waves - 1u);
        float mn = fminf(slot[src][w0][0], slot[src][w1][0]), mx = fmaxf(slot[src][w0][1], slot[src][w1][1]);
        group_minmax<8>(mn, mx, 8);
        if constexpr (CODEC == kFp8)
            group_params_absmax<448>(fmaxf(fabsf(mn), fabsf(mx)), s_l, inv_l);
        else if constexpr (CODEC == kSym)
            group_params_sym<BITS_RS>(fmaxf(fabsf(mn), fabsf(mx)), s_l, inv_l);
        else
            group_params<BITS_RS, HM>(mn, mx, s_l, inv_l, zf_l);
    }

    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        const float s = from_lane(s_l, 8 * j), inv = from_lane(inv_l, 8 * j);
        if constexpr (CODEC == kFp8) {
            float v[E];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const h2 p = as_h2(raw[j][k >> 2][k & 3]);
                v[2 * k] = (float)p.x;
                v[2 * k + 1] = (float)p.y;
            }
            u32 word[4];
            pack_lane_fp8<E>(v, inv, word);
            accumulate_fp8(word, s, acc);
        } else {
            const float zf = from_lane(zf_l, 8 * j);
            const float d_lo = 0.0f - zf, d_hi = (float)((1 << BITS_RS) - 1) - zf;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const h2 p = as_h2(raw[j][k >> 2][k & 3]);
                float t0 = rintf(fmaf((float)p.x, inv, 0.0f));
                float t1 = rintf(fmaf((float)p.y, inv, 0.0f));
                if constexpr (is_asym(CODEC)) {
                    t0 = __builtin_amdgcn_fmed3f(t0, d_lo, d_hi);
                    t1 = __builtin_amdgcn_fmed3f(t1, d_lo, d_hi);
                }
                acc[2 * k] = fmaf(t0, s, acc[2 * k]);
                acc[2 * k + 1] = fmaf(t1, s, acc[2 * k + 1]);
            }
        }
        pin_values(acc);              // sources are folded in one after the other
    }

    // second quantization and final Dequantize: d[i] = the dequantized code before the scale
    float mn, mx;
    lane_minmax(acc, mn, mx);
    wave_minmax_last(mn, mx);
    if (lane == 63u) {
        slot[NSRC][wave][0] = mn;
        slot[NSRC][wave][1] = mx;
    }
    __syncthreads();
    mn = slot[NSRC][lane & (waves - 1u)][0];
    mx = slot[NSRC][lane & (waves - 1u)][1];
    group_minmax<16>(mn, mx, 16);

    float s, inv, d[E];
    if constexpr (is_asym(CODEC)) {
        float zf;
        group_params<BITS_AG, HM>(mn, mx, s, inv, zf);
        constexpr float qmax = (float)((1 << BITS_AG) - 1);
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const float u = rintf(acc[i] * inv) + zf;
            d[i] = __builtin_amdgcn_fmed3f(u, 0.0f, qmax) - zf;
        }
    } else if constexpr (CODEC == kSym) {
        group_params_sym<BITS_AG>(fmaxf(fabsf(mn), fabsf(mx)), s, inv);
#pragma unroll
        for (int i = 0; i < E; ++i) d[i] = rintf(acc[i] * inv) + 0.0f;
    } else {
        group_params_absmax<448>(fmaxf(fabsf(mn), fabsf(mx)), s, inv);
        u32 word[4];
        pack_lane_fp8<E>(acc, inv, word);
        decode_fp8(word, d);
    }
    const rsrc_t ry = make_rsrc(y + e0, (int64_t)piece * 2);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        u32x4 out;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h2 r;
            r.x = (_Float16)(d[8 * k + 2 * i] * s);
            r.y = (_Float16)(d[8 * k + 2 * i + 1] * s);
            out[i] = as_u32(r);
        }
        store_b128_at(out, ry, tid * 16, k * piece);
    }
}

#ifndef FC_SIM_CODEC
#error "compile with -DFC_SIM_CODEC=0..3 (kAsym, kSym, kFp8, kAsymH): one translation unit per quantizer"
#endif

namespace {

constexpr int CODEC = FC_SIM_CODEC;

// Workgroups that a compute unit shall hold at once, 0: as many as fit.  Many rounds of wavefronts: 16 wavefronts per compute unit with two
// sources, 14 with three, 12 from four on, in workgroups of two or more (groups of 8192: two workgroups in every case; of 16384: no
// limit, one workgroup to a compute unit is too few).  INT4, us, without and with so many workgroups: 8192 x 8192, groups of
// 2048, N = 1 42.9 / 16: 42.9, 12: 41.7, 8: 46.9; N = 2 68.3 / 10: 63.1, 8: 60.8, 7: 63.2; N = 3 93.8 / 8: 86.7, 7: 80.9, 6: 83.7; N = 4
// 114.9 / 7: 104.3, 6: 100.7, 5: 106.1; N = 6 163.9 / 7: 157, 6: 154, 5: 150; N = 8 209.6 / 7: 200, 6: 190, 5: 189; groups of 4096 N = 2
// 67.2 / 4: 61.3, 3: 65.1; N = 3 86.7 / 4: 83.3, 3: 81.1; N = 4 109.8 / 3: 101.8, 2: 111.5; N = 8 203.8 / 3: 184.4.  Groups of
// 2048, N = 4, 6.5 M elements 13.4 / 6: 14.2, 13 M 24.2 / 23.6, 26 M 45.9 / 42.4; N = 8 23.1 / 23.5, 42.4 / 41.2, 82.1 / 76.6.  Few sources have
// fewer reads waiting, and it begins later: groups of 2048, N = 2  12 M 13.7 / 8: 14.4, 16 M 18.6 / 18.8, 20 M 22.9 / 22.4; N = 3  12 M 18.7 / 7: 19.1,
// 14 M 21.9 / 21.6.  Two sources in groups of 1024, one wavefront each, or 8192 are best without: 12 M 13.4 / 14.5, 24 M 26.0 / 26.6, 64 M 66.4 / 66.2;
// 14 M 16.2 / 17.5, 32 M 34.9 / 35.4.
int wide_workgroups_per_unit(int n_src, int64_t n_elems, int group)
{
    if (n_src == 1 || group > 8192 || n_elems < (int64_t)(n_src == 2 ? 20 : n_src == 3 ? 14 : 12) << 20) return 0;
    if (n_src == 2 && (group == 1024 || group == 8192)) return 0;
    const int waves = n_src == 2 ? 16 : n_src == 3 ? 14 : 12, per_group = group / 1024;
    return waves / per_group > 2 ? waves / per_group : 2;
}

template <int BITS_RS, int BITS_AG>
hipError_t launch_wide_bits(const uint16_t *x, int n_src, int64_t n_elems, int group, uint16_t *y, hipStream_t stream)
{
    const dim3 grid((unsigned)(n_elems / group)), block(group / 16);
    const int sh = log2_int(group);
    const size_t pad = lds_to_limit(wide_workgroups_per_unit(n_src, n_elems, group),
                                    (size_t)(n_src + 1) * kSimWideMaxWaves * 2 * sizeof(float));
#define FC_SIM_WIDE(N) \
    case N: return launch_kernel_lds(k_allreduce_wide<CODEC, BITS_RS, BITS_AG, N>, grid, block, pad, stream, x, n_elems, sh, y);
    switch (n_src) {
        FC_SIM_WIDE(1) FC_SIM_WIDE(2) FC_SIM_WIDE(3) FC_SIM_WIDE(4)
        FC_SIM_WIDE(5) FC_SIM_WIDE(6) FC_SIM_WIDE(7) FC_SIM_WIDE(8)
    default: return hipErrorInvalidValue;
    }
#undef FC_SIM_WIDE
}

hipError_t launch_wide_codec(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems, int group,
                             void *y_f16, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    if constexpr (CODEC == kFp8) {
        return (bits_rs == 8 && bits_ag == 8) ? launch_wide_bits<8, 8>(x, n_src, n_elems, group, y, stream)
                                              : hipErrorInvalidValue;
    } else {
        if (bits_rs == 4)
            return bits_ag == 4 ? launch_wide_bits<4, 4>(x, n_src, n_elems, group, y, stream)
                                : launch_wide_bits<4, 8>(x, n_src, n_elems, group, y, stream);
        return bits_ag == 4 ? launch_wide_bits<8, 4>(x, n_src, n_elems, group, y, stream)
                            : launch_wide_bits<8, 8>(x, n_src, n_elems, group, y, stream);
    }
}

}  // namespace

#define FC_SIM_WIDE_NAME(name)                                                                                       \
    hipError_t launch_allreduce_wide_##name(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems, \
                                            int group, void *y_f16, hipStream_t stream)                              \
    {                                                                                                                \
        return launch_wide_codec(bits_rs, bits_ag, x_f16, n_src, n_elems, group, y_f16, stream);                     \
    }
#if FC_SIM_CODEC == 0
FC_SIM_WIDE_NAME(asym)
#elif FC_SIM_CODEC == 1
FC_SIM_WIDE_NAME(sym)
#elif FC_SIM_CODEC == 2
FC_SIM_WIDE_NAME(fp8)
#else
FC_SIM_WIDE_NAME(cmeta)
#endif
#undef FC_SIM_WIDE_NAME

}  // namespace fc
