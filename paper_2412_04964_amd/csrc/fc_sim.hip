// fc_sim.hip -- Algorithm 1 in ONE launch for volumes that memory bandwidth bounds.
//
// The paper's design is a single fused kernel around its two exchanges (Section 3.2.3, "Kernel Design").  On one
// device the exchanges are the identity, and the counterpart is a kernel that reads the N binary16 partials once and
// writes the binary16 result once: FinegrainedQuantize of every partial (Eq. 1-2), Dequantize and ReduceSum in
// source order, FinegrainedQuantize of the sum with the second bit-width and the final Dequantize all happen in
// registers, and no code, scale or zero-point travels through HBM.  Per output element that is 2 N + 2 bytes
// instead of the 2 N + 2 (N + 1) (b/8 + 8/g) + ... of the three-kernel sequence: 10 against 15.6 bytes at N = 4,
// INT4, g = 128.  Every rounding of the three-kernel sequence is kept, so the result is bit-identical to
// fc_quantize x N -> fc_dequant_reduce_requant -> fc_dequantize.
//
// Arithmetic, and why the shortcuts are exact:
//  * first quantization (binary16 input): s, 1/s and z come from group_params, the function the stand-alone
//    quantizer uses.  With t = rint(x * (1/s)) the code is q = clamp(t + z, 0, qmax) and Dequantize forms q - z.
//    For binary16 inputs z and t are integers below 2^20 (|z| <= 2^11 * 255), so both additions are exact and
//    q - z = clamp(t, -z, qmax - z): one median-of-three.  x * (1/s) is evaluated as a mixed-precision
//    multiply-add with a +0 addend straight from the binary16 value (widening is exact; adding +0 changes only the
//    sign of a zero product); the sign of a zero difference cannot reach the result, because the sum
//    acc = fma(q - z, s, acc) starts at +0 and a round-to-nearest sum is -0 only if both terms are.
//  * the group's min and max are taken on the binary16 pairs (packed min / max are exact in any format) and widened
//    afterwards; whether a zero minimum is +0 or -0 does not matter to Eq. 1 (the range, |min| and 0 - rint(min/s)
//    are the same).
//  * second quantization (fp32 sums) and final Dequantize: literally Eq. 2 and its inverse in fp32, because the
//    zero-point of a sum can be any fp32 integer: u = rint(acc * (1/s')) + z', q = clamp(u, 0, qmax),
//    y = half((q - z') * s').
//
//  * the other quantizers (one translation unit per quantizer, selected by FC_SIM_CODEC).  Symmetric (Eq. 3-4):
//    max|x| of a lane is max(|min|, |max|) of its packed min / max; neither clamp of Eq. 4 can act on a group's own
//    values, so the first stage contributes rint(x * (1/s)) itself, and the second stage adds +0 to its rint so that
//    a code of zero dequantizes to +0 as the stored integer does.  FP8: both stages go through the same conversion
//    instructions as the stand-alone kernels (the format keeps the sign of zero).  Binary16 metadata: group_params
//    rounds the scale and the zero-point as the stored word does; the zero-point stays an integer below 2^17, so
//    the median-of-three form of the first stage remains exact, lower clamp included.
//
// Decomposition: a lane owns 16 consecutive elements (two 128-bit pieces of binary16 per partial), a wavefront
// 1024, a workgroup of two wavefronts 2048; a group of g <= 1024 elements is g/16 adjacent lanes.  The partials come
// through one landing zone of 2 KB per wavefront, in source order, as buffer-to-LDS loads (nothing sits in vector
// registers while in flight): the next partial's loads are issued as soon as this one's data has been read from
// the zone, so they are in flight while it is folded in (DEPTH = 1; = 2: two zones, two partials ahead).  The binary16
// result leaves through the zone as coalesced 1 KB pieces.
//
// What bounds it: HBM, and the number of reads that wait in the memory system at once.  A bare stream of this shape (four
// 128 MB partials read, one written, no arithmetic) takes 99 to 103 us with 48 to 64 KB in flight per compute unit and
// 107 to 111 with 128 KB and more: past what the latency needs, requests only queue and get in each other's way.  Hence one
// partial at a time instead of all N (two where few wavefronts leave the latency uncovered, launch_sim_src), and, for volumes that take
// several rounds of wavefronts, a limit on the workgroups per compute unit (sim_workgroups_per_unit).  4 partials of 8192 x 8192, INT4, group 128, us: all partials at once 109.7,
// one at a time 108.5, with 10 / 9 / 8 / 7 / 6 workgroups per compute unit 108.3 / 106.5 / 103.0 / 102.0 / 107.7.
#include "fc_device.hpp"
#include "fc_launch.hpp"

namespace fc {

constexpr int kSimLaneElems = 16;
constexpr int kSimWaveElems = 64 * kSimLaneElems;
constexpr int kSimBlockThreads = 128;
constexpr int kSimTileElems = kSimBlockThreads * kSimLaneElems;
static_assert(kSimWaveElems == kFusedAllreduceMaxGroup && kSimTileElems == kFusedAllreduceTileElems,
              "the launcher's applicability test describes this decomposition");

template <int CODEC, int BITS_RS, int BITS_AG, int NSRC, int LPG, int DEPTH>
__global__ __launch_bounds__(kSimBlockThreads) void k_allreduce_fused(const uint16_t *__restrict__ x, int64_t n_elems,
                                                                     int lpg, uint16_t *__restrict__ y)
{
    constexpr int E = kSimLaneElems;
    constexpr int kZone = E * 2 * 64;                                  // bytes of one partial per wavefront: 2 KB
    constexpr int kWaves = kSimBlockThreads / 64;
    constexpr bool HM = CODEC == kAsymH;
    static_assert(DEPTH >= 1 && DEPTH <= NSRC && 2 * (DEPTH - 1) <= kMaxCountedVmem,
                  "landing-zone waits count the loads of the later sources");
    static_assert(CODEC != kFp8 || (BITS_RS == 8 && BITS_AG == 8), "E4M3 codes are bytes");
    __shared__ __attribute__((aligned(16))) uint8_t landing[kWaves][DEPTH][kZone];

    const u32 tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const u32 tile = xcd_tile<xcd_chunk(kSimTileElems * 2)>((u32)((n_elems + kSimTileElems - 1) / kSimTileElems));
    const int64_t e_tile = (int64_t)tile * kSimTileElems;
    const int64_t left = (n_elems - e_tile) * 2;                       // bytes from the tile to the end of a partial

    auto fetch = [&](int j) {
        const rsrc_t rx = make_rsrc(x + (int64_t)j * n_elems + e_tile, left);
        dma_piece(rx, wave * kZone + lane * 16, &landing[wave][j % DEPTH][0]);
        dma_piece(rx, wave * kZone + 1024 + lane * 16, &landing[wave][j % DEPTH][1024]);
    };
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) fetch(j);
    issue_order_fence();

    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < NSRC; ++j) {
        // source j has landed once no more than the loads of the later sources are outstanding
        wait_vmem_outstanding(2 * ((NSRC < j + DEPTH ? NSRC : j + DEPTH) - 1 - j));
        u32x4 a0 = lds_read_b128_issue(&landing[wave][0][lane * (E * 2)], j % DEPTH * kZone);
        u32x4 a1 = lds_read_b128_issue(&landing[wave][0][lane * (E * 2)], j % DEPTH * kZone + 16);
        lds_read_complete(a0);
        lds_read_complete(a1);
        // the zone has been read: it takes the next source but DEPTH - 1
        if (j + DEPTH < NSRC) fetch(j + DEPTH);
        issue_order_fence();
        const h2 p[8] = {as_h2(a0[0]), as_h2(a0[1]), as_h2(a0[2]), as_h2(a0[3]),
                         as_h2(a1[0]), as_h2(a1[1]), as_h2(a1[2]), as_h2(a1[3])};
        h2 lo = pk_min(p[0], p[1]), hi = pk_max(p[0], p[1]);
#pragma unroll
        for (int k = 2; k < 8; ++k) {
            lo = pk_min(lo, p[k]);
            hi = pk_max(hi, p[k]);
        }
        float mn = fminf((float)lo.x, (float)lo.y), mx = fmaxf((float)hi.x, (float)hi.y);
        float s, inv;
        if constexpr (is_asym(CODEC)) {
            group_minmax<LPG>(mn, mx, lpg);
            float zf;
            group_params<BITS_RS, HM>(mn, mx, s, inv, zf);
            const float d_lo = 0.0f - zf, d_hi = (float)((1 << BITS_RS) - 1) - zf;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float t0 = rintf(fmaf((float)p[k].x, inv, 0.0f));
                const float t1 = rintf(fmaf((float)p[k].y, inv, 0.0f));
                acc[2 * k] = fmaf(__builtin_amdgcn_fmed3f(t0, d_lo, d_hi), s, acc[2 * k]);
                acc[2 * k + 1] = fmaf(__builtin_amdgcn_fmed3f(t1, d_lo, d_hi), s, acc[2 * k + 1]);
            }
        } else {
            const float amax = group_max<LPG>(fmaxf(fabsf(mn), fabsf(mx)), lpg);
            if constexpr (CODEC == kSym) {
                group_params_sym<BITS_RS>(amax, s, inv);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    acc[2 * k] = fmaf(rintf(fmaf((float)p[k].x, inv, 0.0f)), s, acc[2 * k]);
                    acc[2 * k + 1] = fmaf(rintf(fmaf((float)p[k].y, inv, 0.0f)), s, acc[2 * k + 1]);
                }
            } else {
                group_params_absmax<448>(amax, s, inv);
                float v[E];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    v[2 * k] = (float)p[k].x;
                    v[2 * k + 1] = (float)p[k].y;
                }
                u32 word[4];
                pack_lane_fp8<E>(v, inv, word);
                accumulate_fp8(word, s, acc);
            }
        }
        pin_values(acc);              // source j is folded in before source j+1 is waited for
    }

    // FinegrainedQuantize of the sums and the final Dequantize: d[i] = the dequantized code before the scale
    float s, inv, d[E];
    if constexpr (is_asym(CODEC)) {
        float mn, mx, zf;
        lane_minmax(acc, mn, mx);
        group_minmax<LPG>(mn, mx, lpg);
        group_params<BITS_AG, HM>(mn, mx, s, inv, zf);
        constexpr float qmax = (float)((1 << BITS_AG) - 1);
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const float u = rintf(acc[i] * inv) + zf;
            d[i] = __builtin_amdgcn_fmed3f(u, 0.0f, qmax) - zf;
        }
    } else {
        const float amax = group_max<LPG>(lane_absmax(acc), lpg);
        if constexpr (CODEC == kSym) {
            group_params_sym<BITS_AG>(amax, s, inv);
#pragma unroll
            for (int i = 0; i < E; ++i) d[i] = rintf(acc[i] * inv) + 0.0f;
        } else {
            group_params_absmax<448>(amax, s, inv);
            u32 word[4];
            pack_lane_fp8<E>(acc, inv, word);
            decode_fp8(word, d);
        }
    }
    u32x4 *mine = reinterpret_cast<u32x4 *>(&landing[wave][0][lane * (E * 2)]);
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
        mine[k] = out;
    }
    const rsrc_t ry = make_rsrc(y + e_tile, left);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const u32x4 o = *reinterpret_cast<const u32x4 *>(&landing[wave][0][k * 1024 + lane * 16]);
        __builtin_amdgcn_raw_buffer_store_b128(o, ry, wave * kZone + k * 1024 + lane * 16, 0, kStreamStorePolicy);
    }
}

#ifndef FC_SIM_CODEC
#error "compile with -DFC_SIM_CODEC=0..3 (kAsym, kSym, kFp8, kAsymH): one translation unit per quantizer"
#endif

namespace {

constexpr int CODEC = FC_SIM_CODEC;

// Workgroups that a compute unit shall hold at once, 0: as many as fit.  From 18 * 2^20 elements per partial on (over four rounds of
// wavefronts) the chip would otherwise have more reads waiting than the memory system serves well.  With few sources more of the
// wavefronts are at the start or the end of their tile, and the limit is higher.  INT4, group 128, us, without a limit and with so many
// workgroups: N = 2  8192 x 8192 63.5, 10: 61.9, 8: 63.2, 7: 66.2; N = 3 86.0, 9: 82.7, 8: 82.0, 7: 85; N = 4 109.5, 8: 103.0, 7: 102.2; N = 5 131.8,
// 8: 126.2, 7: 121.2, 6: 127.8; N = 6 151.8, 148.9, 142.2, 149.3; N = 8 205.4, 196.1, 187.9, 194.3.  N = 4 x 4096: 8 M elements 15.3 / 15.9 with 8,
// 16 M 28.4 / 28.9, 20 M 35.4 / 35.2, 24 M 42.3 / 41.2, 32 M 56.0 / 53.5.  N = 1: no gain from any limit.
// A minimum and a maximum over more than 8 lanes take instructions that fewer wavefronts do not cover: asymmetric, group 512, N = 2
// without / 10: 18 M 20.8 / 21.8, 32 M 34.6 / 35.7, 64 M 66.5 / 67.7 (group 32 66.6 / 66.1, symmetric 66.1 / 64.5); N = 6  8 / 7: 24 M 60.6 / 62.2,
// 40 M 96.7 / 97.6.
int sim_workgroups_per_unit(int n_src, int64_t n_elems, int group)
{
    if (n_src == 1 || n_elems < (int64_t)18 << 20) return 0;
    const bool more = is_asym(CODEC) && group > 128;
    if (n_src == 2) return more ? 0 : 10;
    return n_src <= 4 || (n_src == 6 && more) ? 8 : 7;
}

template <int BITS_RS, int BITS_AG, int NSRC>
hipError_t launch_sim_src(const uint16_t *x, int64_t n_elems, int group, uint16_t *y, hipStream_t stream)
{
    const dim3 grid((unsigned)((n_elems + kSimTileElems - 1) / kSimTileElems)), block(kSimBlockThreads);
    const int lpg = group / kSimLaneElems;
    // Less than two rounds of wavefronts: a wavefront's chain of loads bounds the call, two at a time shorten it.  us, group 128, all
    // at once / one / two at a time: INT4 N = 2 (two are all)  3.5 M elements 4.81 / 5.08;  N = 3  2.5 M 5.00 / 5.41 / 4.90;  N = 4  2.5 M 6.14 /
    // 6.27 / 5.82;  N = 6  2 M 6.95 / 6.97 / 5.95;  N = 8  1.25 M 6.84 / 7.24 / 6.57   3 M 13.97 / 10.73 / 10.36   4 M 16.69 / 12.99 / 13.35;  symmetric
    // N = 4  1.75 M 4.38 / 4.87 / 4.02;  binary16 metadata N = 2  3.5 M 4.87 / 5.50;  N = 3  3.5 M 6.31 / 6.57 / 6.30;  N = 4  1.75 M 4.76 / 5.30 / 4.68   3 M 6.90 /
    // 7.38 / 6.83.  Where the buffers are not cached (700 MB of them) one at a time is up to 8 % faster with two or three sources; where two sets of them
    // stay in the caches two at a time go on to win: symmetric N = 2  4 M 4.78 / 4.26, binary16 metadata N = 2  5 M 6.49 / 6.07, N = 4  3.5 M 7.60 / 7.03.
    if constexpr (NSRC >= 2)
        if (n_elems <= (int64_t)(NSRC == 2 ? 10 : NSRC == 3 ? 8 : NSRC == 4 ? 7 : 6) << 19)
            return lpg == 8 ? launch_kernel(k_allreduce_fused<CODEC, BITS_RS, BITS_AG, NSRC, 8, 2>, grid, block, stream, x,
                                            n_elems, lpg, y)
                            : launch_kernel(k_allreduce_fused<CODEC, BITS_RS, BITS_AG, NSRC, 0, 2>, grid, block, stream, x,
                                            n_elems, lpg, y);
    const size_t pad = lds_to_limit(sim_workgroups_per_unit(NSRC, n_elems, group), kSimTileElems * 2);
    if (lpg == 8)                                                      // g = 128: the lane pattern is a constant
        return launch_kernel_lds(k_allreduce_fused<CODEC, BITS_RS, BITS_AG, NSRC, 8, 1>, grid, block, pad, stream, x, n_elems,
                                 lpg, y);
    return launch_kernel_lds(k_allreduce_fused<CODEC, BITS_RS, BITS_AG, NSRC, 0, 1>, grid, block, pad, stream, x, n_elems, lpg, y);
}

template <int BITS_RS, int BITS_AG>
hipError_t launch_sim_bits(const uint16_t *x, int n_src, int64_t n_elems, int group, uint16_t *y, hipStream_t stream)
{
    switch (n_src) {
    case 1: return launch_sim_src<BITS_RS, BITS_AG, 1>(x, n_elems, group, y, stream);
    case 2: return launch_sim_src<BITS_RS, BITS_AG, 2>(x, n_elems, group, y, stream);
    case 3: return launch_sim_src<BITS_RS, BITS_AG, 3>(x, n_elems, group, y, stream);
    case 4: return launch_sim_src<BITS_RS, BITS_AG, 4>(x, n_elems, group, y, stream);
    case 5: return launch_sim_src<BITS_RS, BITS_AG, 5>(x, n_elems, group, y, stream);
    case 6: return launch_sim_src<BITS_RS, BITS_AG, 6>(x, n_elems, group, y, stream);
    case 7: return launch_sim_src<BITS_RS, BITS_AG, 7>(x, n_elems, group, y, stream);
    case 8: return launch_sim_src<BITS_RS, BITS_AG, 8>(x, n_elems, group, y, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sim_codec(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems, int group,
                            void *y_f16, hipStream_t stream)
{
    const uint16_t *x = static_cast<const uint16_t *>(x_f16);
    uint16_t *y = static_cast<uint16_t *>(y_f16);
    if constexpr (CODEC == kFp8) {
        return (bits_rs == 8 && bits_ag == 8) ? launch_sim_bits<8, 8>(x, n_src, n_elems, group, y, stream)
                                              : hipErrorInvalidValue;
    } else {
        if (bits_rs == 4)
            return bits_ag == 4 ? launch_sim_bits<4, 4>(x, n_src, n_elems, group, y, stream)
                                : launch_sim_bits<4, 8>(x, n_src, n_elems, group, y, stream);
        return bits_ag == 4 ? launch_sim_bits<8, 4>(x, n_src, n_elems, group, y, stream)
                            : launch_sim_bits<8, 8>(x, n_src, n_elems, group, y, stream);
    }
}

}  // namespace

#if FC_SIM_CODEC == 0
hipError_t launch_allreduce_fused_asym(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems,
                                       int group, void *y_f16, hipStream_t stream)
{
    return launch_sim_codec(bits_rs, bits_ag, x_f16, n_src, n_elems, group, y_f16, stream);
}
#elif FC_SIM_CODEC == 1
hipError_t launch_allreduce_fused_sym(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems,
                                      int group, void *y_f16, hipStream_t stream)
{
    return launch_sim_codec(bits_rs, bits_ag, x_f16, n_src, n_elems, group, y_f16, stream);
}
#elif FC_SIM_CODEC == 2
hipError_t launch_allreduce_fused_fp8(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems,
                                      int group, void *y_f16, hipStream_t stream)
{
    return launch_sim_codec(bits_rs, bits_ag, x_f16, n_src, n_elems, group, y_f16, stream);
}
#else
hipError_t launch_allreduce_fused_cmeta(int bits_rs, int bits_ag, const void *x_f16, int n_src, int64_t n_elems,
                                        int group, void *y_f16, hipStream_t stream)
{
    return launch_sim_codec(bits_rs, bits_ag, x_f16, n_src, n_elems, group, y_f16, stream);
}
#endif

}  // namespace fc
