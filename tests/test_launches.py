"""Which kernel a call launches, and with what grid, on both sides of the limits of the dispatch.  Nothing runs: see launches.py.  That the
kernels on both sides agree with the oracle is what the GPU tests check."""
import pytest

from launches import allreduce, allreduce_rot, dequantize, dequantize_rot, fused, launches, quantize, quantize_rot

M = 1 << 20


def kernels(*calls):
    """the kernels of each call, which has to succeed"""
    out = []
    for call, (rc, seen) in zip(calls, launches(calls)):
        assert rc == 0 and seen, "%s %s: %d %s" % (*call, rc, seen)
        out.append([s[0] for s in seen])
    return out


@pytest.mark.parametrize("quantizer", ["asym", "sym", "cmeta"])
@pytest.mark.parametrize("group", [32, 64, 128, 256, 512, 1024, 4096, 16384])
def test_the_largest_4_bit_volume_is_launched(quantizer, group):
    # 2^36 elements: 2^31 threads with 32 elements each, while 16 each would be 2^32, which the runtime refuses
    for call in (quantize(quantizer, 1 << 36, group, 4), dequantize(quantizer, 1 << 36, group, 4), fused(quantizer, 2, 1 << 36, group, 4, 4)):
        (rc, seen), = launches([call])
        assert rc == 0 and len(seen) == 1, "%s: %d %s" % (call[0], rc, seen)


def forms(make, limits):
    """limits: [(what make takes, elements, the kernel's beginning up to there, the beginning above)].  One row of 8192 is one step"""
    calls = [make(*what, elems) for what, limit, _, _ in limits for elems in (limit, limit + 8192)]
    got = kernels(*calls)
    for (what, limit, upto, above), a, b in zip(limits, got[::2], got[1::2]):
        assert a[0].startswith(upto) and b[0].startswith(above), "%s at %.2f M elements: %s, then %s" % (what, limit / M, a, b)


def test_quantizer_forms():
    # 8 elements per lane; 16 in workgroups of 256; 16 in workgroups of 64; 32
    forms(lambda q, bits, group, elems: quantize(q, elems, group, bits), [
        (("asym", 4, 128), 7 * M // 2, "k_quantize_small<4,0,0>", "k_quantize<4,8,0,16,256>"), (("asym", 4, 128), 8 * M, "k_quantize<4,8,0,16,256>", "k_quantize<4,8,0,16,64>"),
        (("sym", 4, 32), 4 * M, "k_quantize_small<4,1,0>", "k_quantize<4,2,1,16,256>"), (("cmeta", 4, 64), 8 * M, "k_quantize<4,4,3,16,256>", "k_quantize<4,4,3,16,64>"),
        (("asym", 4, 256), 5 * M // 2, "k_quantize_small<4,0,0>", "k_quantize<4,8,0,32,128>"), (("asym", 4, 256), 36 * M - 8192, "k_quantize<4,8,0,32,128>", "k_quantize<4,0,0,16,64>"),
        (("sym", 4, 512), 36 * M - 8192, "k_quantize<4,0,1,32,256>", "k_quantize<4,0,1,16,64>"), (("asym", 4, 1024), 3 * M // 2, "k_quantize_small<4,0,1>", "k_quantize<4,0,0,32,256>"),
        (("cmeta", 4, 1024), 36 * M - 8192, "k_quantize<4,0,3,32,256>", "k_quantize<4,0,3,16,64>"), (("asym", 4, 2048), 3 * M, "k_quantize_small<4,0,1>", "k_quantize<4,0,0,32,256>"),
        (("sym", 4, 2048), 3 * M // 2, "k_quantize_small<4,1,1>", "k_quantize<4,0,1,32,256>"), (("sym", 4, 8192), 2 * M, "k_quantize_small<4,1,1>", "k_quantize_wide<4,1,1,256>"),
        (("asym", 8, 512), 3 * M // 2, "k_quantize_small<8,0,0>", "k_quantize<8,0,0,16,256>"), (("asym", 8, 1024), M, "k_quantize_small<8,0,1>", "k_quantize<8,0,0,16,256>"),
        (("sym", 8, 256), M, "k_quantize_small<8,1,0>", "k_quantize<8,0,1,16,256>"), (("fp8", 8, 1024), M, "k_quantize_small<8,2,1>", "k_quantize<8,0,2,16,256>"),
        (("sym", 8, 2048), 2 * M, "k_quantize_small<8,1,1>", "k_quantize_wide<8,1,1,128>")])


def test_wide_quantizer_leaves_room_at_large_volumes():
    # LDS beyond the kernel's own limits the workgroups per compute unit, 4-bit codes in groups of 4096 from 36 * 2^20 elements on
    for quantizer, bits, elems, limited in (("asym", 4, 36 * M, True), ("sym", 4, 64 * M, True), ("cmeta", 4, 36 * M - 8192, False), ("asym", 8, 64 * M, False)):
        (rc, seen), = launches([quantize(quantizer, elems, 16384 // bits, bits)])
        assert rc == 0 and seen[0][0].startswith("k_quantize_wide<%d,1" % bits) and seen[0][2] == 128
        room = 160 * 1024 // (seen[0][3] + 128 * (128 // bits) * 2 + 16)
        assert (room == 10) == limited, "%s %d bits, %d elements: %d" % (quantizer, bits, elems, room)


def test_dequantizer_forms():
    forms(lambda q, group, elems: dequantize(q, elems, group, 4), [
        (("asym", 32), 8 * M, "k_dequantize<4,0,16>", "k_dequantize<4,0,32>"), (("sym", 128), 5 * M, "k_dequantize<4,1,16>", "k_dequantize<4,1,32>"),
        (("cmeta", 8192), 5 * M, "k_dequantize<4,3,16>", "k_dequantize<4,3,32>")])
    for elems, limited in ((48 * M - 8192, False), (48 * M, True)):
        (rc, seen), = launches([dequantize("sym", elems, 128, 4)])
        assert rc == 0 and (seen[0][3] > 0) == limited


def test_partials_in_flight():
    # the last template argument: two at a time up to 10 to 6 * 2^19 elements, one at a time above
    forms(lambda q, n_src, group, elems: allreduce(q, n_src, elems, group, 8, 8), [
        (("asym", 2, 128), 5 * M, "k_allreduce_fused<0,8,8,2,8,2>", "k_allreduce_fused<0,8,8,2,8,1>"),
        (("cmeta", 3, 32), 4 * M, "k_allreduce_fused<3,8,8,3,0,2>", "k_allreduce_fused<3,8,8,3,0,1>"),
        (("sym", 4, 128), 7 * M // 2, "k_allreduce_fused<1,8,8,4,8,2>", "k_allreduce_fused<1,8,8,4,8,1>"),
        (("fp8", 8, 512), 3 * M, "k_allreduce_fused<2,8,8,8,0,2>", "k_allreduce_fused<2,8,8,8,0,1>")])
    assert kernels(allreduce("asym", 1, 2 * M, 128)) == [["k_allreduce_fused<0,8,8,1,8,1>"]]


def test_all_reduce_workgroups_per_compute_unit():
    # 4 KB of LDS of the kernel's own; what the launch asks for beyond that leaves room for so many in 160 KB (0: asks for nothing)
    cases = [("asym", 2, 18 * M, 128, 10), ("asym", 2, 18 * M, 512, 0), ("cmeta", 2, 64 * M, 256, 0), ("sym", 2, 64 * M, 512, 10), ("asym", 4, 18 * M, 512, 8),
             ("asym", 6, 24 * M, 512, 8), ("asym", 6, 24 * M, 128, 7), ("fp8", 6, 24 * M, 512, 7), ("asym", 8, 24 * M, 512, 7), ("asym", 3, 18 * M - 8192, 128, 0)]
    for case, (rc, seen) in zip(cases, launches([allreduce(q, n, elems, g) for q, n, elems, g, _ in cases])):
        assert rc == 0 and seen[0][0].startswith("k_allreduce_fused")
        assert (160 * 1024 // (seen[0][3] + 4096) if seen[0][3] else 0) == case[-1], "%s %s" % (case, seen)


def test_all_reduce_of_wide_groups():
    # which kernel takes groups of 1024, and where the wide one leaves room
    forms(lambda q, n, group, elems: allreduce(q, n, elems, group, 8, 8), [
        (("sym", 1, 1024), M, "k_allreduce_wide<1", "k_allreduce_fused<1"), (("fp8", 3, 1024), 3 * M // 2, "k_allreduce_wide<2", "k_allreduce_fused<2"),
        (("asym", 4, 1024), 4 * M, "k_allreduce_wide<0", "k_allreduce_fused<0"), (("cmeta", 1, 1024), 4 * M, "k_allreduce_wide<3", "k_allreduce_fused<3")])
    cases = [("asym", 2, 20 * M - 8192, 2048, False), ("sym", 2, 20 * M, 2048, True), ("asym", 2, 64 * M, 1024, False), ("fp8", 2, 64 * M, 8192, False),
             ("cmeta", 2, 20 * M, 4096, True), ("asym", 3, 14 * M - 8192, 4096, False), ("asym", 3, 14 * M, 8192, True), ("asym", 4, 12 * M, 1024, True),
             ("sym", 8, 12 * M, 2048, True), ("sym", 8, 12 * M - 8192, 2048, False), ("asym", 1, 64 * M, 2048, False)]
    for case, (rc, seen) in zip(cases, launches([allreduce(q, n, elems, g) for q, n, elems, g, _ in cases])):
        assert rc == 0 and seen[0][0].startswith("k_allreduce_wide") and (seen[0][3] > 0) == case[-1], "%s %s" % (case, seen)


def test_fused_step_forms():
    # the launch-bound kernel up to 1024 wavefronts times 2 to 6, by quantizer, code widths and fan-in
    small, bulk = "k_fused_small<", "k_dequant_reduce_requant"
    forms(lambda q, n, group, b, elems: fused(q, n, elems, group, *b), [
        (("asym", 2, 128, (4, 4)), 5 * M // 2, small, bulk), (("asym", 2, 32, (4, 8)), 2 * M, small, bulk), (("asym", 4, 128, (4, 8)), 2 * M, small, bulk),
        (("asym", 5, 128, (4, 8)), 5 * M // 2, small, bulk), (("cmeta", 3, 256, (4, 8)), 3 * M // 2, small, bulk), (("cmeta", 3, 256, (4, 4)), 2 * M, small, bulk),
        (("cmeta", 8, 128, (4, 8)), 2 * M, small, bulk), (("sym", 2, 128, (4, 8)), 3 * M, small, bulk), (("sym", 4, 32, (8, 4)), 3 * M // 2, small, bulk),
        (("fp8", 4, 256, ()), 5 * M // 4, small, bulk), (("asym", 1, 128, (8, 8)), 3 * M // 4, small, bulk), (("asym", 8, 8192, (8, 8)), 7 * M // 2, small, "k_dequant_reduce_requant_wide<")])
    # the rule that test_fused_at_the_limit_of_the_launch_bound_kernel works with
    for name, pairs in (("sym", ((4, 4), (4, 8), (8, 4), (8, 8))), ("cmeta", ((4, 4), (4, 8), (8, 4), (8, 8))), ("fp8", ((8, 8),))):
        for n in (1, 2, 3, 4, 5, 8):
            for (bits_in, bits_out), lanes in [(p, l) for p in pairs for l in (16, 32)]:
                waves = 3 if n == 1 and bits_in == 8 else 2 if n == 1 else (6 if lanes < 32 else 5) if bits_in == 8 else 6 if name == "sym" else 3 if bits_out == 8 and n <= 4 else 4
                limit = waves * 1024 * (2048 // bits_in)
                a, b = kernels(*[fused(name, n, elems, lanes * 32 // bits_in, bits_in, bits_out) for elems in (limit, limit + 1024)])
                assert a[0].startswith(small) and b[0].startswith(bulk), "%s N=%d %d>%d %d lanes: %s, then %s" % (name, n, bits_in, bits_out, lanes, a, b)
    got = kernels(fused("sym", 2, M // 16, 1024), fused("fp8", 2, M // 16, 1024), fused("asym", 2, M // 16, 1024), fused("sym", 3, M // 16, 1024), fused("sym", 2, M // 16, 2048))
    assert [k[0].startswith(small) for k in got] == [False, False, True, True, True], got


def test_rotated_codec_forms():
    fine, rows, registers = "k_quantize_rot_fine<", "k_quantize_rot_rows<", "k_quantize_rot<"
    def block(q, bits, hidden, elems):
        return quantize_rot(q, elems // hidden * hidden, hidden, 128, bits)
    def both(cases):
        calls = [block(q, bits, hidden, elems) for q, bits, hidden, limit, _, _ in cases for elems in (limit, limit + hidden)]
        got = kernels(*calls)
        for (q, bits, hidden, limit, upto, above), a, b in zip(cases, got[::2], got[1::2]):
            assert a[0].startswith(upto) and b[0].startswith(above), "%s %d bits h=%d %.2f M: %s, then %s" % (q, bits, hidden, limit / M, a, b)
    both([("asym", 4, 1024, 5 * M // 4, fine, rows), ("sym", 4, 1024, 2 * M, rows, registers), ("asym", 8, 5120, 5 * M // 4, fine, rows), ("sym", 8, 1024, 2 * M, rows, registers),
          ("asym", 4, 2048, 3 * M // 2, fine, registers), ("sym", 8, 2048, M, fine, rows), ("asym", 8, 2048, 2 * M, rows, registers), ("fp8", 8, 2048, M, fine, rows),
          ("fp8", 8, 2048, 4 * M, rows, registers), ("asym", 4, 4096, M, fine, registers), ("sym", 8, 4096, M, fine, registers), ("fp8", 8, 4096, 4 * M, rows, registers),
          ("fp8", 8, 8192, M, registers, registers), ("asym", 4, 8192, M, registers, registers)])
    got = kernels(*[dequantize_rot(q, elems, hidden, 128, bits) for q, bits, hidden, elems in
                    (("asym", 4, 2048, 2 * M), ("asym", 4, 2048, 2 * M + 2048), ("sym", 8, 8192, M), ("sym", 8, 8192, M + 8192), ("asym", 8, 1024, 2 * M), ("fp8", 8, 1024, 3 * M))])
    assert [k[0].split("<")[0] for k in got] == ["k_dequantize_rot" + s for s in ("_fine", "", "_fine", "", "_rows", "")]


def test_rotated_all_reduce_in_steps():
    # the last volume in steps and the next one, by code, block and number of sources: where the one launch has all sources at once, and
    # where it would take them in turn
    at_once = [("asym", 4, 2048, 8, 2), ("fp8", 8, 2048, 5, 3), ("asym", 4, 4096, 3, 4), ("sym", 4, 4096, 4, 4), ("asym", 4, 4096, 5, 8), ("sym", 8, 4096, 6, 8), ("asym", 4, 4096, 7, 10),
               ("fp8", 8, 4096, 3, 6), ("fp8", 8, 4096, 5, 9), ("asym", 4, 8192, 4, 10), ("asym", 8, 8192, 4, 8), ("fp8", 8, 8192, 3, 8), ("fp8", 8, 8192, 4, 16), ("asym", 4, 8192, 6, 32),
               ("sym", 8, 8192, 6, 30), ("asym", 4, 8192, 7, 30), ("asym", 4, 8192, 8, 25), ("sym", 8, 8192, 8, 22), ("fp8", 8, 8192, 7, 28)]
    in_turn = [("asym", 4, 1024, 5, 30), ("asym", 4, 1024, 8, 30), ("sym", 8, 1024, 6, 20), ("asym", 8, 1024, 7, 22), ("fp8", 8, 1024, 5, 33), ("asym", 4, 2048, 6, 37), ("asym", 8, 2048, 8, 25),
               ("fp8", 8, 2048, 7, 33), ("asym", 4, 4096, 5, 38), ("sym", 8, 4096, 6, 32), ("fp8", 8, 4096, 4, 44), ("fp8", 8, 4096, 8, 45), ("asym", 4, 8192, 5, 32), ("sym", 8, 8192, 5, 30),
               ("asym", 4, 8192, 8, 38), ("fp8", 8, 8192, 6, 38)]
    cases = at_once + in_turn
    got = kernels(*[allreduce_rot(q, n, elems, h, 128, b, b) for q, b, h, n, limit in cases for elems in (limit << 16, (limit << 16) + h)])
    for case, a, b in zip(cases, got[::2], got[1::2]):
        assert len(a) == 2 and a[1].startswith("k_reduce_rot_fine") and len(b) == 1, "%s: %s, then %s" % (case, a, b)
    # all sources at once up to a volume, and in steps past it
    cases = [("asym", 4, 2048, 6, M), ("sym", 8, 2048, 7, M), ("fp8", 8, 1024, 8, M), ("asym", 4, 2048, 5, 3 * M // 2), ("fp8", 8, 1024, 5, 3 * M // 2), ("asym", 4, 4096, 5, M), ("fp8", 8, 4096, 8, M),
             ("fp8", 8, 4096, 4, 2 * M), ("asym", 4, 8192, 8, 2 * M), ("fp8", 8, 8192, 7, 2 * M)]
    got = kernels(*[allreduce_rot(q, n, elems, h, 128, b, b) for q, b, h, n, limit in cases for elems in (limit, limit + h)])
    for case, a, b in zip(cases, got[::2], got[1::2]):
        assert len(a) == 1 and len(b) == 2, "%s: %s, then %s" % (case, a, b)
    # coarse groups: the first limit lies 2^17 elements lower up to eight, six, four sources; padded slabs of blocks of 1024 never
    cases = [("asym", 4, 4096, 7, 10), ("asym", 4, 4096, 6, 6), ("fp8", 8, 2048, 8, 1), ("asym", 4, 8192, 4, 8), ("asym", 4, 8192, 8, 25)]
    got = kernels(*[allreduce_rot(q, n, elems, h, 1024, b, b) for q, b, h, n, limit in cases for elems in (limit << 16, (limit << 16) + h)])
    assert [len(k) for k in got] == [2, 1] * len(cases), got
    assert [len(k) for k in kernels(allreduce_rot("asym", 8, M + 3 * 1024, 1024, 1024, 4, 4), allreduce_rot("asym", 8, M + 4 * 1024, 1024, 1024, 4, 4))] == [1, 2]


def test_rotated_all_reduce_in_one_launch():
    # all sources at once with 8 elements per lane; side by side; one after the other
    fine, spread, plain = "k_allreduce_rot_fine<", "k_allreduce_rot_spread<", "k_allreduce_rot<"
    cases = [("asym", 1, 1024, 5 * M // 4, fine, plain), ("sym", 1, 2048, 3 * M // 2, fine, plain), ("fp8", 1, 4096, 2 * M, fine, plain), ("asym", 2, 1024, 3 * M // 4, fine, spread),
             ("asym", 2, 2048, M, fine, spread), ("fp8", 2, 4096, M, fine, spread), ("sym", 3, 1024, M // 2, fine, spread), ("asym", 2, 8192, 2 * M, spread, plain), ("sym", 3, 4096, 2 * M, spread, plain),
             ("asym", 5, 8192, 31 * M // 16, plain, plain), ("sym", 6, 8192, 2 * M, spread, plain)]
    got = kernels(*[allreduce_rot(q, n, elems, h, 128, 8, 8) for q, n, h, limit, _, _ in cases for elems in (limit, limit + h)])
    for case, a, b in zip(cases, got[::2], got[1::2]):
        assert len(a) == len(b) == 1 and a[0].startswith(case[4]) and b[0].startswith(case[5]), "%s: %s, then %s" % (case, a, b)
