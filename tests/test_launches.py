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
