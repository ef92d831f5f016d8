"""The fused step's cases once more at volumes past every limit of its launch-bound kernel (at most 6144 wavefronts of 512
four-bit elements, 3 * 2^20, or 7 * 2^19 in groups of 8192), where the bulk kernels take them; and both kernels on the two sides of each limit.  Run with
``-m gpu`` on an MI355X."""
import numpy as np
import pytest

import oracle
import test_gpu_parity
from test_gpu_parity import (Guarded, dev, fc, test_fused_adversarial_sums, test_fused_arbitrary_scales_and_zero_points,  # noqa: F401
                             test_fused_extreme_scales, test_fused_matches_oracle, test_fused_scales_around_the_exponent_limit,
                             test_fused_source_stride_with_padding, test_upper_clamp_is_exercised)
from test_gpu_parity_abi import (plain_lib, test_fused_with_odd_metadata_strides,                                         # noqa: F401
                                 test_hand_ordered_and_plain_landing_reads_agree_with_the_oracle)
from test_gpu_small_variants import PAIRS, test_fused_small_and_bulk, wire                                                # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def volumes_past_the_limit(monkeypatch):
    monkeypatch.setattr(test_gpu_parity, "BULK_ELEMS", 9 << 19)


@pytest.mark.parametrize("name", ["asym"] + list(PAIRS))
@pytest.mark.parametrize("n_src", [1, 2, 3, 4, 6, 8])
def test_fused_on_both_sides_of_every_limit(fc, name, n_src):
    # 1024 wavefronts and up to six times as many, by quantizer, code width, fan-in and the lanes of a group; rows do not depend on each other
    t, h = 7, 4096
    sfx = "" if name == "asym" else "_" + name
    pairs = [(4, 4), (4, 8), (8, 4), (8, 8)] if name == "asym" else PAIRS[name]
    for bits_in, bits_out in pairs:
        for lanes in (16, 32):
            g = lanes * 32 // bits_in
            bits = () if name == "fp8" else (bits_in, bits_out)
            if name == "asym":
                x = test_gpu_parity.synth_inputs.make_partials_stress(n_src, t, h, n_src % 6, seed=lanes + n_src)
                few = [np.stack(p) for p in zip(*[oracle.quantize(x[j], g, bits_in) for j in range(n_src)])]
            else:
                few = list(wire(name, n_src, t, h, g, bits_in, seed=lanes + n_src))
            want = [dev(np.ascontiguousarray(a).view(np.uint8))
                    for a in getattr(oracle, "dequant_reduce_requant" + sfx)(*few, h, g, *bits)]
            few = [dev(a.view(np.int32)) if a.dtype == np.uint32 else dev(a) for a in few]
            for k in (2, 3, 4, 5, 6):
                limit = k * 1024 * (2048 // bits_in) // h
                for rows in (limit, limit + 1):
                    pick = torch.arange(rows, device="cuda") % t
                    outs = [Guarded((rows, h * bits_out // 8), torch.uint8)]
                    outs += [Guarded((rows, h // g), few[1].dtype) for _ in few[1:]]
                    getattr(fc, "dequant_reduce_requant" + sfx)(*[w[:, pick] for w in few], h, g, *bits, out=tuple(o.t for o in outs))
                    torch.cuda.synchronize()
                    for got, w in zip(outs, want):
                        got.check()
                        assert torch.equal(got.t.view(torch.uint8), w[pick]), "%s N=%d g=%d %d->%d rows=%d" % (
                            name, n_src, g, bits_in, bits_out, rows)


@pytest.mark.parametrize("name", ["asym"] + list(PAIRS))
@pytest.mark.parametrize("n_src", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("bits_in, group, limits", [(4, 1024, (3 << 18, 3 << 19, 2 << 20)), (4, 4096, (3 << 18, 3 << 19, 2 << 20)),
                                                    (8, 512, (1 << 17, 1 << 18)), (8, 2048, (1 << 17, 1 << 18)), (8, 8192, (2 << 20, 7 << 19))])
def test_fused_groups_of_several_wavefronts(fc, name, n_src, bits_in, group, limits):
    # a group that is a workgroup up to these volumes, the bulk kernels' above them
    t, h = 7, max(4096, group)
    sfx = "" if name == "asym" else "_" + name
    for bits_out in (4, 8):
        if name != "asym" and (bits_in, bits_out) not in PAIRS[name]:
            continue
        bits = () if name == "fp8" else (bits_in, bits_out)
        if name == "asym":
            x = test_gpu_parity.synth_inputs.make_partials_stress(n_src, t, h, n_src % 6, seed=group + n_src)
            few = [np.stack(p) for p in zip(*[oracle.quantize(x[j], group, bits_in) for j in range(n_src)])]
        else:
            few = list(wire(name, n_src, t, h, group, bits_in, seed=group + n_src))
        want = [dev(np.ascontiguousarray(a).view(np.uint8))
                for a in getattr(oracle, "dequant_reduce_requant" + sfx)(*few, h, group, *bits)]
        few = [dev(a.view(np.int32)) if a.dtype == np.uint32 else dev(a) for a in few]
        for rows in {1, 3} | {limit // h + more for limit in limits for more in (0, 1)}:
            pick = torch.arange(rows, device="cuda") % t
            outs = [Guarded((rows, h * bits_out // 8), torch.uint8)]
            outs += [Guarded((rows, h // group), few[1].dtype) for _ in few[1:]]
            getattr(fc, "dequant_reduce_requant" + sfx)(*[w[:, pick] for w in few], h, group, *bits, out=tuple(o.t for o in outs))
            torch.cuda.synchronize()
            for got, w in zip(outs, want):
                got.check()
                assert torch.equal(got.t.view(torch.uint8), w[pick]), "%s N=%d g=%d %d->%d rows=%d" % (
                    name, n_src, group, bits_in, bits_out, rows)
