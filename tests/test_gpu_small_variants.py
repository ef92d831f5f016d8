"""The launch-bound kernels of the symmetric, FP8 and compact-metadata quantizers (fused step and one-launch all-reduce),
on both sides of their size limit: a case as given, and the same case with its token rows repeated up to the bulk kernels'
volumes.  Both must give the oracle's bits.  Run with ``-m gpu`` on an MI355X."""
import numpy as np
import pytest

import oracle
import synth_inputs
from test_gpu_parity import BULK_ELEMS, Guarded, bulk_reps, dev, fc, first_diff, same_bits, tile_tokens  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PAIRS = {"sym": [(4, 4), (4, 8), (8, 4), (8, 8)], "cmeta": [(4, 4), (4, 8), (8, 4), (8, 8)], "fp8": [(8, 8)]}
SHAPES = [(7, 2176, 128), (1, 32, 32), (3, 1056, 32), (5, 2048, 64), (2, 4096, 256), (3, 1536, 512), (31, 8192, 128)]


def wire(name, n_src, tokens, hidden, group, bits, seed):
    """codes and metadata of every source: quantized rows in the first source, arbitrary legal ones in the others"""
    rng = np.random.default_rng(seed)
    x = synth_inputs.make_partials_stress(n_src, tokens, hidden, seed % synth_inputs.STRESS_KINDS, seed=seed)
    q = {"sym": lambda r: oracle.quantize_sym(r, group, bits), "fp8": lambda r: oracle.quantize_fp8(r, group),
         "cmeta": lambda r: oracle.quantize_cmeta(r, group, bits)}[name]
    parts = [q(x[j]) for j in range(n_src)]
    c = np.stack([p[0] for p in parts])
    m = np.stack([p[1] for p in parts])
    for j in range(1, n_src, 2):
        c[j] = rng.integers(0, 256, size=c[j].shape, dtype=np.uint8)          # every code, -2^(n-1) included
        if name == "fp8":
            c[j][(c[j] & 0x7F) == 0x7F] = 0x7E                                # no NaN bytes
        if name != "cmeta":
            m[j] = np.exp(rng.uniform(-100, 60, size=m[j].shape)).astype(np.float32)
    return c, m


@pytest.mark.parametrize("name", list(PAIRS))
@pytest.mark.parametrize("n_src", [1, 2, 3, 5, 8])
def test_fused_small_and_bulk(fc, name, n_src):
    ref = getattr(oracle, "dequant_reduce_requant_" + name)
    gpu = getattr(fc, "dequant_reduce_requant_" + name)
    meta_type = torch.int32 if name == "cmeta" else torch.float32
    for bits_in, bits_out in PAIRS[name]:
        for k, (t, h, g) in enumerate(SHAPES):
            bits = () if name == "fp8" else (bits_in, bits_out)
            c, m = wire(name, n_src, t, h, g, bits_in, seed=10 * n_src + k)
            want = ref(c, m, h, g, *bits)
            for reps in (1, bulk_reps(t, h)):
                if reps > 1 and (k % 3 or t * h < 1024):
                    continue                                                  # the bulk kernels on every third shape
                cr, mr = tile_tokens(c, reps), tile_tokens(m, reps)
                co = Guarded((t * reps, h * bits_out // 8), torch.uint8)
                mo = Guarded((t * reps, h // g), meta_type)
                gpu(dev(cr), dev(mr.view(np.int32)) if name == "cmeta" else dev(mr), h, g, *bits, out=(co.t, mo.t))
                torch.cuda.synchronize()
                for part, got, w in zip(("codes", "metadata"), (co, mo), want):
                    got.check()
                    a = got.t.cpu().numpy()
                    b = tile_tokens(w, reps)
                    assert same_bits(a.view(np.uint8), b.view(np.uint8)), "%s N=%d %dx%d g=%d %d->%d x%d %s: %s" % (
                        name, n_src, t, h, g, bits_in, bits_out, reps, part, first_diff(a.view(np.uint8), b.view(np.uint8)))


@pytest.mark.parametrize("name", list(PAIRS))
@pytest.mark.parametrize("n_src", [1, 2, 3, 4, 5, 8])
def test_fused_at_the_limit_of_the_launch_bound_kernel(fc, name, n_src):
    # the largest volume of the launch-bound kernel (a number of wavefronts, by quantizer, widths and fan-in) and the next row on the
    # bulk kernel; 6 rows of 8-bit codes are the largest volume of few sources that is too small for it
    t, h = 6, 1024
    meta_type = torch.int32 if name == "cmeta" else torch.float32
    for (bits_in, bits_out), lanes in [(p, l) for p in PAIRS[name] for l in (16, 32)]:
        g = lanes * 32 // bits_in
        bits = () if name == "fp8" else (bits_in, bits_out)
        c, m = wire(name, n_src, t, h, g, bits_in, seed=n_src)
        want = [dev(np.ascontiguousarray(a).view(np.uint8)) for a in getattr(oracle, "dequant_reduce_requant_" + name)(c, m, h, g, *bits)]
        few_c, few_m = dev(c), dev(m.view(np.int32)) if name == "cmeta" else dev(m)
        waves = 3 if n_src == 1 and bits_in == 8 else 2 if n_src == 1 else (6 if lanes < 32 else 5) if bits_in == 8 else \
            6 if name == "sym" else 3 if bits_out == 8 and n_src <= 4 else 4
        limit = waves * 1024 * (2048 // bits_in)                              # elements
        for rows in (6, 7, limit // h, limit // h + 1):
            pick = torch.arange(rows, device="cuda") % t
            co = Guarded((rows, h * bits_out // 8), torch.uint8)
            mo = Guarded((rows, h // g), meta_type)
            getattr(fc, "dequant_reduce_requant_" + name)(few_c[:, pick], few_m[:, pick], h, g, *bits, out=(co.t, mo.t))
            torch.cuda.synchronize()
            for got, w in zip((co, mo), want):
                got.check()
                assert torch.equal(got.t.view(torch.uint8), w[pick]), "%s N=%d %d->%d rows=%d" % (name, n_src, bits_in, bits_out, rows)


@pytest.mark.parametrize("name", ["asym", "cmeta"])
@pytest.mark.parametrize("n_src", [1, 2, 3, 4])
@pytest.mark.parametrize("group", [256, 512, 1024, 2048, 4096, 8192])
def test_fused_wide_groups_where_the_fold_changes(fc, name, n_src, group):
    # 4-bit codes, groups from 1024 on, at most 256 workgroups (4096 elements each, 8192 for the widest groups): another fold than
    # above that; groups from 256 on, two or three sources, 4 -> 8 bit: the same fold from 6 * 2^20 up to 32 * 2^20 elements.
    # Rows with ordinary, huge, fractional and out-of-reach metadata.
    t, sfx = 5, "" if name == "asym" else "_cmeta"
    rng = np.random.default_rng(group + n_src)
    x = synth_inputs.make_partials(n_src, t, group, seed=group + n_src)
    parts = [getattr(oracle, "quantize" + sfx)(x[j], group, 4) for j in range(n_src)]
    wire = [np.stack(p) for p in zip(*parts)]
    wire[0][:] = rng.integers(0, 256, size=wire[0].shape, dtype=np.uint8)
    if name == "asym":
        wire[1][:, 1], wire[2][:, 2], wire[2][-1, 3], wire[2][0, 4] = 2.0 ** 105, 2.5, 5000.0, -1700.0
    else:
        halves = wire[1].view(np.uint16).reshape(n_src, t, -1, 2)
        halves[:, 2, :, 1], halves[-1, 3, :, 1] = np.float16(2.5).view(np.uint16), np.float16(5000.0).view(np.uint16)
    few = [dev(w.view(np.int32) if w.dtype == np.uint32 else w) for w in wire]
    for bits_out in (4, 8):
        want = [dev(np.ascontiguousarray(a).view(np.uint8))
                for a in getattr(oracle, "dequant_reduce_requant" + sfx)(*wire, group, group, 4, bits_out)]
        limit = 256 * (8192 if group == 8192 else 4096)
        volumes = [1, limit // group, limit // group + 1, 2 * limit // group + 3]
        if bits_out == 8 and n_src in (2, 3):
            volumes += [v // group + more for v in (6 << 20, 32 << 20) for more in (0, 1)]
        for rows in volumes:
            pick = torch.arange(rows, device="cuda") % t
            outs = [Guarded((rows, group * bits_out // 8), torch.uint8)]
            outs += [Guarded((rows, 1), few[1].dtype) for _ in few[1:]]
            getattr(fc, "dequant_reduce_requant" + sfx)(*[w[:, pick] for w in few], group, group, 4, bits_out,
                                                        out=tuple(o.t for o in outs))
            torch.cuda.synchronize()
            for got, w in zip(outs, want):
                got.check()
                assert torch.equal(got.t.view(torch.uint8), w[pick]), "%s N=%d g=%d ->%d rows=%d" % (name, n_src, group, bits_out, rows)


@pytest.mark.parametrize("name", list(PAIRS))
@pytest.mark.parametrize("n_src", [1, 2, 4, 7, 8])
def test_allreduce_small_and_bulk(fc, name, n_src):
    ref, gpu = getattr(oracle, "allreduce_sim_" + name), getattr(fc, "allreduce_sim_" + name)
    for bits_rs, bits_ag in PAIRS[name]:
        for k, (t, h, g) in enumerate(SHAPES):
            bits = () if name == "fp8" else (bits_rs, bits_ag)
            x = synth_inputs.make_partials_stress(n_src, t, h, (k + n_src) % synth_inputs.STRESS_KINDS, seed=k + 50 * n_src)
            if k == 0:
                x[:, 0] = -0.0                                                # groups of negative zeros
                x[0, 1, ::2] = np.float16(-0.0)
            want = ref(x, g, *bits)
            for reps in (1, bulk_reps(t, h)):
                if reps > 1 and (k % 3 or t * h < 1024):
                    continue
                xr = tile_tokens(x, reps)
                assert (xr[0].size > BULK_ELEMS) == (reps > 1)
                y = Guarded((t * reps, h), torch.float16)
                gpu(dev(xr.view(np.uint16)).view(torch.float16), g, *bits, out=y.t)
                torch.cuda.synchronize()
                y.check()
                a, b = y.t.cpu().numpy().view(np.uint16), tile_tokens(want, reps).view(np.uint16)
                assert same_bits(a, b), "%s N=%d %dx%d g=%d %d->%d x%d: %s" % (name, n_src, t, h, g, bits_rs, bits_ag, reps,
                                                                              first_diff(a, b))


@pytest.mark.parametrize("name", ["asym"] + list(PAIRS))
@pytest.mark.parametrize("n_src,limit", [(4, 1 << 20), (7, (6 << 20) // 7), (8, 1 << 20)])
def test_allreduce_at_the_limit_of_the_launch_bound_kernel(fc, name, n_src, limit):
    # the largest volume of the launch-bound kernel and the next row on the bulk kernel, from a few rows of every kind
    t, h, g = 6, 1024, 128
    bits = () if name == "fp8" else (4, 8)
    sfx = "" if name == "asym" else "_" + name
    x = np.concatenate([synth_inputs.make_partials_stress(n_src, 1, h, k % synth_inputs.STRESS_KINDS, seed=k + n_src)
                        for k in range(t)], axis=1)
    want = dev(getattr(oracle, "allreduce_sim" + sfx)(x, g, *bits).view(np.int16))
    few = dev(x.view(np.uint16)).view(torch.float16)
    for rows in (limit // h, limit // h + 1):
        pick = torch.arange(rows, device="cuda") % t
        y = Guarded((rows, h), torch.float16)
        getattr(fc, "allreduce_sim" + sfx)(few[:, pick], g, *bits, out=y.t)
        torch.cuda.synchronize()
        y.check()
        assert torch.equal(y.t.view(torch.int16), want[pick]), "%s N=%d rows=%d" % (name, n_src, rows)
