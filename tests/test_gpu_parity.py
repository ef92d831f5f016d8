"""GPU parity: every entry point of the C-ABI library against the CPU oracle on
the same seeded inputs.  Codes, scales and zero-points must match bit for bit;
the final float16 output is additionally checked against the benchmark
contract's tolerance (1e-3 relative) although bit equality is what is expected
and asserted.  Run with ``-m gpu`` on an MI355X."""
import numpy as np
import pytest

import oracle
import synth_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GUARD = 16384     # bytes of poison on each side of every output buffer: the largest tile that one workgroup writes
POISON = 0xA5


@pytest.fixture(scope="module")
def fc():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests selected but no GPU is visible")
    import paper_2412_04964_amd as m
    m.lib()            # raises if libfc.so was not built: there is no fallback
    return m


class Guarded:
    """Device buffer with poisoned guard bands; .t is the usable tensor."""

    def __init__(self, shape, dtype):
        n = int(np.prod(shape)) * torch.empty(0, dtype=dtype).element_size()
        pad = (-n) % 16
        self.raw = torch.full((GUARD + n + pad + GUARD,), POISON, dtype=torch.uint8, device="cuda")
        self.n = n
        self.t = self.raw[GUARD:GUARD + n].view(dtype).view(*shape)

    def check(self):
        raw = self.raw.cpu().numpy()
        assert (raw[:GUARD] == POISON).all(), "write before the buffer"
        assert (raw[GUARD + self.n:] == POISON).all(), "write past the buffer"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def same_bits(a, b):
    a = np.ascontiguousarray(a); b = np.ascontiguousarray(b)
    return a.shape == b.shape and a.tobytes() == b.tobytes()


def first_diff(a, b):
    a = np.ascontiguousarray(a).ravel(); b = np.ascontiguousarray(b).ravel()
    ia = a.view(np.uint32) if a.dtype == np.float32 else a
    ib = b.view(np.uint32) if b.dtype == np.float32 else b
    idx = np.flatnonzero(ia != ib)
    return "%d mismatches, first at %s: gpu=%r ref=%r" % (idx.size, idx[:5], a[idx[:5]], b[idx[:5]])


def gpu_quantize(fc, x16, group, bits):
    t, h = x16.shape
    c = Guarded((t, h * bits // 8), torch.uint8)
    s = Guarded((t, h // group), torch.float32)
    z = Guarded((t, h // group), torch.float32)
    fc.quantize(dev(x16.view(np.uint16)).view(torch.float16), group, bits, out=(c.t, s.t, z.t))
    torch.cuda.synchronize()
    for g in (c, s, z):
        g.check()
    return c.t.cpu().numpy(), s.t.cpu().numpy(), z.t.cpu().numpy()


# fc_dequant_reduce_requant has two kernels: a launch-bound one (one code word per lane and source) up to 6144 wavefronts of it, i.e.
# at most 3 * 2^20 elements (7 * 2^19 in groups of 8192), and the bulk kernel above.  Groups never cross token rows, so repeating the
# token rows of a case gives the same case at another volume: here one with workgroups of several wavefronts, which the launch-bound
# kernel still takes in part; test_gpu_parity_bulk.py runs the cases once more at volumes past every limit.
BULK_ELEMS = 1 << 20


def bulk_reps(tokens, hidden):
    return -(-(BULK_ELEMS + 1) // (tokens * hidden))


def tile_tokens(a, reps):
    """repeat the token axis (the last but one) of codes / scales / zero-points / expected outputs"""
    return np.concatenate([np.asarray(a)] * reps, axis=-2) if reps > 1 else np.asarray(a)


def gpu_fused(fc, c, s, z, hidden, group, bits_in, bits_out):
    """the fused step on the case as given and on the case repeated up to the bulk kernel's volumes; both results
    must be the same bits (the first is returned)"""
    results = []
    for reps in (1, bulk_reps(c.shape[1], hidden)):
        cr, sr, zr = tile_tokens(c, reps), tile_tokens(s, reps), tile_tokens(z, reps)
        t = cr.shape[1]
        co = Guarded((t, hidden * bits_out // 8), torch.uint8)
        so = Guarded((t, hidden // group), torch.float32)
        zo = Guarded((t, hidden // group), torch.float32)
        fc.dequant_reduce_requant(dev(cr), dev(sr), dev(zr), hidden, group, bits_in, bits_out,
                                  out=(co.t, so.t, zo.t))
        torch.cuda.synchronize()
        for g in (co, so, zo):
            g.check()
        results.append((co.t.cpu().numpy(), so.t.cpu().numpy(), zo.t.cpu().numpy(), reps))
    small, big = results
    for name, a, b in zip(("codes", "scales", "zeros"), small[:3], big[:3]):
        assert same_bits(tile_tokens(a, big[3]), b), "bulk kernel differs from the small-volume call: %s: %s" % (
            name, first_diff(tile_tokens(a, big[3]), b))
    return small[:3]


def gpu_dequantize(fc, c, s, z, hidden, group, bits):
    y = Guarded((c.shape[0], hidden), torch.float16)
    fc.dequantize(dev(c), dev(s), dev(z), hidden, group, bits, out=y.t)
    torch.cuda.synchronize()
    y.check()
    return y.t.cpu().numpy()


def assert_triplet(got, want, what):
    for name, g, w in zip(("codes", "scales", "zeros"), got, want):
        assert same_bits(g, w), "%s %s: %s" % (what, name, first_diff(g, w))


def assert_f16(got, want, scale_per_elem, what):
    # contract tolerance first (1e-3 relative, floored by the group's step), then exact bits
    g = got.astype(np.float64); w = want.astype(np.float64)
    tol = 1e-3 * np.maximum(np.abs(w), scale_per_elem)
    fin = np.isfinite(w)
    assert np.all(np.abs(g[fin] - w[fin]) <= tol[fin]), what
    assert same_bits(got.view(np.uint16), want.view(np.uint16)), \
        "%s: %s" % (what, first_diff(got.view(np.uint16), want.view(np.uint16)))


# shapes: several workgroup tiles (8192 elements each) plus a ragged tail
SHAPES = [(16, 4096), (3, 1056), (5, 8192), (1, 32), (7, 2080), (33, 4096 + 2048)]


def groups_for(hidden):
    return [g for g in (32, 64, 128, 256, 512, 1024) if hidden % g == 0]


# --------------------------------------------------------------------------- #
# fc_quantize
# --------------------------------------------------------------------------- #

@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("shape", SHAPES)
def test_quantize_matches_oracle(fc, bits, shape):
    t, h = shape
    x = synth_inputs.make_partials(1, t, h, seed=t + h, outlier_frac=0.01)[0]
    for group in groups_for(h):
        assert_triplet(gpu_quantize(fc, x, group, bits), oracle.quantize(x, group, bits),
                       "quantize %s g=%d b=%d" % (shape, group, bits))


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("group", [32, 64, 128, 256])
def test_quantize_adversarial_groups(fc, bits, group):
    x = synth_inputs.adversarial_groups(group, seed=group)
    assert_triplet(gpu_quantize(fc, x, group, bits), oracle.quantize(x, group, bits),
                   "adversarial g=%d b=%d" % (group, bits))


def test_quantize_tiny_config_seed0(fc):
    w = synth_inputs.WORKLOADS["tiny"]
    x = synth_inputs.make_workload(w)
    for j in range(w.n_src):
        assert_triplet(gpu_quantize(fc, x[j], w.group, w.bits_in), oracle.quantize(x[j], w.group, w.bits_in),
                       "tiny source %d" % j)


# --------------------------------------------------------------------------- #
# fc_dequant_reduce_requant
# --------------------------------------------------------------------------- #

def oracle_stage1(x, group, bits):
    parts = [oracle.quantize(x[j], group, bits) for j in range(x.shape[0])]
    return tuple(np.stack([p[i] for p in parts]) for i in range(3))


@pytest.mark.parametrize("bits_in,bits_out", [(4, 4), (8, 8), (4, 8), (8, 4)])
@pytest.mark.parametrize("n_src", [1, 2, 3, 4, 5, 6, 7, 8])
def test_fused_matches_oracle(fc, bits_in, bits_out, n_src):
    for (t, h) in [(16, 4096), (3, 1056), (7, 2080)]:
        x = synth_inputs.make_partials(n_src, t, h, seed=10 * n_src + bits_in)
        for group in groups_for(h)[:4]:
            c, s, z = oracle_stage1(x, group, bits_in)
            want = oracle.dequant_reduce_requant(c, s, z, h, group, bits_in, bits_out)
            got = gpu_fused(fc, c, s, z, h, group, bits_in, bits_out)
            assert_triplet(got, want, "fused N=%d %dx%d g=%d %d->%d" % (n_src, t, h, group, bits_in, bits_out))


@pytest.mark.parametrize("bits_in,bits_out", [(4, 4), (8, 8), (4, 8)])
def test_fused_large_groups(fc, bits_in, bits_out):
    t, h = 5, 8192
    x = synth_inputs.make_partials(3, t, h, seed=77)
    for group in (256, 512, 1024):
        c, s, z = oracle_stage1(x, group, bits_in)
        want = oracle.dequant_reduce_requant(c, s, z, h, group, bits_in, bits_out)
        assert_triplet(gpu_fused(fc, c, s, z, h, group, bits_in, bits_out), want, "fused g=%d" % group)


@pytest.mark.parametrize("bits_in", [4, 8])
def test_fused_arbitrary_scales_and_zero_points(fc, bits_in):
    # slices whose zero-points are huge, negative, fractional or mixed inside one
    # wavefront: exercises the general (fp32) dequantize path next to the fast one
    rng = np.random.default_rng(5)
    n_src, t, h, group = 4, 6, 4096, 128
    c = rng.integers(0, 256, size=(n_src, t, h * bits_in // 8), dtype=np.uint8)
    s = np.exp(rng.uniform(-12, 8, size=(n_src, t, h // group))).astype(np.float32)
    z = np.rint(rng.uniform(-20, 300, size=(n_src, t, h // group))).astype(np.float32)
    z[0, :, ::3] = rng.uniform(-3e6, 3e6, size=z[0, :, ::3].shape).astype(np.float32)
    z[1, :, 1::5] += 0.25
    z[2, 1] = -1700.0
    z[2, 2] = 1000.0
    z[2, 3] = -1701.0
    z[2, 4] = 1001.0
    z[3, 0] = 2.0 ** 24 + 2
    for bits_out in (4, 8):
        want = oracle.dequant_reduce_requant(c, s, z, h, group, bits_in, bits_out)
        assert_triplet(gpu_fused(fc, c, s, z, h, group, bits_in, bits_out), want,
                       "arbitrary meta %d->%d" % (bits_in, bits_out))


@pytest.mark.parametrize("bits_in", [4, 8])
def test_fused_extreme_scales(fc, bits_in):
    # source scales from the smallest subnormal to 1e35: sums that are subnormal or vanish (the constant-group
    # rule of Eq. 1 on tiny ranges), and output scales beyond 2^100 (the reciprocal's slow branch)
    rng = np.random.default_rng(15)
    n_src, t, h, group = 2, 9, 2048, 128
    ladder = np.array([1.4e-45, 1e-42, 1e-40, 1.1754944e-38, 1.2e-38, 1e-30, 1.0, 1e30, 2.0 ** 100, 2.0 ** 101, 1e35],
                      np.float32)
    c = rng.integers(0, 256, size=(n_src, t, h * bits_in // 8), dtype=np.uint8)
    s = ladder[rng.integers(0, ladder.size, size=(n_src, t, h // group))]
    s[:, 0] = ladder[0]; s[:, 1] = ladder[3]; s[:, 2] = ladder[8]; s[:, 3] = ladder[10]     # uniform rows too
    s[0, 4] = ladder[9]; s[1, 4] = ladder[1]
    z = np.rint(rng.uniform(-20, 300, size=s.shape)).astype(np.float32)
    for bits_out in (4, 8):
        want = oracle.dequant_reduce_requant(c, s, z, h, group, bits_in, bits_out)
        assert np.isfinite(want[1]).all() and (want[1] > 2.0 ** 100).any() and (want[1] < 1e-37).any()
        assert_triplet(gpu_fused(fc, c, s, z, h, group, bits_in, bits_out), want,
                       "extreme scales %d->%d" % (bits_in, bits_out))
        y = oracle.dequantize(*want, h, group, bits_out)
        got = gpu_dequantize(fc, *want, h, group, bits_out)
        assert same_bits(got.view(np.uint16), y.view(np.uint16)), "extreme scales, dequantize"


@pytest.mark.parametrize("n_src,group", [(1, 128), (2, 1024), (3, 32), (4, 128), (4, 8192), (5, 128)])
@pytest.mark.parametrize("scale", [1.4e-45, 1e-40, 2.0 ** 104 * (1 - 2.0 ** -24), 2.0 ** 104, 2.0 ** 115, -3.5])
def test_fused_scales_around_the_exponent_limit(fc, n_src, group, scale):
    # 4-bit codes are dequantized with part of the exponent moved into the scale: the largest scale that may take it,
    # the first that may not, subnormal and negative ones; every nibble position, zero-points at both ends of the
    # short path; the most sources that take it and one more.  Ordinary rows meet general ones in the same launch.
    rng = np.random.default_rng(16)
    t, h = 5, 8192
    c = rng.integers(0, 256, size=(n_src, t, h // 2), dtype=np.uint8)
    s = np.full((n_src, t, h // group), scale, np.float32)
    s[:, 2] = rng.uniform(0.01, 2.0, size=s[:, 2].shape).astype(np.float32)
    z = np.rint(rng.uniform(-20, 30, size=s.shape)).astype(np.float32)
    z[0, 0], z[0, 1], z[-1, 3], z[-1, 4] = -1700.0, 1000.0, -0.0, 0.0
    for bits_out in (4, 8):
        want = oracle.dequant_reduce_requant(c, s, z, h, group, 4, bits_out)
        assert np.isfinite(want[1]).all()
        assert_triplet(gpu_fused(fc, c, s, z, h, group, 4, bits_out), want, "scale %g -> %d" % (scale, bits_out))


def test_fused_adversarial_sums(fc):
    # sums that are constant, zero, or nearly constant on a large offset
    group = 128
    a = synth_inputs.adversarial_groups(group, seed=1)
    x = np.stack([a, (-a.astype(np.float32)).astype(np.float16), a[::-1].copy()])
    for bits in (4, 8):
        c, s, z = oracle_stage1(x, group, bits)
        for n in (2, 3):
            want = oracle.dequant_reduce_requant(c[:n], s[:n], z[:n], a.shape[1], group, bits, bits)
            assert_triplet(gpu_fused(fc, c[:n], s[:n], z[:n], a.shape[1], group, bits, bits), want,
                           "adversarial sums b=%d n=%d" % (bits, n))


def test_fused_source_stride_with_padding(fc):
    # sources separated by more than one slab (stride > slab size), at a launch-bound and at a bulk volume
    n_src, t0, h, group, bits = 3, 4, 2048, 128, 4
    x = synth_inputs.make_partials(n_src, t0, h, seed=9)
    c0, s0, z0 = oracle_stage1(x, group, bits)
    want0 = oracle.dequant_reduce_requant(c0, s0, z0, h, group, bits, bits)
    for reps in (1, bulk_reps(t0, h)):
        c, s, z = tile_tokens(c0, reps), tile_tokens(s0, reps), tile_tokens(z0, reps)
        want = tuple(tile_tokens(w, reps) for w in want0)
        t = t0 * reps
        cp = torch.zeros((n_src, t + 2, h // 2), dtype=torch.uint8, device="cuda")
        sp = torch.zeros((n_src, t + 1, h // group), dtype=torch.float32, device="cuda")
        zp = torch.zeros_like(sp)
        cp[:, :t] = dev(c); sp[:, :t] = dev(s); zp[:, :t] = dev(z)
        co = torch.empty((t, h // 2), dtype=torch.uint8, device="cuda")
        so = torch.empty((t, h // group), dtype=torch.float32, device="cuda")
        zo = torch.empty_like(so)
        rc = fc.lib().fc_dequant_reduce_requant(cp.data_ptr(), cp.stride(0), sp.data_ptr(), zp.data_ptr(),
                                                sp.stride(0), n_src, t, h, group, bits, bits,
                                                co.data_ptr(), so.data_ptr(), zo.data_ptr(),
                                                torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        torch.cuda.synchronize()
        assert_triplet((co.cpu().numpy(), so.cpu().numpy(), zo.cpu().numpy()), want, "padded stride x%d" % reps)


def _clamp_case_groups(group, n_groups, rng):
    """fp16 groups whose largest rounded value exceeds qmax - z by one step (the upper clamp of
    Eq. 2 acts): range 7.5 with both ends on .5 ties, so s = 0.5 (4 bit) and the ends round apart."""
    rows = []
    for k in range(n_groups):
        off = float(rng.integers(-40, 40))
        body = rng.uniform(-1.5, 5.5, size=group)
        body[rng.integers(0, group)] = -1.75
        body[rng.integers(0, group - 1) + (1 if body[0] == -1.75 else 0)] = 5.75
        if not (body == -1.75).any():
            body[0] = -1.75
        rows.append(body + off)
    return np.concatenate(rows).astype(np.float16)


@pytest.mark.parametrize("group", [32, 128])
def test_upper_clamp_is_exercised(fc, group):
    rng = np.random.default_rng(group)
    x = np.stack([_clamp_case_groups(group, 4096 // group, rng) for _ in range(8)])
    want = oracle.quantize(x, group, 4)
    # the case set really triggers the clamp: some group's top code comes from t + z = 16
    xf = x.astype(np.float32).reshape(8, -1, group)
    t_top = np.rint(xf.max(-1) * (np.float32(1) / want[1])) + want[2]
    assert (t_top > 15).any()
    assert_triplet(gpu_quantize(fc, x, group, 4), want, "clamp quantize g=%d" % group)
    # same through the fused kernel: one 8-bit source with scale 0.25 and zero-point 100 whose codes
    # 93..123 dequantize exactly to -1.75..5.75, so the requantized sums hit the clamp as well
    t, h = 8, 4096
    codes = rng.integers(94, 123, size=(1, t, h), dtype=np.uint8)
    cg = codes.reshape(1, t, h // group, group)
    cg[..., 3] = 93
    cg[..., 17] = 123
    s = np.full((1, t, h // group), 0.25, np.float32)
    z = np.full((1, t, h // group), 100.0, np.float32)
    want_f = oracle.dequant_reduce_requant(codes, s, z, h, group, 8, 4)
    acc = oracle.dequant_reduce_f32(codes, s, z, h, group, 8).reshape(t, h // group, group)
    assert (np.rint(acc.max(-1) * (np.float32(1) / want_f[1])) + want_f[2] > 15).all()
    assert_triplet(gpu_fused(fc, codes, s, z, h, group, 8, 4), want_f, "clamp fused g=%d" % group)


# --------------------------------------------------------------------------- #
# fc_dequantize
# --------------------------------------------------------------------------- #

@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("shape", [(16, 4096), (3, 1056), (7, 2080)])
def test_dequantize_matches_oracle(fc, bits, shape):
    t, h = shape
    x = synth_inputs.make_partials(1, t, h, seed=3)[0]
    for group in groups_for(h)[:4]:
        c, s, z = oracle.quantize(x, group, bits)
        want = oracle.dequantize(c, s, z, h, group, bits)
        got = gpu_dequantize(fc, c, s, z, h, group, bits)
        assert_f16(got, want, np.repeat(s, group, axis=1), "dequantize %s g=%d b=%d" % (shape, group, bits))


@pytest.mark.parametrize("bits", [4, 8])
def test_dequantize_extremes(fc, bits):
    # adversarial groups (float16 extremes, subnormals), overflow to infinity, odd zero-points
    group = 128
    x = synth_inputs.adversarial_groups(group, seed=2)
    c, s, z = oracle.quantize(x, group, bits)
    h = x.shape[1]
    want = oracle.dequantize(c, s, z, h, group, bits)
    assert_f16(gpu_dequantize(fc, c, s, z, h, group, bits), want, np.repeat(s, group, axis=1), "extremes")
    rng = np.random.default_rng(8)
    s2 = np.exp(rng.uniform(-30, 12, size=s.shape)).astype(np.float32)
    z2 = z.copy(); z2[:, ::2] = rng.uniform(-5e4, 5e4, size=z2[:, ::2].shape).astype(np.float32)
    want = oracle.dequantize(c, s2, z2, h, group, bits)
    got = gpu_dequantize(fc, c, s2, z2, h, group, bits)
    assert same_bits(got.view(np.uint16), want.view(np.uint16)), first_diff(got.view(np.uint16), want.view(np.uint16))
    assert np.isinf(want.astype(np.float32)).any() and (want.view(np.uint16) & 0x7C00 == 0).any()


# --------------------------------------------------------------------------- #
# fc_allreduce_sim
# --------------------------------------------------------------------------- #

@pytest.mark.parametrize("name", ["tiny"])
def test_allreduce_sim_tiny_config(fc, name):
    w = synth_inputs.WORKLOADS[name]
    x = synth_inputs.make_workload(w)
    want = oracle.allreduce_sim(x, w.group, w.bits_in, w.bits_out)
    y = Guarded((w.tokens, w.hidden), torch.float16)
    fc.allreduce_sim(dev(x.view(np.uint16)).view(torch.float16), w.group, w.bits_in, w.bits_out, out=y.t)
    torch.cuda.synchronize(); y.check()
    c, s, z = oracle_stage1(x, w.group, w.bits_in)
    so = oracle.dequant_reduce_requant(c, s, z, w.hidden, w.group, w.bits_in, w.bits_out)[1]
    assert_f16(y.t.cpu().numpy(), want, np.repeat(so, w.group, axis=1), "allreduce_sim tiny")


@pytest.mark.parametrize("bits_rs,bits_ag", [(8, 8), (4, 4), (4, 8)])
@pytest.mark.parametrize("n_src", [2, 4, 8])
def test_allreduce_sim_matches_oracle(fc, bits_rs, bits_ag, n_src):
    t, h, group = 9, 4096, 128
    x = synth_inputs.make_partials(n_src, t, h, seed=n_src)
    want = oracle.allreduce_sim(x, group, bits_rs, bits_ag)
    got = fc.allreduce_sim(dev(x.view(np.uint16)).view(torch.float16), group, bits_rs, bits_ag)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    assert same_bits(got.view(np.uint16), want.view(np.uint16)), first_diff(got.view(np.uint16), want.view(np.uint16))


def test_empty_input_is_a_noop(fc):
    x = torch.empty((0, 4096), dtype=torch.float16, device="cuda")
    c, s, z = fc.quantize(x, 128, 4)
    assert c.shape == (0, 2048) and s.shape == (0, 32)
    y = fc.allreduce_sim(torch.empty((4, 0, 4096), dtype=torch.float16, device="cuda"), 128, 4, 4)
    assert y.shape == (0, 4096)
    torch.cuda.synchronize()


# --------------------------------------------------------------------------- #
# full benchmark shapes, in the launch configuration the benchmark times:
# the whole tensor goes through the GPU, sampled token rows are checked
# against the oracle (groups never cross rows, so a row is self-contained)
# --------------------------------------------------------------------------- #

@pytest.mark.parametrize("name", ["llama3_8b_prefill", "llama3_70b_prefill", "wide_fanin", "decode"])
def test_full_size_configs_on_sampled_rows(fc, name):
    w = synth_inputs.WORKLOADS[name]
    x = synth_inputs.make_partials_device(w.n_src, w.tokens, w.hidden, w.seed, "cuda",
                                          w.outlier_frac, w.outlier_gain)
    rows = np.unique(np.concatenate([[0, 1, w.tokens - 1],
                                     np.random.default_rng(1).integers(0, w.tokens, 61)]))
    rows = rows[rows < w.tokens]
    ridx = torch.from_numpy(rows).cuda()
    stage1 = [fc.quantize(x[j], w.group, w.bits_in) for j in range(w.n_src)]
    c = torch.stack([p[0] for p in stage1]); s = torch.stack([p[1] for p in stage1])
    z = torch.stack([p[2] for p in stage1])
    co, so, zo = fc.dequant_reduce_requant(c, s, z, w.hidden, w.group, w.bits_in, w.bits_out)
    y = fc.dequantize(co, so, zo, w.hidden, w.group, w.bits_out)
    y2 = fc.allreduce_sim(x, w.group, w.bits_in, w.bits_out)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))

    xs = x[:, ridx].cpu().numpy()
    oc, os_, oz = oracle_stage1(xs, w.group, w.bits_in)
    assert_triplet((c[:, ridx].cpu().numpy(), s[:, ridx].cpu().numpy(), z[:, ridx].cpu().numpy()),
                   (oc, os_, oz), name + " stage 1")
    want = oracle.dequant_reduce_requant(oc, os_, oz, w.hidden, w.group, w.bits_in, w.bits_out)
    assert_triplet((co[ridx].cpu().numpy(), so[ridx].cpu().numpy(), zo[ridx].cpu().numpy()), want,
                   name + " fused")
    wy = oracle.dequantize(*want, w.hidden, w.group, w.bits_out)
    assert_f16(y[ridx].cpu().numpy(), wy, np.repeat(want[1], w.group, axis=1), name + " output")
    # properties that hold at any size: every code in range is automatic for 4/8 bit fields;
    # scales positive and finite, zero-points integral
    assert bool((so > 0).all()) and bool(torch.isfinite(so).all())
    assert bool((zo == torch.round(zo)).all())


def _by_row_blocks(fn, n_rows, blocks=16):
    """fn(r0, r1) on contiguous row blocks in host threads (the oracle is scalar C; ctypes drops the GIL)."""
    from concurrent.futures import ThreadPoolExecutor
    edges = np.linspace(0, n_rows, min(blocks, n_rows) + 1).astype(int)
    with ThreadPoolExecutor(8) as ex:
        return list(ex.map(lambda k: fn(int(edges[k]), int(edges[k + 1])), range(len(edges) - 1)))


# every element of the benchmark volumes, all three stages, against the oracle (groups never cross token rows,
# so the oracle runs on row blocks in parallel); the headline shape also on the other two seeds
@pytest.mark.parametrize("name,seed", [("llama3_8b_prefill", 0), ("llama3_70b_prefill", 0), ("llama3_70b_prefill", 1),
                                       ("llama3_70b_prefill", 2), ("wide_fanin", 0), ("decode", 0),
                                       ("llama3_70b_prefill_int6", 0)])
def test_full_size_configs_every_element(fc, name, seed):
    w = synth_inputs.WORKLOADS[name]
    x = synth_inputs.make_partials_device(w.n_src, w.tokens, w.hidden, seed, "cuda", w.outlier_frac, w.outlier_gain)
    stage1 = [fc.quantize(x[j], w.group, w.bits_in) for j in range(w.n_src)]
    c = torch.stack([p[0] for p in stage1]); s = torch.stack([p[1] for p in stage1])
    z = torch.stack([p[2] for p in stage1])
    del stage1
    co, so, zo = fc.dequant_reduce_requant(c, s, z, w.hidden, w.group, w.bits_in, w.bits_out)
    y = fc.dequantize(co, so, zo, w.hidden, w.group, w.bits_out)
    torch.cuda.synchronize()
    xh = x.cpu().numpy()
    got1 = (c.cpu().numpy(), s.cpu().numpy(), z.cpu().numpy())
    got2 = (co.cpu().numpy(), so.cpu().numpy(), zo.cpu().numpy())
    goty = y.cpu().numpy()
    del x, c, s, z, co, so, zo, y

    def block(r0, r1):
        o1 = oracle_stage1(xh[:, r0:r1], w.group, w.bits_in)
        o2 = oracle.dequant_reduce_requant(*o1, w.hidden, w.group, w.bits_in, w.bits_out)
        oy = oracle.dequantize(*o2, w.hidden, w.group, w.bits_out)
        bad = []
        for what, got, want in (("stage 1", tuple(g[:, r0:r1] for g in got1), o1),
                                ("fused", tuple(g[r0:r1] for g in got2), o2)):
            for part, g_, w_ in zip(("codes", "scales", "zeros"), got, want):
                if not same_bits(g_, w_):
                    bad.append("%s %s rows [%d,%d): %s" % (what, part, r0, r1, first_diff(g_, w_)))
        if not same_bits(goty[r0:r1].view(np.uint16), oy.view(np.uint16)):
            bad.append("output rows [%d,%d): %s" % (r0, r1, first_diff(goty[r0:r1].view(np.uint16), oy.view(np.uint16))))
        return bad

    bad = sum(_by_row_blocks(block, w.tokens), [])
    assert not bad, "%s seed %d: %s" % (name, seed, "; ".join(bad[:4]))


@pytest.mark.parametrize("variant", ["asym", "sym", "fp8", "cmeta", "rot"])
def test_entry_points_capture_into_a_hip_graph_and_replay(fc, variant):
    # the library only enqueues kernels on the caller's stream (no allocation, no memset, no sync), so a
    # whole all-reduce captures into a HIP graph; every replay, with eager work in between, must
    # reproduce the eager result
    w = synth_inputs.WORKLOADS["decode"]
    x = synth_inputs.make_workload(w)
    xd = dev(x.view(np.uint16)).view(torch.float16)
    y = torch.empty((w.tokens, w.hidden), dtype=torch.float16, device="cuda")
    ws = torch.empty(fc.allreduce_sim_workspace_bytes(w.n_src, w.tokens, w.hidden, w.group, w.bits_in, w.bits_out),
                     dtype=torch.uint8, device="cuda")
    gpu_sim, cpu_sim = {
        "asym": (lambda: fc.allreduce_sim(xd, w.group, w.bits_in, w.bits_out, out=y, workspace=ws),
                 lambda a: oracle.allreduce_sim(a, w.group, w.bits_in, w.bits_out)),
        "sym": (lambda: fc.allreduce_sim_sym(xd, w.group, w.bits_in, w.bits_out, out=y, workspace=ws),
                lambda a: oracle.allreduce_sim_sym(a, w.group, w.bits_in, w.bits_out)),
        "fp8": (lambda: fc.allreduce_sim_fp8(xd, w.group, out=y, workspace=ws),
                lambda a: oracle.allreduce_sim_fp8(a, w.group)),
        "cmeta": (lambda: fc.allreduce_sim_cmeta(xd, w.group, w.bits_in, w.bits_out, out=y, workspace=ws),
                  lambda a: oracle.allreduce_sim_cmeta(a, w.group, w.bits_in, w.bits_out)),
        "rot": (lambda: fc.allreduce_sim_rot(xd, w.group, w.bits_in, w.bits_out, fc.QUANTIZER_ASYM, out=y, workspace=ws),
                lambda a: oracle.allreduce_sim_rot(a, w.group, w.bits_in, w.bits_out, oracle.ASYM)),
    }[variant]
    want = cpu_sim(x)
    gpu_sim()                                                                       # eager, loads the kernels
    torch.cuda.synchronize()
    assert same_bits(y.cpu().numpy().view(np.uint16), want.view(np.uint16))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        gpu_sim()
    for rep in range(4):
        y.fill_(7.0); ws.fill_(0x5A)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        assert same_bits(got.view(np.uint16), want.view(np.uint16)), "replay %d: %s" % (
            rep, first_diff(got.view(np.uint16), want.view(np.uint16)))
        # new input for the next replay: the graph reads the buffers, not captured values
        x = synth_inputs.make_partials(w.n_src, w.tokens, w.hidden, seed=100 + rep)
        xd.copy_(dev(x.view(np.uint16)).view(torch.float16))
        want = cpu_sim(x)


@pytest.mark.parametrize("n_src", [1, 3, 8])
def test_stream_reference_is_the_xor_of_its_inputs(fc, n_src):
    rng = np.random.default_rng(n_src)
    nbytes = 3 * 4096 + 1040                 # several tiles and a ragged tail
    src = rng.integers(0, 256, size=(n_src, nbytes), dtype=np.uint8)
    out = Guarded((nbytes,), torch.uint8)
    fc.stream_reference(dev(src), out.t)
    torch.cuda.synchronize(); out.check()
    assert np.array_equal(out.t.cpu().numpy(), np.bitwise_xor.reduce(src, axis=0))


def test_rank_shares_compose_to_the_whole(fc):
    # sharding by token rows (rank r reduces rows [r T/N, (r+1) T/N) of every source): running the fused
    # kernel once per share, with offset pointers and the full-slab strides, reproduces the single launch
    # (shares small enough for the launch-bound kernel, and shares the bulk kernel takes)
    n_src, t0, h, group, bits = 4, 24, 4096, 128, 4
    x = synth_inputs.make_partials(n_src, t0, h, seed=21)
    c0, s0, z0 = oracle_stage1(x, group, bits)
    want0 = oracle.dequant_reduce_requant(c0, s0, z0, h, group, bits, bits)
    for reps in (1, n_src * bulk_reps(t0, h)):
        c, s, z = tile_tokens(c0, reps), tile_tokens(s0, reps), tile_tokens(z0, reps)
        want = tuple(tile_tokens(w, reps) for w in want0)
        t = t0 * reps
        cd, sd, zd = dev(c), dev(s), dev(z)
        co = torch.empty((t, h // 2), dtype=torch.uint8, device="cuda")
        so = torch.empty((t, h // group), dtype=torch.float32, device="cuda")
        zo = torch.empty_like(so)
        share = t // n_src
        st = torch.cuda.current_stream().cuda_stream
        for r in range(n_src):
            r0 = r * share
            rc = fc.lib().fc_dequant_reduce_requant(
                cd[0, r0].data_ptr(), cd.stride(0), sd[0, r0].data_ptr(), zd[0, r0].data_ptr(), sd.stride(0),
                n_src, share, h, group, bits, bits, co[r0].data_ptr(), so[r0].data_ptr(), zo[r0].data_ptr(), st)
            assert rc == 0
        torch.cuda.synchronize()
        assert_triplet((co.cpu().numpy(), so.cpu().numpy(), zo.cpu().numpy()), want, "row shares x%d" % reps)
