"""GPU parity of the rotation entry points (Hadamard transform fused into the first
quantization and the last dequantization; paper Section 4) against the CPU oracle,
bit for bit, through the C ABI.  Run with ``-m gpu`` on an MI355X."""
import numpy as np
import pytest

import oracle
import synth_inputs
from test_gpu_parity import Guarded, dev, first_diff, same_bits, fc  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

QUANTIZERS = [(oracle.ASYM, 4), (oracle.ASYM, 8), (oracle.SYM, 4), (oracle.SYM, 8), (oracle.FP8, 8)]


def groups_of(hidden):
    return [g for g in (32, 128, 1024, 2048, 4096, 8192) if g <= hidden and hidden % g == 0]


# power-of-two rows (one block) and rows rotated block by block: 5 x 1024 (the rotation table's LLaMA-2-13B
# row), 3 x 1024, 7 x 1024, 3 x 2048, 3 x 4096, and a single block of 1024
HIDDENS = [2048, 4096, 8192, 1024, 5120, 3072, 7168, 6144, 12288]


def gpu_quantize_rot(fc, x16, group, bits, quantizer):
    t, h = x16.shape
    c = Guarded((t, h * bits // 8), torch.uint8)
    s = Guarded((t, h // group), torch.float32)
    z = Guarded((t, h // group), torch.float32)
    fc.quantize_rot(dev(x16.view(np.uint16)).view(torch.float16), group, bits, quantizer, out=(c.t, s.t, z.t))
    torch.cuda.synchronize()
    for g in (c, s, z):
        g.check()
    return c.t.cpu().numpy(), s.t.cpu().numpy(), z.t.cpu().numpy()


def assert_rot_triplet(got, want, quantizer, what):
    names = ("codes", "scales", "zeros") if quantizer == oracle.ASYM else ("codes", "scales")
    for name, g, w in zip(names, got, want):
        assert same_bits(g, w), "%s %s: %s" % (what, name, first_diff(g, w))


@pytest.mark.parametrize("quantizer,bits", QUANTIZERS)
@pytest.mark.parametrize("hidden", HIDDENS)
def test_quantize_rot_matches_oracle(fc, quantizer, bits, hidden):
    # 5 rows: with 1024-element blocks (two to a workgroup) 5 x 5, 5 x 3 and 5 x 7 blocks end in a half-filled chunk
    x = synth_inputs.make_partials(1, 5, hidden, seed=hidden + bits)[0]
    for group in groups_of(hidden):
        want = oracle.quantize_rot(x, group, bits, quantizer)
        got = gpu_quantize_rot(fc, x, group, bits, quantizer)
        assert_rot_triplet(got, want, quantizer, "quantize_rot h=%d g=%d b=%d q=%d" % (hidden, group, bits, quantizer))


@pytest.mark.parametrize("hidden", [2048, 4096, 8192])
def test_quantize_rot_special_rows(fc, hidden):
    # rows that rotate to a single spike (Walsh functions), a spike that rotates to a flat row, zeros,
    # binary16 extremes, and values whose transform rounds in every stage
    import scipy.linalg
    H = scipy.linalg.hadamard(hidden).astype(np.float32)
    rng = np.random.default_rng(hidden)
    x = np.zeros((8, hidden), np.float16)
    x[0] = H[3] * 0.5
    x[1] = H[hidden - 1] * -2.0
    x[2, 7] = 1000.0
    x[4] = 60000.0 * H[hidden // 2 + 1]
    x[5] = (rng.standard_normal(hidden) * np.exp(rng.uniform(-8, 8, hidden))).astype(np.float16)
    x[6] = np.float16(6e-8) * (np.arange(hidden) % 5)
    x[7] = rng.standard_normal(hidden) * 1e-3 + 3.0
    for quantizer, bits in QUANTIZERS:
        for group in (128, hidden):
            want = oracle.quantize_rot(x, group, bits, quantizer)
            got = gpu_quantize_rot(fc, x, group, bits, quantizer)
            assert_rot_triplet(got, want, quantizer, "special rows h=%d g=%d b=%d q=%d" % (hidden, group, bits, quantizer))


@pytest.mark.parametrize("quantizer,bits", QUANTIZERS)
@pytest.mark.parametrize("hidden", HIDDENS)
def test_dequantize_rot_matches_oracle(fc, quantizer, bits, hidden):
    x = synth_inputs.make_partials(1, 3, hidden, seed=hidden + 7)[0]
    rng = np.random.default_rng(hidden + bits)
    for group in groups_of(hidden)[::2]:
        c, s, z = oracle.quantize_rot(x, group, bits, quantizer)
        cases = [(c, s, z)]
        # arbitrary codes and metadata: every code value, scales over many binades, odd zero-points
        c2 = rng.integers(0, 256, size=c.shape, dtype=np.uint8)
        if quantizer == oracle.FP8:
            c2[(c2 & 0x7F) == 0x7F] = 0x7E
        s2 = np.exp(rng.uniform(-10, 6, size=s.shape)).astype(np.float32)
        z2 = np.rint(rng.uniform(-20, 300, size=s.shape)).astype(np.float32)
        z2[0, ::3] = rng.uniform(-3e4, 3e4, size=z2[0, ::3].shape).astype(np.float32)
        cases.append((c2, s2, z2))
        for cc, ss, zz in cases:
            want = oracle.dequantize_rot(cc, ss, zz, hidden, group, bits, quantizer)
            y = Guarded((cc.shape[0], hidden), torch.float16)
            fc.dequantize_rot(dev(cc), dev(ss), dev(zz), hidden, group, bits, quantizer, out=y.t)
            torch.cuda.synchronize(); y.check()
            got = y.t.cpu().numpy()
            assert same_bits(got.view(np.uint16), want.view(np.uint16)), \
                "dequantize_rot h=%d g=%d b=%d q=%d: %s" % (hidden, group, bits, quantizer,
                                                          first_diff(got.view(np.uint16), want.view(np.uint16)))


@pytest.mark.parametrize("quantizer,bits_rs,bits_ag", [(oracle.ASYM, 4, 4), (oracle.ASYM, 4, 8), (oracle.ASYM, 8, 8),
                                                       (oracle.SYM, 4, 4), (oracle.FP8, 8, 8)])
def test_allreduce_sim_rot_matches_oracle(fc, quantizer, bits_rs, bits_ag):
    for n_src, t, hidden, group in ((4, 5, 4096, 128), (2, 3, 8192, 8192), (8, 3, 2048, 2048), (3, 4, 8192, 1024),
                                    (4, 7, 5120, 1024), (2, 3, 5120, 128), (3, 1, 1024, 32), (2, 5, 12288, 4096)):
        x = synth_inputs.make_partials(n_src, t, hidden, seed=n_src + hidden)
        want = oracle.allreduce_sim_rot(x, group, bits_rs, bits_ag, quantizer)
        y = Guarded((t, hidden), torch.float16)
        fc.allreduce_sim_rot(dev(x.view(np.uint16)).view(torch.float16), group, bits_rs, bits_ag, quantizer, out=y.t)
        torch.cuda.synchronize(); y.check()
        got = y.t.cpu().numpy()
        assert same_bits(got.view(np.uint16), want.view(np.uint16)), \
            "allreduce_sim_rot N=%d h=%d g=%d: %s" % (n_src, hidden, group,
                                                      first_diff(got.view(np.uint16), want.view(np.uint16)))


@pytest.mark.parametrize("quantizer,bits", QUANTIZERS)
@pytest.mark.parametrize("tokens,hidden", [(1, 1024), (1, 5120), (3, 2048), (3, 3072)])
def test_partial_last_tile_stays_inside_the_buffers(fc, quantizer, bits, tokens, hidden):
    # blocks of 1024 and 2048 lie 4096 elements to a workgroup: here the last one holds 1024 or 2048 (one wavefront has
    # half of its elements, the other none).  Nothing past the end of codes, metadata and result may be written; the
    # guard bands reach further than a tile.
    x = synth_inputs.make_partials(2, tokens, hidden, seed=hidden + tokens)
    for group in (32, 1024):
        want = oracle.quantize_rot(x[0], group, bits, quantizer)
        assert_rot_triplet(gpu_quantize_rot(fc, x[0], group, bits, quantizer), want, quantizer, "h=%d g=%d" % (hidden, group))
        y = Guarded((tokens, hidden), torch.float16)
        fc.dequantize_rot(*[dev(a) for a in want], hidden, group, bits, quantizer, out=y.t)
        torch.cuda.synchronize(); y.check()
        ref = oracle.dequantize_rot(*want, hidden, group, bits, quantizer)
        assert same_bits(y.t.cpu().numpy().view(np.uint16), ref.view(np.uint16))
        y = Guarded((tokens, hidden), torch.float16)
        fc.allreduce_sim_rot(dev(x.view(np.uint16)).view(torch.float16), group, bits, bits, quantizer, out=y.t)
        torch.cuda.synchronize(); y.check()
        ref = oracle.allreduce_sim_rot(x, group, bits, bits, quantizer)
        assert same_bits(y.t.cpu().numpy().view(np.uint16), ref.view(np.uint16))


# elements: both sides of every volume at which the rotated quantizer and dequantizer change their form
VOLUMES = [1 << 20, (1 << 20) + 1, 1 << 21, (1 << 21) + 1, 5 << 19, (5 << 19) + 1, 3 << 20, (3 << 20) + 1, 1 << 22, (1 << 22) + 1,
           5 << 20, (5 << 20) + 1, 6 << 20, (6 << 20) + 1, 7 << 20, (7 << 20) + 1, 1 << 24, (1 << 24) + 1]


@pytest.mark.parametrize("quantizer,bits", QUANTIZERS)
@pytest.mark.parametrize("hidden", [1024, 3072, 2048, 4096])
def test_both_forms_give_the_same_bits(fc, quantizer, bits, hidden):
    # rows of every kind, a few of them (compared with the oracle) and repeated up to the volumes of the other form; the
    # number of rows is odd just above each limit, where blocks of 1024 and 2048 leave a partial last tile
    rng = np.random.default_rng(hidden + bits)
    x = synth_inputs.make_partials(1, 6, hidden, seed=hidden)[0]
    x[1] = 0
    x[2] = (rng.standard_normal(hidden) * np.exp(rng.uniform(-8, 8, hidden))).astype(np.float16)
    x[3] = rng.standard_normal(hidden) * 1e-3 + 3.0
    x[4] = np.float16(6e-8) * (np.arange(hidden) % 5)
    few = dev(x.view(np.uint16)).view(torch.float16)
    for group in (32, 1024):
        want = oracle.quantize_rot(x, group, bits, quantizer)
        s2, z2 = want[1].copy(), want[2].copy()
        s2[5] = np.exp(rng.uniform(-10, 6, size=s2[5].shape))
        if quantizer == oracle.ASYM:
            z2[5, ::3] = rng.uniform(-3e4, 3e4, size=z2[5, ::3].shape)
        wants = [dev(a) for a in want[:3 if quantizer == oracle.ASYM else 2]]
        metas = [dev(s2), dev(z2)]
        back = dev(oracle.dequantize_rot(want[0], s2, z2, hidden, group, bits, quantizer).view(np.int16))
        for volume in VOLUMES:
            rows = volume // hidden if volume % 2 == 0 else (volume // hidden + 1) | 1
            pick = torch.arange(rows, device="cuda") % 6
            c = Guarded((rows, hidden * bits // 8), torch.uint8)
            s, z = [Guarded((rows, hidden // group), torch.float32) for _ in range(2)]
            fc.quantize_rot(few[pick], group, bits, quantizer, out=(c.t, s.t, z.t))
            y = Guarded((rows, hidden), torch.float16)
            fc.dequantize_rot(wants[0][pick], metas[0][pick], metas[1][pick], hidden, group, bits, quantizer, out=y.t)
            torch.cuda.synchronize()
            for g in (c, s, z, y): g.check()
            what = "h=%d g=%d rows=%d " % (hidden, group, rows)
            for got, w in zip((c.t, s.t, z.t), wants):
                assert torch.equal(got.view(torch.uint8), w[pick].view(torch.uint8)), what + "quantize"
            assert torch.equal(y.t.view(torch.int16), back[pick]), what + "dequantize"


@pytest.mark.parametrize("quantizer,bits", QUANTIZERS)
@pytest.mark.parametrize("hidden", [8192, 12288])
def test_wide_blocks_both_layouts_every_group(fc, quantizer, bits, hidden):
    # Blocks of 8192 quantize in one layout of the lanes up to 2^21 elements and in another above, where a group of 256 elements and
    # more spans wavefronts; blocks of 4096 (hidden 12288) lay groups of 512 and more across them.  Every group, rows of every
    # kind, compared with the oracle and repeated up to both sides of the limit.
    rng = np.random.default_rng(hidden + bits)
    x = synth_inputs.make_partials(1, 5, hidden, seed=hidden + 1)[0]
    x[1] = (rng.standard_normal(hidden) * np.exp(rng.uniform(-8, 8, hidden))).astype(np.float16)
    x[2] = rng.standard_normal(hidden) * 1e-3 + 3.0
    x[3] = np.float16(6e-8) * (np.arange(hidden) % 5)
    x[4, ::2] = np.float16(-0.0)
    few = dev(x.view(np.uint16)).view(torch.float16)
    n_meta = 3 if quantizer == oracle.ASYM else 2
    for group in (32, 64, 128, 256, 512, 1024, 2048, 4096, 8192):
        if hidden % group:
            continue
        wants = [dev(a) for a in oracle.quantize_rot(x, group, bits, quantizer)[:n_meta]]
        for rows in (5, (1 << 21) // hidden, (1 << 21) // hidden + 1):
            pick = torch.arange(rows, device="cuda") % 5
            c = Guarded((rows, hidden * bits // 8), torch.uint8)
            s, z = [Guarded((rows, hidden // group), torch.float32) for _ in range(2)]
            fc.quantize_rot(few[pick], group, bits, quantizer, out=(c.t, s.t, z.t))
            torch.cuda.synchronize()
            for g in (c, s, z): g.check()
            for got, w in zip((c.t, s.t, z.t), wants):
                assert torch.equal(got.view(torch.uint8), w[pick].view(torch.uint8)), "h=%d g=%d rows=%d" % (hidden, group, rows)


# by block: for INT4 and FP8 the two limits of the steps of three to eight sources
STEPS = {1024: (((0, 0, 0, 0, 0, 0), (0, 0, 30, 31, 30, 30)), ((0, 0, 0, 0, 0, 0), (0, 0, 33, 31, 28, 29))),
         2048: (((0, 0, 2, 2, 2, 2), (0, 0, 37, 37, 36, 33)), ((0, 0, 3, 3, 3, 3), (0, 0, 34, 32, 33, 32))),
         4096: (((4, 4, 8, 8, 10, 10), (0, 0, 38, 39, 36, 37)), ((6, 6, 9, 8, 10, 10), (0, 44, 40, 40, 41, 45))),
         8192: (((0, 10, 0, 32, 30, 25), (0, 0, 32, 0, 36, 38)), ((8, 16, 0, 32, 28, 24), (0, 0, 38, 38, 38, 42)))}


@pytest.mark.parametrize("quantizer,n_src", [(oracle.ASYM, 3), (oracle.ASYM, 4), (oracle.ASYM, 6), (oracle.ASYM, 8), (oracle.SYM, 5), (oracle.SYM, 7),
                                             (oracle.SYM, 8), (oracle.FP8, 2), (oracle.FP8, 3), (oracle.FP8, 4), (oracle.FP8, 6), (oracle.FP8, 7),
                                             (oracle.FP8, 8)])
@pytest.mark.parametrize("hidden", [1024, 2048, 3072, 4096, 8192])
def test_allreduce_sim_rot_on_both_sides_of_the_limit(fc, quantizer, n_src, hidden):
    # the steps, which write the workspace, and the one launch, which leaves it alone: up to a first limit (2^16 elements; by block, code
    # and number of sources) the steps run, up to a second where the one launch takes the sources in turn.  Slabs of a length that
    # needs padding never run in steps in blocks of 1024.  A few rows (compared with the oracle) are repeated up to the limits.
    bits = 8 if quantizer == oracle.FP8 else 4
    block = hidden & -hidden
    first, second = (STEPS[block][quantizer == oracle.FP8][i][n_src - 3] if n_src >= 3 else 0 for i in range(2))
    turns = {1024: (2 << 20, 2 << 20, 3 << 19), 2048: (2 << 20, 2 << 20, 3 << 19), 4096: (2 << 20, 2 << 20), 8192: (2 << 20, 2 << 20, 0, 2 << 20, 2 << 20, 2 << 20)}[block]
    turns = turns[n_src - 3] if n_src - 3 < len(turns) else 1 << 20      # past so many elements the one launch takes the sources in turn
    x = synth_inputs.make_partials(n_src, 5, hidden, seed=hidden + n_src)
    x[:, 1] = 0
    x[0, 2] = np.float16(6e-8) * (np.arange(hidden) % 5)
    x[:, 3] += np.float16(300.0)
    few = dev(x.view(np.uint16)).view(torch.float16)
    for group in (128, 1024):
        want = dev(oracle.allreduce_sim_rot(x, group, bits, bits, quantizer).view(np.int16))
        few_limit = max(first - 2 * (group == 1024 and n_src <= {1024: 8, 2048: 8, 4096: 6, 8192: 4}[block]), 0) << 16
        edges = {limit // hidden + more for limit in (few_limit, turns, second << 16) for more in (0, 1, 4)}
        for rows in sorted({1, 2, 5, 12} | edges - {0}):
            pick = torch.arange(rows, device="cuda") % 5
            need = fc.allreduce_sim_workspace_bytes(n_src, rows, hidden, group, bits, bits)
            space = torch.full((need + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            y = Guarded((rows, hidden), torch.float16)
            fc.allreduce_sim_rot(few[:, pick], group, bits, bits, quantizer, out=y.t, workspace=space[:need])
            torch.cuda.synchronize(); y.check()
            assert (space[need:] == 0xA5).all(), "written past the workspace"
            elems = rows * hidden
            steps = elems <= few_limit or turns < elems <= second << 16
            steps = steps and (elems // group % 4 == 0 or block != 1024)
            assert bool((space[:need] != 0xA5).any()) == steps, "N=%d h=%d g=%d rows=%d: form" % (n_src, hidden, group, rows)
            assert torch.equal(y.t.view(torch.int16), want[pick]), "N=%d h=%d g=%d rows=%d" % (n_src, hidden, group, rows)


@pytest.mark.parametrize("quantizer,n_src", [(oracle.ASYM, 3), (oracle.ASYM, 4), (oracle.ASYM, 8), (oracle.SYM, 5), (oracle.FP8, 3), (oracle.FP8, 7)])
@pytest.mark.parametrize("hidden", [2048, 4096, 8192])
def test_allreduce_sim_rot_few_coarse_groups(fc, quantizer, n_src, hidden):
    # one to seven groups per partial: the three steps lay one partial's metadata right behind the other's, not on multiples of 16 bytes
    bits = 8 if quantizer == oracle.FP8 else 4
    for group, rows in ((hidden, 1), (hidden, 2), (hidden, 7), (hidden // 2, 1), (hidden // 2, 3)):
        x = synth_inputs.make_partials_stress(n_src, rows, hidden, (rows + n_src) % synth_inputs.STRESS_KINDS, seed=hidden + rows)
        need = fc.allreduce_sim_workspace_bytes(n_src, rows, hidden, group, bits, bits)
        space = torch.full((need + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        y = Guarded((rows, hidden), torch.float16)
        fc.allreduce_sim_rot(dev(x.view(np.uint16)).view(torch.float16), group, bits, bits, quantizer, out=y.t, workspace=space[:need])
        torch.cuda.synchronize(); y.check()
        assert (space[need:] == 0xA5).all(), "written past the workspace"
        want = oracle.allreduce_sim_rot(x, group, bits, bits, quantizer)
        assert same_bits(y.t.cpu().numpy().view(np.uint16), want.view(np.uint16)), "N=%d h=%d g=%d rows=%d" % (n_src, hidden, group, rows)


def test_rot_rejects_unsupported_rows_and_empty_is_noop(fc):
    x = torch.zeros((2, 2560), dtype=torch.float16, device="cuda")           # 5 x 512: blocks below 1024
    with pytest.raises(fc.FcError):
        fc.quantize_rot(x, 128, 4)
    with pytest.raises(fc.FcError):
        fc.quantize_rot(torch.zeros((2, 4096), dtype=torch.float16, device="cuda"), 128, 4, fc.QUANTIZER_FP8)
    c, s, z = fc.quantize_rot(torch.empty((0, 4096), dtype=torch.float16, device="cuda"), 128, 4)
    assert c.shape == (0, 2048) and z.shape == (0, 32)
    torch.cuda.synchronize()


def test_rot_full_size_on_sampled_rows(fc):
    # the headline shape with per-token groups (where the paper finds the rotation pays off)
    w = synth_inputs.WORKLOADS["llama3_70b_prefill"]
    g = w.hidden
    x = synth_inputs.make_partials_device(w.n_src, w.tokens, w.hidden, 11, "cuda", w.outlier_frac, w.outlier_gain)
    rows = np.unique(np.concatenate([[0, w.tokens - 1], np.random.default_rng(5).integers(0, w.tokens, 20)]))
    ridx = torch.from_numpy(rows).cuda()
    y = fc.allreduce_sim_rot(x, g, w.bits_in, w.bits_out)
    stage1 = [fc.quantize_rot(x[j], g, w.bits_in) for j in range(w.n_src)]
    torch.cuda.synchronize()
    xs = x[:, ridx].cpu().numpy()
    for j in range(w.n_src):
        want = oracle.quantize_rot(xs[j], g, w.bits_in)
        got = tuple(a[ridx].cpu().numpy() for a in stage1[j])
        assert_rot_triplet(got, want, oracle.ASYM, "full size stage 1 source %d" % j)
    want = oracle.allreduce_sim_rot(xs, g, w.bits_in, w.bits_out)
    got = y[ridx].cpu().numpy()
    assert same_bits(got.view(np.uint16), want.view(np.uint16)), first_diff(got.view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("hidden", [8192, 5120])
def test_rot_volume_beyond_2_to_32_elements(fc, hidden):
    # element indices and the byte offsets of the input pass 2^32 inside the tensor (for hidden 5120 the blocks of
    # 1024 also end in a half-filled chunk); sampled token rows against the oracle
    group, bits = 128, 4
    tokens = (1 << 32) // hidden + 3
    free, _ = torch.cuda.mem_get_info()
    if free < 40 * (1 << 30):
        pytest.skip("needs 40 GB of free device memory")
    g = torch.Generator(device="cuda"); g.manual_seed(hidden)
    x = torch.empty((tokens, hidden), dtype=torch.float16, device="cuda")
    chunk = 1 << 16
    for r0 in range(0, tokens, chunk):
        r1 = min(tokens, r0 + chunk)
        x[r0:r1] = (torch.randn((r1 - r0, hidden), generator=g, device="cuda") * (1.0 + (r0 // chunk) % 3)).half()
    c, s, z = fc.quantize_rot(x, group, bits)
    y = fc.dequantize_rot(c, s, z, hidden, group, bits)
    torch.cuda.synchronize()
    marks = [0, 1, (1 << 31) // hidden, (1 << 32) // hidden - 1, (1 << 32) // hidden, tokens - 2, tokens - 1]
    rows = np.unique(np.array(marks + list(np.random.default_rng(hidden).integers(0, tokens, 12))))
    ridx = torch.from_numpy(rows).cuda()
    xs = x[ridx].cpu().numpy()
    want = oracle.quantize_rot(xs, group, bits, oracle.ASYM)
    got = (c[ridx].cpu().numpy(), s[ridx].cpu().numpy(), z[ridx].cpu().numpy())
    assert_rot_triplet(got, want, oracle.ASYM, "rows around 2^32 elements, hidden %d" % hidden)
    wy = oracle.dequantize_rot(*want, hidden, group, bits, oracle.ASYM)
    assert same_bits(y[ridx].cpu().numpy().view(np.uint16), wy.view(np.uint16)), "dequantize_rot around 2^32 elements"


@pytest.mark.parametrize("quantizer,bits_rs,bits_ag", [(oracle.ASYM, 4, 8), (oracle.SYM, 8, 4), (oracle.FP8, 8, 8)])
@pytest.mark.parametrize("hidden", [1024, 3072, 2048, 4096, 12288, 8192])
def test_one_launch_allreduce_every_group_and_value_kind(fc, quantizer, bits_rs, bits_ag, hidden):
    # every group a block allows (inside a quad of lanes up to all wavefronts of the block), fan-ins 1 ... 8, an odd
    # number of blocks (half-filled workgroups), values that reach huge zero-points and the top clamp, and rows of
    # zeros of both signs (FP8 keeps the sign of a zero code)
    block = hidden & -hidden
    groups = [g for g in (32, 64, 128, 256, 512, 1024, 2048, 4096, 8192) if g <= block]
    for k, group in enumerate(groups):
        for n_src, kind in (((k % 8) + 1, k % synth_inputs.STRESS_KINDS), (3, 2), (2, None)):
            if kind is None:
                x = np.zeros((n_src, 3, hidden), np.float16)
                x[:, 0] = -0.0
                x[0, 1, ::2] = -0.0
                x[1, 2, block // 2:] = np.float16(-0.0)
                x[1, 2, 5] = 3.0
            else:
                x = synth_inputs.make_partials_stress(n_src, 3, hidden, kind, seed=hidden + group)
            want = oracle.allreduce_sim_rot(x, group, bits_rs, bits_ag, quantizer)
            y = Guarded((3, hidden), torch.float16)
            fc.allreduce_sim_rot(dev(x.view(np.uint16)).view(torch.float16), group, bits_rs, bits_ag, quantizer, out=y.t)
            torch.cuda.synchronize(); y.check()
            got = y.t.cpu().numpy()
            assert same_bits(got.view(np.uint16), want.view(np.uint16)), "q=%d N=%d h=%d g=%d kind %s: %s" % (
                quantizer, n_src, hidden, group, kind, first_diff(got.view(np.uint16), want.view(np.uint16)))


@pytest.mark.parametrize("quantizer,bits_rs,bits_ag", [(oracle.ASYM, 4, 8), (oracle.SYM, 8, 4), (oracle.FP8, 8, 8)])
@pytest.mark.parametrize("hidden", [1024, 3072, 2048, 4096, 12288, 8192])
def test_one_launch_allreduce_both_forms_every_group(fc, quantizer, bits_rs, bits_ag, hidden):
    # launches of at most a workgroup per compute unit (2^20 elements in blocks of 4096, 2^21 in blocks of 8192) have a form of
    # their own, in blocks of 8192 also a layout: the value kinds above in five rows, repeated up to both sides of these limits
    for k, group in enumerate(g for g in (32, 64, 128, 256, 512, 1024, 2048, 4096, 8192) if g <= hidden & -hidden):
        n_src = 1 + k % 3
        x = synth_inputs.make_partials_stress(n_src, 5, hidden, k % synth_inputs.STRESS_KINDS, seed=hidden + group)
        x[:, 1] = np.float16(-0.0)
        x[0, 2, ::2] = 0
        few = dev(x.view(np.uint16)).view(torch.float16)
        want = dev(oracle.allreduce_sim_rot(x, group, bits_rs, bits_ag, quantizer).view(np.int16))
        for rows in (limit // hidden + more for limit in (1 << 20, 1 << 21) for more in (0, 1)):
            pick = torch.arange(rows, device="cuda") % 5
            y = Guarded((rows, hidden), torch.float16)
            fc.allreduce_sim_rot(few[:, pick], group, bits_rs, bits_ag, quantizer, out=y.t)
            torch.cuda.synchronize(); y.check()
            assert torch.equal(y.t.view(torch.int16), want[pick]), "N=%d h=%d g=%d rows=%d" % (n_src, hidden, group, rows)


@pytest.mark.parametrize("quantizer,bits", [(oracle.ASYM, 4), (oracle.SYM, 4), (oracle.FP8, 8)])
@pytest.mark.parametrize("hidden", [1024, 2048, 4096, 8192])
def test_full_chip_runs_repeat(fc, quantizer, bits, hidden):
    # a volume that fills the chip several times over, eight times: the rotated kernels give the same bits every time, and
    # the one-launch all-reduce those of the three steps (a register overwritten while a store still reads it shows
    # in a few wavefronts in ten thousand, never at the sizes of the other tests)
    tokens, group, n_src = (1 << 25) // hidden, 128, 2
    x = synth_inputs.make_partials_device(n_src, tokens, hidden, hidden + bits, "cuda", 0.01, 20.0)
    parts = [[t for t in fc.quantize_rot(x[j], group, bits, quantizer) if t is not None] for j in range(n_src)]
    coded = [torch.stack(p) for p in zip(*parts)]
    fused = {oracle.ASYM: fc.dequant_reduce_requant, oracle.SYM: fc.dequant_reduce_requant_sym,
             oracle.FP8: fc.dequant_reduce_requant_fp8}[quantizer]
    total = fused(*coded, hidden, group, *(() if quantizer == oracle.FP8 else (bits, bits)))
    c, s, z = (*total, None)[:3]
    want = fc.dequantize_rot(c, s, z, hidden, group, bits, quantizer).clone()
    for _ in range(8):
        again = [t for t in fc.quantize_rot(x[0], group, bits, quantizer) if t is not None]
        for a, b in zip(again, parts[0]):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
        y = fc.dequantize_rot(c, s, z, hidden, group, bits, quantizer)
        assert torch.equal(y.view(torch.int16), want.view(torch.int16)), "dequantize_rot does not repeat"
        y = fc.allreduce_sim_rot(x, group, bits, bits, quantizer)
        assert torch.equal(y.view(torch.int16), want.view(torch.int16)), "one launch differs from the three steps"


@pytest.mark.parametrize("quantizer,bits", [(oracle.ASYM, 4), (oracle.ASYM, 8), (oracle.SYM, 4), (oracle.SYM, 8)])
@pytest.mark.parametrize("hidden", [1024, 2048, 4096, 8192])
def test_dequantize_rot_signs_of_zero(fc, quantizer, bits, hidden):
    # the short form of large volumes drops signs of zero inside the transform, the literal one keeps them, and the wavefronts (2048
    # elements) of one block may take different ones: rows that cancel to zeros everywhere, with zero-points and
    # scales out of the short form's reach in all, in one and in none of the wavefronts; fractional zero-points and
    # subnormal scales whose products underflow to -0.  The result must agree in every bit, zeros included.
    group, rows = 128, 12
    rng = np.random.default_rng(hidden + bits)
    top = 1 << bits
    q = np.zeros((rows, hidden), np.uint8)
    s = np.ones((rows, hidden // group), np.float32)
    z = np.zeros((rows, hidden // group), np.float32)
    per_wave = min(2048, hidden) // group
    z[1] = -3000.0                                     # constant rows: one spike, zeros elsewhere
    z[2, :per_wave] = -3000.0
    z[3, -per_wave:] = 3000.0
    q[4:6] = 5
    z[4:6] = 5.0                                       # q - z = 0 everywhere
    s[5, ::3] = np.float32(1e-39)
    z[6] = np.float32(1e-9)                            # d = -1e-9, times a subnormal scale: -0
    s[6] = np.float32(1e-40)
    z[7, :per_wave] = np.float32(1e-9)
    s[7, :per_wave] = np.float32(1e-40)
    s[8, -1] = np.float32(1e-42)
    q[9] = rng.integers(0, top, hidden)
    z[9, ::5] = 2500.0
    q[10] = rng.integers(0, top, hidden)
    q[11] = rng.integers(0, top, hidden)
    s[11] = np.exp(rng.uniform(-95, 60, s.shape[1])).astype(np.float32)
    codes = q if bits == 8 else (q[:, ::2] | (q[:, 1::2] << 4)).astype(np.uint8)
    want = oracle.dequantize_rot(codes, s, z, hidden, group, bits, quantizer)
    y = Guarded((rows, hidden), torch.float16)
    fc.dequantize_rot(dev(codes), dev(s), dev(z), hidden, group, bits, quantizer, out=y.t)
    torch.cuda.synchronize(); y.check()
    got = y.t.cpu().numpy()
    for r in range(rows):
        assert same_bits(got[r].view(np.uint16), want[r].view(np.uint16)), \
            "row %d h=%d b=%d q=%d: %s" % (r, hidden, bits, quantizer, first_diff(got[r].view(np.uint16), want[r].view(np.uint16)))
    # the same rows over and over in volumes past the limits of the launch-bound forms, which have the literal form only
    pick = torch.arange((4 << 20) // hidden + 1, device="cuda") % rows
    y = Guarded((pick.numel(), hidden), torch.float16)
    fc.dequantize_rot(dev(codes)[pick], dev(s)[pick], dev(z)[pick], hidden, group, bits, quantizer, out=y.t)
    torch.cuda.synchronize(); y.check()
    same = (y.t.view(torch.int16) == dev(want.view(np.int16))[pick]).all(dim=1)
    assert same.all(), "rows %s of 12, h=%d b=%d q=%d" % (sorted(set((torch.nonzero(~same)[:, 0] % rows).tolist())), hidden, bits, quantizer)


@pytest.mark.parametrize("quantizer", [oracle.ASYM, oracle.SYM, oracle.FP8])
@pytest.mark.parametrize("n_src", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("hidden", [1024, 2048, 4096, 8192])
def test_allreduce_sim_rot_sources_side_by_side(fc, quantizer, n_src, hidden):
    # few elements: the sources of a block go side by side through one workgroup, up to 2^21 elements and one round of workgroups, in two
    # rounds from six sources on in blocks of 8192; shorter blocks with 8 elements per lane up to 2^21 elements of all sources together, less in
    # blocks of 1024 and of a single source.
    # Rows on both sides of that, an odd number of blocks of 1024 among them
    bits = 8 if quantizer == oracle.FP8 else 4
    waves = max(1, hidden // 2048)
    parts = min(n_src, 4 if hidden == 8192 else 8)
    limit = min(1 << 21, 256 * (16 // (waves * parts)) * waves * 2048) // hidden
    x = synth_inputs.make_partials(n_src, 5, hidden, seed=hidden + n_src, outlier_frac=0.01)
    x[:, 1] = 0
    x[0, 2] = np.float16(6e-8) * (np.arange(hidden) % 5)
    x[:, 3] += np.float16(300.0)
    x[n_src - 1, 4] = np.float16(-0.0)
    few = dev(x.view(np.uint16)).view(torch.float16)
    for group in (64, hidden):
        want = dev(oracle.allreduce_sim_rot(x, group, bits, bits, quantizer).view(np.int16))
        quarters = {1024: 6 - (n_src == 1), 2048: 8 - 2 * (n_src == 1)}.get(hidden, 8)
        fine = (quarters << 18) // n_src // hidden
        for rows in (1, 3, fine, fine + 1, limit - 1, limit, limit + 1):
            pick = torch.arange(rows, device="cuda") % 5
            y = Guarded((rows, hidden), torch.float16)
            fc.allreduce_sim_rot(few[:, pick], group, bits, bits, quantizer, out=y.t)
            torch.cuda.synchronize(); y.check()
            assert torch.equal(y.t.view(torch.int16), want[pick]), "N=%d h=%d g=%d rows=%d" % (n_src, hidden, group, rows)


@pytest.mark.parametrize("quantizer,bits", [(oracle.ASYM, 4), (oracle.ASYM, 8), (oracle.SYM, 4), (oracle.SYM, 8), (oracle.FP8, 8)])
@pytest.mark.parametrize("hidden", [1024, 2048, 4096, 8192])
def test_rot_codecs_on_both_sides_of_the_volume_limits(fc, quantizer, bits, hidden):
    # 2^20, 5 * 2^18, 3 * 2^19, 2^21, 5 * 2^19 and 2^22 elements, where other forms of the rotated quantizer and dequantizer take over
    x = synth_inputs.make_partials(1, 5, hidden, seed=hidden + bits, outlier_frac=0.01)[0]
    x[1] = 0
    x[2] = np.float16(6e-8) * (np.arange(hidden) % 5)
    x[3] += np.float16(300.0)
    x[4, ::3] = np.float16(-0.0)
    few = dev(x.view(np.uint16)).view(torch.float16)
    for group in (32, 256, hidden):
        coded = oracle.quantize_rot(x, group, bits, quantizer)
        back = dev(oracle.dequantize_rot(*coded, hidden, group, bits, quantizer).view(np.int16))
        want = [dev(np.ascontiguousarray(a).view(np.uint8)) for a in coded[:3 if quantizer == oracle.ASYM else 2]]
        for limit in (1 << 20, 5 << 18, 3 << 19, 1 << 21, 5 << 19, 1 << 22):
            for rows in (1, limit // hidden, limit // hidden + 1):
                pick = torch.arange(rows, device="cuda") % 5
                got = fc.quantize_rot(few[pick], group, bits, quantizer)
                what = "h=%d g=%d rows=%d" % (hidden, group, rows)
                for a, w in zip(got, want):
                    assert torch.equal(a.view(torch.uint8), w[pick]), what
                y = Guarded((rows, hidden), torch.float16)
                fc.dequantize_rot(got[0], got[1], got[2] if quantizer == oracle.ASYM else None, hidden, group, bits, quantizer, out=y.t)
                torch.cuda.synchronize(); y.check()
                assert torch.equal(y.t.view(torch.int16), back[pick]), what


@pytest.mark.parametrize("quantizer", [oracle.ASYM, oracle.SYM])
@pytest.mark.parametrize("bits_rs,bits_ag", [(4, 8), (8, 4)])
@pytest.mark.parametrize("hidden,group", [(1024, 32), (3072, 1024), (2048, 2048), (4096, 64), (8192, 8192), (8192, 512)])
def test_allreduce_sim_rot_in_steps(fc, quantizer, bits_rs, bits_ag, hidden, group):
    # few rows of many sources: the sum, its codes and the inverse transform in one launch.  Zero-points far outside the codes, sums that
    # cancel to zero, partials of -0 and subnormals, groups of less and more than a wavefront
    short = hidden & -hidden <= 2048
    for n_src in (6 if short else 5, 7, 8):
        rows = (1 << 20) // hidden + 1 if short else 12
        x = synth_inputs.make_partials(n_src, 12, hidden, seed=hidden + group + n_src, outlier_frac=0.01)
        x[:, 1] = 0
        x[:, 2] = np.float16(-0.0)
        x[:, 3] += np.float16(300.0)
        x[1::2, 4] = -x[: n_src // 2 * 2 : 2, 4]
        x[:, 5] = np.float16(6e-8) * (np.arange(hidden) % 5)
        x[:, 6] *= np.float16(60.0)
        want = oracle.allreduce_sim_rot(x, group, bits_rs, bits_ag, quantizer).view(np.uint16)
        pick = np.arange(rows) % 12
        need = fc.allreduce_sim_workspace_bytes(n_src, rows, hidden, group, bits_rs, bits_ag)
        space = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
        y = Guarded((rows, hidden), torch.float16)
        fc.allreduce_sim_rot(dev(x.view(np.uint16)).view(torch.float16)[:, torch.from_numpy(pick).cuda()], group, bits_rs, bits_ag, quantizer, out=y.t, workspace=space)
        torch.cuda.synchronize(); y.check()
        assert hidden // group * rows % 4 or (space != 0xA5).any(), "not in steps: N=%d h=%d g=%d" % (n_src, hidden, group)
        assert np.array_equal(y.t.cpu().numpy().view(np.uint16), want[pick]), "N=%d h=%d g=%d %d->%d" % (n_src, hidden, group, bits_rs, bits_ag)
