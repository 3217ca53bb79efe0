"""Parity of the norm-and-sign quantizer (cgx_qsgd_* through the C ABI) with the CPU oracle.

Bar as for the min/max form: packed stream and meta bit-exact; sums bit-exact against
the oracle's ordered binary32 sum and within 1e-6 * sum_w |deq_w| of its binary64 sum.
Chunks fed to the reduce come from the oracle's quantizer, never from the GPU.
"""
import numpy as np
import pytest

from paper_2111_08617_amd import binding as cgx
from paper_2111_08617_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "these tests need the MI355X"
    cgx.lib()
    return t


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def no_one_bit(w):
    """The same workload with its 1-bit layers widened to 2 bits (a sign bit alone carries no level)."""
    w.bits = np.where(w.bits == 1, 2, w.bits).astype(np.uint8)
    return w


def gpu_quantize(torch, grad, offsets, bits, bucket, seed, dt):
    plan = cgx.Plan(offsets, bits, bucket, dt)
    pb, mb = cgx.cgx_qsgd_sizes(plan)
    packed = torch.full((pb + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    meta = torch.full((mb // 4 + 16,), -7.0, dtype=torch.float32, device="cuda")
    g = grad if isinstance(grad, torch.Tensor) else dev(torch, grad)
    cgx.cgx_qsgd_quantize(g, plan, seed, packed, meta)
    torch.cuda.synchronize()
    p, m = packed.cpu().numpy(), meta.cpu().numpy()
    assert (p[pb:] == 0xA5).all() and (m[mb // 4:] == -7.0).all(), "wrote past the reported sizes"
    return p[:pb], m[:mb // 4]


def device_chunks(torch, chunks, metas):
    dp = [dev(torch, c) for c in chunks]
    dm = [dev(torch, m) if m.size else torch.zeros(4, device="cuda") for m in metas]
    return dp, dm


def gpu_reduce(torch, chunks, metas, offsets, bits, bucket, dt):
    plan = cgx.Plan(offsets, bits, bucket, dt)
    dp, dm = device_chunks(torch, chunks, metas)
    total = torch.full((plan.n + 16,), 123.0, dtype=torch.float32, device="cuda")
    cgx.cgx_qsgd_dequant_reduce(dp, dm, plan, total)
    torch.cuda.synchronize()
    out = total.cpu().numpy()
    assert (out[plan.n:] == 123.0).all(), "wrote past the end of the sum"
    return out[:plan.n], total


def gpu_fused(torch, chunks, metas, offsets, bits, bucket, dt, seed, layered=False):
    """layered: the same plan with its bucket size given layer by layer, which always runs in chunks of 2048 elements."""
    plan = cgx.LayeredPlan(offsets, bits, np.full(len(bits), bucket, np.int32), dt) if layered else cgx.Plan(offsets, bits, bucket, dt)
    pb, mb = cgx.cgx_qsgd_sizes(cgx.Plan(offsets, bits, bucket, wl.F32))
    dp, dm = device_chunks(torch, chunks, metas)
    packed = torch.full((pb + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    meta = torch.full((mb // 4 + 16,), -7.0, dtype=torch.float32, device="cuda")
    fused = cgx.cgx_qsgd_layered_dequant_reduce_requantize if layered else cgx.cgx_qsgd_dequant_reduce_requantize
    fused(dp, dm, plan, seed, packed, meta)
    torch.cuda.synchronize()
    p, m = packed.cpu().numpy(), meta.cpu().numpy()
    assert (p[pb:] == 0xA5).all() and (m[mb // 4:] == -7.0).all(), "wrote past the reported sizes"
    return p[:pb], m[:mb // 4]


def assert_same_chunk(gp, gm, op, om, what=""):
    assert gm.tobytes() == om.tobytes(), f"{what}: meta differs in {int((gm.view(np.uint32) != om.view(np.uint32)).sum())} words"
    if not np.array_equal(gp, op):
        bad = np.nonzero(gp != op)[0]
        raise AssertionError(f"{what}: packed differs in {bad.size} bytes, first at {bad[:5]}")


def assert_sum_parity(got, ref, what=""):
    g, r = got.view(np.uint32), ref["sum32"].view(np.uint32)
    assert np.array_equal(g, r), f"{what}: {int((g != r).sum())} sums differ from the ordered binary32 sum"
    err = np.abs(got.astype(np.float64) - ref["sum64"])
    assert (err <= 1e-6 * ref["abs64"] + 1e-45).all(), f"{what}: worst relative error {np.max(err / (ref['abs64'] + 1e-300))}"


def full_cycle(torch, oracle, w, W, what=""):
    chunks, metas = [], []
    for peer in range(W):
        g = w.gradient(peer)
        seed = w.quant_seed(peer)
        op, om = oracle.qsgd_quantize(g, w.offsets, w.bits, w.bucket, seed, w.dt)
        if peer < 2:
            gp, gm = gpu_quantize(torch, g, w.offsets, w.bits, w.bucket, seed, w.dt)
            assert_same_chunk(gp, gm, op, om, f"{what} quantize peer {peer}")
        chunks.append(op)
        metas.append(om)
    ref = oracle.qsgd_dequant_reduce(chunks, metas, w.offsets, w.bits, w.bucket, w.dt)
    got, total = gpu_reduce(torch, chunks, metas, w.offsets, w.bits, w.bucket, w.dt)
    assert_sum_parity(got, ref, f"{what} reduce")
    rp, rm = gpu_quantize(torch, total[:w.n], w.offsets, w.bits, w.bucket, 99, wl.F32)
    op, om = oracle.qsgd_quantize(got, w.offsets, w.bits, w.bucket, 99, wl.F32)
    assert_same_chunk(rp, rm, op, om, f"{what} requantize")
    if W <= cgx.MAX_FUSED_PEERS:
        fp, fm = gpu_fused(torch, chunks, metas, w.offsets, w.bits, w.bucket, w.dt, 99)
        op, om = oracle.qsgd_quantize(ref["sum32"], w.offsets, w.bits, w.bucket, 99, wl.F32)
        assert_same_chunk(fp, fm, op, om, f"{what} fused reduce+requantize")
        if w.dt == wl.F32:            # short binary32 buffers run in chunks of 1024 elements; here in chunks of 2048
            fp, fm = gpu_fused(torch, chunks, metas, w.offsets, w.bits, w.bucket, w.dt, 99, layered=True)
            assert_same_chunk(fp, fm, op, om, f"{what} fused reduce+requantize, a bucket size per layer")


@pytest.mark.parametrize("seed", range(24))
def test_random_plans(torch, oracle, seed):
    """Seeded random plans (1-bit layers widened to 2 bits) through the whole cycle."""
    w = no_one_bit(wl.random_plan(seed))
    if w.n == 0:
        pytest.skip("empty plan (covered by the edge cases)")
    full_cycle(torch, oracle, w, W=w.W, what=f"random plan {seed} (bucket {w.bucket}, bits {w.bits.tolist()})")


@pytest.mark.parametrize("dt", [wl.F32, wl.F16], ids=["f32", "f16"])
@pytest.mark.parametrize("bucket", [32, 96, 128, 512, 4096, 8192])
def test_edge_case_plan(torch, oracle, bucket, dt):
    """Bit widths 2..8, pass-through, empty, tiny and ragged layers, odd offsets."""
    w = no_one_bit(wl.tiny_mixed(seed=bucket + dt, dt=dt, bucket=bucket))
    full_cycle(torch, oracle, w, W=3, what=f"qsgd tiny_mixed B={bucket}")


@pytest.mark.parametrize("dt", [wl.F32, wl.F16], ids=["f32", "f16"])
@pytest.mark.parametrize("bucket", [32, 64, 128, 256, 512, 1024, 2048])
def test_vectorised_path_all_bit_widths(torch, oracle, bucket, dt):
    sizes = [2048 * 3, 2048 * 2 + 40, 8, 2048, 2048 * 5 + 1000, 2048 * 4, 16384, 2048 + bucket, 6144, 8192 * 2 + 24]
    bits = [2, 2, 0, 3, 4, 5, 0, 6, 7, 8]
    w = wl.Workload("chunks", [(s,) for s in sizes], np.array(bits, np.uint8), bucket, dt, 4, 2000 + bucket,
                    wl._normal, np.linspace(0.01, 2.0, len(sizes)))
    full_cycle(torch, oracle, w, W=4, what=f"qsgd chunks B={bucket}")


@pytest.mark.parametrize("W", [1, 5, 16, 17, 40])
def test_peer_counts(torch, oracle, W):
    """Every peer-block size of a launch, and more peers than one launch takes."""
    sizes = [2048 * 2, 2048 + 24, 2048 * 3, 100]
    w = wl.Workload("peers", [(s,) for s in sizes], np.array([4, 3, 8, 0], np.uint8), 128, wl.F32, W, 77 + W,
                    wl._normal, np.ones(len(sizes)))
    full_cycle(torch, oracle, w, W=W, what=f"qsgd W={W}")


def test_signed_zeros_constant_and_non_finite_values(torch, oracle):
    """Zeros of either sign decode to +0; a non-finite value zeroes the bucket's unit; both
    sides agree bit for bit."""
    rng = np.random.default_rng(5)
    n, B = 2048 * 3 + 200, 128
    x = rng.standard_normal(n).astype(np.float32)
    x[:B] = 0.0
    x[5] = -0.0
    x[B:2 * B] = -3.5                                   # constant bucket: every level is the top one
    x[2 * B + 3] = np.inf
    x[3 * B + 9] = -np.inf
    x[4 * B + 1] = np.nan
    x[5 * B:6 * B] = np.float32(1e-42) * rng.integers(-3, 4, B)   # subnormal magnitudes
    x[-150:] = np.abs(x[-150:])                          # a one-signed ragged tail
    off, bits = np.array([0, n], np.int64), np.array([4], np.uint8)
    op, om = oracle.qsgd_quantize(x, off, bits, B, 11)
    gp, gm = gpu_quantize(torch, x, off, bits, B, 11, wl.F32)
    assert_same_chunk(gp, gm, op, om, "qsgd special values")
    ref = oracle.qsgd_dequant_reduce([op, op], [om, om], off, bits, B)
    got, _ = gpu_reduce(torch, [op, op], [om, om], off, bits, B, wl.F32)
    assert np.array_equal(got.view(np.uint32), ref["sum32"].view(np.uint32))
    assert not np.signbit(got[5]) and got[5] == 0.0 and (got[B:2 * B] == -7.0).all()


def test_resnet50_config_full_size(torch, oracle):
    """161 tensors, 25.6M elements, 4 bit, bucket 1024, small tensors pass-through, W = 8."""
    full_cycle(torch, oracle, no_one_bit(wl.resnet50()), W=8, what="qsgd resnet50")


@pytest.mark.parametrize("name", ["gpt2_medium", "bert_base", "decoder_1p3b"])
def test_large_configs_full_size(torch, oracle, name):
    """gpt2_medium (355M elements, binary16 storage, 4 bit, bucket 128), bert_base (109M, widths from
    {2,3,4,8}, bucket 512: the odd width) and decoder_1p3b (1.3G, widths from {2,4,8}, bucket 1024):
    quantize the full buffer; reduce over W = 8, requantize and the fused form on one rank's 1/8 share."""
    w = no_one_bit(wl.WORKLOADS[name]())
    g = w.gradient(0, threads=16)
    gp, gm = gpu_quantize(torch, g, w.offsets, w.bits, w.bucket, w.quant_seed(0), w.dt)
    op, om = oracle.qsgd_quantize(g, w.offsets, w.bits, w.bucket, w.quant_seed(0), w.dt)
    assert_same_chunk(gp, gm, op, om, f"qsgd {name} quantize")
    del g, gp, op
    first, sub_off, sub_bits = wl.share_subplan(w.offsets, w.bits, w.bucket, w.W, 5)
    m = int(sub_off[-1])
    chunks, metas = [], []
    for peer in range(w.W):
        x = w.gradient(peer, first, first + m, threads=16)
        op, om = oracle.qsgd_quantize(x, sub_off, sub_bits, w.bucket, w.quant_seed(peer), w.dt)
        chunks.append(op)
        metas.append(om)
    ref = oracle.qsgd_dequant_reduce(chunks, metas, sub_off, sub_bits, w.bucket, w.dt)
    got, total = gpu_reduce(torch, chunks, metas, sub_off, sub_bits, w.bucket, w.dt)
    assert_sum_parity(got, ref, f"qsgd {name} share reduce")
    fp, fm = gpu_fused(torch, chunks, metas, sub_off, sub_bits, w.bucket, w.dt, 7)
    op, om = oracle.qsgd_quantize(ref["sum32"], sub_off, sub_bits, w.bucket, 7, wl.F32)
    assert_same_chunk(fp, fm, op, om, f"qsgd {name} share fused reduce+requantize")
    rp, rm = gpu_quantize(torch, got, sub_off, sub_bits, w.bucket, 7, wl.F32)
    assert_same_chunk(rp, rm, op, om, f"qsgd {name} share requantize")


@pytest.mark.parametrize("dt", [wl.F32, wl.F16], ids=["f32", "f16"])
@pytest.mark.parametrize("bucket", [4096, 8192])
def test_buckets_longer_than_a_chunk(torch, oracle, bucket, dt):
    sizes = [bucket * 3, bucket + 40, 8, bucket * 2, bucket * 2 + 1000, 4, bucket, 16384, bucket * 4 + 24, 100, bucket * 2]
    bits = [2, 2, 0, 3, 4, 5, 0, 6, 7, 8, 4]
    w = wl.Workload("wide", [(s,) for s in sizes], np.array(bits, np.uint8), bucket, dt, 3, 600 + bucket,
                    wl._normal, np.linspace(0.01, 2.0, len(sizes)))
    full_cycle(torch, oracle, w, W=3, what=f"qsgd wide B={bucket}")


@pytest.mark.parametrize("dt", [wl.F32, wl.F16], ids=["f32", "f16"])
@pytest.mark.parametrize("bucket", [32, 512, 8192])
def test_layers_that_start_anywhere(torch, oracle, bucket, dt):
    sizes = [2048 * 3 + 1, 2048 * 2, 7, 8192 + 3, 2048 * 4 + 2, 1, 8192 * 2, 4096 + 5, 2048 * 5, 3, 8192 + 4096]
    bits = [4, 2, 0, 3, 8, 0, 0, 5, 2, 0, 7]
    w = wl.Workload("shifted", [(s,) for s in sizes], np.array(bits, np.uint8), bucket, dt, 3, 800 + bucket,
                    wl._normal, np.linspace(0.01, 2.0, len(sizes)))
    full_cycle(torch, oracle, w, W=3, what=f"qsgd shifted B={bucket}")


@pytest.mark.parametrize("dt", [wl.F32, wl.F16], ids=["f32", "f16"])
@pytest.mark.parametrize("bits", range(2, 9))
@pytest.mark.parametrize("start", [0, 2, 4, 7])
def test_draws_follow_where_the_tiles_start(torch, oracle, start, bits, dt):
    """Quantized tiles on multiples of 8 elements, on even and on odd ones; both signs of the top level (of a norm whose scale
    is rounded up) and zeros of either sign."""
    sizes = [start] * (start > 0) + [2048 * 3 + 8 * 5 + 3]
    w = wl.Workload("start", [(s,) for s in sizes], np.array([0] * (start > 0) + [bits], np.uint8), 128, dt, 2, 60 + start,
                    wl._normal, np.full(len(sizes), 0.3))
    full_cycle(torch, oracle, w, W=2, what=f"start {start} bits {bits}")
    levels = ((1 << bits - 1) - 1) * 65536
    a = next(a for a in 1.0 + np.arange(1, 1024) / 1024 if float(np.float32(levels) / np.float32(a)) * a > levels)
    g = np.array([-a, 0.0, a, -0.0], w.gradient(0).dtype)[np.arange(w.n) % 4]
    op, om = oracle.qsgd_quantize(g, w.offsets, w.bits, w.bucket, 3, w.dt)
    gp, gm = gpu_quantize(torch, g, w.offsets, w.bits, w.bucket, 3, w.dt)
    assert_same_chunk(gp, gm, op, om, "top levels and zeros")


@pytest.mark.parametrize("dt", [wl.F32, wl.F16], ids=["f32", "f16"])
@pytest.mark.parametrize("bits", range(2, 9))
@pytest.mark.parametrize("bucket", [96, 128, 4096])
def test_ends_within_a_group_where_all_values_have_one_sign(torch, oracle, bucket, bits, dt):
    """Layers that end 1 to 7 elements into a group of 8, all values negative or all positive."""
    shifted = lambda rng, n, scale: (scale + 0.7 * rng.standard_normal(n)).astype(np.float32)
    sizes = [length for end in range(1, 8) for length in (end, 8 * 5 + end, bucket + end, 2048 + bucket + 8 * 3 + end)]
    w = wl.Workload("one sign", [(s,) for s in sizes], np.full(len(sizes), bits, np.uint8), bucket, dt, 2, 60 + bits, shifted,
                    np.where(np.arange(len(sizes)) // 2 % 2 == 0, -3.0, 3.0))
    full_cycle(torch, oracle, w, W=2, what="one sign")


@pytest.mark.parametrize("bits", range(2, 9))
@pytest.mark.parametrize("bucket", [32, 96, 1024])
def test_units_of_any_size(torch, oracle, bucket, bits):
    """Chunks with units that a quantizer of another program may write: the smallest, subnormal and small ones, the
    largest, zeros of either sign, negative ones and values that are not finite; every code occurs."""
    n, W = 2048 * 2 + 96 * 5, 5
    off, widths = np.array([0, n], np.int64), np.array([bits], np.uint8)
    rng = np.random.default_rng(bits * 10000 + bucket)
    x = rng.standard_normal(n).astype(np.float32)
    chunk, meta = oracle.qsgd_quantize(x, off, widths, bucket, 1)
    small = np.float32(2.0 ** -120)
    special = np.array([1.4e-45, 1e-40, 1.1754942e-38, np.nextafter(small, np.float32(0)), -small, 0.0, -0.0, small, -1.0, 1.0, 3e38,
                        np.inf, np.nan], np.float32)
    chunks = [rng.integers(0, 256, chunk.size, dtype=np.uint8) for _ in range(W)]
    for units in (special, special[5:]):       # with subnormal units in a chunk, and without
        metas = [rng.choice(units, meta.size).astype(np.float32) for _ in range(W)]
        ref = oracle.qsgd_dequant_reduce(chunks, metas, off, widths, bucket, wl.F32)["sum32"]
        got, _ = gpu_reduce(torch, chunks, metas, off, widths, bucket, wl.F32)
        same = got.view(np.uint32) == ref.view(np.uint32)
        assert (same | (np.isnan(got) & np.isnan(ref))).all(), f"{bits} bits, buckets of {bucket}: sums differ"
