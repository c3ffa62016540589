"""GPU parity of the several-workgroup TopK engine at the edges of its
exchanges, bit for bit against the CPU oracle: last chunks that are barely or
almost filled, one to 256 workgroups per segment, more segments than are
resident at once, every layout (runs per thread), and data that takes each way
through the exchanges -- chunks whose magnitudes differ by octaves (the
window guesses miss), a gap around the threshold, ties in one key per
workgroup (multiplicities), many distinct keys on the prefix (records
overflow), all zeros, thresholds among the subnormals."""
import pytest
import torch

from gpu_helpers import TORCH, assert_bits_equal, check_block_table, raw

pytestmark = pytest.mark.gpu


def make(kind, shape, dt, seed):
    g = torch.Generator().manual_seed(seed)
    z = torch.randn(shape, generator=g)
    L = shape[-1]
    if kind == "ties":           # few distinct magnitudes
        z = torch.randint(-4, 5, shape, generator=g).float() * 0.25
    elif kind == "zero":
        z = torch.zeros(shape)
    elif kind == "octaves":      # chunk magnitudes from 2^-10 to 2^6
        z = z * torch.exp2(torch.linspace(-10, 6, L).round())
    elif kind == "gap":          # a tenth of the values far above the rest
        z = torch.where(torch.rand(shape, generator=g) < 0.1, z.sign() * (4 + z.abs()), z * 0.01)
    elif kind == "dense":        # everything inside one narrow magnitude interval
        z = 1.0 + torch.rand(shape, generator=g) * 2.0 ** -9
    return z.to(TORCH[dt])


# (n_seg, seg_len, dtype, kind): chunk lengths are 2048 r elements for 4-byte
# types (r = 1, 2, 4, 6) and 4096 r for 2-byte types (r = 1, 2, 3)
SHAPES = [(1, 32769, "f16"), (1, 36865, "bf16"), (3, 40960, "f16"), (2, 12288 * 4 + 1, "f32"), (9, 61441, "f32"),
          (5, 100003, "f16"), (70, 33000, "bf16"), (8, 200001, "f16"), (1, 400003, "f32"), (1, 1100001, "bf16"),
          (1, 2500003, "f32"), (1, 3145728, "bf16")]
KINDS = ["normal", "ties", "zero", "octaves", "gap", "dense"]
CASES = [(n, L, dt, KINDS[(i + j) % len(KINDS)]) for i, (n, L, dt) in enumerate(SHAPES) for j in (0, 3)] + [
    (2, 70001, dt, kind) for dt in ("f32", "bf16") for kind in KINDS]


@pytest.mark.parametrize("n_seg,L,dt,kind", CASES)
def test_group_parity(tc, orc, n_seg, L, dt, kind):
    for k in sorted({1, L // 10, L - 1}):
        x = make(kind, (n_seg, L), dt, 7)
        e0 = (make("normal", (n_seg, L), "f32", 8) * 0.01) if kind in ("normal", "octaves") else torch.zeros(n_seg, L)
        ed = e0.cuda().reshape(-1).contiguous()
        pl = tc.ef_step_topk(x.cuda(), ed, k, n_seg)
        torch.cuda.synchronize()
        oi, ov, oe = orc.ef_topk(raw(x), dt, e0.numpy(), n_seg, L, k)
        what = f"{n_seg}x{L} {dt} {kind} k={k}"
        assert_bits_equal(raw(pl.idx), oi, f"idx {what}")
        assert_bits_equal(raw(pl.val), ov, f"val {what}")
        assert_bits_equal(raw(ed).reshape(n_seg, L), oe, f"e {what}")
        check_block_table(pl.blk, oi, L, what)
    assert tc.device_errors() == 0


def tiny(shape, dt, b, seed):
    """zeros and, denser in the first half of a segment than in the second,
    subnormal or barely normal magnitudes whose key has b in bits 30..19"""
    g = torch.Generator().manual_seed(seed)
    p = torch.where(torch.arange(shape[-1]) < shape[-1] // 2, 0.13, 0.08)
    low = torch.randint(0 if b else 1, 1 << 19, shape, generator=g)
    key = torch.where(torch.rand(shape, generator=g) < p, (b << 19) + low, 0)
    key += torch.randint(0, 2, shape, generator=g) << 31
    if dt == "bf16":
        return (key >> 16).to(torch.int32).to(torch.int16).view(torch.bfloat16)
    return torch.where(key >= 1 << 31, key - (1 << 32), key).to(torch.int32).view(torch.float32)


@pytest.mark.parametrize("b", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("L,dt", [(40000, "f32"), (70001, "f32"), (40000, "bf16"), (70001, "bf16")])
def test_group_threshold_near_zero(tc, orc, L, dt, b):
    """k-th magnitudes in the lowest bins of the first histogram: with k a tenth
    of the segment the workgroups of its first half guess bin b and those of
    its second half bin 0, whose window has no neighbour below"""
    n, k = 2, L // 10
    x = tiny((n, L), dt, b, 11)
    ids = torch.arange(n, dtype=torch.int64)
    ed, eo = torch.zeros(n * L, device="cuda"), torch.zeros(n, L).numpy()
    md = torch.zeros((n, L), dtype=TORCH[dt], device="cuda")
    mo = raw(md).copy()
    plain = tc.topk_compress(x.cuda(), k, n)
    ef = tc.ef_step_topk(x.cuda(), ed, k, n)
    aq = tc.aqsgd_step(x.cuda(), md, ids.cuda(), k)
    torch.cuda.synchronize()
    pi, pv = orc.topk_compress(raw(x), dt, n, L, k)
    oi, ov, oe = orc.ef_topk(raw(x), dt, eo, n, L, k)
    ai, av = orc.aqsgd_send(raw(x), mo, dt, ids.numpy(), k)
    for what, pl, wi, wv in (("plain", plain, pi, pv), ("EF", ef, oi, ov), ("AQ-SGD", aq, ai, av)):
        assert_bits_equal(raw(pl.idx), wi, f"idx {what}")
        assert_bits_equal(raw(pl.val), wv, f"val {what}")
        check_block_table(pl.blk, wi, L, what)
    assert_bits_equal(raw(ed).reshape(n, L), oe, "e")
    assert_bits_equal(raw(md), mo, "m")
    assert tc.device_errors() == 0


@pytest.mark.parametrize("n_seg,L,dt", [(1, 40000, "f32"), (2, 300001, "f32"), (1, 3000000, "f32"), (20, 65000, "f32"),
                                        (2, 300001, "bf16")])
@pytest.mark.parametrize("spread", [2.0 ** -9, 2.0 ** -6])
def test_group_records_overflow(tc, orc, n_seg, L, dt, spread):
    """distinct keys on T's prefix in every workgroup, in some, and in none that
    ranks before: with the prefix from the windows, and with one that a digit
    pass gave (chunks of other magnitudes make the windows miss)"""
    g = torch.Generator().manual_seed(19)
    for miss in (False, True):
        x = 1.0 + torch.rand((n_seg, L), generator=g) * spread
        x[:, L // 2:L // 2 + L // 4] = 1.0 + spread / 3          # one key, many times
        if miss:
            x[:, :L // 5] *= 2.0 ** -8
        x = x.to(TORCH[dt])
        for k in (1, L // 10, L // 2, L * 7 // 8):
            e = torch.zeros(n_seg * L, device="cuda")
            pl = tc.ef_step_topk(x.cuda(), e, k, n_seg)
            torch.cuda.synchronize()
            oi, ov, oe = orc.ef_topk(raw(x), dt, torch.zeros(n_seg, L).numpy(), n_seg, L, k)
            what = f"{n_seg}x{L} {dt} spread {spread} miss {miss} k={k}"
            assert_bits_equal(raw(pl.idx), oi, f"idx {what}")
            assert_bits_equal(raw(pl.val), ov, f"val {what}")
            assert_bits_equal(raw(e).reshape(n_seg, L), oe, f"e {what}")
    assert tc.device_errors() == 0


def test_group_aqsgd_repeated_activations(tc, orc):
    """the same two activations in turn: after a few visits the changes have a
    gap around the threshold, repeat in few values, or are all zero"""
    n, L = 3, 60001
    k = L * 3 // 10
    m0 = make("normal", (n, L), "f16", 1)
    acts = [(m0.float() + 0.1 * make("normal", (n, L), "f32", 2 + v)).half() for v in range(2)] + [m0]
    ids = torch.arange(n, dtype=torch.int64)
    md, mo = m0.cuda(), raw(m0).copy()
    for v in [0, 1] * 4 + [2] * 5:
        a = acts[v]
        pl = tc.aqsgd_step(a.cuda(), md, ids.cuda(), k)
        torch.cuda.synchronize()
        oi, ov = orc.aqsgd_send(raw(a), mo, "f16", ids.numpy(), k)
        assert_bits_equal(raw(pl.idx), oi, f"idx visit of {v}")
        assert_bits_equal(raw(pl.val), ov, f"val visit of {v}")
        assert_bits_equal(raw(md), mo, f"m visit of {v}")
    assert tc.device_errors() == 0
