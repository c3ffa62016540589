"""GPU parity of the one-wavefront TopK engine (rows of up to 2048 elements),
bit for bit against the CPU oracle, where its layout and its threshold search
can go wrong: rows that end inside a piece of four, inside a wavefront's 256
elements or just past them, rows and pointers that are not 16-byte aligned,
one to all entries kept, and data that takes each way through the search --
the window over the first guess misses the threshold (magnitudes over many
octaves, one value far above the rest, subnormals), one bin holds every key,
few distinct magnitudes, all zeros, half zeros."""
import numpy as np
import pytest
import torch

from gpu_helpers import TORCH, assert_bits_equal, check_block_table, raw

pytestmark = pytest.mark.gpu

KINDS = ["normal", "relu", "ties", "zero", "octaves", "spike", "dense", "tiny"]
LENGTHS = [1, 2, 3, 4, 5, 63, 255, 256, 257, 511, 768, 1021, 1024, 1025, 1537, 2047, 2048]
N = 5


def make(kind, shape, dt, seed):
    g = torch.Generator().manual_seed(seed)
    z = torch.randn(shape, generator=g)
    if kind == "relu":
        z = torch.relu(z)
    elif kind == "ties":
        z = torch.randint(-4, 5, shape, generator=g).float() * 0.25
    elif kind == "zero":
        z = torch.zeros(shape)
    elif kind == "octaves":
        z = z * torch.exp2((torch.rand(shape, generator=g) * 24 - 14).round())
    elif kind == "spike":
        z[:, 0] = 60000.0
    elif kind == "dense":
        z = 1.0 + torch.rand(shape, generator=g) * 2.0 ** -9
    elif kind == "tiny":
        z = z * (1e-41 if dt != "f16" else 1e-6)
    return z.to(TORCH[dt])


def shifted(t, off):
    """the same values on the device, `off` elements past an aligned address"""
    flat = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    v = flat[off:off + t.numel()]
    v.copy_(t.reshape(-1))
    return v


def counts(L):
    return sorted({1, min(3, L), -(-L // 10), max(1, L // 2), L - 1 or 1, L})


CASES = [(L, ("f32", "bf16", "f16")[(i + j) % 3], KINDS[(3 * i + j) % len(KINDS)], (i + j) % 3 if j else 0)
         for i, L in enumerate(LENGTHS) for j in range(4)]


@pytest.mark.parametrize("L,dt,kind,off", CASES)
def test_rows_plain_and_ef(tc, orc, L, dt, kind, off):
    x = make(kind, (N, L), dt, 11)
    xd = shifted(x, off).view(N, L)
    for k in counts(L):
        what = f"{N}x{L} {dt} {kind} +{off} k={k}"
        pl = tc.topk_compress(xd, k, N)
        torch.cuda.synchronize()
        oi, ov = orc.topk_compress(raw(x), dt, N, L, k)
        assert_bits_equal(raw(pl.idx), oi, f"idx {what}")
        assert_bits_equal(raw(pl.val), ov, f"val {what}")
        check_block_table(pl.blk, oi, L, what)
        e = (make("normal", (N, L), "f32", 12) * 0.1).numpy() if kind in ("normal", "relu") else np.zeros((N, L), np.float32)
        ed = shifted(torch.from_numpy(e), off)
        for step in range(3):        # later steps: the residual crowds below the threshold
            pl = tc.ef_step_topk(xd, ed, k, N)
            torch.cuda.synchronize()
            oi, ov, e = orc.ef_topk(raw(x), dt, e, N, L, k)
            assert_bits_equal(raw(pl.idx), oi, f"EF idx {what} step {step}")
            assert_bits_equal(raw(pl.val), ov, f"EF val {what} step {step}")
            assert_bits_equal(raw(ed).reshape(N, L), e, f"EF e {what} step {step}")
    assert tc.device_errors() == 0


@pytest.mark.parametrize("L,dt,kind,off", CASES[1::2])
def test_rows_aqsgd(tc, orc, L, dt, kind, off):
    if kind == "spike" and dt == "f16":
        kind = "octaves"             # (differences of 60000 overflow binary16)
    m0 = make(kind, (2 * N, L), dt, 21)
    ids = torch.tensor([7, 0, 9, 3, 4], dtype=torch.int64)
    acts = [(m0[ids].float() + 0.1 * make("normal", (N, L), "f32", 22 + v)).to(TORCH[dt]) for v in range(2)]
    for k in counts(L):
        md, mo = shifted(m0, off).view(2 * N, L), raw(m0).copy()
        for v in (0, 1, 0, 1, 0, 0):   # repeats: differences in few values, then zero
            pl = tc.aqsgd_step(shifted(acts[v], off).view(N, L), md, ids.cuda(), k)
            torch.cuda.synchronize()
            oi, ov = orc.aqsgd_send(raw(acts[v]), mo, dt, ids.numpy(), k)
            what = f"{L} {dt} {kind} +{off} k={k} visit {v}"
            assert_bits_equal(raw(pl.idx), oi, f"idx {what}")
            assert_bits_equal(raw(pl.val), ov, f"val {what}")
            assert_bits_equal(raw(md), mo, f"m {what}")
    assert tc.device_errors() == 0


def ways(kind, L, dt, seed):
    """rows that take each way through the threshold's search"""
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((N, L), generator=g)
    if kind == "gap":            # a tenth far above the rest: T on either side of it
        z = torch.where(torch.rand((N, L), generator=g) < 0.1, z.sign() * (4 + z.abs()), z * 0.01)
    elif kind == "sparse":       # few non-zero values
        z = torch.where(torch.rand((N, L), generator=g) < 0.03, z, 0.0 * z)
    elif kind == "far":          # the smaller half more than 16 octaves below the larger
        z = torch.where(torch.rand((N, L), generator=g) < 0.5, z, z * 2.0 ** -20)
    elif kind == "alike":        # one magnitude but for a few keys, zeros among them
        z = torch.where(torch.rand((N, L), generator=g) < 0.02, z.round(), 1.5 * z.sign())
    elif kind == "narrow":       # distinct values in one bin of the first window
        z = 1.0 + torch.rand((N, L), generator=g) * 2.0 ** -9
    return z.to(TORCH[dt])


@pytest.mark.parametrize("dt", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("kind", ["gap", "sparse", "far", "alike", "narrow"])
@pytest.mark.parametrize("L", [5, 64, 255, 768, 2048])
def test_rows_ways_through_the_search(tc, orc, L, kind, dt):
    x = ways(kind, L, dt, 41)
    for k in sorted({1, min(2, L), 3, -(-L // 50), -(-L // 10), -(-L // 8), -(-L * 45 // 100), -(-L * 6 // 10), L}):
        e = np.zeros((N, L), np.float32)
        ed = torch.zeros(N * L, device="cuda")
        for step in range(2):
            pl = tc.ef_step_topk(x.cuda(), ed, k, N)
            torch.cuda.synchronize()
            oi, ov, e = orc.ef_topk(raw(x), dt, e, N, L, k)
            what = f"{N}x{L} {dt} {kind} k={k} step {step}"
            assert_bits_equal(raw(pl.idx), oi, f"idx {what}")
            assert_bits_equal(raw(pl.val), ov, f"val {what}")
            assert_bits_equal(raw(ed).reshape(N, L), e, f"e {what}")
        pl = tc.topk_compress(x.cuda(), k, N)
        oi, ov = orc.topk_compress(raw(x), dt, N, L, k)
        assert_bits_equal(raw(pl.idx), oi, f"plain idx {N}x{L} {dt} {kind} k={k}")
        assert_bits_equal(raw(pl.val), ov, f"plain val {N}x{L} {dt} {kind} k={k}")
    assert tc.device_errors() == 0


def test_more_rows_than_resident(tc, orc):
    n, L, k = 9001, 65, 7
    x = make("normal", (n, L), "f32", 31)
    pl = tc.topk_compress(x.cuda(), k, n)
    torch.cuda.synchronize()
    oi, ov = orc.topk_compress(raw(x), "f32", n, L, k)
    assert_bits_equal(raw(pl.idx), oi, "idx")
    assert_bits_equal(raw(pl.val), ov, "val")
    assert tc.device_errors() == 0
