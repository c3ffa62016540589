"""GPU parity of quantization groups spread over several workgroups, bit for
bit against the CPU oracle: groups in up to six rounds of what is resident at
once (three sets of min / max slots take turns, or with more than fifteen
workgroups per group one set is cleared between barriers), ragged and aligned lengths, minima and maxima of
either sign of zero; two calls in a row share one workspace."""
import numpy as np
import pytest
import torch

from gpu_helpers import TORCH, assert_bits_equal, raw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_grp,G,dt,bits", [(600, 16385, "f32", 4), (530, 20000, "bf16", 2), (40, 300001, "f32", 3),
                                             (2, 1000003, "f16", 8), (3, 16384 * 15, "f16", 6),
                                             (64, 768, "bf16", 4), (5, 2047, "f32", 8), (300, 4, "f16", 1)])
def test_exchange_parity(tc, orc, n_grp, G, dt, bits):
    g = torch.Generator().manual_seed(n_grp + G)
    e = torch.zeros(n_grp * G, device="cuda")
    eo = np.zeros((n_grp, G), np.float32)
    for t in range(2):
        x = torch.randn((n_grp, G), generator=g)
        x[0] = -0.0 if t else 0.0            # a constant group: lo = hi = +0
        x = x.to(TORCH[dt])
        codes, meta = tc.ef_step_quant(x.cuda(), e, bits, n_grp)
        torch.cuda.synchronize()
        oc, om, eo = orc.ef_quant(raw(x), dt, eo, n_grp, G, bits)
        what = f"{n_grp}x{G} {dt} b={bits} step {t}"
        assert np.array_equal(codes.cpu().numpy().ravel(), np.asarray(oc).view(np.uint8).ravel()), f"codes {what}"
        assert_bits_equal(raw(meta), np.asarray(om).reshape(n_grp, 2), f"meta {what}")
        assert_bits_equal(raw(e).reshape(n_grp, G), np.asarray(eo).reshape(n_grp, G), f"e {what}")
    assert tc.device_errors() == 0


@pytest.mark.parametrize("n_grp,G", [(1300, 16392), (1300, 16387), (180, 15 * 16384)])
def test_slots_are_written_again(tc, orc, n_grp, G):
    """more than four groups in turn on the same workgroups (two and fifteen
    each; at most 256 and 34 groups are resident), so that each of the three
    sets of slots is written a second time; every group has a minimum and
    maximum of its own, each in another workgroup's part, that a stale slot would
    replace.  The values of one block are shared, so that the oracle can be asked
    per group: lo and hi come from the first and last element."""
    b = 4
    g = torch.Generator().manual_seed(23)
    body = torch.randn((1, G), generator=g).clamp(-3, 3)
    lo = -4.0 - (torch.arange(n_grp) * 7 % n_grp).float() / n_grp * 60     # neighbours in no order
    hi = 4.0 + (torch.arange(n_grp) * 11 % n_grp).float() / n_grp * 60
    x = body.expand(n_grp, G).contiguous()
    x[:, 0], x[:, G - 1] = lo, hi
    codes, meta = tc.quant_pack(x.cuda(), b, n_grp)
    torch.cuda.synchronize()
    assert_bits_equal(raw(meta)[:, 0], lo.numpy(), "lo")
    some = sorted(set(range(0, n_grp, max(1, n_grp // 40))) | {n_grp - 1})   # codes of some groups, whole
    oc, om = orc.quant_pack(raw(x[some]), "f32", len(some), G, b)
    got = codes.cpu().numpy()[some]
    assert np.array_equal(got.ravel(), np.asarray(oc).view(np.uint8).ravel()), "codes"
    assert_bits_equal(raw(meta)[some], np.asarray(om).reshape(-1, 2), "meta")
    scale = ((hi - lo) / np.float32(2 ** b - 1)).numpy()                     # binary32, as the codec defines it
    assert_bits_equal(raw(meta)[:, 1], scale, "scale")
    assert tc.device_errors() == 0


@pytest.mark.parametrize("G", [1, 2, 3, 5, 6, 7, 2045, 2047, 2050, 16383, 16387, 32771])
@pytest.mark.parametrize("dt,bits,off", [("f32", 4, 0), ("bf16", 2, 1), ("f16", 32, 3)])
def test_unaligned_groups(tc, orc, G, dt, bits, off):
    """groups that end inside a piece of four elements, at addresses aligned to
    their elements only"""
    n = 3
    g = torch.Generator().manual_seed(G)
    x = torch.randn((n, G), generator=g).to(TORCH[dt])
    e0 = torch.randn((n, G), generator=g) * 0.1
    xd = torch.empty(n * G + 8, dtype=TORCH[dt], device="cuda")[off:off + n * G].view(n, G)
    ed = torch.empty(n * G + 8, device="cuda")[off:off + n * G]
    xd.copy_(x)
    ed.copy_(e0.reshape(-1))
    codes, meta = tc.ef_step_quant(xd, ed, bits, n)
    torch.cuda.synchronize()
    oc, om, eo = orc.ef_quant(raw(x), dt, e0.numpy(), n, G, bits)
    assert np.array_equal(codes.cpu().numpy().ravel(), np.asarray(oc).view(np.uint8).ravel()), "codes"
    assert_bits_equal(raw(meta), np.asarray(om).reshape(n, 2), "meta")
    assert_bits_equal(raw(ed).reshape(n, G), np.asarray(eo).reshape(n, G), "e")
    assert tc.device_errors() == 0
