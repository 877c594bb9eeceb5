"""Precision of the contractions that run fp32 operands as three bf16 parts each and accumulate six of the nine partial products
(the dense volume, both gradients): the relative error in the 2-norm against fp64.

Normal operands, D = 256: all six products leave 6e-9 out, and without any one of the three smallest (hi * lo, lo * hi, mid * mid) the
result is off by 2.5e-6 or more (the first test, on the CPU).  What fp32 accumulation adds is 2^-24 = 6e-8 a rounding, a few of
them in the 2-norm.  RMS_TOL lies between: a lost product fails, rounding does not."""
import numpy as np
import pytest

from oracle import corr_oracle as oracle
from paper_2505_16942_amd import synth

torch = pytest.importorskip("torch")
RMS_TOL = 6e-7
SIX = [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]


def _rel(got, want):
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


def _parts(v):
    v = torch.from_numpy(v)
    out = []
    for _ in range(3):
        p = v.to(torch.bfloat16).float()
        out.append(p.numpy().astype(np.float64))
        v = v - p
    return out


def test_every_product_counts():
    rng = np.random.default_rng(0)
    a, b = (rng.standard_normal((n, 256)).astype(np.float32) for n in (200, 300))
    pa, pb = _parts(a), _parts(b)
    assert all(np.array_equal(sum(p), v.astype(np.float64)) for p, v in ((pa, a), (pb, b)))      # 24 bits: nothing is left over
    want = a.astype(np.float64) @ b.T.astype(np.float64)
    assert _rel(sum(pa[i] @ pb[j].T for i, j in SIX), want) < RMS_TOL / 50
    for lost in SIX:
        assert _rel(sum(pa[i] @ pb[j].T for i, j in SIX if (i, j) != lost), want) > 4 * RMS_TOL, lost


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 256])
def test_full_volume(D):
    from paper_2505_16942_amd import binding as b
    dev = torch.device("cuda:0")
    f1, f2, c = synth.small_case(7, 1, 28, 40, D, flow_range=6.0)
    want = oracle.lookup(f1, f2, c, L=2, r=4)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=2, reps=b.CORR_REP_F32)
    rel = _rel(b.corr_sample(t1, pyr, tc, r=4, mode=b.CORR_MODE_FULLVOLUME).cpu().numpy().astype(np.float64), want)
    pyr.destroy()
    print("full volume D=%d: %.2e" % (D, rel), flush=True)
    assert rel < RMS_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("D,r", [(64, 4), (128, 3), (256, 4), (256, 1), (512, 4)])
def test_gradient(D, r):
    from paper_2505_16942_amd import binding as b
    dev = torch.device("cuda:0")
    f1, f2, c = synth.small_case(9 + r, 1, 28, 40, D, flow_range=6.0)
    d_out = np.random.default_rng(D).standard_normal((1, 4 * (2 * r + 1) ** 2, 28, 40)).astype(np.float32)
    want1, want2 = oracle.backward(f1, f2, c, d_out, L=4, r=r)
    t1, t2, tc, tg = (torch.from_numpy(a).to(dev) for a in (f1, f2, c, d_out))
    pyr = b.corr_pyramid_build(t1, t2, L=4, reps=b.CORR_REP_F32)
    g1, g2 = b.corr_sample_backward(pyr, tc, tg, r=r)
    rel = [_rel(g.cpu().numpy().astype(np.float64), w) for g, w in ((g1, want1), (g2, want2))]
    pyr.destroy()
    print("gradient D=%d r=%d: d_fmap1 %.2e, d_fmap2 %.2e" % (D, r, *rel), flush=True)
    assert max(rel) < RMS_TOL
