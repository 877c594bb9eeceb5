"""Infinities, NaNs and values beyond bf16's range in the kernels that split fp32 operands into three bf16 parts (the dense
volume and the gradient): what the fp64 oracle leaves finite stays finite and right, the rest is not."""
import numpy as np
import pytest

from oracle import corr_oracle as oracle
from paper_2505_16942_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

INF, NAN, HUGE = np.float32("inf"), np.float32("nan"), np.float32(3.4e38)     # the largest bf16 is 3.39e38


def _binding():
    from paper_2505_16942_amd import binding
    binding.load_library()
    return binding


def _check(got, want, tol, what, kinds=True, axis=1):
    """The same elements finite (with `kinds` every infinity of the oracle's the same one: where it adds infinities of both
    signs tap by tap and has NaN, weights that were summed first may leave one), finite ones within tol of the largest of
    their slice along `axis` (the slices' magnitudes differ by 38 orders)."""
    got = got.cpu().numpy().astype(np.float64)
    ok = np.isfinite(want)
    print(what, "not finite:", int((~ok).sum()), "of", ok.size, flush=True)
    assert 0 < (~ok).sum() < ok.size // 2, what
    assert np.array_equal(np.isfinite(got), ok), what
    if kinds:
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)]), what
    rest = tuple(i for i in range(want.ndim) if i != axis)
    most = np.where(ok, np.abs(want), 0.0).max(axis=rest, keepdims=True)
    err = np.where(ok, np.abs(np.where(ok, got, 0.0) - np.where(ok, want, 0.0)), 0.0)
    assert np.all(err <= tol * most), what


def test_full_volume():
    b = _binding()
    dev = torch.device("cuda:0")
    H, W, D = 20, 36, 96
    f1, f2, c = synth.small_case(41, 1, H, W, D, flow_range=4.0)
    f1[0, 3, 4, 5], f1[0, 60, 11, 30], f1[0, 70, 17, 2] = INF, NAN, -INF
    f2[0, 8, 9, 9], f2[0, 50, 2, 33] = -INF, NAN
    f1[0, 21, 15, 16] = HUGE                             # its hi part is infinity, its products are finite
    f2[0, 21] *= np.float32(1e-6)
    ref = oracle.lookup(f1, f2, c, L=4, r=4)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=4, reps=b.CORR_REP_F32)
    got = b.corr_sample(t1, pyr, tc, r=4, mode=b.CORR_MODE_FULLVOLUME)
    flat = lambda a: a.reshape(1, 324, H * W)            # a slice is a query
    _check(flat(got), flat(ref), 1e-5, "full volume", kinds=False, axis=2)
    # level 0: the deeper levels pool the volume, where infinities of both signs meet, and not the features
    _check(flat(got)[:, :81], flat(ref)[:, :81], 1e-5, "full volume, level 0", axis=2)
    pyr.destroy()
