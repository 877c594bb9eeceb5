"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element
by element on the same seeded inputs.

Bar (fp32 path, all three modes): max|err| <= 1e-4 * max|C|, with max|C| the
largest magnitude in the oracle's output for that input.  bf16 mode has its
own absolute bound, set by the features' fourth moments (tests/tolerances.py).
"""
import numpy as np
import pytest

from oracle import corr_oracle as oracle
from paper_2505_16942_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from tolerances import FP32_TOL, bf16_bound


def _binding():
    from paper_2505_16942_amd import binding
    binding.load_library()
    return binding


FORMS = {"one workgroup per level": -4, "two workgroups per item": -2, "decided by item count": 1 << 30, "one workgroup per item": 0}


@pytest.fixture(autouse=True, params=list(FORMS))
def block_kernel_form(request):
    """Every test of this file runs four times: small inputs take the block kernel with one workgroup per
    (item, level) or two per item, decided by the item count; large ones one workgroup per item.  Forcing each form in turn covers the
    edge cases of all of them (ragged maps, missing levels, null queries, D > 256, r < 4) at sizes the oracle
    handles in seconds."""
    b = _binding()
    prev = b.corr_debug_set_level_split(FORMS[request.param])
    yield request.param
    b.corr_debug_set_level_split(prev)


def _run(f1, f2, c, L, r, mode, prec=0, reps=3):
    b = _binding()
    dev = torch.device("cuda:0")
    t1, t2, tc = (torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=L, reps=reps)
    K = 2 * r + 1
    out = torch.full((f1.shape[0], L * K * K, f1.shape[2], f1.shape[3]), float("nan"),
                     dtype=torch.float32, device=dev)
    b.corr_sample(t1, pyr, tc, r=r, out=out, mode=mode, prec=prec)
    torch.cuda.synchronize()
    res = out.cpu().numpy()
    stats = b.corr_last_block_stats(pyr, r) if mode == b.CORR_MODE_BLOCK else None
    pyr.destroy()
    return res, stats


def _check(res, ref, tol_rel, what, bound=None):
    """bound: absolute; default tol_rel * max|C|."""
    assert res.shape == ref.shape
    assert np.all(np.isfinite(res)), what + ": non-finite output (an element was not written?)"
    maxc = float(np.abs(ref).max())
    err = float(np.abs(res.astype(np.float64) - ref).max())
    if bound is None:
        bound = tol_rel * max(maxc, 1e-30)
    print("%s: max|err| = %.3e, max|C| = %.3f, bound = %.3e" % (what, err, maxc, bound), flush=True)
    assert err <= bound, what


SMALL = [
    # B, H, W, D, L, flow_range
    (1, 21, 35, 64, 3, 7.0),      # ragged vs cells, odd level sizes
    (2, 16, 24, 32, 4, 12.0),     # batch, smallest D, level 3 is 2x3
    (1, 8, 8, 256, 4, 3.0),       # level 3 is a single pixel
    (1, 37, 53, 96, 2, 40.0),     # many windows partly or wholly outside
    (1, 19, 27, 224, 4, 5.0),     # seven channel chunks
    (1, 18, 22, 288, 4, 5.0),     # more channels than a wave holds at a time: two groups (8 + 1 chunks)
    (1, 12, 20, 1024, 3, 6.0),    # largest D: four full groups
]


@pytest.mark.parametrize("case", SMALL)
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_small_cases_all_modes(case, mode):
    B, H, W, D, L, fr = case
    print("case", case, "mode", mode, flush=True)
    f1, f2, c = synth.small_case(100 + H, B, H, W, D, flow_range=fr)
    ref = oracle.lookup(f1, f2, c, L=L, r=4)
    res, _ = _run(f1, f2, c, L, 4, mode)
    _check(res, ref, FP32_TOL, "small %s mode %d" % (case, mode))


def test_feature_maps_not_16_byte_aligned():
    """W % 4 == 0 but the caller's maps start 4 bytes past a 16-byte boundary: the build must not
    use aligned vector loads there."""
    b = _binding()
    dev = torch.device("cuda:0")
    B, H, W, D, L = 1, 16, 24, 64, 3
    f1, f2, c = synth.small_case(41, B, H, W, D, flow_range=4.0)
    ref = oracle.lookup(f1, f2, c, L=L, r=4)
    n = f1.size
    big1 = torch.empty(n + 4, dtype=torch.float32, device=dev)
    big2 = torch.empty(n + 4, dtype=torch.float32, device=dev)
    t1 = big1[1:1 + n].view(B, D, H, W)
    t2 = big2[1:1 + n].view(B, D, H, W)
    t1.copy_(torch.from_numpy(f1)); t2.copy_(torch.from_numpy(f2))
    assert t1.data_ptr() % 16 == 4 and t1.is_contiguous()
    pyr = b.corr_pyramid_build(t1, t2, L=L, reps=3)
    tc = torch.from_numpy(c).to(dev)
    for mode in (b.CORR_MODE_BLOCK, b.CORR_MODE_ONDEMAND):
        res = b.corr_sample(t1, pyr, tc, mode=mode)
        _check(res.cpu().numpy(), ref, FP32_TOL, "unaligned maps mode %d" % mode)
    pyr.destroy()


@pytest.mark.parametrize("mode,reps", [(0, 1), (1, 2)])
def test_pyramid_bytes_equal_the_host_estimate(mode, reps):
    """corr_workspace_bytes (host arithmetic) is what a pyramid built for that mode holds."""
    b = _binding()
    dev = torch.device("cuda:0")
    B, H, W, D, L = 2, 37, 53, 96, 3
    f = torch.zeros((B, D, H, W), device=dev)
    pyr = b.corr_pyramid_build(f, f, L=L, reps=reps)
    assert pyr.bytes() == b.corr_workspace_bytes(mode, B, H, W, D, L, 4)
    if mode == 1:      # the dense volume appears with the first full-volume lookup
        c = torch.zeros((B, 2, H, W), device=dev)
        b.corr_sample(f, pyr, c, mode=b.CORR_MODE_FULLVOLUME)
        assert pyr.bytes() == b.corr_workspace_bytes(b.CORR_MODE_FULLVOLUME, B, H, W, D, L, 4)
    pyr.destroy()


def test_bf16_only_representation():
    """CORR_REP_BF16 (hi parts alone, half the bytes) serves bf16 mode with the same bits as the hi
    halves of CORR_REP_SPLIT; a representation that was not rebuilt for the current pair is refused."""
    b = _binding()
    dev = torch.device("cuda:0")
    B, H, W, D, L = 2, 26, 38, 96, 4
    f1, f2, c = synth.small_case(71, B, H, W, D, flow_range=10.0)
    ref = oracle.lookup(f1, f2, c, L=L, r=4)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    p_hi = b.corr_pyramid_build(t1, t2, L=L, reps=b.CORR_REP_BF16)
    got_hi = b.corr_sample(t1, p_hi, tc, prec=b.CORR_PREC_BF16)
    _check(got_hi.cpu().numpy(), ref, None, "bf16 mode on hi-only records", bound=bf16_bound(f1, f2, ref))
    with pytest.raises(b.CorrError) as e:
        b.corr_sample(t1, p_hi, tc)                                   # bf16x3 needs the lo parts
    assert e.value.status == b.CORR_ERR_MISSING_REP
    assert p_hi.bytes() < b.corr_workspace_bytes(b.CORR_MODE_BLOCK, B, H, W, D, L, 4)
    p_sp = b.corr_pyramid_build(t1, t2, L=L, reps=b.CORR_REP_SPLIT)
    got_sp = b.corr_sample(t1, p_sp, tc, prec=b.CORR_PREC_BF16)
    assert torch.equal(got_hi, got_sp)
    p_hi.destroy(); p_sp.destroy()
    # all three representations, then a rebuild of one of them only: the others are stale
    p_all = b.corr_pyramid_build(t1, t2, L=L, reps=7)
    _check(b.corr_sample(t1, p_all, tc).cpu().numpy(), ref, FP32_TOL, "bf16x3 with all representations")
    assert torch.equal(b.corr_sample(t1, p_all, tc, prec=b.CORR_PREC_BF16), got_sp)
    b.corr_pyramid_build(t2, t1, L=L, reps=b.CORR_REP_SPLIT, pyramid=p_all)      # another pair
    with pytest.raises(b.CorrError) as e:
        b.corr_sample(t2, p_all, tc, mode=b.CORR_MODE_ONDEMAND)
    assert e.value.status == b.CORR_ERR_MISSING_REP
    ref2 = oracle.lookup(f2, f1, c, L=L, r=4)
    _check(b.corr_sample(t2, p_all, tc, prec=b.CORR_PREC_BF16).cpu().numpy(), ref2, None,
           "bf16 mode after a split-only rebuild reads the split records", bound=bf16_bound(f2, f1, ref2))
    p_all.destroy()


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_channels_last_output(mode):
    """CORR_OUT_NHWC holds the same values as CORR_OUT_NCHW, taps contiguous per query; every
    element is written (NaN prefill), null queries and untouched levels included."""
    b = _binding()
    dev = torch.device("cuda:0")
    B, H, W, D, L = 2, 21, 35, 64, 3
    f1, f2, c = synth.small_case(61, B, H, W, D, flow_range=30.0)     # many windows partly or wholly outside
    c[0, :, 3, 5] = np.float32(1e9)                                    # a null query
    c[1, 0, 7, 9] = np.float32(np.nan)
    ref_c = np.where(np.isfinite(c) & (np.abs(c) <= 2.0 ** 20), c, np.float32(-1e5))   # same taps: all zero
    ref = oracle.lookup(f1, f2, ref_c, L=L, r=4)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=L, reps=3)
    out = torch.full((B, H, W, L * 81), float("nan"), dtype=torch.float32, device=dev)
    b.corr_sample(t1, pyr, tc, out=out, mode=mode, layout=b.CORR_OUT_NHWC)
    res = out.permute(0, 3, 1, 2).contiguous().cpu().numpy()
    _check(res, ref, FP32_TOL, "channels-last mode %d" % mode)
    nchw = b.corr_sample(t1, pyr, tc, mode=mode)
    assert torch.equal(nchw, out.permute(0, 3, 1, 2)), "the two layouts hold different values"
    pyr.destroy()


def test_lookups_replayed_from_a_hip_graph():
    """corr_sample allocates nothing and clears its own counters with kernels, so a caller may
    capture a sequence of lookups; every replay must equal the eager result."""
    b = _binding()
    dev = torch.device("cuda:0")
    B, H, W, D, L = 1, 30, 44, 64, 4
    f1, f2, c0 = synth.small_case(51, B, H, W, D, flow_range=9.0)
    _, _, c1 = synth.small_case(52, B, H, W, D, flow_range=9.0)
    t1, t2 = torch.from_numpy(f1).to(dev), torch.from_numpy(f2).to(dev)
    tcs = [torch.from_numpy(c0).to(dev), torch.from_numpy(c1).to(dev)]
    outs = [torch.empty((B, L * 81, H, W), device=dev) for _ in range(2)]
    pyr = b.corr_pyramid_build(t1, t2, L=L)

    def job():
        for t in range(2):
            b.corr_sample(t1, pyr, tcs[t], out=outs[t])

    job()
    torch.cuda.synchronize()
    eager = [o.clone() for o in outs]
    _check(eager[0].cpu().numpy(), oracle.lookup(f1, f2, c0, L=L, r=4), FP32_TOL, "eager lookup 0")
    _check(eager[1].cpu().numpy(), oracle.lookup(f1, f2, c1, L=L, r=4), FP32_TOL, "eager lookup 1")
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            job()
    torch.cuda.synchronize()
    for rep in range(4):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(outs[0], eager[0]) and torch.equal(outs[1], eager[1]), "replay %d" % rep
        b.corr_sample(t1, pyr, tcs[1], out=outs[0])          # the program's own eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(outs[0], eager[1])
    pyr.destroy()


@pytest.mark.parametrize("r", [1, 2, 3])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_other_radii(r, mode):
    f1, f2, c = synth.small_case(7, 1, 19, 23, 64, flow_range=5.0)
    ref = oracle.lookup(f1, f2, c, L=3, r=r)
    res, _ = _run(f1, f2, c, 3, r, mode)
    _check(res, ref, FP32_TOL, "r=%d mode %d" % (r, mode))


@pytest.mark.parametrize("r", [1, 2, 3])
def test_other_radii_block_mode_four_levels_far_motion_and_layouts(r):
    """Block mode at r < 4: four levels, windows partly outside, null queries,
    bf16 mode and the channels-last layout."""
    b = _binding()
    dev = torch.device("cuda:0")
    B, H, W, D, L = 2, 33, 41, 96, 4
    f1, f2, c = synth.small_case(80 + r, B, H, W, D, flow_range=25.0)
    c[1, :, 2, 3] = np.float32(-1e6)
    ref = oracle.lookup(f1, f2, c, L=L, r=r)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=L, reps=b.CORR_REP_SPLIT)
    K = 2 * r + 1
    out = torch.full((B, L * K * K, H, W), float("nan"), dtype=torch.float32, device=dev)
    b.corr_sample(t1, pyr, tc, r=r, out=out)
    _check(out.cpu().numpy(), ref, FP32_TOL, "block r=%d" % r)
    stats = b.corr_last_block_stats(pyr, r)
    assert stats["query_levels"] == B * H * W * L and 0 < stats["null_query_levels"] < B * H * W * L
    o16 = b.corr_sample(t1, pyr, tc, r=r, prec=b.CORR_PREC_BF16)
    _check(o16.cpu().numpy(), ref, None, "block bf16 r=%d" % r, bound=bf16_bound(f1, f2, ref))
    ocl = torch.full((B, H, W, L * K * K), float("nan"), dtype=torch.float32, device=dev)
    b.corr_sample(t1, pyr, tc, r=r, out=ocl, layout=b.CORR_OUT_NHWC)
    assert torch.equal(ocl.permute(0, 3, 1, 2), out)
    pyr.destroy()


def test_both_block_kernel_forms_give_the_same_bits():
    b = _binding()
    dev = torch.device("cuda:0")
    f1, f2, c = synth.small_case(55, 2, 40, 56, 96, flow_range=15.0)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=4)
    prev = b.corr_debug_set_level_split(0)
    fused = b.corr_sample(t1, pyr, tc)
    for form, limit in FORMS.items():
        b.corr_debug_set_level_split(limit)
        assert torch.equal(b.corr_sample(t1, pyr, tc), fused), form
    b.corr_debug_set_level_split(prev)
    pyr.destroy()


def test_tiny_config_block_and_bf16():
    cfg = synth.config("tiny")
    f1, f2 = synth.features(cfg)
    c = synth.coords(cfg)
    ref = oracle.lookup(f1, f2, c, L=cfg["L"], r=cfg["r"])
    res, stats = _run(f1, f2, c, cfg["L"], cfg["r"], 0, prec=0, reps=1)
    print("stats", stats, flush=True)
    _check(res, ref, FP32_TOL, "tiny block bf16x3")
    assert stats["query_levels"] == 46 * 62 * 4
    res16, _ = _run(f1, f2, c, cfg["L"], cfg["r"], 0, prec=1, reps=1)
    _check(res16, ref, None, "tiny block bf16", bound=bf16_bound(f1, f2, ref))
    res_od, _ = _run(f1, f2, c, cfg["L"], cfg["r"], 1, reps=2)
    _check(res_od, ref, FP32_TOL, "tiny ondemand")


def test_special_coordinates():
    # integer coords, non-finite, huge, exactly on borders, all outside
    B, H, W, D, L = 1, 24, 40, 64, 4
    f1, f2, c = synth.small_case(5, B, H, W, D, flow_range=6.0, integer_coords=True)
    c[0, 0, 0, 0] = np.nan
    c[0, 1, 0, 1] = np.inf
    c[0, 0, 0, 2] = -np.inf
    c[0, 0, 0, 3] = 3e38
    c[0, 1, 0, 4] = -1e30
    c[0, 0, 1, :] = -1.0
    c[0, 0, 2, :] = W
    c[0, 1, 3, :] = H - 1
    c[0, 0, 4, :] = -13.0          # everything out at level 0, partly in at level 1+
    c[0, 0, 5, :] = W + 200.0
    c[0, 0, 6, :] = 1048576.0      # at the clamp limit
    c[0, 0, 7, :] = 2097152.0      # beyond it
    ref = oracle.lookup(f1, f2, c, L=L, r=4)
    for mode in (0, 1, 2):
        res, _ = _run(f1, f2, c, L, 4, mode)
        _check(res, ref, FP32_TOL, "special coords mode %d" % mode)
        assert np.all(res[0, :, 0, :5] == 0.0)


@pytest.mark.parametrize("fill", ["nan", "far"])
def test_no_query_in_range(fill):
    """Degenerate lookup: every query is out of range at every level, so there is no work item at
    all; every output is written as zero, and the next ordinary lookup on the pyramid is unaffected."""
    b = _binding()
    dev = torch.device("cuda:0")
    B, H, W, D, L = 2, 20, 28, 64, 4
    f1, f2, c = synth.small_case(91, B, H, W, D, flow_range=6.0)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    bad = torch.full_like(tc, float("nan") if fill == "nan" else 5000.0)
    pyr = b.corr_pyramid_build(t1, t2, L=L, reps=3)
    for mode in (0, 1):
        for layout, shape in ((b.CORR_OUT_NCHW, (B, L * 81, H, W)), (b.CORR_OUT_NHWC, (B, H, W, L * 81))):
            out = torch.full(shape, float("nan"), dtype=torch.float32, device=dev)
            b.corr_sample(t1, pyr, bad, out=out, mode=mode, layout=layout)
            assert torch.count_nonzero(out).item() == 0 and not torch.isnan(out).any()
    assert b.corr_last_block_stats(pyr)["items"] == 0
    ref = oracle.lookup(f1, f2, c, L=L, r=4)
    _check(b.corr_sample(t1, pyr, tc).cpu().numpy(), ref, FP32_TOL, "lookup after an empty one")
    pyr.destroy()


def test_determinism_and_pyramid_reuse():
    b = _binding()
    dev = torch.device("cuda:0")
    f1, f2, c = synth.small_case(9, 1, 30, 44, 128, flow_range=9.0)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=4, reps=1)
    o1 = b.corr_sample(t1, pyr, tc).clone()
    o2 = b.corr_sample(t1, pyr, tc).clone()
    # rebuild into the same pyramid from different features, then back
    b.corr_pyramid_build(t2, t1, L=4, reps=1, pyramid=pyr)
    o3 = b.corr_sample(t2, pyr, tc).clone()
    b.corr_pyramid_build(t1, t2, L=4, reps=1, pyramid=pyr)
    o4 = b.corr_sample(t1, pyr, tc).clone()
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(o1, o4)
    assert not torch.equal(o1, o3)
    ref = oracle.lookup(f2, f1, c, L=4, r=4)
    _check(o3.cpu().numpy(), ref, FP32_TOL, "swapped features")
    pyr.destroy()


def test_error_paths():
    b = _binding()
    dev = torch.device("cuda:0")
    f = torch.zeros((1, 48, 16, 16), device=dev)            # D not a multiple of 32
    with pytest.raises(b.CorrError) as e:
        b.corr_pyramid_build(f, f, L=4)
    assert e.value.status == b.CORR_ERR_UNSUPPORTED
    f = torch.zeros((1, 64, 4, 16), device=dev)             # level 3 would be empty
    with pytest.raises(b.CorrError) as e:
        b.corr_pyramid_build(f, f, L=4)
    assert e.value.status == b.CORR_ERR_INVALID_ARG
    f = torch.zeros((1, 64, 16, 16), device=dev)
    pyr = b.corr_pyramid_build(f, f, L=2, reps=1)
    c = torch.zeros((1, 2, 16, 16), device=dev)
    with pytest.raises(b.CorrError) as e:
        b.corr_sample(f, pyr, c, mode=b.CORR_MODE_ONDEMAND)
    assert e.value.status == b.CORR_ERR_MISSING_REP
    with pytest.raises(b.CorrError) as e:
        b.corr_sample(f, pyr, c, r=5)
    assert e.value.status == b.CORR_ERR_UNSUPPORTED
    pyr.destroy()
    # the 8K dense volume is reported, not run
    assert b.corr_full_volume_bytes(1, 540, 960, 4) == 1427549184000
    big = b.corr_full_volume_bytes(1, 540, 960, 4)
    free_b, _ = torch.cuda.mem_get_info()
    assert big > free_b


@pytest.mark.parametrize("B,H,W,D,L,r,nhwc", [(1, 8, 8, 32, 4, 4, 0), (1, 8, 17, 64, 4, 3, 1), (2, 16, 12, 96, 2, 1, 0),
                                              (1, 9, 71, 256, 1, 4, 0), (3, 33, 10, 160, 3, 2, 1), (1, 35, 66, 32, 4, 4, 0)])
def test_full_volume_tiles_and_remainders(B, H, W, D, L, r, nhwc):
    """Full-volume mode where its kernels' tiles end: 64 x 128 of the product, 8 x 32 of the pooling, 16 queries of the
    sampling; levels of one row or column, every radius, both layouts."""
    b = _binding()
    dev = torch.device("cuda:0")
    f1, f2, c = synth.small_case(900 + H * W, B, H, W, D, flow_range=6.0)
    c[0, :, 0, 0] = (-0.5, -0.25)                      # half outside
    c[0, :, 0, 1] = (W - 0.5, H - 0.25)
    c[0, :, 1, 0] = np.float32("nan")
    ref = oracle.lookup(f1, f2, c, L=L, r=r)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    pyr = b.corr_pyramid_build(t1, t2, L=L, reps=b.CORR_REP_F32)
    got = b.corr_sample(t1, pyr, tc, r=r, mode=b.CORR_MODE_FULLVOLUME, layout=b.CORR_OUT_NHWC if nhwc else b.CORR_OUT_NCHW)
    got = got.cpu().numpy()
    _check(np.moveaxis(got, 3, 1) if nhwc else got, ref, 1e-5, "full volume %dx%dx%d D=%d L=%d r=%d" % (B, H, W, D, L, r))
    pyr.destroy()


@pytest.mark.parametrize("D", [32, 96, 128, 160, 192, 224, 288, 352, 512, 544])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_block_channel_loops(D, r):
    """Every length of the block kernel's channel loop, full and not, alone and in groups, at every radius and in both
    precisions."""
    b = _binding()
    f1, f2, c = synth.small_case(60 + D + r, 1, 19, 37, D, flow_range=8.0)
    ref = oracle.lookup(f1, f2, c, L=4, r=r)
    got, _ = _run(f1, f2, c, 4, r, b.CORR_MODE_BLOCK, reps=b.CORR_REP_SPLIT)
    _check(got, ref, FP32_TOL, "block D=%d r=%d" % (D, r))
    got, _ = _run(f1, f2, c, 4, r, b.CORR_MODE_BLOCK, prec=b.CORR_PREC_BF16, reps=b.CORR_REP_BF16)
    _check(got, ref, None, "block bf16 D=%d r=%d" % (D, r), bound=bf16_bound(f1, f2, ref))


@pytest.mark.parametrize("D", [32, 128, 160, 192, 224, 352, 480, 512])
def test_block_channel_loops_channels_last(D):
    """Channels-last kernels of every loop length and group size, at every radius: the same values as NCHW, bit for bit, in both
    precisions; the reduced one also reads the hi parts of a split pyramid."""
    b = _binding()
    dev = torch.device("cuda:0")
    f1, f2, c = synth.small_case(61 + D, 1, 19, 37, D, flow_range=8.0)
    t1, t2, tc = (torch.from_numpy(a).to(dev) for a in (f1, f2, c))
    split = b.corr_pyramid_build(t1, t2, L=4, reps=b.CORR_REP_SPLIT)
    hi = b.corr_pyramid_build(t1, t2, L=4, reps=b.CORR_REP_BF16)
    for r in (1, 2, 3, 4):
        for pyr, prec in ((split, b.CORR_PREC_BF16X3), (split, b.CORR_PREC_BF16), (hi, b.CORR_PREC_BF16)):
            out = torch.full((1, 19, 37, 4 * (2 * r + 1) ** 2), float("nan"), device=dev)
            b.corr_sample(t1, pyr, tc, r=r, prec=prec, layout=b.CORR_OUT_NHWC, out=out)
            want = b.corr_sample(t1, pyr, tc, r=r, prec=prec)
            assert torch.equal(out.permute(0, 3, 1, 2), want), (D, r, prec)
            if pyr is split and prec == b.CORR_PREC_BF16:
                of_split = want
            elif pyr is hi:
                assert torch.equal(of_split, want), (D, r)
    split.destroy()
    hi.destroy()
