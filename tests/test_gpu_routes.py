"""The sizes at which the library changes kernels, against the oracle: the
marching count pass building halo bits of its own (or not), the rays per
workgroup of cone steps, the rays per wave of the uniform fill and of fused
inference."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_fused import _assert_same, _cuda, _nacc, _three_step
from test_gpu_march import BOX, compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rays", [16415, 16416])
def test_uniform_own_halo(n_rays):
    """Halo bits of a 32^3 grid (128 words) are built from 16,416 rays on."""
    mask = synth.random_mask(32 ** 3, 0.02, 11)
    o, d = synth.rays_toward_origin(n_rays, 61)
    compare(o, d, mask, 32, BOX, 0.0, 1e10, 0.0137)


@pytest.mark.parametrize("n_grids,n_rays", [(64, 1), (65, 64), (66, 64), (66, 200)])
def test_cone_many_grids(n_grids, n_rays):
    """64^3 grids have 1,024 halo words each; a call of n rays builds up to
    65,536 + 16 n words (66 grids: not for 64 rays, but for 200)."""
    mask = synth.random_mask(n_grids * 64 ** 3, 0.01, 12)
    o, d = synth.rays_toward_origin(n_rays, 62)
    gid = np.random.default_rng(5).integers(0, n_grids, n_rays).astype(np.int32)
    compare(o, d, mask, 64, BOX, 0.0, 1e10, 0.006, cone=1 / 256, n_grids=n_grids, grid_id=gid)


@pytest.mark.parametrize("n_rays", [104857, 104858])
def test_contraction_many_chunks(n_rays):
    """2,512 candidates, 40 chunks a ray, 4.2 million chunks."""
    mask = synth.random_mask(64 ** 3, 0.01, 13)
    o, d = synth.rays_unbounded(n_rays, 63)
    compare(o, d, mask, 64, np.array(synth.CONTRACT_BOX, np.float32), 0.2, 1e4, synth.STEP_1024,
            cone=1 / 256, lookup=2, max_per_ray=64)


@pytest.mark.parametrize("n_rays", [1, 5, 8191, 8192, 16384, 32768, 65536, 131072])
def test_cone_rays_per_workgroup(n_rays):
    """4 to 64 rays a workgroup; rays that start at the near plane (inside
    the box), outside it, and both in a wave."""
    mask = synth.random_mask(16 ** 3, 0.05, 21)
    o, d = synth.rays_toward_origin(n_rays, 65)
    for step in (1, 2):
        o[::step] *= 0.1
        compare(o, d, mask, 16, BOX, 0.05, 1e10, 0.02, cone=1 / 64, dt_max=0.2)
        o[::step] *= 10.0


@pytest.mark.parametrize("base,levels,dt,cone", [
    (1.0, 5, 0.02, 1 / 256),       # a level or two per segment of 8 steps
    (0.0625, 9, 0.2, 1 / 16),      # many levels per segment
    (2.0 ** -62, 3, 2.0 ** -66, 0.01),  # scales near the end of the exponent range
    (2.0 ** -40, 3, 2.0 ** -44, 0.01),
])
def test_cone_cascade_levels(base, levels, dt, cone):
    res = 16
    mask = synth.random_mask(levels * res ** 3, 0.2, 22)
    o, d = synth.rays_toward_origin(700, 66)
    o = (o * np.float32(0.3 * base)).astype(np.float32)
    box = np.array([-base] * 3 + [base] * 3, np.float32)
    compare(o, d, mask, res, box, 0.01 * base, base * 2.0 ** levels, dt, cone=cone, n_grids=levels, lookup=1)


@pytest.mark.parametrize("res,p_occ", [(4, 0.5), (12, 0.5), (12, 0.95), (20, 1.0), (32, 0.5), (64, 0.97), (64, 0.002)])
@pytest.mark.parametrize("near,far,dt,cone", [
    (0.2, 1e4, 0.01, 1 / 256),
    (0.0, 1e10, 0.005, 1 / 128),   # steps that may stall by their size alone
    (0.2, 3.0, 0.02, 1 / 256),     # rays ending inside a segment
    (0.2, 40.0, 0.0005, 1 / 4096),  # past the stored chunks
    (40000.0, 1e6, 0.001, 1e-9),   # stalled from the start
])
def test_cone_contraction_cells(res, p_occ, near, far, dt, cone):
    """Segments decided by the cells within their bounds, and not: sparse,
    ragged and full grids, rows of cells that cross words."""
    mask = synth.random_mask(res ** 3, p_occ, 23)
    o, d = synth.rays_unbounded(150, 67)
    compare(o, d, mask, res, np.array(synth.CONTRACT_BOX, np.float32), near, far, dt, cone=cone, lookup=2)


@pytest.mark.parametrize("n_rays,dt", [(1, 0.0137), (63, 0.0137), (2049, 0.0137), (4095, 0.0025),
                                       (4096, 0.0025), (8192, 0.0025), (16384, 0.0137), (16385, 0.00125)])
@pytest.mark.parametrize("cap", [0, 70])
def test_uniform_fill_rays_per_wave(n_rays, dt, cap):
    """1, 2, 4 and 8 rays per wave of the fill; 6, 33 and 64 stored chunks
    (the last one with rays going on past them); full and ragged masks; rays
    cut by the cap."""
    for p_occ in (0.05, 1.0):
        mask = synth.random_mask(16 ** 3, p_occ, 14)
        o, d = synth.rays_toward_origin(n_rays, 64)
        compare(o, d, mask, 16, BOX, 0.0, 1e10, dt, max_per_ray=cap)


@pytest.mark.parametrize("n_rays", [3, 39999, 40000, 159999, 160000, 399999, 400000])
def test_fused_rays_per_workgroup(n_rays):
    """4, 8, 16 and 32 rays per workgroup of the fused inference kernel."""
    nacc = _nacc()
    scene = synth.blob_scene(6, 71)
    grid = nacc.OccupancyGrid(synth.BOX_1_5, 32)
    grid.set_occupancy(_cuda(synth.initial_occupancy(scene, 32, synth.BOX_1_5)), 0.01)
    field = nacc.BlobField(scene)
    o, d = (_cuda(a) for a in synth.rays_toward_origin(n_rays, 72, jitter_std=0.5))
    ref = _three_step(nacc, field, grid, o, d, 0.0, 1e10, 0.02, 1e-4)
    _assert_same(nacc.render_fused(field, o, d, grid, 0.0, 1e10, 0.02, 1e-4, return_kept=True), ref)


@pytest.mark.parametrize("n_blobs,contract,odd_peak", [(1, False, None), (64, False, None), (65, False, None),
                                                       (150, True, None), (70, False, float("inf")),
                                                       (70, False, -3.0)])
def test_fused_leaves_out_far_blobs(n_blobs, contract, odd_peak):
    """Narrow blobs, most of them too far from a chunk of samples to
    contribute; more blobs than lanes; a peak whose product is not zero where
    its exponential is; a scene in contracted coordinates."""
    nacc = _nacc()
    scene = synth.blob_scene(n_blobs, 73, radius_range=(0.02, 0.3))
    scene.contract = contract
    grid = nacc.OccupancyGrid(synth.BOX_1_5, 64)
    grid.set_occupancy(_cuda(synth.initial_occupancy(scene, 64, synth.BOX_1_5)), 0.01)
    if odd_peak is not None:
        scene.peaks[n_blobs // 2] = odd_peak
    field = nacc.BlobField(scene)
    o, d = synth.rays_toward_origin(2000, 74, jitter_std=0.3)
    o, d = _cuda(o), _cuda(d * np.float32(1.7))
    ref = _three_step(nacc, field, grid, o, d, 0.0, 1e10, 0.004, 1e-4)
    assert int((ref["packed"][:, 1] > 0).sum()) > 100
    _assert_same(nacc.render_fused(field, o, d, grid, 0.0, 1e10, 0.004, 1e-4, return_kept=True), ref)


@pytest.mark.parametrize("n_rays", [1, 65, 255, 256, 257, 4097, 65537, 131072, 524288, 524289])
@pytest.mark.parametrize("waves", [1, 4, 16])
def test_starts_and_totals(n_rays, waves):
    """Starts and total of the marched layout at the edges of the parts their
    sums come in (1 to 16 workgroups per 64 rays; one launch up to 8,192
    parts, then the scan): the exclusive sums of the counts, which do not
    depend on the launch parameters."""
    nacc = _nacc()
    lib = nacc._lib
    scene = synth.blob_scene(6, 75)
    grid = nacc.OccupancyGrid(synth.BOX_1_5, 32)
    grid.set_occupancy(_cuda(synth.initial_occupancy(scene, 32, synth.BOX_1_5)), 0.01)
    o, d = (_cuda(a) for a in synth.rays_toward_origin(n_rays, 76, jitter_std=0.5))
    before = lib.get_tuning()
    try:
        lib.set_tuning(march_waves_per_group=waves)
        packed, ri, ts, _ = nacc.ray_marching(o, d, grid, 0.0, 1e10, 0.02)
    finally:
        lib.set_tuning(**before)
    count = packed[:, 1].long()
    assert int(count.sum()) == ri.numel() == ts.numel()
    assert torch.equal(packed[:, 0].long(), count.cumsum(0) - count)
    assert torch.equal(ri.long(), torch.repeat_interleave(torch.arange(n_rays, device="cuda"), count))


@pytest.mark.parametrize("n_rays", [1, 5, 16383, 16384, 32768, 131072, 131073, 262144, 262145, 600000])
def test_prune_rays_per_wave(n_rays):
    """1, 2, 4, 8 and 16 rays per wave of the pruning kernels: rays of no, one
    and many chunks, some cut, most samples of some below the threshold;
    against the flags' definition in plain torch on the kept samples and the
    rendering kernel's cut."""
    nacc = _nacc()
    rng = np.random.default_rng(77)
    count = rng.choice([0, 1, 63, 64, 65, 130, 200], n_rays, p=[0.4, 0.25, 0.1, 0.1, 0.05, 0.05, 0.05])
    start = np.concatenate([[0], np.cumsum(count)[:-1]])
    packed = _cuda(np.stack([start, count], 1).astype(np.int32))
    e = int(count.sum())
    g = torch.Generator(device="cuda").manual_seed(78)
    ts = torch.rand(e, generator=g, device="cuda")
    te = ts + 0.01
    sig = torch.rand(e, generator=g, device="cuda") ** 4 * 200.0
    out, ri, ts_o, te_o, sg_o = nacc.prune_samples(packed, ts, te, sig, 1e-2, 0.05)
    kept = torch.empty(n_rays, dtype=torch.int32, device="cuda")
    rgb = torch.zeros((e, 3), device="cuda")
    c3, a1, d1 = (torch.empty((n_rays, k), device="cuda") for k in (3, 1, 1))
    nacc._lib.render_fwd(packed, ts, te, sig, rgb, 1e-2, c3, a1, d1, None, kept)
    ray = torch.repeat_interleave(torch.arange(n_rays, device="cuda"), _cuda(count))
    alpha = -torch.expm1(-sig.double() * (te - ts).double())
    sure = (alpha - 0.05).abs() > 1e-6  # away from the threshold
    before_cut = torch.arange(e, device="cuda") - _cuda(start)[ray] < kept.long()[ray]
    want = before_cut & (alpha >= 0.05)
    if bool(sure.all()):
        assert torch.equal(ri.long(), ray[want])
        for got, src in ((ts_o, ts), (te_o, te), (sg_o, sig)):
            assert torch.equal(got, src[want])
    n_out = out[:, 1].long()
    assert torch.equal(out[:, 0].long(), n_out.cumsum(0) - n_out) and int(n_out.sum()) == ri.numel()
    low = torch.zeros(n_rays, dtype=torch.long, device="cuda").index_add_(0, ray, (want & sure).long())
    high = torch.zeros(n_rays, dtype=torch.long, device="cuda").index_add_(0, ray, (want | (before_cut & ~sure)).long())
    assert bool(((n_out >= low) & (n_out <= high)).all())


@pytest.mark.parametrize("res,p_occ", [(4, 0.1), (12, 0.02), (20, 0.002), (100, 1e-5), (128, 2e-6), (160, 1e-5),
                                       (512, 1e-6), (516, 1e-7)])
def test_skip_buffer_of_any_resolution(res, p_occ):
    """Distances and halo bits of grids whose rows fill words, end inside
    them, or hold several (and of the first grid that takes the passes per
    axis): against scipy."""
    from scipy.ndimage import distance_transform_cdt, maximum_filter
    nacc = _nacc()
    n = 2
    mask = synth.random_mask(n * res ** 3, p_occ, 80 + res)
    mask[-1] = 1
    grid = nacc.OccupancyGrid(BOX, res, n_grids=n)
    grid.set_occupancy(_cuda(mask.astype(np.float32)), 0.5)
    torch.cuda.synchronize()
    buf = grid.skip.cpu().numpy()
    c, h = res // 4, res // 2
    words = -(-h ** 3 // 64) * 2
    halo = np.unpackbits(buf[-(-2 * c ** 3 * n // 256) * 256:].reshape(n, 4 * words), axis=1, bitorder="little")
    for i in range(n):
        m = mask[i * res ** 3:(i + 1) * res ** 3].reshape(res, res, res).astype(bool)
        coarse = m.reshape(c, 4, c, 4, c, 4).any(axis=(1, 3, 5))
        far = distance_transform_cdt(~coarse, metric="chessboard") if coarse.any() else np.full(coarse.shape, 15)
        assert np.array_equal(buf[i * c ** 3:(i + 1) * c ** 3], np.minimum(far, 15).ravel()), f"distances {i}"
        near = maximum_filter(m, size=5, mode="constant").reshape(h, 2, h, 2, h, 2).any(axis=(1, 3, 5))
        assert np.array_equal(halo[i, :h ** 3], near.ravel()) and not halo[i, h ** 3:].any(), f"halo {i}"


@pytest.mark.parametrize("n_cells", [32, 992, 1024, 4096, 4128, 100000])
def test_pack_runs(n_cells):
    """Cells short of, at and past the 1,024 of a wave and the 4,096 of a
    workgroup; values at the threshold and NaN are not above it."""
    lib = _nacc()._lib
    rng = np.random.default_rng(n_cells)
    occ = rng.choice(np.array([0.0, 0.01, 0.02, -1.0, np.nan, np.inf], np.float32), n_cells)
    bits = torch.full((n_cells // 32 + 1,), -1, dtype=torch.int32, device="cuda")
    lib.grid_pack(_cuda(occ), 0.01, bits[:-1])
    got = np.unpackbits(bits.cpu().numpy().view(np.uint8), bitorder="little")
    assert np.array_equal(got[:n_cells], occ > np.float32(0.01)) and got[n_cells:].all()


@pytest.mark.parametrize("ch", list(range(1, 18)) + [20, 23, 24, 28, 31, 33, 47, 49])
@pytest.mark.parametrize("shift", [0, 1])
def test_attribute_rows_of_any_width(ch, shift):
    """Every channel of a row of any width, at 16-byte aligned addresses or
    not, is rendered and gets its gradient as the only channel of a call of
    its own, bit for bit; nothing beside the rows is written."""
    nacc = _nacc()
    packed, ts, te, sg, _ = synth.ragged_render_inputs(300, 81, mean_count=90.0)
    packed, ts, te, sg = (_cuda(a) for a in (packed, ts, te, sg))
    e, n = ts.numel(), packed.shape[0]
    g = torch.Generator(device="cuda").manual_seed(82)
    attrs = torch.randn(e * ch + shift, generator=g, device="cuda")[shift:].view(e, ch)
    g_out = torch.randn((n, ch), generator=g, device="cuda")
    bg = torch.rand(ch, generator=g, device="cuda")
    lib = nacc._lib

    def render(a, go, b, pad):
        k = a.shape[1]
        out, op, dep = (torch.empty((n, j), device="cuda") for j in (k, 1, 1))
        lib.render_attrs_fwd(packed, ts, te, sg, a, 1e-2, 0.05, b, out, op, dep)
        ga = torch.full((e * k + pad + 4,), 7.0, device="cuda")
        gs = torch.empty_like(ts)
        lib.render_attrs_bwd(packed, ts, te, sg, a, 1e-2, 0.05, b, go, None, None, gs, ga[pad:pad + e * k].view(e, k))
        assert bool((ga[:pad] == 7.0).all()) and bool((ga[pad + e * k:] == 7.0).all())
        return out, ga[pad:pad + e * k].view(e, k)

    out, ga = render(attrs, g_out, bg, shift)
    for k in range(ch):
        one = render(attrs[:, k:k + 1].contiguous(), g_out[:, k:k + 1].contiguous(), bg[k:k + 1].contiguous(), 0)
        assert torch.equal(out[:, k:k + 1].contiguous().view(torch.int32), one[0].view(torch.int32)), f"out {k}"
        assert torch.equal(ga[:, k:k + 1].contiguous().view(torch.int32),
                           one[1].contiguous().view(torch.int32)), f"g_attrs {k}"


@pytest.mark.parametrize("read", [(0,), (1,), (2,), (0, 2), (1, 2)])
@pytest.mark.parametrize("attrs", [False, True])
def test_gradients_of_unread_outputs(read, attrs):
    """A loss that leaves outputs out gives the gradients of one that reads
    them times zero, exactly: zero gradients add zeros."""
    import paper_2210_04847_amd as nacc
    gen = torch.Generator().manual_seed(5)
    counts = torch.tensor([0, 3, 64, 65, 200, 1])
    starts = torch.cumsum(counts, 0) - counts
    packed = torch.stack([starts, counts], 1).to(torch.int32).cuda()
    e = int(counts.sum())
    ts = torch.rand(e, generator=gen).cuda()
    sig0, at0 = torch.rand(e, generator=gen).cuda(), torch.rand(e, 3, generator=gen).cuda()
    grads = []
    for zeros in (False, True):
        sig, at = sig0.clone().requires_grad_(), at0.clone().requires_grad_()
        outs = (nacc.render_attrs if attrs else nacc.rendering)(packed, ts, ts + 0.01, sig, at)
        loss = sum((outs[i] ** 2).sum() for i in read)
        if zeros:
            loss = loss + sum((outs[i] * 0.0).sum() for i in range(3) if i not in read)
        loss.backward()
        grads.append((sig.grad, at.grad))
    for a, b in zip(*grads):
        assert torch.equal(a, b)


def test_cone_starts_past_one_launch():
    """More than 8,192 parts of 32 rays: scanned, a wave placing two."""
    mask = synth.random_mask(8 ** 3, 0.05, 24)
    o, d = synth.rays_unbounded(262144 + 33, 68)
    compare(o, d, mask, 8, np.array(synth.CONTRACT_BOX, np.float32), 0.2, 20.0, 0.012, cone=1e-6, lookup=2)


@pytest.mark.parametrize("n_rays", [1, 15, 2048, 4097, 8192, 32768])
@pytest.mark.parametrize("cap", [0, 9, 100])
def test_cone_fill_rays_per_wave(n_rays, cap):
    """1 to 16 rays a wave, listed in whole blocks (rays from the near plane)
    or by segments; rays cut by the cap; more than 64 tasks a wave."""
    for p_occ in (0.05, 1.0):
        mask = synth.random_mask(16 ** 3, p_occ, 25)
        o, d = synth.rays_toward_origin(n_rays, 69)
        for scale in (0.1, 1.0):
            compare((o * np.float32(scale)).astype(np.float32), d, mask, 16, BOX, 0.05, 1e10, 0.01, cone=1 / 512,
                    max_per_ray=cap)


@pytest.mark.parametrize("res,dt,p_occ,cap", [
    (16, 0.0005, 0.02, 0), (16, 0.0005, 0.97, 70),  # more candidates than stored chunks: windows
    (8, 0.02, 1.0, 0),                              # every segment inside occupied cells
    (16, 0.03, 0.99, 0), (32, 0.0137, 0.98, 0), (64, 0.004, 0.995, 0),  # segments of 8 to 32
    (64, 0.05, 0.5, 0),                             # rays too fast for segments
    (64, 0.0137, 0.03, 5),
])
@pytest.mark.parametrize("n_rays,n_grids", [(60, 1), (16900, 1), (18500, 1), (17401, 2)])
def test_box_count(res, dt, p_occ, cap, n_rays, n_grids):
    """Uniform steps by halo bits, and (from 16,384 rays and twice the halo
    words on) by hole bits: grids of solid parts with gaps."""
    if n_rays > 60 and res == 16 and dt < 0.001:
        n_rays = 16500
    mask = synth.random_mask(n_grids * res ** 3, p_occ, 26).reshape(n_grids, res, res, res)
    if p_occ > 0.9:
        mask[:, res // 2:] = 1
    o, d = synth.rays_toward_origin(n_rays, 70)
    gid = np.random.default_rng(6).integers(0, n_grids, n_rays).astype(np.int32)
    kw = dict(n_grids=n_grids, grid_id=gid) if n_grids > 1 else {}
    compare(o, d, mask.reshape(-1), res, BOX, 0.0, 1e10, dt, max_per_ray=cap, **kw)


@pytest.mark.parametrize("n_rays", [65535, 65536])
def test_contraction_rays_per_workgroup(n_rays):
    """40 chunks a ray: 16 and 32 rays a workgroup of the cone count."""
    mask = synth.random_mask(64 ** 3, 0.01, 27)
    o, d = synth.rays_unbounded(n_rays, 71)
    compare(o, d, mask, 64, np.array(synth.CONTRACT_BOX, np.float32), 0.2, 1e4, synth.STEP_1024,
            cone=1 / 256, lookup=2, max_per_ray=64)


@pytest.mark.parametrize("n_rays", [1, 900, 8200, 16500])
@pytest.mark.parametrize("res,dt,p_occ", [(64, 0.0137, 0.02), (32, 0.004, 0.3), (16, 0.0009, 0.05), (8, 0.0011, 1.0),
                                          (64, 0.05, 0.5)])
@pytest.mark.parametrize("cap", [1, 7, 130, 4000])
def test_box_count_in_turns(n_rays, res, dt, p_occ, cap):
    """Rays capped after the first candidates, in a later turn, in the second
    window of stored chunks, and never; 1 to 16 rays a wave."""
    if dt < 0.003:
        n_rays = min(n_rays, 900)
    mask = synth.random_mask(res ** 3, p_occ, 28).reshape(res, res, res)
    mask[:res // 4, :, ::3] = 0
    o, d = synth.rays_toward_origin(n_rays, 72)
    compare(o, d, mask.reshape(-1), res, BOX, 0.0, 1e10, dt, max_per_ray=cap)


@pytest.mark.parametrize("res,dt,p_occ,cap", [
    (16, 0.0009, 0.05, 0), (16, 0.0009, 0.97, 70),  # windows of stored chunks
    (8, 0.02, 1.0, 0), (16, 0.03, 0.3, 0), (32, 0.0137, 0.5, 9), (64, 0.004, 0.1, 0),  # segments of 8 to 32
    (64, 0.05, 0.5, 0),                             # rays too fast for segments
])
@pytest.mark.parametrize("n_rays,n_grids", [(1, 2), (70, 3), (4100, 7), (19000, 3)])
def test_box_count_of_several_grids(res, dt, p_occ, cap, n_rays, n_grids):
    """Lookups of eight runs a load: rays of different grids in a wave, some
    with no grid; full and partly filled rounds; 1 to 4 rays a wave."""
    if dt < 0.001:
        n_rays = min(n_rays, 300)
    mask = synth.random_mask(n_grids * res ** 3, p_occ, 29)
    o, d = synth.rays_toward_origin(n_rays, 73)
    gid = np.random.default_rng(7).integers(-1, n_grids + 1, n_rays).astype(np.int32)
    gid[0] = n_grids - 1
    compare(o, d, mask, res, BOX, 0.0, 1e10, dt, max_per_ray=cap, n_grids=n_grids, grid_id=gid)


def _check_skip(nacc, res, n, mask):
    """Distances and halo bits of n grids, against scipy (as above), for as
    many different ones as `mask` [m, res, res, res] holds, repeated."""
    from scipy.ndimage import distance_transform_cdt, maximum_filter
    m = mask.shape[0]
    lib = nacc._lib
    desc = lib.grid_desc(BOX[:3], BOX[3:], res, n)
    words = np.packbits(mask.reshape(m, -1), axis=1, bitorder="little").view(np.int32)
    bits = _cuda(words).repeat(-(-n // m), 1)[:n].reshape(-1)
    buf = torch.full((lib.grid_skip_bytes(desc),), 77, dtype=torch.uint8, device="cuda")
    lib.grid_build_skip(bits, desc, buf)
    c, h = res // 4, res // 2
    hw = -(-h ** 3 // 64) * 8  # bytes of a grid's halo bits
    field = buf[:n * c ** 3].view(n, -1)
    halo = buf[-(-2 * c ** 3 * n // 256) * 256:].view(n, hw)
    want_f = np.empty((m, c ** 3), np.uint8)
    want_h = np.zeros((m, hw), np.uint8)
    for i in range(m):
        coarse = mask[i].reshape(c, 4, c, 4, c, 4).any(axis=(1, 3, 5))
        far = distance_transform_cdt(~coarse, metric="chessboard") if coarse.any() else np.full(coarse.shape, 15)
        want_f[i] = np.minimum(far, 15).ravel()
        near = maximum_filter(mask[i].astype(bool), size=5, mode="constant").reshape(h, 2, h, 2, h, 2)
        b = np.packbits(near.any(axis=(1, 3, 5)).ravel(), bitorder="little")
        want_h[i, :b.size] = b
    for got, want, name in ((field, want_f, "distances"), (halo, want_h, "halo bits")):
        w = _cuda(want).repeat(-(-n // m), 1)[:n]
        assert torch.equal(got, w), f"{name} of {n} grids of {res}^3"


@pytest.mark.parametrize("res,n", [(4, 1), (4, 2048), (4, 2049), (4, 300001), (8, 3), (8, 1024), (8, 1025), (16, 512),
                                   (16, 513), (32, 256), (32, 257), (44, 186), (44, 187), (48, 187)])
def test_skip_buffer_of_many_small_grids(res, n):
    """Either side of the number of planes up to which small grids are built
    plane by plane; grids of one word a plane and less."""
    mask = np.stack([synth.random_mask(res ** 3, p, 90 + i).reshape(res, res, res)
                     for i, p in enumerate((0.0, 1.0, 0.5, 4 / res ** 3, 1 / res ** 3, 1 / res ** 3, 0.02))])
    _check_skip(_nacc(), res, n, mask)


def test_skip_buffer_of_very_many_grids():
    """4.2 million grids of 4^3 cells: as many planes, past 2^32 threads with
    1,024 a plane."""
    mask = np.stack([synth.random_mask(64, p, 97 + i).reshape(4, 4, 4) for i, p in enumerate((0.02, 0.0, 0.3))])
    _check_skip(_nacc(), 4, (1 << 22) + 5, mask)


@pytest.mark.parametrize("n_blobs", [1, 15, 16])
@pytest.mark.parametrize("n_sets", [1, 3])
def test_fused_few_blobs(n_blobs, n_sets):
    """Either side of the number of blobs from which far ones are left out,
    with one set of centres and with several."""
    nacc = _nacc()
    scene = synth.moving_blob_scene(n_blobs, n_sets, 75) if n_sets > 1 else synth.blob_scene(n_blobs, 75)
    grid = nacc.OccupancyGrid(synth.BOX_1_5, 32)
    grid.set_occupancy(torch.ones(32 ** 3), 0.5)
    field = nacc.BlobField(scene)
    o, d = (_cuda(a) for a in synth.rays_toward_origin(1500, 76, jitter_std=0.4))
    ray_set = torch.arange(1500, dtype=torch.int32, device="cuda") % n_sets if n_sets > 1 else None
    packed, ri, ts, te = nacc.ray_marching(o, d, grid, 0.0, 1e10, 0.01)
    sig, rgb = field.samples(o, d, ri, ts, te, ray_set)
    color, opacity, depth = nacc.rendering(packed, ts, te, sig, rgb, early_stop_eps=1e-4)
    got = nacc.render_fused(field, o, d, grid, 0.0, 1e10, 0.01, 1e-4, ray_set=ray_set)
    assert float(opacity.max()) > 0.5
    for g, want in zip(got, (color, opacity, depth)):
        assert torch.equal(g.reshape(-1).view(torch.int32), want.reshape(-1).view(torch.int32))
