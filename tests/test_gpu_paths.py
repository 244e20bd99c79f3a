"""The kernels' size and layout edges: each path a dispatch can take, at the
sizes where it can go wrong, against the oracle or the general path."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bcf():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    import paper_2311_16121_amd as bcf
    return bcf


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def material(bcf, sizes, levels, dims, seed, bias=None, signed=False):
    """(device material, oracle material) of bounded random blocks."""
    g = synth.rng(seed)
    texs = [synth.bounded_blocks(synth.chain_blocks(w, h, L), g, signed=signed).reshape(-1)
            for (w, h), L in zip(sizes, levels)]
    params = synth.mlp_params(dims, synth.rng(seed + 1))
    bias = bias or [0.0] * len(sizes)
    return (bcf.Material.from_host(texs, sizes, levels, dims, params, bias, signed),
            oracle.Material(texs, sizes, levels, dims, params, bias, signed))


@pytest.mark.parametrize("sizes,dims", [([(64, 64)] * 4, (12, 16, 16, 9)), ([(64, 32)] * 2, (6, 64, 24, 16)),
                                        ([(64, 64), (32, 32), (16, 16)], (9, 33, 11))])
def test_fp32_decode_and_calibration_share_a_workspace(bcf, sizes, dims):
    """BCF_FP32 evaluates what BCF_FP32_MFMA does, bit for bit, also after a
    calibration wrote its own operands into the same workspace."""
    levels = [max(s).bit_length() for s in sizes]
    mat, host = material(bcf, sizes, levels, dims, seed=90)
    q = synth.uniform_queries(501, synth.rng(91), float(levels[0] - 1))
    ws, wsm = bcf.prepare(mat, bcf.Precision.FP32), bcf.prepare(mat, bcf.Precision.FP32_MFMA)
    want = bcf.decode(mat, wsm, dev(q), bcf.Precision.FP32_MFMA).cpu().numpy()
    assert np.array_equal(bcf.decode(mat, ws, dev(q)).cpu().numpy(), want)
    absmax = torch.empty(len(dims) - 1, device="cuda")
    import ctypes as C
    assert bcf.lib.bcf_calibrate(C.byref(mat.c), C.c_void_p(ws.data_ptr()), C.c_void_p(dev(q).data_ptr()), len(q),
                                 C.c_void_p(absmax.data_ptr()), None) == 0
    torch.cuda.synchronize()
    assert np.array_equal(bcf.decode(mat, ws, dev(q)).cpu().numpy(), want)
    assert np.abs(want - oracle.decode(host, q)).max() <= 1e-5
    # z0's largest magnitude: one binary32 filter against binary64, so a few ulp
    assert abs(float(absmax[0]) - np.abs(oracle.sample(host, q)).max()) <= 1e-6


@pytest.mark.parametrize("n,dims", [(1, (12, 32, 32, 10)), (15, (12, 16, 1)), (17, (9, 32, 16)), (63, (12, 16, 16, 8)),
                                    (65, (12, 32, 32, 32, 16)), (130, (3, 16, 16, 16, 3))])
def test_training_backward_over_ragged_groups(bcf, n, dims):
    """The backward's groups of 16 samples and chunks of 64, partly filled, at
    every depth and width of its tiles, against the binary64 oracle. The bar is
    the training tests' (2e-4 of a tensor's largest gradient: binary32 sums)."""
    from oracle import train as T
    g = synth.rng(700 + n)
    texs = []
    for _ in range(dims[0] // 3):
        nb = synth.chain_blocks(32, 32, 6)
        texs.append(T.TrainTexture(32, 32, 6, endpoints=g.uniform(0.0, 31.0, (nb, 4, 3)).astype(np.float32),
                                   indices=g.uniform(0.0, 1.0, (nb, 16)).astype(np.float32),
                                   partitions=g.integers(0, 32, nb).astype(np.uint8), lod_bias=0.0))
    params = synth.mlp_params(dims, g).astype(np.float32)
    q = synth.uniform_queries(n, g, 5.0)
    go = g.standard_normal((n, dims[-1])).astype(np.float32)
    geo = bcf.TrainGeometry([32] * len(texs), [6] * len(texs), [dev(t.partitions) for t in texs], dims,
                            straight_through=True)
    g_end, g_idx, g_par = bcf.train_backward(geo, [dev(t.endpoints) for t in texs], [dev(t.indices) for t in texs],
                                             dev(params), dev(q), dev(go))
    _, r_end, r_idx, r_par = T.gradients(texs, dims, params, q, go, True)
    for got, ref in list(zip(g_end, r_end)) + list(zip(g_idx, r_idx)) + [(g_par, r_par)]:
        ref = np.asarray(ref)
        err = np.abs(got.cpu().numpy().reshape(ref.shape) - ref).max()
        assert err <= 2e-4 * max(np.abs(ref).max(), 1e-30)


@pytest.mark.parametrize("n,res", [(300, 64), (5000, 1024), (3000, 2048)])
def test_training_scatter_with_an_infinite_gradient(bcf, n, res):
    """One sample's infinite dL/dG makes its own texels' gradients non-finite
    (its region then sums in floats) and leaves every other gradient what it is
    without that sample, to the rounding of binary32 sums (1e-5 of the largest)."""
    g = synth.rng(900 + n)
    levels = res.bit_length()
    nb = synth.chain_blocks(res, res, levels)
    dims = (6, 16, 4)
    geo = bcf.TrainGeometry([res] * 2, [levels] * 2, [dev(g.integers(0, 32, nb).astype(np.uint8))] * 2, dims)
    ends = [dev(g.uniform(0.0, 31.0, (nb, 4, 3)).astype(np.float32)) for _ in range(2)]
    idxs = [dev(g.uniform(0.0, 1.0, (nb, 16)).astype(np.float32)) for _ in range(2)]
    p = dev(synth.mlp_params(dims, g).astype(np.float32))
    q = synth.uniform_queries(n, g, 2.0)             # fine levels, so that few texels are touched
    go = g.standard_normal((n, 4)).astype(np.float32)
    go[7] = 0.0
    want = bcf.train_backward(geo, ends, idxs, p, dev(q), dev(go))
    go[7] = np.inf
    got = bcf.train_backward(geo, ends, idxs, p, dev(q), dev(go))
    some = 0
    for a, b in zip(got[0] + got[1], want[0] + want[1]):
        a, b = a.cpu().numpy(), b.cpu().numpy()
        ok = np.isfinite(a)
        some += (~ok).sum()
        assert np.isfinite(b).all() and ok.mean() > 0.5
        assert np.abs(a[ok] - b[ok]).max() <= 1e-5 * np.abs(b).max()
    assert some > 0


@pytest.mark.parametrize("sizes,levels", [([(64, 64)] * 4, 7), ([(32, 64)] * 3, 7), ([(4, 4)] * 3, 3), ([(1, 8)] * 4, 4),
                                          ([(2, 2)] * 4, 2)])
@pytest.mark.parametrize("shift,straight", [(0, True), (1, True), (1, False)])
def test_training_packed_texels_equal_the_images(bcf, sizes, levels, shift, straight):
    """Pyramids of one geometry go through packed positions: the same outputs,
    bit for bit, as from float images (which a pyramid with another bias
    forces). Parameters 16-byte aligned and not (shift)."""
    g = synth.rng(950)
    dims = (12, 16, 16, 5) if len(sizes) == 4 else (9, 16, 16, 5)
    nb = [synth.chain_blocks(w, h, levels) for w, h in sizes]

    def moved(x):
        flat = torch.zeros(x.size + shift, device="cuda")
        flat[shift:] = dev(x.reshape(-1))
        return flat[shift:].view(x.shape)

    ends = [moved(g.uniform(-1.0, 64.0, (n, 4, 3)).astype(np.float32)) for n in nb]
    idxs = [moved(g.uniform(-0.1, 1.1, (n, 16)).astype(np.float32)) for n in nb]
    parts = [dev(g.integers(0, 256, n).astype(np.uint8)) for n in nb]
    p = dev(synth.mlp_params(dims, g).astype(np.float32))
    q = synth.uniform_queries(1000, g, float(levels))
    q[:, :2] = q[:, :2] * 3.0 - 1.0
    q[:, 2] -= 0.5
    go = dev(g.standard_normal((len(q), 5)).astype(np.float32))

    def geometry(bias):
        return bcf.TrainGeometry(sizes, [levels] * len(sizes), parts, dims, bias, straight_through=straight)

    # a bias that rounds away (|s| + 1e-30) makes the geometries differ
    one, other = geometry([0.0] * len(sizes)), geometry([0.0] * (len(sizes) - 1) + [1e-30])
    assert torch.equal(bcf.train_forward(one, ends, idxs, p, dev(q)), bcf.train_forward(other, ends, idxs, p, dev(q)))
    # one sample at a time: no sum has an order to differ in
    for k in range(0, 1000, 125):
        (ge, gi, gp), (re, ri, rp) = (bcf.train_backward(geo, ends, idxs, p, dev(q[k:k + 1]), go[k:k + 1])
                                      for geo in (one, other))
        for a, b in list(zip(ge, re)) + list(zip(gi, ri)) + [(gp, rp)]:
            assert torch.equal(a, b)


@pytest.mark.parametrize("n,grid,out_dim", [
    (1, 0, 1), (5, 0, 3), (63, 0, 9), (64, 0, 16), (65, 0, 7), (129, 0, 10), (4097, 0, 3),      # linear items
    (32768, 0, 1), (32769, 0, 1), (33001, 0, 5),                                               # linear strips
    (1, 1, 1), (7, 3, 1), (70, 7, 3), (81, 9, 9), (15 * 8 + 4, 15, 16), (33 * 17, 33, 10), (201 * 173 - 5, 201, 7)])
def test_decode_stores_every_row_and_nothing_else(bcf, n, grid, out_dim):
    """Linear launches and images whose rows leave 1..3 floats over, in outputs
    at every four-byte alignment, with the bytes around them kept."""
    mat, host = material(bcf, [(64, 64)] * 4, [7] * 4, (12, 16, out_dim), seed=130)
    q = synth.uniform_queries(n, synth.rng(131), 6.0)
    want = oracle.decode(host, q)
    ws = bcf.prepare(mat, bcf.Precision.FP32)
    for shift in range(4):
        buf = torch.full((64 + n * out_dim + 64,), -77.0, device="cuda")
        out = buf[64 + shift - 4:][:n * out_dim].view(n, out_dim)
        bcf.decode(mat, ws, dev(q), grid_width=grid, out=out)
        got = buf.cpu().numpy()
        lo = 64 + shift - 4
        assert np.abs(got[lo:lo + n * out_dim].reshape(n, out_dim) - want).max() <= 1e-5
        assert (got[:lo] == -77.0).all() and (got[lo + n * out_dim:] == -77.0).all()


@pytest.mark.parametrize("n_tex,size,levels", [(3, (64, 64), 7), (3, (8, 2), 4), (3, (1, 32), 6), (3, (256, 4), 1),
                                               (2, (64, 64), 7), (2, (2, 16), 3), (1, (64, 64), 7), (1, (1, 1), 1)])
def test_pyramids_of_one_geometry_in_each_count(bcf, n_tex, size, levels):
    """One to three pyramids of one geometry: the packed scratch of three, the
    two-slot filter of one and two, single and batched, whole and touched."""
    dims = (3 * n_tex, 16, 10)
    mats, hosts = zip(*(material(bcf, [size] * n_tex, [levels] * n_tex, dims, seed=140 + k, bias=[-0.5] * n_tex)
                        for k in range(2)))
    q = synth.uniform_queries(1500, synth.rng(143), float(levels))
    offsets = np.array([0, 1000, 1500], np.int32)
    wants = [oracle.decode(hosts[0], q[:1000]), oracle.decode(hosts[1], q[1000:])]
    for prec, tol in (("FP32", 1e-5), ("FP16", 2e-3)):
        p = bcf.Precision[prec]
        batch = bcf.Batch(list(mats), p, ws_fill=0xFF)
        batch.unpack_touched(dev(q), dev(offsets))
        touched = batch.decode(dev(q), dev(offsets)).cpu().numpy()
        batch.unpack()
        assert np.array_equal(batch.decode(dev(q), dev(offsets)).cpu().numpy(), touched)
        for k, part in enumerate((slice(0, 1000), slice(1000, 1500))):
            single = bcf.decode(mats[k], bcf.prepare(mats[k], p), dev(q[part]), p).cpu().numpy()
            assert np.array_equal(single, touched[part])
            assert np.abs(single - wants[k]).max() <= tol
    # z0's largest magnitude: one binary32 filter against binary64, so a few ulp
    absmax = bcf.calibrate(mats[0], dev(q)).cpu().numpy()
    assert abs(float(absmax[0]) - np.abs(oracle.sample(hosts[0], q)).max()) <= 1e-6


@pytest.mark.parametrize("sizes", [[(64, 64), (32, 32), (16, 16), (8, 8)], [(64, 32)] * 2, [(32768, 4)], [(4, 32768)],
                                   [(16384, 4)] * 3, [(4, 16384)] * 4])
@pytest.mark.parametrize("n,grid,out_dim", [(1, 0, 2), (321, 0, 7), (40 * 21, 40, 8), (33 * 17 - 2, 33, 5),
                                            (150 * 140, 150, 10)])
def test_every_layout_under_every_item_kind(bcf, sizes, n, grid, out_dim):
    """Runs of 64 queries, tiles and tiles with ragged rows over each texel
    layout, up to the longest rows and columns a level may have."""
    levels = [3] * len(sizes)
    mat, host = material(bcf, sizes, levels, (3 * len(sizes), 16, out_dim), seed=150)
    q = synth.uniform_queries(n, synth.rng(151), 2.0)
    got = bcf.decode(mat, bcf.prepare(mat, bcf.Precision.FP32), dev(q), grid_width=grid).cpu().numpy()
    pick = np.unique(np.linspace(0, n - 1, 1500).astype(int))
    assert np.abs(got[pick] - oracle.decode(host, q[pick])).max() <= 1e-5


@pytest.mark.parametrize("precision", ["FP32", "FP16", "BF16", "FP8"])
@pytest.mark.parametrize("sizes,dims,signed", [([(64, 64)] * 4, (12, 16, 1), False), ([(8, 4)], (3, 64, 64, 64, 16), True),
                                               ([(64, 32), (16, 16)], (6, 33, 24, 7), True)])
def test_decode_without_a_workspace_equals_one_with(bcf, precision, sizes, dims, signed):
    """The launch that unpacks and converts the operands together, against
    bcf_prepare and bcf_decode, bit for bit."""
    p = bcf.Precision[precision]
    mat, _ = material(bcf, sizes, [max(s).bit_length() for s in sizes], dims, seed=160, signed=signed)
    q = dev(synth.uniform_queries(300, synth.rng(161), 4.0))
    if precision == "FP8":
        mat.set_act_absmax(bcf.calibrate(mat, q))
    want = bcf.decode(mat, bcf.prepare(mat, p), q, p)
    assert torch.equal(bcf.decode_noalloc(mat, q, p).view(torch.int32), want.view(torch.int32))


def test_training_backward_in_batches_equals_its_parts(bcf):
    """More samples than the workspace of a small material sorts at once: the
    gradients are the sums of two calls' that each fit one batch."""
    sizes, levels, dims, n = [(32, 32)] * 4, [6] * 4, (12, 16, 4), 700_003
    g = torch.Generator("cuda").manual_seed(170)
    blocks = [sum(max((s >> l) // 4, 1) ** 2 for l in range(6)) for s, _ in sizes]
    ends = [60.0 * torch.rand((b, 4, 3), device="cuda", generator=g) for b in blocks]
    idxs = [torch.rand((b, 16), device="cuda", generator=g) for b in blocks]
    parts = [torch.randint(0, 32, (b,), device="cuda", generator=g, dtype=torch.uint8) for b in blocks]
    n_par = sum(a * b + b for a, b in zip(dims[:-1], dims[1:]))
    params = torch.randn(n_par, device="cuda", generator=g) * 0.3
    q = torch.rand((n, 3), device="cuda", generator=g) * torch.tensor([1.0, 1.0, 5.0], device="cuda")
    go = torch.rand((n, 4), device="cuda", generator=g)
    geo = bcf.TrainGeometry(sizes, levels, parts, dims)

    def flat(r):
        return [t.double() for t in r[0] + r[1] + [r[2]]]

    whole = flat(bcf.train_backward(geo, ends, idxs, params, q, go))
    halves = [flat(bcf.train_backward(geo, ends, idxs, params, q[s], go[s]))
              for s in (slice(0, 350_000), slice(350_000, n))]
    for w, a, b in zip(whole, *halves):
        # fp32 sums of some hundred partial sums each way, in any order
        assert float((w - a - b).abs().max()) <= 1e-3 * float(w.abs().max()) + 1e-12


@pytest.mark.parametrize("n_mats", [1, 63, 64, 65, 130])
def test_batches_around_the_materials_a_wave_holds(bcf, n_mats):
    """Items found from the lanes and from the table, with empty materials at
    both ends and in between: whole and touched unpacks equal single decodes."""
    g = synth.rng(180)
    mats = [material(bcf, [(16, 16), (16, 16), (16, 16)] if k % 2 else [(32, 16), (16, 16), (8, 8)], [3, 3, 3],
                     (9, 16, 3), seed=181 + k)[0] for k in range(5)]
    mats = [mats[k % 5] for k in range(n_mats)]
    counts = g.integers(0, 3, n_mats) * g.integers(1, 150, n_mats)
    counts[0] = 0 if n_mats > 1 else 100
    counts[-1] = 0 if n_mats > 1 else 100
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    q = dev(synth.uniform_queries(int(offsets[-1]), g, 2.0))
    batch = bcf.Batch(mats, bcf.Precision.FP16, ws_fill=0xFF)
    batch.unpack_touched(q, dev(offsets))
    touched = batch.decode(q, dev(offsets))
    batch.unpack()
    assert torch.equal(batch.decode(q, dev(offsets)), touched)
    for k in np.flatnonzero(counts):
        part = slice(int(offsets[k]), int(offsets[k + 1]))
        assert torch.equal(bcf.decode(mats[k], bcf.prepare(mats[k], bcf.Precision.FP16), q[part], bcf.Precision.FP16),
                           touched[part])


@pytest.mark.parametrize("n_tex,signed", [(4, False), (3, True), (2, False)])
def test_a_large_scratch_unpacks_the_same_past_the_caches(bcf, n_tex, signed):
    """decode() of few queries stores a scratch above 64 MiB non-temporally, of
    many ordinarily: the same texels, so the same bits."""
    sizes, levels = [(2048, 2048)] * n_tex, [12] * n_tex
    g = synth.rng(190)
    block = synth.bounded_blocks(4096, g, signed=signed).reshape(-1)
    texs = [np.resize(np.roll(block, 16 * 7 * t), 16 * synth.chain_blocks(2048, 2048, 12)) for t in range(n_tex)]
    dims = (3 * n_tex, 16, 5)
    mat = bcf.Material.from_host(texs, sizes, levels, dims, synth.mlp_params(dims, g), [0.0] * n_tex, signed)
    ws = bcf.prepare(mat, bcf.Precision.FP16)
    assert ws.numel() > 64 << 20
    q = dev(synth.uniform_queries(900_000, g, 11.0))
    many = bcf.decode(mat, ws, q, bcf.Precision.FP16)
    assert torch.equal(bcf.decode(mat, ws, q[:5000], bcf.Precision.FP16), many[:5000])
    bcf.unpack(mat, ws)
    assert torch.equal(bcf.decode_unpacked(mat, ws, q, bcf.Precision.FP16), many)
