"""Edges of the decode calls: the largest materials that fit the library's own
workspace, and unpacks that must store every texel."""
import numpy as np
import pytest

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


def material(bcf, sizes, levels, dims, seed, signed=False):
    """Pyramids of the same bounded random blocks over and over, each rolled."""
    g = synth.rng(seed)
    block = synth.bounded_blocks(4096, g, signed=signed).reshape(-1)
    texs = [np.resize(np.roll(block, 16 * 7 * t), 16 * synth.chain_blocks(w, h, n))
            for t, ((w, h), n) in enumerate(zip(sizes, levels))]
    return bcf.Material.from_host(texs, sizes, levels, dims, synth.mlp_params(dims, g), [0.0] * len(sizes), signed)


@pytest.mark.parametrize("sizes,levels,dims,fits", [
    # texel scratch and row-major operands 67,107,584, 67,108,608 and 67,108,864 (= 64 MiB) bytes
    ([(512, 4096), (512, 8192)], [3, 5], (6, 64, 64, 10), True),
    ([(1, 1), (8192, 256), (512, 8192)], [1, 4, 4], (9, 32, 32, 10), True),
    ([(8192, 256), (4096, 1024)], [9, 5], (6, 16, 16, 8), True),
    ([(8192, 256), (4096, 1024)], [9, 5], (6, 16, 16, 11), False)])
def test_fp32_materials_that_just_fit_the_librarys_workspace(bcf, sizes, levels, dims, fits):
    """BCF_FP32 counts its operands' true rows against the 64 MiB."""
    mat = material(bcf, sizes, levels, dims, 300)
    q = dev(synth.uniform_queries(2000, synth.rng(301), max(levels) - 1.0))
    if not fits:
        with pytest.raises(bcf.BcfError, match="status 2.*workspace"):
            bcf.decode_noalloc(mat, q)
        return
    want = bcf.decode(mat, bcf.prepare(mat), q)
    assert torch.equal(bcf.decode_noalloc(mat, q).view(torch.int32), want.view(torch.int32))


def test_calibration_evaluates_the_prepared_parameters(bcf):
    """Until it is prepared again, a workspace decodes and calibrates with the
    parameters that bcf_prepare converted."""
    import ctypes as C
    dims = (6, 33, 24, 7)
    mat = material(bcf, [(64, 32)] * 2, [7, 7], dims, 310)
    q = dev(synth.uniform_queries(700, synth.rng(311), 6.0))
    ws = bcf.prepare(mat)

    def evaluate():
        absmax = torch.empty(len(dims) - 1, device="cuda")
        assert bcf.lib.bcf_calibrate(C.byref(mat.c), C.c_void_p(ws.data_ptr()), C.c_void_p(q.data_ptr()), len(q),
                                     C.c_void_p(absmax.data_ptr()), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        return bcf.decode(mat, ws, q), absmax

    before = evaluate()
    assert torch.equal(before[1], bcf.calibrate(mat, q))
    mat.params.mul_(2.0)
    after = evaluate()
    assert all(torch.equal(a, b) for a, b in zip(before, after))
    ws = bcf.prepare(mat)
    assert float(evaluate()[1][1]) > 1.5 * float(before[1][1])


def three_pyramids(bcf, n_mats, res, per, seed):
    """(batch on a workspace of ones, materials, queries, offsets) of three pyramids of one geometry."""
    levels = res.bit_length()
    mats = [material(bcf, [(res, res)] * 3, [levels] * 3, (9, 16, 5), seed + k) for k in range(min(n_mats, 3))]
    mats = [mats[k % len(mats)] for k in range(n_mats)]
    q = synth.uniform_queries(n_mats * per, synth.rng(seed + 9), levels - 1.0)
    q[:, :2] = q[:, :2] * 3.0 - 1.0
    offsets = np.arange(0, n_mats * per + 1, per, dtype=np.int32)
    return bcf.Batch(mats, bcf.Precision.FP16, ws_fill=0xFF), mats, dev(q), dev(offsets)


@pytest.mark.parametrize("n_mats,res", [(9, 512), (5, 1024)])
def test_three_pyramids_in_a_large_scratch_are_marked(bcf, n_mats, res):
    """Above 64 MiB the touched unpack marks the blocks of packed materials of
    three pyramids: decodes equal the single materials', on texels of NaN."""
    per = 333
    batch, mats, q, offsets = three_pyramids(bcf, n_mats, res, per, 320)
    batch.unpack_touched(q, offsets)
    got = batch.decode(q, offsets)
    elsewhere = q.roll(per, 0) + torch.tensor([0.37, 0.37, 0.0], device="cuda")
    partly = batch.decode(elsewhere, offsets)
    batch.unpack()
    assert not torch.equal(batch.decode(elsewhere, offsets), partly)      # blocks that no query touched were not there
    for k, mat in enumerate(mats):
        part = slice(k * per, (k + 1) * per)
        want = bcf.decode(mat, bcf.prepare(mat, bcf.Precision.FP16), q[part], bcf.Precision.FP16)
        assert torch.equal(got[part], want)


@pytest.mark.parametrize("n_mats,res", [(1, 64), (7, 512), (70, 64)])
def test_three_pyramids_in_a_small_scratch_are_unpacked_whole(bcf, n_mats, res):
    """Up to 64 MiB it unpacks them whole: any decode equals the single one."""
    per = 65
    batch, mats, q, offsets = three_pyramids(bcf, n_mats, res, per, 340)
    batch.unpack_touched(q[:1], torch.zeros_like(offsets))
    got = batch.decode(q, offsets)
    for k, mat in enumerate(mats):
        part = slice(k * per, (k + 1) * per)
        want = bcf.decode(mat, bcf.prepare(mat, bcf.Precision.FP16), q[part], bcf.Precision.FP16)
        assert torch.equal(got[part], want)


def test_touched_blocks_of_more_than_a_gigabyte(bcf):
    """Above 1 GiB of scratch the touched blocks are stored past the caches:
    decodes equal the single material's, on texels of ones."""
    mat = material(bcf, [(2048, 2048)] * 4, [12] * 4, (12, 16, 5), 360)
    n_mats, per = 9, 1111
    batch = bcf.Batch([mat] * n_mats, bcf.Precision.FP16, ws_fill=0xFF)
    assert batch.ws.numel() > 1 << 30
    q = dev(synth.uniform_queries(n_mats * per, synth.rng(361), 11.0))
    offsets = dev(np.arange(0, n_mats * per + 1, per, dtype=np.int32))
    batch.unpack_touched(q, offsets)
    want = bcf.decode(mat, bcf.prepare(mat, bcf.Precision.FP16), q, bcf.Precision.FP16)
    assert torch.equal(batch.decode(q, offsets), want)


@pytest.mark.parametrize("n", [(1 << 24) - 1, 1 << 24, (1 << 24) + 4097])
def test_marks_of_many_queries_beyond_an_l2(bcf, n):
    """From 2^24 queries on, marks of more than 4 MiB are set by two rounds of
    workgroups: decodes equal the single material's, on texels of ones."""
    mat = material(bcf, [(2048, 2048)] * 4, [12] * 4, (12, 16, 5), 370)
    n_mats, pool = 13, 65536
    batch = bcf.Batch([mat] * n_mats, bcf.Precision.FP16, ws_fill=0xFF)
    few = dev(synth.uniform_queries(pool, synth.rng(371), 11.0))
    q = few.repeat(n // pool + 1, 1)[:n].contiguous()
    offsets = dev(np.linspace(0, n, n_mats + 1).astype(np.int32))
    batch.unpack_touched(q, offsets)
    want = bcf.decode(mat, bcf.prepare(mat, bcf.Precision.FP16), few, bcf.Precision.FP16)
    assert torch.equal(batch.decode(q, offsets), want.repeat(n // pool + 1, 1)[:n])


@pytest.mark.parametrize("sizes,signed", [([(2048, 2048)] * 4, False), ([(2048, 2048)] * 3, True), ([(4096, 4096)], False),
                                          ([(4096, 2048), (2048, 2048), (2048, 1024)], True)])
def test_unpacks_past_the_caches_store_every_texel(bcf, sizes, signed):
    """Above 128 MiB of scratch the unpack of few points, of an image and by
    itself (of pyramids of their own) stores past the caches, of many points and
    of a large image ordinarily: on a scratch of ones each leaves texels from
    which every query decodes to the same bits, within 2e-3 of the oracle."""
    import oracle
    levels, dims, bias = [s[0].bit_length() for s in sizes], (3 * len(sizes), 16, 5), [0.0] * len(sizes)
    g = synth.rng(380)
    block = synth.bounded_blocks(4096, g, signed=signed).reshape(-1)
    texs = [np.resize(np.roll(block, 16 * 7 * t), 16 * synth.chain_blocks(w, h, n))
            for t, ((w, h), n) in enumerate(zip(sizes, levels))]
    params = synth.mlp_params(dims, g)
    mat = bcf.Material.from_host(texs, sizes, levels, dims, params, bias, signed)
    p = bcf.Precision.FP16
    ws = bcf.prepare(mat, p)
    offset, size = (int(x) for x in ws[24:40].cpu().numpy().view(np.uint64))     # of the scratch, from the header
    assert size > 128 << 20
    q = synth.uniform_queries(6 * (1 << 20), g, levels[0] - 1.0)
    q[:4000, :2] = np.round(q[:4000, :2] * 256) / 256                            # block corners and wrap columns
    qd, few = dev(q), 5000

    def decode(**kw):
        return bcf.decode_unpacked(mat, ws, qd, p, **kw).view(torch.int32)

    def spoil():
        ws[offset:offset + size] = 0xFF

    want = None
    for unpack in (lambda: bcf.decode(mat, ws, qd, p), lambda: bcf.decode(mat, ws, qd[:few], p),
                   lambda: bcf.decode(mat, ws, qd[:few], p, grid_width=100), lambda: bcf.unpack(mat, ws),
                   lambda: bcf.decode(mat, ws, qd, p, grid_width=4096)):
        spoil()
        unpack()
        got = decode()
        want = got if want is None else want
        assert torch.equal(got, want)
    host = oracle.Material(texs, sizes, levels, dims, params, bias, signed)
    assert np.abs(want[:few].view(torch.float32).cpu().numpy() - oracle.decode(host, q[:few])).max() <= 2e-3
