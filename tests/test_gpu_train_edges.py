"""Training edges: parameters that no texel uses, gradients of very different
size side by side, pyramids whose scatter windows do not fit, and batches of
samples, against the binary64 oracle or the call's own parts."""
import numpy as np
import pytest

import synth
from oracle import train as T

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


@pytest.mark.parametrize("n_tex", [1, 3])
@pytest.mark.parametrize("straight", [False, True])
@pytest.mark.parametrize("bad", [np.nan, np.inf, 3e38])
def test_parameters_that_no_texel_uses_change_nothing(bcf, n_tex, straight, bad):
    """The 2 x 2 and 1 x 1 levels keep the top left of their blocks. Whatever
    the other texels' indices and the endpoints of a subset without a texel
    hold, the other gradients are what they are without it, bit for bit (one
    sample a call: no sum has an order to differ in), and theirs are 0."""
    g = synth.rng(1200)
    dims, levels, first = (3 * n_tex, 16, 4), 4, 4 + 1          # 8 x 8: four blocks, then one per level
    nb = synth.chain_blocks(8, 8, levels)
    assert nb == first + 2
    ends = [g.uniform(0.0, 63.0, (nb, 4, 3)).astype(np.float32) for _ in range(n_tex)]
    idxs = [g.uniform(0.0, 1.0, (nb, 16)).astype(np.float32) for _ in range(n_tex)]
    parts = [np.zeros(nb, np.uint8) for _ in range(n_tex)]       # mask 0xCCCC: subset 1 is columns 2 and 3
    params = synth.mlp_params(dims, g).astype(np.float32)
    geo = bcf.TrainGeometry([8] * n_tex, [levels] * n_tex, [dev(p) for p in parts], dims, straight_through=straight)
    unused = np.ones((2, 16), bool)
    unused[0, [0, 1, 4, 5]] = False                              # 2 x 2
    unused[1, 0] = False                                         # 1 x 1
    bad_ends, bad_idxs = [e.copy() for e in ends], [x.copy() for x in idxs]
    for e, x in zip(bad_ends, bad_idxs):
        e[first:, 2:] = bad
        x[first:][unused] = bad
    for q in synth.uniform_queries(8, g, 1.0) + np.array([0.0, 0.0, 2.0], np.float32):
        go = dev(g.standard_normal((1, 4)).astype(np.float32))
        want = bcf.train_backward(geo, [dev(e) for e in ends], [dev(x) for x in idxs], dev(params), dev(q[None]), go)
        got = bcf.train_backward(geo, [dev(e) for e in bad_ends], [dev(x) for x in bad_idxs], dev(params),
                                 dev(q[None]), go)
        for a, b in zip(got[0] + got[1] + [got[2]], want[0] + want[1] + [want[2]]):
            assert torch.equal(a, b)
        for ge, gi in zip(got[0], got[1]):
            assert not ge[first:, 2:].any() and not gi[first:][dev(unused)].any()
            assert ge[first:, :2].any() and gi[first:].any()


@pytest.mark.parametrize("ratio", [1e-4, 1e-9, 1e-13, 1e-20])
@pytest.mark.parametrize("count", [3, 200])
def test_small_gradients_beside_large_ones(bcf, ratio, count):
    """Samples of one 64th of the material whose dL/dG is `ratio` times that of
    the samples next to it: the gradients of the texels that only they touch
    are as accurate (2e-4 of their largest, the training tests' bar) as without
    the neighbours."""
    g = synth.rng(1250 + count)
    res, dims = 256, (3, 16, 4)                                  # a 64th is four texels
    nb = synth.chain_blocks(res, res, 1)
    tex = T.TrainTexture(res, res, 1, endpoints=g.uniform(0.0, 63.0, (nb, 4, 3)).astype(np.float32),
                         indices=g.uniform(0.0, 1.0, (nb, 16)).astype(np.float32),
                         partitions=g.integers(0, 32, nb).astype(np.uint8), lod_bias=0.0)
    params = synth.mlp_params(dims, g).astype(np.float32)
    geo = bcf.TrainGeometry([res], [1], [dev(tex.partitions)], dims)
    for loud, quiet in (((0, 0), (1, 0)), ((10, 21), (10, 20)), ((33, 33), (32, 32))):
        def inside(cell, n):
            return np.concatenate([(np.array(cell) + g.uniform(0.15, 0.85, (n, 2))) / 64.0, np.zeros((n, 1))],
                                  axis=1).astype(np.float32)
        q = np.concatenate([inside(loud, count), inside(quiet, count)])
        go = g.standard_normal((2 * count, 4))
        go[count:] *= ratio
        order = g.permutation(2 * count)
        q, go = q[order], go[order].astype(np.float32)
        got = bcf.train_backward(geo, [dev(tex.endpoints)], [dev(tex.indices)], dev(params), dev(q), dev(go))
        _, r_end, r_idx, _ = T.gradients([tex], dims, params, q, go, False)
        block = quiet[1] * 64 + quiet[0]                         # texels 4 cell .. 4 cell + 3: one block
        for a, ref in ((got[0][0], r_end[0]), (got[1][0], r_idx[0])):
            a, ref = a.cpu().numpy()[block].reshape(-1), ref[block].reshape(-1)
            assert np.abs(ref).max() > 0.0
            assert np.abs(a - ref).max() <= 2e-4 * np.abs(ref).max()


def window_sums(size, level, cells):
    """Sums (three a texel) of a level's scatter window: a region of cells x
    cells 64ths spans that share of the level, and two texels more a side."""
    return 3 * int(np.prod([min(max(s >> level, 1), -(-cells * max(s >> level, 1) // 64) + 2) for s in size]))


def windows_that_fit(size, levels, cells):
    """Levels with a window, and the bytes these take, of a pool of 72 KB."""
    used, fit = 0, 0
    for level in reversed(range(levels)):
        more = 8 * window_sums(size, level, cells)
        if used + more > 72 * 1024:
            break
        used, fit = used + more, fit + 1
    return fit, used


def pyramids(sizes, levels, seed, e_hi=31.0):
    g = synth.rng(seed)
    texs = []
    for (w, h), n in zip(sizes, levels):
        nb = synth.chain_blocks(w, h, n)
        texs.append(T.TrainTexture(w, h, n, endpoints=g.uniform(0.0, e_hi, (nb, 4, 3)).astype(np.float32),
                                   indices=g.uniform(0.0, 1.0, (nb, 16)).astype(np.float32),
                                   partitions=g.integers(0, 32, nb).astype(np.uint8), lod_bias=0.0))
    return texs, g


def backward(bcf, texs, dims, params, q, go):
    geo = bcf.TrainGeometry([(t.width, t.height) for t in texs], [t.levels for t in texs],
                            [dev(t.partitions) for t in texs], dims)
    return bcf.train_backward(geo, [dev(t.endpoints) for t in texs], [dev(t.indices) for t in texs], dev(params),
                              dev(q), dev(go))


def assert_levels_close(texs, got, ref):
    """Block gradients per level and parameter gradients, within 2e-4 of the
    largest of each (the training tests' bar)."""
    def close(a, b, what):
        scale = np.abs(b).max()
        assert np.abs(a - b).max() <= 2e-4 * max(scale, 1e-30), what

    def host(x):
        return x.double().cpu().numpy() if torch.is_tensor(x) else np.asarray(x)

    for t, tex in enumerate(texs):
        for level, (first, bx, by, _, _) in enumerate(tex.level_blocks()):
            sl = slice(first, first + bx * by)
            for k, name in ((0, "endpoints"), (1, "indices")):
                close(host(got[k][t])[sl], host(ref[k][t])[sl], (t, level, name))
    close(host(got[2]), host(ref[2]), "params")


@pytest.mark.parametrize("sizes,levels,fits", [
    ([(2048, 2048)], [1], [0]),                                    # no window at all, no pool
    ([(2048, 2048)], [12], [11]),                                  # all but level 0
    ([(2048, 2048), (64, 64)], [2, 7], [1, 7]),                    # a pool that the first sizes
    ([(64, 256), (4096, 512), (1024, 1024)], [9, 13, 11], [9, 12, 11]),
    ([(2048, 1024)], [3], [3]),                                    # 72,864 bytes of LDS
    ([(1024, 4096)] * 2, [4] * 2, [3, 3])])
def test_levels_without_a_scatter_window(bcf, sizes, levels, fits):
    """Levels whose windows of 2 x 2 cells do not fit the pool take their taps
    straight to memory, beside levels and pyramids that have windows."""
    assert [windows_that_fit(s, n, 2)[0] for s, n in zip(sizes, levels)] == fits
    texs, g = pyramids(sizes, levels, 1300 + len(levels))
    dims = (3 * len(sizes), 16, 4)
    params = synth.mlp_params(dims, g).astype(np.float32)
    q = synth.uniform_queries(3000, g, max(levels) - 1.0)
    q[:, :2] = q[:, :2] * 3.0 - 1.0
    go = g.standard_normal((len(q), 4)).astype(np.float32)
    got = backward(bcf, texs, dims, params, q, go)
    _, r_end, r_idx, r_par = T.gradients(texs, dims, params, q, go, False)
    assert_levels_close(texs, got, (r_end, r_idx, r_par))


@pytest.mark.parametrize("sizes,levels,n", [([(2048, 2048)], [12], (1 << 19) + 77), ([(4096, 256), (64, 64)], [13, 7], (1 << 19) + 1),
                                            ([(32, 32)] * 4, [6] * 4, 1_200_003), ([(128, 128)] * 3, [8] * 3, 262_145)])
def test_backward_of_many_samples_equals_its_parts(bcf, sizes, levels, n):
    """From 2^19 samples on (single cells above 1024 texels a side, wide
    workgroups, several batches of a small material): the gradients are the
    sums of calls of at most 130,000 samples, and a gradient on the last 70
    samples alone is what those 70 give."""
    texs, g = pyramids(sizes, levels, 1350 + len(levels))
    dims = (3 * len(sizes), 16, 4)
    params = synth.mlp_params(dims, g).astype(np.float32)
    q = synth.uniform_queries(n, g, max(levels) - 1.0)
    go = g.standard_normal((n, 4)).astype(np.float32)
    parts = None
    for first in range(0, n, 130_000):
        part = backward(bcf, texs, dims, params, q[first:first + 130_000], go[first:first + 130_000])
        part = [[x.double() for x in part[0]], [x.double() for x in part[1]], part[2].double()]
        parts = part if parts is None else [[a + b for a, b in zip(parts[0], part[0])],
                                            [a + b for a, b in zip(parts[1], part[1])], parts[2] + part[2]]
    assert_levels_close(texs, backward(bcf, texs, dims, params, q, go), parts)
    go[:-70] = 0.0
    assert_levels_close(texs, backward(bcf, texs, dims, params, q, go), backward(bcf, texs, dims, params, q[-70:], go[-70:]))
