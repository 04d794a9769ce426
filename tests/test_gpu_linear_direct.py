"""Projections whose workgroups keep all of k: the tiles of 16 .. 64 rows of x by 16 .. 64 features, at row counts around the tiles'
edges, feature counts that leave the last tile short or put two outputs into one tile, k of less than a chunk, with a short last
chunk, shorter and longer than the ring, and a multiple of 4096 (where tiles start their walk in different places)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_07590_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2410_07590_amd import binding
    binding.lib()
    return binding

ROWS = [1, 15, 16, 17, 33, 48, 49, 64, 65, 96, 97, 128]
FEATURES = [(32,), (96, 32, 64), (4064,), (2048, 1056)]
DEPTHS = [16, 80, 128, 144, 1040, 4096]


def run(B, x, weights, guard=2):
    M = x.shape[0]
    ys = [torch.full((M + guard, w.shape[0]), float("nan"), dtype=torch.bfloat16, device="cuda") for w in weights]
    feats = [w.shape[0] for w in weights]
    scratch = B.workspace(B.tr_linear_workspace_size(M, feats, x.shape[1]))
    B.tr_linear(x.cuda(), [w.cuda() for w in weights], [y[:M] for y in ys], scratch)
    torch.cuda.synchronize()
    assert all(torch.isnan(y[M:]).all() for y in ys), "rows behind the last one were written"
    return [H.to_f64(y[:M]) for y in ys]


@pytest.mark.parametrize("K", DEPTHS)
@pytest.mark.parametrize("feats", FEATURES, ids=lambda f: "x".join(map(str, f)))
def test_against_fp64(B, feats, K):
    """Row counts one after the other over the same weights, in whichever kernel the call takes (few features with a long k take
    slices).  |err| <= 2^-8 |y| (the rounding of the result) + 1e-3: fp32 sums of up to 4096 products of unit variance over sqrt(K)."""
    rng = np.random.Generator(np.random.PCG64([612, sum(feats), K]))
    weights = [(synth.normal_tensor(rng, (n, K), torch.float32) * K ** -0.5).to(torch.bfloat16) for n in feats]
    xs = synth.normal_tensor(rng, (max(ROWS), K), torch.bfloat16)
    want = [oracle.linear(H.bits(xs), H.bits(w)) for w in weights]
    worst = 0.0
    for M in ROWS:
        for got, w in zip(run(B, xs[:M], weights), want):
            assert np.isfinite(got).all(), M
            err = np.abs(got - w[:M])
            assert (err <= 2.0 ** -8 * np.abs(w[:M]) + 1e-3).all(), "%d rows: max abs err %.3e" % (M, err.max())
            worst = max(worst, float(err.max()))
    print("features %s K %d: max abs err %.3e" % (feats, K, worst))


# tile in blocks of 16 rows and 16 features -> products that take it at the depths of the test below
TILES = {
    (1, 1): [(1, (4064,)), (16, (2048, 1056)), (128, (32,)), (49, (96, 32, 64))],
    (1, 2): [(1, (4128,)), (16, (5536, 64, 32)), (17, (4064,)), (32, (2048, 1056))],
    (1, 3): [(15, (8288,)), (16, (10272,))],
    (1, 4): [(15, (12352,)), (16, (12416, 32))],
    (2, 2): [(17, (8192,)), (32, (4096, 1056, 1056)), (49, (4064,)), (64, (2048, 1056))],
    (2, 3): [(17, (8256,)), (32, (10272,)), (33, (2048, 2080)), (80, (2048, 1056))],
    (2, 4): [(17, (12352,)), (32, (16384,)), (49, (4096, 1056, 1056)), (128, (4096,))],
    (3, 2): [(33, (6176,)), (48, (8192,)), (65, (4096,)), (96, (4096,))],
    (3, 3): [(33, (8288,)), (48, (10272,)), (65, (5536, 64, 32)), (97, (2048, 1056))],
    (3, 4): [(33, (12416, 32)), (48, (16384,)), (81, (6176,)), (128, (2048, 2080))],
    (4, 3): [(49, (8256,)), (64, (10272,)), (97, (5504,)), (128, (5536, 64, 32))],
    (4, 4): [(49, (12352,)), (64, (16384,)), (97, (4096, 1056, 1056)), (128, (6176,))],
}
TILE_DEPTHS = [144, 2064]   # a short last chunk inside the ring, and behind more chunks than the ring and one accumulator take


@pytest.mark.parametrize("tile", TILES, ids=lambda t: "%dx%d" % t)
def test_every_tile_against_fp64(B, tile):
    """The tile is the one that the library says it takes; the bound is that of the test above, for sums of up to 2064 products."""
    for case, (M, feats) in enumerate(TILES[tile]):
        for K in TILE_DEPTHS:
            assert B.lib().tr_linear_direct_tile(M, sum(feats), K) == 16 * tile[0] + tile[1], (M, feats, K)
            g = torch.Generator(device="cuda").manual_seed(615 + case + K)
            draw = lambda *size: torch.randn(size, generator=g, device="cuda")
            x, weights = draw(M, K).bfloat16(), [(draw(n, K) * K ** -0.5).bfloat16() for n in feats]
            for got, w in zip(run(B, x, weights), weights):
                want = H.to_f64(torch.matmul(x.double(), w.double().T))
                err = np.abs(got - want)
                assert (err <= 2.0 ** -8 * np.abs(want) + 1e-3).all(), (M, feats, K, float(err.max()))


@pytest.mark.parametrize("M,N,K", [(5, 3584, 4064), (33, 6144, 4064), (17, 6144, 4080), (128, 4096, 4112), (5, 4096, 4128),
                                   (128, 5120, 4128), (32, 8192, 8192)])
def test_rows_about_a_multiple_of_8_kb_apart(B, M, N, K):
    """Tiles start their walks at different chunks, the short last one among them, and wrap round.  Bound as above."""
    assert B.lib().tr_linear_direct_tile(M, N, K) != 0
    g = torch.Generator(device="cuda").manual_seed(616 + K)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    w = (torch.randn(N, K, generator=g, device="cuda") * K ** -0.5).bfloat16()
    got, = run(B, x, [w])
    want = H.to_f64(torch.matmul(x.double(), w.double().T))
    err = np.abs(got - want)
    assert (err <= 2.0 ** -8 * np.abs(want) + 1e-3).all(), float(err.max())


def test_infinity_stays_in_its_row(B):
    """The pieces of a short last chunk that lie past the end of a row take no part, whatever the row ends in."""
    K, n = 144, 64
    rng = np.random.Generator(np.random.PCG64([613]))
    x = synth.normal_tensor(rng, (20, K), torch.bfloat16)
    x[3, K - 1] = float("inf")
    w = (synth.normal_tensor(rng, (n, K), torch.float32) * K ** -0.5).to(torch.bfloat16)
    got, = run(B, x, [w])
    assert np.array_equal(got[3], np.sign(H.to_f64(w)[:, K - 1]) * np.inf)
    assert np.isfinite(np.delete(got, 3, axis=0)).all()


@pytest.mark.parametrize("M,N,K", [(64, 3584, 3584), (5, 2048, 2048), (128, 4608, 3584), (64, 4608, 3584), (128, 512, 3584),
                                   (128, 4608, 4096), (16, 4096, 4096), (64, 8192, 8192), (16, 512, 512)])
def test_no_less_precise_than_the_slices(B, M, N, K):
    """The error of the fp32 sums alone, all of k in a workgroup against the slices that the call would take otherwise: every
    product has its negative somewhere in the row, so the exact results are zero and what is left is rounding of the sums (a result
    near one hides it behind its own rounding, 2^-9 against 1e-7).  Root mean square over at least 8192 results, known to 1 %;
    a chain of k through the accumulators that is a third longer shows as 15 %."""
    gen = torch.Generator().manual_seed(614 + M + N)
    a, b = (torch.randn(n, K // 2, generator=gen).bfloat16() for n in (M, N))
    places = torch.randperm(K, generator=gen)
    x, w = torch.cat([a, a], 1)[:, places].contiguous().cuda(), torch.cat([b, -b], 1)[:, places].contiguous().cuda()
    need = B.tr_linear_workspace_size(M, [N], K)
    slices = need // (4 * M * N)
    assert slices > 1

    def rms(split):
        y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.tr_set_tuning("lin_split", split)
        try:
            scratch = B.workspace(need)
            scratch.fill_(0x5A)
            B.tr_linear(x, [w], [y], scratch)
            torch.cuda.synchronize()
        finally:
            B.tr_set_tuning("lin_split", 0)
        assert bool((scratch == 0x5A).all()) == (split == 0)   # the slices leave partial sums there, a whole row of k none
        return float(y.double().square().mean().sqrt())

    e = rms(0), rms(slices)
    print("%d x %d x %d: rms error of the sums %.3e, in %d slices %.3e, ratio %.2f" % (M, N, K, e[0], slices, e[1], e[0] / e[1]))
    assert 0 < e[0] <= 1.02 * e[1]
