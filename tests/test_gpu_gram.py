"""hsp_gram at the edges of its tiles: 16-wide blocks, 64- and 128-wide tiles
(the switch between them lies at p = 128), rows short of a stage or a split,
rows that start off 16-byte boundaries, and padding that must not be read as
data (it holds NaN).  Against float64 sums of the same (rounded) design:
entries are sums of N exact products, so |error| <= N 2^-52 sum |x_ij x_ik|,
and sum |x_ij x_ik| <= sqrt(G_jj G_kk)."""
import numpy as np
import pytest

from gpu_util import need_gpu
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("xt", ["f32", "bf16"])
@pytest.mark.parametrize("N,p,ld", [(1, 1, 1), (33, 15, 16), (63, 16, 16), (65, 17, 19), (1000, 64, 64), (517, 65, 72),
                                    (2049, 128, 128), (2048, 129, 136), (999, 145, 145), (131, 255, 256),
                                    (3001, 257, 259), (4100, 400, 400), (20011, 300, 300), (9001, 352, 352),
                                    (9001, 383, 383)])
def test_gram_tile_edges(xt, N, p, ld):
    torch, hsp = need_gpu()
    X = np.random.default_rng(N + p).standard_normal((N, p)).astype(np.float32)
    if xt == "bf16":
        bits = synth.bf16_bits(X)
        X = synth.bf16_to_f32(bits)
        buf = np.full((N, ld), 0x7FC0, np.uint16)
        buf[:, :p] = bits
    else:
        buf = np.full((N, ld), np.nan, np.float32)
        buf[:, :p] = X
    d = torch.from_numpy(buf.ravel()[: (N - 1) * ld + p].copy()).cuda()  # the last row ends at p
    G = torch.full((p, p), np.nan, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    hsp.hsp_gram(d.data_ptr(), hsp.HSP_X_F32 if xt == "f32" else hsp.HSP_X_BF16, N, p, ld, G.data_ptr())
    ref = X.astype(np.float64).T @ X.astype(np.float64)
    got = G.cpu().numpy()
    s = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
    assert np.all(np.abs(got - ref) <= 2 * N * 2.0 ** -52 * s)
    assert np.array_equal(got, got.T)


@pytest.mark.parametrize("xt,N,p,rows", [("f32", 2049, 150, 64), ("bf16", 3000, 140, 192), ("f32", 3000, 60, 128)])
def test_gram_of_row_chunks(xt, N, p, rows):
    """Row splits that end inside a chunk of streamed rows, and go on from one
    chunk to the next: the resident design's G, bit for bit."""
    torch, hsp = need_gpu()
    rng = np.random.default_rng(p)
    X, y = rng.standard_normal((N, p)).astype(np.float32), (rng.random(N) < 0.5).astype(np.uint8)
    G = []
    for stream in (False, True):
        s = hsp.Sampler(X if stream else torch.from_numpy(X).cuda(), y if stream else torch.from_numpy(y).cuda(), seed=1,
                        x_type=xt, x_stream=stream, stream_rows=rows)
        G.append(s.gram())
        s.close()
    assert np.array_equal(G[0], G[1])


@pytest.mark.parametrize("N", [1, 1030])
def test_gram_of_very_many_columns(N):
    """More tiles than one launch of the sum can take (p > 46208; 64- and 128-wide
    ones): small whole numbers, so that every sum is exact."""
    torch, hsp = need_gpu()
    p = 46300
    x = torch.randint(-3, 4, (N, p), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda").float()
    G = torch.full((p, p), float("nan"), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    hsp.hsp_gram(x.data_ptr(), hsp.HSP_X_F32, N, p, p, G.data_ptr())
    d = x.double()
    for i in range(0, p, 4096):
        assert torch.equal(G[i:i + 4096], d[:, i:i + 4096].t().contiguous() @ d)
    del G
    torch.cuda.empty_cache()


@pytest.mark.parametrize("xt,N,p,rows", [("f32", 2500, 129, 64), ("bf16", 2500, 192, 320), ("f32", 3100, 193, 512),
                                         ("bf16", 2100, 257, 64), ("f32", 2400, 384, 128),  # quarters of tiles
                                         ("f32", 2200, 2900, 512), ("bf16", 2100, 2820, 1088)])  # whole ones
def test_gram_of_row_chunks_by_quarters_and_whole_tiles(xt, N, p, rows):
    """A chunk that few blocks have rows of is taken in 64-wide quarters of the
    128-wide tiles: the resident design's G, bit for bit."""
    test_gram_of_row_chunks(xt, N, p, rows)


@pytest.mark.parametrize("xt", ["f32", "bf16"])
@pytest.mark.parametrize("N,p,ld", [(2048, 130, 130), (2049, 130, 131), (2049, 145, 145), (2100, 255, 256), (2500, 383, 383),
                                    (1024, 1025, 1032), (1025, 1025, 1027), (3, 700, 700), (250, 200, 200), (257, 140, 144)])
def test_gram_of_short_designs(xt, N, p, ld):
    """Where 64-wide tiles take over from 128-wide ones (up to N = 1024, or 2048
    with p <= 1024), and where one thread sums an entry's splits (up to four)."""
    test_gram_tile_edges(xt, N, p, ld)
