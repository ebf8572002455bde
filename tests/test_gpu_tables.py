"""Decode tables: code lengths on both sides of the first level (12 bits, 11 for the general table), of the second
level's classes (13, 14, 16, 18 bits) and beyond both, one symbol, flat alphabets, and the alphabet sizes where the
compact table ends.  Every residual in turn, decompressed bit-exactly as the CPU oracle does."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _tensor(counts, values, eb, rng, w):
    """Planes of one row each, whose residuals are the given values the given number of times."""
    res = np.repeat(values, counts)
    rng.shuffle(res)
    res = np.concatenate([res, np.zeros((-res.size) % w, np.int64)]).reshape(-1, w)
    q = np.cumsum(res, axis=1)
    return (q * np.float64(2 * np.float32(eb))).astype(np.float32).reshape(1, -1, 1, w)


@pytest.mark.parametrize("nbins", [64, 4094, 4096, 4098, 16384])
@pytest.mark.parametrize("kind", ["one", "flat", "len12", "len13", "len14", "len16", "len18", "len20", "mixed"])
def test_tables(oracle, nbins, kind):
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(nbins)
    half = nbins // 2 - 1
    if kind == "one":
        values, counts = np.array([0]), np.array([1000])
    elif kind == "flat":
        m = min(nbins - 1, 1500)
        values, counts = np.arange(m) - m // 2, np.full(m, 3)
    elif kind == "mixed":
        m = min(nbins - 1, 700)
        values, counts = np.arange(m) - m // 2, np.maximum(1, (40000 * 0.97 ** np.abs(np.arange(m) - m // 2)).astype(np.int64))
    else:
        deepest = int(kind[3:])                           # counts 1, 1, 2, 4, ...: lengths 1 .. deepest
        counts = 2 ** np.maximum(np.arange(deepest + 1) - 1, 0)
        values = np.concatenate([np.arange(counts.size - 2) - 5, [half, -half]])[::-1]
    eb = 1e-2
    x = _tensor(counts, values, eb, rng, 64)
    box = oracle.compress(x, eb, nbins, 64)
    want = oracle.decompress(box)
    ctx = comet.Context(x.size, nbins)
    dev = torch.from_numpy(box).cuda()
    out = torch.empty(x.shape, device="cuda")
    for hint in (64, 128):                                # both decoders
        ctx.comet_set_chunk_syms(hint)
        out.zero_()
        ctx.comet_decompress(dev, box.size, x.shape, out)
        ctx.comet_sync()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), hint
    info = ctx.comet_peek(dev, box.size)
    if kind.startswith("len"):
        assert info.max_len == int(kind[3:]) or info.n_active != counts.size
    ctx.close()
