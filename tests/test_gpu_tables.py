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


@pytest.mark.parametrize("nbins", [64, 4096, 65536])
def test_incomplete_codes_are_refused(oracle, nbins):
    """A length section that is no complete prefix code, behind a header that is right or wrong itself: the tables kernel
    decides twice, first on the header and then on the lengths, while its sixteen wavefronts run apart.  Refused every
    time, and the next call on the same context is not touched by it."""
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(nbins)
    x = np.maximum(rng.standard_normal((1, 4, 28, 28)), 0.0).astype(np.float32)
    good = oracle.compress(x, 1e-2, nbins, 64)
    want = oracle.decompress(good)
    lens = good[comet.HEADER_BYTES:comet.HEADER_BYTES + nbins]
    used = np.flatnonzero(lens)
    bad = {"incomplete": good.copy(), "oversubscribed": good.copy(), "no code at all": good.copy(), "too long": good.copy(), "header and code": good.copy()}
    section = {k: b[comet.HEADER_BYTES:comet.HEADER_BYTES + nbins] for k, b in bad.items()}
    section["incomplete"][used[-1]] += 1
    section["oversubscribed"][used[-1]] -= 1
    section["no code at all"][:] = 0
    section["too long"][used[-1]] = 58
    section["header and code"][used[0]] += 1
    bad["header and code"][0] ^= 1
    ctx = comet.Context(x.size, nbins)
    out = torch.empty(x.shape, device="cuda")
    dev = {k: torch.from_numpy(b).cuda() for k, b in bad.items()}
    fine = torch.from_numpy(good).cuda()
    for _ in range(3):
        for kind, box in dev.items():
            ctx.comet_decompress(box, good.size, x.shape, out)
            with pytest.raises(comet.CometError) as ei:
                ctx.comet_sync()
            assert ei.value.code == comet.ERR_FORMAT, kind
            out.zero_()
            ctx.comet_decompress(fine, good.size, x.shape, out)
            ctx.comet_sync()
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), kind
    ctx.close()
