"""Decoding of alphabets beyond the compact table (more than 4096 bins) through the table of code lengths: codes on both
sides of its 13 bits, of two codes in 32 bits and of its longest unmarked length, up to the longest a container holds (whose
strips do not fit LDS); numbers of symbols on both sides of the residuals kept in LDS; one symbol; escapes; every chunk size
and decoder, containers of version 2.  Bit-exact against the CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _table(kind, nbins, rng):
    """Code lengths by symbol and the symbols to draw from."""
    lens = np.zeros(nbins, np.uint8)
    half = nbins // 2
    if kind.startswith("deep"):
        k = int(kind[4:])
        syms = np.concatenate([half + np.arange(k) - k // 2, [0]])          # (the escape symbol has the longest code)
        lens[syms] = np.concatenate([np.arange(1, k + 1), [k]])
    else:
        m = int(kind[4:])                                                   # a complete code of m symbols, two lengths apart at most
        syms = np.concatenate([[0], rng.choice(np.arange(1, nbins), m - 1, replace=False)])
        k = int(np.log2(m))
        long2 = 2 * (m - (1 << k))
        lens[syms] = np.concatenate([np.full(long2, k + 1), np.full(m - long2, k)])
    return lens, syms


@pytest.mark.parametrize("nbins", [4098, 8192])
@pytest.mark.parametrize("kind", ["deep13", "deep14", "deep17", "deep32", "deep33", "deep57", "many2", "many2047", "many2048", "many2049", "many4000"])
def test_given_lengths(oracle, nbins, kind):
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(nbins + sum(map(ord, kind)))
    lens, syms = _table(kind, nbins, rng)
    eb, half, shape = 1e-2, nbins // 2, (2, 9, 31, 64)
    n = int(np.prod(shape))
    for weights in ("even", "short"):
        p = None if weights == "even" else 2.0 ** -np.minimum(lens[syms].astype(float), 40)
        draw = rng.choice(syms, n, p=None if p is None else p / p.sum())
        res = np.where(draw == 0, half + 5, draw.astype(np.int64) - half).reshape(shape)
        q = np.cumsum(np.cumsum(res, axis=2), axis=3)
        x = (np.where(np.abs(q) < 2 ** 22, q, 0) * np.float64(2 * np.float32(eb))).astype(np.float32)
        ctx = comet.Context(n, nbins)
        out = torch.empty(shape, device="cuda")
        for chunk in (64, 128, 256):
            box = oracle.compress_with_lengths(x, eb, nbins, chunk, lens)
            want = oracle.decompress(box)
            dev = torch.from_numpy(box).cuda()
            for hint in (64, 128):                        # both decoders
                ctx.comet_set_chunk_syms(hint)
                out.zero_()
                ctx.comet_decompress(dev, box.size, shape, out)
                ctx.comet_sync()
                assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32)), (weights, chunk, hint)
        ctx.close()


@pytest.mark.parametrize("w,kind", [(w, k) for w in (7, 16, 28, 56, 113, 224, 257, 512, 600) for k in (0, 1, 2) if k == 0 or w <= 512])
def test_zero_chunks_and_types(oracle, w, kind):
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(w)
    shape, eb, nbins = (2, 5, 40, w), 1e-3, 65536
    n = int(np.prod(shape))
    x = np.maximum(rng.standard_normal(shape), 0.0).astype(np.float32)
    x[0, 1:3] = 0.0                                       # whole strips and single chunks without words
    x[1, :, 10:20] = 0.0
    x[1, 4, 30, w // 2] = 3e5                             # an escape; the row behind it as well
    ctx = comet.Context(n, nbins)
    ctx.comet_set_zero_chunks(True)
    dt = [torch.float32, torch.float16, torch.bfloat16][kind]
    t = torch.from_numpy(np.minimum(x, 6e4)).cuda().to(dt)
    box = torch.zeros(comet.comet_compress_bound(shape, nbins, 64), dtype=torch.uint8, device="cuda")
    used = ctx.comet_compress(t, eb, nbins, box) if kind == 0 else ctx.comet_compress_16(t, eb, nbins, box)
    host = box[:used].cpu().numpy()
    out = torch.empty_like(t)
    for hint in (64, 256):
        ctx.comet_set_chunk_syms(hint)
        out.zero_()
        (ctx.comet_decompress if kind == 0 else ctx.comet_decompress_16)(box, used, shape, out)
        ctx.comet_sync()
        if kind == 0:
            assert np.array_equal(out.cpu().numpy().view(np.uint32), oracle.decompress(host).view(np.uint32)), hint
        else:
            assert np.array_equal(out.cpu().view(torch.int16).numpy().view(np.uint16), oracle.decompress_16(host, kind).reshape(shape)), hint
    ctx.close()
