"""Code lengths and canonical codes of alphabets at the edges of the code book kernel: the sort's sizes (one and two
keys per thread), the 64 lightest items a merge round looks at, ties of leaves with nodes, and the largest total of
frequencies its 32-bit keys take (2^31 - 2).  Bit-exact against the CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _hist(kind, m, rng):
    if kind == "flat":
        return np.full(m, 7, np.uint64)
    if kind == "doubling":                                # a node weighs what the next leaf weighs, over and over
        return np.minimum(2 ** (np.arange(m) % 24), 2 ** 20).astype(np.uint64)
    if kind == "steps":                                   # many equal leaves beside equal nodes
        return (1 + np.arange(m) // 37).astype(np.uint64)
    if kind == "geometric":
        return np.maximum(1, (1e6 * 0.93 ** np.abs(np.arange(m) - m // 2)).astype(np.uint64))
    return rng.integers(1, 2 ** 14, m).astype(np.uint64)


@pytest.mark.parametrize("m", [1, 2, 3, 62, 63, 64, 65, 66, 128, 129, 512, 513, 1023, 1024, 1025, 1500, 2047, 2048])
@pytest.mark.parametrize("nbins", [2048, 4096, 65536])
def test_edges(oracle, m, nbins):
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(m * 7 + nbins)
    ctx = comet.Context(max_elems=4096, max_nbins=65536)
    lens = torch.empty(nbins, dtype=torch.uint8, device="cuda")
    codes = torch.empty(nbins, dtype=torch.int64, device="cuda")
    for kind in ("flat", "doubling", "steps", "geometric", "random"):
        w = _hist(kind, m, rng)
        totals = [None]
        if kind == "random":
            totals += [2 ** 31 - 2, 2 ** 31 - 1]          # the last total of 32-bit keys, the first of 64-bit ones
        for total in totals:
            f = w.copy()
            if total is not None:
                f[int(np.argmax(f))] += total - int(f.sum())
            h = np.zeros(nbins, np.uint32)
            h[np.sort(rng.choice(nbins, m, replace=False))] = f
            want = oracle.code_lengths(h)
            ctx.comet_stage_codebook(torch.from_numpy(h.view(np.int32)).cuda(), nbins, lens, codes)
            ctx.comet_sync()
            assert np.array_equal(lens.cpu().numpy(), want), (kind, total)
            assert np.array_equal(codes.cpu().numpy().view(np.uint64), oracle.canonical_codes(want)), (kind, total)
    ctx.close()


@pytest.mark.parametrize("nbins,m", [(4096, 2049), (8192, 8192), (8194, 2048), (8194, 2049), (8194, 8194), (9001, 2500), (16384, 16383),
                                     (32768, 5000), (65535, 65535), (65536, 2049), (65536, 4097), (65536, 30000), (65536, 65536)])
def test_more_symbols_than_lds(oracle, nbins, m):
    """Trees in global memory: finished by one workgroup (up to 8192 bins) or by whole grids (more)."""
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(m * 7 + nbins)
    ctx = comet.Context(max_elems=4096, max_nbins=65536)
    lens = torch.empty(nbins, dtype=torch.uint8, device="cuda")
    codes = torch.empty(nbins, dtype=torch.int64, device="cuda")
    for kind in ("flat", "doubling", "steps", "geometric", "random", "largest 32-bit total", "64-bit total"):
        f = _hist("random" if "total" in kind else kind, m, rng)
        if "total" in kind:                               # (the limit of 32-bit weights)
            f[int(np.argmax(f))] += 2 ** 31 - (2 if "largest" in kind else 1) - int(f.sum())
        h = np.zeros(nbins, np.uint32)
        h[np.sort(rng.choice(nbins, m, replace=False))] = f
        want = oracle.code_lengths(h)
        lens.fill_(77)
        codes.fill_(77)
        ctx.comet_stage_codebook(torch.from_numpy(h.view(np.int32)).cuda(), nbins, lens, codes)
        ctx.comet_sync()
        assert np.array_equal(lens.cpu().numpy(), want), kind
        assert np.array_equal(codes.cpu().numpy().view(np.uint64), oracle.canonical_codes(want)), kind
    ctx.close()


@pytest.mark.parametrize("nbins", [4096, 8192])
def test_more_symbols_than_lds_beside_other_work(oracle, nbins):
    """The same by one workgroup, over and over, with its wavefronts slowed down unevenly by kernels on another stream: the
    number of symbols is taken from words of LDS that the construction uses again."""
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(nbins)
    ctx = comet.Context(max_elems=4096, max_nbins=65536)
    side = torch.cuda.Stream()
    busy = torch.randn(1 << 24, device="cuda")
    cases = []
    for m in (2048, 2049, 3000, nbins):
        h = np.zeros(nbins, np.uint32)
        h[np.sort(rng.choice(nbins, m, replace=False))] = rng.integers(1, 1 << 14, m)
        cases.append((torch.from_numpy(h.view(np.int32)).cuda(), torch.from_numpy(oracle.code_lengths(h)).cuda()))
    torch.cuda.synchronize()
    outs = []
    for i in range(40):
        with torch.cuda.stream(side):
            busy.mul_(1.0)
        lens = torch.empty(nbins, dtype=torch.uint8, device="cuda")
        ctx.comet_stage_codebook(cases[i % 4][0], nbins, lens)
        outs.append(lens)
    ctx.comet_sync()
    assert all(torch.equal(lens, cases[i % 4][1]) for i, lens in enumerate(outs))
    ctx.close()
