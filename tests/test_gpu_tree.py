"""Trees of large alphabets whose leaves' weights fit the LDS of the code book kernel: on both sides of the number that fits, of
the items a round takes (8192) and of the nodes a pass of its threads makes (1024); rounds that take leaves alone, nodes
alone and both.  Bit-exact against the CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _weights(kind, m, rng):
    if kind == "ones":                                    # rounds of as many leaves, then nodes, as they may take; one odd one left over
        return np.ones(m, np.uint64)
    if kind == "two levels":                              # a second crop of leaves that weighs what the first one's nodes weigh
        return np.where(np.arange(m) < m // 2, 1, 2).astype(np.uint64)
    if kind == "late":                                    # light leaves, and as many that only come when their tree is almost done
        return np.where(np.arange(m) < m // 2, 1, 9000).astype(np.uint64)
    return np.maximum(1, 3e7 / (1.0 + np.arange(m)) ** 1.2).astype(np.uint64)      # a long tail


@pytest.mark.parametrize("m", [2049, 4097, 8191, 8192, 8193, 8194, 16383, 16385, 24577, 40699, 40700, 40701])
@pytest.mark.parametrize("kind", ["ones", "two levels", "late", "tail"])
def test_trees(oracle, m, kind):
    from paper_2111_09562_amd import comet
    nbins = 65536 if m > 16384 else 16386
    rng = np.random.default_rng(m)
    h = np.zeros(nbins, np.uint32)
    h[rng.permutation(nbins)[:m]] = _weights(kind, m, rng)
    want = oracle.code_lengths(h)
    ctx = comet.Context(max_elems=4096, max_nbins=65536)
    lens = torch.full((nbins,), 77, dtype=torch.uint8, device="cuda")
    codes = torch.full((nbins,), 77, dtype=torch.int64, device="cuda")
    ctx.comet_stage_codebook(torch.from_numpy(h.view(np.int32)).cuda(), nbins, lens, codes)
    ctx.comet_sync()
    assert np.array_equal(lens.cpu().numpy(), want)
    assert np.array_equal(codes.cpu().numpy().view(np.uint64), oracle.canonical_codes(want))
    ctx.close()
