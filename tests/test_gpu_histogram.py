"""Histogram of alphabets larger than the quantise kernel's LDS window (k_code_hist): sizes that are no multiple of the
eight codes a thread loads, one and several workgroups, alphabets at the edges of its own window, bounds that spread the
codes over the innermost bins, the window and what lies outside it, and fields of one value.  Counts are exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nbins", [8192, 8194, 16384, 32766, 32768, 32770, 65536])
@pytest.mark.parametrize("shape", [(1, 1, 1, 5), (1, 3, 7, 19), (1, 64, 28, 28), (3, 17, 41, 53), (4, 16, 112, 113)])
def test_counts(oracle, nbins, shape):
    from paper_2111_09562_amd import comet
    n = int(np.prod(shape))
    rng = np.random.default_rng(nbins + n)
    ctx = comet.Context(max_elems=n, max_nbins=65536)
    codes = torch.empty(n, dtype=torch.int16, device="cuda")
    hist = torch.empty(nbins, dtype=torch.int32, device="cuda")
    rec = torch.empty(4 * n, dtype=torch.int32, device="cuda")
    counts = torch.empty(3, dtype=torch.int64, device="cuda")
    for spread in (0.0, 3.0, 400.0, 0.2 * nbins, 0.6 * nbins):     # standard deviation of the input, in units of twice the bound
        eb = 1e-3
        x = (rng.standard_normal(shape) * spread * 2 * eb).astype(np.float32)
        ctx.comet_stage_quantize(torch.from_numpy(x).cuda(), eb, nbins, codes, hist, rec, counts)
        ctx.comet_sync()
        got = codes.cpu().numpy().view(np.uint16)
        assert np.array_equal(hist.cpu().numpy().view(np.uint32), np.bincount(got, minlength=nbins)), spread
        out = torch.empty(comet.comet_compress_bound(shape, nbins, 64), dtype=torch.uint8, device="cuda")
        used = ctx.comet_compress(torch.from_numpy(x).cuda(), eb, nbins, out)
        assert np.array_equal(out[:used].cpu().numpy(), oracle.compress(x, eb, nbins, 64)), spread
    ctx.close()


@pytest.mark.parametrize("nbins", [8194, 40000, 65536])
@pytest.mark.parametrize("shape", [(64, 64, 128, 129), (2, 69400, 22, 22), (1, 8200, 91, 91), (17, 16, 512, 511), (21, 64, 224, 224), (1, 1, 131080, 512), (9, 4100, 43, 43)])
def test_counts_shared_by_two_kernels(nbins, shape):
    """From 2^26 elements on the quantise kernel counts a run's codes as long as few of them lie outside its window, and the
    second kernel counts the rest: fields that change from row to row, from plane to plane and once, between no code
    outside, a few, about one in 32 (where the line lies) and most of them, so that runs of both kinds and points inside
    a run meet in one slice of the second kernel, and widths that put both off the groups of eight codes it loads."""
    from paper_2111_09562_amd import comet
    n = int(np.prod(shape))
    assert n >= 1 << 26
    g = torch.Generator(device="cuda").manual_seed(nbins + n)
    ctx = comet.Context(max_elems=n, max_nbins=65536)
    codes = torch.empty(n, dtype=torch.int16, device="cuda")
    hist = torch.empty(nbins, dtype=torch.int32, device="cuda")
    rec = torch.empty(4 * n, dtype=torch.int32, device="cuda")
    counts = torch.empty(3, dtype=torch.int64, device="cuda")
    eb = 1e-3
    noise = torch.randn(shape, device="cuda", generator=g)

    def pick(values, where):
        return torch.tensor(values, device="cuda")[torch.randint(len(values), where, device="cuda", generator=g)]
    rows = shape[:3] + (1,)
    n_rows = shape[0] * shape[1] * shape[2]
    once = (torch.arange(n_rows, device="cuda") > 0.4 * n_rows).reshape(rows)
    spread = {"none": torch.full(rows, 5.0, device="cuda"),
              "rows": pick([1.0, 900.0, 1000.0, 2500.0, 9000.0], rows),
              "planes": pick([1.0, 900.0, 1000.0, 2500.0], shape[:2] + (1, 1)),
              "near the line": torch.full(rows, 950.0, device="cuda"),
              "once": torch.where(once, 9000.0, 5.0),
              "few": torch.where(torch.rand(rows, device="cuda", generator=g) < 0.02, 5000.0, 40.0),
              "escapes": torch.where(torch.rand(rows, device="cuda", generator=g) < 0.5, 2.0 * nbins, 40.0)}
    for kind, s in spread.items():
        ctx.comet_stage_quantize((noise * s * (2 * eb)).contiguous(), eb, nbins, codes, hist, rec, counts)
        ctx.comet_sync()
        want = torch.zeros(nbins, dtype=torch.int64, device="cuda")
        for part in codes.split(1 << 25):
            want += torch.bincount(part.to(torch.int64) & 0xffff, minlength=nbins)
        assert bool((hist.to(torch.int64) == want).all()), kind
    ctx.close()


@pytest.mark.parametrize("nbins,shape,want", [(1024, (2, 8, 56, 56), 1), (8192, (2, 8, 56, 56), 1), (8194, (2, 8, 56, 56), 2), (65536, (2, 8, 56, 56), 2), (65536, (1, 1, 8, 600), 1)])
def test_the_histogram_is_timed_with_the_quantiser(nbins, shape, want):
    """The per-kernel timers: an alphabet beyond the sweep's window has its histogram in a kernel of its own, which the
    quantiser's figure includes (planes of more than 512 columns have another sweep, which counts everything)."""
    from paper_2111_09562_amd import comet
    x = torch.randn(shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(nbins)).clamp_min_(0.0)
    ctx = comet.Context(x.numel(), nbins)
    ctx.comet_profile_enable(True)
    ctx.comet_profile_reset()
    box = torch.empty(comet.comet_compress_bound(shape, nbins, 64), dtype=torch.uint8, device="cuda")
    ctx.comet_compress(x, 1e-3, nbins, box)
    assert ctx.comet_profile_read(0)[0] == want
    assert ctx.comet_profile_read(0)[1] > 0.0
    ctx.close()


@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("shape", [(21, 64, 224, 224), (64, 64, 128, 129), (17, 4100, 31, 32)])
def test_16_bit_tensors_shared_by_two_kernels(kind, shape):
    """The same division for 16-bit inputs: the container is the one of the widened tensor, byte for byte."""
    from paper_2111_09562_amd import comet
    nbins, eb = 65536, 1e-3
    n = int(np.prod(shape))
    assert n >= 1 << 26
    g = torch.Generator(device="cuda").manual_seed(n + kind)
    spread = torch.tensor([1.0, 900.0, 1000.0, 9000.0], device="cuda")[torch.randint(4, shape[:3] + (1,), device="cuda", generator=g)]
    x = (torch.randn(shape, device="cuda", generator=g) * spread * (2 * eb)).to([torch.float16, torch.bfloat16][kind - 1])
    ctx = comet.Context(n, nbins)
    boxes = [torch.zeros(4 * n + (1 << 20), dtype=torch.uint8, device="cuda") for _ in range(2)]
    used = [ctx.comet_compress_16(x, eb, nbins, boxes[0]), ctx.comet_compress(x.float(), eb, nbins, boxes[1])]
    assert used[0] == used[1] and torch.equal(boxes[0], boxes[1])
    ctx.close()
