"""Decompression of planes that are cut into bands of rows and segments of columns (wide planes, and planes too few
for a plane per workgroup): bit-exact against the CPU oracle at the edges of bands (rows), segments (64 lanes of one or
two columns) and of the alphabet (escaped residuals within and beyond 16 bits, verbatim values)."""
import numpy as np
import pytest

from paper_2111_09562_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def comet():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_09562_amd import comet as libcomet
    libcomet.lib()
    return libcomet


def _in_bands(ctx, call):
    """Runs a decompression and asserts that it went through the Huffman decoder and the kernels of the bands."""
    ctx.comet_profile_enable(True)
    ctx.comet_profile_reset()
    call()
    ctx.comet_sync()
    assert tuple(ctx.comet_profile_read(k)[0] for k in (5, 4, 8)) == (1, 1, 0)
    ctx.comet_profile_enable(False)


SHAPES = [(1, 2, 8, 513), (1, 1, 9, 640), (2, 1, 17, 514), (1, 3, 64, 767), (1, 1, 65, 1025), (1, 1, 1, 8191), (1, 1, 2, 8192),
          (1, 1, 1100, 128), (1, 2, 300, 129), (1, 1, 130, 512), (3, 2, 131, 385)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("eb,nbins,chunk", [(1e-2, 1024, 64), (1e-3, 16, 64), (1e-4, 65536, 128), (1e-2, 4, 256), (1e-6, 4096, 77)])
def test_bands(comet, oracle, shape, eb, nbins, chunk):
    x = synth.relu_blur(shape, 7, blur=3, shift=-0.2)
    rng = np.random.default_rng(3)
    flat = x.reshape(-1)
    at = rng.choice(flat.size, max(1, flat.size // 97), replace=False)
    flat[at] = rng.choice(np.array([0.0, 3e2, -7e2, 2e4 * eb, -40000 * eb, np.inf, 1e30, 65535.9 * eb], np.float32), at.size)
    want = oracle.compress(x, eb, nbins, chunk)
    ref = oracle.decompress(want)
    ctx = comet.Context(max_elems=x.size, max_nbins=nbins)
    ctx.comet_set_chunk_syms(chunk if chunk in (64, 128, 256) else 64)
    box = torch.from_numpy(want).cuda()
    room = torch.full((x.size + 1,), 7.0, device="cuda")
    out = room[:x.size].view(shape)
    _in_bands(ctx, lambda: ctx.comet_decompress(box, want.size, shape, out))
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    assert float(room[-1]) == 7.0
    room.fill_(7.0)                                      # an output that is not aligned to a pair: one column per lane
    out = room[1:].view(shape)
    ctx.comet_decompress(box, want.size, shape, out)
    ctx.comet_sync()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    assert float(room[0]) == 7.0
    if shape[3] <= 512:
        for name, dt in (("float16", torch.float16), ("bfloat16", torch.bfloat16)):
            half = torch.empty(shape, dtype=dt, device="cuda")
            ctx.comet_decompress_16(box, want.size, shape, half)
            ctx.comet_sync()
            got, exp = half.cpu(), torch.from_numpy(ref).to(dt)
            same = (got.view(torch.int16) == exp.view(torch.int16)) | (torch.isnan(got) & torch.isnan(exp))
            assert bool(same.all()), name
    ctx.close()


# (shape, rows per band): bands grow from 8 rows at 4.7 million elements to 64 at 34 million
TALL = [((4, 5, 33, 8191), 9), ((1, 7, 500, 1999), 13), ((1, 16, 401, 1300), 15), ((2, 4, 1058, 1000), 16), ((1, 9, 1021, 1000), 17), ((1, 40, 500, 510), 19),
        ((2, 16, 480, 854), 24), ((1, 17, 1020, 1001), 33), ((2, 20, 129, 8191), 43), ((2, 17, 1001, 1001), 63), ((3, 11, 1023, 1000), 64)]


@pytest.mark.parametrize("shape,rows", TALL)
def test_tall_bands(comet, oracle, shape, rows):
    """Bands of 9 to 64 rows: the second half of the row loop and its refills, a lane per row beyond the eighth, last bands
    with fewer rows; one and two columns per lane; 16-bit outputs where the planes allow them."""
    n = int(np.prod(shape))
    r = min(64, max(8, n >> 19))
    bands = -(-shape[2] // r)
    assert -(-shape[2] // bands) == rows
    eb, nbins = 1e-3, 1024
    x = synth.relu_blur(shape, 7, blur=3, shift=-0.2)
    rng = np.random.default_rng(3)
    flat = x.reshape(-1)
    at = rng.choice(flat.size, flat.size // 997, replace=False)
    flat[at] = rng.choice(np.array([0.0, 3e2, -7e2, 2e4 * eb, -40000 * eb, np.inf, 1e30, 65535.9 * eb], np.float32), at.size)
    want = oracle.compress(x, eb, nbins, 64)
    ref = torch.from_numpy(oracle.decompress(want)).cuda().view(shape)
    ctx = comet.Context(max_elems=n, max_nbins=nbins)
    box = torch.from_numpy(want).cuda()
    room = torch.full((n + 1,), 7.0, device="cuda")
    for first in (0, 1):                                 # 1: an output that is not aligned to a pair: one column per lane
        room.fill_(7.0)
        out = room[first:first + n].view(shape)
        _in_bands(ctx, lambda: ctx.comet_decompress(box, want.size, shape, out))
        assert torch.equal(out.view(torch.int32), ref.view(torch.int32)), first
        assert float(room[n if first == 0 else 0]) == 7.0
    if shape[3] <= 512:
        for dt in (torch.float16, torch.bfloat16):
            half = torch.empty(shape, dtype=dt, device="cuda")
            _in_bands(ctx, lambda: ctx.comet_decompress_16(box, want.size, shape, half))
            exp = ref.to(dt)
            assert bool(((half.view(torch.int16) == exp.view(torch.int16)) | (torch.isnan(half) & torch.isnan(exp))).all()), dt
    ctx.close()
