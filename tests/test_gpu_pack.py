"""The pack kernel of large alphabets on large tensors (entries of 32 bits in LDS): code words too long for those, symbols at the edges
of the cached range and outside it, the escape symbol, every symbol inside.  Bit-exact against the CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 64 * 512 * 1536 + 64 * 4 + 37                         # segments of just over 512 chunks on 256 compute units, the last chunk short


@pytest.mark.parametrize("nbins", [8194, 65536])
def test_codes_of_every_length(oracle, nbins):
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(nbins)
    lo = (nbins - 8192) // 2
    edge = np.array([0, 1, lo - 1, lo, lo + 8191, lo + 8192, nbins - 1]) % nbins
    syms = np.unique(np.concatenate([edge, rng.choice(nbins, 60, replace=False)]))
    rng.shuffle(syms)
    w = 0.6 ** np.arange(syms.size)                       # lengths 1, 2, 3, ... for as long as the counts last
    codes = syms[np.searchsorted(np.cumsum(w / w.sum()), rng.random(N), side="right").clip(0, syms.size - 1)].astype(np.uint16)
    at = rng.choice(N, 40 * syms.size, replace=False)     # every symbol occurs
    codes[at] = np.tile(syms, 40).astype(np.uint16)
    hist = oracle.histogram(codes, nbins).astype(np.uint64)
    fib = [1, 1]
    while len(fib) < 44:
        fib.append(fib[-1] + fib[-2])
    deep = np.zeros(nbins, np.uint32)                     # a code book of its own: a chain of lengths up to 43
    deep[syms[:44]] = np.array(fib, np.uint32)[::-1]
    deep[syms[44:]] = 1 << 20
    for h in (hist.astype(np.uint32), deep):
        ln = oracle.code_lengths(h)
        assert h is not deep or ln.max() > 31
        want_off, want_payload = oracle.encode(codes, nbins, 64, ln, oracle.canonical_codes(ln))
        lens = torch.empty(nbins, dtype=torch.uint8, device="cuda")
        off = torch.empty((N + 63) // 64, dtype=torch.int32, device="cuda")
        payload = torch.zeros(want_payload.size + 16, dtype=torch.int32, device="cuda")
        pw = torch.zeros(1, dtype=torch.int64, device="cuda")
        big = comet.Context(N, 65536)
        big.comet_stage_codebook(torch.from_numpy(h.view(np.int32)).cuda(), nbins, lens)
        big.comet_stage_encode(torch.from_numpy(codes.view(np.int16)).cuda(), N, nbins, 64, off, payload, pw)
        big.comet_sync()
        assert int(pw.item()) == want_payload.size
        assert np.array_equal(off.cpu().numpy().view(np.uint32), want_off)
        assert np.array_equal(payload.cpu().numpy().view(np.uint32)[:want_payload.size], want_payload)
        big.close()


@pytest.mark.parametrize("chunk", [64, 128, 256])
@pytest.mark.parametrize("zero_chunks", [False, True])
def test_chunk_sizes(oracle, chunk, zero_chunks):
    """Just over 512 chunks of every size per segment, a short chunk at the end; stretches of nothing but the centre code, which
    take no words in a container of version 2.  Code words start at a word, so a tensor that repeats a block of whole
    chunks has the block's words again and again."""
    from paper_2111_09562_amd import comet
    nbins, n = 16384, chunk * 512 * 1536 + 4 * chunk + 37
    rng = np.random.default_rng(chunk)
    block = np.clip(nbins // 2 + np.rint(rng.standard_normal(chunk * 1357) * 2500), 1, nbins - 1).astype(np.uint16)
    block[chunk * 100:chunk * 400] = nbins // 2
    block[chunk * 500 - 3:chunk * 500 + chunk + 5] = nbins // 2
    assert block.min() < (nbins - 8192) // 2                  # (symbols on both sides of the cached range, and in it)
    times, rest = divmod(n, block.size)
    tail = block[:rest]
    hist = oracle.histogram(block, nbins) * np.uint32(times) + oracle.histogram(tail, nbins)
    ln = oracle.code_lengths(hist)
    words = oracle.canonical_codes(ln)
    b_off, b_words = oracle.encode(block, nbins, chunk, ln, words, zero_chunks=zero_chunks)
    t_off, t_words = oracle.encode(tail, nbins, chunk, ln, words, zero_chunks=zero_chunks)
    ctx = comet.Context(n, nbins)
    ctx.comet_set_zero_chunks(zero_chunks)
    lens = torch.empty(nbins, dtype=torch.uint8, device="cuda")
    off = torch.empty((n + chunk - 1) // chunk, dtype=torch.int32, device="cuda")
    total = times * b_words.size + t_words.size
    payload = torch.zeros(total + 16, dtype=torch.int32, device="cuda")
    pw = torch.zeros(1, dtype=torch.int64, device="cuda")
    codes = torch.from_numpy(block.view(np.int16)).cuda().repeat(times + 1)[:n].contiguous()
    ctx.comet_stage_codebook(torch.from_numpy(hist.astype(np.uint32).view(np.int32)).cuda(), nbins, lens)
    ctx.comet_stage_encode(codes, n, nbins, chunk, off, payload, pw)
    ctx.comet_sync()
    assert np.array_equal(lens.cpu().numpy(), ln)
    assert int(pw.item()) == total
    got = payload.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:times * b_words.size].reshape(times, -1), np.broadcast_to(b_words, (times, b_words.size)))
    assert np.array_equal(got[times * b_words.size:total], t_words)
    assert not got[total:].any()
    got = off.cpu().numpy().view(np.uint32)
    steps = np.arange(times, dtype=np.uint64)[:, None] * b_words.size
    assert np.array_equal(got[:times * 1357].reshape(times, -1), (steps + b_off).astype(np.uint32))
    assert np.array_equal(got[times * 1357:], t_off + np.uint32(times * b_words.size))
    ctx.close()


@pytest.mark.parametrize("scale,lo,hi", [(0.2, 0, 1024), (1.9, 1024, 4096), (8.0, 4096, 32768)])
def test_symbols_inside_and_outside_the_range(oracle, scale, lo, hi):
    """Residuals within 1024 (the middle 2048 entries), within 4096 (the 8192 of the pack kernel) and beyond, with a few escapes."""
    from paper_2111_09562_amd import comet
    shape, eb, nbins = (3, 256, 257, 256), 1e-3, 65536
    rng = np.random.default_rng(1)
    x = (rng.random(shape, dtype=np.float32) * np.float32(scale))
    x[:, 1::2, :, :] *= np.float32(0.3)
    x.reshape(-1)[rng.choice(x.size, 500, replace=False)] = 1000.0
    want = oracle.compress(x, eb, nbins, 64)
    used = np.flatnonzero(oracle.parse_container(want)["len"])
    assert lo < np.abs(used[used > 0] - nbins // 2).max() < hi and used[0] == 0
    ctx = comet.Context(x.size, nbins)
    ctx.comet_set_chunk_syms(64)
    box = torch.zeros(want.size + (-want.size) % 16 + 4096, dtype=torch.uint8, device="cuda")
    assert ctx.comet_compress(torch.from_numpy(x).cuda(), eb, nbins, box) == want.size
    assert np.array_equal(box[:want.size].cpu().numpy(), want)
    ctx.close()


@pytest.mark.parametrize("nbins", [64, 1024, 16384])
@pytest.mark.parametrize("chunk", [64, 128])
def test_last_step_with_fewer_chunks(oracle, nbins, chunk):
    """A step is 256 symbols: the last one of a tensor may have chunks of them missing, which take no words.  The payload's own size is
    enough for it, and what lies behind a container stays as it was."""
    from paper_2111_09562_amd import comet
    rng = np.random.default_rng(nbins + chunk)
    ctx = comet.Context(1 << 16, nbins)
    ctx.comet_set_chunk_syms(chunk)
    for n in (chunk, 2 * chunk, 3 * chunk, 5 * chunk, 256 + chunk, 40 * 256 - chunk, 40 * 256 + chunk, 16 * 1024 - 2 * chunk, 3 * chunk - 5):
        x = rng.standard_normal((1, 1, 1, n) if n <= 512 else (1, 1, n // chunk, chunk)).astype(np.float32) if n % chunk == 0 else \
            rng.standard_normal((1, 1, 1, n)).astype(np.float32)
        x.reshape(-1)[:n:7] = 1e5                                 # (escapes: symbol 0 has a code word)
        want = oracle.compress(x, 1e-2, nbins, chunk)
        room = torch.full((want.size // 16 * 16 + 4096,), 77, dtype=torch.uint8, device="cuda")
        assert ctx.comet_compress(torch.from_numpy(x).cuda(), 1e-2, nbins, room) == want.size, n
        assert np.array_equal(room[:want.size].cpu().numpy(), want), n
        assert bool((room[want.size:] == 77).all()), n
        parts = oracle.parse_container(want)
        codes = oracle.decode(parts["len"], parts["chunk_off"], parts["payload"], x.size, chunk)
        hist = oracle.histogram(codes, nbins)
        lens = torch.empty(nbins, dtype=torch.uint8, device="cuda")
        off = torch.empty(parts["n_chunks"], dtype=torch.int32, device="cuda")
        payload = torch.full((parts["payload_words"] + 64,), 7, dtype=torch.int32, device="cuda")
        pw = torch.zeros(1, dtype=torch.int64, device="cuda")
        ctx.comet_stage_codebook(torch.from_numpy(hist.astype(np.uint32).view(np.int32)).cuda(), nbins, lens)
        ctx.comet_stage_encode(torch.from_numpy(codes.view(np.int16)).cuda(), x.size, nbins, chunk, off, payload[:parts["payload_words"]], pw)
        ctx.comet_sync()                                          # (no error: the payload fits)
        assert int(pw.item()) == parts["payload_words"]
        assert np.array_equal(payload.cpu().numpy().view(np.uint32)[:parts["payload_words"]], parts["payload"]), n
        assert bool((payload[parts["payload_words"]:] == 7).all()), n
    ctx.close()
