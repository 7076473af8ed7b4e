"""WordCount and its first-occurrence pass at the edges of the scan: texts
shorter than a 16-byte load, sizes around one 16-byte span for every lane of
the grid and its multiples, words that cross spans and chunks, an arena too
small for the spill regions, and lookup tables at their loads' ends; exactly
the oracle's keys, counts and offsets."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu
LANES = 64 * 16  # of one block


def text_of(n: int, seed: int, longest: int) -> np.ndarray:
    """n bytes of words of 1..longest letters from a small vocabulary (and some
    long runs), separated by one to three whitespace bytes."""
    rng = np.random.default_rng(seed)
    words = [bytes(rng.integers(97, 123, rng.integers(1, longest + 1), dtype=np.uint8))
             for _ in range(3000)]
    pick = rng.zipf(1.3, n // 2 + 8) % len(words)
    seps = [b" ", b"\n", b" \t ", b"\r\n"]
    out, size = [], 0
    for i, k in enumerate(pick):
        w = words[k] * (40 if i % 997 == 5 else 1)
        out.append(w + seps[i % 4])
        size += len(out[-1])
        if size >= n:
            break
    return np.frombuffer(b"".join(out)[:n], dtype=np.uint8).copy()


def check(ctx, text: np.ndarray, offset: int = 0, cap=None):
    buf = torch.zeros(text.size + offset, dtype=torch.uint8, device="cuda")  # ends with the text
    buf[offset:].copy_(torch.from_numpy(text))
    ok, oc, on = oracle.wordcount(text)
    keys, counts, nd, nw = ctx.wordcount(buf[offset:], cap or len(ok) + 3)
    k = keys[:nd].cpu().numpy().view(np.uint64)
    order = np.argsort(k)
    assert nw == on and np.array_equal(k[order], ok)
    assert np.array_equal(counts[:nd].cpu().numpy().view(np.uint64)[order], oc)
    if nd:
        off = ctx.wordcount_locate(buf[offset:], keys, nd).cpu().numpy()[:nd].view(np.uint64)
        assert np.array_equal(off, oracle.wordcount_first(text, k))


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=1 << 30)
    yield c
    c.destroy()


@pytest.mark.parametrize("n", list(range(1, 18)) + [31, 32, 33, 1023, 1024, 1025, 1041])
def test_small(ctx, n):
    rng = np.random.default_rng(n)
    check(ctx, rng.choice(np.frombuffer(b"ab \n", dtype=np.uint8), n))
    check(ctx, np.full(n, ord("x"), dtype=np.uint8), offset=3)


@pytest.mark.parametrize("extra", [-1, 0, 1, 15, 16, 17])
@pytest.mark.parametrize("per", [16, 48, 256])
def test_span_edges(ctx, per, extra):
    # `per` bytes for every lane of one block per CU, and a few more or less
    n = per * LANES * torch.cuda.get_device_properties(0).multi_processor_count + extra
    check(ctx, text_of(n, per + extra, 12), offset=per % 5)


@pytest.mark.parametrize("longest", [1, 40, 300])
def test_word_lengths(ctx, longest):
    check(ctx, text_of(3_000_017, longest, longest), offset=1)


def test_without_spill_regions():
    text = text_of(1 << 21, 5, 9)
    with sc.Context(device=0, arena_bytes=16 << 20) as small:
        check(small, text, offset=2)


@pytest.mark.parametrize("n", [1, 511, 512, 513, 30000])
def test_lookup_table_sizes(ctx, n):
    # n keys, wanted or not in the text, at loads of 1/3 to 2/3; the key 0 last
    text = text_of(1 << 20, n, 8)
    rng = np.random.default_rng(n)
    ok, _, _ = oracle.wordcount(text)
    other = rng.integers(1, 1 << 63, n, dtype=np.uint64)
    keys = np.unique(np.concatenate([ok[rng.permutation(ok.size)[:(n + 1) // 2]], other]))
    keys = np.append(rng.permutation(keys[keys != 0])[:n - 1], np.uint64(0))
    dev = torch.from_numpy(keys.view(np.int64)).cuda()
    off = ctx.wordcount_locate(torch.from_numpy(text).cuda(), dev, n)
    assert np.array_equal(off.cpu().numpy()[:n].view(np.uint64),
                          oracle.wordcount_first(text, keys))
