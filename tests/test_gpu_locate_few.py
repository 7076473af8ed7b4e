"""First occurrences of few keys (a bit per hash value drops the other words, the
last scan block writes the results) and of one more than few, against the
oracle: wanted keys at both ends of texts of one to many blocks, keys that no
word has, the key 0, and a repeated key."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu

FEW = 512


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=1 << 30)
    yield c
    c.destroy()


def text_of(n, seed):
    rng = np.random.default_rng(seed)
    text = rng.integers(97, 123, n).astype(np.uint8)
    text[rng.random(n) < 0.2] = 32
    return text


@pytest.mark.parametrize("n", [5, 16, 4096, 70001, 3_000_017])
@pytest.mark.parametrize("nkeys", [1, 10, FEW - 1, FEW, FEW + 1])
def test_few(ctx, n, nkeys):
    text = text_of(n, n + nkeys)
    rng = np.random.default_rng(nkeys)
    found, _, _ = oracle.wordcount(text)
    rare = found[np.argsort(oracle.wordcount_first(text, found))[-nkeys // 2:]]
    keys = np.unique(np.concatenate([rare, rng.integers(1, 1 << 63, nkeys, dtype=np.uint64)]))
    keys = rng.permutation(np.append(keys[keys != 0][:nkeys - 1], np.uint64(0)))
    dev = torch.from_numpy(keys.view(np.int64)).cuda()
    want = oracle.wordcount_first(text, keys)
    t = torch.from_numpy(text).cuda()
    for _ in range(3):
        off = torch.full((keys.size + 2,), 77, dtype=torch.int64, device="cuda")
        ctx.wordcount_locate(t, dev, keys.size, offsets=off)
        got = off.cpu().numpy().view(np.uint64)
        assert np.array_equal(got[:-2], want) and np.all(got[-2:] == 77)
    # the text that a call passes is the one it reads
    t[:n // 2] = 32
    text[:n // 2] = 32
    off = ctx.wordcount_locate(t, dev, keys.size)
    assert np.array_equal(off.cpu().numpy().view(np.uint64)[:keys.size],
                          oracle.wordcount_first(text, keys))


def test_empty_text_and_repeated_key(ctx):
    keys = torch.tensor([5, 9, 0], dtype=torch.int64, device="cuda")
    text = torch.zeros(0, dtype=torch.uint8, device="cuda")
    assert ctx.wordcount_locate(text, keys).cpu().tolist() == [-1, -1, -1]
    keys[2] = 5
    with pytest.raises(sc.SparkclError) as e:
        ctx.wordcount_locate(torch.full((100,), 97, dtype=torch.uint8, device="cuda"), keys)
    assert e.value.code == sc.EINVAL
