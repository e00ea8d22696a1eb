"""Optional splits must not make the library ask for more than its static scratch array holds where
the low-rank intermediate alone fits it, nor for more on a small batch than on a large one (CPU only:
size queries)."""
import random

import pytest

from tests.test_host_abi import _problem, mb  # noqa: F401  (mb is a fixture)


@pytest.mark.parametrize("seed", range(40))
def test_splits_stay_within_the_static_scratch(mb, seed):  # noqa: F811
    rng = random.Random(seed)
    K = rng.randint(1, 64)
    dtype = rng.choice([mb.MLORA_BF16, mb.MLORA_F32])
    align = rng.choice([1, 8, 64])
    h, d = (max(align, int(2 ** rng.uniform(0, 14)) // align * align) for _ in range(2))
    T = max(K, int(2 ** rng.uniform(3, 16)))
    cuts = sorted(rng.randint(0, T) for _ in range(K - 1))
    ranks = tuple(rng.randint(1, 128) for _ in range(K))
    if all(r % 8 == 0 for r in ranks):
        ranks = (ranks[0] - 1 or 1,) + ranks[1:]
    p = _problem(mb, T=T, h=h, d=d, off=tuple([0] + cuts + [T]), ranks=ranks, s=(1.0,) * K)
    p.c.dtype = dtype
    assert p.validate() == 0
    z, ws = p.saved_bytes(), p.workspace_bytes()
    if z <= mb.MLORA_STATIC_SCRATCH_BYTES:
        assert z <= ws <= mb.MLORA_STATIC_SCRATCH_BYTES, (T, h, d, ranks)
    assert p.recompute_workspace_bytes() == ws + z


def _reserve(p, tokens, ranks, h, d):
    """Sums of one gradient, two blocks per CU: what aligned shapes with whole-chunk ranks ask for at least."""
    most = 0
    for wide in (h, d):
        blocks = len(ranks) * -(-wide // 128)
        s = min(-(-512 // blocks), 16, max(tokens) // 256)
        if blocks < 384 and s > 1:
            most = max(most, -(-s * sum(ranks) * wide * 4 // 256) * 256)
    return most


@pytest.mark.parametrize("seed", range(40))
def test_whole_chunk_ranks_and_the_static_scratch(mb, seed):  # noqa: F811
    """Aligned bf16 shapes with ranks that are multiples of 8: what fits the static scratch with the
    reserved sums still fits with everything, what does not is still refused."""
    rng = random.Random(100 + seed)
    K = rng.randint(1, 16)
    h, d = (64 * int(2 ** rng.uniform(0, 8)) for _ in range(2))
    tokens = [int(2 ** rng.uniform(0, 13)) for _ in range(K)]
    ranks = tuple(8 * rng.randint(1, 16) for _ in range(K))
    off = [sum(tokens[:k]) for k in range(K + 1)]
    p = _problem(mb, T=off[-1], h=h, d=d, off=tuple(off), ranks=ranks, s=(1.0,) * K)
    z, ws = p.saved_bytes(), p.workspace_bytes()
    need = z + _reserve(p, tokens, ranks, h, d)
    assert need <= ws <= need + (64 << 20)
    assert (ws <= mb.MLORA_STATIC_SCRATCH_BYTES) == (need <= mb.MLORA_STATIC_SCRATCH_BYTES)


def _queries(mb, T, shares, h, ds, ranks, dtype):  # noqa: F811
    """Every size query of a batch of T tokens, `shares` of them per task."""
    off = [0]
    for n in shares:
        off.append(off[-1] + T * n // sum(shares))
    ps = [_problem(mb, T=T, h=h, d=d, off=tuple(off), ranks=ranks, s=(1.0,) * len(ranks)) for d in ds]
    for p in ps:
        p.c.dtype = dtype
        assert p.validate() == 0
    return [f() for p in ps for f in (p.workspace_bytes, p.recompute_workspace_bytes, p.w8_workspace_bytes)] + [
        mb.Group(ps).workspace_bytes()]


@pytest.mark.parametrize("case", [
    # h, [d], ranks, shares of the tokens
    (5120, [5120, 5120, 5120], (64,) * 16, (1,) * 16),
    (4096, [4096], (16,) * 4, (1,) * 4),
    (13824, [5120], (8, 16, 32, 64), (5, 1, 0, 2)),
    (4096, [1024, 1024], (128, 100), (3, 1)),
    (1000, [1500], (8, 10, 16), (2, 1, 1)),
])
def test_workspace_for_the_largest_batch_serves_the_smaller_ones(mb, case):  # noqa: F811
    h, ds, ranks, shares = case
    for dtype in (mb.MLORA_BF16, mb.MLORA_F32):
        last = None
        for T in [sum(shares) * n for n in (1, 2, 4, 7, 16, 33, 64, 128, 250, 512, 1000, 1024, 2048, 4096, 8192, 20000)]:
            now = _queries(mb, T, shares, h, ds, ranks, dtype)
            assert last is None or all(a <= b for a, b in zip(last, now)), (T, last, now)
            last = now


@pytest.mark.parametrize("seed", range(30))
def test_workspace_never_falls_with_the_batch(mb, seed):  # noqa: F811
    rng = random.Random(200 + seed)
    K = rng.randint(1, 12)
    align = rng.choice([1, 8, 64, 64])
    h, *ds = (max(align, int(2 ** rng.uniform(0, 13.5)) // align * align) for _ in range(rng.randint(2, 4)))
    ranks = tuple(rng.choice([8, 16, 32, 64, 128]) if seed % 2 else rng.randint(1, 128) for _ in range(K))
    shares = tuple(rng.randint(0, 5) for _ in range(K - 1)) + (1,)
    dtype = rng.choice([mb.MLORA_BF16, mb.MLORA_F32])
    batches = sorted({int(2 ** rng.uniform(0, 15)) for _ in range(25)})
    sizes = [_queries(mb, sum(shares) * n, shares, h, ds, ranks, dtype) for n in batches]
    for n, a, b in zip(batches[1:], sizes, sizes[1:]):
        assert all(x <= y for x, y in zip(a, b)), (sum(shares) * n, a, b)
