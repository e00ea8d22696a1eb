"""Optional splits must not make the library ask for more than its static scratch array holds where
the low-rank intermediate alone fits it (CPU only: size queries)."""
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
