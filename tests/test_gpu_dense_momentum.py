"""Dense momentum on both sides of the size from which u and g go past the caches: small whole numbers and rho = 1/2, whose
results are exact, against plain torch; lengths with a remainder, vectors that begin anywhere, several steps."""
import pytest
import torch

import paper_1903_04488_amd as cs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 12 W d bytes around 150 million
@pytest.mark.parametrize("W,d", [(1, 12_500_000), (1, 12_500_001), (3, 4_166_666), (3, 4_166_667), (8, 1_562_500), (8, 1_562_503), (2, 5)])
@pytest.mark.parametrize("skip", [0, 1])
def test_both_sides_of_the_cache(W, d, skip):
    gen = torch.Generator(device=DEV).manual_seed(d + W)
    u, v, g = ([torch.randint(-8, 9, (d + skip,), device=DEV, generator=gen).float()[skip:] for _ in range(W)] for _ in range(3))
    want_u, want_v = [x.clone() for x in u], [x.clone() for x in v]
    for _ in range(3):
        cs.cs_dense_momentum(u, v, g, 0.5)
        for w in range(W):
            want_u[w] = 0.5 * want_u[w] + g[w]
            want_v[w] += want_u[w]
    for w in range(W):
        assert torch.equal(u[w], want_u[w]) and torch.equal(v[w], want_v[w]), w
