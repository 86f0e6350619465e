"""The grouping of (token, slot) entries by expert around the sizes where it changes form: one and
several entries per thread of the single workgroup (1024), the last count it takes (4096) and the
first of the three-pass form; many experts, and shared groups behind more than 64 routed ones. A
wrong grouping gives wrong rows to an expert, so the layer's output is compared with the oracle
(bounds as in test_gpu_layer). Routing tiles of 16 tokens with 17 to 256 experts ride along."""

import pytest

from paper_2609_34077_amd import _lib as L
from paper_2609_34077_amd import synth
from test_gpu_layer import check_layer

pytestmark = pytest.mark.gpu

# (T, E, K, shared): T K entries
CASES = [(512, 8, 2, 0), (171, 64, 6, 2), (256, 256, 16, 1), (257, 256, 16, 1), (1366, 17, 3, 0), (4096, 16, 1, 8),
         (5, 64, 6, 2), (16, 256, 16, 8)]


@pytest.mark.parametrize("T,E,K,ns", CASES)
def test_permutation_sizes(T, E, K, ns):
    check_layer(synth.LayerConfig(f"perm_t{T}_e{E}_k{K}", T=T, d=64, F=64, E=E, K=K, n_shared=ns,
                                  route_mode=L.ROUTE_SOFT_PRIOR, mask_set=tuple(range(0, E, 3)), seed=E + T))
