"""The serving-batch expert kernels (more tokens than the few-token path takes, few rows per
expert) against the oracle, at the edges of their tiles and of the rule that picks them: row
groups of exactly one tile and one row more (64- and 128-row tiles; a shared expert's group
holds every token), the last batch a rule takes and the first it leaves, d and F that are no
multiple of a workgroup's 128 weight rows, one chunk of the reduction, and a split one. Bounds
as in test_gpu_layer."""

import pytest

from paper_2609_34077_amd import _lib as L
from paper_2609_34077_amd import synth
from test_gpu_layer import check_layer
from test_gpu_lora import check_lora

pytestmark = pytest.mark.gpu


def _cfg(T, E, K, ns, d, F, mode=L.ROUTE_PLAIN, keep=None):
    return synth.LayerConfig(f"batch_t{T}_e{E}_k{K}_s{ns}_d{d}_f{F}_m{mode}", T=T, d=d, F=F, E=E, K=K, n_shared=ns,
                             route_mode=mode, gate_mode=L.GATE_P if ns else L.GATE_RENORM, mask_set=keep, seed=T + d)


KEEP4 = (0, 2, 5, 7)
CASES = [
    _cfg(17, 8, 2, 0, 64, 64),                                        # the smallest batch; one chunk
    _cfg(64, 8, 2, 1, 192, 320),                                      # 64-row tiles: one tile exactly
    _cfg(65, 8, 2, 1, 256, 192),                                      # ... and one row more
    _cfg(120, 8, 2, 0, 128, 2048, L.ROUTE_SOFT_PRIOR, KEEP4),         # 64-row tiles, split reduction
    _cfg(121, 8, 2, 0, 128, 192, L.ROUTE_SOFT_PRIOR, KEEP4),
    _cfg(144, 8, 2, 0, 128, 192, L.ROUTE_SOFT_PRIOR, KEEP4),          # the last batch of 64-row tiles
    _cfg(145, 8, 2, 0, 128, 192, L.ROUTE_SOFT_PRIOR, KEEP4),          # 128-row tiles from here
    _cfg(128, 8, 2, 1, 320, 128),                                     # one tile exactly
    _cfg(129, 8, 2, 1, 128, 2048),                                    # one row more, split reduction
    _cfg(208, 8, 2, 0, 256, 256, L.ROUTE_HARD_MASK, KEEP4),           # the last batch, four experts
    _cfg(209, 8, 2, 0, 256, 256, L.ROUTE_HARD_MASK, KEEP4),           # the many-token path
    _cfg(906, 64, 6, 2, 128, 192, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set())),
    _cfg(800, 64, 6, 2, 128, 192, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set())),   # the last, many experts
    _cfg(801, 64, 6, 2, 128, 192, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set())),
    _cfg(597, 64, 6, 2, 128, 192, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set())),
    _cfg(40, 256, 16, 8, 192, 64),                                    # the most experts and shared experts
    # model widths (many chunks, several column tiles, a down reduction in slices): 64-row tiles, then the
    # first batch of 128-row ones
    _cfg(128, 8, 2, 0, 1152, 2048),
    _cfg(145, 8, 2, 1, 1152, 2048),
    _cfg(100, 16, 2, 0, 1088, 2112, L.ROUTE_SOFT_PRIOR, KEEP4),
    # twelve experts take every token: more row tiles than the batch path keeps, so that the many-token
    # path's tiles run beside it
    _cfg(333, 64, 6, 2, 256, 2048, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set())).with_(delta=25.0),
    _cfg(700, 64, 6, 2, 128, 320, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set())).with_(delta=25.0),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_batch_rows(cfg):
    check_layer(cfg)


@pytest.mark.parametrize("cfg", [c for c in CASES if c.d % 128 == 0], ids=lambda c: c.name)
def test_batch_packed(cfg):
    check_layer(cfg, packed=True)


# the adapters' chunk in front of the weight chunks: 64- and 128-row tiles, a split reduction (only
# its first slice takes the adapters), ragged weight rows, one token
@pytest.mark.parametrize("T,E,K,ns,d,F,rank", [(1, 8, 2, 1, 64, 64, 8), (17, 8, 2, 0, 128, 2048, 16), (129, 8, 2, 1, 192, 320, 4),
                                               (300, 64, 6, 2, 256, 192, 8), (100, 8, 2, 0, 1152, 2048, 8),
                                               (130, 8, 2, 1, 1088, 2048, 5)])
def test_batch_lora(T, E, K, ns, d, F, rank):
    check_lora(_cfg(T, E, K, ns, d, F), rank=rank)


def test_batch_lora_skewed():
    check_lora(_cfg(333, 64, 6, 2, 256, 2048, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set())).with_(delta=25.0), rank=8)


# The serving batches of both model shapes, on tokens of every row tile.
@pytest.mark.parametrize("T,E,K,ns,d,F,mode,keep,packed", [
    (96, 8, 2, 0, 4096, 14336, L.ROUTE_SOFT_PRIOR, KEEP4, True),
    (333, 64, 6, 2, 2048, 1408, L.ROUTE_SOFT_PRIOR, tuple(synth.deepseek_mask_set()), False),
])
def test_batch_model_shapes(T, E, K, ns, d, F, mode, keep, packed):
    check_layer(_cfg(T, E, K, ns, d, F, mode, keep), sample=True, packed=packed)


# the many-token path's last tile of a group: 64, 128, 192 or 256 rows multiplied. Two experts take
# every token, as the shared expert does, so a group holds T rows.
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("T", [129, 192, 193, 256, 257, 320, 321, 449])
def test_tail_rows(T, packed):
    check_layer(_cfg(T, 8, 2, 1, 256, 192, L.ROUTE_HARD_MASK, (0, 5)), packed=packed)


@pytest.mark.parametrize("T", [192, 257, 321])
def test_tail_rows_lora(T):
    check_lora(_cfg(T, 8, 2, 1, 192, 320, L.ROUTE_HARD_MASK, (0, 5)), rank=8)
