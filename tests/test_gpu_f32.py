"""fp32 layers and the fp32 router against the oracle at the edges of their tiles: hidden and FFN
sizes that are no multiple of a 64-value chunk, of a 16-byte unit or of the 32 output columns of a
workgroup, row groups around 32 rows, one token, many experts, shared experts; routers whose
outputs split the reduction (up to 64) or the output tiles, over several layers. Bounds as in
test_gpu_layer and test_gpu_route (fp32: 2e-5 of the largest output)."""

import numpy as np
import pytest
import torch

import gpu_util as U
from oracle import routing as R
from paper_2609_34077_amd import _lib as L
from paper_2609_34077_amd import synth
from test_gpu_layer import check_layer
from test_gpu_route import _inputs

pytestmark = pytest.mark.gpu

# (T, d, F, E, K, shared)
LAYERS = [(1, 64, 64, 4, 2, 0), (33, 3, 5, 2, 1, 0), (33, 50, 70, 5, 2, 0), (40, 36, 100, 8, 2, 1), (65, 64, 33, 1, 1, 1),
          (300, 96, 130, 64, 6, 2), (32, 260, 192, 256, 16, 0)]


@pytest.mark.parametrize("T,d,F,E,K,ns", LAYERS)
def test_f32_layer(T, d, F, E, K, ns):
    check_layer(synth.LayerConfig(f"f32_t{T}_d{d}_f{F}_e{E}", T=T, d=d, F=F, E=E, K=K, n_shared=ns, dtype="f32",
                                  route_mode=L.ROUTE_PLAIN, gate_mode=L.GATE_P if ns else L.GATE_RENORM, seed=T + d))


@pytest.mark.parametrize("T,d,E,K,layers", [(1, 16, 1, 1, 1), (17, 6, 8, 2, 3), (16, 33, 16, 16, 4), (19, 100, 5, 3, 13),
                                            (50, 200, 33, 4, 3), (35, 76, 256, 16, 2)])
def test_f32_router(T, d, E, K, layers):
    U.say(f"f32 route T={T} d={d} E={E} K={K} layers={layers}")
    x, w = _inputs(T, d, E, "f32", T + d, Lyr=layers)
    w = w.reshape(layers, E, d)
    prior = np.stack([synth.concentrated_prior(E, [i % E], 1.0) for i in range(layers)])
    idx, gate, margin = L.maskmoe_route(U.dev(x), U.dev(w), K, L.ROUTE_SOFT_PRIOR, L.GATE_P, prior=prior)
    torch.cuda.synchronize()
    for i in range(layers):
        z = R.router_logits(U.f64(x, "f32"), U.f64(w[i], "f32"))
        U.check_routing(z, idx[i].cpu().numpy(), gate[i].cpu().numpy(), margin[i].cpu().numpy(), K, L.ROUTE_SOFT_PRIOR,
                        L.GATE_P, prior=prior[i])
