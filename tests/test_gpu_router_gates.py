"""The router product in a launch of its own behind every gate and with token-aware priorities: the logits lie in the workspace
and the front kernel, the separate routing pass of the distribution gate and the priorities read them (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import HostLayer, beta_pair, safe_threshold, tae_margin
from test_gpu_parity import _check_layer
from test_gpu_psi import _check, _measured_table

pytestmark = pytest.mark.gpu

# one tile (the grouping in the front kernel's tail), several tiles, the last token count with the launch of its own
BF16 = [("c4_qwen3", dict(d=256, F=128, E=E, n_resident=E // 2), T) for E in (65, 128) for T in (8, 33, 64)]
F32 = [("c4_qwen3", dict(d=256, F=96, E=33, K=4, n_resident=16, dtype="f32"), T) for T in (16, 40)]


@pytest.mark.parametrize("name,over,T", BF16 + F32)
@pytest.mark.parametrize("unique", [False, True])
def test_gates_behind_the_router_launch(name, over, T, unique):
    spec = workloads.scaled(name, **over)
    print("router launch gated", name, over, T, unique, flush=True)
    host = HostLayer(spec, T)
    ids, w = oracle.route_topk(host.f32(host.x), host.f32(host.w_router), host.bias, spec.K)
    tae, margin = tae_margin(w)
    tau, gamma = safe_threshold(tae, 0.35), safe_threshold(margin, 0.75)
    _check_layer(host, unique, tau=tau)
    _check_layer(host, unique, gamma=gamma, rho=2)
    _check_layer(host, unique, tau=tau, gamma=gamma, rho=1)
    closed, open_ = beta_pair(oracle.distribution_delta(ids, host.mask)[0])
    _, ref, _ = _check_layer(host, unique, beta=closed)
    assert ref["stats"]["bypassed"] == 1 and ref["stats"]["n_substituted"] == 0
    _, ref, _ = _check_layer(host, unique, beta=open_, tau=tau)
    assert ref["stats"]["bypassed"] == 0 and ref["stats"]["n_substituted"] > 0


@pytest.mark.parametrize("name,over,T", BF16 + F32)
def test_priorities_behind_the_router_launch(name, over, T):
    spec = workloads.scaled(name, **over)
    print("router launch psi", name, over, T, flush=True)
    table, q = _measured_table(spec)
    host = HostLayer(spec, T)
    host.table = table
    ids, _ = oracle.route_topk(host.f32(host.x), host.f32(host.w_router), host.bias, spec.K)
    closed, open_ = beta_pair(oracle.distribution_delta(ids, host.mask)[0])
    for unique in (False, True):
        _check(host, q, 8.0, unique)
    _check(host, q, 8.0, True, rho=1)
    out, ref = _check(host, q, 8.0, True, beta=open_)
    assert ref["stats"]["bypassed"] == 0 and ref["stats"]["n_substituted"] > 0
    out, ref = _check(host, q, 8.0, False, beta=closed)
    assert ref["stats"]["bypassed"] == 1 and ref["stats"]["n_substituted"] == 0


# one slot a token: U_t never decides (a non-resident expert is no candidate), the gates see one weight; one tile and several
@pytest.mark.parametrize("name,over", [("c2_mixtral_decode", dict(d=256, F=256, K=1)), ("c4_qwen3", dict(d=256, F=128, E=65, K=1, n_resident=30)),
                                       ("c1_tiny", dict(K=1))])
@pytest.mark.parametrize("T", [1, 16, 40])
def test_one_slot_per_token_in_the_layer(name, over, T):
    spec = workloads.scaled(name, **over)
    print("one slot in the layer", name, over, T, flush=True)
    host = HostLayer(spec, T)
    for unique in (False, True):
        for gates in (dict(), dict(tau=0.5), dict(gamma=0.5), dict(gamma=1.5), dict(rho=0), dict(tau=-0.5, rho=1), dict(beta=1.5), dict(beta=0.0)):
            _check_layer(host, unique, **gates)
