"""Layers whose router prefers a few experts, at token counts that take the tiles for few rows per sub-expert: groups of
several of their m-tiles beside groups without a row, with the m-tile table of each dispatch (one
workgroup, the end of the top-k kernel, the place kernel, the stage call's own), against the oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2510_19366_amd import binding as B
from paper_2510_19366_amd import workloads as W
from gpu_util import max_rel, row_rel, run_layer, run_stages, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,S,k_max,d,Is,longest", [
    (16, 16, 2, 4, 128, 96, 15),      # one workgroup for routing and dispatch; tiles of 16 rows, which all tokens fit
    (40, 16, 4, 8, 128, 96, 33),      # the end of the top-k kernel; tiles of 32
    (64, 4, 4, 8, 64, 32, 33),        # tiles of 64
    (100, 16, 4, 8, 448, 352, 65),    # several tiles of 32 per group, two 64-token words
    (200, 16, 4, 4, 256, 64, 97),     # the same; a narrow width
    (200, 64, 8, 32, 256, 64, 97),    # the same; place kernel
    (300, 32, 4, 16, 256, 128, 193),  # and tiles of 64, fewer sub-experts than CUs
    (2000, 64, 8, 4, 256, 64, 385),   # groups of many tiles of 32
    (900, 16, 4, 4, 256, 64, 257),    # the fused kernel, long tiles first
    (1100, 64, 8, 32, 256, 64, 257),  # and more of them
    (160, 50, 4, 32, 256, 64, 65),    # the fused kernel behind one workgroup's table, in the order of the groups
    (120, 50, 4, 60, 832, 192, 65),
    (300, 16, 4, 4, 128, 96, 129),    # place kernel, tiles of 32
    (300, 16, 4, 8, 448, 352, 193),   # and of 64
    (300, 16, 4, 8, 256, 32, 193),
])
def test_layer_with_a_skewed_load(T, N, S, k_max, d, Is, longest):
    k = np.random.default_rng(T).integers(1, k_max + 1, size=T).astype(np.int32)
    wl = W.make_workload("skewed", dtype="bf16", d=d, n_experts=N, n_sub=S, inter_sub=Is, req_tokens=[1] * T,
                         req_k=k, k_max=k_max, seed=T, bias_std=4.0, w_std=0.05)
    ref = O.layer_of(wl, return_all=True)
    assert ref["cnt"].max() >= longest and (ref["cnt"] == 0).any()
    r = run_stages(wl)
    for name in ("ids", "cnt", "off", "sorted_pair", "slot_of_pair"):
        assert np.array_equal(r[name], ref[name]), name
    # bf16: h and y are rounded once each, as in the other layer tests
    assert max_rel(r["y"], ref["y"]) <= 2e-2 and row_rel(r["y"], ref["y"]) <= 4e-2
    assert max_rel(r["out"], ref["out"]) <= 2e-2
    out, dev, ws = run_layer(wl, r["dev"], r["ws"])
    assert np.array_equal(to_np(out), r["out"])
    assert B.moe_prism_status(ws)[0] == 0


@pytest.mark.parametrize("T,path", [(65, "few"), (159, "few"), (384, "few"), (385, "fused")])
def test_narrow_sub_experts_on_both_sides_of_the_few_rows_rule(T, path):
    # 512 sub-experts, 32 picks: up to 24 possible rows for each
    k = np.random.default_rng(T).integers(0, 33, size=T).astype(np.int32)
    wl = W.make_workload("border", dtype="bf16", d=256, n_experts=64, n_sub=8, inter_sub=64, req_tokens=[1] * T,
                         req_k=k, k_max=32, seed=T, bias_std=1.0, w_std=0.05)
    dev = B.to_device(wl)
    assert B.ffn_path(dev["shape"]) == path
    B.moe_prism_timing_enable(True)
    B.moe_prism_timing_read()
    out, _, _ = run_layer(wl, dev)
    calls = {name: v[1] for name, v in B.moe_prism_timing_read().items()}
    B.moe_prism_timing_enable(False)
    assert (calls["ffn_fused"], calls["ffn_gate_up"], calls["ffn_down"]) == ((1, 0, 0) if path == "fused" else (0, 1, 1))
    assert max_rel(to_np(out), O.layer_of(wl)) <= 2e-2


@pytest.mark.parametrize("T,d,Is,path", [(74, 1024, 128, "few"), (396, 1024, 128, "few"), (397, 1024, 128, "fused"),
                                         (397, 2048, 128, "few"), (448, 2048, 128, "few"), (449, 2048, 128, "fused"),
                                         (640, 2048, 192, "few"), (641, 2048, 192, "fused")])
def test_narrow_sub_experts_beyond_that_range(T, d, Is, path):
    # 264 sub-experts, 16 picks: 24 possible rows for each, or the tokens that long phases are worth; short groups beside long ones
    k = np.random.default_rng(T).integers(0, 17, size=T).astype(np.int32)
    wl = W.make_workload("beside", dtype="bf16", d=d, n_experts=33, n_sub=8, inter_sub=Is, req_tokens=[1] * T,
                         req_k=k, k_max=16, seed=T, bias_std=1.0)
    dev = B.to_device(wl)
    assert B.ffn_path(dev["shape"]) == path
    out, _, ws = run_layer(wl, dev)
    tokens = np.arange(0, T, 9)
    ref, _, _ = O.layer_tokens(tokens, wl.x, wl.w_router, wl.router_bias, wl.k_tok, wl.w_gate_up, wl.w_down, wl.k_max,
                               wl.renormalize, wl.routed_scale)
    assert max_rel(to_np(out)[tokens], ref) <= 2e-2
    assert B.moe_prism_status(ws)[0] == 0
