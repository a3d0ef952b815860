"""Top-k by threshold search and the one-workgroup dispatch of small batches, at the sizes where
they change over: mask words of 64 tokens, the token and pair limits, the LDS limit, budgets around one
wave's 64 lanes, and logits with many equal values at the border of the budget."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2510_19366_amd import binding as B
from paper_2510_19366_amd import workloads as W
from gpu_util import max_rel, run_layer, run_stages, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k_max", [(1, 512, 32), (64, 40, 5), (65, 40, 5), (128, 64, 32), (128, 64, 33), (129, 64, 2),
                                       (129, 64, 3), (255, 64, 9),
                                       (255, 1500, 1), (255, 1530, 1), (130, 2100, 66),
                                       # the last of several workgroups or three launches
                                       (128, 64, 50), (128, 64, 51), (129, 64, 15), (129, 64, 16), (255, 64, 8),
                                       # one workgroup with all tokens: waves, elements per lane, LDS; just beyond
                                       (3, 64, 64), (5, 512, 32), (16, 66, 1), (16, 1024, 40), (17, 64, 8),
                                       (16, 1026, 8), (15, 1024, 200), (2, 1024, 512),
                                       (66, 1040, 1024), (128, 64, 40), (128, 64, 41)])
def test_small_batches_match_the_oracle(T, E, k_max):
    k = np.random.default_rng(T).integers(0, k_max + 1, size=T).astype(np.int32)
    wl = W.make_workload("small", dtype="bf16", d=64, n_experts=E // 2, n_sub=2, inter_sub=32,
                         req_tokens=[1] * T, req_k=k, k_max=k_max, seed=T, bias_std=1.0, w_std=0.1)
    r = run_stages(wl)
    ref = O.layer_of(wl, return_all=True)
    for key in ("ids", "cnt", "off", "sorted_pair", "slot_of_pair"):
        assert np.array_equal(r[key], ref[key]), key
    out, dev, ws = run_layer(wl)
    assert max_rel(to_np(out), ref["out"]) <= 2e-2
    # the layer's own tables (picks dispatched by the top-k kernel) equal the stage calls'
    im = B.layer_intermediates(dev["shape"], ws)
    assert np.array_equal(to_np(im["topk_ids"]), ref["ids"])
    for key, name in (("cnt", "group_count"), ("off", "group_offset"), ("sorted_pair", "sorted_pair"),
                      ("slot_of_pair", "slot_of_pair")):
        assert np.array_equal(to_np(im[name]), ref[key]), name


@pytest.mark.parametrize("T,E,k_max,one", [
    (64, 64, 64, 1), (65, 1024, 1024, 1), (66, 1024, 1024, 1), (67, 1024, 853, 1), (67, 1024, 854, 0),
    (100, 128, 71, 1), (100, 128, 72, 0), (128, 64, 40, 1), (128, 64, 41, 0),  # 2560 pairs beyond those of 64 tokens
    (129, 64, 15, 1), (129, 64, 16, 0), (255, 64, 8, 1), (255, 64, 9, 0), (256, 64, 1, 0)])  # 2048 pairs; 255 tokens
def test_batches_that_one_workgroup_dispatches(T, E, k_max, one):
    rng = np.random.default_rng(T + k_max)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k_max].astype(np.int32)
    ids[np.arange(k_max) >= rng.integers(0, k_max + 1, T)[:, None]] = -1
    shape = B.make_shape(T, 64, E, 1, 32, k_max, "bf16")
    ws = B.alloc_workspace(shape)
    B.moe_prism_timing_enable(True)
    B.moe_prism_timing_read()
    tables = B.moe_prism_dispatch(shape, torch.from_numpy(ids).cuda(), ws)
    calls = {name: v[1] for name, v in B.moe_prism_timing_read().items()}
    B.moe_prism_timing_enable(False)
    assert (calls["dispatch_count"], calls["dispatch_place"]) == (1 - one, 1)
    for got, ref in zip(tables, O.dispatch(ids, E)):
        assert np.array_equal(to_np(got), ref)


@pytest.mark.parametrize("values", [2, 9])
@pytest.mark.parametrize("E,k_max", [(64, 64), (130, 65), (512, 63), (520, 200)])
def test_equal_logits_at_the_border_go_to_the_lower_ids(E, k_max, values):
    # every logit is one of a few values (signed zeros and infinities among them): x = 1, one weight
    # per sub-expert plus the bias
    T, d = 40, 64
    rng = np.random.default_rng(E + values)
    x = np.zeros((T, d), np.float32)
    x[np.arange(T), np.arange(T) % 8] = 1.0
    pool = np.array([0.0, -0.0, 1.0, -1.0, 1e-30, -3.0, 65504.0, 0.5, -np.inf], np.float32)[:values]
    w = np.zeros((E, d), np.float32)
    bias = rng.choice(pool, size=E).astype(np.float32)
    k = rng.integers(0, k_max + 1, size=T).astype(np.int32)
    k[:2] = [k_max, 0]
    shape = B.make_shape(T, d, E, 1, 32, k_max, "f32")
    ws = B.alloc_workspace(shape)
    ids, wt, lg = B.moe_prism_route(shape, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(),
                                    torch.from_numpy(bias).cuda(), torch.from_numpy(k).cuda(), ws, want_logits=True)
    torch.cuda.synchronize()
    ref = O.logits(x, w, bias)
    assert np.array_equal(to_np(lg).view(np.uint32), ref.view(np.uint32))
    assert np.array_equal(to_np(ids), O.select(ref, k, k_max))


@pytest.mark.parametrize("low", [float(np.finfo(np.float32).min), -np.inf, 1e30])
@pytest.mark.parametrize("E,k_max", [(64, 2), (64, 8), (130, 16), (512, 32), (4000, 65)])
def test_masked_logits(E, k_max, low):
    # a router bias of the lowest finite value (or infinity; or huge outliers) on half of the
    # sub-experts, and on all but a few in some calls: fewer unmasked ones than picks included
    T, d = 70, 64
    rng = np.random.default_rng(E)
    x = rng.standard_normal((T, d)).astype(np.float32)
    w = (rng.standard_normal((E, d)) * 0.2).astype(np.float32)
    k = rng.integers(0, k_max + 1, size=T).astype(np.int32)
    shape = B.make_shape(T, d, E, 1, 32, k_max, "f32")
    ws = B.alloc_workspace(shape)
    for masked in (1, E // 2, E - k_max // 2, E):
        bias = np.zeros(E, np.float32)
        bias[rng.permutation(E)[:masked]] = low
        ids, _, lg = B.moe_prism_route(shape, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(),
                                       torch.from_numpy(bias).cuda(), torch.from_numpy(k).cuda(), ws, want_logits=True)
        torch.cuda.synchronize()
        ref = O.logits(x, w, bias)
        assert np.array_equal(to_np(lg).view(np.uint32), ref.view(np.uint32))
        assert np.array_equal(to_np(ids), O.select(ref, k, k_max)), masked


@pytest.mark.parametrize("E", [5, 64, 100, 512, 2100])
def test_few_picks_of_equal_and_distinct_logits(E):
    # budgets on both sides of the border between a maximum per pick and the search; few distinct values,
    # so that several lanes, and several elements of a lane, hold the maximum
    T, d, k_max = 90, 64, min(E, 9)
    rng = np.random.default_rng(E)
    for x, w in ((rng.standard_normal((T, d)), rng.standard_normal((E, d))),
                 (np.ones((T, d)), rng.integers(-2, 3, (E, 1)) * np.ones((1, d)))):
        x, w = x.astype(np.float32), w.astype(np.float32)
        k = rng.integers(0, k_max + 1, size=T).astype(np.int32)
        shape = B.make_shape(T, d, E, 1, 32, k_max, "f32")
        ws = B.alloc_workspace(shape)
        ids, _, lg = B.moe_prism_route(shape, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), None,
                                       torch.from_numpy(k).cuda(), ws, want_logits=True)
        torch.cuda.synchronize()
        ref = O.logits(x, w, None)
        assert np.array_equal(to_np(lg).view(np.uint32), ref.view(np.uint32))
        assert np.array_equal(to_np(ids), O.select(ref, k, k_max))


def test_logits_of_more_tokens_than_a_grid_has_rows():
    T, d, E = 4300000, 64, 33  # 32-token tiles: 134 375 rows
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn(T, d, generator=g, device="cuda", dtype=torch.bfloat16)
    w = torch.randn(E, d, generator=g, device="cuda", dtype=torch.bfloat16)

    def route(x):
        shape = B.make_shape(len(x), d, E, 1, 32, 1, "bf16")
        k = torch.ones(len(x), dtype=torch.int32, device="cuda")
        return B.moe_prism_route(shape, x, w, None, k, B.alloc_workspace(shape), want_logits=True)

    ids, wt, lg = route(x)
    ref = torch.cat([x[i:i + 500000].float() @ w.float().T for i in range(0, T, 500000)])
    # a chain of 64 roundings of 2^-24 on sums of 64 terms, |term| <= 30 here, against another order of the same sum
    assert (lg - ref).abs().max() <= 64 * 2.0 ** -24 * 64 * 30
    assert torch.equal(ids[:, 0].long(), lg.argmax(dim=1))
    for t in (0, 2097100, 4194200, T - 300):
        assert all(torch.equal(a, b[t:t + 300]) for a, b in zip(route(x[t:t + 300].contiguous()), (ids, wt, lg)))


@pytest.mark.parametrize("dtype,N,S,change", [("bf16", 128, 4, None), ("bf16", 85, 6, None), ("bf16", 64, 8, None),
                                              ("bf16", 256, 2, None), ("f32", 128, 4, None), ("bf16", 128, 4, (511, 2047)),
                                              ("bf16", 128, 4, (1, 0)), ("bf16", 85, 6, (505, 1030))])
def test_equal_router_rows_are_computed_once_with_the_same_logits(dtype, N, S, change):
    # beyond 2^34 multiply-adds the rows of an expert's sub-experts are compared; against the same rows as experts of their
    # own, which are not: bit for bit, with a bias per sub-expert, and where one element of one row is another
    T, d, E, k_max = 2 ** 23 // (N * S) + 67, 2048, N * S, 9
    g = torch.Generator(device="cuda").manual_seed(N + S)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.empty(T, d, dtype=dt, device="cuda").normal_(generator=g)
    w = torch.empty(N, d, dtype=dt, device="cuda").normal_(0.0, 0.02, generator=g).repeat_interleave(S, dim=0).contiguous()
    if change is not None:
        w[change] = w[change] + 0.5
    bias = torch.empty(E, device="cuda").normal_(generator=g)
    k = torch.full((T,), k_max, dtype=torch.int32, device="cuda")
    for b in (None, bias):
        shared, alone = (B.make_shape(T, d, n, s, 32, k_max, dtype, 1, 1.0) for n, s in ((N, S), (E, 1)))
        got = B.moe_prism_route(shared, x, w, b, k, B.alloc_workspace(shared), want_logits=True)
        ref = B.moe_prism_route(alone, x, w, b, k, B.alloc_workspace(alone), want_logits=True)
        for a, r in zip(got, ref):
            assert torch.equal(a, r)
    tokens = torch.tensor([0, 63, 64, T // 2, T - 1])
    exact = x[tokens].double() @ w.double().T
    bound = 2.0 * d * 2.0 ** -24 * (x[tokens].double().abs() @ w.double().abs().T)  # d roundings of the running sum
    assert ((ref[2][tokens].double() - bias.double() - exact).abs() <= bound + 1e-6).all()


@pytest.mark.parametrize("d", [64, 128, 192, 256, 320, 384, 448, 512])
@pytest.mark.parametrize("T,E", [(1, 5), (33, 70), (3001, 510), (12001, 509)])  # tiles of 32 x 32, 32 x 64, 64 x 64
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_logits_of_every_tile_and_count_of_stages(T, E, d, dtype):
    # fewer stages than the ring holds, and more, with the copies in the waves of the products or apart; small whole
    # numbers, so that every order of the sum is exact
    g = torch.Generator(device="cuda").manual_seed(T + d)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randint(-9, 10, (T, d), generator=g, device="cuda").to(dt)
    w = torch.randint(-9, 10, (E, d), generator=g, device="cuda").to(dt)
    k = torch.ones(T, dtype=torch.int32, device="cuda")
    shape = B.make_shape(T, d, E, 1, 32, 1, dtype)
    ids, _, lg = B.moe_prism_route(shape, x, w, None, k, B.alloc_workspace(shape), want_logits=True)
    ref = x.double() @ w.double().T
    assert torch.equal(lg.double(), ref)
    assert torch.equal(lg.gather(1, ids[:, :1].long()), lg.max(dim=1, keepdim=True).values)


@pytest.mark.parametrize("T,E,k_max,one", [
    (128, 64, 64, 1), (136, 64, 64, 1), (137, 64, 64, 0), (255, 512, 24, 1), (255, 512, 25, 0), (256, 64, 1, 0),  # 4608 pairs, 255 tokens
    (90, 1024, 177, 1), (90, 1024, 178, 0), (65, 1024, 480, 1), (73, 512, 480, 1), (66, 512, 512, 1), (80, 512, 481, 0),  # eight waves, four
    (200, 1706, 3, 1), (200, 1707, 3, 0), (40, 4096, 8, 1),  # 60 KiB of masks
    (8, 64, 9, 1), (9, 64, 9, 1), (8, 1100, 70, 1), (9, 1000, 70, 1)])  # one workgroup for all tokens, the last of two
def test_layer_batches_that_the_top_k_kernel_dispatches(T, E, k_max, one):
    # against the stage calls, whose own rules and kernels are others; skewed, budgets of 0 to k_max
    d, Is = 64, 32
    g = torch.Generator(device="cuda").manual_seed(T + E + k_max)
    shape = B.make_shape(T, d, E, 1, Is, k_max, "f32", 1, 1.0)

    def normal(*size, std):
        return torch.empty(size, device="cuda").normal_(0.0, std, generator=g)
    x, w_r, w_gu, w_dn = normal(T, d, std=1.0), normal(E, d, std=0.02), normal(E, 2 * Is, d, std=0.1), normal(E, d, Is, std=0.1)
    bias = normal(E, std=1.0)
    k = torch.randint(0, k_max + 1, (T,), generator=g, device="cuda", dtype=torch.int32)
    ws = B.alloc_workspace(shape)
    B.moe_prism_timing_enable(True)
    try:
        out = B.moe_prism_layer(shape, x, w_r, bias, k, w_gu, w_dn, ws).clone()
        torch.cuda.synchronize()
        calls = {name: v[1] for name, v in B.moe_prism_timing_read().items()}
    finally:
        B.moe_prism_timing_enable(False)
    assert calls["dispatch_place"] == 1 - one
    ids, wt, _ = B.moe_prism_route(shape, x, w_r, bias, k, ws, want_logits=True)
    _, off, sp, sl = B.moe_prism_dispatch(shape, ids, ws)
    y = B.moe_prism_grouped_ffn(shape, x, w_gu, w_dn, off, sp, ws)
    assert torch.equal(out, B.moe_prism_combine(shape, y, sl, wt, k))


@pytest.mark.parametrize("T,E,k_max", [
    (300, 4, 4), (8000, 4, 3), (16384, 4, 4), (16320, 4, 1), (300, 8, 2), (513, 16, 16), (2000, 32, 4),  # few groups: counts added up by few threads
    (1, 1, 1), (64, 16, 4), (65, 4, 4), (32, 1100, 8), (33, 512, 8), (1, 1024, 257), (8, 4096, 32),  # one workgroup, of 256 threads and of 1024
])
def test_dispatch_of_random_picks(T, E, k_max):
    # against a stable sort of the pairs by sub-expert; budgets of 0 to k_max
    g = torch.Generator(device="cuda").manual_seed(T + E + k_max)
    budget = torch.randint(0, k_max + 1, (T, 1), generator=g, device="cuda")
    load = torch.rand(E, generator=g, device="cuda")
    ids = (torch.rand(T, E, generator=g, device="cuda") + load).topk(k_max, dim=1).indices.int()
    ids[torch.arange(k_max, device="cuda")[None, :] >= budget] = -1
    shape = B.make_shape(T, 64, E, 1, 32, k_max, "bf16")
    cnt, off, sp, sl = B.moe_prism_dispatch(shape, ids, B.alloc_workspace(shape))
    flat = ids.flatten().long()
    count = torch.bincount(flat[flat >= 0], minlength=E)
    P = int(count.sum())
    order = torch.where(flat >= 0, flat, E).sort(stable=True).indices
    assert torch.equal(cnt.long(), count) and torch.equal(off[1:].long(), count.cumsum(0)) and off[0] == 0
    assert torch.equal(sp[:P].long(), order[:P]) and (sp[P:] == -1).all()
    slots = torch.full_like(flat, -1)
    slots[order[:P]] = torch.arange(P, device="cuda")
    assert torch.equal(sl.long(), slots)


@pytest.mark.parametrize("T,E,k_max", [
    (9, 64, 9), (10, 1024, 33), (11, 1024, 33), (12, 853, 9), (13, 512, 9), (12, 512, 512), (16, 128, 128), (16, 128, 12), (16, 128, 13), (16, 129, 12), (17, 128, 20), (13, 17, 17)])
def test_layer_batches_around_one_workgroup_for_all_tokens(T, E, k_max):
    test_layer_batches_that_the_top_k_kernel_dispatches(T, E, k_max, 1)


@pytest.mark.parametrize("dtype,T,E,d", [
    (dtype, T, E, d) for dtype in ("bf16", "f32") for T, E in ((17293, 250), (8100, 510), (25200, 512)) for d in (64, 192, 256, 448, 512)])
def test_logits_where_the_tile_goes_by_the_length_of_a_row(dtype, T, E, d):
    # 32 x 32 with copies by the same waves and apart; the fourth workgroup of 64 x 64 on a CU or 32 x 64; the thirteenth
    test_logits_of_every_tile_and_count_of_stages(T=T, E=E, d=d, dtype=dtype)
