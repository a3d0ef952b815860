"""The grouped FFN's kernels on groups whose sizes are the edges of their tiles (slot blocks of 32
rows, m-tiles of 256, empty groups), at widths with partial weight tiles and a half K stage, and
SwiGLU where its gate is huge or infinite."""
import numpy as np
import pytest
import torch

from paper_2510_19366_amd import binding as B

pytestmark = pytest.mark.gpu

SIZES = [257, 1, 0, 31, 32, 33, 63, 64, 65, 0, 0, 127, 129, 191, 255, 256, 300, 2]
LONG = [257, 320, 321, 352, 384, 385, 0, 448, 449, 511, 512, 513, 576, 577, 640, 769, 1025]
FEW = [1, 0, 33, 0, 0, 30]
ONE = [1, 0, 9, 2, 0, 3]
TWO = [1, 0, 15, 16, 17, 31, 32, 33, 0, 47, 5, 64, 48]
FOUR = [63, 64, 65, 48, 49, 15, 0, 1, 33, 128, 130, 16]
LONG_FOUR = [0, 0, 270, 1, 0, 0, 31, 0, 33, 0, 0, 96, 0, 0, 2, 0, 0, 0, 0, 128]  # 28 rows for each on average: four blocks
LONG_TWO = [0] * 9 + [200] + [0] * 10 + [31, 1, 65] + [0] * 3


def ffn(dtype, x, w_gu, w_dn, group):
    """moe_prism_grouped_ffn of one pick per token, rows back in token order."""
    T, d = x.shape
    E, Is = w_dn.shape[0], w_dn.shape[2]
    shape = B.make_shape(T, d, E, 1, Is, 1, dtype)
    ws = B.alloc_workspace(shape)
    ids = group.to(torch.int32).view(T, 1).cuda()
    _, off, sp, sl = B.moe_prism_dispatch(shape, ids, ws)
    y = B.moe_prism_grouped_ffn(shape, x.cuda(), w_gu.cuda(), w_dn.cuda(), off, sp, ws)
    return y[sl.view(-1).long()].float().cpu()


@pytest.mark.parametrize("dtype,path,sizes,d,Is", [
    ("bf16", "auto", SIZES, 256, 256),    # two-kernel, shortest K of the ring driver
    ("bf16", "auto", LONG, 256, 256),     # groups of several m-tiles, cut evenly
    ("bf16", "auto", SIZES, 448, 288),    # half K stage in the down GEMM; 32 neurons in the last gate-up tile
    ("bf16", "auto", SIZES, 576, 704),    # 64 columns in the last down tile, 64 neurons in the last gate-up tile
    ("bf16", "auto", SIZES, 192, 320),    # gate-up K too short for the ring
    ("bf16", "auto", SIZES, 64, 8192),    # five short items per workgroup: gate-up, one and two slabs of K
    ("bf16", "auto", SIZES, 128, 8192),
    ("bf16", "auto", SIZES, 16384, 32),   # down, half a slab and one and a half
    ("bf16", "auto", SIZES, 16384, 96),
    ("bf16", "auto", SIZES, 256, 64),     # fused, each width
    ("bf16", "auto", SIZES, 576, 128),
    ("bf16", "auto", SIZES, 320, 192),
    ("bf16", "auto", [34, 1, 64, 25] * 65, 320, 64),  # fused, more tiles than CUs: the next tile known from the start, near the end
    ("bf16", "auto", [34, 1, 64, 25] * 65, 832, 64),
    ("bf16", "auto", [300, 1, 64, 25, 0] * 65, 896, 192),
    ("bf16", "auto", [300, 1, 64, 25, 0] * 65, 1408, 192),  # long enough that empty lists draw from the others
    ("bf16", "split", SIZES, 512, 192),   # weight tiles with and without a second half
    ("bf16", "auto", FEW, 64, 32),        # small tiles: one K stage; half a stage
    ("bf16", "auto", FEW, 448, 352),
    ("bf16", "auto", FEW, 2048, 192),
    ("bf16", "auto", ONE, 64, 32),        # at most 16 tokens: one stage, half a stage, more stages than the ring has
    ("bf16", "auto", ONE, 448, 352),
    ("bf16", "auto", ONE, 2048, 192),
    ("bf16", "auto", ONE, 4096, 96),
    ("bf16", "auto", [16], 320, 1024),
    ("bf16", "auto", [0, 17], 576, 160),  # one token more
    # up to 24 rows per group: two blocks of 16 rows at a time, several times (bits at 64 x 32 are compared below; there the
    # rounding of h, 2^-9 of its norm, reaches y times up to the condition number of 64 x 32 weights: 0.0041 in one row)
    ("bf16", "auto", TWO, 128, 96),
    ("bf16", "auto", TWO, 448, 352),
    ("bf16", "auto", TWO, 1024, 160),
    ("bf16", "auto", FOUR, 64, 32),       # up to 56: four; waves without weight rows in the last tiles
    ("bf16", "auto", FOUR, 192, 96),
    ("bf16", "auto", FOUR, 448, 352),
    ("bf16", "auto", FOUR, 1024, 160),
    ("bf16", "auto", LONG_FOUR, 448, 352),  # a group of several m-tiles beside empty ones, in tiles of 64 rows and of 32
    ("bf16", "auto", LONG_FOUR, 128, 96),  # (not 64 x 32: as above)
    ("bf16", "auto", LONG_TWO, 448, 352),
    ("bf16", "auto", LONG_TWO, 128, 96),
    ("bf16", "auto", LONG, 256, 32),      # gate-up of 32 neurons: row blocks of an m-tile as items of their own
    ("bf16", "auto", LONG, 448, 32),
    ("f32", "auto", SIZES, 64, 32),
    ("f32", "auto", SIZES, 320, 96),
    ("f32", "auto", FEW, 256, 128),
    ("f32", "auto", TWO, 64, 32),         # several row blocks per group from the short list
    ("f32", "auto", FOUR, 320, 96),
    ("f32", "auto", [256, 3] * 30 + [40], 64, 640),  # two column blocks per wave
    ("f32", "auto", [300, 600, 1], 64, 32),  # the list of all row blocks
    # many weight tiles, 53 and 57 rows per group on average: on both sides of the border between the lists
    ("f32", "auto", [0, 130, 31] * 13 + [33], 1024, 544),
    ("f32", "auto", [0, 140, 33] * 13 + [34], 1024, 544),
])
def test_group_sizes_at_the_edges_of_the_tiles(dtype, path, sizes, d, Is, monkeypatch):
    monkeypatch.setenv("MOE_PRISM_FFN", path)
    g = torch.Generator().manual_seed(d + Is)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    E, T = len(sizes), sum(sizes)
    group = torch.repeat_interleave(torch.arange(E), torch.tensor(sizes))[torch.randperm(T, generator=g)]
    x = torch.randn(T, d, generator=g).to(dt)
    w_gu = (torch.randn(E, 2 * Is, d, generator=g) * 0.05).to(dt)
    w_dn = (torch.randn(E, d, Is, generator=g) * 0.05).to(dt)
    got = ffn(dtype, x, w_gu, w_dn, group)
    ref = torch.empty(T, d, dtype=torch.float64)
    for e in range(E):
        rows = (group == e).nonzero().view(-1)
        v = x[rows].double() @ w_gu[e].double().T
        a, u = v[:, :Is], v[:, Is:]
        ref[rows] = (a / (1 + torch.exp(-a)) * u) @ w_dn[e].double().T
    err = (got.double() - ref).norm(dim=1) / ref.norm(dim=1)
    # bf16: h and y are rounded once each, 2^-9 at most; fp32: chains of up to d roundings of 2^-24,
    # twice (and expf)
    assert err.max() <= (2 * 2.0 ** -9 if dtype == "bf16" else 2 * d * 2.0 ** -24), int(err.argmax())


@pytest.mark.parametrize("path,T,d,Is", [("auto", 12, 256, 192),    # small tiles
                                         ("auto", 300, 256, 192),   # fused
                                         ("split", 300, 256, 192),  # two-kernel, ring
                                         ("split", 300, 128, 192)])  # two-kernel, short K
def test_swiglu_of_huge_and_infinite_gates(path, T, d, Is, monkeypatch):
    # gate = x[0] 2^64, up = x[1] = 1, output = mean of the (equal) activations
    monkeypatch.setenv("MOE_PRISM_FFN", path)
    gates = torch.tensor([float("inf"), 3e38, 1e20, 100.0, 5.0, 0.0, -5.0, -80.0, -89.0, -100.0, -1e30, -3e38])
    x = torch.zeros(T, d)
    a = gates.repeat(-(-T // len(gates)))[:T]
    x[:, 0] = torch.where(a.isinf(), torch.full_like(a, 2.0 ** 100), a * 2.0 ** -64)  # overflows to infinity
    x[:, 1] = 1.0
    x = x.bfloat16()
    E = 2
    w_gu = torch.zeros(E, 2 * Is, d)
    w_gu[:, :Is, 0] = 2.0 ** 64
    w_gu[:, Is:, 1] = 1.0
    w_dn = torch.full((E, d, Is), 2.0 ** -8)
    got = ffn("bf16", x, w_gu.bfloat16(), w_dn.bfloat16(), torch.arange(T) % E)
    a = x[:, 0].float() * 2.0 ** 64
    h = (a / (1 + torch.exp(-a))).bfloat16().double() * (2.0 ** -8 * Is)
    for t in range(T):
        # one bf16 rounding each of h and y, and the gate's exponential: 2^-20 at a = -80
        torch.testing.assert_close(got[t].double(), h[t].expand(d), rtol=2.0 ** -7, atol=1e-35,
                                   msg=lambda m: f"gate {a[t]}: {m}")


@pytest.mark.parametrize("d,Is", [(64, 32), (320, 32), (2048, 32), (448, 192), (2048, 192), (320, 352), (1024, 704)])
def test_a_rows_bits_do_not_depend_on_the_batch_it_is_in(d, Is):
    # a handful of tokens takes the small tiles, hundreds of them the other drivers; every sum over K
    # is one chain in ascending k in all of them
    g = torch.Generator().manual_seed(d + Is)
    E, T, few, one = 6, 400, 24, 13
    x = torch.randn(T, d, generator=g).bfloat16()
    w_gu = (torch.randn(E, 2 * Is, d, generator=g) * 0.05).bfloat16()
    w_dn = (torch.randn(E, d, Is, generator=g) * 0.05).bfloat16()
    group = torch.randint(0, E, (T,), generator=g)
    whole = ffn("bf16", x, w_gu, w_dn, group)
    assert torch.equal(ffn("bf16", x[:few], w_gu, w_dn, group[:few]), whole[:few])
    assert torch.equal(ffn("bf16", x[:one], w_gu, w_dn, group[:one]), whole[:one])
    for more in (100, 200):  # two and four blocks of 16 rows
        assert torch.equal(ffn("bf16", x[:more], w_gu, w_dn, group[:more]), whole[:more])


@pytest.mark.parametrize("dtype,T,k_max", [("bf16", 40, 8), ("f32", 40, 8), ("bf16", 10, 32)])
def test_a_callers_own_tables_with_groups_of_more_rows_than_tokens(dtype, T, k_max):
    # all pairs of a few tokens in one group of 320 rows: a full m-tile and a second one, in the kernels whose
    # m-tiles otherwise have one or two row blocks
    d, Is, E = 256, 96, 32
    g = torch.Generator().manual_seed(5)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn(T, d, generator=g).to(dt)
    w_gu = (torch.randn(E, 2 * Is, d, generator=g) * 0.05).to(dt)
    w_dn = (torch.randn(E, d, Is, generator=g) * 0.05).to(dt)
    pair = torch.randperm(T * k_max, generator=g).to(torch.int32)
    off = torch.tensor([0] * 3 + [320] * (E - 2), dtype=torch.int32)
    shape = B.make_shape(T, d, E, 1, Is, k_max, dtype)
    y = B.moe_prism_grouped_ffn(shape, x.cuda(), w_gu.cuda(), w_dn.cuda(), off.cuda(), pair.cuda(), B.alloc_workspace(shape))
    v = x[(pair // k_max).long()].double() @ w_gu[2].double().T
    a, u = v[:, :Is], v[:, Is:]
    ref = (a / (1 + torch.exp(-a)) * u) @ w_dn[2].double().T
    err = (y.cpu().double() - ref).norm(dim=1) / ref.norm(dim=1)
    assert err.max() <= (2 * 2.0 ** -9 if dtype == "bf16" else 2 * d * 2.0 ** -24), int(err.argmax())


@pytest.mark.parametrize("T,N,S,k_max,d,Is,combines", [
    (1, 128, 4, 32, 2048, 192, 1),    # 8 columns: 256 workgroups; a block per tile
    (1, 1, 1, 1, 2048, 64, 1),        # one block, of which a wave has two
    (8, 16, 4, 4, 1536, 96, 1), (9, 16, 4, 4, 1600, 32, 1),  # up to 8 rows to a group, and more; half a stage; 200 workgroups
    (17, 3, 1, 2, 1984, 320, 1),      # few groups, tiles of several blocks
    (37, 128, 4, 32, 2048, 192, 1), (78, 128, 4, 32, 2048, 192, 1), (79, 128, 4, 32, 2048, 192, 0),  # 2510 possible rows
    (200, 256, 4, 12, 2048, 64, 1),   # more tiles than threads; the tokens in two turns
    (64, 64, 2, 12, 2048, 704, 1), (129, 64, 2, 12, 2048, 704, 0),  # 12 possible rows to a group
    (64, 64, 2, 12, 1536, 352, 1), (65, 64, 2, 12, 1536, 352, 0),  # 6, where K has half a stage
    (30, 16, 2, 4, 1472, 64, 0), (30, 16, 2, 4, 2112, 64, 0), (30, 16, 2, 4, 3008, 64, 0),  # 3/4 of the CUs; all of them
    (5, 8, 4, 8, 4096, 608, 1), (24, 128, 4, 32, 3136, 192, 1), (25, 128, 4, 32, 3136, 192, 1),  # 16 columns: 196 workgroups; 773
    (48, 128, 4, 32, 3136, 192, 1), (49, 128, 4, 32, 3136, 192, 0),  # and 1553 rows
    (100, 64, 4, 11, 3072, 64, 1), (30, 16, 2, 4, 4160, 64, 0)])
def test_down_projection_and_combine_in_one_kernel(T, N, S, k_max, d, Is, combines):
    # against the stage calls, which do them one after the other: the same sums in the same order, bit for bit.  Budgets of 0 to
    # k_max; a router bias that gives some groups many tokens
    g = torch.Generator(device="cuda").manual_seed(T + d)
    E = N * S
    shape = B.make_shape(T, d, N, S, Is, k_max, "bf16", 1, 1.5)

    def normal(*size, std):
        return torch.empty(size, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, w_r, w_gu, w_dn = normal(T, d, std=1.0), normal(E, d, std=0.02), normal(E, 2 * Is, d, std=0.05), normal(E, d, Is, std=0.05)
    bias = torch.empty(E, device="cuda").normal_(generator=g)
    k = torch.randint(0, k_max + 1, (T,), generator=g, device="cuda", dtype=torch.int32)
    k[0] = k_max
    ws = B.alloc_workspace(shape)
    B.moe_prism_timing_enable(True)
    try:
        out = B.moe_prism_layer(shape, x, w_r, bias, k, w_gu, w_dn, ws)
        torch.cuda.synchronize()
        assert (B.moe_prism_timing_read()["combine"][1] == 0) == bool(combines)
    finally:
        B.moe_prism_timing_enable(False)
    out = out.clone()
    ids, wt, _ = B.moe_prism_route(shape, x, w_r, bias, k, ws, want_logits=True)
    _, off, sp, sl = B.moe_prism_dispatch(shape, ids, ws)
    y = B.moe_prism_grouped_ffn(shape, x, w_gu, w_dn, off, sp, ws)
    ref = B.moe_prism_combine(shape, y, sl, wt, k)
    assert out[k > 0].abs().max() > 0
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("dtype,T,E,k_max,d,Is,picks", [
    ("bf16", 1, 1, 1, 64, 32, 1), ("bf16", 1, 64, 6, 512, 64, 1), ("bf16", 2, 65, 7, 448, 96, 1), ("bf16", 3, 128, 64, 576, 32, 1),
    ("bf16", 4, 129, 40, 1088, 64, 1), ("bf16", 1, 256, 64, 2048, 192, 1), ("bf16", 4, 257, 33, 64, 192, 1),
    ("bf16", 1, 512, 32, 2048, 192, 1), ("bf16", 4, 512, 64, 1024, 128, 1), ("bf16", 4, 512, 8, 320, 352, 1), ("bf16", 2, 512, 2, 1536, 32, 1),
    ("bf16", 5, 512, 8, 320, 192, 0), ("bf16", 1, 513, 8, 320, 192, 0), ("bf16", 4, 128, 65, 320, 64, 0),
    ("f32", 1, 1, 1, 64, 32, 1), ("f32", 2, 5, 5, 128, 96, 1), ("f32", 33, 31, 7, 192, 64, 1), ("f32", 64, 32, 8, 256, 128, 1),
    ("f32", 64, 32, 32, 64, 32, 1), ("f32", 63, 9, 3, 320, 1184, 1),  # the last one: two column blocks per wave
    ("f32", 65, 32, 8, 64, 32, 0), ("f32", 64, 33, 8, 64, 32, 0)])
@pytest.mark.parametrize("renorm,ties", [(1, False), (0, False), (1, True)])
def test_gate_up_that_picks_for_itself(dtype, T, E, k_max, d, Is, picks, renorm, ties):
    # against the stage calls: the same picks, and from them the same sums, bit for bit.  Budgets of 0 to k_max, and of
    # outside of that, which the status reports; ties: logits of two values, so that the picks are the lowest ids
    g = torch.Generator(device="cuda").manual_seed(T * E + d)
    shape = B.make_shape(T, d, E, 1, Is, k_max, dtype, renorm, 1.5)
    dt, bits = (torch.bfloat16, torch.int16) if dtype == "bf16" else (torch.float32, torch.int32)

    def normal(*size, std):
        return torch.empty(size, dtype=dt, device="cuda").normal_(0.0, std, generator=g)
    x, w_r, w_gu, w_dn = normal(T, d, std=1.0), normal(E, d, std=0.02), normal(E, 2 * Is, d, std=0.05), normal(E, d, Is, std=0.05)
    bias = torch.empty(E, device="cuda").normal_(generator=g)
    if ties:
        w_r.zero_()
        bias = (bias > 0).float()
    ws = B.alloc_workspace(shape)
    for budgets in ([k_max] * T, [k_max // 2] * T, [0] * T, torch.randint(-2, k_max + 3, (T,), generator=g, device="cuda").tolist()):
        k = torch.tensor(budgets, dtype=torch.int32, device="cuda")
        ws.fill_(255)
        B.moe_prism_timing_enable(True)
        try:
            out = B.moe_prism_layer(shape, x, w_r, bias, k, w_gu, w_dn, ws).clone()
            torch.cuda.synchronize()
            assert (B.moe_prism_timing_read()["topk"][1] == 0) == bool(picks)
        finally:
            B.moe_prism_timing_enable(False)
        status = B.moe_prism_status(ws)
        ids, wt, _ = B.moe_prism_route(shape, x, w_r, bias, k, ws, want_logits=True)
        assert status[0] == B.moe_prism_status(ws)[0] == int(any(b < 0 or b > k_max for b in budgets))
        _, off, sp, sl = B.moe_prism_dispatch(shape, ids, ws)
        assert status[1] == B.moe_prism_status(ws)[1] == int(off[-1])
        y = B.moe_prism_grouped_ffn(shape, x, w_gu, w_dn, off, sp, ws)
        ref = B.moe_prism_combine(shape, y, sl, wt, k)
        assert torch.equal(out.view(bits), ref.view(bits))


@pytest.mark.parametrize("T,N,S,k_max,d,Is", [
    (1, 128, 4, 32, 2048, 192), (37, 128, 4, 32, 2048, 192), (600, 128, 4, 4, 1600, 64),  # 8 columns; more rows than threads
    (17, 3, 1, 2, 1984, 320), (5, 8, 4, 8, 4096, 608), (48, 128, 4, 32, 3136, 192),       # 16 columns, four stages and three
    (80, 128, 4, 32, 2048, 192)])                                                         # the combine's own kernel
def test_layer_leaves_y_where_its_offsets_say(T, N, S, k_max, d, Is):
    # against the stage calls' y, bit for bit, whichever kernel adds up the picks; rows beyond the pairs are not written
    g = torch.Generator(device="cuda").manual_seed(T + d)
    E = N * S
    shape = B.make_shape(T, d, N, S, Is, k_max, "bf16", 1, 1.0)

    def normal(*size, std):
        return torch.empty(size, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, w_r, w_gu, w_dn = normal(T, d, std=1.0), normal(E, d, std=0.02), normal(E, 2 * Is, d, std=0.05), normal(E, d, Is, std=0.05)
    k = torch.randint(0, k_max + 1, (T,), generator=g, device="cuda", dtype=torch.int32)
    k[0] = k_max - 1 if k_max > 1 else 1
    ws = B.alloc_workspace(shape)
    ws.fill_(255)
    B.moe_prism_layer(shape, x, w_r, None, k, w_gu, w_dn, ws)
    at = B.moe_prism_layer_offsets(shape)["y"]
    y = ws[at:at + T * k_max * d * 2].view(torch.int16).view(T * k_max, d).clone()
    other = B.alloc_workspace(shape)
    ids, _, _ = B.moe_prism_route(shape, x, w_r, None, k, other, want_logits=True)
    _, off, sp, _ = B.moe_prism_dispatch(shape, ids, other)
    ref = B.moe_prism_grouped_ffn(shape, x, w_gu, w_dn, off, sp, other)
    P = int(off[-1])
    assert 0 < P < T * k_max
    assert torch.equal(y[:P], ref[:P].view(torch.int16))
    assert (y[P:] == -1).all()


@pytest.mark.parametrize("dtype,T,E,k_max,d,Is", [
    ("bf16", 1, 1, 1, 64, 32), ("bf16", 2, 65, 7, 448, 96), ("bf16", 4, 129, 40, 1088, 64), ("bf16", 1, 512, 32, 2048, 192), ("bf16", 4, 512, 64, 1024, 128),
    ("f32", 1, 1, 1, 64, 32), ("f32", 2, 5, 5, 128, 96), ("f32", 33, 31, 7, 192, 64), ("f32", 64, 32, 8, 256, 128), ("f32", 64, 32, 32, 64, 32)])
def test_gate_up_that_picks_leaves_the_tables_of_route_and_dispatch(dtype, T, E, k_max, d, Is):
    # every table of the layer's workspace against the stage calls', behind a workspace of 0xff; budgets of 0 to k_max
    g = torch.Generator(device="cuda").manual_seed(T + E + d)
    shape = B.make_shape(T, d, E, 1, Is, k_max, dtype, 1, 1.5)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def normal(*size, std):
        return torch.empty(size, dtype=dt, device="cuda").normal_(0.0, std, generator=g)
    x, w_r, w_gu, w_dn = normal(T, d, std=1.0), normal(E, d, std=0.02), normal(E, 2 * Is, d, std=0.05), normal(E, d, Is, std=0.05)
    k = torch.randint(0, k_max + 1, (T,), generator=g, device="cuda", dtype=torch.int32)
    k[0] = k_max
    ws, other = B.alloc_workspace(shape), B.alloc_workspace(shape)
    ws.fill_(255)
    B.moe_prism_timing_enable(True)
    try:
        B.moe_prism_layer(shape, x, w_r, None, k, w_gu, w_dn, ws)
        torch.cuda.synchronize()
        assert B.moe_prism_timing_read()["topk"][1] == 0
    finally:
        B.moe_prism_timing_enable(False)
    ids, wt, lg = B.moe_prism_route(shape, x, w_r, None, k, other, want_logits=True)
    cnt, off, sp, sl = B.moe_prism_dispatch(shape, ids, other)
    ref = dict(topk_ids=ids, topk_w=wt, group_count=cnt, group_offset=off, sorted_pair=sp, slot_of_pair=sl, logits=lg)
    for name, table in B.layer_intermediates(shape, ws).items():
        assert torch.equal(table.view(torch.int32), ref[name].view(torch.int32)), name


@pytest.mark.parametrize("Is", [32, 64, 96, 128, 160, 192, 224, 256])
@pytest.mark.parametrize("T", [1, 9, 50])
def test_down_projection_and_combine_of_every_count_of_stages(T, Is):
    test_down_projection_and_combine_in_one_kernel(T, 32, 4, 9, 1728, Is, 1)


@pytest.mark.parametrize("T,N,S,k_max,d,Is,combines", [
    (65, 64, 4, 12, 2048, 704, 1), (67, 64, 4, 12, 2048, 704, 0),    # 560 000 elements of h with columns for every CU
    (43, 64, 4, 12, 1536, 192, 1), (44, 64, 4, 12, 1536, 192, 0),    # 100 000 with columns for three quarters
    (83, 64, 4, 12, 3072, 320, 0), (78, 64, 4, 12, 3072, 320, 1),    # 300 000 in 16 columns
    (16, 64, 4, 12, 2048, 608, 1), (17, 64, 4, 12, 2048, 608, 0),    # half a stage
    (6, 64, 4, 12, 1536, 608, 1), (7, 64, 4, 12, 1536, 608, 0), (64, 64, 4, 12, 1536, 224, 1)])
def test_down_projection_and_combine_on_both_sides_of_what_it_reads(T, N, S, k_max, d, Is, combines):
    test_down_projection_and_combine_in_one_kernel(T, N, S, k_max, d, Is, combines)


@pytest.mark.parametrize("T,E,k_max,d,Is,picks", [
    (64, 2, 2, 128, 32, 1), (64, 1, 1, 64, 64, 1), (50, 3, 2, 192, 96, 1),  # fewer tiles than XCDs
    (64, 8, 4, 64, 992, 1), (64, 8, 4, 64, 1024, 1), (64, 8, 5, 64, 992, 1), (64, 8, 5, 64, 1024, 0), (64, 32, 32, 64, 256, 0), (33, 16, 2, 64, 1024, 0)])
def test_gate_up_that_picks_and_the_workgroups_that_write(T, E, k_max, d, Is, picks):
    # fp32: as many tiles as workgroups fit, and room for those that write
    test_gate_up_that_picks_for_itself("f32", T, E, k_max, d, Is, picks, 1, False)
