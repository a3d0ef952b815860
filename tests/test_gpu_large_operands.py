"""Operands and tiles of 4 GiB and more, where byte offsets need 64 bits."""
import pytest
import torch

from paper_2510_19366_amd import binding as B

pytestmark = pytest.mark.gpu


def reference(x, w_gu, w_dn, cols):
    """Rows x through one sub-expert in fp64, the columns `cols`, in slices of the weights."""
    Is, d = w_gu.shape[0] // 2, x.shape[1]
    rows, deep = 1024, 1 << 20
    h = torch.zeros(x.shape[0], Is, dtype=torch.float64, device="cuda")
    for i in range(0, Is, rows):
        n = min(rows, Is - i)
        v = torch.zeros(x.shape[0], 2 * n, dtype=torch.float64, device="cuda")
        for k in range(0, d, deep):
            s = slice(k, k + deep)
            v += x[:, s].double() @ torch.cat([w_gu[i:i + n, s], w_gu[Is + i:Is + i + n, s]]).double().T
        h[:, i:i + n] = v[:, :n] / (1 + torch.exp(-v[:, :n])) * v[:, n:]
    y = torch.zeros(x.shape[0], len(cols), dtype=torch.float64, device="cuda")
    for i in range(0, Is, 8192):
        y += h[:, i:i + 8192] @ w_dn[cols, i:i + 8192].double().T
    return y


@pytest.mark.parametrize("dtype,T,E,d,Is", [
    ("bf16", 32900, 3, 65536, 256),   # activations
    ("bf16", 270, 1, 65536, 16384),   # gate-up weights of one sub-expert
    ("bf16", 70, 1, 65536, 32800),    # both weights, half a K stage in the down projection
    ("bf16", 257, 1, 1 << 23, 32),    # activations and a tile of outputs, short K in the down projection
    ("f32", 65700, 2, 16384, 32),
    ("f32", 40, 1, 65536, 16384),
    ("f32", 70, 1, 65536, 16384),
])
def test_ffn_offsets_beyond_32_bits(dtype, T, E, d, Is):
    torch.cuda.empty_cache()
    g = torch.Generator(device="cuda").manual_seed(d + Is)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32

    def rand(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=dt)

    x, w_gu, w_dn = rand(T, d), rand(E, 2 * Is, d).mul_(d ** -0.5), rand(E, d, Is).mul_(Is ** -0.5)
    assert max(x.nbytes, w_gu[0].nbytes, w_dn[0].nbytes) >= 1 << 32
    ids = torch.randint(0, E, (T, 1), generator=g, device="cuda", dtype=torch.int32)
    shape = B.make_shape(T, d, E, 1, Is, 1, dtype)
    ws = B.alloc_workspace(shape)
    _, off, sp, sl = B.moe_prism_dispatch(shape, ids, ws)
    y = B.moe_prism_grouped_ffn(shape, x, w_gu, w_dn, off, sp, ws)
    pick = torch.cat([torch.arange(0, T, max(1, T // 40), device="cuda"), torch.arange(T - 20, T, device="cuda")])
    cols = torch.unique(torch.cat([torch.arange(0, d, max(1, d // 1500)), torch.arange(d - 64, d)])).cuda()
    for e in range(E):
        t = pick[ids[pick, 0] == e]
        ref = reference(x[t], w_gu[e], w_dn[e], cols)
        err = (y[sl[t].long()][:, cols].double() - ref).norm(dim=1) / ref.norm(dim=1)
        # bf16: h and y are rounded once each, 2^-9 at most; fp32: two chains of up to n roundings of 2^-24
        assert err.max() <= (2 * 2.0 ** -9 if dtype == "bf16" else 2 * max(d, Is) * 2.0 ** -24), (e, int(err.argmax()))
