"""Combine: the wave per 64 column vectors that few tokens take and the workgroup per token of larger
batches, at the edges of both (columns beyond d, batches of rows, more than 64 picks), against a sum
in 64 bits and bit for bit against each other."""
import pytest
import torch

from paper_2510_19366_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,T,d,k_max", [
    ("bf16", 1, 64, 9), ("bf16", 3, 2048, 32), ("bf16", 5, 576, 17), ("bf16", 2, 512, 16), ("bf16", 9, 320, 66),
    ("bf16", 1, 64, 130), ("f32", 1, 64, 9), ("f32", 7, 320, 16), ("f32", 4, 256, 33), ("f32", 2, 576, 100),
])
def test_few_and_many_tokens(dtype, T, d, k_max):
    waves = -(-d // (64 * (8 if dtype == "bf16" else 4)))
    many_tokens = 8 * torch.cuda.get_device_properties(0).multi_processor_count // waves + 1  # a workgroup per token
    g = torch.Generator().manual_seed(d + k_max)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    n = many_tokens * k_max
    # slots of the first T tokens lie in the rows that a call with T tokens has
    slot = torch.cat([torch.randperm(T * k_max, generator=g), T * k_max + torch.randperm(n - T * k_max, generator=g)])
    slot[torch.rand(n, generator=g) < 0.1] = -1
    y = torch.randn(n, d, generator=g).to(dt)
    used = torch.zeros(n, dtype=torch.bool)
    used[slot[slot >= 0]] = True
    y[~used] = float("nan")  # a row without a pick is not part of any sum
    w = torch.rand(n, generator=g)
    k_tok = torch.randint(0, k_max + 1, (many_tokens,), generator=g, dtype=torch.int32)
    k_tok[0] = k_max + 5  # more than there are
    k_tok[T] = -2

    def combine(tokens):
        shape = B.make_shape(tokens, d, 256, 1, 32, k_max, dtype, 1, 1.0)
        m = tokens * k_max
        return B.moe_prism_combine(shape, y[:m].cuda(), slot[:m].to(torch.int32).cuda(), w[:m].cuda(),
                                   k_tok[:tokens].cuda()).cpu()

    many, few = combine(many_tokens), combine(T)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(few.view(bits), many[:T].view(bits))
    for t in range(T):
        kt = min(max(int(k_tok[t]), 0), k_max)
        s = slot[t * k_max:t * k_max + kt]
        rows = torch.where((s >= 0)[:, None], y[s.clamp(min=0)].double(), torch.zeros((), dtype=torch.float64))
        terms = rows * w[t * k_max:t * k_max + kt].double()[:, None]
        ref = terms.sum(0)
        bound = kt * 2.0 ** -24 * terms.abs().sum(0) + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0.0) + 1e-30
        assert ((few[t].double() - ref).abs() <= bound).all()
