"""More heads than a grid's second dimension takes beside the (batch, head) pairs: launches that serve the rows of both (weights of every
head, keys or states of every pair) are split or laid out in one dimension there.  test_launch_limits.py holds every launch to the device's limits on
the host; here the split launches' results are compared with the oracle at the first, the last and the heads around the borders.

Tolerance: the bars of test_gpu_parity.py and test_gpu_value_distill_grad.py."""
import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from oracle import value_distill_grad_oracle as G
from paper_2509_24899_amd import hybrid_attn as ha
from tests.test_gpu_value_distill_grad import GRAD_REL_L2

pytestmark = pytest.mark.gpu


def draw(H, N, d, width, dtype):
    gen = torch.Generator(device="cuda").manual_seed(H)
    # (fp32 values that bf16 holds: both sides then take the ReLU's gates on the same numbers)
    normal = lambda std, *shape: (torch.randn(*shape, generator=gen, device="cuda", dtype=torch.bfloat16) * std).to(dtype)
    maps = [ha.FeatureMap(normal(d ** -0.5, H, width, d), normal(0.1, H, width).float(), normal(width ** -0.5, H, width, width),
                          normal(0.1, H, width).float(), 2) for _ in range(2)]
    return [normal(1.0, 1, H, N, d) for _ in range(3)] + maps


def of_heads(heads, *tensors):
    return [t[:, heads].double().cpu().numpy() for t in tensors]


def oracle_map_of(heads, m):
    return O.FeatureMap(*(t[heads].double().cpu().numpy() for t in (m.w1, m.b1, m.w2, m.b2)), 2)


def test_forward_with_prepared_weights():
    H, N, R = 33000, 7, 2                          # fp32: compaction and weights in one launch, reduction and weights in another
    heads = [0, 1, H - 1, 65535 - H, 65536 - H]
    q, k, v, fq, fk = draw(H, N, 128, 128, torch.float32)
    out = ha.hybrid_attn_forward(q, k, v, fq, fk, R)
    torch.cuda.synchronize()
    want = O.hybrid_attn(*of_heads(heads, q, k, v), oracle_map_of(heads, fq), oracle_map_of(heads, fk), R, 128 ** -0.5)
    got, = of_heads(heads, out)
    assert np.isfinite(got).all() and np.linalg.norm(got - want) <= 5e-3 * np.linalg.norm(want)
    del q, k, v, fq, fk, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("H,width", ((13200, 128), (21900, 256)))
def test_gradient(H, width):
    N, R = 7, 2
    q, k, v, fq, fk = draw(H, N, 128, width, torch.bfloat16)
    heads = [0, 1, H - 2, H - 1, 65535 % H, (65535 + 1) % H]
    _, gq, gk, yt, ys, _ = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, R)
    torch.cuda.synchronize()
    want = G.value_distill_grad(*of_heads(heads, q, k, v), oracle_map_of(heads, fq), oracle_map_of(heads, fk), R, 128 ** -0.5,
                                sign_from=of_heads(heads, yt, ys))
    for got, exact in ((gq, want[0]), (gk, want[1])):
        for n in exact:
            a = got[n][heads].double().cpu().numpy()
            assert np.isfinite(a).all() and np.linalg.norm(a - exact[n]) <= GRAD_REL_L2 * np.linalg.norm(exact[n]), n
    del q, k, v, fq, fk, gq, gk, yt, ys
    torch.cuda.empty_cache()
