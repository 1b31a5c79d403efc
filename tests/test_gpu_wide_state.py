"""State pass of the wide feature maps: 256 and 128 features per workgroup, every activation and several degrees (slices that do and
do not end with a 32-channel block), numbers of linear tokens around its 64-token tiles, 32-token blocks and 128-token chunks, fewer chunks than
chiplets and more, both dtypes and layouts, through the forward.

Tolerance: the bars of test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


def work(N, hid, feat, P, H=1, B=1, R=2, dtype="bf16", seed=0):
    return W.Workload(f"ws_{hid}_{feat}_N{N}_H{H}_{dtype}", B, H, N, 128, dtype, 128, R, hid, feat, poly_degree=P, seed=seed)


@pytest.mark.parametrize("n_linear", (1, 31, 33, 64, 65, 127, 129, 193))
@pytest.mark.parametrize("feat,P", ((512, 4), (384, 3)))
def test_numbers_of_linear_tokens(n_linear, feat, P):
    check("ws", W.make_inputs(work(2 * n_linear, 128, feat, P, H=2, seed=n_linear)))


@pytest.mark.parametrize("act", (ha.HA_ACT_SOFTMAX, ha.HA_ACT_EXP, ha.HA_ACT_RELU))
@pytest.mark.parametrize("feat,P", ((512, 8), (768, 1), (640, 2), (384, 8)))
@pytest.mark.parametrize("dtype", ("bf16", "f32"))
def test_activations_and_degrees(act, feat, P, dtype):
    check("ws_act", W.make_inputs(work(277, 256, feat, P, H=3, R=3, dtype=dtype, seed=feat + P)), act=act, layout="bnhd")


def test_more_chunks_than_chiplets():
    w = work(3000, 128, 512, 2, H=5, B=2, R=4, seed=3)
    check(w.name, W.make_inputs(w), rows=np.arange(0, 3000, 211))


@pytest.mark.parametrize("feat,P,H,dtype", ((768, 6, 64, "bf16"), (640, 2, 80, "f32")))   # eight and four row blocks per workgroup
def test_pre_activations_beyond_the_memory_side_cache(feat, P, H, dtype):
    w = work(1000, 128, feat, P, H=H, B=2, R=16, dtype=dtype, seed=feat)                   # 872 linear tokens: both sides
    assert w.B * w.H * 872 * feat * 4 > 320 << 20
    check(w.name, W.make_inputs(w), rows=np.arange(0, 1000, 97))
