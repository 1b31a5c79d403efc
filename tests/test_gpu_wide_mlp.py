"""The streaming layer kernel of the wide feature maps, through the forward (the gradient suites cover the images it keeps
for the backward pass): widths with and
without a block of four output tiles, shortest and longest contraction, two and three layers, token counts around the
256-token tile and the last idle waves, more heads than a workgroup's run, both dtypes.

Tolerance: the bars of test_gpu_parity.py."""
import numpy as np
import pytest
import torch
import torch

from paper_2509_24899_amd import workloads as W
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


def work(N, hid, feat, mid=0, P=2, H=2, B=1, R=3, dtype="bf16", seed=0):
    return W.Workload(f"wm_{hid}_{mid}_{feat}_N{N}_H{H}_{dtype}", B, H, N, 128, dtype, 128, R, hid, feat, poly_degree=P, d_mid=mid, seed=seed)


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("hid,feat,mid,P", ((128, 384, 0, 3), (768, 128, 0, 2), (384, 640, 0, 4), (256, 512, 0, 4),
                                            (128, 128, 128, 2), (640, 768, 384, 6), (768, 768, 768, 6)))
def test_widths(hid, feat, mid, P, dtype):
    check("wm", W.make_inputs(work(333, hid, feat, mid, P, dtype=dtype, seed=hid + feat)))


@pytest.mark.parametrize("N", (1, 32, 255, 256, 257, 289, 2049))
@pytest.mark.parametrize("mid", (0, 256))
def test_token_counts(N, mid):
    w = work(N, 384, 384, mid, 3, R=0 if N == 1 else 4 if N > 4 else 2, seed=N)
    check(w.name, W.make_inputs(w), rows=W.sample_rows(w, n_random=16) if N > 600 else None)


def test_many_heads():
    w = work(300, 384, 512, 256, 4, H=60, B=3, R=2, seed=9)
    check(w.name, W.make_inputs(w), rows=np.arange(0, 300, 7))


# Work items (256 tokens x 256 channels) around whole rounds of 256: 258 = a round and two items halved (three layers: from x and
# from HBM), 288 and 264 with more of them, 180 (one round, not halved), 270 + 135 (odd multiple of 128: blocks of four throughout)
@pytest.mark.parametrize("B,H,N,hid,feat,mid,R", ((1, 3, 10808, 512, 512, 512, 0), (2, 12, 789, 768, 768, 768, 4), (1, 12, 5503, 384, 256, 0, 8),
                                                  (1, 3, 5000, 768, 768, 0, 4), (1, 3, 11400, 640, 640, 0, 0)))
@pytest.mark.parametrize("dtype", ("bf16", "f32"))
def test_items_beyond_whole_rounds(B, H, N, hid, feat, mid, R, dtype):
    w = work(N, hid, feat, mid, {256: 2, 512: 4, 640: 4, 768: 6}[feat], H=H, B=B, R=R, dtype=dtype, seed=N)
    check(w.name, W.make_inputs(w), rows=np.unique(np.r_[0, 255, 256, N // 2, N - 257:N - 255, N - 1]))


def test_hidden_image_of_halved_items():
    """The backward pass of the 256-wide maps reads the first hidden layer as the layer kernel left it: 264 items for twelve
    heads (eight of them halved) against 22 for one head on its own (blocks of four throughout): the same gradients up to the order
    of fp32 sums (other chunks of tokens; the bar of the headline gradient test)."""
    from paper_2509_24899_amd import hybrid_attn as ha
    w = work(5503, 256, 256, H=12, R=4, seed=5)
    q, k, v, fq, fk = ha.device_inputs(w)

    def grads(a, b):
        def sl(m):
            return ha.FeatureMap(*(t[a:b].contiguous() for t in (m.w1, m.b1, m.w2, m.b2)), m.poly_degree)
        yt = torch.zeros_like(q[:, a:b])
        return ha.hybrid_attn_value_distill_grad(q[:, a:b], k[:, a:b], v[:, a:b], sl(fq), sl(fk), 4, 128, w.scale, y_teacher=yt, teacher_is_cached=True)[1:3]
    every = grads(0, 12)
    for h in (0, 7, 11):
        for m, one in zip(every, grads(h, h + 1)):
            for n in one:
                x, y = m[n][h].double(), one[n][0].double()
                assert float((x - y).norm() / y.norm()) <= 1e-4, (h, n)


def test_a_second_round_of_small_items_is_not_taken():
    """768-wide maps, one head: 40 tiles of tokens are 240 items with blocks of four output tiles, one round on 256 CUs (168 us).
    44 tiles are 264 of them, a second round (236 us, 1.41 times as long), or 132 with blocks of eight (202 us, 1.20).  The medians
    of one process are compared; the line lies halfway."""
    from paper_2509_24899_amd import hybrid_attn as ha
    times = []
    for N in (10232, 11256):
        w = work(N, 768, 768, H=1, R=0, seed=1)
        q, k, v, fq, fk = ha.device_inputs(w)
        out = torch.empty_like(q)
        ws = torch.empty(ha.hybrid_attn_workspace_bytes(ha.make_problem(q, 0, 128, w.scale), fq, fk), dtype=torch.uint8, device="cuda")
        ms = []
        for i in range(25):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(8):
                ha.hybrid_attn_forward(q, k, v, fq, fk, 0, 128, w.scale, out=out, workspace=ws)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b))
        times.append(float(np.median(ms[5:])))
    assert times[1] < 1.305 * times[0], times
