"""Feature maps some of whose output channels are switched off by a bias that stands for minus infinity (for degree 2, the first
or the last half: a whole slice), under the softmax activation: such a channel's feature is zero and nothing else changes, so a channel
softmax that is put together from parts (pairs of tiles, tiles, blocks of 128 channels) must not form its exponentials
against a maximum that is such a value.

From -1e9 down exp(u - max) is zero in float64 as well, so one reference serves all values.  Tolerance: the bars of
test_gpu_parity.py and test_gpu_value_distill_grad.py."""
import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from oracle import value_distill_grad_oracle as G
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_gpu_parity import MAX_ABS, REL_L2, ROW_REL_L2, gpu_forward, metrics, oracle_map, record, worst_row
from test_gpu_value_distill_grad import GRAD_REL_L2, bf16_representable, compare, oracle_forward_pieces, round_io

pytestmark = pytest.mark.gpu

VALUES = (-np.inf, float(np.finfo(np.float32).min), -1e30, -1e20, -1e10, -1e9)
CHANNELS = {
    "first_half": lambda F: slice(0, F // 2),
    "last_half": lambda F: slice(F // 2, F),
    "first_32": lambda F: slice(0, 32),
    "second_quarter_and_last_16": lambda F: np.r_[F // 4:F // 2, F - 16:F],
}


def work(name, d, width, H, N, R, **kw):
    return W.Workload(name, 1, H, N, d, kw.pop("dtype", "bf16"), 128, R, kw.pop("hidden", width), width, seed=N + width, **kw)


PATHS = (
    work("one_wave_per_simd", 128, 128, 6, 131, 2), work("linear_pass", 128, 128, 2, 300, 4), work("rate_0", 128, 128, 6, 300, 0),
    work("large_tiles", 128, 128, 96, 300, 4), work("f32", 128, 128, 6, 131, 4, dtype="f32"), work("d64", 64, 64, 3, 300, 4),
    work("chunk_causal_128", 128, 128, 2, 600, 4, causal_chunk=256), work("phi256", 128, 256, 2, 300, 4),
    work("chunk_causal_256", 128, 256, 2, 600, 4, causal_chunk=256), work("phi384", 128, 384, 1, 300, 2, poly_degree=3),
    work("phi512", 128, 512, 2, 200, 2, hidden=128), work("phi768x3", 128, 768, 1, 300, 4, d_mid=768),
    work("phi512_rounds", 128, 512, 40, 700, 0, hidden=128),
)


@pytest.mark.parametrize("w", PATHS, ids=lambda w: w.name)
@pytest.mark.parametrize("channels", sorted(CHANNELS))
def test_forward_with_masked_channels(w, channels):
    inp = W.make_inputs(w)
    off = CHANNELS[channels](w.d_feat)
    rows = np.arange(0, w.N, 97) if w.H * w.N > 10000 else np.arange(w.N)
    for side in ("phi_q", "phi_k"):
        p = getattr(inp, side)
        kept = p.b2.copy()
        p.b2[:, off] = -np.inf
        maps = oracle_map(inp.phi_q), oracle_map(inp.phi_k)
        if w.causal_chunk:
            ref = O.hybrid_attn_chunk_causal(inp.q, inp.k, inp.v, *maps, w.R, w.scale, w.causal_chunk, rows=rows)
        else:
            ref = O.hybrid_attn(inp.q, inp.k, inp.v, *maps, w.R, w.scale, rows=rows)
        for value in VALUES:
            p.b2[:, off] = value
            print(f"  case {w.name} {channels} {side} {value}", flush=True)
            y = gpu_forward(inp, R=w.rate)[:, :, rows]
            assert np.isfinite(y).all(), f"{side} {value}: non-finite output"
            ma, rl = metrics(y, ref)
            wr, _ = worst_row(y, ref)
            record(f"masked_{w.name}_{channels}_{side}_{value}", ma, rl, row_rel_l2=wr)
            assert ma <= MAX_ABS and rl <= REL_L2 and wr <= ROW_REL_L2, (side, value, ma, rl, wr)
        p.b2[...] = kept


@pytest.mark.parametrize("width,d_mid", ((64, 0), (128, 0), (256, 0), (384, 0), (512, 128)))
@pytest.mark.parametrize("channels", sorted(CHANNELS))
def test_gradient_with_masked_channels(width, d_mid, channels):
    d = min(width, 128)
    w = work(f"masked_grad_{width}", d, width, 2, 413, 4, d_mid=d_mid, hidden=128 if width == 512 else width)
    inp = bf16_representable(W.make_inputs(w))
    off = CHANNELS[channels](width)
    for p in (inp.phi_q, inp.phi_k):
        p.b2[:, off] = -np.inf
    fq, fk, y, yh, den = oracle_forward_pieces(inp, w.R)
    y_r, yh_r = round_io(y, w.dtype), round_io(yh, w.dtype)
    want = G.value_distill_grad(inp.q, inp.k, inp.v, fq, fk, w.R, w.scale, sign_from=(y_r, yh_r))
    yt, ys = (torch.from_numpy(t).to(device="cuda", dtype=torch.bfloat16).contiguous() for t in (y_r, yh_r))
    rd = torch.from_numpy(den).to(device="cuda", dtype=torch.float32).contiguous()
    for value in VALUES[:3]:
        for p in (inp.phi_q, inp.phi_k):
            p.b2[:, off] = value
        q, k, v, dq, dk = ha.to_device(inp)
        print(f"  case {w.name} {channels} {value}", flush=True)
        _, gq, gk, _, _, _ = ha.hybrid_attn_value_distill_grad(q, k, v, dq, dk, w.R, w.block_size, w.scale, y_teacher=yt,
                                                               teacher_is_cached=True, y_student=ys, row_den=rd, student_is_cached=True)
        torch.cuda.synchronize()
        assert compare(f"{w.name}_{channels}_{value}", (gq, gk), want) <= GRAD_REL_L2
