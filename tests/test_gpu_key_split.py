"""Problems of few query tiles split the softmax keys into ranges whose partial sums a second pass merges: every form of
that pass (rate 1, precomputed linear part of the 128-wide, 256-wide and wider maps; two to eight ranges) against the fp64
oracle, with ragged last ranges, rows and tiles, a maximum that sits in any one range, ranges without weight, the denominators
of the gradient call, and equal bits with the fixed workspace and for either block size.  That the shapes of SPLIT_SHAPES are
split is checked on the host (test_abi_host.py); test_ranges, test_row_denominators and test_one_key_far_above_the_others
run just outside the rule, in one range.

Tolerance: the bars of test_gpu_parity.py; row denominators 4e-3 relative (weights and features are rounded to bf16, 2^-9 at
most twice)."""
import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_abi_host import SPLIT_SHAPES
from test_gpu_parity import check, oracle_map

pytestmark = pytest.mark.gpu


def work(N, R, width=128, B=1, H=2, dtype="bf16", seed=0, gain=1.0):
    P = {128: 2, 256: 2, 384: 3}[width]
    return W.Workload(f"ks_R{R}_F{width}_N{N}_B{B}H{H}_{dtype}", B, H, N, 128, dtype, 128, R, width, width, poly_degree=P, seed=seed, qk_gain=gain)


# (key blocks of 32 from a few per range to uneven ranges; the last block and the last tile ragged)
@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("width", (128, 256, 384))
@pytest.mark.parametrize("N,R", ((1560, 4), (700, 1), (2049, 2), (3001, 3), (1025, 1)))
def test_ranges(N, R, width, dtype):
    w = work(N, R, width, H=3, dtype=dtype, seed=N, gain=128 ** 0.5)
    rows = W.sample_rows(w, n_random=32)
    y64, _ = check(w.name, W.make_inputs(w), block_size=64, rows=rows)
    y128, _ = check(w.name, W.make_inputs(w), block_size=128, rows=rows)
    assert np.array_equal(y64, y128)


@pytest.mark.parametrize("at", (0, 700, 1996))
def test_one_key_far_above_the_others(at):
    """Its range holds the maximum of every row that points its way: the other ranges' sums shrink to nothing."""
    w = work(2000, 4, seed=3, gain=128 ** 0.5)
    inp = W.make_inputs(w)
    inp.k[:, :, at - at % 4] *= 8.0
    inp.k[:] = W.round_to_bf16(inp.k)
    check(f"ks_peak_{at}", inp, rows=W.sample_rows(w, n_random=64))


@pytest.mark.parametrize("lo,hi", ((0.0, 0.5), (0.3, 0.7), (0.6, 1.0)))
@pytest.mark.parametrize("N,R,width,dtype", ((2000, 1, 128, "bf16"), (2000, 1, 128, "f32"), (20000, 4, 128, "bf16"), (20000, 4, 256, "bf16"), (20000, 4, 384, "f32")))
def test_ranges_whose_every_logit_is_minus_infinity(N, R, width, dtype, lo, hi):
    """Keys masked with values whose products with the queries overflow to -inf, whole ranges of them: weight zero, as in
    one range."""
    w = work(N, R, width, H=1, dtype=dtype, seed=N + R, gain=128 ** 0.5)
    inp = W.make_inputs(w)
    inp.q[:] = W.round_to_bf16(np.abs(inp.q) + 1)
    a, b = (int(x * N) // R * R for x in (lo, hi))
    inp.k[:, :, a:b:R] = W.round_to_bf16(np.float32([-3e38]))[0]
    check(f"ks_masked_N{N}_R{R}_F{width}_{a}_{b}", inp, rows=np.arange(0, N, N // 40))


@pytest.mark.parametrize("width", (128, 256))
def test_row_denominators(width):
    inp = W.make_inputs(work(1500, 2, width, seed=6, gain=128 ** 0.5))
    w = inp.workload
    q, k, v, fq, fk = ha.to_device(inp)
    _, _, _, _, y, den = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, 2, 128, w.scale, y_teacher=torch.zeros_like(q), teacher_is_cached=True)
    torch.cuda.synchronize()
    assert torch.equal(ha.hybrid_attn_forward(q, k, v, fq, fk, 2, 128, w.scale), y)
    for h in range(w.H):
        _, z = O.linear_state(inp.k[0, h], inp.v[0, h], oracle_map(inp.phi_k), h, 2)
        _, l, _ = O.softmax_part(np.asarray(inp.q[0, h], np.float64), inp.k[0, h], inp.v[0, h], 2, w.scale)
        ref = l + O.feature_map(inp.q[0, h], oracle_map(inp.phi_q), h) @ z
        assert np.abs(den[0, h].double().cpu().numpy() / ref - 1).max() <= 4e-3     # (exp of a rounded logit: 2^-9 at most twice)


@pytest.mark.parametrize("H", (5, 6))                  # five heads: linear part ahead of the query kernel; six: in its epilogue
@pytest.mark.parametrize("N,P,act", ((1, 2, 0), (33, 1, 0), (257, 4, 0), (6528, 2, 0), (6529, 2, 0), (300, 8, 1), (300, 2, 2)))
def test_linear_part_of_the_narrow_maps(N, P, act, H):
    """51 and 52 tiles of 128 queries per head: the border of the rule at five heads."""
    w = W.replace(work(N, 4 if N > 4 else 0, H=H, seed=N), poly_degree=P)
    check(f"ks_lin128_H{H}_N{N}_P{P}_a{act}", W.make_inputs(w), act=act, rows=W.sample_rows(w, n_random=16) if N > 600 else None)


@pytest.mark.parametrize("B,H,N,R,width", ((1, 12, 1560, 4, 128), (1, 1, 20000, 2, 256), (1, 2, 12000, 4, 256), (1, 2, 16000, 1, 128)))
def test_fixed_workspace_gives_the_same_bits(B, H, N, R, width):
    w = work(N, R, width, B, H, seed=N)
    q, k, v, fq, fk = ha.to_device(W.make_inputs(w))
    maps = (None, None) if R == 1 else (fq, fk)
    ref = ha.hybrid_attn_forward(q, k, v, *maps, R, 128, w.scale)
    out = torch.full_like(q, float("nan"))
    ha.hybrid_attn_forward_static(q, k, v, *maps, R, out, 128, w.scale)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


@pytest.mark.parametrize("N,R,width", ((15362, 2, 128), (15488, 2, 128), (7000, 2, 384), (6402, 2, 384)))
def test_block_sizes_agree_where_the_fixed_workspace_ends(N, R, width):
    w = work(N, R, width, seed=N)
    q, k, v, fq, fk = ha.to_device(W.make_inputs(w))
    a, b = (ha.hybrid_attn_forward(q, k, v, fq, fk, R, bs, w.scale) for bs in (64, 128))
    outs = [b]
    for bs in (64, 128):
        try:
            outs.append(ha.hybrid_attn_forward_static(q, k, v, fq, fk, R, torch.full_like(q, float("nan")), bs, w.scale))
        except ha.HybridAttnError as e:
            assert e.status == ha.HA_ERR_WORKSPACE
    torch.cuda.synchronize()
    for other in outs:
        assert torch.equal(a, other)


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("N,R,width,H", SPLIT_SHAPES)
def test_split_shapes(N, R, width, H, dtype):
    w = work(N, R, width, H=H, dtype=dtype, seed=N + R, gain=128 ** 0.5)
    rows = np.unique(np.r_[0:3, 31, 32, 255, 256, np.linspace(0, N - 1, 24).astype(int), N - 34:N])
    inp = W.make_inputs(w)
    y64, _ = check(w.name + "_bs64", inp, block_size=64, rows=rows)
    y128, _ = check(w.name + "_bs128", inp, block_size=128, rows=rows)
    assert np.array_equal(y64, y128)


@pytest.mark.parametrize("at", (0.0, 0.27, 0.5, 0.81, 1.0))
@pytest.mark.parametrize("N,R,width,H", [s for s in SPLIT_SHAPES if s in ((3001, 1, 128, 1), (8321, 2, 128, 1), (6003, 2, 256, 1), (3001, 2, 384, 1))])
def test_the_maximum_in_one_range(N, R, width, H, at):
    """One key far above the others, in the first, a middle or the last range."""
    w = work(N, R, width, H=H, seed=3, gain=128 ** 0.5)
    inp = W.make_inputs(w)
    key = int(at * (N - 1)) // R * R
    inp.k[:, :, key] = W.round_to_bf16(inp.k[:, :, key] * 8.0)
    check(f"{w.name}_peak_{key}", inp, rows=np.unique(np.linspace(0, N - 1, 40).astype(int)))


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("N,R,width,H", [s for s in SPLIT_SHAPES if s[1] > 1 and s[0] < 10000])
def test_denominators_of_split_shapes(N, R, width, H, dtype):
    inp = W.make_inputs(work(N, R, width, H=H, dtype=dtype, seed=6, gain=128 ** 0.5))
    w = inp.workload
    for owner, names in ((inp, ("q", "k", "v")), (inp.phi_q, ("w1", "w2")), (inp.phi_k, ("w1", "w2"))):
        for n in names:                     # (an fp32 call rounds these to bf16 on load: the same values on both sides)
            setattr(owner, n, W.round_to_bf16(getattr(owner, n)))
    q, k, v, fq, fk = ha.to_device(inp)
    _, _, _, _, y, den = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, R, 128, w.scale, y_teacher=torch.zeros_like(q), teacher_is_cached=True)
    torch.cuda.synchronize()
    assert torch.equal(ha.hybrid_attn_forward(q, k, v, fq, fk, R, 128, w.scale), y)
    rows = np.unique(np.r_[0, 255, 256, np.linspace(0, N - 1, 30).astype(int), N - 2, N - 1])
    for h in range(H):
        _, z = O.linear_state(inp.k[0, h], inp.v[0, h], oracle_map(inp.phi_k), h, R)
        qr = np.asarray(inp.q[0, h][rows], np.float64)
        _, l, _ = O.softmax_part(qr, inp.k[0, h], inp.v[0, h], R, w.scale)
        ref = l + O.feature_map(qr, oracle_map(inp.phi_q), h) @ z
        assert np.abs(den[0, h, rows].double().cpu().numpy() / ref - 1).max() <= 4e-3
