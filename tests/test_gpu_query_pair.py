"""Teacher and student of a distillation call in one launch of the query kernel: the same bits as one after the other, which a workspace too
small for both sets of keys brings about; on both sides of the rule's borders (sizes whose tilings differ, more than four rounds of
tiles), through the loss and through the gradient."""
import pytest
import torch

from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,H,N,R,dtype,pairs", (
    (128, 1, 12, 2900, 8, "bf16", True), (64, 1, 12, 2900, 4, "bf16", True), (64, 2, 8, 2500, 2, "f32", True),
    (128, 1, 11, 3001, 8, "f32", True), (64, 1, 11, 3001, 2, "bf16", True),        # 132 tiles: idle workgroups between the two problems
    (128, 1, 12, 9361, 8, "bf16", True), (128, 1, 9, 12001, 3, "f32", True),       # 444 and 423: the teacher's in more than one round
    (128, 2, 11, 3001, 3, "f32", False), (128, 1, 8, 32000, 16, "bf16", False), (128, 1, 8, 33000, 16, "bf16", False),
    (128, 1, 3, 700, 2, "bf16", False), (128, 1, 10, 6500, 2, "bf16", False)))
def test_same_bits_as_one_after_the_other(d, B, H, N, R, dtype, pairs):
    w = W.Workload(f"pair_d{d}_B{B}_H{H}_N{N}_R{R}_{dtype}", B, H, N, d, dtype, 64, R, d, d, seed=N)
    q, k, v, fq, fk = ha.device_inputs(w)
    print(f"  case {w.name}", flush=True)
    p = ha.make_problem(q, R, 64, w.scale)
    lib = ha._lib()
    (_, pq), (_, pk) = ha._fm_ptr(fq), ha._fm_ptr(fk)
    need = lib.hybrid_attn_value_distill_workspace_bytes(ha.ctypes.byref(p), pq, pk)
    least = max(ha.hybrid_attn_workspace_bytes(ha.make_problem(q, r, 64, w.scale), *m) for r, m in ((R, (fq, fk)), (1, (None, None))))
    least = (least + 255) // 256 * 256 + (B * H * 64 * 8 + 255) // 256 * 256          # and the partial sums of the loss
    assert (least < need) == pairs, "one launch" if pairs else "one after the other"
    got = []
    for size in (need, least):
        loss, yt, ys = ha.hybrid_attn_value_distill_loss(q, k, v, fq, fk, R, 64, w.scale,
                                                         workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        got.append((loss, yt, ys))
    teacher = ha.hybrid_attn_forward(q, k, v, None, None, 1, 64, w.scale)
    student = ha.hybrid_attn_forward(q, k, v, fq, fk, R, 64, w.scale)
    torch.cuda.synchronize()
    for loss, yt, ys in got:
        assert torch.equal(yt, teacher) and torch.equal(ys, student) and torch.equal(loss, got[0][0])
    with pytest.raises(ha.HybridAttnError):
        ha.hybrid_attn_value_distill_loss(q, k, v, fq, fk, R, 64, w.scale, workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))


def test_gradient_step_with_its_own_teacher():
    w = W.Workload("pair_step", 1, 12, 2900, 128, "bf16", 64, 4, 128, 128, seed=3)
    q, k, v, fq, fk = ha.device_inputs(w)
    loss, gq, gk, yt, ys, rd = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, 4, 64, w.scale)
    loss2, gq2, gk2, _, ys2, rd2 = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, 4, 64, w.scale, y_teacher=yt.clone(), teacher_is_cached=True)
    torch.cuda.synchronize()
    assert torch.equal(yt, ha.hybrid_attn_forward(q, k, v, None, None, 1, 64, w.scale))
    assert torch.equal(loss, loss2) and torch.equal(ys, ys2) and torch.equal(rd, rd2)
    for a, b in ((gq, gq2), (gk, gk2)):
        assert all(torch.equal(a[n], b[n]) for n in a)
