"""The compiled marshalling of plain calls (csrc/ha_binding.cpp): it takes what is plain, with the results of the Python code, and leaves
everything else to that code, so that no check and no message is lost."""
import dataclasses

import pytest
import torch

from paper_2509_24899_amd import build
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W


def python_only(monkeypatch):
    monkeypatch.setattr(ha, "_BINDING", None)
    monkeypatch.setattr(ha, "_binding", lambda: False)


@pytest.mark.parametrize("fault", ("no compiler", "does not compile"))
def test_the_library_is_built_without_it(fault, monkeypatch, tmp_path, capsys):
    """A machine with hipcc alone builds the library; a module of an earlier build does not stay beside it."""
    stale = tmp_path / "hybridattn_binding.so"
    stale.write_bytes(b"of an earlier build")
    monkeypatch.setenv("HIPCC", "true")
    monkeypatch.setattr(build, "LIB_DIR", str(tmp_path))
    monkeypatch.setattr(build, "BINDING_PATH", str(stale))
    monkeypatch.setattr(build, "binding_command", lambda: [str(tmp_path / "g++")] if fault == "no compiler" else ["false"])
    assert build.build_library() == build.LIB_PATH
    assert not stale.exists() and "was not built" in capsys.readouterr().err


def test_is_built_and_leaves_host_tensors_alone():
    native = ha._binding()
    assert native
    t = torch.zeros(1, 1, 8, 64)
    ws = torch.zeros(1024, dtype=torch.uint8)
    assert native.forward(t, t, t, None, None, 1, 64, None, t, ws, None) is None
    assert native.forward(t, t) is None and native.param_update(t) is None
    assert native.param_update(t, t, 1e-3, 0, None, None, 1, 1.0, 0.9, 0.999, 1e-8, 0.01, None, None) is None
    with pytest.raises(RuntimeError, match="GPU only"):
        ha.hybrid_attn_forward(t, t, t, None, None, 1, out=t, workspace=ws)


@pytest.mark.parametrize("fault", ("not a module", "another torch", "another library", "absent"))
def test_a_module_that_does_not_fit_is_not_used(fault, monkeypatch, tmp_path):
    """A file left over from another torch or another version of the C ABI would read tensors and structs by the wrong layout: the Python
    code takes every call, and the file is looked for once."""
    monkeypatch.setattr(ha, "_BINDING", None)
    if fault in ("not a module", "absent"):
        path = tmp_path / "hybridattn_binding.so"
        if fault == "not a module":
            path.write_bytes(b"left over")
        monkeypatch.setattr(ha, "BINDING_PATH", str(path))
    elif fault == "another torch":
        monkeypatch.setattr(torch.version, "git_version", "0" * 40)
    else:
        class longer(ha.ctypes.Structure):
            _fields_ = ha.ha_problem._fields_ + [("more", ha.ctypes.c_int64)]
        monkeypatch.setattr(ha, "ha_problem", longer)
    if fault == "absent":
        assert ha._binding() is False
    else:
        with pytest.warns(UserWarning, match="build it again"):
            assert ha._binding() is False
    monkeypatch.setattr(ha, "_load_binding", lambda: pytest.fail("looked for a second time"))
    t = torch.zeros(1, 1, 8, 64)
    with pytest.raises(RuntimeError, match="GPU only"):
        ha.hybrid_attn_forward(t, t, t, None, None, 1, out=t, workspace=t)
    with pytest.raises(RuntimeError, match="GPU only"):
        ha.hybrid_attn_param_update(t, t, 1e-3)


@pytest.mark.gpu
@pytest.mark.parametrize("R,maps,dtype,layout", ((1, "none", "bf16", "bhnd"), (3, "square", "f32", "bnhd"), (4, "wide", "bf16", "bnhd"),
                                                 (2, "three", "bf16", "bhnd"), (2, "nobias", "f32", "bhnd")))
def test_same_outputs_as_the_python_code(R, maps, dtype, layout, monkeypatch):
    w = W.Workload(f"binding_{maps}", 2, 2, 150, 128, dtype, 64, R, 256 if maps == "wide" else 128, 256 if maps == "wide" else 128,
                   d_mid=128 if maps == "three" else 0, seed=5)
    q, k, v, fq, fk = ha.to_device(W.make_inputs(w))
    if layout == "bnhd":
        q, k, v = (t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v))
    if maps == "none":
        fq = fk = None
    if maps == "nobias":
        fq, fk = (dataclasses.replace(m, b1=None, b2=None) for m in (fq, fk))
    ws = torch.empty(ha.hybrid_attn_workspace_bytes(ha.make_problem(q, R, 64, w.scale), fq, fk), dtype=torch.uint8, device="cuda")
    outs = [torch.empty_strided(q.shape, q.stride(), dtype=q.dtype, device="cuda") for _ in range(2)]
    assert ha._binding().forward(q, k, v, fq, fk, R, 64, None, outs[0], ws, None) == ha.HA_OK
    python_only(monkeypatch)
    ha.hybrid_attn_forward(q, k, v, fq, fk, R, 64, out=outs[1], workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])


@pytest.mark.gpu
def test_what_is_not_plain_is_left_to_the_python_code():
    w = W.Workload("binding_refused", 1, 2, 100, 128, "bf16", 64, 2, 128, 128, seed=6)
    q, k, v, fq, fk = ha.to_device(W.make_inputs(w))
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(q)
    call = lambda *a: ha._binding().forward(*a, 64, None, out, ws, None)
    assert call(q, k, v, fq, fk, 2) == ha.HA_OK
    assert call(q, k, v, fq, fk, (2, 4)) is None                                     # a variant
    assert call(q, k, v.float(), fq, fk, 2) is None and call(q, k[:, :, :50], v, fq, fk, 2) is None
    assert call(q, k, v, fq, dataclasses.replace(fk, w1=fk.w1[:1]), 2) is None
    assert call(q, k, v, fq, dataclasses.replace(fk, b1=fk.b1.half()), 2) is None
    assert call(q, k, v, fq, dataclasses.replace(fk, w2=fk.w2.transpose(1, 2)), 2) is None
    assert ha._binding().forward(q, k, v, fq, fk, 2, 64, None, out, ws, torch.cuda.current_stream()) is None
    assert call(q, k, v, fq, fk, 0x7fffffff + 1) is None
    torch.cuda.synchronize()
    with pytest.raises(ha.HybridAttnError, match="workspace"):
        ha.hybrid_attn_forward(q, k, v, fq, fk, 2, 64, out=out, workspace=ws[:512])
    with pytest.raises(ValueError, match="w1 must be"):
        ha.hybrid_attn_forward(q, k, v, fq, dataclasses.replace(fk, w1=fk.w1[:1]), 2, 64, out=out, workspace=ws)
    with pytest.raises(ha.HybridAttnError):
        ha.hybrid_attn_forward(q, k, v, fq, fk, -1, 64, out=out, workspace=ws)
