"""The marshalling extension of the serving calls: what it does not take it leaves to the checks of mla.py,
without calling anything (on the CPU: no tensor here is on a GPU)."""
import pytest
import torch

from paper_2502_07864_amd import mla


def test_the_extension_is_the_one_in_the_package():
    mla.lib()
    assert mla._fast.__file__.startswith(str(mla._LIB_PATH.parent))


def test_the_library_loads_without_the_extension(monkeypatch):
    """A package without _marshal (or one built for another torch) still loads, says so, and keeps every check."""
    import sys
    from paper_2502_07864_amd import convert
    monkeypatch.setitem(sys.modules, "paper_2502_07864_amd._marshal", None)      # importing it raises ImportError
    import paper_2502_07864_amd
    monkeypatch.delattr(paper_2502_07864_amd, "_marshal", raising=False)
    monkeypatch.setattr(mla, "_lib", None)
    monkeypatch.setattr(mla, "_fast", None)
    monkeypatch.setattr(convert, "_ready", False)
    with pytest.warns(RuntimeWarning, match="marshalling extension is not loaded"):
        mla.lib()
    assert mla._fast is None and mla.version().startswith("mla-gfx950")
    assert convert.lib().mla_conv_top_eig_workspace_bytes(64, 8) > 0
    with pytest.raises(ValueError, match="GPU tensor"):
        mla.absorb_q(torch.zeros(1, 2, 4), torch.zeros(2, 4, 8), out=torch.zeros(1, 2, 8))


def test_the_library_builds_where_the_extension_cannot(monkeypatch, tmp_path):
    """Neither a missing torch nor a failing compiler keeps the library from being built."""
    import sys
    from paper_2502_07864_amd import build
    monkeypatch.setattr(build, "MARSHAL", tmp_path / "_marshal.so")
    (tmp_path / "bin").mkdir()
    failing = tmp_path / "bin" / "g++"
    failing.write_text("#!/bin/sh\nexit 1\n")
    failing.chmod(0o755)
    monkeypatch.setattr(build.shutil, "which", lambda name: str(failing) if name == "g++" else None)
    monkeypatch.setattr(build, "hipcc", lambda: "/opt/rocm/bin/hipcc")
    with pytest.warns(RuntimeWarning, match="failed on marshal.cpp"):
        assert build.build_marshal() is None
    monkeypatch.setitem(sys.modules, "torch", None)
    with pytest.warns(RuntimeWarning, match="not built"):
        assert build.build_marshal() is None
    assert not (tmp_path / "_marshal.so").exists()


@pytest.mark.parametrize("bad", [torch.zeros(1, 2, 4), torch.zeros(1, 2, 4, dtype=torch.float64), None, 3, "x",
                                 torch.zeros(2, 1, 4).transpose(0, 1)])
def test_arguments_it_does_not_take_are_left_to_the_binding(bad):
    mla.lib()
    w = torch.zeros(2, 4, 8)
    assert mla._fast.absorb_q(bad, w, w) is None
    assert mla._fast.absorb_q(w, w) is None
    assert mla._fast.decode(3, bad, bad, bad, bad, bad, 1.0, 1, None, bad, bad, None, 0) is None
    assert mla._fast.decode(3) is None
    assert mla._fast.merge_out_proj(bad, w, w, None, w, 1, 1, 1, 0) is None
    assert mla._fast.merge_partials(bad, w, None, 1, 1, 1, 1, 0) is None
    assert mla._fast.cache_append(bad, w, w, None, w, w, w, 8, 1.0) is None


def test_the_checks_of_the_binding_still_raise():
    x, w = torch.zeros(1, 2, 4), torch.zeros(2, 4, 8)
    with pytest.raises(ValueError, match="GPU tensor"):
        mla.absorb_q(x, w, out=torch.zeros(1, 2, 8))
    with pytest.raises(ValueError, match="W_UK must be"):
        mla.absorb_q(x, w[:, :3], out=torch.zeros(1, 2, 8))
    with pytest.raises(ValueError, match="shorter than d_c"):
        mla.decode_paged(x, None, torch.zeros(1, 16, 3), torch.zeros(1, 1, dtype=torch.int32), torch.zeros(1, dtype=torch.int32),
                         1.0, workspace=torch.zeros(256, dtype=torch.uint8), out=torch.zeros(1, 2, 4))


@pytest.mark.gpu
def test_wrong_arguments_raise_on_the_gpu_as_before():
    """The same errors whether or not the extension was asked first."""
    dev = "cuda"
    q, kv = torch.zeros(2, 4, 8, device=dev), torch.zeros(3, 16, 16, device=dev)
    table, lens = torch.zeros(2, 1, dtype=torch.int32, device=dev), torch.zeros(2, dtype=torch.int32, device=dev)
    ws, out = torch.empty(1 << 16, dtype=torch.uint8, device=dev), torch.empty(2, 4, 8, device=dev)
    r = torch.zeros(2, 4, 8, device=dev)
    ok = dict(workspace=ws, out=out)
    for args, kw, err in [((q, r[:1], kv, table, lens, 1.0), ok, "q_rope must be"), ((q, r, kv, table.long(), lens, 1.0), ok, "must be int32"),
                          ((q, r, kv, table[:1], lens, 1.0), ok, "page_table must be"), ((q, None, kv, table, lens, 1.0), ok, "q_rope must be"),
                          ((q.transpose(0, 1).contiguous().transpose(0, 1), r, kv, table, lens, 1.0), ok, "contiguous"),
                          ((q, r, kv, table, lens, 1.0), dict(ok, workspace=ws[:64]), "MLA_ERR_WORKSPACE"),
                          ((q, r, kv, table, lens, float("nan")), ok, "MLA_ERR_SHAPE"), ((q, r, kv, table, lens, 1.0), dict(ok, num_splits=0), "MLA_ERR_SHAPE"),
                          ((q, r, kv, table, lens, 1.0), dict(ok, kv_scale=torch.zeros(3, 8, device=dev)), "kv_scale must be"),
                          ((q.double(), r.double(), kv, table, lens, 1.0), ok, "io dtype")]:
        with pytest.raises((ValueError, TypeError, mla.MlaError), match=err):
            mla.decode_paged(*args, **kw)
    assert mla.decode_paged(q, r, kv, table, lens, 1, **ok) is out          # an int for a scale: the binding's own path
    torch.cuda.synchronize()
    assert out.abs().max() == 0
