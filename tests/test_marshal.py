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


# ------------------------------------------------------------------ the native way through each entry point

B, T, H, DC, DR, DH, PAGE, MP, POOL, D = 3, 2, 5, 256, 64, 128, 16, 7, 23, 96      # all different


@pytest.fixture
def calls():
    """name -> (function of mla, dict of its arguments, names of its outputs), outputs holding 3.0."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    bf, f32, u8 = torch.bfloat16, torch.float32, torch.uint8

    def rnd(*shape, dtype=bf):
        return torch.randn(*shape, device="cuda", generator=gen).to(dtype)

    def out(*shape, dtype=bf):
        return torch.full(shape, 3.0, device="cuda", dtype=dtype)

    table = torch.randperm(POOL, device="cuda", generator=gen)[:B * MP].to(torch.int32).view(B, MP)
    table64 = torch.randperm(POOL, device="cuda", generator=gen)[:B * MP].to(torch.int32).view(B, MP)
    lens = torch.tensor([37, 0, 100], dtype=torch.int32, device="cuda")
    pos = torch.tensor([36, 5, 111], dtype=torch.int32, device="cuda")
    codes = torch.randint(0, 0x7E, (POOL, PAGE, DC + DR), dtype=u8, device="cuda", generator=gen)
    scale = torch.rand(POOL, PAGE, device="cuda", generator=gen) * 0.01 + 0.01
    kv, kv64 = rnd(POOL, PAGE, DC + DR), rnd(POOL, 64, DC + DR)

    def ws(rows, splits):
        # zeros: a chunk that no row falls into leaves its partial row as it is
        return torch.zeros(mla.decode_workspace_bytes(B, rows, DC, splits), dtype=u8, device="cuda")

    def step(q, qr, cache, tbl, splits, **kw):
        return dict(q_abs=q, q_rope=qr, kv_cache=cache, page_table=tbl, seq_lens=lens, softmax_scale=0.125, num_splits=splits,
                    workspace=ws(q[0].numel() // DC, splits), **kw)

    def partials(q, qr, cache, tbl, splits, flags=0):
        f = mla.decode_paged if q.dim() == 3 else mla.decode_paged_multi
        return f(**step(q, qr, cache, tbl, splits, flags=flags | mla.FLAG_SKIP_MERGE))

    q, qr, qf = rnd(B, H, DC), rnd(B, H, DR), rnd(B, H, DC, dtype=f32)
    q4, qr4, W_UV = rnd(B, T, H, DC), rnd(B, T, H, DR), rnd(H, DC, DH)
    return {
        "absorb_q": (mla.absorb_q, dict(q_nope=rnd(B, H, DH), W_UK=rnd(H, DH, DC), out=out(B, H, DC)), ["out"]),
        "absorb_q_f32": (mla.absorb_q, dict(q_nope=rnd(B, H, DH, dtype=f32), W_UK=rnd(H, DH, DC, dtype=f32), out=out(B, H, DC, dtype=f32)), ["out"]),
        "out_proj": (mla.out_proj, dict(o_lat=rnd(B, H, DC), W_UV=W_UV, out=out(B, H, DH)), ["out"]),
        "decode": (mla.decode_paged, step(q, qr, kv, table, 2, out=out(B, H, DC), lse=out(B, H, dtype=f32)), ["out", "lse"]),
        "decode_no_rope": (mla.decode_paged, dict(step(qf, None, rnd(POOL, PAGE, DC, dtype=f32), table, 2, out=out(B, H, DC, dtype=f32))), ["out"]),
        "decode_fp8": (mla.decode_paged, step(q, qr, codes, table, 3, kv_scale=scale, out=out(B, H, DC), lse=out(B, H, dtype=f32)), ["out", "lse"]),
        "decode_skip_merge": (mla.decode_paged, step(q, qr, kv64, table64, 2, flags=mla.FLAG_SKIP_MERGE), ["workspace"]),
        "decode_balanced": (mla.decode_paged, step(q, qr, kv64, table64, 2, flags=mla.FLAG_BALANCED, out=out(B, H, DC), lse=out(B, H, dtype=f32)), ["out", "lse"]),
        "decode_multi": (mla.decode_paged_multi, step(q4, qr4, kv, table, 2, out=out(B, T, H, DC), lse=out(B, T, H, dtype=f32)), ["out", "lse"]),
        "merge": (mla.merge_partials, dict(workspace=partials(q, qr, kv, table, 2), B=B, H=H, d_c=DC, num_splits=2, dtype=bf, out=out(B, H, DC),
                                           lse=out(B, H, dtype=f32)), ["out", "lse"]),
        "merge_balanced": (mla.merge_partials, dict(workspace=partials(q, qr, kv64, table64, 2, mla.FLAG_BALANCED), B=B, H=H, d_c=DC, num_splits=2,
                                                    dtype=bf, out=out(B, H, DC), lse=out(B, H, dtype=f32), flags=mla.FLAG_BALANCED), ["out", "lse"]),
        "merge_out_proj": (mla.merge_out_proj, dict(workspace=partials(q, qr, kv, table, 2), W_UV=W_UV, B=B, num_splits=2, o_lat=out(B, H, DC),
                                                    out=out(B, H, DH), lse=out(B, H, dtype=f32)), ["o_lat", "out", "lse"]),
        "merge_out_proj_multi": (mla.merge_out_proj_multi, dict(workspace=partials(q4, qr4, kv, table, 3), W_UV=W_UV, B=B, q_len=T, num_splits=3,
                                                                o_lat=out(B, T, H, DC), out=out(B, T, H, DH), lse=out(B, T, H, dtype=f32)),
                                 ["o_lat", "out", "lse"]),
        "append": (mla.cache_append, dict(x=rnd(B, D), W_DKVR=rnd(D, DC + DR), kv_cache=kv.clone(), page_table=table, positions=pos, d_c=DC,
                                          rope_base=5000.0, workspace=torch.empty(mla.append_workspace_bytes(B, D, DC, DR), dtype=u8, device="cuda")),
                   ["kv_cache"]),
        "append_fp8": (mla.cache_append, dict(x=rnd(B, D), W_DKVR=rnd(D, DC + DR), kv_cache=codes.clone(), kv_scale=scale.clone(), page_table=table,
                                              positions=pos, d_c=DC, workspace=torch.empty(mla.append_workspace_bytes(B, D, DC, DR), dtype=u8, device="cuda")),
                       ["kv_cache", "kv_scale"]),
    }


class Asked:
    """The extension, with what it answered."""
    def __init__(self, fast):
        self.fast, self.answers = fast, []

    def __getattr__(self, name):
        def call(*a):
            self.answers.append(getattr(self.fast, name)(*a))
            return self.answers[-1]
        return call


@pytest.mark.gpu
def test_every_native_call_gives_the_bits_of_the_binding(calls, monkeypatch):
    """The same call with the extension, which has to have made it, and without: outputs, caches and partials bit for
    bit (integers as they lie)."""
    fast = mla._fast
    for name, (f, args, outputs) in calls.items():
        got = {}
        for native in (True, False):
            a = {k: v.clone() if k in outputs else v for k, v in args.items()}
            asked = Asked(fast)
            monkeypatch.setattr(mla, "_fast", asked if native else None)
            f(**a)
            torch.cuda.synchronize()
            assert not native or asked.answers == [0], (name, asked.answers)
            got[native] = {k: a[k].view(torch.uint8) for k in outputs}
        for k in outputs:
            assert torch.equal(got[True][k], got[False][k]), (name, k)
            assert name == "decode_skip_merge" or not torch.equal(got[True][k], args[k].view(torch.uint8)), (name, k)


@pytest.mark.gpu
def test_what_the_native_calls_refuse_the_binding_refuses(calls, monkeypatch):
    """One argument at a time that breaks one check only, everything else as the call takes it: the extension calls
    nothing, and the binding raises."""
    f64, i64 = torch.float64, torch.int64

    def cut(t):                  # the right types, one element short
        return t.flatten()[:-1].clone()

    wrong = {
        "absorb_q": [dict(out=cut), dict(out=lambda t: t.float()), dict(W_UK=lambda t: t[:-1].clone()), dict(W_UK=lambda t: t[:, :-1].clone()),
                     dict(W_UK=lambda t: t.float()), dict(out=lambda t: t.repeat(1, 1, 2)[..., ::2])],
        "out_proj": [dict(out=cut), dict(W_UV=lambda t: t[:, 1:].clone())],
        "decode": [dict(out=cut), dict(lse=cut), dict(out=lambda t: t.float()), dict(lse=lambda t: t.double()), dict(page_table=lambda t: t.to(i64)),
                   dict(seq_lens=lambda t: t.to(i64)), dict(page_table=lambda t: t[:-1].clone()), dict(seq_lens=cut), dict(q_rope=lambda t: t[:, :-1].clone()),
                   dict(q_rope=lambda t: t.float()), dict(q_rope=lambda t: None), dict(kv_cache=lambda t: t[..., :DC - 8].clone()),
                   dict(kv_cache=lambda t: t.half()), dict(q_abs=lambda t: t.to(f64), q_rope=lambda t: t.to(f64)), dict(workspace=lambda t: t[:-256].clone())],
        "decode_fp8": [dict(kv_scale=lambda t: t[:-1].clone()), dict(kv_scale=lambda t: t.to(f64)), dict(kv_scale=lambda t: None)],
        "decode_multi": [dict(out=cut), dict(lse=cut), dict(q_rope=lambda t: t[:, :-1].clone())],
        "merge": [dict(out=cut), dict(lse=cut), dict(lse=lambda t: t.bfloat16()), dict(workspace=lambda t: t[:-256].clone())],
        "merge_out_proj": [dict(o_lat=cut), dict(out=cut), dict(lse=cut), dict(o_lat=lambda t: t.float()), dict(out=lambda t: t.float())],
        "merge_out_proj_multi": [dict(o_lat=cut), dict(out=cut), dict(lse=cut)],
        "append": [dict(positions=cut), dict(positions=lambda t: t.to(i64)), dict(page_table=lambda t: t.to(i64)), dict(page_table=lambda t: t[:-1].clone()),
                   dict(W_DKVR=lambda t: t[:-1].clone()), dict(W_DKVR=lambda t: t.float()), dict(workspace=lambda t: t[:-256].clone())],
        "append_fp8": [dict(kv_scale=cut), dict(kv_scale=lambda t: t.to(f64)), dict(kv_scale=lambda t: None)],
    }
    fast = mla._fast
    for name, cases in wrong.items():
        f, args, _ = calls[name]
        for case in cases:
            a = {**args, **{k: change(args[k]) for k, change in case.items()}}
            asked = Asked(fast)
            monkeypatch.setattr(mla, "_fast", asked)
            with pytest.raises((ValueError, TypeError, mla.MlaError)):
                f(**a)
            assert asked.answers[0] != 0, (name, list(case))      # None, or the entry point's own refusal (a short workspace)
            monkeypatch.setattr(mla, "_fast", None)
            with pytest.raises((ValueError, TypeError, mla.MlaError)):
                f(**a)
    torch.cuda.synchronize()
