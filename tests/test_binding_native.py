"""The native argument checks of the per-step calls against the Python
checks: the same calls are taken, the same ones refused with the same error."""
import ctypes
import warnings

import pytest

import paper_2403_08845_amd as bif

B, H, G, D, MC, MD = 2, 4, 2, 64, 40, 8


def test_host_tensors_are_left_to_the_python_checks():
    torch = pytest.importorskip("torch")
    # a caller of addresses that are never called: nothing here is on a GPU
    c = bif._caller(bif.Dims(B, H, G, D, MC, MD, 0.0), ctypes.c_void_p(16), 0)
    q = torch.zeros(B, H, D, dtype=torch.bfloat16)
    kc = torch.zeros(G, MC, D, dtype=torch.bfloat16)
    kd = torch.zeros(B, G, MD, D, dtype=torch.bfloat16)
    lens = torch.zeros(B, dtype=torch.int32)
    out = torch.zeros(B, H, D)
    assert c.decode(q, kc, kc, kd, kd, lens, None, None, out, 0) is None
    assert c.decode(None, 1, "x", kd, kd, lens, None, None, out, 0) is None
    assert c.append(kd, kd, kd, kd, lens, 0) is None
    with pytest.raises(TypeError):
        c.decode(q, kc)


@pytest.mark.parametrize("obstacle", ["missing", "other torch", "unloadable"])
def test_without_the_native_checks_python_takes_every_call(obstacle, monkeypatch, tmp_path):
    torch = pytest.importorskip("torch")
    monkeypatch.setattr(bif, "_bind", None)
    if obstacle == "missing":
        monkeypatch.setattr(bif, "BIND_PATH", str(tmp_path / "none.so"))
    elif obstacle == "unloadable":
        (tmp_path / "bad.so").write_bytes(b"no library")
        monkeypatch.setattr(bif, "BIND_PATH", str(tmp_path / "bad.so"))
    else:
        monkeypatch.setattr(torch, "__version__", "1.13.0+other")
    dims = bif.Dims(B, H, G, D, MC, MD, 0.0)
    with pytest.warns(RuntimeWarning, match="check their arguments in Python"):
        assert bif._caller(dims, ctypes.c_void_p(16), 0) is None
    with warnings.catch_warnings():
        warnings.simplefilter("error")  # once is enough
        assert bif._caller(dims, ctypes.c_void_p(16), 0) is None


def test_current_stream_without_the_raw_getter(monkeypatch):
    torch = pytest.importorskip("torch")

    class Stream:
        cuda_stream = 7

    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream)
    assert bif._raw_stream_getter()(0) == 7
    assert bif._stream_ptr(None, torch.device("cuda", 0)).value == 7
    assert bif._caller(bif.Dims(B, H, G, D, MC, MD, 0.0), ctypes.c_void_p(16), 0) is not None


def test_the_library_is_built_without_a_host_compiler(monkeypatch, capsys):
    from paper_2403_08845_amd import build
    ran = []
    monkeypatch.setenv("CXX", "/no/such/compiler")
    monkeypatch.setattr(build, "_run", lambda cmd, verbose: ran.append(cmd[0]))
    monkeypatch.setattr(build.os, "replace", lambda a, b: ran.append(b))
    assert build.build() == build.LIB
    assert ran == [build.hipcc(), build.LIB]
    assert "no host compiler" in capsys.readouterr().err


def _args(torch, kv, n):
    cache = torch.bfloat16 if kv == "bf16" else torch.uint8
    w = D // 2 if kv == "int4" else D

    def rows(*shape):
        if kv == "bf16":
            return torch.randn(*shape, w, device="cuda").to(cache)
        return torch.randint(0, 100, (*shape, w), device="cuda", dtype=cache)

    a = dict(q=torch.randn(B, H, n, D, device="cuda").to(torch.bfloat16), Kc=rows(G, MC),
             Vc=rows(G, MC), Kd=rows(B, G, MD), Vd=rows(B, G, MD),
             decode_lens=torch.full((B,), MD, dtype=torch.int32, device="cuda"),
             k_scale=None, v_scale=None,
             out=torch.full((B, H, n, D), float("nan"), device="cuda"))
    if kv != "bf16":
        a["k_scale"] = torch.full((G,), 0.01, device="cuda")
        a["v_scale"] = torch.full((G,), 0.02, device="cuda")
    return a


def _forms(torch, a, kv, n):
    """Argument sets by name: some valid, most one mistake away from it."""
    class Sub(torch.Tensor):
        pass

    yield "valid", a
    yield "subclass", dict(a, q=a["q"].as_subclass(Sub))
    yield "parameter", dict(a, q=torch.nn.Parameter(a["q"], requires_grad=False))
    yield "gradient", dict(a, q=a["q"].clone().requires_grad_())
    if n == 1:
        yield "flat", dict(a, q=a["q"][:, :, 0], out=a["out"][:, :, 0])
        yield "mixed ranks", dict(a, q=a["q"][:, :, 0])
    if kv != "bf16":
        yield "signed codes", dict(a, Kc=a["Kc"].view(torch.int8))
        yield "float codes", dict(a, Vd=a["Vd"].view(torch.float8_e4m3fn))
        yield "double scale", dict(a, k_scale=a["k_scale"].double())
        yield "one scale", dict(a, v_scale=a["v_scale"][:1])
    wide = torch.cat([a["Kd"], a["Kd"]], dim=2)
    yield "strided cache", dict(a, Kd=wide[:, :, ::2])
    yield "sliced cache", dict(a, Kd=wide[:, :, :MD])
    yield "transposed q", dict(a, q=a["q"].transpose(0, 1).contiguous().transpose(0, 1))
    yield "wrong dtype", dict(a, q=a["q"].half())
    yield "wrong rows", dict(a, Kc=a["Kc"][:, :-1].contiguous())
    yield "long lens", dict(a, decode_lens=a["decode_lens"].long())
    yield "half out", dict(a, out=a["out"].half())
    yield "host tensor", dict(a, Vc=a["Vc"].cpu())
    yield "not a tensor", dict(a, Vc=[1, 2])
    yield "none", dict(a, decode_lens=None)
    base = torch.empty(a["q"].numel() + 1, dtype=torch.bfloat16, device="cuda")
    yield "misaligned", dict(a, q=base[1:].view(a["q"].shape))


@pytest.mark.gpu
@pytest.mark.parametrize("kv,n", [("bf16", 1), ("bf16", 2), ("fp8_e4m3", 1), ("int4", 1)])
def test_native_and_python_checks_agree(kv, n):
    import torch
    torch.manual_seed(0)
    with bif.Plan(B, H, G, D, MC, MD, n=n, kv=kv) as plan:
        native = plan._caller
        assert native is not None  # the module that was built loads
        a = _args(torch, kv, n)
        for name, x in _forms(torch, a, kv, n):
            print(f"[case] {kv} n={n} {name}", flush=True)
            seen = []
            for caller in (native, None):
                plan._caller = caller
                x["out"].fill_(float("nan"))
                try:
                    bif.bifattn_decode_scaled(plan, *x.values())
                    torch.cuda.synchronize()
                    seen.append(("ok", x["out"].clone()))
                except Exception as e:
                    seen.append((type(e).__name__, str(e)))
            plan._caller = native
            assert seen[0][0] == seen[1][0], (name, seen)
            if seen[0][0] == "ok":
                assert torch.equal(seen[0][1], seen[1][1]) and torch.isfinite(seen[0][1]).all(), name
            else:
                assert seen[0][1] == seen[1][1], (name, seen)
        # appends, on a stream that is handed over
        new = a["Kd"][:, :, :n].contiguous()
        stream = torch.cuda.current_stream()
        seen = []
        for caller in (native, None):
            plan._caller = caller
            kd, vd = a["Kd"].clone(), a["Vd"].clone()
            lens = torch.full((B,), MD - n - 1, dtype=torch.int32, device="cuda")
            torch.cuda.synchronize()
            bif.bifattn_append_kv(plan, new, new, kd, vd, lens, stream=stream)
            stream.synchronize()
            with pytest.raises(TypeError):
                bif.bifattn_append_kv(plan, new, new, kd, vd, lens.long())
            seen.append((kd, vd, lens))
        plan._caller = native
        assert all(torch.equal(x, y) for x, y in zip(*seen))
        assert bif.bifattn_plan_status(plan) == bif.OK
    with pytest.raises(bif.BifattnError):  # a closed plan is refused, not called
        bif.bifattn_decode_scaled(plan, *a.values())
