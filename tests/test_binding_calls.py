"""Plain calls take the native way through the binding, others Python's: the same results, and the same refusals."""
import os

import pytest
import torch

import paper_2506_22694_amd as vt
from paper_2506_22694_amd import binding, build


class Sub(torch.Tensor):
    pass


def _calls(dev):
    """name -> (call, arguments, results supplied by the caller) of the functions with a native way."""
    n, d, k, m, K = 3, 128, 96, 4, 5
    g = torch.Generator(device=dev).manual_seed(1)
    h = torch.randn(n, d, generator=g, device=dev)
    W = torch.randn(k, d, generator=g, device=dev).mul_(0.1)
    map_ = torch.arange(k, dtype=torch.int32, device=dev)
    cum = torch.linspace(-1, 0, n, device=dev)
    scores = torch.randn(40, generator=g, device=dev)
    ids = torch.randint(-2, k, (1000,), generator=g, device=dev)
    i32 = lambda *s: torch.zeros(s, dtype=torch.int32, device=dev)
    f32 = lambda *s: torch.zeros(s, device=dev)
    ws = None if dev == "cpu" else vt.StepWorkspace(n, k, d, m, h.device)
    return {
        "step": (vt.draft_head_step, dict(h=h, W_trim=W, map_=map_, m=m, ws=ws, out_ids=i32(n, m), out_logp=f32(n, m))),
        "static": (vt.draft_head_step_static, dict(h=h, W_trim=W, map_=map_, m=m, out_ids=i32(n, m), out_logp=f32(n, m))),
        "level": (vt.draft_tree_level, dict(h=h, W_trim=W, map_=map_, m=m, parent_cum=cum, K=K, ws=ws, out=(i32(K), i32(K), f32(K)),
                                            out_ids=i32(n, m), out_logp=f32(n, m))),
        "rerank": (vt.tree_rerank, dict(cum=scores, T=7, out=i32(7))),
        "count": (vt.count_tokens, dict(ids=ids, V=k, counts=torch.zeros(k, dtype=torch.int64, device=dev))),
    }


def _changes(args):
    """(what, changed arguments): calls that are refused, or that are not plain."""
    for name, t in args.items():
        if isinstance(t, torch.Tensor):
            if not name.startswith("out"):      # (what a step writes to was never looked at)
                yield name + " on the host", {**args, name: t.cpu()}
                yield name + " strided", {**args, name: t.repeat_interleave(2, dim=-1)[..., ::2]}
                yield name + " of another type", {**args, name: t.to(torch.float64)}
            yield name + " a subclass", {**args, name: t.as_subclass(Sub)}
            yield name + " a parameter", {**args, name: torch.nn.Parameter(t, requires_grad=False)}
            yield name + " no tensor", {**args, name: 3}
        elif isinstance(t, int):
            # (counts[V] are the caller's to supply: a larger V is not for trying)
            for v in (0, -1, 1 << 40, True, 2.0) + ((1 << 20,) if name != "V" else ()):
                yield f"{name} = {v}", {**args, name: v}
    if "h" in args:
        yield "a row shorter", {**args, "h": args["h"][:, :-4].contiguous()}
        yield "a map shorter", {**args, "map_": args["map_"][1:].clone()}
        yield "no rows", {**args, "h": args["h"][:0]}
        yield "a dimension more", {**args, "h": args["h"][None]}


def _outcome(call, args):
    args = {a: t.detach().clone() if a == "counts" and isinstance(t, torch.Tensor) else t for a, t in args.items()}
    try:
        r = call(**args)
    except Exception as e:
        return type(e), str(e)
    return [t.clone() for t in (r if isinstance(r, tuple) else (r,))]


def _compare(monkeypatch, dev, seen):
    native = binding._bind
    for name, (call, args) in _calls(dev).items():
        for what, changed in [("plain", args), *_changes(args)]:
            got = []
            for way in (native, None):
                monkeypatch.setattr(binding, "_bind", way)
                got.append(_outcome(call, changed))
            a, b = got
            seen.append((name, what, isinstance(a, tuple)))
            if isinstance(a, tuple) or isinstance(b, tuple):
                assert a == b, (name, what, a, b)
            else:
                assert all(torch.equal(x.cpu(), y.cpu()) for x, y in zip(a, b)), (name, what)
    monkeypatch.setattr(binding, "_bind", native)


def test_the_native_way_is_built():
    vt.load_library()
    assert binding._bind is not None


def test_a_native_way_built_for_another_torch_is_left_alone(monkeypatch):
    L = vt.load_library()
    monkeypatch.setattr(binding, "_bind", None)
    monkeypatch.setattr(binding, "BIND_ABI", binding.BIND_ABI.replace(torch.__version__, "1.0.0"))
    binding._connect(L)
    assert binding._bind is None
    # ... and built anew
    src = os.path.join(build.CSRC, "vt_bind.cpp")
    assert build._binding_stale(build._binding_command(src), [])
    monkeypatch.undo()
    assert not build._binding_stale(build._binding_command(src), [])


def test_a_binding_that_does_not_build_is_left_out(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "BIND", str(tmp_path / "_vt_bind.so"))
    monkeypatch.setattr(build, "BIND_STAMP", str(tmp_path / "vt_bind.command"))
    monkeypatch.setattr(build, "PKG", str(tmp_path))
    monkeypatch.setenv("CXX", str(tmp_path / "no such compiler"))
    with pytest.warns(UserWarning, match="left out"):
        build.build_binding()
    assert not os.path.exists(build.BIND)


def test_host_tensors_are_refused_the_same_way(monkeypatch):
    vt.load_library()
    seen = []
    _compare(monkeypatch, "cpu", seen)
    assert seen and all(refused for _, _, refused in seen)


@pytest.mark.gpu
def test_both_ways_answer_the_same(monkeypatch):
    vt.load_library()
    seen = []
    _compare(monkeypatch, "cuda", seen)
    assert sum(not refused for _, what, refused in seen if what == "plain") == 5


@pytest.mark.gpu
def test_plain_calls_take_the_native_way(monkeypatch):
    taken = []

    class Spy:
        def __getattr__(self, name):
            def f(*a):
                taken.append((name, getattr(native, name)(*a)))
                return taken[-1][1]
            return f
    vt.load_library()
    native = binding._bind
    monkeypatch.setattr(binding, "_bind", Spy())
    for call, args in _calls("cuda").values():
        call(**args)
    assert taken == [("step", 0), ("step_static", 0), ("level", 0), ("rerank", 0), ("count", 0)]


def test_calls_without_their_results_do_not_try_the_native_way(monkeypatch):
    class Refuses:
        def __getattr__(self, name):
            raise AssertionError(f"{name} is tried")
    vt.load_library()
    monkeypatch.setattr(binding, "_bind", Refuses())
    host = _calls("cpu")
    ws = object.__new__(vt.StepWorkspace)      # (what a host tensor is refused with comes before anything is read of it)
    for name, missing in (("step", ("out_ids", "out_logp")), ("level", ("out_ids", "out_logp", "out")), ("rerank", ("out",))):
        call, args = host[name]
        for gone in missing:
            with pytest.raises(ValueError):
                call(**{**args, **({"ws": ws} if "ws" in args else {}), gone: None})
