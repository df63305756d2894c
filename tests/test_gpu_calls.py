"""The binding's native marshalling (csrc/calls.cpp) against its general code: the same call through both returns the same tensors, the
caller's own where it gave some, and what one refuses the other refuses with the same words.  On the CPU: what it leaves to the general
code."""
import os
import sys
import warnings

import numpy as np
import pytest
import torch

import paper_2508_16201_amd as package
from paper_2508_16201_amd import binding as B, build

gpu = pytest.mark.gpu


native_code = pytest.mark.skipif(torch.version.hip is None, reason="no torch for ROCm: there is no native code")


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(B.LIB_PATH) or (build.torch_with_gpus() and not os.path.exists(build.CALLS)):
        build.build()


def both(monkeypatch, call):
    """call(), by the native route, which has to take it, and by the general one."""
    native, taken = B._load_calls(), []

    class Watched:
        def __getattr__(self, name):
            def f(*args):
                got = getattr(native, name)(*args)
                taken.append(got is not None)
                return got
            return f

    results = []
    for route in (Watched(), B._NoCalls()):
        monkeypatch.setattr(B, "_calls", route)
        results.append(call())
    torch.cuda.synchronize()
    assert taken == [True]
    return results


def same(a, b):
    a, b = (x if isinstance(x, tuple) else (x,) for x in (a, b))
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert (x is None) == (y is None)
        if x is not None:
            assert x.dtype == y.dtype and x.shape == y.shape and x.stride() == y.stride() and x.device == y.device
            assert torch.equal(x.contiguous().view(torch.uint8), y.contiguous().view(torch.uint8))


def bf16(*shape, seed=1):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def i32(*x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


@gpu
@pytest.mark.parametrize("sampling", [False, True])
@pytest.mark.parametrize("given", [False, True])
def test_accept(monkeypatch, sampling, given):
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    t, x = torch.randn((2, 4, 1000), generator=g, device="cuda"), torch.randint(1000, (2, 3), generator=g, device="cuda", dtype=torch.int32)
    more = dict(draft_logits=t[:, :3].contiguous(), uniforms=torch.rand((2, 4), generator=g, device="cuda"), temperature=2) if sampling else {}
    if given:
        more.update(n_accepted=i32(0, 0), out_tokens=torch.zeros((2, 4), dtype=torch.int32, device="cuda"),
                    workspace=B.new_workspace(B.accept_workspace_bytes(2, 3, 1000, sampling)))
    a, b = both(monkeypatch, lambda: tuple(r.clone() if given else r for r in B.accept(t, x, **more)))
    same(a, b)
    if given:
        assert B.accept(t, x, **more)[0] is more["n_accepted"]


@gpu
@pytest.mark.parametrize("more", [{}, {"norm_mode": 1}, {"row_lse": True}, {"beta": 1, "scores": True, "workspace": True}])
def test_score(monkeypatch, more):
    q, k = bf16(20, 4, 64), bf16(2, 320, 64).permute(1, 0, 2)
    more = dict(more)
    if more.get("row_lse"):
        more["row_lse"] = torch.full((20, 4), 6.0, device="cuda")
    if more.get("workspace"):
        more["workspace"] = B.new_workspace(B.score_workspace_bytes(20, 320, 300, 4, 2, 64))

    def call():
        m = dict(more)
        if m.get("scores"):
            m["scores"] = torch.ones(300, device="cuda")
        return B.score(q, k, 0, 300, -1, 0.125, **m)
    same(*both(monkeypatch, call))


@gpu
def test_select_and_count(monkeypatch):
    s = torch.rand(500, device="cuda")
    same(*both(monkeypatch, lambda: B.select(s, i32(20), i32(50), 50)))
    same(*both(monkeypatch, lambda: B.select(s, i32(20), i32(50), 50, want_flags=False, keep_idx=torch.zeros(50, dtype=torch.int32, device="cuda"))))
    cu, keep = i32(0, 200, 500), i32(0, 30, 80)
    same(*both(monkeypatch, lambda: B.select(s, i32(9, 9), i32(30, 50), 80, cu_video=cu, cu_keep=keep, max_n_video=300)))
    same(*both(monkeypatch, lambda: B.top_p_count(s, 0.4)))
    same(*both(monkeypatch, lambda: B.top_p_count(s, 1, cu_video=cu, max_n_video=300, max_count=i32(20, 400), count=i32(0, 0))))


@gpu
def test_gather(monkeypatch):
    k, v = bf16(3, 2, 120, 64).permute(0, 2, 1, 3), bf16(3, 2, 120, 64, seed=2).permute(0, 2, 1, 3)
    keep = torch.arange(0, 100, 3, dtype=torch.int32, device="cuda")
    same(*both(monkeypatch, lambda: B.gather_kv(k, v, 0, 100, keep)))

    def into():
        return B.gather_kv(k, v, 5, 100, keep, *(torch.zeros((3, 2, 54, 64), dtype=torch.bfloat16, device="cuda").permute(0, 2, 1, 3) for _ in "kv"))
    same(*both(monkeypatch, into))
    cu = dict(cu_keys=i32(0, 50, 120), cu_video=i32(0, 40, 100), cu_keep=i32(0, 14, 34))
    idx = torch.cat([keep[:14], torch.arange(20, dtype=torch.int32, device="cuda")])
    same(*both(monkeypatch, lambda: B.gather_kv(k, v, 0, 100, idx, **cu)))


@gpu
@pytest.mark.parametrize("more", [{}, {"want_lse": True}, {"num_splits": 3, "out": True, "workspace": True}, {"tree": True}, {"batch": True}])
def test_attention(monkeypatch, more):
    q, k, v = bf16(6, 8, 128), bf16(2, 900, 128).permute(1, 0, 2), bf16(2, 900, 128, seed=2).permute(1, 0, 2)
    m = {n: x for n, x in more.items() if n in ("want_lse", "num_splits")}
    if "out" in more:
        m["out"] = torch.zeros_like(q)
    if "workspace" in more:
        m["workspace"] = B.new_workspace(B.decode_attn_workspace_bytes(1, 6, 900, 8, 2, 128, 3))
    if "tree" in more:
        m["ancestor_mask"] = torch.tensor([1, 3, 5, 11, 19, 37], dtype=torch.int64, device="cuda")
    if "batch" in more:
        m.update(cu_q=i32(0, 2, 6), cu_kv=i32(0, 300, 900), max_q_len=4, max_kv_len=600)
    same(*both(monkeypatch, lambda: B.decode_attn(q, k, v, 0.1, **m).clone() if "out" in more else B.decode_attn(q, k, v, 0.1, **m)))


# numbers as NumPy and Python programs have them (1 / np.sqrt(d) is an np.float64), parameters, flags that are not True or False
@gpu
@pytest.mark.parametrize("num", [np.float64, np.float32, int, bool])
def test_plain_numbers_of_other_types(monkeypatch, num):
    q, k = bf16(6, 8, 128), bf16(900, 2, 128)
    same(*both(monkeypatch, lambda: B.decode_attn(q, k, k, num(1) / num(8) if num is np.float32 else num(1))))
    same(*both(monkeypatch, lambda: B.score(q, k, 0, 800, -1, num(1), norm_mode=1, beta=num(1), scores=torch.ones(800, device="cuda"))))
    t, x = torch.randn((2, 3, 500), generator=torch.Generator("cuda").manual_seed(5), device="cuda"), i32(3, 4, 5, 6).view(2, 2)
    same(*both(monkeypatch, lambda: B.accept(t, x, draft_logits=t[:, :2].contiguous(), uniforms=torch.full((2, 3), 0.5, device="cuda"), temperature=num(1))))
    same(*both(monkeypatch, lambda: B.top_p_count(torch.rand(500, generator=torch.Generator("cuda").manual_seed(6), device="cuda"), num(1))))


@gpu
def test_plain_sizes_flags_and_tensors_of_other_types(monkeypatch):
    n = np.int64
    q, k, s = bf16(6, 8, 128), bf16(3, 900, 2, 128), torch.rand(500, generator=torch.Generator("cuda").manual_seed(6), device="cuda")
    same(*both(monkeypatch, lambda: B.score(q, k[0], n(0), n(800), n(-1), np.float64(0.1), norm_mode=n(1))))
    same(*both(monkeypatch, lambda: B.select(s, i32(20), i32(50), n(50), want_flags=1)))
    same(*both(monkeypatch, lambda: B.select(s, i32(20), i32(50), 50, want_flags=0)))
    same(*both(monkeypatch, lambda: B.select(s, i32(20), i32(50), n(50), want_flags=None, max_n_video=n(500))))
    same(*both(monkeypatch, lambda: B.decode_attn(q, k[0], k[1], 0.1, want_lse=1, num_splits=n(3), cu_q=i32(0, 2, 6), cu_kv=i32(0, 300, 900),
                                                  max_q_len=n(4), max_kv_len=n(600))))
    p = torch.nn.Parameter(k[0], requires_grad=False)
    same(*both(monkeypatch, lambda: B.decode_attn(torch.nn.Parameter(q, requires_grad=False), p, p, 0.1)))


@gpu
def test_gather_of_keys_alone_and_into_one_destination(monkeypatch):
    k, v = bf16(3, 120, 2, 64), bf16(3, 120, 2, 64, seed=2)
    keep = torch.arange(0, 100, 3, dtype=torch.int32, device="cuda")
    dst = lambda: torch.zeros((3, 54, 2, 64), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    same(*both(monkeypatch, lambda: B.gather_kv(k, None, 0, 100, keep)))
    same(*both(monkeypatch, lambda: B.gather_kv(k, None, 0, 100, keep, dst())))
    same(*both(monkeypatch, lambda: B.gather_kv(k, v, 0, 100, keep, dst())))
    same(*both(monkeypatch, lambda: B.gather_kv(k, v, 0, 100, keep, None, dst())))


@gpu
def test_calls_are_ordered_on_the_current_stream(monkeypatch):
    """Inputs that a side stream writes behind a pause: a call that went elsewhere would meet what was there before."""
    side, q, k = torch.cuda.Stream(), bf16(6, 8, 128), bf16(900, 2, 128)
    want, s = B.decode_attn(q, k, k, 0.1), torch.rand(500, generator=torch.Generator("cuda").manual_seed(6), device="cuda")
    kept = B.select(s, i32(20), i32(50), 50)[0]
    torch.cuda.synchronize()

    def call():
        late_q, late_s, k_top, budget = torch.zeros_like(q), torch.zeros_like(s), i32(20), i32(50)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)
            late_q.copy_(q)
            late_s.copy_(s)
            got = B.decode_attn(late_q, k, k, 0.1), B.select(late_s, k_top, budget, 50)[0]
        side.synchronize()
        return got
    for route in (B._load_calls(), B._NoCalls()):
        monkeypatch.setattr(B, "_calls", route)
        same(call(), (want, kept))


@gpu
def test_what_is_refused_is_refused_in_the_same_words(monkeypatch):
    t, x = torch.randn((1, 3, 100), device="cuda"), torch.zeros((1, 2), dtype=torch.int32, device="cuda")
    q, k = bf16(4, 8, 128), bf16(50, 2, 128)
    calls = [lambda: B.accept(t.transpose(1, 2), x), lambda: B.accept(t.cpu(), x), lambda: B.accept(t, x, workspace=t.new_empty(8, dtype=torch.uint8)),
             lambda: B.accept(t[0], x), lambda: B.accept(t, None), lambda: B.accept(np.zeros((1, 3, 100)), x),
             lambda: B.score(q, k, 0, 40, -1, 0.1, beta=0.5), lambda: B.score(q, k, 0, 40, -1, 0.1, beta=-1e-50), lambda: B.score(q, k, 0, 60, -1, 0.1), lambda: B.score(q[..., ::2], k, 0, 40, -1, 0.1),
             lambda: B.score(q, k, 0, -1, -1, 0.1), lambda: B.score(q, k, 0, 40, -1, 0.1, row_lse=torch.zeros(4, 8)),
             lambda: B.select(t[0, 0], x[0], x[0], 5, cu_video=x[0]), lambda: B.top_p_count(t[0, 0], 0.4, cu_video=x[0]),
             lambda: B.gather_kv(q, q, 0, 2, x[0]), lambda: B.gather_kv(k[None], k[None].transpose(1, 2), 0, 2, x[0]), lambda: B.gather_kv(k[None], None, 0, 2, x[0], None, q[None]),
             lambda: B.decode_attn(q, k, k[::2], 0.1), lambda: B.decode_attn(q, k, k, -1.0), lambda: B.decode_attn(q, k, k, 0.1, out=q.transpose(0, 1)),
             lambda: B.decode_attn(q, k, k, 0.1, cu_q=x[0], cu_kv=x[0]), lambda: B.decode_attn(q, k, k, 0.1, workspace=t.new_empty(8), num_splits=-1)]
    native = B._load_calls()
    for n, call in enumerate(calls):
        said = []
        for route in (native, B._NoCalls()):
            monkeypatch.setattr(B, "_calls", route)
            with pytest.raises(Exception) as e:
                call()
            said.append((type(e.value), str(e.value)))
        assert said[0] == said[1], (n, said)


@native_code
def test_what_is_left_to_the_general_code():
    native = B._load_calls()
    t, x = torch.zeros(1, 3, 9), torch.zeros((1, 2), dtype=torch.int32)

    class Kind(torch.Tensor):
        pass

    for a in (t, t.as_subclass(Kind), torch.nn.Parameter(t), t.numpy(), t.to("meta"), None, 3):
        assert native.accept(a, x, None, None, 1.0, None, None, None) is None
        assert native.score(a, a, 0, 2, -1, 0.1, 0, None, 0.0, None, None) is None
        assert native.select(a, x, x, 2, None, None, None, True, None) is None
        assert native.top_p_count(a, 0.4, None, None, None, None) is None
        assert native.gather_kv(a, a, 0, 2, x, None, None, None, None, None) is None
        assert native.decode_attn(a, a, a, 0.1, None, None, None, None, None, False, 0, None, None) is None
    with pytest.raises(TypeError):
        native.accept(t)
    with pytest.raises(TypeError):
        native.connect(1)


@native_code
def test_what_is_left_is_left_at_once():
    """A call that is not plain costs it what a look at a tensor or two costs, not an exception (2.4 us, as long as a launch)."""
    import timeit
    native, t, x = B._load_calls(), torch.zeros(1, 3, 9), torch.zeros((1, 2), dtype=torch.int32)
    once = lambda f: min(timeit.repeat(f, number=500, repeat=20)) / 500  # noqa: E731
    look = once(lambda: t.stride())
    for f in (lambda: native.accept(t, x, None, None, 1.0, None, None, None), lambda: native.gather_kv(t, None, 0, 2, x, None, None, None, None, None),
              lambda: native.decode_attn(t, t, t, 0.1, None, None, None, None, None, False, 0, None, None)):
        assert f() is None and once(f) < 6 * look


def test_without_the_native_code_every_call_is_left(monkeypatch):
    """A library without _calls.so beside it serves every call, after one warning; what is missing is the faster way there."""
    monkeypatch.setattr(B, "_calls", None)
    monkeypatch.setattr(B, "_raw_stream", lambda device: 0)
    monkeypatch.delattr(package, "_calls", raising=False)
    monkeypatch.setitem(sys.modules, package.__name__ + "._calls", None)
    t, x = torch.zeros((1, 3, 9)), torch.zeros((1, 2), dtype=torch.int32)
    with pytest.warns(RuntimeWarning, match="_calls.so"), pytest.raises(ValueError, match="on the GPU"):
        B.accept(t, x, n_accepted=x[0, :1], out_tokens=x, workspace=t)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        with pytest.raises(ValueError, match="on the GPU"):
            B.accept(t, x, n_accepted=x[0, :1], out_tokens=x, workspace=t)


@native_code
def test_the_native_code_is_of_the_library_and_the_torch_it_is_used_with(monkeypatch):
    """Another interface behind the same names, or objects laid out otherwise, is noticed before a call reaches it."""
    monkeypatch.setattr(B, "_raw_stream", lambda device: 0)
    native = B._load_calls()
    at = {name: 1 for name in native.functions}
    with pytest.raises(ImportError, match="version"):
        native.connect(B.version() + 1, at)
    with pytest.raises(KeyError, match=native.functions[-1]):
        native.connect(B.version(), {name: 1 for name in native.functions[:-1]})
    later = B.version() + 1
    class Older:                                               # (what was compiled before it said what for)
        connect = native.connect
    for where, name, what in ((B, "version", lambda: later), (torch, "__version__", "1.0.0+other"), (package, "_calls", Older)):
        with monkeypatch.context() as m:
            m.setattr(where, name, what)
            m.setattr(B, "_calls", None)
            with pytest.warns(RuntimeWarning, match="_calls.so"):
                assert isinstance(B._load_calls(), B._NoCalls)


@pytest.mark.parametrize("hip", [None, "7.0"])
def test_the_native_code_is_built_where_there_is_a_torch_for_it(monkeypatch, capsys, hip):
    made = []
    monkeypatch.setattr(torch.version, "hip", hip)
    monkeypatch.setattr(build, "_run", lambda cmd, verbose, what: made.append(cmd[cmd.index("-o") + 1]))
    assert build.build() == build.LIB and made == [build.LIB] + [build.CALLS] * (hip is not None)
    assert ("left out" in capsys.readouterr().out) == (hip is None)
