"""The native marshalling of binding.py against its step-by-step path: the same outputs bit for bit, under the same names and in
the same order, over the forms a call can have; what is not of the ordinary form is declined before anything happens."""
import gc
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

B = pytest.importorskip("paper_2506_02850_amd.binding")


class Declines:
    """Stands in for the native module: every call takes the step-by-step path."""
    def __getattr__(self, name):
        return lambda *a: None


class Watched:
    """The native module, and whether each call was taken (True) or declined (False)."""
    def __init__(self):
        self.host, self.taken = B._host, []

    def __getattr__(self, name):
        def call(*a):
            res = getattr(self.host, name)(*a)
            self.taken.append(res is not None)
            return res
        return call


def both(monkeypatch, call, taken):
    """The outputs of a call through the native module and step by step.  taken: what the native module does with it, [] where it is
    not asked."""
    with monkeypatch.context() as m:
        watched = Watched()
        m.setattr(B, "_host", watched)
        native = call()
    assert watched.taken == taken
    with monkeypatch.context() as m:
        m.setattr(B, "_host", Declines())
        plain = call()
    torch.cuda.synchronize()
    return native, plain


def check_same(native, plain):
    if isinstance(native, torch.Tensor):
        native, plain = {"": native}, {"": plain}
    assert list(native) == list(plain)
    for name, t in native.items():
        u = plain[name]
        if isinstance(t, torch.Tensor):
            assert t.dtype == u.dtype and t.shape == u.shape and t._base is None, name
            if name != "workspace":
                assert torch.equal(t, u), name
        else:
            assert t == u, name


# ---- without a GPU: declined, and the step-by-step path reports as it always has -----------------------------------------
def test_calls_off_the_gpu_are_declined_and_reported():
    f = torch.zeros(4, 6, 16)
    none = [None] * 9
    assert B._host.prefill_prune(torch.zeros(3, 4), 0, 1, torch.zeros(1), [1], *none, 0, False, B._stream) is None
    assert B._host.segment_compress(f, 2, 3, 2, torch.zeros(16), 0.5, 0.5, 1, 2, 0, 0, 0, None, None, B._stream) is None
    assert B._host.kv_compact([f], [f], None, [None], None, None, B._stream) is None
    with pytest.raises(ValueError, match="grid_h"):
        B.metok_segment_compress(f, 2, 2, 2, torch.zeros(16), 0.5, 0.5, 1, 2)
    with pytest.raises(ValueError, match="k_all is required"):
        B.metok_prefill_prune(torch.zeros(3, 4), 0, 1, torch.zeros(1), [1], q_text=torch.zeros(1, 1, 32))
    with pytest.raises(TypeError):
        B._host.prefill_prune(f)


@pytest.mark.parametrize("bad", [dict(k="3"), dict(k=np.int64(2)), dict(alpha="x"), dict(out=[1]), dict(feats=None), dict(feats=np.zeros((4, 6, 16)))])
def test_arguments_of_other_types_are_declined(bad):
    a = dict(feats=torch.zeros(4, 6, 16), gh=2, gw=3, k=2, text=torch.zeros(16), alpha=0.5, beta=0.5, s1=1, s2=2, sim=0, red=0, edge=0, ws=None, out=None)
    a.update(bad)
    assert B._host.segment_compress(*a.values(), B._stream) is None
    assert B._host.segment_compress_batched(*a.values(), B._stream) is None


def in_a_new_interpreter(before):
    code = before + """
import warnings
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    from paper_2506_02850_amd import binding as B
import torch
print([str(w.message) for w in said])
print(B.metok_preset(B.MODEL_LONGVA_7B)["s1"], type(B._host).__name__)
try:
    B.metok_segment_compress(torch.zeros(4, 6, 16), 2, 3, 2, torch.zeros(16), 0.5, 0.5, 1, 2)
except ValueError as e:
    print(e)
"""
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert p.returncode == 0, p.stderr
    return p.stdout


@pytest.mark.parametrize("before,said", [("import sys; sys.modules['paper_2506_02850_amd._host'] = None", "None in sys.modules"),
                                         ("import torch; torch.__version__ = '1.0'", "this is 1.0")])
def test_the_binding_works_without_its_native_part(before, said):
    out = in_a_new_interpreter(before)
    assert said in out and "ctypes" in out and "_StepByStep" in out and "must live on the GPU" in out


def test_the_native_part_is_loaded_where_it_fits():
    out = in_a_new_interpreter("")
    assert "ctypes" not in out and "module" in out and "must live on the GPU" in out


@pytest.mark.parametrize("commands", [[["false"]], [["no-such-compiler"]]])
def test_a_native_part_that_cannot_be_built_is_reported(monkeypatch, tmp_path, commands):
    from paper_2506_02850_amd import build
    target = str(tmp_path / "_host.so")
    monkeypatch.setattr(build, "host_commands", lambda obj, target: commands)
    assert commands[0][0] in build.build_host(target) and not os.path.exists(target)


# ---- on the GPU -----------------------------------------------------------------------------------------------------------
def frames(batch, T=9, gh=4, gw=5, d=64, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(T + d)
    lead = (batch,) if batch else ()
    return (torch.randn(lead + (T, gh * gw, d), generator=g, device="cuda").to(dtype), torch.randn(lead + (d,), generator=g, device="cuda").to(dtype))


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [0, 1, 3])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("form", ["fresh", "given", "workspace", "numpy", "out_dtype"])
def test_stage1_calls(monkeypatch, batch, dtype, form):
    f, t = frames(batch, dtype=dtype)
    call = B.metok_segment_compress_batched if batch else B.metok_segment_compress
    lead = (batch,) if batch else ()
    cap = B.metok_compress_encoder_tokens_capacity_rows(9, 4, 5, 1, 2) + 3
    kw, k = {}, 3
    if form == "given":
        kw["out"] = dict(out_tokens=torch.zeros(lead + (cap, 64), dtype=dtype, device="cuda"), token_event=torch.zeros(lead + (cap,), dtype=torch.int32, device="cuda"),
                         sim=torch.zeros(lead + (8,), device="cuda"), event_score=None)
    if form == "workspace":
        kw["workspace"] = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    if form == "numpy":
        k = np.int32(3)
    if form == "out_dtype":
        kw["out_dtype"] = torch.float32

    def run():
        r = call(f, 4, 5, k, t, 0.5, 0.45, 1, 2, sim_mode=B.SIM_TOKEN_MEAN, event_reduce=B.EVENT_MAX, pool_edge=B.POOL_CEIL, **kw)
        torch.cuda.synchronize()
        if form == "given":
            assert r["out_tokens"] is kw["out"]["out_tokens"] and r["sim"] is kw["out"]["sim"]
        res = {}
        for name, x in r.items():           # rows behind a video's own are not written unless the caller cleared them
            if name in ("out_tokens", "token_event") and form != "given":
                x = x.clone()
                ends = r["frame_offsets"].view(-1, 10)[:, -1].tolist()
                for b, end in enumerate(ends):
                    (x[b] if batch else x)[end:] = 0
            res[name] = x.clone()
        return res

    check_same(*both(monkeypatch, run, {"numpy": [False], "out_dtype": []}.get(form, [True])))


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [0, 2])
@pytest.mark.parametrize("form", ["attention", "scores", "bare", "given", "in_place", "static", "tuple", "workspace", "strides"])
def test_stage2_calls(monkeypatch, batch, form):
    g = torch.Generator(device="cuda").manual_seed(5)
    lead = (batch,) if batch else ()
    n, S, D = 70, 90, 64
    hidden = torch.randn(lead + (S, D), generator=g, device="cuda")
    seg = torch.randint(0, 2, lead + (n,), generator=g, device="cuda").int()
    ev = torch.randint(0, 4, lead + (n,), generator=g, device="cuda").int()
    quota = [[20, 9], [15, 20]] if batch else [20, 9]
    kw = dict(q_text=torch.randn(lead + (4, 6, 32), generator=g, device="cuda"), k_all=torch.randn(lead + (2, S, 32), generator=g, device="cuda"),
              token_event=ev, event_weight=torch.rand(lead + (4,), generator=g, device="cuda"),
              orig_idx=torch.arange(n, device="cuda").int().expand(lead + (n,)).contiguous(), score_mode=B.SCORE_VISUAL_ONLY)
    if form in ("scores", "bare"):
        kw = dict(scores=torch.rand(lead + (n,), generator=g, device="cuda"), **(kw if form == "scores" else {}))
        for name in ("q_text", "k_all"):
            kw.pop(name, None)
    if form == "tuple":
        quota = tuple(tuple(q) for q in quota) if batch else tuple(quota)
    if form == "static":
        if batch:
            pytest.skip("the static call takes one video")
        kw["static_scratch"] = True
    if form == "workspace":
        kw["workspace"] = torch.empty(1 << 21, dtype=torch.uint8, device="cuda")
    if form == "strides":
        if not batch:
            pytest.skip("one video has no strides")
        kw.update(keep_stride=40, out_row_stride=60)
    keep = 35 if batch else 29
    if form == "given":
        kw["out"] = dict(kept_idx=torch.zeros(lead + (keep,), dtype=torch.int32, device="cuda"), orig_idx_out=torch.zeros(lead + (keep,), dtype=torch.int32, device="cuda"),
                         hidden_out=torch.zeros(lead + (S - n + keep, D), device="cuda"))
    call = B.metok_prefill_prune_batched if batch else B.metok_prefill_prune

    def run():
        h = hidden.clone()
        if form == "in_place":
            kw["hidden_out"] = h if batch else h[:S - n + 29]
        r = call(h, 8, n, seg, quota, **kw)
        torch.cuda.synchronize()
        if form == "in_place":
            assert r["hidden_out"] is kw["hidden_out"]
        res = {}
        for name, x in r.items():
            if isinstance(x, torch.Tensor):
                x = x.clone()
                if batch and x.shape[1] != n:                       # what lies behind a video's own entries is unspecified
                    for b, kept in enumerate(r["n_keep"]):
                        x[b, kept + (S - n if name == "hidden_out" else 0):] = 0
            res[name] = x
        return res

    check_same(*both(monkeypatch, run, [True]))


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["dense", "paged", "relink", "relink_lens", "tuple", "given", "empty"])
def test_stage3_calls(monkeypatch, form):
    g = torch.Generator(device="cuda").manual_seed(9)
    L, Bn, H, rows, dh, ps = 3, 2, 2, 96, 64, 16
    paged = form in ("paged", "relink", "relink_lens")
    shape = (Bn * rows // ps, H, ps, dh) if paged else (Bn, H, rows, dh)
    table = torch.randperm(Bn * rows // ps, generator=g, device="cuda").int().view(Bn, -1)
    kv = torch.randn((L, 2) + shape, generator=g, device="cuda").to(torch.bfloat16)
    idx = [None, torch.arange(0, rows, 3, device="cuda").int().expand(Bn, -1).contiguous(), torch.arange(16, 64, device="cuda").int().expand(Bn, -1).contiguous()]
    if form == "empty":
        idx[1] = torch.empty((Bn, 0), dtype=torch.int32, device="cuda")
    given = torch.zeros(L, dtype=torch.int32, device="cuda")

    def run():
        x = kv.clone()
        k, v = [x[i, 0] for i in range(L)], [x[i, 1] for i in range(L)]
        ix = idx
        if form == "tuple":
            k, v, ix = tuple(k), tuple(v), tuple(idx)
        if form.startswith("relink"):
            r = B.metok_kv_relink_paged(k, v, table, ix, len_in=[rows] * L if form == "relink_lens" else None)
        elif form == "paged":
            r = {"new_len": B.metok_kv_compact_paged(k, v, table, ix)}
        elif form == "given":
            r = {"new_len": B.metok_kv_compact(k, v, ix, given)}
            assert r["new_len"] is given
        else:
            r = {"new_len": B.metok_kv_compact(k, v, ix)}
        torch.cuda.synchronize()
        # rows behind the kept ones are unspecified where rows moved between workgroups; the whole cache is the same here
        return {**{name: t.clone() for name, t in r.items()}, "kv": x}

    check_same(*both(monkeypatch, run, [form != "empty"]))


@pytest.mark.gpu
def test_refusals_of_the_library_are_raised():
    f, t = frames(0)
    with pytest.raises(B.MetokError, match="k must be in"):
        B.metok_segment_compress(f, 4, 5, 99, t, 0.5, 0.5, 1, 2)
    with pytest.raises(B.MetokError, match="workspace"):
        B.metok_segment_compress(f, 4, 5, 2, t, 0.5, 0.5, 1, 2, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    with pytest.raises(ValueError, match="contiguous"):
        B.metok_segment_compress(f.transpose(0, 1).contiguous().transpose(0, 1), 4, 5, 2, t, 0.5, 0.5, 1, 2)
    with pytest.raises(ValueError, match="out"):
        B.metok_segment_compress(f, 4, 5, 2, t, 0.5, 0.5, 1, 2, out=dict(sim=torch.zeros(3, device="cuda")))


def native_calls():
    """The six native functions on small inputs, each as a function of the stream function it is given."""
    f, t = frames(0)
    fb, tb = frames(2)
    g = torch.Generator(device="cuda").manual_seed(11)
    n, S, D = 70, 90, 64
    hidden, seg, scores = (torch.randn(S, D, generator=g, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda"),
                           torch.rand(n, generator=g, device="cuda"))
    two = lambda x: torch.stack([x, x])
    kv = [torch.randn(2, 2, 96, 64, generator=g, device="cuda") for _ in range(2)]
    pools, table = [x.view(12, 2, 16, 64) for x in kv], torch.arange(12, device="cuda").int().view(2, 6)
    idx = [torch.arange(0, 96, 3, device="cuda").int().expand(2, -1).contiguous()]
    shape = (4, 5, 3)
    rest = (0.5, 0.45, 1, 2, 0, 0, 0, None, None)
    nothing = [None] * 5
    H = B._host
    return {
        "segment_compress": lambda s: H.segment_compress(f, *shape, t, *rest, s),
        "segment_compress_batched": lambda s: H.segment_compress_batched(fb, *shape, tb, *rest, s),
        "prefill_prune": lambda s, static=False: H.prefill_prune(hidden, 8, n, seg, [29], *nothing, scores, hidden[:S - n + 29], None, None, 0, static, s),
        "prefill_prune_batched": lambda s: H.prefill_prune_batched(two(hidden), 8, n, two(seg), [[29], [15]], *nothing, two(scores), None, None, None, 0, None, None, s),
        "kv_compact": lambda s: H.kv_compact(kv[:1], kv[1:], None, idx, None, None, s),
        "kv_relink_paged": lambda s: H.kv_relink_paged(pools[:1], pools[1:], table, idx, None, None, s),
    }


NATIVE_CALLS = ["segment_compress", "segment_compress_batched", "prefill_prune", "prefill_prune_batched", "kv_compact", "kv_relink_paged"]


@pytest.mark.gpu
@pytest.mark.parametrize("name", NATIVE_CALLS)
def test_nothing_that_can_fail_follows_the_launch(name):
    """Had the wrapping of the results failed behind the launch, the step-by-step path would launch the call again, on data that an
    in-place call has already moved.  The results are Python objects: with a collection due at every other one that is made, one
    made after the stream was asked for, the last thing before the launch, would show."""
    call, handles, late = native_calls()[name], [B._stream()], []

    def watch(phase, info):
        if not handles:
            late.append(phase)

    before = gc.get_threshold()
    gc.collect()
    gc.callbacks.append(watch)
    gc.set_threshold(1)
    try:
        res = call(handles.pop)
        gc.disable()
    finally:
        gc.callbacks.remove(watch)
        gc.set_threshold(*before)
        gc.enable()
    torch.cuda.synchronize()
    assert res is not None and not handles and not late


class Refuses:
    def __bool__(self):
        raise LookupError("asked for its truth")


@pytest.mark.gpu
@pytest.mark.parametrize("name", NATIVE_CALLS)
def test_errors_of_the_stream_function_are_raised(name):
    """A signal's exception is raised wherever Python code runs, here in the stream function: it must not be taken for a reason
    to decline."""
    def interrupted():
        raise KeyboardInterrupt
    with pytest.raises(KeyboardInterrupt):
        native_calls()[name](interrupted)


@pytest.mark.gpu
def test_errors_of_the_arguments_are_raised():
    asked = []

    def stream():
        asked.append(1)
        return B._stream()
    # a truth value that is no bool belongs to the step-by-step path; nothing goes on beside the error
    assert native_calls()["prefill_prune"](stream, Refuses()) is None and not asked

    class Key(str):
        __hash__ = str.__hash__

        def __eq__(self, other):
            raise KeyboardInterrupt
    f, t = frames(0)
    with pytest.raises(KeyboardInterrupt):
        B._host.segment_compress(f, 4, 5, 3, t, 0.5, 0.45, 1, 2, 0, 0, 0, None, {Key("sim"): None}, stream)
