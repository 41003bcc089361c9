"""The binding's two host paths: a call that leaves its outputs to the library
(marshalled natively) gives the bits of the same call with its stream given
(marshalled in Python), and arguments that the native path does not take end
where they ended before: converted, or refused with the same exception. Which path
a call took is read off the native functions, which return None for what they do
not take."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


class _Recorder:
    """The native functions, noting of each call whether it was taken."""

    def __init__(self, native):
        self.native, self.taken = native, []

    def __getattr__(self, name):
        f = getattr(self.native, name)

        def call(*args):
            out = f(*args)
            self.taken.append(out is not None)
            return out

        return call


@pytest.fixture
def native(monkeypatch):
    import paper_2509_23866_amd as dart

    rec = _Recorder(dart._nat(required=True))
    monkeypatch.setattr(dart, "_native", rec)
    return rec


def _case(T=300, V=1003, dtype="bf16"):
    import torch

    g = torch.Generator(device="cuda").manual_seed(T)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    lens = np.r_[np.full(9, 30), T - 270]
    off = torch.from_numpy(np.r_[0, np.cumsum(lens)].astype(np.int32)).cuda()
    i32 = lambda *v: torch.tensor(v, dtype=torch.int32, device="cuda")  # noqa: E731
    return dict(z=(rnd(T, V) * 3).to(torch.bfloat16 if dtype == "bf16" else torch.float32),
                y=torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32),
                old=-rnd(T).abs(), roll=-rnd(T).abs(), ref=-rnd(T).abs(), adv=rnd(T), off=off,
                R=rnd(4), traj=i32(0, 3, 5, 8, 10), grp=i32(0, 2, 4), gso=i32(0, 5, 10),
                h=rnd(T, 64).to(torch.bfloat16), w=rnd(V, 64).to(torch.bfloat16))


def _calls(c):
    """name -> (call with no outputs given, the same on the Python path)."""
    import torch

    import paper_2509_23866_amd as dart

    T = c["y"].numel()
    st = torch.cuda.current_stream()
    tok = dart.dart_tok_stats(c["z"], c["y"], stream=st)
    sel = lambda **k: dart.dart_select_tis_loss_fwd(  # noqa: E731
        tok[1], tok[0], c["old"], c["roll"], c["adv"], c["off"], 0.7, 0.2, 0.28, 2.0, **k)
    coef, mask = sel(stream=st)[4], sel(stream=st)[1]
    ex = lambda kl, **k: dart.dart_tis_loss_fwd_ex(  # noqa: E731
        tok[0], c["old"], c["roll"], c["adv"], c["off"], mask, 0.2, 0.28, 2.0, logp_ref=c["ref"],
        kl=kl, beta=0.1, aggregation="step_mean", ratio="step_geomean", **k)
    up = lambda **k: dart.policy_update(  # noqa: E731
        c["z"], c["y"], c["old"], c["roll"], c["adv"], c["off"], 0.7, 0.2, 0.28, 2.0, **k)
    values = lambda d: tuple(d[k] for k in sorted(d))  # noqa: E731
    both = lambda f: (f, lambda: f(stream=st))  # noqa: E731
    return {
        "tok_stats": both(lambda **k: dart.dart_tok_stats(c["z"], c["y"], **k)),
        "tok_stats inv_temp": both(lambda **k: dart.dart_tok_stats(c["z"], c["y"], inv_temp=1.3, **k)),
        "select_loss": both(sel),
        "select_loss no stats": both(lambda **k: sel(with_stats=False, **k)),
        "loss_ex": both(lambda **k: ex("k3", **k)),
        "loss_ex no kl": both(lambda **k: ex("none", **k)),
        "grad": both(lambda **k: (dart.dart_tis_grad(c["z"], c["y"], tok[0], tok[2], coef, **k),)),
        "grad skip": both(lambda **k: (dart.dart_tis_grad(
            c["z"], c["y"], tok[0], tok[2], coef, inv_temp=0.8, skip_zero_rows=True, **k),)),
        "advantage": both(lambda **k: dart.dart_grpo_advantage(c["R"], c["traj"], c["grp"],
                                                               c["off"], T=T, **k)),
        "advantage, T from the device": both(lambda **k: dart.dart_grpo_advantage(
            c["R"], c["traj"], c["grp"], c["off"], **k)),
        "groups": both(lambda **k: dart.dart_step_select_groups(tok[1], c["off"], c["gso"], 0.6,
                                                                **k)),
        "lmhead": both(lambda **k: dart.dart_lmhead_tok_stats(c["h"], c["w"], c["y"], **k)),
        "lmhead inv_temp": both(lambda **k: dart.dart_lmhead_tok_stats_ex(c["h"], c["w"], c["y"],
                                                                          0.9, **k)),
        "update": both(lambda **k: values(up(**k))),
    }


def _equal(a, b, name):
    import torch

    assert len(a) == len(b), name
    for x, y in zip(a, b):
        assert (x is None) == (y is None), name
        if x is not None:
            assert x.dtype == y.dtype and x.shape == y.shape and x.device == y.device, name
            raw = lambda t: t.contiguous().view(torch.uint8)  # noqa: E731
            assert torch.equal(raw(x), raw(y)), name


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_native_and_python_calls_agree(dtype, native):
    import torch

    for name, (ordinary, python) in _calls(_case(dtype=dtype)).items():
        native.taken.clear()
        a = ordinary()
        # T read from the device is the Python path's
        assert native.taken == ["from the device" not in name], name
        native.taken.clear()
        b = python()
        assert native.taken == [], name
        torch.cuda.synchronize()
        _equal(a, b, name)


def test_native_calls_run_on_the_current_stream(native):
    """Captured into a graph: a replay computes what it finds in the inputs, so every
    launch went to the capturing stream."""
    import torch

    c = _case()
    s = torch.cuda.Stream()
    for name, (ordinary, python) in _calls(c).items():
        if "from the device" in name:  # reads back: not for a capture
            continue
        ordinary()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        native.taken.clear()
        with torch.cuda.graph(graph, stream=s):
            a = ordinary()
        assert native.taken == [True], name
        for x in a:
            if x is not None:
                x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        _equal(a, python(), name)


def test_gradient_into_a_given_tensor(native):
    import torch

    import paper_2509_23866_amd as dart

    c = _case()
    out = dart.policy_update(c["z"], c["y"], c["old"], c["roll"], c["adv"], c["off"], 0.7, 0.2,
                             0.28, 2.0)
    buf = torch.empty_like(c["z"])
    got = dart.policy_update(c["z"], c["y"], c["old"], c["roll"], c["adv"], c["off"], 0.7, 0.2,
                             0.28, 2.0, dlogits=buf)
    assert got["dlogits"] is buf and torch.equal(buf, out["dlogits"])
    own = c["z"].clone()
    dz = dart.dart_tis_grad(own, c["y"], out["logp"], out["lse"], out["tok_coef"], dlogits=own)
    assert dz is own and torch.equal(own, buf)
    assert native.taken == [True] * 3


def test_what_the_native_path_does_not_take(native):
    """Numbers of other types are converted; wrong types, shapes, devices and
    layouts raise what they raised, and a failing C call names itself."""
    import torch

    import paper_2509_23866_amd as dart

    c = _case()
    z, y = c["z"], c["y"]
    want = dart.dart_tok_stats(z, y, inv_temp=1.5)
    plain = dart.dart_tok_stats(z, y)
    assert native.taken == [True, True]
    native.taken.clear()
    for it in (np.float32(1.5), torch.tensor(1.5)):
        for a, b in zip(dart.dart_tok_stats(z, y, inv_temp=it), want):
            assert torch.equal(a, b)

    class Sub(torch.Tensor):
        pass

    assert torch.equal(dart.dart_tok_stats(z.as_subclass(Sub), y)[0], plain[0])
    for bad, exc in (((z, y.long()), ValueError), ((z, y[:-1]), ValueError),
                     ((z, y.cpu()), ValueError), ((z.half(), y), TypeError),
                     ((z.t(), y), ValueError), ((z, [0] * 300), TypeError),
                     ((z.cpu(), y.cpu()), ValueError)):
        with pytest.raises(exc):
            dart.dart_tok_stats(*bad)
    assert native.taken and not any(native.taken)
    for it in (0.0, -1.0, float("nan"), float("inf")):
        with pytest.raises(dart.DartError, match="dart_tok_stats_ex"):
            dart.dart_tok_stats(z, y, inv_temp=it)
    with pytest.raises(dart.DartError, match="dart_tok_stats failed"):
        dart.policy_update(z[:0], y[:0], *(c[k][:0] for k in ("old", "roll", "adv")), c["off"][:1],
                           0.5, 0.2, 0.28, 2.0)
    with pytest.raises(dart.DartError, match="dart_select_tis_loss_fwd"):
        dart.policy_update(z, y, c["old"], c["roll"], c["adv"], c["off"], 1.5, 0.2, 0.28, 2.0)
    with pytest.raises(ValueError):
        dart.policy_update(z, y, c["old"], c["roll"], c["adv"][::2], c["off"], 0.5, 0.2, 0.28, 2.0)
    with pytest.raises(KeyError):
        dart.dart_tis_loss_fwd_ex(c["old"], c["old"], c["roll"], c["adv"], c["off"],
                                  torch.ones(10, dtype=torch.uint8, device="cuda"), 0.2, 0.28, 2.0,
                                  kl="k9")
