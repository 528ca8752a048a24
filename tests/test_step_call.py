"""The native call of a generation step: what it takes itself, what it leaves to the
general way, and that both ways are the same step."""
import subprocess
import sys

import pytest
import torch

B, Hh, D, HEAVY, RECENT = 1, 3, 64, 5, 4


@pytest.fixture(scope="module")
def hb():
    from paper_2306_14048_amd import binding
    return binding


def test_only_exact_plain_tensors_are_taken(hb):
    """On the CPU: everything that is not the plain case is left to the caller (1), before the
    library is called (the handle is not a cache)."""
    spec = hb._step_call.step_spec(torch.empty(1), B, Hh, D, hb.H2O_F16)
    good = torch.zeros(B, Hh, D, dtype=torch.float16)
    assert hb._step_call.decode_step(spec, None, good, good, good, good, 0) == 1       # a closed cache

    class Sub(torch.Tensor):
        pass
    for bad in (good.float(), good[:, :2], torch.zeros(B, Hh, 2 * D, dtype=torch.float16)[..., ::2],
                good.reshape(Hh, D), good.to(torch.bfloat16), good.as_subclass(Sub), good.to_sparse(), None, 5,
                torch.empty(B, Hh, D, dtype=torch.float16, device="meta")):
        for at in range(4):
            args = [good] * 4
            args[at] = bad
            assert hb._step_call.decode_step(spec, 1, *args, 0) == 1, (at, type(bad))
    with pytest.raises(TypeError):
        hb._step_call.decode_step(spec, None, good, good, good, good)
    with pytest.raises(ValueError):
        hb._step_call.decode_step(None, None, good, good, good, good, 0)
    with pytest.raises(TypeError):
        hb._step_call.step_spec(None, B, Hh, D, hb.H2O_F16)


def test_binding_without_the_native_call():
    """The library alone is enough: the import says that steps are slower and goes on."""
    code = ("import sys, warnings\n"
            "sys.modules['paper_2306_14048_amd._step_call'] = None\n"
            "with warnings.catch_warnings(record=True) as w:\n"
            "    warnings.simplefilter('always')\n"
            "    from paper_2306_14048_amd import binding\n"
            "assert binding._step_call is None and 'native step call' in str(w[-1].message), w\n"
            "assert binding.h2o_status_str(0)\n")
    subprocess.run([sys.executable, "-c", code], check=True)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
def test_native_and_general_call_are_the_same_step(hb, dtype, monkeypatch):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(3)
    draw = lambda *s: torch.randn(s, generator=gen, device=dev).to(dtype)  # noqa: E731
    steps = [tuple(draw(B, Hh, D) for _ in range(3)) for _ in range(24)]

    class Sub(torch.Tensor):
        pass
    side = torch.cuda.Stream()

    def run(way):
        with monkeypatch.context() as m:
            if way == "without the native call":
                m.setattr(hb, "_step_call", None)
            c = hb.H2OCache(B, Hh, D, HEAVY, RECENT, dtype, device=dev)
        if way in ("subclass", "without the native call"):      # one condition, not a call per tensor
            monkeypatch.setattr(c, "_expect", None, raising=False)
        torch.cuda.synchronize()
        outs = []
        for q, k, v in steps:
            out = torch.empty_like(q)
            if way == "native":
                c.decode_step(q, k, v, out)
            elif way == "entry point":
                hb.h2o_decode_step(c.handle, q, k, v, out)
            elif way == "subclass":                              # not the plain case: checked and called in Python
                c.decode_step(q.as_subclass(Sub), k, v, out)
            elif way == "without the native call":
                c.decode_step(q, k, v, out)
            elif way == "stream object":
                c.decode_step(q, k, v, out, side)
            elif way == "raw stream":
                c.decode_step(q, k, v, out, side.cuda_stream)
            else:
                with torch.cuda.stream(side):
                    c.decode_step(q, k, v, out)
            outs.append(out)
        torch.cuda.synchronize()
        state = [x.clone() for x in c.views()]
        c.close()
        with pytest.raises(hb.H2OError):
            c.decode_step(*steps[0], outs[0])                    # closed
        return outs + state
    ref = run("native")
    for way in ("entry point", "subclass", "without the native call", "stream object", "raw stream", "current stream"):
        for a, b in zip(ref, run(way)):
            assert torch.equal(a, b), way


@pytest.mark.gpu
def test_refusals_are_said(hb):
    dev = torch.device("cuda:0")
    c = hb.H2OCache(B, Hh, D, HEAVY, RECENT, torch.float16, device=dev)
    x = torch.zeros(B, Hh, D, dtype=torch.float16, device=dev)
    for bad, err in ((x.float(), ValueError), (x.cpu(), ValueError), (x[:, :2], ValueError), (None, None), (3, TypeError)):
        for at in range(4):
            args = [x] * 4
            args[at] = bad
            with pytest.raises(err or hb.H2OError):
                c.decode_step(*args)
    odd = torch.zeros(x.numel() + 1, dtype=torch.float16, device=dev)[1:].view_as(x)
    with pytest.raises(hb.H2OError):
        c.decode_step(odd, x, x, x)                              # not 16-byte aligned: the library refuses it
    assert c.tokens_seen == 0
