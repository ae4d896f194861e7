"""The native argument marshalling (ext/marshal.cpp) against the Python definitions it stands in for: the same results, the same
errors, outputs given or made."""
import inspect
import os
import shutil
import subprocess
import sys

import pytest
import torch

import paper_2409_09099_amd as sste
from paper_2409_09099_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_native_functions_stand_in_for_the_python_ones():
    assert binding._marshal is not None, "_marshal.so is not built"
    for name, fn in binding._PYTHON.items():
        assert getattr(sste, name) is getattr(binding._marshal, name) and fn.__name__ == name


def test_native_functions_keep_signature_and_documentation():
    for name, fn in binding._PYTHON.items():
        want, got = inspect.signature(fn).parameters, inspect.signature(getattr(sste, name)).parameters
        assert [(p.name, p.default, p.kind) for p in got.values()] == [(p.name, p.default, p.kind) for p in want.values()], name
        assert getattr(sste, name).__doc__ == inspect.getdoc(fn)


def test_a_module_that_cannot_be_loaded_is_reported(tmp_path):
    """A _marshal.so that does not fit raises when the package is imported; without one the Python definitions serve."""
    pkg = tmp_path / "paper_2409_09099_amd"
    shutil.copytree(os.path.join(ROOT, "paper_2409_09099_amd"), pkg, ignore=shutil.ignore_patterns("*.so", "csrc", "ext", "__pycache__"))
    run = lambda: subprocess.run([sys.executable, "-c", "import paper_2409_09099_amd as s; print(s.linear_fwd.__module__)"], cwd=tmp_path,  # noqa: E731
                                 capture_output=True, text=True, timeout=100)
    assert run().stdout.strip() == "paper_2409_09099_amd.binding"
    (pkg / "_marshal.so").write_bytes(b"not a module")
    r = run()
    assert r.returncode != 0 and "ImportError" in r.stderr, r.stderr[-500:]


def test_update_step_takes_numbers_only():
    """Anything else that could pass for a float (a GPU tensor would synchronise) is refused, as through ctypes."""
    table = torch.zeros(64, dtype=torch.uint8)
    sste.library()
    for alpha in (torch.tensor(0.1), "0.1", None):
        with pytest.raises(TypeError):
            binding._marshal.update_batch_launch(table, 1, 1, 0, 0, alpha)


@pytest.mark.parametrize("call,error", [
    (lambda: sste.linear_fwd(torch.zeros(4, 64), None, None, 8), ValueError),              # not on the GPU
    (lambda: sste.linear_fwd(torch.zeros(4, 64), None, None), TypeError),                  # missing argument
    (lambda: sste.linear_fwd(torch.zeros(4, 64), None, None, 8, beta=1.0), TypeError),     # unknown keyword
    (lambda: sste.linear_dgrad(1, 2, 3, 4, 5, 6, 7, 8, 9), TypeError),                     # too many positions
    (lambda: sste.linear_wgrad(torch.zeros(4), torch.zeros(4, 4), 0, 0), ValueError),      # not 2-D
    (lambda: sste.cast_fp8(torch.zeros(4, 64), X=1, scale=1.0), TypeError),                # given twice
])
def test_errors_are_those_of_the_python_definitions(call, error):
    with pytest.raises(error):
        call()


def test_a_cxx_exception_becomes_a_python_error():
    """A tensor without storage (tracing) must raise, as through the Python definitions, and not end the process."""
    code = (
        "import torch, paper_2409_09099_amd as s\n"
        "from torch.func import vmap\n"
        "from torch._subclasses.fake_tensor import FakeTensorMode\n"
        "s.library()\n"
        "z = lambda *n, t=torch.bfloat16: torch.empty(n, dtype=t, device='cuda')\n"
        "def mapped():\n"
        "    vmap(lambda w: s.project_pack(w, 1.0, vals=w, meta=w))(z(2, 16, 64))\n"
        "with FakeTensorMode(allow_non_fake_inputs=True):\n"
        "    for call in (lambda: s.project_pack(z(16, 64), 1.0, vals=z(16, 32), meta=z(16, 8)), lambda: s.linear_fwd(z(4, 64), z(16, 32), z(16, 8), 16),\n"
        "                 lambda: s.cast_fp8(z(4, 64), 1.0), mapped):\n"
        "        try:\n"
        "            call()\n"
        "        except Exception as e:\n"
        "            print('raised', type(e).__name__, flush=True)\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.count("raised") == 4, (r.returncode, r.stdout, r.stderr[-2000:])


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", ["bf16", "e4m3"])
def test_same_results_as_the_python_definitions(fmt):
    T, O, I = 192, 80, 128
    g = torch.Generator(device="cuda").manual_seed(3)
    normal = lambda r, c, s: torch.empty((r, c), dtype=torch.bfloat16, device="cuda").normal_(0, s, generator=g)  # noqa: E731
    W, X, dY, H = normal(O, I, 0.02), normal(T, I, 1.0), normal(T, O, 1e-3), normal(T, I, 1.0)
    dt = sste.BF16 if fmt == "bf16" else sste.F8E4M3
    ws = 1.0 if fmt == "bf16" else 2e-4
    Q, amax = torch.empty((T, I), dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda")
    calls = {
        "project_pack": [((W, 1.4), dict(val_dtype=dt, val_scale=ws)), ((W, 1.4, dt, ws, *sste.packed_buffers(O, I, dt, "cuda")), dict(gamma=0.5, amax_out=amax))],
        "cast_fp8": [((X, 0.01), {}), ((X, 0.01, sste.F8E5M2), dict(Q=Q, amax_out=amax)), ((X, 0.01), dict(store=False))],
    }
    vals, meta = binding._PYTHON["project_pack"](W, 1.4, dt, ws)
    if fmt == "e4m3":
        X, dY = binding._PYTHON["cast_fp8"](X, 0.01)[0], binding._PYTHON["cast_fp8"](dY, 1e-5)[0]
    Z, A, dW = torch.empty((T, O), dtype=torch.bfloat16, device="cuda"), torch.empty((T, O), dtype=torch.bfloat16, device="cuda"), torch.ones((O, I), device="cuda")
    Z8 = torch.empty((T, O), dtype=torch.uint8, device="cuda")
    calls.update({
        "linear_fwd": [((X, vals, meta, O, dt), {}), ((X[3:], vals, meta), dict(O=O, dtype=dt, x_scale=2, w_scale=ws, Z=Z[3:]))],
        "linear_fwd_ex": [((X, vals, meta, O, dt), {}), ((X, vals, meta, O, dt, 1.0, ws, sste.F8E4M3, 0.5), dict(Z=Z8, amax_out=amax))],
        "linear_fwd_act": [((X, vals, meta, O, dt), {}), ((X, vals, meta, O, dt), dict(A=A, store_pre=False)), ((X, vals, meta, O, dt), dict(H=Z, A=A))],
        "linear_dgrad": [((dY, vals, meta, I, dt), {}), ((dY, vals, meta, I), dict(dtype=dt, dy_scale=0.5, dX=torch.empty((T, I), dtype=torch.bfloat16, device="cuda")))],
        "linear_dgrad_act": [((dY, vals, meta, I, H, dt), {}), ((dY, vals, meta, I, H, dt), dict(act=sste.ACT_NONE))],
        "linear_wgrad": [((dY[:128], X[:128], 1, 2, dt), {}), ((dY[:128], X[:128], 2 ** 64 - 1, -1), dict(dtype=dt, first_token=128, dW=dW))],
        "sgd_project_pack": [((W.clone(), dW, 0.1, 1.4, dt, ws), {}), ((W.float(), dW, 0.1, 1.4, dt, ws), dict(zip(("vals", "meta"), sste.packed_buffers(O, I, dt, "cuda"))))],
    })

    def flat(r):
        return [t.clone() for t in (r if isinstance(r, tuple) else (r,)) if t is not None]
    for name, variants in calls.items():
        for args, kw in variants:
            if name == "sgd_project_pack":            # in place: each side its own weight
                args = (args[0].clone(),) + args[1:]
            want = flat(binding._PYTHON[name](*((args[0].clone(),) + args[1:] if name == "sgd_project_pack" else args), **kw))
            got = flat(getattr(sste, name)(*args, **kw))
            torch.cuda.synchronize()
            assert len(got) == len(want) and all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, want)), (name, kw.keys())
    with pytest.raises(sste.SsteError) as e:
        sste.linear_fwd(X, vals, meta, O + 4, dt)
    assert e.value.status == 7 and "multiple of 8" in str(e.value)
    with pytest.raises(ValueError):
        sste.linear_wgrad(dY[:64], X[:128], 1, 2, dt)
