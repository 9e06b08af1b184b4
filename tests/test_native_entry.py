"""The Python entry points of the hot calls in native code (csrc/python)."""
import os
import shutil
import subprocess
import sys
import threading
import time

import pytest
import torch

from paper_2106_09236_amd import binding as psa


def _inputs(B=4, H=4, L=512, U=16):
    g = torch.Generator().manual_seed(3)
    Q, K, V = (torch.randn((B, H, L, 64), generator=g).cuda() for _ in range(3))
    idx = torch.randint(0, L, (B, H, L, U), generator=g, dtype=torch.int32).cuda()
    return Q, K, V, idx


def _calls():
    """name -> a call with everything brought along, so that nothing but the entry point itself can let other threads run"""
    Q, K, V, idx = _inputs()
    B, H, L, _ = Q.shape
    out, X, Y = torch.empty_like(Q), Q.reshape(B, L, H * 64), torch.empty((B, L, H * 64), device="cuda")
    ws = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")
    matrices = [torch.randn((H * 64, H * 64), device="cuda") / 16 for _ in range(4)]
    weights = psa.make_weights(*matrices)
    sel = torch.arange(32, dtype=torch.int32, device="cuda").expand(B, H, 32).contiguous()
    u = torch.full((B,), 32, dtype=torch.int32, device="cuda")
    keep = (matrices,)
    return {
        "fwd": lambda: psa.probsparse_attn_fwd(Q, K, V, None, idx, 5.0, out=out, workspace=ws),
        "opt": lambda: psa.probsparse_attn_fwd_opt(Q, K, V, None, idx, psa.U_RATIO, 0.5, psa.FILL_VALUE, out=out, workspace=ws, taps=False),
        "indices": lambda: psa.probsparse_attn_fwd_with_indices(Q, K, V, None, sel, u, psa.FILL_MEAN, out=out, workspace=ws),
        "mhsa": lambda: (psa.probsparse_mhsa_fwd(X, weights, None, idx, psa.U_LOG, 5.0, psa.FILL_MEAN, Y=Y, workspace=ws), keep),
        "bwd": lambda: psa.probsparse_attn_bwd(Q, K, V, None, sel, u, Q, psa.FILL_MEAN, workspace=ws),
    }


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["fwd", "opt", "indices", "mhsa", "bwd"])
def test_other_threads_run_during_calls(name):
    # The other thread waits for the interpreter and has a few microseconds of each call in which it can be had: how soon it wakes is up
    # to the machine (threads of a library that still spin after an earlier test keep the CPUs busy), so calls go on until it has run.
    # An entry point that keeps the interpreter lets it run in none of them, however many.
    call = _calls()[name]
    call()
    torch.cuda.synchronize()
    ticks, stop = [0], threading.Event()

    def other():
        while not stop.is_set():
            ticks[0] += 1
            time.sleep(0)
    interval = sys.getswitchinterval()
    thread = threading.Thread(target=other)
    sys.setswitchinterval(1000.0)                # a thread that does not let go of the interpreter keeps it
    during, end = 0, time.monotonic() + 60.0
    try:
        thread.start()
        while ticks[0] == 0:
            time.sleep(0.001)
        while during == 0 and time.monotonic() < end:
            before = ticks[0]
            results = [call() for _ in range(200)]   # (kept: freeing a tensor lets other threads run as well)
            during = ticks[0] - before
            results.clear()
            torch.cuda.synchronize()
    finally:
        stop.set()
        thread.join()
        sys.setswitchinterval(interval)
    assert during > 0


@pytest.mark.parametrize("module", [None, "not a shared object"])
def test_library_loads_without_the_module(tmp_path, module):
    # the package with its library only, or with a module that cannot be loaded
    here = os.path.dirname(psa.LIB_PATH)
    package = tmp_path / os.path.basename(here)
    package.mkdir()
    for name in ("__init__.py", "binding.py", "libprobsparse.so"):
        shutil.copy(os.path.join(here, name), package)
    if module is not None:
        (package / "_native.so").write_text(module)
    code = ("from paper_2106_09236_amd import binding as psa; s = psa.make_shape(1, 4, 128, 25, psa.PSA_F32); "
            "assert psa.LIB_PATH.startswith(%r), psa.LIB_PATH; assert psa.u_max(s, 5.0) == 25; "
            "print(psa.probsparse_describe_plan(s, psa.PsaOptions(psa.U_LOG, psa.FILL_MEAN, 5.0))['measure'], "
            "psa._fast().attn_bwd(1, 2, 3))" % str(tmp_path))
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.split() == ["lds", "None"], r.stderr
    assert ("cannot be loaded" in r.stderr) == (module is not None)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["fwd", "opt", "indices", "mhsa", "bwd"])
def test_ctypes_path_gives_the_same(name, monkeypatch):
    call = _calls()[name]

    def outputs():
        r = call()
        r = r[0] if name == "mhsa" else r
        return [t.clone() for t in (r if isinstance(r, tuple) else (r,))]
    native = outputs()
    assert psa._native is not psa._CtypesOnly
    monkeypatch.setattr(psa, "_native", psa._CtypesOnly)
    for a, b in zip(native, outputs()):
        assert torch.equal(a, b)


@pytest.mark.gpu
def test_a_status_is_raised_without_a_second_attempt(monkeypatch):
    # a workspace that is too small is refused on the host; the ctypes path, which would call the library again, is not entered
    Q, K, V, idx = _inputs(1, 4, 128, 8)
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    sel, u = torch.zeros((1, 4, 1), dtype=torch.int32, device="cuda"), torch.ones(1, dtype=torch.int32, device="cuda")
    X = torch.zeros((1, 128, 256), device="cuda")
    eye = torch.eye(256, device="cuda")
    weights = psa.make_weights(eye, eye, eye, eye)
    entered = []
    monkeypatch.setattr(psa, "_require_dev", lambda *ts: entered.append(ts))
    for call in (lambda: psa.probsparse_attn_fwd(Q, K, V, None, idx, 5.0, workspace=small),
                 lambda: psa.probsparse_attn_fwd_opt(Q, K, V, None, idx, psa.U_RATIO, 0.5, psa.FILL_MEAN, workspace=small, taps=False),
                 lambda: psa.probsparse_attn_fwd_with_indices(Q, K, V, None, sel, u, workspace=small),
                 lambda: psa.probsparse_attn_bwd(Q, K, V, None, sel, u, Q, workspace=small),
                 lambda: psa.probsparse_mhsa_fwd(X, weights, None, idx, psa.U_LOG, 5.0, psa.FILL_MEAN, workspace=small)):
        with pytest.raises(psa.ProbSparseError) as e:
            call()
        assert e.value.code == -5 and not entered          # PSA_ERR_WORKSPACE
