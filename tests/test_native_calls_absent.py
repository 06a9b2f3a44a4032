"""The torch functions where the native calls were not built for this Python or
torch: a warning, and the same results and errors."""
import os
import subprocess
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NOT_BUILT = "sys.modules['paper_1905_03136_amd._calls'] = None"
OTHER_TORCH = "import types; m = types.ModuleType('_calls'); m.torch_version = '1.0'; " \
              "sys.modules['paper_1905_03136_amd._calls'] = m; import paper_1905_03136_amd as p; p._calls = m"


@pytest.mark.parametrize("how", [NOT_BUILT, OTHER_TORCH], ids=["not built", "another torch"])
def test_import_and_errors(how):
    script = """
import sys, warnings
%s
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    from paper_1905_03136_amd import api
assert [x.category for x in w if "native calls" in str(x.message)] == [RuntimeWarning], w
assert api._calls is None
import torch
x = torch.zeros(4, 2, dtype=torch.float64)
for call in (lambda: api.tsmttsm(x, x), lambda: api.tsmm(x, x[:2])):
    try:
        call()
    except ValueError:
        continue
    raise SystemExit("CPU tensors were taken")
""" % how
    r = subprocess.run([sys.executable, "-c", script], cwd=ROOT, text=True, timeout=300, stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT)
    assert r.returncode == 0, r.stdout


def test_built_for_this_torch():
    from paper_1905_03136_amd import api
    assert api._calls is not None and api._calls.torch_version == torch.__version__


@pytest.mark.gpu
def test_same_results(monkeypatch):
    from paper_1905_03136_amd import api, inputs
    A = inputs.device_uniform(10007, 5, 97, inputs.STREAM_A, False, "cuda:0")
    B = inputs.device_uniform(10007, 3, 97, inputs.STREAM_B, False, "cuda:0")
    X = A[:5, :4]
    want = api.tsmttsm(A, B), api.tsmm(A, X, alpha=2.0)
    monkeypatch.setattr(api, "_calls", None)
    got = api.tsmttsm(A, B), api.tsmm(A, X, alpha=2.0)
    assert all(torch.equal(g, w) for g, w in zip(got, want))
