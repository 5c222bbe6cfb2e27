"""md_autotune launches the form of the steps that the context runs: the fused one,
which writes the drifted positions to the second position buffer, after NVE steps;
the plain one after steps under the thermostat, which are not fused."""
import pytest

import initconf
from gpu_common import lib_params
from test_gpu_brick import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", [0, 1])
@pytest.mark.parametrize("T0", [None, 1.0])
def test_tuned_form(torch_cuda, path, T0):  # noqa: F811
    torch = torch_cuda
    from paper_1105_5613_amd import System
    n = 9001  # no other array has 32 n bytes
    print(f"case autotune form path={path} T0={T0}", flush=True)
    s = initconf.fcc_system(n, seed=5, temperature=1.0)
    sysm = System(lib_params(path=path), [n], [s["L"]], allocator="torch")
    sysm.set_state(s["x"], s["v"], s["type"])
    sysm.step(5, T0=T0)
    pos = [b for b in sysm.allocator.blocks.values() if n * 32 <= b.numel() < n * 32 + 4096]
    assert len(pos) == 2
    before = [b.clone() for b in pos]
    sysm.autotune(reps=2)
    torch.cuda.synchronize()
    changed = sum(not torch.equal(a, b) for a, b in zip(before, pos))
    assert changed == (1 if T0 is None else 0)
    sysm.close()
