"""A box that outgrows the tiles of cells while the caller's allocator refuses
the gather buffers: the call reports MD_ENOMEM, the context stays usable, and
goes on once there is memory."""
import numpy as np
import pytest

import initconf
from gpu_common import lib_params
from test_gpu_brick import converging_box, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture
def limited(monkeypatch):
    """System(..., allocator="torch") with a refusal: limit[0] is a count of
    allocations to grant first (None: no refusal), or a function of the bytes
    held and asked for."""
    from paper_1105_5613_amd import md
    limit = [None]

    class Limited(md.TorchAllocator):
        def __init__(self, stream):
            super().__init__(stream)
            grant = self._fns[0]

            def alloc(u, nbytes, hip_stream):
                if callable(limit[0]):
                    if not limit[0](self.bytes_held(), int(nbytes)):
                        return None
                elif limit[0] is not None:
                    if limit[0] <= 0:
                        return None
                    limit[0] -= 1
                return grant(u, nbytes, hip_stream)
            self._fns = (md.ALLOC_FN(alloc), self._fns[1], grant)
            self.struct = md.Allocator(self._fns[0], self._fns[1], None)
    monkeypatch.setattr(md, "TorchAllocator", Limited)
    return limit


def crowded():
    s = initconf.fcc_system(16000, rho=0.7, seed=15, temperature=0.5)
    x = s["x"].copy()
    x[:, 0] *= 0.55
    return s, x


def forces(sysm):
    sysm.forces()
    return sysm.get_forces().cpu().numpy()


# buffers of the switch: the list, and in the mixed form two sets of records;
# asked for with the tiles' list held, and again without it
@pytest.mark.parametrize("precision,grants", [(0, 0), (1, 0), (1, 1), (1, 2)])
def test_refused_at_the_first_build(torch_cuda, limited, precision, grants):  # noqa: F811
    from paper_1105_5613_amd import MDError, System, md
    print(f"case refused build precision={precision} grants={grants}", flush=True)
    s, x = crowded()
    ref = System(lib_params(precision=precision, path=1), [s["n"]], [s["L"]])
    ref.set_state(x, s["v"], s["type"])
    F = forces(ref)
    ref.close()
    sysm = System(lib_params(precision=precision), [s["n"]], [s["L"]], allocator="torch")
    for _ in range(2):
        sysm.set_state(x, s["v"], s["type"])
        limited[0] = grants
        for _ in range(2):
            with pytest.raises(MDError) as ex:
                sysm.forces()
            assert ex.value.code == md.MD_ENOMEM, ex.value
            limited[0] = 0
        with pytest.raises(MDError):  # no forces to give
            sysm.get_forces()
        xs, vs, _ = sysm.get_state()
        assert np.array_equal(vs.cpu().numpy(), s["v"])
        limited[0] = None
    assert np.array_equal(forces(sysm), F)  # the gather kernels' bits
    sysm.step(3)
    assert np.isfinite(sysm.observables()[0]["E"])
    sysm.close()
    assert sysm.allocator.bytes_held() == 0


@pytest.mark.parametrize("precision", [0, 1])
def test_room_for_one_list_only(torch_cuda, limited, precision):  # noqa: F811
    from paper_1105_5613_amd import System
    print(f"case room for one list precision={precision}", flush=True)
    s, x = crowded()  # rows of up to 150: a capacity of 256 does not grow
    ref = System(lib_params(precision=precision, path=1, max_neighbors=256), [s["n"]], [s["L"]], allocator="torch")
    ref.set_state(x, s["v"], s["type"])
    F = forces(ref)
    gather = max(t.numel() for t in ref.allocator.blocks.values())
    ref.close()
    sysm = System(lib_params(precision=precision, max_neighbors=256), [s["n"]], [s["L"]], allocator="torch")
    room = sysm.allocator.bytes_held() + gather - 1
    limited[0] = lambda held, asked: held + asked <= room
    sysm.set_state(x, s["v"], s["type"])
    assert np.array_equal(forces(sysm), F)
    sysm.close()


@pytest.mark.parametrize("graphs", [0, 4])
def test_refused_inside_a_run(torch_cuda, limited, graphs):  # noqa: F811
    """The box condenses during md_step: MD_ENOMEM with the state of the
    interrupted step, from which a context with memory goes on."""
    from paper_1105_5613_amd import MDError, System, md
    print(f"case refused run graphs={graphs}", flush=True)
    s, v = converging_box()
    sysm = System(lib_params(dt=0.002, graph_steps=graphs), [s["n"]], [s["L"]], allocator="torch")
    sysm.set_state(s["x"], v, s["type"])
    sysm.step(8)
    limited[0] = 0
    with pytest.raises(MDError) as ex:
        for _ in range(30):
            sysm.step(8)
    assert ex.value.code == md.MD_ENOMEM, ex.value
    xs, vs, img = sysm.get_state()  # reports nothing left behind
    assert bool(torch_cuda.isfinite(xs).all() & torch_cuda.isfinite(vs).all())
    with pytest.raises(MDError) as ex:
        sysm.step(8)
    assert ex.value.code == md.MD_ENOMEM, ex.value
    limited[0] = None
    sysm.step(8)
    F = sysm.get_forces().cpu().numpy()
    assert np.isfinite(F).all() and len(sysm.autotune(reps=1)["tried"]) > 2
    sysm.close()
