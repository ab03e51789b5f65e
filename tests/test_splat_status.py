"""lib.splat with a workspace: one that is too small or empty is replaced; every
other status of the first render is raised, a device error above all (no GPU:
the library is replaced by one that reports chosen statuses)."""
import ctypes as C

import pytest
import torch

from paper_0811_2055_amd import lib


class Fake:
    def __init__(self, codes):
        self.codes, self.sizes = list(codes), []

    def splat_render(self, x, y, z, m, n, cam, sp, ws, ws_bytes, img, stream):
        self.sizes.append(ws_bytes)
        return self.codes.pop(0)

    def splat_plan(self, n, cam, sp, out):
        out._obj.value = 4096
        return lib.LOD_OK

    def lod_status_string(self, code):
        return str(code).encode()


def _splat(monkeypatch, codes, ws_bytes):
    fake = Fake(codes)
    monkeypatch.setattr(lib, "load", lambda: fake)
    monkeypatch.setattr(lib, "_stream", lambda: C.c_void_p())
    t = torch.zeros(3)
    lib.splat(t, t, t, t, lib.Camera.ortho(8, 8), workspace=torch.zeros(ws_bytes, dtype=torch.uint8))
    return fake


@pytest.mark.parametrize("codes,code", [(["LOD_EDEVICE", "LOD_OK"], "LOD_EDEVICE"),
                                        (["LOD_EUNSUPPORTED", "LOD_OK"], "LOD_EUNSUPPORTED"),
                                        (["LOD_EINVAL", "LOD_EINVAL"], "LOD_EINVAL"),
                                        (["LOD_ENOMEM", "LOD_EDEVICE"], "LOD_EDEVICE")])
def test_status_is_raised(monkeypatch, codes, code):
    with pytest.raises(lib.LodError) as err:
        _splat(monkeypatch, [getattr(lib, c) for c in codes], 8192)
    assert err.value.code == getattr(lib, code)


def test_small_workspace_is_replaced(monkeypatch):
    assert _splat(monkeypatch, [lib.LOD_ENOMEM, lib.LOD_OK], 256).sizes == [256, 4096]
    assert _splat(monkeypatch, [lib.LOD_EINVAL, lib.LOD_OK], 0).sizes == [0, 4096]    # no address to check
    assert _splat(monkeypatch, [lib.LOD_OK], 8192).sizes == [8192]
