"""Workspaces hold the buffers that the handle's calls may use, and no others
(host only: sizes, no device)."""
import ctypes as C
import os

import pytest


@pytest.fixture(scope="module")
def lib():
    import paper_1107_5463_amd as smc
    if not os.path.exists(smc.lib_path()):
        from paper_1107_5463_amd import build
        build.build()
    try:
        return smc.load_library()
    except OSError as e:  # pragma: no cover - HIP runtime missing on this host
        pytest.skip(f"cannot load libsmc.so: {e}")


def _bytes(lib, *args, **kw):
    import paper_1107_5463_amd as smc
    return lib.smc_workspace_bytes(C.byref(smc.make_params(*args, **kw)))


# up to 7 << 18 sites bricks take two copies of the spins; larger 2D XY lattices one,
# where two sweeps a pass are the faster way (from about L = 2450)
@pytest.mark.parametrize("L,copies", [(512, 2), (1352, 2), (1360, 0), (2048, 0), (2400, 0), (2600, 1), (4096, 1)])
def test_xy_copies(lib, monkeypatch, L, copies):
    for v in ("SMC_XY_MARCH", "SMC_CONT_KERNEL", "SMC_CONT_ROWS", "SMC_CONT_SPL"):
        monkeypatch.delenv(v, raising=False)
    partials = 48 * (L * L // 512)
    spare = _bytes(lib, 2, 2, L, delta=1.0) - copies * 8 * L * L - partials
    assert 0 <= spare <= 48 * 1024 + 4 * 256
    # couplings a bond and other dimensions never march
    assert _bytes(lib, 2, 2, 2600, J_kind=1, delta=1.0) < 8 * 2600 * 2600


def test_forced_passes_have_their_buffer(lib, monkeypatch):
    monkeypatch.delenv("SMC_XY_MARCH", raising=False)
    plain = _bytes(lib, 2, 2, 2048, delta=1.0)
    monkeypatch.setenv("SMC_XY_MARCH", "18")
    assert _bytes(lib, 2, 2, 2048, delta=1.0) == plain + 8 * 2048 * 2048
    monkeypatch.setenv("SMC_XY_MARCH", "0")
    assert _bytes(lib, 2, 2, 4096, delta=1.0) < 8 * 4096 * 4096
