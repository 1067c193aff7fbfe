"""Which kernels calls launch, on a runtime that records launches instead of
running them."""
import pytest

from host_util import on_host


@pytest.mark.parametrize("N", [160, 320])
def test_gradient_lonlat_below_a_thousand_tiles(N):
    """d/dlon and d/dlat read their scales by position, so the packed sweep
    cannot serve them, and the register-staged one leaves most of the chip
    idle on a mesh of a few hundred tiles: flat and column forms."""
    result = on_host(f"""
m = P.Mesh({N})
result = [(nlev, dt, launches(L.atlas_nabla_gradient_lonlat, m.handle, IN, nlev, dt, OUT, None)[-1][0])
          for nlev in (1, 4, 12, 23, 24, 37, 64, 137, 200) for dt in (F64, F32)]
""")
    for nlev, dt, kernel in result:
        assert ("k_flat" if nlev < 24 else "k_col") in kernel, (nlev, dt, kernel)


def test_gradient_lonlat_on_many_tiles():
    """A mesh of a thousand tiles and more: the register-staged sweep from 20
    levels in FP32 (to 79) and from 48 in FP64."""
    result = on_host("""
m = P.Mesh(500)
result = [(nlev, dt, launches(L.atlas_nabla_gradient_lonlat, m.handle, IN, nlev, dt, OUT, None)[-1][0])
          for nlev in (1, 4, 12, 19, 20, 23, 24, 47, 48, 79, 80, 137, 200) for dt in (F64, F32)]
""")
    for nlev, dt, kernel in result:
        staged = nlev >= 48 if dt == 1 else 20 <= nlev < 80
        want = "k_sweepv" if staged else "k_flat" if nlev < 24 else "k_col"
        assert want in kernel, (nlev, dt, kernel)
