"""Regular grids: their polar rows refer to the far half of the parallel, so
no built-in shape walks tiles there, a sweep asked for is refused where the
runs do not fit, and every form gives the general form's bits."""
import pytest
import torch

import paper_1908_06091_amd as P

pytestmark = pytest.mark.gpu
_OPS = {"grad": P.ATLAS_OP_GRADIENT, "div": P.ATLAS_OP_DIVERGENCE, "lapl": P.ATLAS_OP_LAPLACIAN}


@pytest.fixture(scope="module")
def mesh():
    n = 100  # 91 tiles of 32 x 32, parallels of 400 nodes
    m = P.Mesh(nx=P.regular_gaussian_nx(n))
    yield m
    m.close()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nlev", [1, 20, 130])
@pytest.mark.parametrize("op", ["grad", "div", "lapl"])
def test_builtin_shapes(mesh, op, nlev, dtype):
    code = _OPS[op]
    g = torch.Generator().manual_seed(nlev)
    shape = (mesh.nnodes, nlev) + ((2,) if op == "div" else ())
    x = torch.randn(shape, generator=g, dtype=torch.float64).to(dtype).cuda()
    assert mesh.shape_of(code, nlev, x)["variant"] in (P.VARIANT_COLUMN, P.VARIANT_FLAT)
    want = mesh.apply(code, x, launch=P.Launch(P.VARIANT_FLAT, 512, 64, 0, 0, 0))
    assert torch.equal(mesh.apply(code, x), want)
    if op == "lapl":
        fused = P.Launch(P.VARIANT_FUSED, 768, 0, 0, 0, 0)
        assert torch.equal(mesh.apply(code, x, launch=fused), want)
    elif op == "div" and nlev >= 2:
        with pytest.raises(P.AtlasError, match="too large"):
            mesh.apply(code, x, launch=P.Launch(P.VARIANT_SWEEP, 512, 0, 0, 0, 0))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nlev", [1, 2, 3, 23, 24, 47])
@pytest.mark.parametrize("op", ["grad", "div"])
def test_many_tiles(op, nlev, dtype):
    """Short columns on a mesh of many tiles: larger blocks of the flat form,
    and 24 to 47 levels on lane vectors; block ends inside and past rows."""
    m = P.Mesh(nx=P.regular_gaussian_nx(48), layout=(2, 8))
    code = _OPS[op]
    g = torch.Generator().manual_seed(nlev)
    shape = (m.nnodes, nlev) + ((2,) if op == "div" else ())
    x = torch.randn(shape, generator=g, dtype=torch.float64).to(dtype).cuda()
    sh = m.shape_of(code, nlev, x)
    if nlev < 24:
        assert (sh["variant"], sh["block_threads"]) == (P.VARIANT_FLAT, 1024)
    got = m.apply(code, x)
    assert torch.equal(got, m.apply(code, x, launch=P.Launch(P.VARIANT_FLAT, 256, 32, 0, 0, 0)))
    m.close()
