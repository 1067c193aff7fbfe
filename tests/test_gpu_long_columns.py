"""Columns above 256 levels in the column form (256 at a time with one level
per lane; lane vectors; the built-in choice) and FP32 vector columns of 193 to
256 levels (one chunk of four levels per lane): the flat form's bits, whose
values the parity tests pin to the oracle, on triangles and on
quadrilaterals (whose polar rows have three edges)."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_06091_amd as P
    return P


def _same(a, b):
    return torch.equal(a.isnan(), b.isnan()) and torch.equal(torch.nan_to_num(a), torch.nan_to_num(b))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("grid", ["O12", "S24x12"])
def test_column_equals_flat(P, grid, dtype):
    if grid == "O12":
        gm = P.Mesh(12)
    else:
        nx, lat = P.lonlat_grid(24, 12)
        gm = P.Mesh(nx=nx, lat=lat, shifted=True, quads=True)
    for nlev in (193, 255, 256, 257, 319, 320, 321, 511, 512, 513, 769):
        for op in (P.ATLAS_OP_GRADIENT, P.ATLAS_OP_DIVERGENCE, P.ATLAS_OP_CURL):
            print(f"long columns {grid} op={op} nlev={nlev} {dtype}", flush=True)
            shape = (gm.nnodes, nlev) + ((2,) if op != P.ATLAS_OP_GRADIENT else ())
            g = torch.Generator(device="cuda")
            g.manual_seed(nlev)
            x = torch.randn(shape, dtype=dtype, device="cuda", generator=g)
            x.view(-1)[::1009] = float("inf")
            x.view(-1)[::1499] = float("nan")
            want = gm.apply(op, x, launch=P.Launch(P.VARIANT_FLAT, 256, 32, 0, 0, 0))
            for launch in (None, P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 1),
                           P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 0)):
                out = torch.full_like(want, 7.0)
                got = gm.apply(op, x, out=out, launch=launch)
                assert _same(got, want), (op, nlev, launch)
