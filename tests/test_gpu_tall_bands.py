"""Bands of more than 62 parallels, whose pieces' tables of runs no longer fit
a wavefront's lanes (entries from 64 on are read when they are needed): the
wave-specialised sweep and fused Laplacian against the column form, whose
values the parity tests pin to the oracle."""
import pytest

from test_gpu_sweep_cuts import _field, _mesh, _same

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# 92 parallels: windows of 92 (the last run of the table is its 91st entry); a
# first band of 63 whose table ends on entry 63 and, with the Laplacian's two
# rings, 64; one of 62
LAYOUTS = [(92, 24), (63, 40), (62, 16), (64, 9)]


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_06091_amd as P
    return P


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("layout", LAYOUTS)
def test_sweep_of_tall_bands(P, layout, dtype):
    gm = _mesh(P, 46, layout)
    for nlev in (4, 5, 37, 96, 137):
        for op in (P.ATLAS_OP_GRADIENT, P.ATLAS_OP_DIVERGENCE, P.ATLAS_OP_CURL):
            print(f"tall bands {layout} op={op} nlev={nlev} {dtype}", flush=True)
            x = _field(gm, nlev, op != P.ATLAS_OP_GRADIENT, dtype, special=nlev % 2 == 1)
            ref = gm.apply(op, x, launch=P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 0))
            for block in (512, 1024):
                got = gm.apply(op, x, out=torch.full_like(ref, float("nan")),
                               launch=P.Launch(P.VARIANT_SWEEP, block, 0, 0, 0, 0))
                torch.cuda.synchronize()
                assert _same(got, ref), (op, nlev, block)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("layout", LAYOUTS)
def test_fused_laplacian_of_tall_bands(P, layout, dtype):
    gm = _mesh(P, 46, layout)
    for nlev in (4, 5, 37, 96, 137):
        print(f"tall bands {layout} lapl nlev={nlev} {dtype}", flush=True)
        x = _field(gm, nlev, False, dtype, special=nlev % 2 == 1)
        ref = gm.apply(P.ATLAS_OP_LAPLACIAN, x, launch=P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 0))
        for block in (512, 768):
            got = gm.apply(P.ATLAS_OP_LAPLACIAN, x, out=torch.full_like(ref, float("nan")),
                           launch=P.Launch(P.VARIANT_FUSED, block, 0, 0, 0, 0))
            torch.cuda.synchronize()
            assert _same(got, ref), (nlev, block)
