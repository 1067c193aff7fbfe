"""The wave-specialised fused Laplacian over its cuts of the tiles, level
chunks, lanes per position and elements per lane: the bits of the two passes
(whose values the parity tests pin to the oracle), at level counts on both
sides of every switch, with infinities and NaN, and as the built-in shape."""
import pytest

from test_gpu_sweep_cuts import _field, _mesh, _same

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LEVELS = (2, 3, 4, 5, 8, 9, 16, 17, 24, 25, 40, 41, 48, 63, 64, 65, 80, 96, 129, 137, 161, 321)


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_06091_amd as P
    return P


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("N,layout", [(33, None), (48, (8, 16)), (24, (3, 2)), (120, None)])
def test_fused_equals_two_passes(P, N, layout, dtype):
    gm = _mesh(P, N, layout)
    for nlev in LEVELS:
        print(f"fused lapl O{N} {layout} nlev={nlev} {dtype}", flush=True)
        x = _field(gm, nlev, False, dtype, special=nlev % 2 == 1)
        two = gm.apply(P.ATLAS_OP_LAPLACIAN, x, launch=P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 0))
        for block, chunk in ((320, 0), (1024, 0), (768, 19)):
            one = gm.apply(P.ATLAS_OP_LAPLACIAN, x,
                           launch=P.Launch(P.VARIANT_FUSED, block, 0, chunk, 0, 0))
            torch.cuda.synchronize()
            assert _same(one, two), (nlev, block, chunk)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("N,nlev", [(160, 45), (160, 137), (240, 24), (240, 137)])
def test_built_in_shape(P, N, nlev, dtype):
    gm = _mesh(P, N, None)
    print(f"built-in lapl O{N} nlev={nlev} {dtype}", flush=True)
    x = _field(gm, nlev, False, dtype, special=False)
    two = gm.apply(P.ATLAS_OP_LAPLACIAN, x, launch=P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 0))
    out = torch.full_like(two, float("nan"))
    gm.laplacian(x, out=out)
    torch.cuda.synchronize()
    assert torch.equal(out, two)
