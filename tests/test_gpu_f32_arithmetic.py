"""FP32 fields: every operator forms its sums in FP64 on the promoted values
and rounds once, so an FP32 result is the FP64 operator's result on the
promoted field to one rounding.  Bound: half an ulp for that rounding and
half more where the two FP64 values (fused and unfused multiply-adds) fall
on different sides of a rounding boundary, 2^-23 |r|, plus the FP64 rounding
of sums whose terms exceed the result, 2^-40 max|r|."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_06091_amd as P
    return P


_meshes = {}


def _forms(P):
    L = P.Launch
    return {"default": None, "column": L(P.VARIANT_COLUMN, 256, 16, 0, 0, 0),
            "one level per lane": L(P.VARIANT_COLUMN, 256, 16, 0, 0, 1),
            "flat": L(P.VARIANT_FLAT, 512, 64, 0, 0, 0),
            "sweep": L(P.VARIANT_SWEEP, 1024, 0, 0, 0, 0),
            "staged sweep": L(P.VARIANT_SWEEP, 768, 0, 0, 1, 0),
            "flux": L(P.VARIANT_FLUX, 1024, 0, 0, 0, 0)}


@pytest.mark.parametrize("N,nlev", [(2, 1), (16, 3), (16, 64), (24, 137), (8, 300)])
@pytest.mark.parametrize("op", ["grad", "div", "curl"])
def test_f32_is_the_f64_result_rounded(P, op, N, nlev):
    print(f"f32 arithmetic {op} O{N} nlev={nlev}", flush=True)
    if N not in _meshes:
        _meshes[N] = P.Mesh(N)
    gm = _meshes[N]
    code = {"grad": P.ATLAS_OP_GRADIENT, "div": P.ATLAS_OP_DIVERGENCE, "curl": P.ATLAS_OP_CURL}[op]
    shape = (gm.nnodes, nlev) if op == "grad" else (gm.nnodes, nlev, 2)
    g = torch.Generator(device="cuda")
    g.manual_seed(7 * N + nlev)
    x = 1e2 + torch.randn(shape, device="cuda", generator=g)
    ref = gm.apply(code, x.double())
    bits = None
    for name, launch in _forms(P).items():
        got = gm.apply(code, x, launch=launch)
        torch.cuda.synchronize()
        err = (got.double() - ref).abs()
        bound = 2.0 ** -23 * ref.abs() + 2.0 ** -40 * ref.abs().max()
        assert bool((err <= bound).all()), (name, float((err - bound).max()))
        bits = got if bits is None else bits
        assert torch.equal(got, bits), name
