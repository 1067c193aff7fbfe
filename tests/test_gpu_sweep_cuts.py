"""The wave-specialised sweep over its cuts of the tiles, level chunks, lanes
per position and elements per lane: each must give the bits of the column
form (whose values the parity tests pin to the oracle), at level counts on
both sides of every switch, on meshes with and without bands to cut, and for
fields that hold infinities and NaN."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LEVELS = (2, 3, 4, 5, 8, 9, 16, 17, 31, 33, 40, 41, 47, 64, 65, 80, 81, 96, 97, 129, 137, 161, 300)


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_06091_amd as P
    return P


_meshes = {}


def _mesh(P, N, layout):
    if (N, layout) not in _meshes:
        _meshes[N, layout] = P.Mesh(N, layout=layout)
    return _meshes[N, layout]


def _field(gm, nlev, vector, dtype, special):
    g = torch.Generator(device="cuda")
    g.manual_seed(nlev)
    shape = (gm.nnodes, nlev, 2) if vector else (gm.nnodes, nlev)
    x = torch.randn(shape, dtype=dtype, device="cuda", generator=g)
    if special:
        x.view(-1)[::1009] = float("inf")
        x.view(-1)[::1499] = float("nan")
        x.view(-1)[::1151] = -torch.finfo(dtype).max
    return x


def _same(a, b):
    return torch.equal(torch.nan_to_num(a, nan=1.25), torch.nan_to_num(b, nan=1.25)) and \
        torch.equal(a.isnan(), b.isnan())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("op", ["grad", "div", "curl"])
@pytest.mark.parametrize("N,layout", [(33, None), (48, (8, 16)), (16, (64, 64)), (24, (3, 2))])
def test_sweep_equals_column(P, N, layout, op, dtype):
    gm = _mesh(P, N, layout)
    code = {"grad": P.ATLAS_OP_GRADIENT, "div": P.ATLAS_OP_DIVERGENCE, "curl": P.ATLAS_OP_CURL}[op]
    for nlev in LEVELS:
        print(f"sweep {op} O{N} {layout} nlev={nlev} {dtype}", flush=True)
        x = _field(gm, nlev, op != "grad", dtype, special=nlev % 2 == 1)
        ref = gm.apply(code, x, launch=P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 0))
        for block, chunk in ((512, 0), (1024, 0), (768, 17)):
            got = gm.apply(code, x, launch=P.Launch(P.VARIANT_SWEEP, block, 0, chunk, 0, 0))
            torch.cuda.synchronize()
            assert _same(got, ref), (nlev, block, chunk)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_one_pass_divergence_and_curl(P, dtype):
    """A mesh whose divergence runs the sweep (O320): both outputs of the one
    pass are bitwise the separate operators'."""
    gm = _mesh(P, 320, None)
    for nlev in (2, 5, 16, 37, 47, 64, 91, 96, 97, 137):
        print(f"div_curl O320 nlev={nlev} {dtype}", flush=True)
        uv = _field(gm, nlev, True, dtype, special=nlev % 2 == 1)
        d, c = gm.div_curl(uv)
        col = P.Launch(P.VARIANT_COLUMN, 256, 16, 0, 0, 0)
        assert _same(d, gm.apply(P.ATLAS_OP_DIVERGENCE, uv, launch=col)), nlev
        assert _same(c, gm.apply(P.ATLAS_OP_CURL, uv, launch=col)), nlev
