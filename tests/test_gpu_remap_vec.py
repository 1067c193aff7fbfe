"""The remap's vector form (several columns per lane, a few targets per
workgroup) against the flat form, column by column: the same bits at every
column count around its switches, for more and for fewer targets than
sources, polar targets and a ragged last workgroup included."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_06091_amd as P
    return P


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("source,target", [(8, 21), (24, 9)])
def test_columns_equal_single_columns(P, source, target, dtype):
    r = P.Remap(P.Mesh(source), P.Mesh(target))
    for ncol in (4, 5, 7, 8, 9, 15, 31, 33, 47, 49, 63, 64, 65, 79, 81, 95, 97, 137):
        print(f"remap O{source} to O{target} {ncol} columns {dtype}", flush=True)
        g = torch.Generator(device="cuda")
        g.manual_seed(ncol)
        x = torch.randn(r.nsource, ncol, dtype=dtype, device="cuda", generator=g)
        got = r.apply(x, out=torch.full((r.ntarget, ncol), float("nan"), dtype=dtype, device="cuda"))
        for c in range(ncol):
            assert torch.equal(got[:, c], r.apply(x[:, c].contiguous())), (ncol, c)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("source,target", [(8, 21), (24, 9)])
def test_infinities_and_nan(P, source, target, dtype):
    r = P.Remap(P.Mesh(source), P.Mesh(target))
    for ncol in (8, 33, 64, 137):
        print(f"remap special O{source} to O{target} {ncol} columns {dtype}", flush=True)
        g = torch.Generator(device="cuda")
        g.manual_seed(ncol)
        x = torch.randn(r.nsource, ncol, dtype=dtype, device="cuda", generator=g)
        x.view(-1)[::409] = float("inf")
        x.view(-1)[::499] = float("nan")
        x.view(-1)[::601] = -torch.finfo(dtype).max
        x.view(-1)[::701] = -float("inf")
        got = r.apply(x, out=torch.zeros((r.ntarget, ncol), dtype=dtype, device="cuda"))
        for c in range(ncol):
            one = r.apply(x[:, c].contiguous())
            assert torch.equal(got[:, c].isnan(), one.isnan()), (ncol, c)
            assert torch.equal(got[:, c].nan_to_num(nan=1.25), one.nan_to_num(nan=1.25)), (ncol, c)
