"""Which kernels calls launch, on a runtime that records launches instead of
running them."""
import pytest

from host_util import on_host


@pytest.mark.parametrize("N,layout,first", [
    # first levels of the register-staged sweep (FP64, FP32)
    (160, None, (999, 999)), (240, None, (180, 999)), (320, None, (100, 161)),
    (400, None, (60, 161)), (500, None, (48, 161)), (320, (16, 24), (91, 201)),
    (320, (8, 16), (999, 999)),
])
def test_gradient_lonlat(N, layout, first):
    """d/dlon and d/dlat read their scales by position, so the packed sweep
    cannot serve them, and the register-staged one needs many tiles or long
    columns: flat and column forms before.  (FP32 from 20 to 79 levels on large
    meshes besides; not 241 to 256 levels.)"""
    result = on_host(f"""
m = P.Mesh({N}, layout={layout!r})
result = [(nlev, dt, launches(L.atlas_nabla_gradient_lonlat, m.handle, IN, nlev, dt, OUT, None)[-1][0])
          for nlev in (1, 4, 12, 19, 20, 23, 24, 37, 47, 48, 59, 60, 79, 80, 90, 91, 99, 100, 137,
                       160, 161, 179, 180, 200, 201, 240, 241, 256, 257, 300) for dt in (F64, F32)]
""")
    for nlev, dt, kernel in result:
        staged = nlev >= first[1 - dt] and not 240 < nlev <= 256
        if N == 500:
            staged |= (dt == 0 and 20 <= nlev < 80) or (dt == 1 and nlev >= 48)
        want = "k_sweepv" if staged else "k_flat" if nlev < 24 else "k_col"
        assert want in kernel, (nlev, dt, kernel)


def _forms(N, layout, calls):
    return on_host(f"""
m = P.Mesh({N}, layout={layout!r})
result = [apply(m, op, nlev, dt)[-1][0] for op, nlev, dt in {calls!r}]
""")


@pytest.mark.parametrize("N,layout,calls", [
    # (operator, levels, dtype) of calls too short for the sweep, and the
    # shortest that take it
    (500, None, [(0, 2, 1), (1, 2, 1), (1, 4, 0), (0, 4, 0)]),
    (320, None, [(0, 3, 1), (0, 4, 0), (1, 4, 0), (1, 3, 1)]),
    (640, None, [(0, 2, 1), (1, 2, 0)]),
    (320, (8, 16), [(0, 8, 1), (0, 9, 0), (1, 6, 0), (1, 5, 1)]),
    (160, None, [(0, 12, 1), (0, 13, 0), (1, 12, 0), (1, 11, 1)]),
    (160, (8, 8), [(0, 3, 1), (0, 10, 0), (1, 20, 0), (1, 1, 1)]),
])
def test_short_columns_keep_the_flat_form(N, layout, calls):
    for call, kernel in zip(calls, _forms(N, layout, calls)):
        assert "k_flat" in kernel, (call, kernel)


@pytest.mark.parametrize("N,layout,calls", [
    (500, None, [(0, 3, 1), (1, 3, 1), (0, 5, 0), (1, 5, 0)]),
    (320, None, [(0, 4, 1), (0, 5, 0), (1, 5, 0), (1, 4, 1)]),
    (640, None, [(0, 3, 1), (1, 1, 1), (1, 3, 0), (0, 4, 0)]),
    (320, (8, 16), [(0, 9, 1), (0, 10, 0), (1, 7, 0), (1, 6, 1), (1, 137, 0), (1, 260, 0)]),
    (160, None, [(0, 13, 1), (0, 14, 0), (1, 13, 0), (1, 12, 1)]),
    (160, (8, 8), [(0, 60, 1), (1, 260, 1), (0, 170, 0)]),
    (640, (8, 8), [(0, 22, 1), (1, 14, 0)]),
    (640, (8, 16), [(0, 7, 1), (1, 5, 1), (0, 7, 0)]),
    (256, None, [(1, 193, 0), (1, 200, 0)]), (180, None, [(1, 260, 0)]),
])
def test_longer_columns_take_the_sweep(N, layout, calls):
    for call, kernel in zip(calls, _forms(N, layout, calls)):
        assert "k_sweepw" in kernel, (call, kernel)


def test_columns_on_small_tiles_keep_the_column_form():
    for kernel in _forms(160, (8, 8), [(0, 37, 1), (1, 137, 0), (1, 60, 1), (0, 60, 0)]):
        assert "k_col" in kernel, kernel
    for kernel in _forms(320, (8, 16), [(1, 104, 0), (1, 200, 0)]):
        assert "k_col" in kernel, kernel
    for kernel in _forms(200, None, [(1, 220, 0), (1, 260, 0)]):
        assert "k_col" in kernel, kernel


def test_one_pass_divergence_and_curl_of_short_columns():
    """Two results from one read: the sweep from the first vector."""
    result = on_host("""
m = P.Mesh(500)
result = [launches(L.atlas_nabla_div_curl, m.handle, IN, nlev, dt, OUT, OUT2, None)
          for nlev, dt in ((1, F64), (2, F64), (2, F32), (4, F32))]
""")
    for calls in result:
        assert len(calls) == 1 and "k_sweepw" in calls[0][0], calls


def test_long_fp32_columns_on_lane_vectors():
    """FP32 vector columns of 193 to 256 levels in one chunk of four levels
    per lane; FP32 gradients above 256 levels on lane vectors."""
    result = on_host("""
m = P.Mesh(nx=P.regular_gaussian_nx(24))
result = [apply(m, op, nlev, F32)[0][0] for op, nlev in ((DIV, 193), (CURL, 256), (GRAD, 257), (GRAD, 300))]
result.append(launches(L.atlas_nabla_div_curl, m.handle, IN, 200, F32, OUT, OUT2, None)[0][0])
""")
    result.append(_forms(200, None, [(1, 220, 0)])[0])
    div, curl, g257, g300, both, o200 = result
    assert "k_colvIfLi1ELi4ELi1E" in o200
    assert "k_colvIfLi1ELi4ELi1E" in div and "k_colvIfLi2ELi4ELi1E" in curl
    assert "k_colvIfLi0E" in g257 and "k_colvIfLi0E" in g300
    assert "k_colv_dcIfLi4ELi1E" in both


@pytest.mark.parametrize("N,nlev,dt,lanes,elements,pieces,lds", [
    # chunks of 13 to 16 vectors, two workgroups to a compute unit: on half
    # tiles, two elements on 16 lanes
    (640, 80, 1, 16, 2, 3440 * 3, 68320),
    (640, 60, 1, 16, 2, 3440 * 2, 72224),
    (640, 120, 1, 16, 2, 3440 * 4, 72224),
    (640, 100, 1, 16, 2, 3440 * 4, 64416),
    (640, 170, 0, 16, 2, 3440 * 3, 72800),
    # 72 levels would leave chunks of 12
    (640, 72, 1, 16, 5, 3440, 154208),
    # one chunk of 38 stays one
    (640, 75, 1, 16, 5, 3440, 162016),
    # not eight lanes with four or five elements ...
    (640, 30, 1, 16, 2, 1720, 133920),
    (640, 36, 1, 16, 3, 1720, 155616),
    (640, 80, 0, 16, 3, 3440, 92320),
    # ... but for 34 to 36 of FP32
    (640, 72, 0, 8, 5, 1720, 156704),
])
def test_fused_laplacian_chunks(N, nlev, dt, lanes, elements, pieces, lds):
    (name, blocks, threads, used), = on_host(f"""
m = P.Mesh({N})
result = apply(m, LAPL, {nlev}, {dt})
""")
    assert f"k_lsweepwI{'d' if dt else 'f'}Li{lanes}ELi{elements}E" in name
    assert (blocks, used) == ((pieces + 7) // 8 * 8, lds)
    assert threads == 512 or 2 * lds > 160 * 1024


@pytest.mark.parametrize("N,nlev,dt,fused", [
    (160, 46, 1, False), (160, 47, 1, True), (160, 128, 1, True),
    (120, 80, 1, False), (120, 81, 1, True),
    (180, 36, 1, False), (180, 37, 1, True), (200, 30, 1, True),
    (200, 60, 1, True), (320, 37, 1, True),
    (200, 149, 0, False), (200, 150, 0, True), (220, 124, 0, False), (220, 137, 0, True),
    (320, 63, 0, False), (320, 64, 0, True), (320, 80, 0, True), (256, 137, 0, True),
])
def test_fused_laplacian_on_few_tiles(N, nlev, dt, fused):
    names = [k[0] for k in on_host(f"m = P.Mesh({N})\nresult = apply(m, LAPL, {nlev}, {dt})")]
    assert len(names) == (1 if fused else 2) and ("k_lsweepw" in names[0]) == fused, names


@pytest.mark.parametrize("N", [2, 16, 160])
def test_upload_takes_few_allocations(N):
    """A small mesh's upload is bound by its allocations and copies: its arrays
    come in one, beside the packed records'."""
    assert on_host(f"""
m = P.Mesh({N})
result = H.host_hip_allocs()
""") <= 10


@pytest.mark.parametrize("N,share", [(160, 0.9), (160, 0.73), (500, 0.83)])
def test_a_mesh_that_fits_without_the_sweeps_plans(N, share):
    """Where the device has no room for the wave-specialised forms' plans and
    records, a mesh goes without them and its calls take the other forms."""
    result = on_host(f"""
m = P.Mesh({N})
full = H.host_hip_used()
m.close()
left = H.host_hip_used()
H.host_hip_limit(int({share} * full))
m = P.Mesh({N})
used = H.host_hip_used() - left
names = [apply(m, op, nlev, dt)[-1][0] for op in (GRAD, DIV, CURL) for dt in (F64, F32)
         for nlev in (1, 5, 37, 137, 300)]
names += [launches(L.atlas_nabla_div_curl, m.handle, IN, nlev, dt, OUT, OUT2, None)[-1][0]
          for dt in (F64, F32) for nlev in (5, 37, 137)]
H.host_hip_limit(-1)  # (two passes ask for their intermediate)
names += [apply(m, LAPL, nlev, dt)[-1][0] for dt in (F64, F32) for nlev in (1, 37, 137)]
result = [int(m.info.device_bytes), used, left, names]
""")
    assert result[0] == result[1] and result[2] == 0
    assert not [n for n in result[3] if "sweepw" in n], result[3]


def test_a_mesh_too_large_for_the_device_is_refused():
    assert on_host("""
H.host_hip_limit(20 << 20)
try:
    P.Mesh(160)
    result = "uploaded"
except P.AtlasError as e:
    result = [str(e), H.host_hip_used()]
""")[1] == 0


def test_arrays_read_once_leave_the_store():
    """What only the packing of the records reads is freed after it."""
    used, wide = on_host("""
m = P.Mesh(320)
result = [H.host_hip_used(), int(m.info.nnodes)]
""")
    assert used < 1550 * wide


@pytest.mark.parametrize("op", [0, 1, 2, 3])
def test_fp32_flux_form_takes_no_flux_workspace(op):
    """FP32 fields run the column form in its place: only a Laplacian's
    gradient needs memory."""
    used, flux64 = on_host(f"""
m = P.Mesh(80)
flux = P.Launch(P.VARIANT_FLUX, 256, 0, 0, 0, 0)
before = H.host_hip_used()
names = apply(m, {op}, 40, F32, flux)
used = H.host_hip_used() - before
assert all("k_col" in n[0] for n in names), names
assert any("flux" in n[0] for n in apply(m, {op}, 40, F64, flux))
result = [used, H.host_hip_used() - before]
""")
    V = sum(4 * (20 + 4 * j) for j in range(80)) // 2
    assert used <= (V * 40 * 8 + 4096 if op == 3 else 0)
    assert flux64 > used


_TUNE = """
import ctypes
def tune(m, nlev, dt):
    best, ms = P.Launch(), ctypes.c_float()
    names = launches(L.atlas_autotune, m.handle, LAPL, IN, nlev, dt, OUT, OUT2, None,
                     ctypes.byref(best), ctypes.byref(ms))
    return best, [(n, t) for n, g, t, l in names if "lsweep" in n]
"""


def test_autotuned_laplacian_tries_the_built_in_block():
    """... and every block once that the fused form launches differently with."""
    result = on_host(_TUNE + """
m = P.Mesh(320)
result = []
for nlev, dt in ((137, F64), (80, F64), (37, F64), (200, F32)):
    built = apply(m, LAPL, nlev, dt)[-1]
    best, fused = tune(m, nlev, dt)
    result.append([built, best.variant, best.block_threads, fused, apply(m, LAPL, nlev, dt)[-1]])
""")
    for built, variant, block, fused, now in result:
        assert "k_lsweepw" in built[0] and variant == 5
        assert fused[0][1] == built[2] == block  # (all equal on this clock: the first is kept)
        blocks = [t for _, t in fused]
        assert sorted(set(blocks)) == sorted({512, 768, built[2]})
        assert len(blocks) == 4 * len(set(blocks))  # a warm-up and three timed
        assert now == built


def test_autotuned_laplacian_keeps_the_faster_form():
    """The two passes where the fused form is slower."""
    result = on_host(_TUNE + """
H.host_hip_slow(b"k_lsweep")
m = P.Mesh(320)
best, fused = tune(m, 137, F64)
names = [n[0] for n in apply(m, LAPL, 137, F64)]
result = [best.variant, len(fused), names]
""")
    assert result[0] != 5 and result[1] > 0 and len(result[2]) == 2
    assert not [n for n in result[2] if "lsweep" in n]


@pytest.mark.parametrize("layout", [(92, 24), (63, 40), (62, 16), (64, 9)])
def test_tall_bands_run_the_wave_specialised_forms(layout):
    """The layouts of test_gpu_tall_bands.py, by explicit launch shapes."""
    result = on_host(f"""
m = P.Mesh(46, layout={layout!r})
result = []
for nlev in (4, 5, 37, 96, 137):
    for dt in (F64, F32):
        for block in (512, 1024):
            result += [apply(m, op, nlev, dt, P.Launch(P.VARIANT_SWEEP, block, 0, 0, 0, 0))[-1][0]
                       for op in (GRAD, DIV, CURL)]
        for block in (512, 768):
            result.append(apply(m, LAPL, nlev, dt, P.Launch(P.VARIANT_FUSED, block, 0, 0, 0, 0))[-1][0])
""")
    assert len(result) == 80
    for name in result:
        assert "sweepw" in name, name


def test_built_in_forms_of_the_parity_cases():
    """Which of the sizes that other tests compare as "built in" take the
    one-pass Laplacian (FP64 first) and the one-pass sweep."""
    fused, dc = on_host("""
fused = []
for N, nlev in ((160, 45), (160, 137), (240, 24), (240, 137)):
    m = P.Mesh(N)
    for dt in (F64, F32):
        names = [n[0] for n in apply(m, LAPL, nlev, dt)]
        fused.append("k_lsweepw" in names[0] if len(names) == 1 else False)
    m.close()
m = P.Mesh(320)
dc = [launches(L.atlas_nabla_div_curl, m.handle, IN, nlev, dt, OUT, OUT2, None)
      for nlev in (2, 5, 16, 37, 47, 64, 91, 96, 97, 137) for dt in (F64, F32)]
result = [fused, [[n[0] for n in c] for c in dc]]
""")
    assert fused == [False, False, True, False, True, False, True, True]
    # 2 levels: flat; 37 and 47 (FP32: 47): two column passes; FP32 above: one
    forms = ["".join(sorted({f for f in ("flat", "sweepw", "colv_dc", "colvI") if f in "".join(c)}))
             for c in dc]
    assert forms == (["flat"] * 2 + ["sweepw"] * 4 + ["colvI", "sweepw"] + ["colvI"] * 2 +
                     ["sweepw", "colv_dc"] * 5)


@pytest.mark.parametrize("nlev,positions", [(2, 256), (3, 256), (4, 256), (5, 204), (20, 51)])
def test_flat_blocks_of_large_meshes(nlev, positions):
    """A block's values are one pass of its threads, or a part of one."""
    V, launch = on_host(f"""
m = P.Mesh(nx=P.regular_gaussian_nx(400))
result = [int(m.info.nnodes), apply(m, GRAD, {nlev}, F32)[-1]]
""")
    name, blocks, threads, _ = launch
    per = (V + positions - 1) // positions
    assert "k_flat" in name and threads == 1024 and blocks == (per + 7) // 8 * 8


def test_built_in_laplacians_that_take_no_memory():
    """The one pass needs no workspace, so a Laplacian on such a mesh can be
    called during a capture or on several streams at once: by values alone, also
    on tiles of few nodes and at the fewest values."""
    result = on_host("""
result = []
for N, layout, calls in ((320, (4, 4), [(4, F64), (37, F64), (260, F64), (64, F32)]),
                         (320, (8, 8), [(4, F64), (137, F64), (33, F32), (260, F32)]),
                         (180, None, [(37, F64), (40, F64), (184, F32)])):
    m = P.Mesh(N, layout=layout)
    H.host_hip_limit(H.host_hip_used())
    result += [[n[0] for n in apply(m, LAPL, nlev, dt)] for nlev, dt in calls]
    H.host_hip_limit(-1)
    m.close()
""")
    for names in result:
        assert len(names) == 1 and "lsweepw" in names[0], names


@pytest.mark.parametrize("nlev,tried", [(10, False), (23, False), (24, True), (137, True)])
def test_batch_tuning_of_short_columns(nlev, tried):
    """One level per lane is no candidate for a batch's short columns: what it
    gains alone it loses in the persistent kernel."""
    names = on_host(f"""
m = P.Mesh(48)
item = (P._abi.WorkItem * 1)()
item[0].mesh, item[0].op, item[0].nlev, item[0].in_, item[0].out = m.handle, GRAD, {nlev}, IN, OUT
cfg, batch = P._abi.BatchConfig(F32, 0, 1, 0, 0, -1), ctypes.c_void_p()
result = [n[0] for n in launches(L.atlas_batch_build, item, 1, ctypes.byref(cfg), None,
                                 ctypes.byref(batch))]
""")
    assert any("k_columnIf" in n for n in names) == tried, names
    assert any("k_colvIf" in n for n in names) and any("k_flatIf" in n for n in names)
