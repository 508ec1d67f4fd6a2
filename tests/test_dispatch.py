"""Which kernels a call launches, over which grid, for shapes that no test
device holds, and what a context keeps when memory is short: the library's host
side over a stand-in for the HIP runtime (hip_stub.c), without a GPU."""
from __future__ import annotations

import pytest

from hip_stub import host_calls  # noqa: F401  (fixture)


def test_ordinary_calls_launch(host_calls):
    """The stand-in serves the library: a step of each dimension launches its
    kernels within the runtime's limits, and destroy frees what create took."""
    out = host_calls(r'''
out = []
for shape in ((200, 1, 1), (300, 200, 1), (800, 700, 1), (20, 18, 17)):
    h = create(shape)
    stub.stub_clear()
    rc = L.weno_l2is_step(h, U, 1e-3)
    out.append([rc, launches()])
    L.weno_l2is_destroy(h)
    out[-1].append(stub.stub_used())
''')
    for (rc, ls, used), k in zip(out, ("row_kernel<3", "tile2d_kernel", "row_kernel<4", "fused3d_kernel")):
        assert rc == 0 and used == 0
        assert sum(k in r[0] for r in ls) == 3


@pytest.mark.parametrize("nx,ny,kw", [(2, 40_000_000, {"hybrid": 2}), (64, 21_000_001, {"hybrid": 2, "split": 1}),
                                      (1, 100_000_000, {"hybrid": 2, "split": 2})])
def test_tall_grids_launch(host_calls, nx, ny, kw):
    """2D grids with every face WENO of more tiles than one launch holds:
    accepted, and every tile has its workgroup."""
    rcs, ls = host_calls(f'''
h = create(({nx}, {ny}, 1), **{kw!r})
stub.stub_clear()
rcs = [L.weno_l2is_rhs_ctx(h, U, V), L.weno_l2is_step(h, U, 1e-9), L.weno_l2is_advance(h, U, 2, 1.0)]
out = [rcs, launches()]
''')
    assert rcs == [0, 0, 0]
    tiles = -(-nx // 63) * -(-ny // 3)
    stages = [r for r in ls if "tile2d_kernel<3" in r[0]]
    assert all(r[1] * r[4] < 1 << 32 and r[2:4] == [1, 1] and r[4] == 448 for r in stages)
    assert sum(r[1] for r in stages) == (1 + 3 + 6) * tiles


@pytest.mark.parametrize("kw", [{}, {"split": 1}, {"bc": [1, 1, 4, 5, 1, 1]}])
def test_wide_grids_take_the_tile_kernel(host_calls, kw):
    """2D grids wider than the row kernel's 32-bit column offsets reach run on
    the tile kernel, however they are tuned; the widest that they reach, on the
    row kernel."""
    out = host_calls(f'''
out = []
for nx in (1 << 29, (1 << 29) + 1, 700_000_000):
    h = create((nx, 2, 1), **{kw!r})
    for tune in ((0, 0, 0), (2, 0, 0), (0, 2, 0), (3, 0, 0)):
        assert L.weno_l2is_tune(h, *tune) == 0
        stub.stub_clear()
        rcs = [L.weno_l2is_rhs_ctx(h, U, V), L.weno_l2is_step(h, U, 1e-9), L.weno_l2is_advance(h, U, 2, 1.0)]
        out.append([nx, rcs, launches()])
''')
    for nx, rcs, ls in out:
        assert rcs == [0, 0, 0]
        row = sum("row_kernel<4" in r[0] for r in ls)
        tiles = sum(r[1] for r in ls if "tile2d_kernel<3" in r[0])
        assert (row, tiles) == ((10, 0) if nx == 1 << 29 else (0, 10 * -(-nx // 63)))
        assert nx == 1 << 29 or not any("ghost_fill" in r[0] for r in ls)  # the tile kernel forms them


# a batched engine; admit(k): a run of scheme k (0: the default one, whose stage
# kernels are a build of their own) from device memory
BATCH = r'''
b = C.c_void_p()
assert L.weno_l2is_batch_create(1 << 28, 64, None, C.byref(b)) == 0
def admit(scheme, shape=(100, 80, 1)):
    p = capi.params_default(*shape, 0.1, split=2 if scheme else 0)
    slot = C.c_int(-1)
    assert L.weno_l2is_batch_admit(b, *shape, 0.1, 1.4, C.byref(p), U, 0, 1.0, C.byref(slot), None) == 0
    return slot.value
def fetch(slot):
    assert L.weno_l2is_batch_fetch(b, slot, V, 0, None, None, None) == 0
'''


def test_batch_graph_outlives_its_launches(host_calls):
    """No captured graph is destroyed before the stream has run what was
    launched of it: a run of another scheme class, a new launch shape, more
    work items than the tables held, and destroy."""
    lines = host_calls(BATCH + r'''
admit(0); admit(0)
assert L.weno_l2is_batch_advance(b, 3) == 0
s = admit(1)
assert L.weno_l2is_batch_advance(b, 2) == 0
assert L.weno_l2is_batch_tune(b, 1, 0) == 0
assert L.weno_l2is_batch_advance(b, 2) == 0
assert L.weno_l2is_batch_tune(b, 0, 512) == 0
assert L.weno_l2is_batch_advance(b, 2) == 0
admit(0, (400, 400, 1)); admit(0, (700, 700, 1))
assert L.weno_l2is_batch_advance(b, 2) == 0
fetch(s)
assert L.weno_l2is_batch_advance(b, 2) == 0
L.weno_l2is_batch_destroy(b)
out = log()
''')
    running, destroyed = set(), 0
    for l in lines:
        op, *a = l.split()
        if op == "graph":
            running.add(a[0])
        elif op == "sync":
            running.clear()
        elif op == "destroy":
            assert a[0] not in running, lines
            destroyed += 1
    assert destroyed >= 3 and sum(l.startswith("graph") for l in lines) == 13


def test_batch_scheme_classes_keep_their_graphs(host_calls):
    """Runs of another scheme that come and go switch between two captured
    graphs; neither is captured again."""
    lines = host_calls(BATCH + r'''
admit(0)
for k in range(6):
    s = admit(1)
    assert L.weno_l2is_batch_advance(b, 1) == 0
    fetch(s)
    assert L.weno_l2is_batch_advance(b, 1) == 0
out = log()
L.weno_l2is_batch_destroy(b)
''')
    graphs = [l.split()[1] for l in lines if l.startswith("graph")]
    assert graphs == ["1", "2"] * 6
    assert sum(l == "capture" for l in lines) == 2


@pytest.mark.parametrize("nx", [1 << 27, (1 << 27) + 1])
def test_cached_rhs_keeps_to_the_3d_march_width(host_calls, nx):
    """The stateless right-hand side of one shape with the hybrid switch (whose
    cached context holds a face buffer), then with every face WENO: rows wider
    than the 32-bit offsets of the kernels per direction take the stage kernel
    with per-cell corrections, as on a context made for that scheme."""
    out = host_calls(f'''
def names():
    return sorted(n.split("(")[0].split("<")[0].split("::")[-1] for n, *_ in launches())
out = []
shape = ({nx}, 2, 2)
for hybrid in (0, 2, 0):
    p = capi.params_default(*shape, 0.1, hybrid=hybrid)
    stub.stub_clear()
    assert L.weno_l2is_rhs(U, *shape, 0.1, 1.4, C.byref(p), V) == 0
    out.append(names())
h = create(shape, hybrid=2)
stub.stub_clear()
assert L.weno_l2is_rhs_ctx(h, U, V) == 0
out.append(names())
''')
    hybrid, every, again, ctx = out
    march = nx <= 1 << 27
    assert ("weno3d_x_kernel" in every) == march and ("weno_fix3d_kernel" in every) == (not march)
    assert "weno_flist3d_kernel" not in every
    assert [n for n in ctx if "reset" not in n] == [n for n in every if "reset" not in n]
    assert "weno_flist3d_kernel" in hybrid and "weno_flist3d_kernel" in again


@pytest.mark.parametrize("shape,zchunk", [((1, 100_000_000, 2), 1), ((2, 3, 90_000_000), 1), ((3, 70_000_000, 2), 0),
                                          ((64, 50, 40), 1), ((64, 50, 40), 2_000_000_000)])
def test_3d_march_lengths_launch(host_calls, shape, zchunk):
    """Any tuned length of the marches along y and z launches: every cell has
    its lane, within the runtime's limit."""
    rcs, ls = host_calls(f'''
h = create({shape}, hybrid=2)
assert L.weno_l2is_tune(h, 0, {zchunk}, 0) == 0
stub.stub_clear()
rcs = [L.weno_l2is_rhs_ctx(h, U, V), L.weno_l2is_step(h, U, 1e-9)]
out = [rcs, launches()]
''')
    nx, ny, nz = shape
    assert rcs == [0, 0]
    marches = [r for r in ls if "weno3d_march_kernel" in r[0]]
    assert len(marches) == 8
    for name, gx, gy, gz, threads in marches:
        assert gx * threads < 1 << 32 and (gy, gz, threads) == (1, 1, 64)
        groups, n = (-(-nx * nz // 64), ny) if name.split(",")[1].strip() == "1" else (-(-nx * ny // 64), nz)
        assert gx % groups == 0 and 1 <= gx // groups <= n
        if zchunk == 1 and groups * n * 64 < 1 << 32:
            assert gx == groups * n


@pytest.mark.parametrize("bc", [0, 1])
def test_longest_1d_grids(host_calls, bc):
    """advance() of 1D grids near 2^31 cells (223 GB with their context): those
    whose positions would run past 2^31 in the whole-step kernels take the
    stage kernels."""
    out = host_calls(f'''
out = []
for n in (505, (1 << 31) - 1 - (1 << 20), (1 << 31) - (1 << 20)):
    h = create((n, 1, 1), bc=[{bc}, {bc}, 1, 1, 1, 1])
    stub.stub_clear()
    rc = L.weno_l2is_advance(h, U, 3, 1.0)
    out.append([n, rc, launches()])
''')
    for n, rc, ls in out:
        assert rc == 0
        line = [r for r in ls if "line_step_kernel" in r[0]]
        stage = [r for r in ls if "row_kernel<3" in r[0]]
        assert (len(line), len(stage)) == ((3, 0) if n < (1 << 31) - (1 << 20) else (0, 9))
        for name, gx, _, _, threads in ls:  # a lane's first index and one stride beyond the grid
            if "line_cfl" in name:
                assert n + gx * threads < 1 << 31
        for _, gx, _, _, threads in line:
            assert gx == -(-n // 46) and gx * 46 + 64 < 1 << 31 and gx * threads < 1 << 32


@pytest.mark.parametrize("split", [1, 2])
def test_3d_sums_leave_room(host_calls, split):
    """3D with every face WENO and a splitting other than LLF: where the running
    sums, with what else the context needs and the caller's state, do not fit
    the device, create() keeps the per-cell corrections; with the memory that
    those need it succeeds."""
    out = host_calls(f'''
shape, n = (64, 60, 50), 64 * 60 * 50
def used(capacity, expect=0, **kw):
    stub.stub_capacity(capacity)
    h = create(shape, hybrid=2, split={split}, expect=expect)
    if expect:
        return stub.stub_used()
    u = stub.stub_used()
    stub.stub_capacity(1 << 62)
    stub.stub_clear()
    assert L.weno_l2is_step(h, U, 1e-9) == 0
    march = any("weno3d_x" in r[0] for r in launches())
    L.weno_l2is_destroy(h)
    return [u, march]
full = used(1 << 62)
cells = full[0] - 80 * n
out = [full, cells]
out += [used(c) for c in (full[0] + 40 * n, full[0] + 40 * n - 1, full[0], full[0] - 1, cells)]
out.append(used(cells - 1, expect=capi.E_NOMEM))
''')
    full, cells, room, less, tight, short, least, refused = out
    assert full[1] and room == full
    assert less == tight == short == least == [cells, False]
    assert refused == 0


@pytest.mark.parametrize("nx,ny,kw,tile", [(500, 400, {}, True), (900, 700, {"hybrid": 2}, True), (900, 700, {}, False)])
def test_2d_face_once_buffers_leave_room(host_calls, nx, ny, kw, tile):
    """The face-once buffers of a 2D grid that the tile kernel serves are not
    needed: short of memory a context does without them, and with rows set by
    tune() takes per-cell corrections then."""
    out = host_calls(f'''
shape, n = ({nx}, {ny}, 1), {nx} * {ny}
def used(capacity, expect=0):
    stub.stub_capacity(capacity)
    h = create(shape, expect=expect, **{kw!r})
    if expect:
        return [stub.stub_used(), None, None]
    u = stub.stub_used()
    stub.stub_capacity(1 << 62)
    kinds = []
    for rows in (0, 5):
        assert L.weno_l2is_tune(h, 0, rows, 0) == 0
        stub.stub_clear()
        assert L.weno_l2is_step(h, U, 1e-9) == 0
        names = " ".join(r[0] for r in launches())
        kinds.append("tile" if "tile2d" in names else "face" if "row_face" in names else "cell")
    L.weno_l2is_destroy(h)
    return [u, *kinds]
full = used(1 << 62)
out = [n, full, used(full[0] + 32 * n), used(full[0] + 32 * n - 1, 0), used(full[0], 0)]
out.append(used(full[0] - 1, {0 if tile else -6}))
''')
    n, full, room, less, tight, short = out
    assert full[1:] == ["tile" if tile else "face", "face"] and room == full
    if tile:
        assert less == tight == short == [full[0] - 68 * n, "tile", "cell"]
    else:
        assert less == tight == full and short[0] == 0


def test_batch_rows_name_two_builds(host_calls):
    """The rows that the autotuner tries each have their build of the stage
    kernels, and a value that names the build in use captures nothing."""
    out = host_calls(BATCH + r'''
from paper_1908_02464_amd import autotune
admit(0)
out = []
for rows in autotune.BATCH_ROWS + (3, 4, 16, 62, 2, 1, 0):
    assert L.weno_l2is_batch_tune(b, rows, 0) == 0
    stub.stub_clear()
    assert L.weno_l2is_batch_advance(b, 1) == 0
    out.append([rows, sum(l == "capture" for l in log(False)), sorted({n for n, *_ in launches() if "batch_stage" in n})])
out = [len(autotune.BATCH_ROWS), out]
L.weno_l2is_batch_destroy(b)
''')
    n, runs = out
    builds = [tuple(k) for _, c, k in runs[:n]]
    assert all(c == 1 for _, c, _ in runs[:n]) and len(set(builds)) == n
    assert [c for _, c, _ in runs[n:]] == [0, 0, 0, 0, 1, 0, 0]


@pytest.mark.parametrize("shape,kw", [((900, 1, 1), {"hybrid": 2}), ((900, 1, 1), {"split": 1}), ((800, 700, 1), {}),
                                      ((24, 20, 18), {})])
def test_captured_stages_clear_their_lists(host_calls, shape, kw):
    """A stage with a correction list that is captured into a graph clears the
    list's counters itself, since a replay starts from what the last one left;
    so does every stage of that context afterwards, and none before."""
    out = host_calls(f'''
h = create({shape}, stream=1 << 12, **{kw!r})
def calls():
    stub.stub_clear()
    assert [L.weno_l2is_rhs_ctx(h, U, V), L.weno_l2is_step(h, U, 1e-9)] == [0, 0]
    return ["reset" if "reset" in n else "stage" for n, *_ in launches()
            if "reset" in n or "row_kernel" in n or "fused3d_kernel" in n]
out = [calls(), calls()]
stub.stub_capturing(1)
out.append(calls())
stub.stub_capturing(0)
out.append(calls())
''')
    first, eager, captured, after = out
    assert first == ["reset"] * 2 + ["stage"] * 4 and eager == ["stage"] * 4
    assert captured == after == (["reset"] * 2 + ["stage"]) * 4
