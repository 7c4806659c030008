"""fsg_simulate_noalloc, the entry point for callers that cannot allocate
device memory (its workspace is a static device array): through the C-ABI,
two calls in a row -- the second on a smaller graph with fewer replicates,
so stale contents of the shared array would show -- give the bits of
fsg_simulate with a caller workspace (and of the oracle); a run larger than
the array is refused before anything is launched."""
import numpy as np
import pytest

from paper_2603_14895_amd import workloads as W
from tests.gpu_util import assert_same, gpu_run, log, oracle_run

pytestmark = pytest.mark.gpu


def _noalloc(gnp, model, seeds, B, key, replicate_offset=0, **kw):
    import torch
    from paper_2603_14895_amd import fsg
    ptr, src = gnp
    g = fsg.DeviceGraph(ptr, src)
    prm, _keep = fsg.make_params(model, **kw)
    states = torch.empty((g.n, B), dtype=torch.uint8, device="cuda")
    counts = torch.empty(g.n, dtype=torch.int32, device="cuda")
    seeds = np.ascontiguousarray(seeds, dtype=np.int32)
    info = fsg.fsg_simulate_noalloc(g.handle, prm, seeds.ctypes.data, seeds.size, B,
                                    replicate_offset, key, None, states.data_ptr(),
                                    counts.data_ptr(), fsg._stream_ptr())
    out = (states.cpu().numpy(), counts.cpu().numpy().astype(np.uint32), int(info.steps_run),
           int(info.absorbed))
    g.close()
    return out


def test_noalloc_matches_workspace_entry_point_twice():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    log(f"[noalloc] static scratch {fsg.lib().fsg_simulate_noalloc_limit()} bytes")
    # first call: SIR, 1024 replicates (16 words per node), heavy rows
    big = W.chung_lu(20000, 12.0, 2.5, 3101).numpy()
    seeds = W.uniform_seeds(20000, 40, 3102)
    kw = dict(beta=0.04, gamma=0.1, max_steps=40)
    log("[noalloc] call 1: SIR n=20000 B=1024")
    a = _noalloc(big, "sir", seeds, 1024, 0xA110C, replicate_offset=3, **kw)
    ref = gpu_run(big, "sir", seeds, 1024, 0xA110C, replicate_offset=3, **kw)
    assert_same(a, ref, "noalloc SIR vs fsg_simulate")
    assert_same(a, oracle_run(big, "sir", seeds, 1024, 0xA110C, replicate_offset=3, **kw),
                "noalloc SIR vs oracle")
    # second call, smaller: IC on 3000 nodes, 100 replicates, to absorption
    small = W.chung_lu(3000, 8.0, 2.5, 3103).numpy()
    s2 = W.uniform_seeds(3000, 7, 3104)
    log("[noalloc] call 2: IC n=3000 B=100")
    b = _noalloc(small, "ic", s2, 100, 0xB0B, p=0.1, max_steps=-1)
    ref2 = gpu_run(small, "ic", s2, 100, 0xB0B, p=0.1, max_steps=-1)
    assert_same(b, ref2, "noalloc IC vs fsg_simulate")
    assert_same(b, oracle_run(small, "ic", s2, 100, 0xB0B, p=0.1, max_steps=-1),
                "noalloc IC vs oracle")
    # and once more at the first size: the array is reused, nothing stale
    c = _noalloc(big, "sir", seeds, 1024, 0xA110C, replicate_offset=3, **kw)
    assert_same(c, ref, "noalloc SIR again")


def test_noalloc_refuses_runs_beyond_the_array():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    gnp = W.chung_lu(200000, 4.0, 2.5, 3105).numpy()
    g = fsg.DeviceGraph(*gnp)
    prm, _ = fsg.make_params("sir", beta=0.02, gamma=0.1, max_steps=5)
    need = fsg.fsg_sim_workspace_size(g.handle, prm, 4096, None)
    assert need > fsg.lib().fsg_simulate_noalloc_limit()
    seeds = np.array([1, 2], dtype=np.int32)
    with pytest.raises(fsg.FsgError) as e:
        fsg.fsg_simulate_noalloc(g.handle, prm, seeds.ctypes.data, 2, 4096, 0, 1, None, None,
                                 None, fsg._stream_ptr())
    assert e.value.code == fsg.FSG_EWORKSPACE and "static scratch" in str(e.value)
    g.close()


def test_noalloc_accepts_what_fits_with_the_largest_tiles():
    """A run whose default tiles need more than the scratch holds, but which
    fits with the largest default tile, is run with that."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    kw = dict(beta=0.1, gamma=0.2, max_steps=6)
    limit = fsg.lib().fsg_simulate_noalloc_limit()
    prm, _keep = fsg.make_params("sir", **kw)

    def ring(n):  # node v pulls from its four predecessors
        v = np.arange(n, dtype=np.int64)
        src = ((v[:, None] - np.arange(1, 5)) % n).astype(np.int32)
        return np.arange(n + 1, dtype=np.int64) * 4, np.ascontiguousarray(src.ravel())

    def needs(n):
        ptr, src = ring(n)
        g = fsg.fsg_graph_create(n, 4 * n, ptr.ctypes.data, src.ctypes.data)
        out = [fsg.fsg_sim_workspace_size(g, prm, 1024, fsg.make_schedule(s))
               for s in (dict(), dict(tile_edges=4096))]
        fsg.fsg_graph_destroy(g)
        return out

    lo, hi = 100000, 200000  # largest n whose run fits with the largest tiles
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if needs(mid)[1] <= limit else (lo, mid)
    assert needs(lo)[0] > limit >= needs(lo)[1]
    gnp = ring(lo)
    seeds = W.uniform_seeds(lo, 50, 3111)
    assert_same(_noalloc(gnp, "sir", seeds, 1024, 0xF17, **kw),
                gpu_run(gnp, "sir", seeds, 1024, 0xF17, **kw), "noalloc at the scratch's limit")


def test_noalloc_without_the_row_table():
    """A run that fits the scratch but for the table of its tiles' rows by
    in-degree is run without it."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    kw = dict(beta=0.1, gamma=0.2, max_steps=6)
    limit = fsg.lib().fsg_simulate_noalloc_limit()
    prm, _keep = fsg.make_params("sir", **kw)
    sched = dict(tile_edges=4096)

    def ring(n, k=4):  # node v pulls from its k predecessors
        v = np.arange(n, dtype=np.int64)
        src = ((v[:, None] - np.arange(1, k + 1)) % n).astype(np.int32)
        return np.arange(n + 1, dtype=np.int64) * k, np.ascontiguousarray(src.ravel())

    def need(n):
        ptr, src = ring(n)
        g = fsg.fsg_graph_create(n, 4 * n, ptr.ctypes.data, src.ctypes.data)
        out = fsg.fsg_sim_workspace_size(g, prm, 1024, fsg.make_schedule(sched))
        fsg.fsg_graph_destroy(g)
        return out

    lo, hi = 100000, 200000
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if need(mid) <= limit else (lo, mid)
    n = lo + lo // 100  # a hundredth more: 8 of some 400 bytes a row are the table's
    assert need(n) > limit
    gnp = ring(n)
    seeds = W.uniform_seeds(n, 50, 3111)
    assert_same(_noalloc(gnp, "sir", seeds, 1024, 0xF18, **kw),
                gpu_run(gnp, "sir", seeds, 1024, 0xF18, **kw), "noalloc without the row table")


# (nodes, in-arcs of each, model, replicates, schedule): runs that need within
# half a percent of the array
AT_THE_LIMIT = [
    (8000, 1000, "sir", 22336, None), (4000, 1500, "lt", 3520, None), (1000, 5000, "ic", 67008, None),
    (4000, 1024, "ic", 6976, dict(heavy_threshold=64)), (1000, 5000, "sir", 832, dict(heavy_threshold=64)),
    (4000, 1024, "lt", 3520, dict(heavy_threshold=600)), (4000, 1500, "lt", 3520, dict(tile_edges=64)),
]


@pytest.mark.parametrize("n,deg,model,B,sched", AT_THE_LIMIT)
def test_noalloc_at_the_limit_with_wide_rows(n, deg, model, B, sched):
    """Runs on wide rows whose tables do not fit beside the planes: with the
    smallest workspace (those rows light, merges by a launch), the same
    result."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_14895_amd import fsg
    v = np.arange(n, dtype=np.int64)
    src = np.ascontiguousarray(((v[:, None] - np.arange(1, deg + 1)) % n).astype(np.int32).ravel())
    g = fsg.DeviceGraph(np.arange(n + 1, dtype=np.int64) * deg, src)
    kw = dict(ic=dict(p=1.0 / deg, max_steps=3), lt=dict(max_steps=3),
              sir=dict(beta=1.5 / deg, gamma=0.2, max_steps=3))[model]
    seeds = W.uniform_seeds(n, n // 50, 3201)
    prm, _keep = fsg.make_params(model, **kw)
    schedule = fsg.make_schedule(sched) if sched else None
    assert fsg.fsg_sim_workspace_size(g.handle, prm, B, schedule) > 0.99 * fsg.lib().fsg_simulate_noalloc_limit()
    sim = fsg.Simulation(g, model, B, schedule=sched, want_states=False, **kw)
    want = sim.run(seeds, 0x11A1)
    counts = torch.empty(n, dtype=torch.int32, device="cuda")
    info = fsg.fsg_simulate_noalloc(g.handle, prm, seeds.ctypes.data, seeds.size, B, 0, 0x11A1, schedule,
                                    None, counts.data_ptr(), fsg._stream_ptr())
    assert int(info.steps_run) == int(want.steps_run) and torch.equal(counts, sim.counts)
    g.close()
