"""CPU tests of the library's host code over a stand-in for the HIP runtime
(fake_hip): what it waits for, allocates, frees and launches."""

from tests import fake_hip


def test_table_free_waits_for_the_tables_device(tmp_path):
    """The dL/dv rows are given back only after a wait for the device they
    belong to, whatever device is current, and the current one stays."""
    r = fake_hip.run(tmp_path, """
t = build(64)
assert backward(t, 1000) == 0 and backward(t, 1 << 20) == 0   # the rows, grown once
H.hipSetDevice(1)
log()
L.pwl_table_free(t)
d = ctypes.c_int(-1)
H.hipGetDevice(ctypes.byref(d))
result([log(), d.value, H.fake_live()])
""")
    calls, current, live = r
    given_back = [i for i, c in enumerate(calls) if c[0] in ("freeasync", "free")]
    assert len(given_back) == 3 and live == 0                     # two workspaces and the table
    assert ["devicesync", "0"] in calls[:given_back[0]]
    assert ["devicesync", "1"] not in calls
    assert all(calls[i][2] == "0" for i in given_back)            # with the table's device current
    assert current == 1


def test_rows_taken_under_capture_are_not_the_graphs(tmp_path):
    """A workspace that is first needed, or outgrown, while the caller's stream
    records a graph is device memory of the table's own: what the
    stream-ordered allocator gives then exists only while the graph runs."""
    r = fake_hip.run(tmp_path, """
out = []
for first in (None, 1000):                  # first needed under capture; outgrown under capture
    t = build(64)
    if first:
        assert backward(t, first) == 0
    H.fake_capture(0x5000, 1)
    log()
    assert backward(t, 1 << 20, 0x5000) == 0, L.pwl_last_error()
    H.fake_capture(0x5000, 0)
    out.append(log())
    log()
    assert backward(t, 1 << 20) == 0        # later calls use the same rows
    out.append(log())
    L.pwl_table_free(t)
    assert H.fake_live() == 0
result(out)
""")
    for captured, later in (r[:2], r[2:]):
        kinds = [c[0] for c in captured]
        assert "graphmalloc" not in kinds and kinds.count("malloc") == 1, kinds
        assert kinds.count("launch") == 2
        assert [c[0] for c in later] == ["launch", "launch"]


def test_rows_grow_in_short_memory(tmp_path):
    """With no memory for twice the rows a call takes what it needs, however
    often, after giving the outgrown ones back (all but those a captured graph
    uses), as when each growth freed the rows before it."""
    r = fake_hip.run(tmp_path, """
t = build(64)
base = H.fake_live()
need = lambda k: 4 * 65 * k                    # k workgroups of 256 threads: 1024 k points
live, waited = [], []
for k in range(1, 101):
    H.fake_malloc_limit(need(k))
    log()
    H.fake_capture(0x5000, int(k == 7))
    st = backward(t, 1024 * k, 0x5000)
    H.fake_capture(0x5000, 0)
    assert st == 0, (k, st, L.pwl_last_error())
    calls = log()
    given = [i for i, c in enumerate(calls) if c[0].startswith("free")]
    waited.append(not given or "devicesync" in [c[0] for c in calls[:given[0]]])
    live.append(H.fake_live() - base)
H.fake_malloc_limit(need(100) - 4)
refused = backward(t, 1024 * 120)
H.fake_malloc_limit(1 << 40)
after = backward(t, 1024 * 100)
L.pwl_table_free(t)
result([live, waited, refused, after, H.fake_live()])
""")
    live, waited, refused, after, end = r
    assert live[:6] == [1, 2, 1, 1, 1, 1]      # (the second is twice the first); growth gave the outgrown back ...
    assert max(live[6:8]) == 2 and live[8:] == [2] * 92   # ... but not under capture, nor the graph's
    assert all(waited)
    assert refused == -2 and after == 0 and end == 0


def test_kde_launches_cover_narrow_images_and_few_frames(tmp_path):
    """An image's tiles pad its rows by little more than threads of four pixels
    must, whatever its width; a small image's window rows are split over more
    waves even if there is one frame of them."""
    r = fake_hip.run(tmp_path, """
import re
out = []
sigma = (ctypes.c_float * 3)(6, 6, 6)
for h, w, T, rad in ((100000, 1, 2, 1), (100000, 3, 2, 1), (60000, 8, 2, 2), (62500, 16, 2, 1), (30000, 33, 2, 2),
                     (15384, 65, 16, 2), (14000, 97, 2, 2), (7692, 130, 16, 2), (7000, 200, 4, 2), (1080, 1920, 16, 2),
                     (288, 352, 1, 32), (288, 352, 1, 5), (480, 640, 1, 12)):
    log()
    assert L.pwl_kde(None, 2, A, A, h, w, T, rad, sigma, A, None) == 0
    (c,) = [c for c in log() if c[0] == "launch"]
    S = int(re.search(r"k_kdeILin?[0-9]+ELi([124])ELb[01]EE", c[1]).group(1))
    out.append((h, w, T, S, int(c[2]) * int(c[3]) * int(c[4]) // S))
result(out)
""")
    for H, W, T, S, threads in r:
        least = H * ((W + 3) // 4)
        assert threads >= least
        assert threads <= 1.17 * least + 1024, (H, W)      # a sixth, and the last rows
        if T == 1:
            assert S == 4, (H, W, S)


def test_batched_dv_of_few_tables_is_no_long_chain(tmp_path):
    """However many units a table's points are cut into, a thread of the second
    kernel adds no more of its partial sums than when a unit was a whole slice
    of 65536 points (or 64, a few rounds of loads)."""
    r = fake_hip.run(tmp_path, """
out = []
for T in (1, 2, 4, 16):
    tabs = [build(1024) for _ in range(T)]
    for total in (1 << 20, 10000000, 1 << 25, 45000000):
        b = batch(tabs, [total * k // T for k in range(T + 1)])
        log()
        assert L.pwl_batch_eval_backward(b, A, A, A, A, A, None) == 0
        k, red = [c for c in log() if c[0] == "launch"]
        out.append([T, total, int(k[2]), int(red[4]) // 256])
        L.pwl_batch_free(b)
result(out)
""")
    for T, total, units, parts in r:
        assert units // (T * parts) <= max(64, total // 65536 // T + 1), (T, total, units, parts)


def test_batch_units_of_large_tables_stay_long(tmp_path):
    """Units are cut short for small tables, where a launch has few of them, but
    not for tables whose images take as long to copy as a short unit's points;
    and a unit per table that needs no cutting keeps the full workgroup."""
    r = fake_hip.run(tmp_path, """
out = []
for N, T, total in ((4096, 512, 10000000), (4096, 512, 45000000), (4096, 64, 45000000), (4096, 512, 131072),
                    (16, 512, 10000000), (64, 64, 100003)):
    tabs = [build(N) for _ in range(T)]
    b = batch(tabs, [total * k // T for k in range(T + 1)])
    log()
    assert L.pwl_batch_eval(b, A, A, None) == 0
    assert L.pwl_batch_eval_backward(b, A, A, A, A, A, None) == 0
    fwd, bwd, _ = [c for c in log() if c[0] == "launch"]
    out.append([int(fwd[2]), int(fwd[4]), int(bwd[2]), int(bwd[4])])
    L.pwl_batch_free(b)
    for t in tabs:
        L.pwl_table_free(t)
result(out)
""")
    (_, _, a, _), (_, _, b, _), (_, _, c, _), (_, threads, _, bthreads), (_, _, d, _), (e, _, f, _) = r
    assert a <= 664 and b <= 1885 and c <= 750   # slices of 65536, 32768 and 65536 points, split at the tables
    assert threads == 1024 and bthreads == 1024
    assert d >= 512 and e >= 40 and f >= 40


def test_batch_creation_uploads_at_once(tmp_path):
    """Creating a batch copies the tables' descriptors, their deepest cells and
    everything else in one copy each, however many lists the plan has."""
    r = fake_hip.run(tmp_path, """
tabs = [build(n) for n in (16, 300, 4096)]
log()
b = batch(tabs, [0, 1 << 20, 1 << 22, 1 << 24])
result([c[0] for c in log()])
""")
    assert r.count("copy") == 3 and r.count("malloc") == 1 and r.count("launch") == 1


def test_large_launches_have_full_workgroups(tmp_path):
    """The sizes the GPU tests of the staging take: 1024 threads of four vectors
    past one and a half workgroups per compute unit forward, the tuned shape past
    one backward, and 256 threads of one vector for small launches."""
    r = fake_hip.run(tmp_path, """
out = []
L.pwl_set_launch.argtypes = [i32] * 4
for N in (300, 1024, 4096):
    t = build(N)
    for shape, n in (((4, 1024, 32), 256 * 1024 * 4 * 4 * 3 // 2 + 4099), ((1, 256, 32), 50000)):
        assert L.pwl_set_launch(0, *shape) == 0
        log()
        assert L.pwl_eval(t, None, A, A, n, None) == 0
        c = log()[0]
        out.append([c[1], int(c[4]), shape])
    for shape in ((2, 768, 1), (4, 1024, 1)):
        assert L.pwl_set_launch(1, *shape) == 0
        log()
        assert backward(t, 256 * shape[1] * shape[0] * 4 + 4099) == 0
        c = [c for c in log() if c[0] == "launch"][0]
        out.append([c[1], int(c[4]), shape])
result(out)
""")
    for name, threads, (unroll, block, _) in r:
        assert threads == block and "ILi%dE" % unroll in name, (name, threads)
