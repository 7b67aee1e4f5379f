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
