"""Point arrays at every 4-byte offset from each other's 16-byte boundaries,
and tables around the sizes at which the staging changes (one word per
thread, or a copy loop), with workgroups from one wave to sixteen: forward
and fused backward against the FP64 oracle on the GPU's own table, and bit
for bit against the same points in aligned arrays."""

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests.gpu_util import GRAD_TOL, Y_TOL, device, launch_shape, library, records_layout, say

pytestmark = pytest.mark.gpu


def _at(dev, a, shift):
    """a copied to the device, `shift` elements past a 16-byte boundary."""
    base = torch.empty(len(a) + 8, dtype=torch.float32, device=dev)
    v = base[shift:shift + len(a)]
    v.copy_(torch.from_numpy(a))
    return v


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 63, 257, 4099, 70001])
def test_every_phase(n):
    import paper_1510_02975_amd as P
    library()
    dev = device()
    say("phases, n=%d" % n)
    t = P.pwl_build(O.GAUSSIAN, (1.0, 1.0), -5.0, 5.0, 100, O.OPTIMAL, O.PROJ)
    d = P.pwl_table_download(t)
    X, v = d["knots"].astype(np.float64), d["values"].astype(np.float64)
    xh, gh = W.normal_points(n, 2.5, 7), W.upstream_grad(n, 8)
    x64, g64 = xh.astype(np.float64), gh.astype(np.float64)
    yr, _, dvr = O.evaluate_backward(X, v, x64, g64)
    _, _, wk = O.evaluate_backward(X, np.zeros(len(X)), x64, np.abs(g64))
    y0, dx0, _ = P.pwl_eval_backward(t, _at(dev, xh, 0), _at(dev, gh, 0), want=("y", "dx"))
    assert np.max(np.abs(y0.cpu().numpy() - yr)) <= Y_TOL
    guard = torch.tensor([7.0] * 4, device=dev)
    for px in range(4):
        x = _at(dev, xh, px)
        for py in range(4):
            base = torch.full((n + 8,), 7.0, device=dev)
            y = base[4 + py - 4:][:n] if py else base[:n]
            P.pwl_eval(t, x, y)
            assert torch.equal(y, y0), (px, py)
            assert torch.equal(base[py + n:][:4], guard[:len(base[py + n:][:4])])   # nothing written past the end
            assert torch.all(base[:py] == 7.0)
    for phases in ((0, 1, 2, 3), (3, 3, 0, 1), (1, 0, 0, 2), (2, 1, 3, 3), (0, 0, 1, 1)):
        x, g = _at(dev, xh, phases[0]), _at(dev, gh, phases[1])
        yb, db = (torch.full((n + 8,), 7.0, device=dev) for _ in range(2))
        y, dx = yb[phases[2]:][:n], db[phases[3]:][:n]
        _, _, dv = P.pwl_eval_backward(t, x, g, y=y, dx=dx)
        assert torch.equal(y, y0) and torch.equal(dx, dx0), phases
        for b, p in ((yb, phases[2]), (db, phases[3])):
            assert torch.all(b[:p] == 7.0) and torch.all(b[p + n:] == 7.0), phases
        assert np.all(np.abs(dv.cpu().numpy() - dvr) <= GRAD_TOL * wk + 1e-30), phases
        _, _, dv1 = P.pwl_eval_backward(t, x, g, want=("dv",))
        assert np.all(np.abs(dv1.cpu().numpy() - dvr) <= GRAD_TOL * wk + 1e-30), phases
    z = _at(dev, xh, 1)
    assert torch.equal(P.pwl_eval(t, z, z), y0)      # in place
    t.free()


@pytest.mark.parametrize("N", [63, 64, 127, 192, 193, 255, 256, 511, 512, 768, 769, 1023, 1024, 1025, 2048,
                               3072, 3073, 4095, 4096])
@pytest.mark.parametrize("shape", [(1, 64, 1), (2, 256, 2), (4, 1024, 32)], ids=["64", "256", "1024"])
def test_staging_sizes(N, shape):
    """The Lorentzian's map has 8 N cells up to N = 2048 (the map is then the
    section that decides), the Gaussian's 4 N."""
    import paper_1510_02975_amd as P
    library()
    dev = device()
    n = 50021
    for func, a, b in ((O.GAUSSIAN, -5.0, 5.0), (O.LORENTZIAN, -20.0, 20.0)):
        t = P.pwl_build(func, (1.0, 1.0), a, b, N, O.OPTIMAL, O.INTERP)
        d = P.pwl_table_download(t)
        X, v = d["knots"].astype(np.float64), d["values"].astype(np.float64)
        xh, gh = W.uniform_points(a - 0.5, b + 0.5, n, N), W.upstream_grad(n, 3)
        xh[:N + 1] = d["knots"]
        x64, g64 = xh.astype(np.float64), gh.astype(np.float64)
        yr, _, dvr = O.evaluate_backward(X, v, x64, g64)
        _, _, wk = O.evaluate_backward(X, np.zeros(len(X)), x64, np.abs(g64))
        x, g = torch.from_numpy(xh).to(dev), torch.from_numpy(gh).to(dev)
        vo = torch.from_numpy((1.0 + 0.5 * np.cos(np.arange(N + 1))).astype(np.float32)).to(dev)
        with launch_shape(P, P.KERNEL_FORWARD, shape), launch_shape(P, P.KERNEL_BACKWARD, shape[:2] + (1,)):
            y = P.pwl_eval(t, x)
            yb, _, dv = P.pwl_eval_backward(t, x, g)
            yo = P.pwl_eval(t, x, v_override=vo)
            ybo, _, _ = P.pwl_eval_backward(t, x, g, v_override=vo, want=("y",))
            assert np.array_equal(P.pwl_locate(t, x).cpu().numpy(), O.locate(X, x64))
        assert np.max(np.abs(y.cpu().numpy() - yr)) <= Y_TOL
        assert torch.equal(yb, y) and torch.equal(yo, ybo)
        yor = O.evaluate(X, vo.cpu().numpy().astype(np.float64), x64)
        assert np.max(np.abs(yo.cpu().numpy() - yor)) <= 4e-6 * 1.5
        assert np.all(np.abs(dv.cpu().numpy() - dvr) <= GRAD_TOL * wk + 1e-30)
        t.free()


@pytest.mark.parametrize("N", [64, 4096])
@pytest.mark.parametrize("vectors_per_cu", [1, 256, 512, 768, 1024, 2048, 4096])
def test_small_launch_edges(N, vectors_per_cu):
    """Point counts one vector to either side of where the shape of a small
    launch changes: every point and every gradient against the oracle."""
    import paper_1510_02975_amd as P
    library()
    dev = device()
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    t = P.pwl_build(O.GAUSSIAN, (1.0, 1.0), -5.0, 5.0, N, O.OPTIMAL, O.PROJ)
    d = P.pwl_table_download(t)
    X, v = d["knots"].astype(np.float64), d["values"].astype(np.float64)
    for n in (4 * cus * vectors_per_cu - 3, 4 * cus * vectors_per_cu, 4 * cus * vectors_per_cu + 5):
        xh, gh = W.normal_points(n, 1.5, 5), W.upstream_grad(n, 6)
        x64, g64 = xh.astype(np.float64), gh.astype(np.float64)
        yr, _, dvr = O.evaluate_backward(X, v, x64, g64)
        _, _, wk = O.evaluate_backward(X, np.zeros(len(X)), x64, np.abs(g64))
        x, g = torch.from_numpy(xh).to(dev), torch.from_numpy(gh).to(dev)
        y = P.pwl_eval(t, x)
        yb, _, dv = P.pwl_eval_backward(t, x, g)
        say("small launches N=%d n=%d" % (N, n))
        assert np.max(np.abs(y.cpu().numpy() - yr)) <= Y_TOL
        assert torch.equal(yb, y)
        assert np.all(np.abs(dv.cpu().numpy() - dvr) <= GRAD_TOL * wk + 1e-30)
    t.free()


@pytest.mark.parametrize("layout", ["packed", "pairs"])
@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 191, 192, 193, 767, 768, 769, 1024, 1025, 3071, 3072, 3073, 4096])
def test_staging_sizes_of_other_records(N, layout):
    """The other record layouts around the sizes where their image is staged
    through registers or copied, with the table's values and with given ones."""
    import paper_1510_02975_amd as P
    library()
    dev = device()
    t = P.pwl_build(O.LORENTZIAN, (1.0, 1.0), -20.0, 20.0, N, O.OPTIMAL, O.INTERP)
    d = P.pwl_table_download(t)
    X = d["knots"].astype(np.float64)
    xh = np.concatenate([d["knots"], W.uniform_points(-21.0, 21.0, 30011, N)]).astype(np.float32)
    x = torch.from_numpy(xh).to(dev)
    vh = (1.0 + 0.5 * np.cos(np.arange(N + 1))).astype(np.float32)
    vo = torch.from_numpy(vh).to(dev)
    with records_layout(P, {"packed": P.RECORDS_PACKED, "pairs": P.RECORDS_PAIRS}[layout]):
        for shape in ((1, 64, 1), (2, 256, 2), (4, 1024, 32)):
            with launch_shape(P, P.KERNEL_FORWARD, shape):
                y, yo = P.pwl_eval(t, x), P.pwl_eval(t, x, v_override=vo)
            for got, v in ((y, d["values"]), (yo, vh)):
                ref = O.evaluate(X, v.astype(np.float64), xh.astype(np.float64))
                assert np.max(np.abs(got.cpu().numpy() - ref)) <= Y_TOL * max(1.0, np.max(np.abs(v)))
    t.free()


@pytest.mark.parametrize("layout", ["packed", "soa", "pairs"])
@pytest.mark.parametrize("N", [1023, 1024, 1025, 2047, 2048, 3071, 3072, 3073, 4096])
def test_staging_in_full_workgroups(N, layout):
    """The same thresholds in the 1024-thread workgroups of large launches
    (more than one and a half of them per compute unit): a section's first
    word per thread, its further words and the copied rest of a map of 8 N
    cells, up to three records per thread and past them.  Bit for bit what
    small launches of 256 threads give for the same points, with the table's
    values and with given ones."""
    import paper_1510_02975_amd as P
    library()
    dev = device()
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    n = cus * 1024 * 4 * 4 * 3 // 2 + 4 * 1024 + 3
    t = P.pwl_build(O.LORENTZIAN, (1.0, 1.0), -20.0, 20.0, N, O.OPTIMAL, O.INTERP)
    assert t.info()[5] == (8 * N if N <= 2048 else 4 * N)
    d = P.pwl_table_download(t)
    x = torch.empty(n, device=dev).uniform_(-21.0, 21.0, generator=torch.Generator(device=dev).manual_seed(N))
    x[:N + 1] = torch.from_numpy(d["knots"]).to(dev)
    vo = torch.from_numpy((1.0 + 0.5 * np.cos(np.arange(N + 1))).astype(np.float32)).to(dev)
    say("full workgroups N=%d %s n=%d" % (N, layout, n))
    with records_layout(P, {"packed": P.RECORDS_PACKED, "soa": P.RECORDS_SOA, "pairs": P.RECORDS_PAIRS}[layout]):
        with launch_shape(P, P.KERNEL_FORWARD, (4, 1024, 32)):
            y, yo = P.pwl_eval(t, x), P.pwl_eval(t, x, v_override=vo)
        with launch_shape(P, P.KERNEL_FORWARD, (1, 256, 32)):
            step = 50000
            for b in range(0, n, step):
                xs = x[b:b + step]
                assert torch.equal(y[b:b + step], P.pwl_eval(t, xs)), b
                assert torch.equal(yo[b:b + step], P.pwl_eval(t, xs, v_override=vo)), b
    t.free()


@pytest.mark.parametrize("N", [300, 1024, 2048, 4096])
@pytest.mark.parametrize("shape", [(2, 768, 1), (4, 1024, 1), (2, 1024, 2)], ids=["2x768", "4x1024", "2x1024"])
def test_backward_in_full_workgroups(N, shape):
    """The fused backward past its small launches: y and dx bit for bit, and
    dL/dv within the gradients' bound, what calls on pieces of the points give."""
    import paper_1510_02975_amd as P
    library()
    dev = device()
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    n = cus * shape[1] * shape[0] * 4 + 4099
    t = P.pwl_build(O.LORENTZIAN, (1.0, 1.0), -20.0, 20.0, N, O.OPTIMAL, O.PROJ)
    gen = torch.Generator(device=dev).manual_seed(N)
    x = torch.empty(n, device=dev).uniform_(-21.0, 21.0, generator=gen)
    g = torch.empty(n, device=dev).normal_(generator=gen)
    vo = torch.from_numpy((1.0 + 0.5 * np.cos(np.arange(N + 1))).astype(np.float32)).to(dev)
    say("full backward workgroups N=%d shape %s n=%d" % (N, shape, n))
    for v in (None, vo):
        with launch_shape(P, P.KERNEL_BACKWARD, shape):
            y, dx, dv = P.pwl_eval_backward(t, x, g, v_override=v)
        want, weight = (torch.zeros(N + 1, dtype=torch.float64, device=dev) for _ in range(2))
        step = 100000
        for b in range(0, n, step):
            xs, gs = x[b:b + step], g[b:b + step]
            ys, dxs, dvs = P.pwl_eval_backward(t, xs, gs, v_override=v)
            assert torch.equal(y[b:b + step], ys) and torch.equal(dx[b:b + step], dxs), b
            want += dvs
            weight += P.pwl_eval_backward(t, xs, gs.abs(), v_override=v, want=("dv",))[2]
        assert torch.all((dv - want).abs() <= GRAD_TOL * weight + 1e-30)
    t.free()
