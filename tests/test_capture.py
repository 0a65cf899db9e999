"""Maps under stream capture.  A map call plans on the host and stages its plan in
memory that the thread's next call rewrites, so a graph of it would read another
call's plan when it is replayed: the call is refused, in either precision, and
leaves nothing in the graph.  On the host runtime for tests, and captured on a GPU."""
import fake_hip
import pytest

CODE = r"""
g, t, out = dd.Grid(0, 0, %s, %s, 48, 40), (C.c_double * 2)(1e-5, 1e-3), buf(2 * 48 * 40)
calls = [lambda p: lib.dd_damage_map(s.handle, C.byref(g), t, 2, p, ptr(out), 1, None),
         lambda p: lib.dd_damage_sweep(s.handle, C.byref(g), 1e-5, 1e-3, 2, p, ptr(out), 1, None)]
s = scan(32, 32, "random", seed=1)
for prec in (0, 1):
    for call in calls:
        ok(call(prec))
        launches()
        fake.fake_capture(1)
        rc = call(prec)
        fake.fake_capture(0)
        assert rc == -3, rc
        names = [name for name, _, _ in launches() if "lag_rows" not in name]
        assert not names, names
        ok(call(prec))
"""


@pytest.mark.parametrize("px", ["1e-9", "0.37e-9"], ids=["lattice", "fp64"])
def test_refused(tmp_path, px):
    fake_hip.run(tmp_path, CODE % (px, px))


@pytest.mark.gpu
def test_refused_on_gpu():
    import numpy as np
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd

    scan = dd.Scan(32, 32, "random", seed=1)
    args = (0.0, 0.0, 1e-9, 1e-9, 48, 40, [1e-5, 1e-3], "fp64")
    want = scan.damage_map(*args).cpu().numpy()
    x = torch.zeros(4, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x += 1
        with pytest.raises(dd.DDError):
            scan.damage_map(*args)
    graph.replay()
    torch.cuda.synchronize()
    assert x.tolist() == [1.0] * 4
    assert np.array_equal(scan.damage_map(*args).cpu().numpy(), want)
