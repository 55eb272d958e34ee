"""GPU: the graph build refuses slices whose total degree 2m_s reaches 2^31, also where the sums
of repeated pairs leave 32 bits (to 0, to a negative value, or to a small positive one), from
host and from device edge lists; totals right below the bound are built as given."""
import ctypes as C

import numpy as np
import pytest

from paper_2608_03695_amd import gen

pytestmark = pytest.mark.gpu

TOP = 2 ** 31 - 1


def _graph(weights, extra=()):
    """Two slices; the second holds the edge (0, 1) once per weight, then the extra edges."""
    edges = [(2, 3, 1)], [(0, 1, w) if k % 2 else (1, 0, w) for k, w in enumerate(weights)]
    return gen.from_edge_lists(5, [edges[0], edges[1] + list(extra)], weighted=True, name="heavy")


def _create(mslm, tg, on_device):
    if not on_device:
        g = mslm.Graph(tg, 1)
        info = g.info()
        g.close()
        return info
    import torch
    d, keep = mslm._desc(tg, 1)
    dev = [torch.from_numpy(a).cuda() for a in keep[1:4]]
    torch.cuda.synchronize()
    d.src, d.dst, d.weight = (t.data_ptr() for t in dev)
    d.flags |= mslm.MSLM_INPUT_ON_DEVICE
    h, out = C.c_void_p(), [C.c_int64() for _ in range(3)]
    mslm._check(mslm.load().mslm_create(C.byref(d), None, C.byref(h)))
    mslm._check(mslm.load().mslm_graph_info(h, *map(C.byref, out)))
    mslm.load().mslm_destroy(h)
    return dict(zip(("n_supra", "nnz", "two_m"), (x.value for x in out)))


@pytest.mark.parametrize("on_device", [False, True], ids=["host", "device"])
@pytest.mark.parametrize("weights", [[2 ** 30] * 4, [TOP, TOP], [TOP] * 4 + [5], [2 ** 30],
                                     [2 ** 29] * 2], ids=["zero", "negative", "small", "one", "two"])
def test_totals_beyond_the_bound_are_refused(weights, on_device):
    from paper_2608_03695_amd import mslm
    with pytest.raises(mslm.MslmError) as e:
        _create(mslm, _graph(weights), on_device)
    assert e.value.status == mslm.MSLM_EOVERFLOW


@pytest.mark.parametrize("on_device", [False, True], ids=["host", "device"])
@pytest.mark.parametrize("count", [1, 2, 255, 32767, 32768, 32769, 70001])
def test_totals_below_the_bound_are_built(count, on_device):
    """As many copies of an edge as one block totals, one fewer and one more."""
    from paper_2608_03695_amd import mslm
    most = 2 ** 30 - 1
    weights = [most // count] * count
    weights[0] += most - sum(weights) - 3
    info = _create(mslm, _graph(weights, [(3, 4, 3)]), on_device)
    assert info == dict(n_supra=10, nnz=2 + 4 + 10, two_m=2 + 2 * most)


def test_unweighted_totals_count_every_listed_edge():
    from paper_2608_03695_amd import mslm
    tg = gen.from_edge_lists(4, [[(0, 1)] * 7 + [(2, 3)], [], [(1, 2)] * 5000], name="repeats")
    g = mslm.Graph(tg, 1)
    assert g.info()["two_m"] == 16 + 10000
    g.close()
