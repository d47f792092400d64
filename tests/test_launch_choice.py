"""Which launch a tuning gets: the autotuner's winner is no slower than the
untuned call, and a shape index past a class's list is the untuned call."""
import ctypes

import pytest

from paper_1311_5304_amd import _binding as B
from paper_1311_5304_amd import autotune

FRAME = {"width": 256, "height": 256, "h": (2, 1, 1), "v": (2, 1, 1), "qsel": (0, 1, 1)}


@pytest.mark.parametrize("untuned", [5.5, 6.5])
def test_tuned_is_no_slower_than_untuned(monkeypatch, untuned):
    """A clock that knows the candidates' times: 6.0 ms for one of them, more
    for the others, and what the library's own choice takes."""
    now = {}
    monkeypatch.setattr(autotune, "shapes", lambda *a: [{"mcus_x": 16, "mcus_y": 2, "threads": 192, "resident_per_cu": 3,
                                                         "cu_count": 256}] * 2)
    monkeypatch.setattr(B, "mjd_ctx_get_tuning", lambda ctx: {"seg_subtiles": 0, "workgroups": 0, "shape": 0})
    monkeypatch.setattr(B, "mjd_ctx_set_tuning", lambda ctx, seg, wg, shape=0: now.update(seg=seg, wg=wg, shape=shape))

    def clock(fn, reps, warmup=3):
        if (now["seg"], now["wg"], now["shape"]) == (0, 0, 0):
            return untuned
        return 6.0 + 0.1 * (now["seg"] != 2) + 0.1 * (now["shape"] != 1)
    monkeypatch.setattr(autotune, "_time_ms", clock)
    best, table = autotune.tune(None, FRAME, [None], None, B.MJD_UPSAMPLE_SIMPLE, [None])
    assert all(r["seg_subtiles"] > 0 for r in table)
    got = (best["seg_subtiles"], best["shape"])
    assert got == ((0, 0) if untuned < 6.0 else (2, 1))
    entry = autotune._entry(best, table, ("seg_subtiles", "workgroups_per_cu"))
    assert entry["seg_subtiles"] == best["seg_subtiles"] and entry["workgroups"] == best["workgroups"]
    assert now == {"seg": 0, "wg": 0, "shape": 0}


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class KernelNodeParams(ctypes.Structure):
    """hipKernelNodeParams"""
    _fields_ = [("block", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", Dim3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


@pytest.mark.gpu
@pytest.mark.parametrize("h,v,mode,width,height", [(2, 2, "simple", 256, 256), (2, 1, "simple", 256, 256),
                                                   (1, 1, "fancy", 256, 256), (2, 1, "fancy", 256, 256),
                                                   (2, 1, "fancy", 1921, 1081), (2, 2, "fancy", 1024, 768)])
def test_index_past_the_list_is_the_default_launch(h, v, mode, width, height):
    """The captured launch (kernel, grid, lanes) is that of no tuning at all."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_5304_amd as M

    hip = ctypes.CDLL("libamdhip64.so")
    ctx = M.Context(0)
    frame = {"width": width, "height": height, "h": (h, 1, 1), "v": (v, 1, 1), "qsel": (0, 1, 1)}
    g = M.mjd_geometry_of(frame)
    coef = torch.zeros((g["n_blocks"] * 64,), dtype=torch.int16, device="cuda")
    qt = torch.ones(256, dtype=torch.int16, device="cuda")
    out = torch.empty((height, width, 3), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()

    def launch(shape):
        M.mjd_ctx_set_tuning(ctx, 0, 0, shape)
        M.mjd_decode(ctx, frame, coef, qt, M.UPSAMPLE[mode], out, 3 * width, 0, g["mcus_y"], stream)
        torch.cuda.synchronize()
        graph, n = ctypes.c_void_p(), ctypes.c_size_t()
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 2) == 0  # relaxed
        M.mjd_decode(ctx, frame, coef, qt, M.UPSAMPLE[mode], out, 3 * width, 0, g["mcus_y"], stream)
        assert hip.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0 and n.value == 1
        nodes, p = (ctypes.c_void_p * 1)(), KernelNodeParams()
        assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(nodes[0]), ctypes.byref(p)) == 0
        seen = (p.func, p.grid.x, p.block.x)
        assert hip.hipGraphDestroy(graph) == 0
        return seen

    try:
        default, past = launch(0), launch(200)
        print(h, v, mode, width, height, default[1:], past[1:], flush=True)
        assert default[2] in (128, 192, 256, 512) and past == default
        listed = launch(1)
        assert listed != default
    finally:
        M.mjd_ctx_set_tuning(ctx, 0, 0, 0)
        ctx.close()
