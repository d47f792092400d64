"""The batch kernel's segment queue when not every workgroup is resident: more
workgroups than the device holds, and two batches at once on two streams.
Every launch, replays included, writes the bytes that the single-image kernel
writes (compared with the oracle elsewhere): whole numbers, no tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1311_5304_amd as mod
    return mod


@pytest.fixture(scope="module")
def ctx(M):
    c = M.Context(0)
    yield c
    c.close()


def images(M, ctx, seed, n):
    """(jobs, expected) of n images of mixed size and sampling."""
    rng = np.random.default_rng(seed)
    jobs, expected = [], []
    for i in range(n):
        w, h = int(rng.integers(200, 1500)), int(rng.integers(200, 1500))
        s = ((1, 1), (2, 1), (2, 2))[i % 3]
        frame = {"width": w, "height": h, "h": (s[0], 1, 1), "v": (s[1], 1, 1), "qsel": (0, 1, 1)}
        k = M.mjd_geometry_of(frame)["n_blocks"]
        coef = torch.from_numpy((rng.standard_normal((k, 64)) * (40 / (1 + np.arange(64)))).astype(np.int16)).cuda()
        qt = torch.from_numpy(rng.integers(1, 17, 256).astype(np.int16)).cuda()
        expected.append(M.decode(ctx, frame, coef, qt, "fancy"))
        jobs.append((frame, coef, qt, torch.empty_like(expected[-1]), 3 * w))
    torch.cuda.synchronize()
    return jobs, expected


def check(jobs, expected, what):
    torch.cuda.synchronize()
    for i, (j, e) in enumerate(zip(jobs, expected)):
        assert torch.equal(j[3], e), (what, i)
        j[3].fill_(0xA5)


@pytest.mark.parametrize("seg", [1, 3])
def test_more_workgroups_than_are_resident(M, ctx, seg):
    jobs, expected = images(M, ctx, seg, 24)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for workgroups in (1, 7, 2 * cus, 2 * cus + 1, 4 * cus, 1 << 20):
        M.mjd_ctx_set_tuning(ctx, seg, workgroups, 0)
        try:
            b = M.Batch(ctx, jobs, M.MJD_UPSAMPLE_FANCY)
        finally:
            M.mjd_ctx_set_tuning(ctx, 0, 0, 0)
        info = b.info()
        assert info["workgroups"] == min(workgroups, info["segments"])
        print(seg, workgroups, info, flush=True)
        for graph in (False, True, True):
            b.launch(use_graph=graph)
            check(jobs, expected, (workgroups, graph))
        b.close()


def test_two_batches_at_once(M, ctx):
    sets = [images(M, ctx, 10 + k, 12) for k in range(2)]
    streams = [torch.cuda.Stream() for _ in sets]
    for workgroups in (0, 1 << 20):
        M.mjd_ctx_set_tuning(ctx, 2, workgroups, 0)
        try:
            plans = [M.Batch(ctx, jobs, M.MJD_UPSAMPLE_FANCY) for jobs, _ in sets]
        finally:
            M.mjd_ctx_set_tuning(ctx, 0, 0, 0)
        for rep in range(3):
            torch.cuda.synchronize()
            for _ in range(3):
                for p, s in zip(plans, streams):
                    p.launch(use_graph=False, stream=s)
            torch.cuda.synchronize()
            for jobs, expected in sets:
                check(jobs, expected, (workgroups, rep))
        for p in plans:
            p.close()
