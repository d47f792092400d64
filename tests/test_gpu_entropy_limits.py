"""GPU entropy decoding at the edges of its dispatch, each reached for sure
(the batch says how it is decoded): more stream bytes than one pass over them
holds, more chunks than the small workgroups hold, long and short split
intervals together, and chains of chunks that break.  Coefficients are whole
numbers: no tolerance."""
import random

import numpy as np
import pytest

from synth import encode, fast_bitstream, images

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LUMA = {"444": (1, 1), "422": (2, 1), "420": (2, 2)}


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


def job(M, data, coef=None):
    scan, _ = M.mjd_parse(data)
    off = M.mjd_restart_index(data, scan)
    d_jpg = torch.zeros(-(-len(data) // 16) * 16, dtype=torch.uint8, device="cuda")
    d_jpg[:len(data)] = torch.from_numpy(np.frombuffer(data, dtype=np.uint8).copy()).cuda()
    if coef is None:
        coef = torch.full((M.mjd_geometry_of(M.scan_frame(scan))["n_blocks"] * 64,), 0x5A5A, dtype=torch.int16, device="cuda")
    return scan, off, d_jpg, len(data), coef


def photograph(w, h, quality, interval=0, seed=3, samp="420"):
    """(coefficients, file)"""
    frame, coef, qt = encode.encode_rgb(images.texture_rgb(w, h, seed, sigma=12), samp, quality)
    return coef, fast_bitstream.write_jpeg(frame, coef, qt, restart_interval=interval)


def check(M, ctx, streams):
    """Decodes the streams as one batch, twice; how it was decoded."""
    jobs = [job(M, data) for _, data in streams]
    b = M.EntropyBatch(ctx, jobs)
    for rep in range(2):
        for j in jobs:
            j[4].fill_(0x5A5A)
        b.launch()
        assert b.status() == -1
        for i, ((coef, _), j) in enumerate(zip(streams, jobs)):
            assert np.array_equal(j[4].cpu().numpy().reshape(-1, 64), coef), (rep, i)
    s = b.splits()
    b.close()
    return s


@pytest.mark.parametrize("quality", [95, 98])
@pytest.mark.parametrize("interval", [0, 64])
def test_dense_photographs_break_chains(M, ctx, quality, interval):
    print(f"1024x768, quality {quality}, markers every {interval}", flush=True)
    s = check(M, ctx, [photograph(1024, 768, quality, interval, seed) for seed in (3, 31)])
    assert s["intervals"] > 1
    if interval == 0:
        assert s["mended"] > 4


def periodic(seed, w=512, h=256):
    """(coefficients, file) of blocks that repeat every one to three MCUs: a
    lane that starts in the wrong place may never find the right one."""
    rng = np.random.default_rng(seed)
    samp = ("420", "444", "422")[seed % 3]
    hy, vy = LUMA[samp]
    bpm, n = hy * vy + 2, (w // (8 * hy)) * (h // (8 * vy))
    period = int(rng.integers(1, 4))
    pat = np.zeros((period * bpm, 64), dtype=np.int16)
    m = rng.random(pat.shape) < rng.choice([0.05, 0.2, 0.5, 0.9])
    pat[m] = rng.integers(-3, 4, int(m.sum()))
    if rng.random() < 0.5:
        pat[:] = pat[rng.integers(0, period * bpm)]
    pat[:, 0] = rng.integers(-5, 6)
    coef = np.tile(pat, (n // period + 1, 1))[:n * bpm]
    frame = {"width": w, "height": h, "h": (hy, 1, 1), "v": (vy, 1, 1), "qsel": (0, 1, 1)}
    return coef, fast_bitstream.write_jpeg(frame, coef, np.ones((4, 64), dtype=np.uint16))


def test_content_that_repeats(M, ctx):
    """Chains that break at every place, and lanes that go on for long."""
    s = check(M, ctx, [periodic(seed) for seed in (0, 5, 10, 31, 42, 44)])
    assert s["intervals"] == 6 and s["mended"] > 6


def test_damage_after_a_break_is_found(M, ctx):
    coef, data = photograph(640, 480, 98)
    scan, _ = M.mjd_parse(data)
    rnd = random.Random(8)
    bad = 0
    for k in range(8):
        b = bytearray(data)
        p = rnd.randrange((scan.data_offset + scan.data_end) // 2, scan.data_end)
        if b[p] != 0xFF and b[p - 1] != 0xFF:
            b[p] ^= 1 << rnd.randrange(7)
        b = bytes(b)
        host = np.zeros_like(coef)
        try:
            s2, _ = M.mjd_parse(b)
            M.mjd_entropy_decode(b, s2, M.mjd_restart_index(b, s2), host, 0, 30, 1)
            ok = True
        except M.MjdError:
            ok = False
        j = job(M, b)
        e = M.EntropyBatch(ctx, [j])
        e.launch()
        if ok:
            assert e.status() == -1
            assert np.array_equal(j[4].cpu().numpy().reshape(-1, 64), host)
        else:
            with pytest.raises(M.MjdError) as ei:
                e.status()
            assert ei.value.code == -5
        assert e.splits()["mended"] > 0
        e.close()
        bad += not ok
    assert bad > 0


def test_more_chunks_than_small_workgroups_hold(M, ctx):
    """The 512-lane shape that follows the boundaries of a large batch, and
    long and short split intervals in one list."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    streams = [photograph(2000, 1504, 85), photograph(2000, 1504, 88, 125, 7, "422")]
    chunks = sum(len(d) for _, d in streams) // 128
    streams *= 3 * 96 * cus // chunks + 1
    s = check(M, ctx, streams)
    assert s["chunks"] > 3 * 96 * cus and s["intervals"] > 188


def test_long_and_short_split_intervals(M, ctx):
    s = check(M, ctx, [photograph(200, 120, 85), photograph(800, 500, 85), photograph(300, 200, 85, 40, 3, "444"),
                       photograph(900, 500, 80)])
    assert s["intervals"] > 4 and s["chunks"] > 2 * 512


def test_captured_and_on_two_streams(M, ctx):
    """Launches of a graph, with eager work between them, and two batches at
    once: split intervals, whole ones and broken chains."""
    sets = [[photograph(640, 480, 98), photograph(400, 300, 85, 2)], [photograph(640, 480, 95, 40, 31), periodic(10)]]
    jobs = [[job(M, data) for _, data in streams] for streams in sets]
    batches = [M.EntropyBatch(ctx, j) for j in jobs]

    def check_and_clear(which):
        torch.cuda.synchronize()
        for (coef, _), j in zip(sets[which], jobs[which]):
            assert np.array_equal(j[4].cpu().numpy().reshape(-1, 64), coef), which
            j[4].fill_(0x5A5A)

    batches[0].launch()
    check_and_clear(0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        batches[0].launch()
    for rep in range(4):
        torch.zeros(1 << 20, device="cuda").sum()
        graph.replay()
        check_and_clear(0)
        assert batches[0].status() == -1 and batches[0].splits()["mended"] > 0
    streams = [torch.cuda.Stream() for _ in batches]
    for rep in range(3):
        torch.cuda.synchronize()
        for b, s in zip(batches, streams):
            b.launch(s)
        for k, b in enumerate(batches):
            check_and_clear(k)
            assert b.status() == -1
    for b in batches:
        b.close()


def test_more_bytes_than_a_pass_holds(M, ctx):
    """1.3 GB of intervals of an MCU row, decoded in two passes, with a long
    interval at the end of the list, which many lanes decode."""
    frame, coef, qt = encode.encode_rgb(images.texture_rgb(2000, 1504, 7, sigma=12), "420", 85)
    exp = torch.from_numpy(coef.reshape(-1)).cuda()
    jobs = []
    for interval in (125, 0):
        data = fast_bitstream.write_jpeg(frame, coef, qt, restart_interval=interval)
        scan, off, d_jpg, _, _ = job(M, data, exp)
        copies = 1_300_000_000 // len(data) if interval else 1
        # every 40th has coefficients of its own, the others share theirs
        own = [torch.zeros_like(exp) for _ in range(copies // 40 + 1)]
        jobs += [(scan, off, d_jpg, len(data), own[i // 40] if i % 40 == 0 else own[-1]) for i in range(copies)]
    assert sum(j[3] for j in jobs) > 1_290_000_000
    print(f"{len(jobs)} jobs of {jobs[0][3]} bytes", flush=True)
    b = M.EntropyBatch(ctx, jobs)
    assert b.splits()["intervals"] >= 1
    outs = {j[4].data_ptr(): j[4] for j in jobs}.values()
    for rep in range(2):
        for c in outs:
            c.fill_(0x5A5A)
        b.launch()
        assert b.status() == -1
        for c in outs:
            assert torch.equal(c, exp), rep
    b.close()
