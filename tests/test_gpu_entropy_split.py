"""GPU parity of intervals that the entropy kernels decode in chunks: one
long interval per stream (no restart markers), over samplings, contents and
lengths at which the chunking can go wrong, every coefficient equal to the
encoder's; corrupted streams are rejected exactly when the host decoder
rejects them.  Coefficients are whole numbers: no tolerance."""
import random

import numpy as np
import pytest

from synth import bitstream, encode, images

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SENTINEL = 0x5A5A
LUMA = {"444": (1, 1), "422": (2, 1), "420": (2, 2), "440": (1, 2), "411": (4, 1)}


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


def job(M, data):
    scan, _ = M.mjd_parse(data)
    off = M.mjd_restart_index(data, scan)
    d_jpg = torch.zeros(-(-len(data) // 16) * 16, dtype=torch.uint8, device="cuda")
    d_jpg[:len(data)] = torch.from_numpy(np.frombuffer(data, dtype=np.uint8).copy()).cuda()
    f = M.scan_frame(scan)
    g, _ = M.mjd_variant_geometry(M.make_variant(f, f.get("ncomp", 3)))
    d_coef = torch.full((g["n_blocks"] * 64,), SENTINEL, dtype=torch.int16, device="cuda")
    return scan, off, d_jpg, len(data), d_coef


def check(M, ctx, streams):
    """streams: (coefficients, file); all in one batch, launched twice."""
    jobs = [job(M, data) for _, data in streams]
    b = M.EntropyBatch(ctx, jobs)
    for rep in range(2):
        for j in jobs:
            j[4].fill_(SENTINEL)
        b.launch()
        assert b.status() == -1
        for i, ((coef, data), j) in enumerate(zip(streams, jobs)):
            got = j[4].cpu().numpy().reshape(-1, 64)
            assert np.array_equal(got, coef), (rep, i, len(data))
    b.close()


def frame_of(w, h, samp):
    hy, vy = LUMA[samp]
    return {"width": w, "height": h, "h": (hy, 1, 1), "v": (vy, 1, 1), "qsel": (0, 1, 1)}


def ones():
    return np.ones((4, 64), dtype=np.uint16)


@pytest.mark.parametrize("samp,quality", [("420", 50), ("420", 92), ("422", 85), ("444", 75)])
def test_photographs_without_markers(M, ctx, samp, quality):
    rgb = images.texture_rgb(333, 250, 31, sigma=12)
    frame, coef, qt = encode.encode_rgb(rgb, samp, quality)
    check(M, ctx, [(coef, bitstream.write_jpeg(frame, coef, qt))])


@pytest.mark.parametrize("samp", ["440", "411", "420", "gray"])
def test_dense_blocks_of_every_sampling(M, ctx, samp):
    """Blocks longer than a part of a chunk, codes past both look-ups."""
    if samp == "gray":
        frame = {"width": 200, "height": 160, "h": (1, 1, 1), "v": (1, 1, 1), "qsel": (0, 0, 0), "ncomp": 1}
        n = 25 * 20
    else:
        frame = frame_of(160, 128, samp)
        n = (160 // (8 * LUMA[samp][0])) * (128 // (8 * LUMA[samp][1])) * (LUMA[samp][0] * LUMA[samp][1] + 2)
    rng = np.random.default_rng(5)
    size = np.minimum(rng.geometric(0.3, size=(n, 64)), 10)
    mag = (1 << (size - 1)) + (rng.random((n, 64)) * (1 << (size - 1))).astype(np.int64)
    coef = np.where(rng.random((n, 64)) < 0.5, -mag, mag).astype(np.int16)
    coef[:, 0] = rng.integers(-1023, 1024, size=n)
    coef[rng.random((n, 64)) < 0.2] = 0
    sparse = coef.copy()
    sparse[rng.random((n, 64)) < 0.9] = 0
    qt = ones()
    check(M, ctx, [(c, bitstream.write_jpeg(frame, c, qt)) for c in (coef, sparse)])


def test_all_ones_bits_cross_tiles_and_chunks(M, ctx):
    """Magnitudes of ones: stuffed bytes at every place of the 16-byte lanes
    and the 4096-byte tiles that drop them."""
    frame = frame_of(256, 192, "444")
    n = 32 * 24 * 3
    coef = np.zeros((n, 64), dtype=np.int16)
    coef[:, 1:24] = 1023
    coef[::3, 30] = 1
    coef[::7, 40] = -5
    data = bitstream.write_jpeg(frame, coef, ones())
    assert data.count(b"\xFF\x00") > len(data) // 8 and len(data) > 3 * 4096
    check(M, ctx, [(coef, data)])


def test_lengths_around_chunks(M, ctx):
    """Streams of every length class from one byte to three chunks."""
    streams, lengths = [], set()
    rng = np.random.default_rng(9)
    for n in range(1, 60):
        frame = {"width": 8 * n, "height": 8, "h": (1, 1, 1), "v": (1, 1, 1), "qsel": (0, 0, 0), "ncomp": 1}
        coef = np.zeros((n, 64), dtype=np.int16)
        coef[:, 0] = rng.integers(-60, 61, size=n)
        coef[:, 1:8] = rng.integers(-9, 10, size=(n, 7))
        data = bitstream.write_jpeg(frame, coef, ones())
        scan, _ = M.mjd_parse(data)
        lengths.add(int(scan.data_end - scan.data_offset))
        streams.append((coef, data))
    assert min(lengths) < 16 and max(lengths) > 384
    check(M, ctx, streams)


def tiled(w, h, seed, amplitude, side):
    """A texture that repeats: lanes that start in the wrong place of the MCU
    may stay there, and chains of chunks break."""
    rng = np.random.default_rng(seed)
    t = np.rint(rng.random((side, side, 3)) * amplitude + 100).astype(np.uint8)
    return np.tile(t, (h // side, w // side, 1))


@pytest.mark.parametrize("amplitude,side,samp,quality", [(10, 16, "420", 75), (80, 32, "420", 90), (6, 16, "420", 60),
                                                         (60, 8, "444", 85), (20, 16, "422", 80), (0, 16, "420", 85)])
def test_repeating_textures(M, ctx, amplitude, side, samp, quality):
    streams = []
    for seed in range(3):
        frame, coef, qt = encode.encode_rgb(tiled(512, 384, seed, amplitude, side), samp, quality)
        streams.append((coef, bitstream.write_jpeg(frame, coef, qt)))
    check(M, ctx, streams)


def test_split_and_whole_intervals_in_one_batch(M, ctx):
    """Long and short intervals of several jobs together."""
    streams = []
    for i, ri in enumerate((0, 1, 7, 64)):
        rgb = images.texture_rgb(256, 160, 50 + i, sigma=12)
        frame, coef, qt = encode.encode_rgb(rgb, ("420", "444", "422", "420")[i], 85)
        streams.append((coef, bitstream.write_jpeg(frame, coef, qt, restart_interval=ri)))
    check(M, ctx, streams)


def test_corruption_is_found_like_on_the_host(M, ctx):
    rnd = random.Random(3)
    rgb = images.texture_rgb(256, 160, 77, sigma=12)
    seen = {True: 0, False: 0}
    for samp in ("420", "444"):
        frame, coef, qt = encode.encode_rgb(rgb, samp, 85)
        data = bitstream.write_jpeg(frame, coef, qt)
        scan, _ = M.mjd_parse(data)
        off = M.mjd_restart_index(data, scan)
        g = M.mjd_geometry_of(frame)
        for k in range(24):
            b = bytearray(data)
            for _ in range(rnd.choice((1, 1, 2, 5))):
                p = rnd.randrange(scan.data_offset, scan.data_end)
                if b[p] != 0xFF and b[p - 1] != 0xFF:
                    b[p] = rnd.randrange(255)
            if k % 6 == 0:  # bytes are missing at the end
                b = b[:scan.data_end - 40 - k] + b[scan.data_end:]
            b = bytes(b)
            try:
                s2, _ = M.mjd_parse(b)
                o2 = M.mjd_restart_index(b, s2)
                host = np.zeros((g["n_blocks"], 64), dtype=np.int16)
                M.mjd_entropy_decode(b, s2, o2, host, 0, g["mcus_y"], 1)
                host_ok = True
            except M.MjdError as e:
                assert e.code == -5
                host_ok = False
            j = job(M, b)
            e = M.EntropyBatch(ctx, [j])
            e.launch()
            if host_ok:
                assert e.status() == -1
                assert np.array_equal(j[4].cpu().numpy().reshape(-1, 64), host)
            else:
                with pytest.raises(M.MjdError) as ei:
                    e.status()
                assert ei.value.code == -5 and ei.value.bad_job == 0
            e.close()
            seen[host_ok] += 1
    assert seen[True] > 3 and seen[False] > 8
