"""GPU entropy decoding of batches at the limits of its memory: more stream
bytes than one pass over them holds.  Coefficients are whole numbers: no
tolerance."""
import numpy as np
import pytest

from synth import encode, fast_bitstream, images

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


def test_more_bytes_than_a_pass_holds(M, ctx):
    """1.3 GB of intervals of an MCU row, decoded in two passes, with a long
    interval at the end of the list, which many lanes decode."""
    frame, coef, qt = encode.encode_rgb(images.texture_rgb(2000, 1504, 7, sigma=12), "420", 85)
    exp = torch.from_numpy(coef.reshape(-1)).cuda()
    jobs = []
    for interval in (125, 0):
        data = fast_bitstream.write_jpeg(frame, coef, qt, restart_interval=interval)
        scan, _ = M.mjd_parse(data)
        off = M.mjd_restart_index(data, scan)
        d_jpg = torch.zeros(-(-len(data) // 16) * 16, dtype=torch.uint8, device="cuda")
        d_jpg[:len(data)] = torch.from_numpy(np.frombuffer(data, dtype=np.uint8).copy()).cuda()
        copies = 1_300_000_000 // len(data) if interval else 1
        # every 40th has coefficients of its own, the others share theirs
        own = [torch.zeros_like(exp) for _ in range(copies // 40 + 1)]
        jobs += [(scan, off, d_jpg, len(data), own[i // 40] if i % 40 == 0 else own[-1]) for i in range(copies)]
    assert sum(j[3] for j in jobs) > 1_290_000_000
    print(f"{len(jobs)} jobs of {jobs[0][3]} bytes", flush=True)
    b = M.EntropyBatch(ctx, jobs)
    outs = {j[4].data_ptr(): j[4] for j in jobs}.values()
    for rep in range(2):
        for c in outs:
            c.fill_(0x5A5A)
        b.launch()
        assert b.status() == -1
        for c in outs:
            assert torch.equal(c, exp), rep
    b.close()
