"""The look-up tables of the GPU entropy kernels (CPU only): compiled with g++
and compared, for every 16-bit front of a stream, with the canonical code of
T.81 Annex C walked code by code."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from synth import bitstream, encode, images

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBDIR = os.path.join(ROOT, "paper_1311_5304_amd", "_lib")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    if not os.path.exists(os.path.join(LIBDIR, "libmjd.so")):
        pytest.skip("libmjd.so is not built")
    exe = str(tmp_path_factory.mktemp("tables") / "entropy_tables_host")
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1311_5304_amd", "csrc"),
                    os.path.join(ROOT, "tests", "entropy_tables_host.cpp"), "-o", exe, "-L", LIBDIR, "-lmjd",
                    "-Wl,-rpath," + LIBDIR], check=True)
    return exe


def photograph():
    return encode.encode_rgb(images.texture_rgb(160, 120, 3, sigma=12), "420", 85)


def flat():
    """Two or three symbols: most of the code space belongs to no code."""
    return encode.encode_rgb(np.full((64, 64, 3), 90, np.uint8), "444", 85)


def dense():
    """Over 150 symbols with halving frequencies: codes of 11 to 16 bits under
    more prefixes than the second look-up has room for."""
    rng = np.random.default_rng(2)
    frame = encode.make_frame(160, 160, "444")
    n = 20 * 20 * 3
    size = np.minimum(rng.geometric(0.5, size=(n, 64)), 10)
    mag = (1 << (size - 1)) + (rng.random((n, 64)) * (1 << (size - 1))).astype(np.int64)
    coef = np.where(rng.random((n, 64)) < 0.5, -mag, mag).astype(np.int16)
    coef[:, 0] = rng.integers(-1023, 1024, size=n)
    coef[rng.random((n, 64)) < rng.random((n, 1))] = 0
    return frame, coef, np.ones((4, 64), dtype=np.uint16)


@pytest.mark.parametrize("content", [photograph, flat, dense])
def test_tables_follow_the_canonical_code(harness, tmp_path, content):
    frame, coef, qt = content()
    path = tmp_path / "s.jpg"
    path.write_bytes(bitstream.write_jpeg(frame, coef, qt))
    r = subprocess.run([harness, str(path)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr)
    assert int(r.stdout) >= 4 * 65536
