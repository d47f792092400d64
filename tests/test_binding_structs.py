"""The binding's packed structs hold what setting each field holds, for every
kind of number a caller may pass, and refuse what that refuses.  No GPU."""
import ctypes

import numpy as np
import pytest

from paper_1311_5304_amd import _binding as B


def by_field(job):
    frame, coef, qt, rgb, pitch = job
    j = B.mjd_job()
    if isinstance(frame, B.mjd_frame):
        j.frame = frame
    else:
        j.frame.width, j.frame.height = int(frame["width"]), int(frame["height"])
        for c in range(3):
            j.frame.h[c], j.frame.v[c] = int(frame["h"][c]), int(frame["v"][c])
            j.frame.qsel[c] = int(frame.get("qsel", (0, 1, 1))[c])
    j.d_coef, j.d_qt, j.d_rgb, j.pitch = coef, qt, rgb, int(pitch)
    return bytes(j)


FRAMES = [
    {"width": 257, "height": 190, "h": (2, 1, 1), "v": (2, 1, 1), "qsel": (3, 2, 1)},
    {"width": 65535, "height": 1, "h": [1, 1, 1], "v": [1, 1, 1]},
    {"width": np.int64(33), "height": np.uint16(47), "h": np.array([2, 1, 1]), "v": (1, 1, 1), "qsel": (0, 1, 1)},
    {"width": 33.0, "height": "47", "h": (2.0, 1, 1), "v": (1, True, 1), "qsel": (0, 1, 1)},  # what int() takes
    {"width": -1, "height": 1 << 33, "h": (257, 1, 1), "v": (-1, 1, 1), "qsel": (0, 1, 300)},  # what C truncates
]


@pytest.mark.parametrize("frame", FRAMES + [B.mjd_frame(width=9, height=8)], ids=range(len(FRAMES) + 1))
@pytest.mark.parametrize("pitch", [771, np.int32(771), 771.0, (1 << 40) + 5])
def test_jobs_equal_their_fields(frame, pitch):
    job = (frame, 0x7F0012345670, 0x10, 0xFFFFFFFFFFFFFFF1, pitch)
    arr = B._job_array([job, job])
    n = ctypes.sizeof(B.mjd_job)
    assert bytes(arr) == 2 * by_field(job) and n * 2 == len(bytes(arr))
    if not isinstance(frame, B.mjd_frame):
        assert bytes(B.make_frame(frame)) == by_field(job)[:ctypes.sizeof(B.mjd_frame)]


@pytest.mark.parametrize("frame,error", [({"width": 8, "height": 8, "h": (1, 1, 1)}, KeyError),
                                         ({"width": 8, "height": 8, "h": (1, 1), "v": (1, 1, 1)}, IndexError),
                                         ({"width": None, "height": 8, "h": (1, 1, 1), "v": (1, 1, 1)}, TypeError),
                                         ({"width": "x", "height": 8, "h": (1, 1, 1), "v": (1, 1, 1)}, ValueError)])
def test_bad_frames_raise(frame, error):
    with pytest.raises(error):
        B.make_frame(frame)
    with pytest.raises(error):
        B._job_array([(frame, 0, 0, 0, 24)])
