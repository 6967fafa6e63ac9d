"""The binding's marshalling, on the CPU: a frame takes its counts and times from
any integer-like value, and its pose from any array of twelve numbers."""
import ctypes

import numpy as np
import pytest

from paper_2204_12876_amd import _emx

POSE = np.arange(12, dtype=np.float64).reshape(3, 4) / 7


@pytest.mark.parametrize("n", [5, np.int64(5), np.int32(5), np.uint8(5), 5.0, True + 4])
def test_frame_count_types(n):
    f = _emx.make_frame(16, 32, 48, n, POSE, n)
    assert (f.x, f.y, f.z, f.n, f.t_ms) == (16, 32, 48, 5, 5)


@pytest.mark.parametrize("pose", [POSE, POSE.astype(np.float32), POSE.tolist(), POSE.reshape(12),
                                  np.asfortranarray(POSE), POSE[:, ::-1][:, ::-1]])
def test_frame_pose_forms(pose):
    f = _emx.make_frame(0, 0, 0, 1, pose, 0)
    want = np.asarray(pose, np.float64).reshape(12)
    assert list(f.pose) == want.tolist()
    assert (f.x, f.n, f.t_ms) == (None, 1, 0)
    assert ctypes.sizeof(f) == ctypes.sizeof(_emx.Frame)


@pytest.mark.parametrize("pose", [None, POSE[:2], np.zeros((4, 4))])
def test_frame_pose_of_another_size_is_refused(pose):
    with pytest.raises(ValueError):
        _emx.make_frame(0, 0, 0, 1, pose, 0)


def test_stream_without_the_private_function(monkeypatch):
    """Another torch may not have the raw lookup: the public one serves."""
    import torch

    import paper_2204_12876_amd as emx

    class Stream:
        cuda_stream = 1234

    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(emx, "_raw_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream)
    assert emx._stream(torch.device("cuda:0")) == 1234
