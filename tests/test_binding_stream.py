"""The binding asks torch for its stream again after a fork: a child of a process that has used the GPU gets torch's error, not a
handle of its parent's."""
import os
import types

import pytest
import torch

from paper_2602_15563_amd import kmq


def test_a_forked_child_gets_no_handle_of_its_parent(monkeypatch):
    monkeypatch.setattr(kmq, "_torch_c", types.SimpleNamespace(_cuda_getDevice=lambda: 0, _cuda_getCurrentRawStream=lambda device: 7))
    assert kmq._stream() == 7                              # as after a first call on the GPU

    def refused():
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
    monkeypatch.setattr(torch.cuda, "current_stream", refused)
    pid = os.fork()
    if pid == 0:
        status = 1
        try:
            kmq._stream()
        except RuntimeError:
            status = 0
        finally:
            os._exit(status)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
    assert kmq._stream() == 7


@pytest.mark.skipif(torch.cuda.is_available(), reason="needs a machine without a GPU")
def test_no_gpu_is_torchs_error():
    with pytest.raises(RuntimeError):
        kmq._stream()
