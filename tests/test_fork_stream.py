"""A child forked after the parent used its device (CPU only): the binding asks
torch for the current stream anew, so that torch's own refusal of a forked
child stands."""
import os

from paper_2608_12123_amd import rc_cohort as rc


class _FakeTorchC:
    """What the binding keeps of torch once a device has been initialised."""
    @staticmethod
    def _cuda_getDevice():
        return 0

    @staticmethod
    def _cuda_getCurrentRawStream(device):
        return 0x5EED


def test_no_stream_of_the_parent_in_a_forked_child(monkeypatch):
    monkeypatch.setattr(rc, "_torch_c", _FakeTorchC)
    assert rc._current_stream() == 0x5EED
    pid = os.fork()
    if pid == 0:
        code = 1
        try:
            code = 0 if rc._torch_c is None else 3
        finally:
            os._exit(code)
    _, status = os.waitpid(pid, 0)
    assert os.WIFEXITED(status) and os.WEXITSTATUS(status) == 0
    assert rc._current_stream() == 0x5EED  # the parent's is as it was
