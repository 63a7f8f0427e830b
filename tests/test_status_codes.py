"""What Simulator.check_status makes of a call's status: a HIP error that the
run left is the library's own exception, and every status word is judged as
mc_check_status judges it."""
import pytest


def _mc():
    import paper_2105_13324_amd as mc
    return mc


def _simulator(ends):
    mc = _mc()
    s = mc.Simulator.__new__(mc.Simulator)
    s._ends = ends
    return s


def test_hip_error_is_the_librarys_exception():
    mc = _mc()

    class Failed:
        def cpu(self):
            raise RuntimeError("HIP error: an illegal memory access was encountered")

    with pytest.raises(mc.McError, match="HIP error.*illegal memory access"):
        _simulator(Failed()).check_status()


@pytest.mark.gpu
def test_status_words_as_the_library_judges_them():
    import torch
    mc = _mc()
    ends = torch.zeros(5, dtype=torch.int64, device="cuda")
    s = _simulator(ends)
    bits = [getattr(mc, n) for n in dir(mc) if n.startswith("STATUS_")]
    assert len(bits) >= 8
    for word in [0] + bits + [a | b for a in bits for b in bits]:
        ends[0] = word
        rc = mc._lib.mc_check_status(ends.data_ptr(), mc._stream_ptr())
        if rc in (mc.MC_EINVAL, mc.MC_EOVERFLOW):
            with pytest.raises(mc.McError, match=mc._lib.mc_error_string(rc).decode()):
                s.check_status()
        else:
            assert int(s.check_status()[0]) == word
