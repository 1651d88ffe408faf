"""GPU tests of what md_energy waits for: its read-back is ordered after the
stream it is given and, through the null stream, after every other blocking
stream; a stream under capture is refused."""
import ctypes

import numpy as np
import pytest

from paper_1107_2619_amd import inputs
from tests.gpu_helpers import announce

pytestmark = pytest.mark.gpu
STREAM_NON_BLOCKING = 1
CAPTURE_RELAXED = 2


@pytest.fixture(scope="module")
def md():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_2619_amd import md as _md

    return _md


@pytest.fixture(scope="module")
def hip(md):
    """The HIP runtime this process has loaded."""
    import torch

    torch.zeros(1, device="cuda:0")
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64.so" in line)
    lib = ctypes.CDLL(path)
    for name in ("hipStreamDestroy", "hipStreamSynchronize"):
        getattr(lib, name).argtypes = [ctypes.c_void_p]
    lib.hipStreamCreateWithFlags.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint]
    lib.hipStreamBeginCapture.argtypes = [ctypes.c_void_p, ctypes.c_int]
    lib.hipStreamEndCapture.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_void_p)]
    lib.hipGraphDestroy.argtypes = [ctypes.c_void_p]
    return lib


def _stream(hip, flags):
    s = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(s), flags) == 0
    return s


@pytest.mark.parametrize("steps_on,read_on", [("blocking", "blocking"), ("blocking", "null"), ("null", "blocking"),
                                              ("null", "own"), ("own", "own")])
def test_energy_waits_for_the_steps(md, hip, steps_on, read_on):
    """Steps of several milliseconds on one stream, the energies read on
    another: those of the last step, bitwise as read on the stream of the steps."""
    import torch

    announce(f"energy read on {read_on}, steps on {steps_on}")
    s = inputs.bcc_fe(60, temperature=600.0, seed=61, skin=0.4)
    want = md.Simulation(s)
    want.step(30)
    ref = want.energy()

    streams = {"null": None, "own": _stream(hip, STREAM_NON_BLOCKING)}
    made = [streams["own"]]
    sim = md.Simulation(s)
    sim.eam_forces()
    first = sim.energy()
    sim.state_changed()
    torch.cuda.synchronize()

    def on(kind):
        if kind == "null":
            return torch.cuda.stream(torch.cuda.default_stream())
        h = streams.get(kind) or _stream(hip, 0)
        if kind == "blocking":
            made.append(h)
        return torch.cuda.stream(torch.cuda.ExternalStream(h.value))

    with on(steps_on):
        sim.step(30)
    with on(read_on):
        got = sim.energy()
    torch.cuda.synchronize()
    for h in made:
        assert hip.hipStreamDestroy(h) == 0
    assert got.pe[0] == ref.pe[0] and got.ke[0] == ref.ke[0] and got.pe[0] != first.pe[0]
    assert np.array_equal(got.virial, ref.virial)


def test_energy_refuses_a_capturing_stream(md, hip):
    """During a capture there is nothing to read: MD_ERR_DEVICE, and the context
    works on once the capture has ended."""
    announce("energy under capture")
    import torch

    s = inputs.bcc_fe(5, seed=62, displace=0.05)
    sim = md.Simulation(s)
    sim.eam_forces()
    ref = sim.energy()
    torch.cuda.synchronize()
    h, graph = _stream(hip, STREAM_NON_BLOCKING), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(h, CAPTURE_RELAXED) == 0
    try:
        with torch.cuda.stream(torch.cuda.ExternalStream(h.value)):
            with pytest.raises(md.MDError) as e:
                sim.energy()
        assert e.value.code == md.MD_ERR_DEVICE
    finally:
        hip.hipStreamEndCapture(h, ctypes.byref(graph))  # (ends with an error where the capture was cut short)
        if graph.value:
            hip.hipGraphDestroy(graph)
        hip.hipGetLastError()
        assert hip.hipStreamDestroy(h) == 0
    assert np.array_equal(sim.energy().pe, ref.pe)
