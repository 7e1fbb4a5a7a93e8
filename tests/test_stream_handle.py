"""The binding's stream handle from several threads: a thread that asks while another one asks
for the first time gets the handle too, wherever the other one has got to."""
import sys
import threading
import types

from paper_2202_07388_amd import qdw


def test_first_call_in_two_threads(monkeypatch):
    cuda = types.SimpleNamespace(current_stream=lambda: None)
    calls = types.SimpleNamespace(_cuda_getCurrentRawStream=lambda device: 100 + device, _cuda_getDevice=lambda: 3)
    monkeypatch.setattr(qdw, "_torch", lambda: types.SimpleNamespace(cuda=cuda, _C=calls))
    cached = [n for n in vars(qdw) if n in ("_stream_calls", "_raw_stream", "_current_device")]
    assert cached
    for n in cached:
        monkeypatch.setattr(qdw, n, None)
    seen = []

    def ask():
        try:
            seen.append(qdw._stream())
        except TypeError as e:
            seen.append(e)

    # another thread asks before every bytecode of the first call
    def step(frame, event, arg):
        if frame.f_code is qdw._stream.__code__:
            frame.f_trace_opcodes = True
            if event == "opcode":
                keep = {n: getattr(qdw, n) for n in cached}
                t = threading.Thread(target=ask)
                t.start()
                t.join()
                for n, v in keep.items():  # leave the first call where it was
                    setattr(qdw, n, v)
        return step

    before = sys.gettrace()
    sys.settrace(step)
    try:
        assert qdw._stream() == 103
    finally:
        sys.settrace(before)
    assert len(seen) > 10 and all(h == 103 for h in seen), seen
