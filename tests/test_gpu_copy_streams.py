"""The streams a step's large copy runs on belong to nobody else: neither torch's pool, which deals out 32 of a device over and over, nor
another session's capture."""
import gc

import pytest
import torch

from paper_2508_08438_amd import inputs, pipeline

pytestmark = pytest.mark.gpu


def _session(seed):
    s = pipeline.Session(inputs.small_random(seed=seed, n_seq=8, max_blocks=24, n_req=3, vocab=50, attn=inputs.AttnShape(8, 2, 128, "bf16")))
    s.prepare()
    return s


def test_no_stream_of_the_pool(monkeypatch):
    monkeypatch.setattr(pipeline, "GATHER_BESIDE_BYTES", 0)
    a, b = _session(1), _session(2)
    own = [a.side.cuda_stream, a.side_capture.cuda_stream, b.side_capture.cuda_stream]
    assert a.side is b.side and len(set(own)) == 3
    assert not set(own) & {torch.cuda.Stream().cuda_stream for _ in range(100)}


def test_session_gives_its_capture_stream_back(monkeypatch):
    monkeypatch.setattr(pipeline, "GATHER_BESIDE_BYTES", 0)
    from paper_2508_08438_amd import binding as skv
    gone = []
    destroy = skv._stream_destroy
    monkeypatch.setattr(skv, "_stream_destroy", lambda h: (gone.append(h), destroy(h)))
    a = _session(4)
    h = a.side_capture.cuda_stream
    a.capture_step()
    a.replay()
    torch.cuda.synchronize()
    del a
    gc.collect()
    assert gone == [h]
