"""What the build does beside compiling: it notices a library built for another torch, and leaves no compiler running behind a failure.  No GPU."""
import subprocess

import pytest
import torch

from paper_2509_09090_amd import build


def test_another_torch_makes_the_calls_stale(monkeypatch):
    monkeypatch.setattr(build, "_older", lambda built, sources: False)
    assert not build.is_stale()
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".1")
    assert build.is_stale()
    monkeypatch.undo()
    monkeypatch.setattr(build, "_older", lambda built, sources: False)
    monkeypatch.setattr(torch, "__version__", torch.__version__[:-1])
    assert build.is_stale()


@pytest.mark.parametrize("calls,hipcc", [("sleep 0.3", "/bin/false"), ("false", "/bin/true")])
def test_every_compiler_is_waited_for(monkeypatch, calls, hipcc):
    started = []
    popen = subprocess.Popen

    def recorded(*args, **kwargs):
        started.append(popen(*args, **kwargs))
        return started[-1]
    monkeypatch.setattr(build.subprocess, "Popen", recorded)
    monkeypatch.setattr(build, "_calls_command", calls.split)
    monkeypatch.setattr(build, "HIPCC", hipcc)
    with pytest.raises(RuntimeError):
        build.build()
    assert len(started) == 1 + len(build.SOURCES) and all(p.returncode is not None for p in started)
