"""A build that fails leaves the package folder as it was."""
import os

import pytest

from paper_2601_10819_amd import build as b


@pytest.mark.parametrize("fails", ["msda_vis.hip", "msda_torch.cpp", "link"])
def test_failed_build_leaves_nothing(monkeypatch, fails):
    def run(cmd):
        out = cmd[cmd.index("-o") + 1]
        source = [os.path.basename(c) for c in cmd if c in b.SOURCES + [b.TORCH_SOURCE]]
        if fails in source or (fails == "link" and not source):
            return 1, "refused"
        with open(out, "w") as f:
            f.write("built")
        return 0, ""

    monkeypatch.setattr(b, "_run", run)
    state = lambda: {f: os.stat(os.path.join(b.PKG, f)).st_mtime_ns for f in os.listdir(b.PKG)
                     if f != "__pycache__"}
    before = state()
    with pytest.raises(RuntimeError, match="refused"):
        b.build()
    assert state() == before
