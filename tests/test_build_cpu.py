"""What a build leaves behind when one of its steps fails.  No compiler runs: the commands are written down."""
import subprocess

import pytest

from paper_2407_12077_amd import build as b


@pytest.fixture
def steps(monkeypatch, tmp_path):
    """[(program, the rest)] in order; `fail` names what fails: a compiled source's name, "link" or "g++"."""
    log, fail, running = [], set(), []

    class Compiler:
        def __init__(self, cmd):
            self.source, self.returncode = cmd[cmd.index("-c") + 1].rsplit("/", 1)[1], None
            log.append(("compile", self.source))
            running.append(self)

        def wait(self):
            if self.returncode is None:
                running.remove(self)
            self.returncode = int(self.source in fail)
            return self.returncode

    def check_call(cmd):
        step = "g++" if cmd[0] == "g++" else "link"
        if step in fail:
            raise FileNotFoundError(step) if step == "g++" else subprocess.CalledProcessError(1, cmd)
        log.append((step, cmd[cmd.index("-o") + 1]))

    monkeypatch.setattr(b.subprocess, "Popen", Compiler)
    monkeypatch.setattr(b.subprocess, "check_call", check_call)
    monkeypatch.setattr(b, "PKG", str(tmp_path))
    return log, fail, running


def test_library_does_not_wait_for_the_extension(steps):
    log, fail, running = steps
    fail.add("g++")                                           # no g++, or no Python headers
    with pytest.raises(FileNotFoundError):
        b.build()
    assert log[-1] == ("link", b.LIB) and [s for k, s in log if k == "compile"] == b.SOURCES and not running


def test_no_compiler_is_left_running(steps):
    log, fail, running = steps
    fail.add(b.SOURCES[0])
    with pytest.raises(subprocess.CalledProcessError):
        b.build()
    assert not running and not [s for k, s in log if k != "compile"]


def test_library_then_extension(steps):
    log = steps[0]
    assert b.build() == b.LIB and log[len(b.SOURCES):] == [("link", b.LIB), ("g++", b.CALL)]
