"""What the build takes for up to date: an object, and the library, are older than a change of the flags that build.py holds."""
import os

from paper_2506_02572_amd import build


def test_a_change_of_flags_makes_objects_and_library_stale(tmp_path, monkeypatch):
    csrc = tmp_path / "csrc"
    include = tmp_path / "include"
    csrc.mkdir(), include.mkdir()
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "CSRC", str(csrc))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libhata.so"))
    monkeypatch.setattr(build, "OBJ", str(tmp_path / "_build"))
    monkeypatch.setattr(build, "HEADERS", ["a.h", os.path.join("..", "include", "b.h")])
    monkeypatch.setattr(build, "SOURCES", ["one.hip", "two.hip"])
    files = [csrc / "one.hip", csrc / "two.hip", csrc / "a.h", include / "b.h", tmp_path / "build.py", tmp_path / "libhata.so"]
    (tmp_path / "_build").mkdir()
    objects = [tmp_path / "_build" / "one.o", tmp_path / "_build" / "two.o"]
    for f in files + objects:
        f.write_text("")

    def age(path, t):
        os.utime(path, (t, t))

    def rebuilt():
        """The sources that a build of what changed compiles."""
        done = []

        def fake(cmd, **kw):
            done.extend(os.path.basename(c) for c in cmd if c.endswith(".hip"))
            return type("Result", (), {"returncode": 0, "stdout": ""})()
        monkeypatch.setattr(build.subprocess, "run", fake)
        state = build.stale()
        build.build(force=False)
        return state, sorted(done)

    for f in files[:5]:
        age(f, 1000)
    for f in objects + [files[5]]:
        age(f, 2000)
    assert rebuilt() == (False, [])
    for changed, compiled in ((tmp_path / "build.py", ["one.hip", "two.hip"]), (csrc / "two.hip", ["two.hip"]),
                              (include / "b.h", ["one.hip", "two.hip"])):
        age(changed, 3000)
        assert rebuilt() == (True, compiled), changed
        age(changed, 1000)
    os.remove(tmp_path / "libhata.so")
    assert rebuilt()[0]
