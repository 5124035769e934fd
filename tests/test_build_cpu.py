"""Builds that run side by side do not disturb each other: every one ends with a whole library in place."""
import os
import stat
import threading

from paper_2607_19438_amd import build

# stands in for hipcc: takes a while, then writes its output from its inputs (a link reads the objects)
COMPILER = """#!/bin/sh
out=; in=
while [ $# -gt 0 ]; do
  case "$1" in
    -o) out=$2; shift;;
    -target-feature|-Xclang) ;;
    -*) ;;
    *) in="$in $1";;
  esac
  shift
done
sleep "0.$(( $$ % 4 ))"
cat $in > "$out" || exit 1
"""


def test_two_builds_at_once(tmp_path, monkeypatch):
    cc = tmp_path / "cc"
    cc.write_text(COMPILER)
    cc.chmod(cc.stat().st_mode | stat.S_IXUSR)
    src = [tmp_path / "a.hip", tmp_path / "b.hip"]
    for s in src:
        s.write_text(s.name + "\n")
    lib = tmp_path / "lib.so"
    monkeypatch.setattr(build, "HIPCC", str(cc))
    monkeypatch.setattr(build, "FLAGS", [])
    monkeypatch.setattr(build, "SOURCES", [str(s) for s in src])
    monkeypatch.setattr(build, "LIB", str(lib))
    errors = []

    def one():
        try:
            for _ in range(3):
                build.build()
                assert lib.read_text() == "a.hip\nb.hip\n"
        except Exception as e:
            errors.append(e)

    threads = [threading.Thread(target=one) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[0]
    assert sorted(os.listdir(tmp_path)) == ["a.hip", "b.hip", "cc", "lib.so"]       # nothing left behind
