"""What a build leaves beside the library: nothing, also where the compiler fails or
leaves intermediate files of its own next to its output."""
import os
import stat

import pytest

from paper_2511_19204_amd import build, hazards

# -c src -o obj: an object, an intermediate beside it and a resource remark; else: links
HIPCC = """#!/bin/sh
while [ $# -gt 0 ]; do
  if [ "$1" = -c ]; then src=$2; fi
  if [ "$1" = -o ]; then out=$2; fi
  shift
done
: > "$out"
if [ -n "$src" ]; then
  : > "$out-6b83dd3e.o.tmp"
  echo "x.hip:1:1: remark: Function Name: kernel"
  echo "x.hip:1:1: remark:     ScratchSize [bytes/lane]: 0"
  %s
fi
"""


@pytest.mark.parametrize("fails", [False, True])
def test_a_build_leaves_no_intermediate_files(tmp_path, monkeypatch, fails):
    tools, out = tmp_path / "tools", tmp_path / "out"
    tools.mkdir()
    out.mkdir()
    exe = tools / "hipcc"
    exe.write_text(HIPCC % ("exit 1" if fails else "exit 0"))
    exe.chmod(exe.stat().st_mode | stat.S_IXUSR)
    monkeypatch.setenv("PATH", f"{tools}{os.pathsep}{os.environ['PATH']}")
    monkeypatch.setattr(build, "LIB", str(out / "libmppi.so"))
    monkeypatch.setattr(hazards, "check", lambda lib: None)
    if fails:
        with pytest.raises(RuntimeError, match="hipcc failed"):
            build.build()
        assert os.listdir(out) == []
    else:
        build.build()
        assert os.listdir(out) == ["libmppi.so"]
