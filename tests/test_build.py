"""Builds at the same time do not touch each other's files."""
import os
import subprocess
import sys
import textwrap

from paper_2305_05988_amd import build

# a compiler that waits, and whose output names the objects it was made of
COMPILER = """\
#!/bin/sh
for out; do :; done
sleep 0.5
if [ "$1" = --offload-arch=gfx950 ] && [ "$4" != -O3 ] && [ "$2" = -fPIC ]; then
  shift 3
  while [ "$1" != -o ]; do cat "$1"; shift; done > "$out"
else
  echo "$TAG" > "$out"
fi
"""


def test_two_builds_at_once(tmp_path):
    cc, lib = tmp_path / "cc", tmp_path / "lib.so"
    cc.write_text(COMPILER)
    cc.chmod(0o755)
    before = set(os.listdir(os.path.join(build.HERE, "csrc")))
    code = textwrap.dedent(f"""
        from paper_2305_05988_amd import build
        build.HIPCC, build.LIB = {str(cc)!r}, {str(lib)!r} + TAG
        build.build()
    """)
    running = []
    for tag in "ab":
        running.append(subprocess.Popen([sys.executable, "-c", f"TAG = {tag!r}\n" + code], cwd=build.ROOT,
                                        env={**os.environ, "TAG": tag}))
    assert [p.wait(timeout=60) for p in running] == [0, 0]
    for tag in "ab":
        assert (tmp_path / f"lib.so{tag}").read_text() == f"{tag}\n" * len(build.SOURCES)
    assert set(os.listdir(os.path.join(build.HERE, "csrc"))) == before
    assert sorted(os.listdir(tmp_path)) == ["cc", "lib.soa", "lib.sob"]
