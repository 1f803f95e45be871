"""Two builds at once (a test worker and a user, say) do not take each other's
objects away, and a failing one leaves nothing behind.  The compiler is a stub
that writes its output after a while and links only objects that exist."""
import glob
import os
import threading
import time

import pytest

from paper_2604_22718_amd import build

STUB = """#!/bin/sh
for a in "$@"; do
  if [ "$prev" = -o ]; then out="$a"; fi
  case "$a" in *.o) [ "$prev" = -o ] || [ -e "$a" ] || { echo "no $a" >&2; exit 1; };; esac
  case "$a" in *rtt_pass.hip) [ -z "$FAIL_PASS" ] || exit 1;; esac
  prev="$a"
done
sleep 0.3
echo built > "$out"
"""


@pytest.fixture
def stub(tmp_path, monkeypatch):
    exe = tmp_path / "hipcc"
    exe.write_text(STUB)
    exe.chmod(0o755)
    monkeypatch.setattr(build, "HIPCC", str(exe))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "librtt.so"))
    return tmp_path


def leftovers(tmp_path):
    return glob.glob(os.path.join(build.CSRC, "*.o")) + glob.glob(str(tmp_path / "librtt.so.*"))


def test_two_builds_at_once(stub):
    errors = []

    def run():
        try:
            build.build()
        except Exception as e:   # noqa: BLE001 - the thread's failure is the test's
            errors.append(e)

    threads = [threading.Thread(target=run) for _ in range(2)]
    for t in threads:
        t.start()
        time.sleep(0.15)   # the second links while the first cleans up
    for t in threads:
        t.join()
    assert not errors and (stub / "librtt.so").exists() and not leftovers(stub)


def test_failed_build_leaves_nothing(stub, monkeypatch, capsys):
    monkeypatch.setenv("FAIL_PASS", "1")
    with pytest.raises(RuntimeError):
        build.build()
    assert not (stub / "librtt.so").exists() and not leftovers(stub)
