"""Every digit-pass sort of a bulk insertion starts from a cleared histogram,
whatever the sizes of the parts sorted before it (the library's host code on the
CPU, with stand-in launchers)."""
import os

from _kernel_source import HERE, run_host_code


def test_histogram_is_clear_for_every_part(tmp_path):
    r = run_host_code(tmp_path, os.path.join(HERE, "bulk_histogram.cpp"),
                      wrap=["_ZN3lsm11launch_sortERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerEPi"])
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "0 began with counts left over" in r.stdout
