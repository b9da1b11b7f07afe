"""The scratch of padding and of large digit passes, and what the host tells the
bucket sort of its batches' padding (the library's layout and host code on the
CPU, with stand-in launchers)."""
import os

from _kernel_source import HERE, excerpt, run_host_code

PARTS = [
    r"^constexpr int kLsdThreads = ", r"^constexpr int kLsdItems = ", r"^constexpr uint32_t kLsdTile = ",
    r"^constexpr uint32_t kLsdMaxGroups = ", r"^struct LsdGrid \{", r"^inline LsdGrid lsd_grid\(",
]
LAUNCHERS = [
    "_ZN3lsm14launch_scatterERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE",
    "_ZN3lsm14launch_bucketsERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE",
    "_ZN3lsm16launch_sort_stepERKNS_8SortArgsES2_P12ihipStream_tPKNS_6KTimerE",
]


def test_padding_and_digit_counts(tmp_path):
    (tmp_path / "kernel_gen.inc").write_text(excerpt(PARTS))
    r = run_host_code(tmp_path, os.path.join(HERE, "pad_layout.cpp"), wrap=LAUNCHERS)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "padding and digit counts: ok" in r.stdout
