"""Sizes of buffers that several kernels share, at the ends of their ranges: host
constants of the library's internal header, compiled and printed. No kernel runs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1302_4587_amd", "csrc")


def _values(tmp_path, *exprs):
    """The integer values of expressions over lm_internal.h, on the host."""
    src, exe = tmp_path / "probe.hip", tmp_path / "probe"
    body = "".join(f'printf("%lld\\n", (long long)({e}));' for e in exprs)
    src.write_text(f'#include <cstdio>\n#include "lm_internal.h"\nusing namespace lm;\nint main() {{ {body} return 0; }}\n')
    hipcc = os.environ.get("HIPCC") or "/opt/rocm/bin/hipcc"
    r = subprocess.run([hipcc, "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return [int(x) for x in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()]


def test_phase_log_of_a_batch_fits_its_buffer(tmp_path):
    """The sums of a batch's phase log (16 bytes a phase) stay inside the buffer of the partial results they borrow,
    and hold every phase of a graph without self-loops (two vertices a phase at least)."""
    sizes = (1, 2, 3, 4095, 32767, 32768, 32769, 65535, 65536)
    room, largest, *recs = _values(tmp_path, "kMaxFirstRanges * 2 * sizeof(Part)", "kSoloMaxN",
                                   *(f"solo_log_records({n})" for n in sizes))
    assert largest == sizes[-1]
    for n, k in zip(sizes, recs):
        assert 16 * k <= room and k >= n // 2, n


def test_phases_past_the_log_have_no_record(tmp_path):
    """A graph with self-loops (refused only by the input check) can have a phase per vertex, more than a batch's log has
    records: phase t's record, 1-based, exists exactly for t up to the records."""
    recs, n = _values(tmp_path, "solo_log_records(kSoloMaxN)", "kSoloMaxN")
    at = (1, 2, recs - 1, recs, recs + 1, n - 1, n)
    assert _values(tmp_path, *(f"solo_log_slot({t}, {recs})" for t in at)) == [t - 1 if t <= recs else -1 for t in at]


def test_row_numbers_near_the_limit(tmp_path):
    """Rows past the last one, of up to 2^31 - 1, are the end and never wrap below zero."""
    n = 2**31 - 1
    at = [(0, 0, n), (0, 64, 64), (0, 63, 64), (n - 63, 62, n), (n - 63, 63, n), (n - 63, 64, n), (n - 63, 192, n), (n - 1, 64, n), (5, 700, 6)]
    got = _values(tmp_path, *(f"row_or_end({r}, {i}u, {m})" for r, i, m in at))
    assert got == [min(r + i, m) for r, i, m in at]


# (graphs, vertices of each, average degree, stream-ordered, whether one workgroup each is the faster way by a fifth or more)
SIDES = [
    (2, 8000, 8, 1, True), (128, 30000, 8, 1, True), (128, 60000, 8, 1, True), (512, 8000, 8, 1, True), (4000, 36, 3, 1, True), (64000, 740, 4, 1, True),
    (2, 30000, 8, 1, False), (8, 30000, 8, 1, False), (8, 60000, 8, 1, False), (32, 60000, 8, 1, False),
    (16000, 36, 3, 1, False), (64000, 36, 3, 1, False), (16000, 140, 5, 1, False),
    (2, 60000, 8, 0, True), (32, 60000, 8, 0, True), (64000, 740, 4, 0, True), (8000, 36, 3, 0, True),
    (2, 60000, 64, 0, False), (4, 4000, 250, 0, False), (24000, 36, 3, 0, False), (128000, 140, 5, 0, False),
]


@pytest.mark.parametrize("graphs,n,degree,stream_ordered,solo", SIDES)
def test_batches_one_workgroup_each(tmp_path, graphs, n, degree, stream_ordered, solo):
    """The rule for a weighted batch of equal graphs falls on the side that measured faster."""
    N, T, a = graphs * n, graphs * n * degree, stream_ordered
    most, entries = _values(tmp_path, f"solo_graph_limit({N}, {a})", f"solo_entry_limit({N}, {T}, false, {a})")
    assert (graphs <= most and n * degree <= entries) == solo
