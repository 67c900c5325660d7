"""The rows that the decoding loop's kernels read of a sequence's trace (csrc/trace_rows.h), on the CPU: over all states that rounds can
reach, none lies outside the trace.  A read past its end may fault on the GPU or go unseen, so the rules themselves are checked."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2411_18462_amd", "csrc", "trace_rows.h")


def _run(tmp_path, body):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(f'#include <algorithm>\n#include <cstdio>\n#include <cstdlib>\n#include "{HEADER}"\nusing namespace svip;\n{body}')
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                           str(src), "-o", str(exe)])
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-2000:]
    assert int(p.stdout.split()[-1]) > 1000                        # states looked at


@pytest.mark.parametrize("gamma_max", [1, 2, 7, 40])
def test_step_by_step_rounds_stay_inside_the_trace(tmp_path, gamma_max):
    """A round may begin wherever the trace holds cap + 1 rows from its position on.  All positions up to gamma_max are launched for the
    whole batch: a sequence of a smaller limit (the Heuristic rule's) has stopped by then, and its row is still requested."""
    _run(tmp_path, """
int main()
{
    const int gamma_max = %d;
    long seen = 0;
    for (int L = gamma_max + 1; L < 3 * gamma_max + 60; ++L)
        for (int cap = 1; cap <= gamma_max; ++cap)
            for (int pos = 0; pos + cap + 1 <= L; ++pos)
                for (int j = 0; j < gamma_max; ++j, ++seen) {
                    const int row = pos + step_row(j, cap);
                    const bool drafting_ok = j >= cap || row == pos + j;
                    if (row < pos || row > L - 2 || !drafting_ok) {
                        std::printf("L %%d cap %%d pos %%d step %%d: row %%d\\n", L, cap, pos, j, row);
                        return 1;
                    }
                }
    std::printf("%%ld\\n", seen);
}
""" % gamma_max)


def test_the_statistics_kernels_take_their_row_from_the_rule():
    """Both kernels that request a row before its stop flag is looked at."""
    text = open(os.path.join(ROOT, "paper_2411_18462_amd", "csrc", "draft_kernels.h")).read()
    for kernel in ("k_draft_stats(DraftArgs a)", "k_draft_step(DraftArgs a)"):
        body = text[text.index(kernel):]
        body = body[:body.index("request_stop_flag(a, b)")]
        assert "step_row_offset(a, b)" in body and "draft_row_offset(a, b, a.step_j)" not in body, kernel


def test_rows_of_the_greedy_stream(tmp_path):
    """Of every running sequence a launch reads at least one further row (or the loop would launch for ever), none outside the trace, and
    none past what a round of it can reach -- also where a call asks for fewer tokens than one before it did, so that the sequence has
    them already."""
    _run(tmp_path, """
int main()
{
    long seen = 0;
    for (int gamma_max = 1; gamma_max <= 5; ++gamma_max)
    for (int L = gamma_max + 1; L <= 14; ++L)
    for (int start = 0; start < L; ++start)
    for (int max_new : {0, 1, 2, 5, 9, 30, 2147483647})
    for (int cap = 1; cap <= gamma_max; ++cap)
    for (int pos = start; pos + cap + 1 <= L; ++pos)
    for (int drafted = -1; drafted < cap; ++drafted)
    for (int ahead : {1, 2, 7})
    for (int group : {1, 3, 128}) {
        const int n = stream_rows(pos, drafted, cap, start, L, gamma_max, max_new, ahead, group);
        const int known = drafted > 0 ? drafted : 0;
        const long long tokens = (long long)start + max_new, last = std::max(tokens - 1 + gamma_max, (long long)pos + cap);   // target row
        ++seen;
        if (n < 1 || n > group || pos + known + n > L - 1 || pos + known + n > last) {
            std::printf("gamma_max %d L %d start %d max_new %d cap %d pos %d drafted %d ahead %d group %d: %d\\n", gamma_max, L, start,
                        max_new, cap, pos, drafted, ahead, group, n);
            return 1;
        }
    }
    std::printf("%ld\\n", seen);
}
""")
