"""The two waves of the adjoint's workgroup leave their loop of barriers after
the same barrier, whatever the schedule: every interleaving of a wave that may
give up in any iteration and one that only follows, over the flags the kernel
uses (sigk_stop.h) and, as a control, over a single flag, which fails."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2502_20392_amd", "csrc")

MODEL = r"""
#include <cstdio>
#include <set>
#include <tuple>
#include "sigk_stop.h"
struct OneFlag {
    int raised;
    void clear() { raised = 0; }
    void raise(int) { raised = 1; }
    bool test(int) const { return raised != 0; }
};
// Each wave: 0 work (wave 0 raises in iteration `give`), 1 at the barrier,
// 2 read the outcome; -1 left, with the iteration it left after.
template <class F> struct State {
    F f;
    int at[2], k[2], out[2];
};
template <class F> bool explore(State<F> s, int give) {
    bool ok = true, any = false;
    // the barrier opens when both waves stand at it
    if (s.at[0] == 1 && s.at[1] == 1) {
        s.at[0] = s.at[1] = 2;
        return explore(s, give);
    }
    for (int w = 0; w < 2; ++w) {
        State<F> n = s;
        if (s.at[w] == 0) {
            if (w == 0 && s.k[0] == give) n.f.raise(s.k[0]);
            n.at[w] = 1;
        } else if (s.at[w] == 2) {
            const bool leave = s.f.test(s.k[w]) || s.k[w] < 0;
            if (leave) { n.at[w] = -1; n.out[w] = s.k[w]; }
            else { n.at[w] = 0; --n.k[w]; }
        } else
            continue;
        any = true;
        ok = explore(n, give) && ok;
    }
    if (!any) return s.at[0] == -1 && s.at[1] == -1 && s.out[0] == s.out[1];
    return ok;
}
template <class F> int bad() {
    int n = 0;
    for (int last = 0; last < 5; ++last)
        for (int give = -2; give <= last; ++give) {  // -2: never
            State<F> s{};
            s.f.clear();
            s.k[0] = s.k[1] = last;
            n += !explore(s, give);
        }
    return n;
}
int main() { std::printf("%d %d\n", bad<sigk::StopFlags>(), bad<OneFlag>()); }
"""


def test_both_waves_leave_after_the_same_barrier(tmp_path):
    src = tmp_path / "model.cpp"
    src.write_text(MODEL)
    exe = tmp_path / "model"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    kernel, single = map(int, subprocess.run([str(exe)], capture_output=True, text=True,
                                             check=True, timeout=60).stdout.split())
    assert kernel == 0
    assert single > 0  # the exploration does find the early leaver


def test_kernel_uses_these_flags():
    text = open(os.path.join(CSRC, "sigk_bwd.hip")).read()
    assert "sweep_two(int wave, StopFlags& stop)" in text and "*stop = 1" not in text
