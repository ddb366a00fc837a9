"""The rule by which the CG kernels read the iteration at which a run stops
(csrc/cg_stop.h), run on the host over every interleaving of one block's waves:
each wave reads the solver state before or after another block of the launch has
recorded this iteration's stop.  All waves must take part in the block's sum or
none, and all must go on or stop together with the beta of a quiet launch."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0910_2950_amd", "csrc")

MODEL = r"""
#include <climits>
#include <cstdio>
#include <initializer_list>
#include "cg_stop.h"
using namespace fgi;

struct State { int stop_at, base0; double rr[2], rr_stop, beta; };
constexpr int W = 4;               // waves of a block
static const double part[W] = {0.25, 0.5, 1.0, 2.0};   // each wave's part of the partials

// one block: wave w reads its own copy of the state; returns the number of faults
static int block(const State* seen, int iter, bool go_ref, double beta_ref) {
    int faults = 0, arrived = 0;
    for (int w = 0; w < W; w++) {  // who reaches the sum's barrier
        double b = 0;
        bool in = false;
        cg_open(seen[w], iter, false, [&] { in = true; return 0.0; }, [](double, double, bool) {}, b);
        arrived |= in << w;
    }
    if (arrived != 0 && arrived != (1 << W) - 1) faults++;
    double total = 0;
    for (int w = 0; w < W; w++)
        if (arrived >> w & 1) total += part[w];
    for (int w = 0; w < W; w++) {
        double b = 0;
        const bool go = cg_open(seen[w], iter, false, [&] { return total; }, [](double, double, bool) {}, b);
        if (go != go_ref || (go && b != beta_ref)) faults++;
    }
    return faults;
}

int main() {
    int faults = 0, runs = 0;
    for (int iter : {4, 5})
        for (int base0 : {0, iter})
            for (double rr_stop : {1.0, 3.75, 10.0})                // 3.75 = the sum of part
                for (int before : {2, iter - 1, iter, INT_MAX}) {   // stop_at as earlier launches left it
                    State quiet{before, base0, {7.5, 7.5}, rr_stop, 0.125};
                    const double rr = 3.75, be = iter == base0 ? 0.125 : rr / 7.5;
                    const bool stop = iter != base0 && rr <= rr_stop, go = before > iter && !stop;
                    // what block 0 leaves
                    State after = quiet;
                    double b = 0;
                    int wrote = 0;
                    cg_open(quiet, iter, true, [&] { return rr; },
                            [&](double r, double bb, bool s) {
                                wrote = 1;
                                after.rr[iter & 1] = r;
                                if (s) after.stop_at = iter;
                                else after.beta = bb;
                            },
                            b);
                    if (wrote != (before > iter && iter != base0)) faults++;
                    if (after.stop_at != (stop && before > iter ? iter : before)) faults++;
                    for (int mask = 0; mask < (1 << W); mask++) {   // who reads before, who after
                        State seen[W];
                        for (int w = 0; w < W; w++) seen[w] = mask >> w & 1 ? after : quiet;
                        faults += block(seen, iter, go, be);
                        runs++;
                    }
                }
    // a site block beside the one that records the stop acts alike on both readings
    for (int before : {2, 4, 5, INT_MAX})
        if (cg_leaves(before, 5, true) != cg_leaves(before > 5 ? 5 : before, 5, true)) faults++;
    if (!cg_leaves(5, 5, false) || cg_leaves(6, 5, false)) faults++;
    printf("%d runs, %d faults\n", runs, faults);
    return faults != 0;
}
"""


def test_every_interleaving_of_a_block(tmp_path):
    src, exe = tmp_path / "model.cpp", tmp_path / "model"
    src.write_text(MODEL)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert r.stdout.startswith("768 runs"), r.stdout


CUTS = r"""
#include <climits>
#include <cstdio>
#include <initializer_list>
#include "cg_stop.h"
using fgi::cg_cut;
int main() {
    int faults = 0;
    for (int batch : {1, 3, 8, 1024})
        for (int base0 : {0, 1, 7, 10, 1000})
            for (int maxiter : {base0 + 1, base0 + 7, base0 + 8, base0 + 9, 20000, INT_MAX - 8, INT_MAX - 1, INT_MAX}) {
                const int cut = cg_cut(base0, maxiter, batch);
                if (cut < maxiter) faults++;   // never short of the limit, and less than a batch past it
                if (cut != INT_MAX && ((cut - base0) % batch || cut - maxiter >= batch)) faults++;
                if (cut == INT_MAX && maxiter < INT_MAX - batch) faults++;
            }
    printf("%d faults\n", faults);
    return faults != 0;
}
"""


def test_cut_off_of_a_run(tmp_path):
    src, exe = tmp_path / "cuts.cpp", tmp_path / "cuts"
    src.write_text(CUTS)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", CSRC, str(src),
                    "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
