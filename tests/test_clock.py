"""Phase timings of a solve (csrc/dd_clock.h): the stamps' bookkeeping, compiled for the CPU and driven with an in-order
model of a stream in the order the outer solvers use it, far past the number of slots; and on the GPU the timings that
long solves report."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1412_2629_amd", "csrc")

# Each phase takes a known number of ticks on the model's clock, so every total is known exactly.  late: nothing runs
# before the host waits; otherwise everything runs at once.
MODEL = r"""
#include <cstdio>
#include <cstdlib>
#include <functional>
#include "dd_clock.h"
struct Stream {
    std::vector<std::function<void()>> queue;
    unsigned long long now = 1000000;
    bool late;
    void put(std::function<void()> f) { if (late) queue.push_back(f); else f(); }
    void run(long ticks) { put([=] { now += ticks; }); }
    void wait() { for (auto &f : queue) f(); queue.clear(); }
} st;
struct Device {
    void stamp(unsigned long long *p) { st.put([=] { *p = st.now; }); }
    void wait() { st.wait(); }
    double ms_per_tick() const { return 1; }
};
typedef dd::Clock<Device> Clock;
typedef dd::Timer<Device> Timer;
enum { SAP = 100, OP = 7, GS = 13, OTHER = 5, IDLE = 3 };
int main(int argc, char **argv)
{
    const int kind = atoi(argv[1]), m = atoi(argv[2]), steps = atoi(argv[3]);
    st.late = atoi(argv[4]);
    unsigned long long slots[dd::CLOCK_SLOTS];
    Clock clk(Device(), slots);
    double sap = 0, op = 0, gs = 0, other = 0;
    long nop = 0, nother = 0;
    for (int k = 0, j = 0; k < steps; k++) {
        if (kind == 0) {   // a timer for each phase, the later ones starting where the one before ended
            { Timer t(clk, &sap); st.run(SAP); }
            { Timer t(clk, &op, true); st.run(OP); }
            { Timer t(clk, &gs, true); st.run(GS - 1); st.wait(); st.run(1); }
        } else {           // stamps taken directly, the last one by a kernel, read at each step
            const long t0 = clk.mark();
            st.run(SAP);
            const long t1 = clk.mark();
            st.run(OP);
            const long t2 = clk.mark(), t3 = clk.slot();
            st.run(GS);
            Device().stamp(clk.at(t3));
            clk.add(t0, t1, &sap);
            clk.add(t1, t2, &op);
            clk.add(t2, t3, &gs);
            st.wait();
            clk.collect();
        }
        nop++;
        st.run(IDLE);
        if (++j < m && k + 1 < steps) continue;
        j = 0;   // a cycle's end
        { Timer t(clk, &other); st.run(OTHER); }
        { Timer t(clk, &op, true); st.run(OP); }
        nop++;
        st.wait();
        { Timer t(clk, &other); st.run(OTHER); st.wait(); }
        nother += 2;
    }
    clk.finish();
    printf("%g %g %g %g\n", sap - (double)steps * SAP, op - (double)nop * OP, gs - (double)steps * GS,
           other - (double)nother * OTHER);
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("clock")
    (d / "model.cpp").write_text(MODEL)
    exe = str(d / "model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(d / "model.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("late", [0, 1])
@pytest.mark.parametrize("kind,m", [(0, 16), (0, 8), (0, 3), (1, 16)])
@pytest.mark.parametrize("steps", [1, 10, 16, 17, 30, 79, 500])
def test_sums_past_the_slots(model, kind, m, steps, late):
    out = subprocess.run([model, str(kind), str(m), str(steps), str(late)], check=True, capture_output=True, text=True)
    assert [float(v) for v in out.stdout.split()] == [0, 0, 0, 0]


@pytest.mark.gpu
@pytest.mark.parametrize("kind,deflate", [("fgcr", 0), ("fgmres_dr", 6), ("fgcr_mixed", 0)])
def test_timings_of_a_long_solve(kind, deflate):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests.gpu_cases import Case, dev
    case = Case("4^4/2^4", (4, 4, 4, 4), (2, 2, 2, 2), 0.16, 1.0, 0.3, 603)
    ctx = case.context()
    ctx.set_schwarz("additive")
    ctx.set_sap(4, 2, "f32")
    ctx.set_solver(16, 1e-9, 40)
    ctx.set_outer(kind, deflate)
    for _ in range(2):
        _, info, st = ctx.solve(dev(case.source(31)))
        i = info[0]
        parts = [i[k] for k in ("t_sap_ms", "t_A_ms", "t_gs_ms", "t_other_ms")]
        print(kind, i)
        assert st == 0 and i["iters"] >= 25
        assert min(parts) > 0 and sum(parts) <= i["t_total_ms"]
        # four cycles of two launches each against one launch: the preconditioner is the larger part
        assert i["t_sap_ms"] > i["t_A_ms"]
