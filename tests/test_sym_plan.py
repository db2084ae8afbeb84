"""The work split of the all-pairs kernels (host code of the library, CPU only):
every unordered pair of superblocks once, runs that cut the cells without gaps,
slots within the scratch, and indices within 64 bits up to 2^30 particles."""

import os
import subprocess

import pytest

from paper_1901_08532_amd import build

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "sym_plan.h"
using namespace h6;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s (n %d block %d ncomp %d cap %lld)\n", __LINE__, #c, P.n, P.block, ncomp, (long long)cap); std::exit(1); } } while (0)

// runs and cells of a plan; slots: those the scratch holds
static void runs_of_plan(const SymPlan &P, int ncomp, int64_t cap) {
    const int64_t slots = cap / ((int64_t)ncomp * P.n);
    CHECK(P.first_cell(0) == 0 && P.first_cell(P.nsb) == P.cells && P.cells > 0);
    auto start = [&](int64_t r) { return r * P.cells / P.runs; };
    CHECK(start(0) == 0 && start(P.runs) == P.cells && P.runs > 0);
    const int step = P.runs > 4096 ? P.runs / 4096 : 1;
    for (int64_t r = 0; r < P.runs; r += step) {
        const int64_t a = start(r), b = start(r + 1);
        CHECK(a < b && a >= 0 && b <= P.cells);
        CHECK(P.run_of(a) == r && P.run_of(b - 1) == r);
    }
    const int sstep = P.nsb > 4096 ? P.nsb / 4096 : 1;
    for (int64_t I = 0; I < P.nsb; I += sstep) {
        const int cnt = P.run_count((int)I);
        CHECK(cnt >= 0 && P.slots_j + cnt <= slots);
        if (cnt) CHECK(P.first_run((int)I) >= 0 && P.first_run((int)I) + cnt <= P.runs);
    }
    if (P.ordered) {
        CHECK(P.runs == P.nsb);
        for (int64_t I = 0; I < P.nsb; I += sstep)
            CHECK(P.first_run((int)I) == I && P.run_count((int)I) == 1 && start(I) == P.first_cell((int)I));
    }
}

int main() {
    h6_ctx_s ctx;
    for (int64_t n : {1, 64, 255, 256, 257, 512, 513, 1025, 5000, 5121, 8192, 33001, 70001, 262144, 1000000})
        for (int block : {256, 512, 1024})
            for (int ncomp : {1, 4, 6, 9, 10, 13})
                for (int64_t per : {2, 5, 0}) {  // a context's two scratch sizes, the allocation-free one
                    const int64_t cap = per ? 9 * std::max<int64_t>(per * n, (int64_t)1 << 21) : (int64_t)1 << 22;
                    ctx.partial_cap = cap;
                    SymPlan P;
                    const SymCost cost{36.0f, 3.0f};
                    int d = 0;
                    const int nd = ((int)n + block - 1) / block / 2 + 1;
                    while (sym_plan(&ctx, (int)n, block, ncomp, cost, d, &P)) {
                        CHECK(P.d0 == d && P.d1 > d && P.d1 <= nd && !P.ordered);
                        runs_of_plan(P, ncomp, cap);
                        d = P.d1;
                    }
                    P.n = (int)n, P.block = block;
                    CHECK(d == nd || d == 0);  // all batches, or none
                    CHECK(d == nd || cap / ((int64_t)ncomp * n) < 3 || per == 0);
                    // every unordered pair of superblocks once over the offsets
                    const int nsb = ((int)n + block - 1) / block;
                    if (nsb <= 64) {
                        std::vector<int> seen(nsb * nsb, 0);
                        for (int I = 0; I < nsb; ++I)
                            for (int q = 0; q < nd; ++q) {
                                if (2 * q == nsb && nsb > 1 && I >= nsb / 2) continue;
                                const int J = (I + q) % nsb;
                                ++seen[I * nsb + J];
                                if (q) ++seen[J * nsb + I];
                            }
                        for (int s : seen) CHECK(s == 1);
                    }
                }
    for (int64_t n : {(int64_t)1, (int64_t)256, (int64_t)1000, (int64_t)350000000, (int64_t)1 << 30})
        for (int ncomp : {7, 10, 13}) {
            const int64_t cap = 18 * n;
            const int nsb = (int)((n + 255) / 256);
            int d = 0;
            while (d < nsb) {
                const SymPlan P = sym_plan_ordered((int)n, 256, d);
                CHECK(P.d0 == d && P.d1 > d && P.d1 <= nsb && P.nsb == nsb);
                if (d == 0 || P.d1 == nsb || d % 1000 == 0) runs_of_plan(P, ncomp, cap);
                d = P.d1;
            }
        }
    // third law at the largest sizes, in the smaller scratch
    for (int64_t n : {(int64_t)350000000, (int64_t)1 << 30}) {
        const int ncomp = 6;
        const int64_t cap = ctx.partial_cap = 18 * n;
        SymPlan P;
        for (int d : {0, 1, 5}) {
            const SymCost cost{36.0f, 3.0f};
            const bool planned = sym_plan(&ctx, (int)n, 512, ncomp, cost, d, &P);
            if (!planned) P.n = (int)n, P.block = 512;
            CHECK(planned);
            runs_of_plan(P, ncomp, cap);
        }
    }
    std::printf("ok\n");
}
"""


def test_plans(tmp_path):
    src, exe = tmp_path / "plans.hip", str(tmp_path / "plans")
    src.write_text(SOURCE)
    lib = os.path.dirname(build.LIB)
    r = subprocess.run([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-I" + build.INCLUDE, "-I" + build.CSRC,
                        str(src), "-o", exe, "-L" + lib, "-l:libh6.so", "-Wl,-rpath," + lib],
                       capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail(r.stderr[-2000:])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
