"""Units of rows that wait for units of lower numbers, on a model of a device that has little room: workgroups are dealt to its XCDs in
turn, each starts those dealt to it in their order as its places become free, and a unit keeps its place until every lower one has
started (csrc/units.hpp, compiled here for the CPU)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_19004_amd", "csrc")

MODEL = r"""
#include <cstdio>
#include <cstdlib>
#include <deque>
#include <vector>
#include "units.hpp"
using namespace ocean;

// Units that finish, of `units`.  Workgroup 0, which gives the places, holds one of XCD 0's from the start.
static int64_t finished(int64_t units, int xcds, int room, bool by_xcd)
{
    std::vector<std::deque<int64_t>> dealt(xcds), running(xcds);
    for (int64_t w = 0; w < units; ++w) dealt[(w + 1) % xcds].push_back(unit_of_workgroup(w, units, by_xcd));
    std::vector<char> started(units, 0);
    int64_t lead = 0, done = 0;   // units before `lead` have started
    for (bool moved = true; moved;) {
        moved = false;
        for (int x = 0; x < xcds; ++x) {
            while (!dealt[x].empty() && (int)running[x].size() < room - (x == 0)) {
                started[dealt[x].front()] = 1;
                running[x].push_back(dealt[x].front());
                dealt[x].pop_front();
                moved = true;
            }
        }
        while (lead < units && started[lead]) ++lead;
        for (int x = 0; x < xcds; ++x)
            for (size_t i = 0; i < running[x].size();)
                if (running[x][i] <= lead) {
                    running[x].erase(running[x].begin() + i);
                    ++done;
                    moved = true;
                } else {
                    ++i;
                }
    }
    return done;
}

int main(int argc, char **argv)
{
    const int64_t units = atoll(argv[1]);
    const int xcds = atoi(argv[2]), room = atoi(argv[3]);
    std::vector<char> seen(units, 0);
    for (int by = 0; by < 2; ++by)
        for (int64_t w = 0; w < units; ++w) seen[unit_of_workgroup(w, units, by)] |= 1 << by;
    bool all = true;
    for (int64_t u = 0; u < units; ++u) all = all && seen[u] == 3;
    printf("%d %lld %lld\n", all, (long long)finished(units, xcds, room, units_by_xcd(xcds * CUS_PER_XCD)), (long long)finished(units, xcds, room, true));
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("units")
    (d / "model.cpp").write_text(MODEL)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "model.cpp"), "-o", str(d / "model")], check=True)
    return lambda *a: [int(x) for x in subprocess.run([str(d / "model"), *map(str, a)], check=True, capture_output=True, text=True).stdout.split()]


@pytest.mark.parametrize("units", [1, 63, 64, 65, 128, 1000, 4096])
@pytest.mark.parametrize("xcds", [1, 2, 4, 8])
@pytest.mark.parametrize("room", [2, 3, 7, 64])
def test_every_unit_finishes(model, units, xcds, room):
    every_unit_once, finished, _ = model(units, xcds, room)
    assert every_unit_once == 1
    assert finished == units


def test_the_order_for_eight_xcds_would_stall_on_one(model):
    """What the rule keeps a partition of one XCD from, beside another kernel or with large rows (the model sees it)."""
    assert model(1000, 1, 40)[2] < 1000
