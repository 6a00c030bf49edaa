"""The count of places for workgroups that wait for each other (psd_places.h), compiled for the host: no mix of threads holds more
than there are, what is given back can be taken again, and a launch that does not fit is refused at once."""
import os
import subprocess

SRC = r"""
#include <stdio.h>
#include <thread>
#include <vector>
#include "psd_places.h"
using psd::Places;
int main() {
    Places p;
    if (p.take(8)) return 1;              // none before the device is known
    p.open(387);
    if (p.total() != 384) return 2;       // whole rounds of the dies
    if (Places::of(1) != 8 || Places::of(192) != 192 || Places::of(193) != 200) return 3;
    if (!p.take(192) || !p.take(192) || p.take(8)) return 4;
    p.give(192);
    if (!p.take(184) || !p.take(8) || p.take(8)) return 5;
    p.give(384);
    if (p.take(392)) return 6;
    std::atomic<int> held{0}, most{0}, granted{0}, refused{0};
    std::vector<std::thread> ts;
    for (int t = 0; t < 6; ++t)
        ts.emplace_back([&, t] {
            for (int i = 0; i < 20000; ++i) {
                const int n = Places::of(8 + (i * 37 + t * 101) % 249);
                if (!p.take(n)) { refused++; continue; }
                const int now = held.fetch_add(n) + n;
                for (int m = most.load(); now > m && !most.compare_exchange_weak(m, now);) {}
                granted++;
                held.fetch_sub(n);
                p.give(n);
            }
        });
    for (auto& t : ts) t.join();
    printf("most held %d of 384, granted %d, refused %d\n", most.load(), granted.load(), refused.load());
    if (most > 384 || granted == 0) return 7;
    return p.take(384) ? 0 : 8;           // everything is back
}
"""


def test_places_are_never_handed_out_twice(tmp_path):
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_12966_amd", "csrc")
    (tmp_path / "t.cpp").write_text(SRC)
    exe = str(tmp_path / "t")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-pthread", "-I", csrc, "-o", exe, str(tmp_path / "t.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, (res.returncode, res.stdout)
