"""The words through which the windows of a sequence learn each other's rows (csrc/sc_gsc_words.h): whatever moments a reader's
two words come from, rows it accepts are those of all windows of the segment.  Compiled for the host, all orders tried."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <stdio.h>
#include <algorithm>
#include <vector>
#include "sc_gsc_words.h"
using namespace sc;
int main() {
    long long looks = 0, accepted = 0, wrong = 0;
    // slots of a segment, and the largest number of tokens that its words hold
    for (int slots : {1, 2, 3, 15, 16, 17, 31, 32, 1025}) {
        const int bits = segment_bits(slots);
        const long long most = std::min((1ll << (32 - bits)) - 1, (long long)kPubValue);
        wrong += !segment_holds(slots, most) + segment_holds(slots, most + 1) + ((1 << bits) <= slots) + (bits > 1 && (1 << (bits - 1)) > slots);
        for (int windows = 0; windows <= std::min(slots, 5); ++windows) {
            std::vector<int> rows;
            for (int w = 0; w < windows; ++w) rows.push_back(w == 0 ? (int)(most - 128 * (windows - 1)) : (w * 41) % 128 + 1);
            if (windows > 1) std::swap(rows[0], rows[1]);
            long long total = 0;
            for (int r : rows) total += r;
            std::vector<int> order(windows);
            for (int i = 0; i < windows; ++i) order[i] = i;
            do {
                // values of `part` after every addition; `upto` is filed by somebody who has seen all of them, with the rows before
                std::vector<uint32_t> part = {segment_start(windows)};
                for (int i : order) part.push_back(part.back() + segment_added(rows[i], bits));
                const long long before = most - total;
                for (uint32_t p : part)
                    for (int filed = 0; filed < 2; ++filed) {
                        const uint32_t upto = filed ? kPubRows | (uint32_t)(before + total) : 0u;
                        ++looks;
                        if (upto & kPubRows) { ++accepted; wrong += (long long)(upto & kPubValue) != before + total; }
                        if (segment_complete(p, bits)) { ++accepted; wrong += segment_rows(p, bits) != total; }
                        else wrong += p == part.back();
                    }
            } while (std::next_permutation(order.begin(), order.end()));
        }
    }
    printf("%lld %lld %lld\n", looks, accepted, wrong);
    return wrong != 0;
}
"""


def test_every_pair_of_words_gives_all_rows_or_none(tmp_path):
    src, exe = tmp_path / "words.cpp", tmp_path / "words"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_14303_amd", "csrc"), "-o", str(exe), str(src)])
    looks, accepted, wrong = map(int, subprocess.run([str(exe)], capture_output=True, text=True).stdout.split())
    assert wrong == 0 and 0 < accepted < looks
