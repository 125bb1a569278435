"""Into how many pieces signature calls cut long paths, and how many short ones share a wavefront: the plan's rules at shapes
where the counts were timed (the times stand beside the rules in the plan header)."""
import os
import re
import subprocess

import pytest

from paper_2509_10613_amd import binding as sk

T, LL = sk.SK_FLAG_TIME_AUG, sk.SK_FLAG_LEAD_LAG


def number(text, key):
    return int(re.search(r"\b%s=(\d+)" % key, text).group(1))


@pytest.mark.parametrize("B,L,d,N,flags,forward,backward", [
    (40, 2048, 7, 5, 0, 4, 1), (200, 100, 3, 3, 0, 8, 8), (100, 200, 4, 3, 0, 16, 16), (4, 1024, 8, 3, 0, 32, 32),
    (32, 1024, 5, 4, T, 16, 16), (16, 1024, 16, 4, 0, 4, 1), (128, 256, 4, 6, 0, 4, 1), (8000, 500, 2, 3, 0, 16, 4),
    (64, 128, 12, 3, 0, 4, 1), (3000, 200, 3, 2, 0, None, 4), (1000, 20, 3, 3, 0, 1, 1), (10, 24, 2, 3, 0, 1, 1),
])
def test_pieces(B, L, d, N, flags, forward, backward):
    if forward is not None:
        assert number(sk.signature_describe(B, L, d, N, flags, sk.SK_F64), "pieces_per_path") == forward
    text = sk.signature_bwd_describe(B, L, d, N, flags, sk.SK_F64)
    assert number(text, "pieces_per_path") == backward
    # an empty piece would be one that starts past the path
    assert number(text, "segments_per_piece") * backward < 2 * (L - 1) + backward


@pytest.mark.parametrize("B,L,d,N,paths", [(50, 9, 2, 3, 2), (3000, 9, 2, 3, 3), (40000, 9, 2, 3, 32), (5000, 30, 4, 3, 5)])
def test_paths_per_wave(B, L, d, N, paths):
    text = sk.signature_describe(B, L, d, N, 0, sk.SK_F64)
    assert number(text, "paths_per_wave") == paths
    assert number(text, "grid") * 4 * paths >= B > (number(text, "grid") - 1) * 4 * paths


def test_adjoint_slots(tmp_path):
    # every channel count and level whose signatures have fewer than 2^31 entries (and a kernel that multiplies pieces)
    source, program = tmp_path / "slots.cpp", str(tmp_path / "slots")
    source.write_text("""
#include <cstdio>
#include "sg_plan.h"
int main()
{
    unsigned start[16], shift[16];
    for (int N = 1; N <= sg::kPiecesMaxN; ++N)
        for (int D = 1; D <= 40000; D = D < 200 ? D + 1 : D + 97) {
            const int64_t n = sg::sig_length(D, N);
            if (n == 0 || n >= ((int64_t)1 << 31)) break;
            const uint64_t slots = sg::adjoint_slots(D, N, start, shift);
            uint64_t words = 1;
            bool ok = slots < ((uint64_t)1 << 31) && slots >= start[N + 1] && slots % (1u << shift[1]) == 0 && start[1] == 0;
            for (int k = 1; k <= N; ++k) {
                words *= (uint64_t)D;
                ok = ok && start[k + 1] - start[k] == words << shift[k] && start[k] % (1u << shift[k]) == 0 && (k == 1 || shift[k] <= shift[k - 1]);
            }
            if (!ok) std::printf("D = %d, N = %d: %llu\\n", D, N, (unsigned long long)slots);
        }
}
""")
    csrc = os.path.join(os.path.dirname(sk.LIB_PATH), "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", csrc, str(source), "-o", program], check=True)
    out = subprocess.run([program], check=True, capture_output=True, text=True).stdout
    assert out == ""
