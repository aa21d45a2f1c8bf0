"""work_deal (lstm_pipe.h): how the chunks of a group are dealt to the 64 workers of a two-layer launch.  The function's
own source is compiled for the host and walked as pipe_worker and the consumer walk it.  CPU only."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    """(G, cap) -> (sets, parts) for every width and group sizes on both sides of the rule."""
    text = open(os.path.join(ROOT, "paper_2210_05064_amd", "csrc", "lstm_pipe.h")).read()
    rule = re.search(r"struct WorkDeal \{.*?\n\};\n.*?\n}\n", text, re.S).group(0)
    tmp = tmp_path_factory.mktemp("deal")
    (tmp / "deal.cpp").write_text(
        "#include <cstdio>\n#include <initializer_list>\n#define __host__\n#define __device__\nconstexpr int WORK_COUNT = 64;\n" + rule +
        "int main() { for (int G = 4; G <= 32; ++G) for (int cap : {0, 1, 16, 17, 3000})\n"
        '    printf("%d %d %d %d\\n", G, cap, work_deal(G, cap).sets, 1 << work_deal(G, cap).share); }\n')
    subprocess.check_call(["g++", "-o", str(tmp / "deal"), str(tmp / "deal.cpp")])
    rows = [tuple(map(int, l.split())) for l in subprocess.check_output([str(tmp / "deal")], text=True).splitlines()]
    return {(g, cap): (sets, parts) for g, cap, sets, parts in rows}


def widths():
    """Workers that hold the weights of a supported width: 16 units each up to 512, 32 above."""
    return sorted({h // 16 for h in range(64, 513, 64)} | {h // 32 for h in range(576, 1025, 64)})


@pytest.mark.parametrize("G", widths())
def test_every_chunk_goes_to_one_whole_set(deal, G):
    for cap in (1, 16, 17, 3000):
        sets, parts = deal[G, cap]
        for g in range(3):
            for n in (1, 2, 3, 7, 64):
                for descend in (False, True):
                    done = {}
                    for w in range(64):
                        team = w // G
                        if team >= sets * parts:
                            continue
                        first = (team // parts + g) % sets
                        at, step = (n - 1 - first, -sets) if descend else (first, sets)
                        while 0 <= at < n:
                            done.setdefault(at, []).append((team % parts, w % G))
                            at += step
                    want = sorted((p, r) for p in range(parts) for r in range(G))   # what the consumer counts: G * parts
                    assert sorted(done) == list(range(n)) and all(sorted(d) == want for d in done.values())


@pytest.mark.parametrize("G", widths())
def test_no_whole_team_stays_idle(deal, G):
    """A width whose weights fit the workers several times: few pieces or many, no further team would fit."""
    for cap in (1, 16, 17, 3000):
        sets, parts = deal[G, cap]
        assert 64 - G * sets * parts < G


@pytest.mark.parametrize("G", widths())
def test_shares_of_a_chunk(deal, G):
    """The teams of a set take whole tiles of 16 rows, all of them, each once."""
    parts = deal[G, 3000][1]
    for total in (1, 15, 16, 17, 170, 2730):
        tiles = (total + 15) // 16
        edge = [min(tiles * k // parts * 16, total) for k in range(parts + 1)]
        assert edge[0] == 0 and edge[-1] == total and edge == sorted(edge)


def test_even_slices_of_the_contraction(tmp_path):
    """work_even: eight slices that cover all blocks of every width below 512, at most four each, and the two waves of a
    SIMD (slices s and s + 4) share the work as evenly as the SIMDs can."""
    text = open(os.path.join(ROOT, "paper_2210_05064_amd", "csrc", "lstm_pipe.h")).read()
    rule = re.search(r"inline __host__ __device__ int work_even.*?}\n", text, re.S).group(0)
    (tmp_path / "even.cpp").write_text(
        "#include <cstdio>\n#define __host__\n#define __device__\nconstexpr int REC_WAVES = 8;\n" + rule +
        'int main() { for (int b = 4; b < 32; b += 4) for (int s = 0; s <= 8; ++s) printf("%d\\n", work_even(b, s)); }\n')
    subprocess.check_call(["g++", "-o", str(tmp_path / "even"), str(tmp_path / "even.cpp")])
    first = [int(v) for v in subprocess.check_output([str(tmp_path / "even")], text=True).split()]
    for k, blocks in enumerate(range(4, 32, 4)):
        at = first[9 * k:9 * k + 9]
        n = [b - a for a, b in zip(at, at[1:])]
        assert at[0] == 0 and at[8] == blocks and min(n) >= 0 and max(n) <= 4
        simd = [n[s] + n[s + 4] for s in range(4)]
        assert max(simd) - min(simd) <= (0 if blocks % 4 == 0 else 1)
