"""work_deal (lstm_pipe.h) for the 32 workers that each product of a three-layer launch has: every share of every chunk taken once, and as many
of them as the consumer counts.  The function's own source, compiled for the host and walked as pipe_worker does.  CPU only."""
import os
import re
import subprocess

import pytest

from tests.test_worker_deal import ROOT, widths

WORKERS = 32


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    text = open(os.path.join(ROOT, "paper_2210_05064_amd", "csrc", "lstm_pipe.h")).read()
    rule = re.search(r"struct WorkDeal \{.*?\n\};\n.*?\n}\n", text, re.S).group(0)
    assert re.search(r"TRIPLE_WORK_COUNT = REC_MAX_GROUP;", text)
    tmp = tmp_path_factory.mktemp("deal")
    (tmp / "deal.cpp").write_text(
        "#include <cstdio>\n#include <initializer_list>\n#define __host__\n#define __device__\nconstexpr int WORK_COUNT = 64;\n" + rule +
        "int main() { for (int G = 4; G <= 32; ++G) for (int cap : {0, 1, 16, 17, 3000})\n"
        f'    printf("%d %d %d %d\\n", G, cap, work_deal(G, cap, {WORKERS}).sets, work_deal(G, cap, {WORKERS}).share); }}\n')
    subprocess.check_call(["g++", "-o", str(tmp / "deal"), str(tmp / "deal.cpp")])
    rows = [tuple(map(int, l.split())) for l in subprocess.check_output([str(tmp / "deal")], text=True).splitlines()]
    return {(g, cap): (sets, share) for g, cap, sets, share in rows}


@pytest.mark.parametrize("G", widths())
def test_every_share_of_every_chunk_once(deal, G):
    assert WORKERS // G >= 1
    for cap in (1, 16, 17, 3000):
        sets, share = deal[G, cap]
        assert sets >= 1 and (sets << share) * G <= WORKERS
        need = sorted((p, r) for p in range(1 << share) for r in range(G))   # what the consumer waits for: G << share
        for g in range(2):
            for n in (1, 2, 3, 7, 64):
                for descend in (False, True):
                    taken = {}
                    for worker in range(WORKERS):
                        team = worker // G
                        if team >= sets << share:
                            continue
                        first = ((team >> share) + g) % sets
                        at, step = (n - 1 - first, -sets) if descend else (first, sets)
                        while 0 <= at < n:
                            taken.setdefault(at, []).append((team & ((1 << share) - 1), worker % G))
                            at += step
                    assert sorted(taken) == list(range(n)) and all(sorted(t) == need for t in taken.values())


@pytest.mark.parametrize("G", widths())
def test_shares_cover_the_rows(deal, G):
    parts = 1 << deal[G, 3000][1]
    for total in (1, 15, 16, 17, 170, 2730):
        tiles = (total + 15) // 16
        edge = [min((tiles * k >> deal[G, 3000][1]) << 4, total) for k in range(parts + 1)]
        assert edge[0] == 0 and edge[-1] == total and edge == sorted(edge)
