"""Which rows the queries of one launch gather and how large their tiles of source
walks are, over every mix of graphs: the library's own rule, compiled for the host.
"""
import itertools
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Reads "kind units graph..." lines; prints the launch's rows and each query's tile.
PROGRAM = """
#include <iostream>
#include <sstream>
#include "common.hpp"
using namespace srk;
int main() {
    // graphs: 0 within an XCD's L2, 1 beyond it, 2 with many hubs, 3 not packed
    Graph gs[4];
    for (Graph &g : gs) { g.n_active = 1000; g.m_slots = 1 << 22; g.obits = 23; }
    gs[0].m_slots = 1 << 16;
    gs[2].n_hubs = HUB_ROWS - 1;
    gs[3].obits = 0;
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        int kind, graph;
        long long units;
        in >> kind >> units;
        std::vector<QueryDesc> d;
        std::vector<const Graph *> g;
        while (in >> graph) {
            g.push_back(&gs[graph]);
            QueryDesc q{};
            q.kind = kind;
            q.tile_nodes = tile_nodes_for(gs[graph], kind, 9502, 64);
            d.push_back(q);
        }
        std::vector<QueryDesc *> pd;
        for (QueryDesc &q : d) pd.push_back(&q);
        std::cout << rows_of(settle_tiles(g.data(), pd.data(), pd.size(), units));
        for (QueryDesc &q : d) std::cout << ' ' << q.tile_nodes;
        std::cout << std::endl;
    }
}
"""
E, PACKED, HUBS, MIXED = range(4)
FULL = {0: 24576, 1: 24576, 2: 20480}
SMALL = 12288


@pytest.mark.skipif(not shutil.which(HIPCC), reason="hipcc not present")
def test_small_tiles_only_with_packed_rows_of_many_hubs(tmp_path):
    src, exe = tmp_path / "rows.cpp", str(tmp_path / "rows")
    src.write_text("#include <vector>\n" + PROGRAM)
    csrc = os.path.join(ROOT, "paper_2304_04015_amd", "csrc")
    subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-std=c++17", "-I", csrc,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=120)
    cases = [(kind, units, mix) for kind in FULL for units in (1000, 1 << 30)
             for count in (1, 2, 3) for mix in itertools.product(range(4), repeat=count)]
    text = "".join(f"{k} {u} {' '.join(map(str, m))}\n" for k, u, m in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
    for (kind, units, mix), line in zip(cases, out.splitlines()):
        rows, *tiles = map(int, line.split())
        hubs_alone = set(mix) == {2} and kind != 2 and units < 1 << 30
        packs = {1} & set(mix)                      # (the stratified kind has no small tiles)
        none = set(mix) & {2, 3}
        want = HUBS if hubs_alone else E if not packs else MIXED if none else PACKED
        assert rows == want, (kind, units, mix, rows)
        assert set(tiles) == {SMALL if rows == HUBS else FULL[kind]}, (kind, units, mix, tiles)
    assert len(out.splitlines()) == len(cases)
