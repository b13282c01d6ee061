"""The affinity's work distribution (csrc/mpm_work.h) on the CPU: over equal and ragged
batches, every block of every image belongs to exactly one workgroup of one launch."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "mpm_work.h"
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <tuple>
#include <vector>
using namespace mpm;

static long shapes = 0;

template <WorkOrder ORDER, bool SPLIT, bool TAB>
static void check(const std::vector<int>& nb, int log_groups, int slots)
{
    const int B = (int)nb.size();
    std::vector<int32_t> items(B + 1, 0), diags(B + 1, 0);
    for (int b = 0; b < B; ++b) {
        items[b + 1] = items[b] + work_items(ORDER, nb[b]);
        diags[b + 1] = diags[b] + nb[b];
    }
    const WorkShape shape(ORDER, B, nb[0] ? nb[0] : 1);
    const WorkCounts<TAB> c{shape, items.data(), diags.data()};
    std::map<std::tuple<int, int, int>, int> seen;
    int least = 1 << 30, most = 0;
    for (int g = 0; g < 1 << log_groups; ++g) {
        const WorkShare s = work_share(c, B, g, log_groups, slots, SPLIT);
        least = s.cnt < least ? s.cnt : least;
        most = s.cnt > most ? s.cnt : most;
        if (2 * s.ndef > slots || (s.ndef && (s.cnt - s.ndef) % slots)) { std::printf("rounds\n"); std::exit(1); }
        for (int slot = 0; slot < slots; ++slot) {
            int from = s.cnt > slot && s.lo < items[B] ? work_image(c, B, s.lo) : 0;
            for (int r = slot; r < s.cnt - s.ndef; r += slots) {
                const WorkBlock k = work_block<ORDER, SPLIT>(c, s, r, from);
                if (k.b < from) { std::printf("backwards\n"); std::exit(1); }
                from = k.b;
                ++seen[{k.b, k.q, k.t}];
            }
        }
        for (int e = 0; e < s.ndef; ++e) {
            const WorkBlock k = work_deferred(c, B, s, e);
            ++seen[{k.b, k.q, k.t}];
        }
    }
    if (most - least > 1) { std::printf("unbalanced\n"); std::exit(1); }
    long want = 0;
    for (int b = 0; b < B; ++b)
        for (int q = 0; q < nb[b]; ++q)
            for (int t = 0; t < nb[b]; ++t) {
                if (ORDER == kOrderSymmetric && t < q) continue;
                if (ORDER == kOrderBand && t != q) continue;
                ++want;
                if (seen[{b, q, t}] != 1) {
                    std::printf("B=%d block (%d, %d, %d) taken %d times\n", B, b, q, t, seen[{b, q, t}]);
                    std::exit(1);
                }
            }
    if ((long)seen.size() != want) { std::printf("%zu items, %ld blocks\n", seen.size(), want); std::exit(1); }
    ++shapes;
}

template <WorkOrder ORDER, bool SPLIT>
static void all(std::vector<int> n, int nb, int log_groups, int slots, std::mt19937& rng)
{
    check<ORDER, SPLIT, false>(n, log_groups, slots);
    check<ORDER, SPLIT, true>(n, log_groups, slots);
    for (int& v : n) v = (int)(rng() % (nb + 1));  // empty images among them
    check<ORDER, SPLIT, true>(n, log_groups, slots);
}

int main()
{
    std::mt19937 rng(7);
    for (int B : {1, 2, 3, 7, 8, 9, 16, 24, 33, 64, 65})
        for (int nb : {1, 2, 3, 4, 5, 9, 16})
            for (int groups : {0, 3})
                for (int slots : {256 >> groups, 512 >> groups, 5}) {
                    const std::vector<int> n(B, nb);
                    all<kOrderFull, false>(n, nb, groups, slots, rng);
                    all<kOrderSymmetric, false>(n, nb, groups, slots, rng);
                    all<kOrderSymmetric, true>(n, nb, groups, slots, rng);
                    all<kOrderBand, false>(n, nb, groups, slots, rng);
                }
    for (int B = 1; B < 200; ++B) {  // the places are a permutation of the images
        const WorkShape shape(kOrderFull, B, 1);
        std::vector<int> hit(B, 0);
        for (int i = 0; i < B; ++i) {
            const int b = work_place(i, shape.run);
            if (b < 0 || b >= B || hit[b]++) { std::printf("place %d of %d: %d\n", i, B, b); return 1; }
        }
    }
    for (uint32_t d : {1u, 2u, 3u, 7u, 10u, 36u, 136u, 4096u, 65535u, 65536u, 1000003u, 0x7fffffffu}) {
        const FixedDiv f(d);
        for (uint32_t k = 0; k < 100000; ++k) {
            const uint32_t v = (k < 1000 ? k : k < 2000 ? 0x7fffffffu - (k - 1000) : rng()) & 0x7fffffffu;
            if ((uint32_t)f((int)v) != v / d) { std::printf("%u / %u\n", v, d); return 1; }
        }
    }
    std::printf("%ld\n", shapes);
    return 0;
}
"""


def _run(tmp_path, text, result=int):
    """The driver's output (the number of batches it checked)."""
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src = tmp_path / "work.cpp"
    src.write_text(text)
    exe = tmp_path / "work"
    csrc = os.path.join(ROOT, "paper_2604_05718_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined,address", "-I", csrc,
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return result(r.stdout)


def test_every_block_exactly_once(tmp_path):
    assert _run(tmp_path, DRIVER) > 1000


# Shares below one round of the slots: with `lone`, where every share has two slots an item,
# those of diagonal blocks only run as halves; no others.
LONE_MAIN = r"""
int main()
{
    for (int B = 1; B <= 70; ++B)
        for (int nb : {1, 2, 3})
            for (int slots : {1, 2, 5, 16, 32}) {
                const WorkShape shape(kOrderSymmetric, B, nb);
                const WorkCounts<false> c{shape, nullptr, nullptr};
                std::map<std::tuple<int, int, int>, int> seen;
                for (int g = 0; g < 8; ++g) {
                    const WorkShare s = work_share(c, B, g, 3, slots, true, true);
                    const WorkShare t = work_share(c, B, g, 3, slots, true, false);
                    const int m = s.cnt % slots;
                    const int diags = work_diags_before(c, B, s.lo + s.cnt) - work_diags_before(c, B, s.lo);
                    const bool defers = m > 0 && 2 * m <= slots && diags >= m;
                    const int most = (c.items(B) + 7) / 8;
                    if (s.ndef != (defers && (s.cnt > slots || 2 * most <= slots) ? m : 0) || t.ndef != (defers && s.cnt > slots ? m : 0)) {
                        std::printf("B=%d nb=%d slots=%d", B, nb, slots);
                        return 1;
                    }
                    if (s.cnt < slots && s.ndef && s.ndef != s.cnt) { std::printf("a part"); return 1; }
                    for (int r = 0; r < s.cnt - s.ndef; ++r) {
                        const WorkBlock k = work_block<kOrderSymmetric, true>(c, s, r, 0);
                        ++seen[{k.b, k.q, k.t}];
                    }
                    for (int e = 0; e < s.ndef; ++e) {
                        const WorkBlock k = work_deferred(c, B, s, e);
                        if (k.q != k.t) { std::printf("off the diagonal"); return 1; }
                        ++seen[{k.b, k.q, k.t}];
                    }
                }
                if ((int)seen.size() != B * nb * (nb + 1) / 2) { std::printf("%zu blocks", seen.size()); return 1; }
                for (auto& e : seen)
                    if (e.second != 1) { std::printf("taken twice"); return 1; }
                ++shapes;
            }
    std::printf("%ld", shapes);
    return 0;
}
"""


SHARES_MAIN = r"""
int main()
{
    const int rows = 256, slots = 32;
    std::mt19937 rng(11);
    for (int k = 0; k < 60; ++k) {
        const int B = 1 + (int)(rng() % 120);
        std::vector<int> n(B);
        for (int& v : n) v = (int)(rng() % 4 == 0 ? 0 : rng() % 1400);
        std::vector<int32_t> items(B + 1, 0), diags(B + 1, 0);
        const WorkShape shape(kOrderSymmetric, B, 6);
        for (int i = 0; i < B; ++i) {
            const int nb = (n[work_place(i, shape.run)] + rows - 1) / rows;
            items[i + 1] = items[i] + work_items(kOrderSymmetric, nb);
            diags[i + 1] = diags[i] + nb;
        }
        const WorkCounts<true> c{shape, items.data(), diags.data()};
        for (int v : n) std::printf("%d ", v);
        std::printf("|");
        for (int lone = 0; lone < 2; ++lone)
            for (int g = 0; g < 8; ++g) std::printf(" %d", work_share(c, B, g, 3, slots, true, lone != 0).ndef);
        std::printf("/");
        ++shapes;
    }
    return 0;
}
"""


def test_shares_in_python_match_the_header(tmp_path):
    from work_shares import deferred

    head = DRIVER[:DRIVER.index("int main()")].replace("static void", "[[maybe_unused]] static void")
    batches = [b for b in _run(tmp_path, head + SHARES_MAIN, str).split("/") if b]
    assert len(batches) == 60
    some = 0
    for b in batches:
        ns, got = ([int(v) for v in part.split()] for part in b.split("|"))
        assert deferred(ns) + deferred(ns, lone=True) == got
        some += any(got[:8])
    assert some >= 10


def test_lone_diagonals_are_deferred_once(tmp_path):
    # The driver's batch checks stay in the program, unused.
    head = DRIVER[:DRIVER.index("int main()")].replace("static void", "[[maybe_unused]] static void")
    assert _run(tmp_path, head + LONE_MAIN) == 70 * 3 * 5
