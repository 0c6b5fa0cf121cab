"""The rule that picks the form of a CRT-halves launch (csrc/launch_rule.cpp, built
here for the host) against measured times: whatever it picks takes no more than
6 % longer than the fastest form measured for that shape."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2111_11924_amd", "csrc")
BITS = [128, 256, 512, 1024, 2048, 3072, 4096, 6144, 8192]

# bits, keys, chunks per key: ms of the group form (G), the lane form (L) and
# Montgomery products (M), 256 compute units; blinded: with two lanes per number (T)
PLAIN = [
    (1024, 64, 64, dict(G=0.86, L=1.06)), (1024, 256, 256, dict(G=4.58, L=1.96)),
    (1024, 1024, 64, dict(L=2.82, M=2.06)), (1024, 512, 192, dict(L=3.68, M=2.93)),
    (2048, 64, 64, dict(G=2.72, M=5.41)), (2048, 256, 64, dict(G=5.91, L=4.07, M=5.45)),
    (2048, 1024, 64, dict(L=8.89, M=11.3)), (2048, 256, 256, dict(G=23.4, L=8.35)),
    (3072, 64, 64, dict(G=4.57, M=17.8)), (3072, 256, 64, dict(G=17.7, L=14.2, M=17.9)),
    (3072, 256, 96, dict(L=24.35, M=18.7)), (3072, 256, 192, dict(L=29.5, M=36.0)),
    (3072, 512, 64, dict(L=37.9, M=18.8)), (3072, 512, 128, dict(L=45.1, M=36.0)),
    (3072, 512, 192, dict(L=62.6, M=55.0)), (3072, 1024, 64, dict(L=53.8, M=36.0)),
    (4096, 64, 64, dict(G=8.19, M=41.3)), (4096, 256, 64, dict(G=31.9, L=57.1, M=42.1)),
    (4096, 256, 96, dict(L=57.8, M=45.1)), (4096, 256, 192, dict(L=58.2, M=85.5)),
    (4096, 384, 64, dict(G=47.3, L=85.5, M=42.4)), (4096, 512, 64, dict(L=113.8, M=45.1)),
    (4096, 512, 128, dict(L=115.0, M=86.4)), (4096, 512, 192, dict(L=116.7, M=131.2)),
    (4096, 1024, 64, dict(L=226.6, M=86.4)), (4096, 256, 256, dict(L=62.0, M=86.4)),
    (6144, 64, 64, dict(G=30.5, M=68.0)), (6144, 128, 64, dict(G=59.6, M=66.3)),
    (6144, 256, 64, dict(G=117.4, M=111.5)), (6144, 512, 64, dict(G=235.1, M=221.7)),
    (8192, 64, 64, dict(G=67.4, M=146.2)), (8192, 128, 64, dict(G=132.3, M=154.2)),
    (8192, 256, 64, dict(G=262.0, M=260.1)), (8192, 512, 64, dict(G=524.6, M=515.4)),
]
BLINDED = [
    (1024, 512, 192, dict(L=4.72, M=4.27)), (1024, 1024, 64, dict(L=2.48, M=2.84)),
    (2048, 512, 192, dict(L=21.6, M=20.7)), (2048, 1024, 64, dict(L=12.1, M=13.9)),
    (2048, 256, 256, dict(L=11.3, M=13.9)), (3072, 256, 96, dict(L=29.2, M=22.4)),
    (3072, 256, 192, dict(L=34.1, M=42.8)), (3072, 512, 64, dict(L=46.7, M=23.2)),
    (3072, 1024, 64, dict(L=66.7, M=43.8)), (4096, 192, 64, dict(L=74.8, M=50.4, T=44.6)),
    (4096, 256, 64, dict(L=75.2, M=50.6, T=44.8)), (4096, 512, 64, dict(L=149.6, M=57.0)),
    (4096, 256, 192, dict(L=79.5, M=101.2)), (4096, 256, 256, dict(L=85.6, M=107.0)),
    (4096, 1024, 64, dict(L=298.5, M=107.0)),
]
# partial rounds of group blocks, tiles with some of their parts
PARTIAL = [
    (2048, 18, 567, dict(G=5.61, L=4.04, M=5.46)), (2048, 228, 25, dict(G=3.13, L=3.98, M=5.48)),
    (2048, 160, 64, dict(G=4.60, L=3.95, M=5.45)), (2048, 228, 33, dict(G=5.43, L=3.95, M=5.48)),
    (2048, 40, 150, dict(G=3.07, L=3.95, M=5.45)), (3072, 130, 102, dict(G=18.5, L=22.4, M=17.9)),
    (3072, 80, 64, dict(G=7.47, L=13.1, M=17.8)), (3072, 200, 25, dict(G=8.97, L=13.9, M=17.9)),
    (3072, 43, 281, dict(G=14.8, L=14.1)), (4096, 43, 281, dict(G=26.0, L=29.3)),
    (4096, 41, 360, dict(G=32.2, L=29.1)), (4096, 200, 25, dict(G=16.3, L=57.2, M=42.1)),
    (4096, 40, 200, dict(G=19.9, L=29.3, M=41.9)), (6144, 40, 64, dict(G=31.1, M=68.1)),
    (6144, 50, 25, dict(G=16.0, M=68.3)), (8192, 30, 40, dict(G=34.8, M=142.0)),
]

DRIVER = r"""
#include "launch_rule.cpp"
#include <cstdio>
#include <cstdlib>
namespace pmk { uint64_t table_words_per_slot(int, int, int) { return 1; } }
using namespace pmk;
int main(int argc, char **argv) {
    if (argc > 1) {  // keys, chunks per key, tiles of a round, tiles of a group: the cuts
        const unsigned keys = std::atoi(argv[1]), n = keys * std::atoi(argv[2]);
        std::vector<uint32_t> km(n);
        for (unsigned i = 0; i < n; ++i) km[i] = i % keys;
        for (uint64_t c : whole_round_cuts(km.data(), n, keys, std::atoi(argv[3]), std::atoi(argv[4])))
            std::printf("%llu\n", (unsigned long long)c);
        return 0;
    }
    ClassRun r{};
    unsigned blinded;
    r.fill_lanes = 8;
    r.tail_lanes = 1;
    r.fold = std::getenv("NO_FOLD") ? nullptr : (const uint8_t *)&blinded;
    while (std::scanf("%u %d %u %u %u %u %u", &blinded, &r.cls, &r.ntiles, &r.parts, &r.ngroups, &r.group_tiles,
                      &r.grid_cap) == 7) {
        const char *f;
        r.share = blinded == 3 ? 4 : 0;  // four classes side by side
        if (blinded == 3) blinded = 0;
        if (blinded == 2) f = fills_chip(r, 4, 256) ? "alone" : "beside";
        else if (!blinded) f = group_launch(r, 256) ? "G" : mont_launch(r, 256) || !fold_lane(kClassBits[r.cls]).nl ? "M" : "L";
        else f = 2 * r.ntiles <= 512 && joint_two_lanes(r, 256) ? "T" : joint_mont_launch(r, 256) ? "M" : "L";
        std::puts(f);
    }
}
"""


def shape(blinded, bits, keys, chunks, cap=0):
    per = 4 if bits in (3072, 4096) else (2 if bits < 3072 else 4)
    tiles, parts = -(-chunks // 64), -(-chunks // 16)
    groups = -(-tiles // per)
    return f"{blinded} {BITS.index(bits)} {keys * tiles} {keys * parts} {keys * groups} {-(-tiles // groups)} {cap}"


# groups of mixed sizes, the last ones spread over blocks (L): job tiles, parts, groups of
# the shape, ms
MIXED = [(4096, 722, 1240, 140, 4, dict(L=35.5, M=42.7)), (4096, 1044, 1900, 174, 4, dict(L=49.0, M=84.1)),
         (3072, 722, 1240, 140, 4, dict(L=23.9, M=17.9)), (3072, 1044, 1900, 174, 4, dict(L=25.5, M=37.0)),
         (4096, 506, 810, 129, 4, dict(G=31.4, M=42.6)), (3072, 544, 855, 129, 4, dict(G=19.2, L=23.0, M=17.8)),
         (3072, 436, 697, 128, 4, dict(G=15.6, L=14.9, M=18.0))]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("rule")
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", str(d / "driver.cpp"), "-o", exe], check=True)
    return lambda lines, *args: subprocess.run([exe, *map(str, args)], input="\n".join(lines), check=True,
                                               capture_output=True, text=True).stdout.split()


@pytest.mark.parametrize("blinded,rows", [(0, PLAIN), (0, PARTIAL), (1, BLINDED)])
def test_pick_is_near_the_fastest_form(rule, blinded, rows):
    picks = rule([shape(blinded, b, k, c) for b, k, c, _ in rows])
    assert len(picks) == len(rows)
    slow = [(b, k, c, p, ms) for (b, k, c, ms), p in zip(rows, picks) if ms.get(p, 1e9) > 1.06 * min(ms.values())]
    assert not slow


def test_partial_round_over_blocks_counts(rule):
    picks = rule([f"0 {BITS.index(b)} {jt // 2} {parts} {g} {most} 0" for b, jt, parts, g, most, _ in MIXED])
    slow = [(row, p) for row, p in zip(MIXED, picks) if row[5].get(p, 1e9) > 1.06 * min(row[5].values())]
    assert not slow


@pytest.mark.parametrize("bits,keys,chunks,form", [
    # with all four 15.7 ms, 29.6 where the 4096-bit class takes the lane form
    (3072, 36, 71, "G"), (4096, 36, 71, "G"), (4096, 128, 64, "L"), (2048, 128, 64, "L")])
def test_classes_side_by_side(rule, bits, keys, chunks, form):
    assert rule([shape(3, bits, keys, chunks)]) == [form]


@pytest.mark.parametrize("bits,waves", [(1024, 1), (2048, 2), (3072, 4), (4096, 4), (6144, 7), (8192, 8)])
def test_grid_limit_below_a_block(rule, bits, waves):
    """A limit on the resident waves below a group block's waves leaves one-wave blocks."""
    caps = range(1, waves + 2)
    picks = rule([shape(0, bits, 4, 16, cap) for cap in caps])
    assert [p == "G" for p in picks] == [cap >= waves for cap in caps]


@pytest.mark.parametrize("bits,keys,chunks,where", [
    # 200 group blocks of one or two waves leave room beside them on 1,024 SIMDs, 800 do not
    (1024, 100, 16, "beside"), (2048, 112, 16, "beside"), (1024, 100, 64, "alone"), (1024, 406, 64, "alone"), (2048, 406, 64, "alone"), (3072, 406, 64, "alone"), (4096, 406, 64, "alone"),
    (4096, 64, 64, "alone")])
def test_classes_that_fill_the_chip(rule, bits, keys, chunks, where):
    assert rule([shape(2, bits, keys, chunks)]) == [where]


@pytest.mark.parametrize("keys,chunks,round_,group,cuts", [
    (256, 256, 512, 4, []),               # a cut after two tiles of each key would split its group of four
    (256, 512, 512, 4, [256 * 256]),      # 1,024 tiles in whole groups
    (256, 26 * 64, 1024, 2, [256 * 256, 256 * 256 * 3]),
    (64, 256, 16, 1, [64 * 64, 64 * 64 * 3])])
def test_slices_keep_whole_groups(rule, keys, chunks, round_, group, cuts):
    assert [int(x) for x in rule([], keys, chunks, round_, group)] == cuts


@pytest.mark.parametrize("bits", [1024, 2048, 3072, 4096, 6144, 8192])
@pytest.mark.parametrize("keys,chunks", [(1, 7), (64, 64), (256, 256)])
def test_without_fold_tables(rule, monkeypatch, bits, keys, chunks):
    monkeypatch.setenv("NO_FOLD", "1")
    assert rule([shape(0, bits, keys, chunks)]) == ["M"]
    if bits <= 4096:
        assert rule([shape(1, bits, keys, chunks)]) in (["M"], ["T"])
