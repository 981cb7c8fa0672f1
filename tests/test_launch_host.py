"""The host arithmetic of the launches (csrc/flashoptim_launch.h), compiled into a small program: table sizes at their
limits and the cutting of work into launches, without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def _run(tmp_path, body):
    """Compiles `body` as main()'s statements behind the header and returns the lines that it prints."""
    src, exe = tmp_path / "launch.cpp", tmp_path / "launch"
    src.write_text('#include <cstdio>\n#include "flashoptim_launch.h"\nint main() {\n' + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-O1", "-I",
                    os.path.join(ROOT, "paper_2602_23349_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()


def test_coarse_tables_never_exceed_their_entries(tmp_path):
    # the step without allocation writes the table into a fixed array of 16384 entries: totals just above
    # 16384 * 2^k, where total >> k is 16384 but the last, partial entry makes one more
    totals = sorted({t for k in range(18) for d in range(-3, 5) if 0 < (t := (16384 << k) + d) <= 0x7fffffff} | {1, 2, 3, 0x7fffffff})
    out = _run(tmp_path, "const long long totals[] = {" + ", ".join(f"{t}LL" for t in totals) + "};\n"
               "for (long long t : totals) std::printf(\"%lld %u %lld\\n\", t, fo::coarse_shift(t), "
               "(long long)fo::coarse_entries(t, fo::coarse_shift(t)));")
    assert len(out) == len(totals)
    for line, total in zip(out, totals):
        t, shift, entries = (int(x) for x in line.split())
        assert t == total and entries <= 16384, line
        assert (entries - 1) << shift < total <= entries << shift, line          # every workgroup has its entry
        assert shift == 0 or -(-total // (1 << (shift - 1))) > 16384, line        # no coarser than needed


@pytest.mark.parametrize("threads", [64, 256, 512, 1024])
def test_launches_stay_below_the_work_item_limit_and_cover_every_workgroup(tmp_path, threads):
    # the checkpoint copy (1024 lanes per 16 KB piece, the header's workgroup behind the last one) reaches the limit of
    # one launch, 2^32 - 1 work-items, at 64 GiB: 2^22 - 1 pieces fit, with the header's workgroup 2^22 - 2
    most = (2**32 - 1) // threads
    totals = [0, 1, most - 1, most, most + 1, most + 2, 2 * most, 2 * most + 1, 5 * most + 7]
    out = _run(tmp_path, "const long long totals[] = {" + ", ".join(f"{t}LL" for t in totals) + "};\n"
               "for (long long t : totals) {\n"
               f"    for (long long first = 0, n; first < t; first += n) {{ n = fo::launch_span(t, first, {threads}); "
               "std::printf(\"%lld %lld \", first, n); }\n    std::printf(\"\\n\");\n}")
    assert len(out) == len(totals)
    for line, total in zip(out, totals):
        spans = [int(x) for x in line.split()]
        first, n = spans[::2], spans[1::2]
        assert all(0 < k and k * threads < 2**32 for k in n), line
        assert len(n) == -(-total // most) and sum(n) == total and first == [sum(n[:i]) for i in range(len(n))], line


def test_every_copy_runs_as_its_own_check_decided(tmp_path):
    # five unpacks with one word, admitted or refused in every combination, the copies of admitted ones held back by their
    # streams for as long as one likes: every order in which checks and copies can run
    out = _run(tmp_path, """
    long long orders = 0, wrong = 0;
    auto go = [&](auto& self, unsigned admitted, int next, unsigned pending, uint64_t word) -> void {
        if (next == 5 && !pending) { ++orders; return; }
        for (int k = 0; k < next; ++k)
            if (pending >> k & 1) {
                wrong += fo::verdict_admits(word, k + 1) != (bool)(admitted >> k & 1);
                self(self, admitted, next, pending & ~(1u << k), word);
            }
        if (next < 5 && !(pending & ~admitted))
            self(self, admitted, next + 1, pending | 1u << next, fo::verdict_word(next + 1, admitted >> next & 1));
    };
    const uint64_t before[] = {0, ~(uint64_t)0};
    for (uint64_t first : before)
        for (unsigned admitted = 0; admitted < 32; ++admitted) go(go, admitted, 0, 0, first);
    std::printf("%lld %lld\\n", orders, wrong);
    """)
    orders, wrong = (int(x) for x in out[0].split())
    assert orders > 5000 and wrong == 0


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="needs the HIP headers")
def test_one_generation_of_workgroups_is_not_held_back(tmp_path):
    # 256 compute units with eight workgroups of 256 lanes each: 2048 of them, or 2^22 elements (k_proj and v_proj of a Llama layer)
    src, exe = tmp_path / "resident.cpp", tmp_path / "resident"
    src.write_text("""#include <cstdio>
#include "flashoptim_device.h"
int main() {
    for (int kind = 0; kind < 3; ++kind)
        for (bool direct : {false, true})
            for (long long blocks : {1, 2047, 2048, 2049, 100000}) {
                const long long elems = blocks * fo::chunk_elems(true, true, fo::StepShape::kUsual);
                std::printf("%lld %d\\n", blocks, fo::step_resident(kind, true, true, fo::StepShape::kUsual, direct, elems, false));
            }
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2602_23349_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) == 30
    for line in lines:
        blocks, resident = (int(x) for x in line.split())
        assert resident == 0 if blocks <= 2048 else resident in (6, 7), line


def test_look_up_finds_every_workgroup_in_few_steps(tmp_path):
    # lists of many small entries beside large ones, and every shift that their coarse tables could have
    out = _run(tmp_path, """
    const int n = 3000;
    static uint32_t begin[n + 1], size[n], coarse[70000];
    uint32_t seed = 1, wrong = 0, over = 0, looked = 0;
    for (int list = 0; list < 6; ++list) {
        for (int i = 0; i < n; ++i) {
            seed = seed * 1664525u + 1013904223u;
            size[i] = list == 0 ? 1 : list == 1 ? (i == n - 1 ? 60000 : 1) : list == 2 ? (i ? 1 : 60000) : list == 3 ? 1 + (seed >> 28) :
                      list == 4 ? (i % 1000 == 500 ? 5000 : 1 + (seed >> 31)) : 1 + (i & 1) * 9;
        }
        begin[0] = 0;
        for (int i = 0; i < n; ++i) begin[i + 1] = begin[i] + size[i];
        const uint32_t total = begin[n];
        for (uint32_t shift = 0; shift < 18; ++shift) {
            const uint32_t entries = (uint32_t)fo::coarse_entries(total, shift);
            for (uint32_t j = 0, t = 0; j < entries; ++j) {
                while (begin[t + 1] <= j << shift) ++t;
                coarse[j] = t;
            }
            coarse[entries] = n - 1;
            uint32_t most = 0;                               // halvings of a whole entry
            while ((1u << most) <= (shift < 12 ? 1u << shift : (uint32_t)n)) ++most;
            for (uint32_t b = 0, t = 0; b < total; ++b) {
                uint32_t reads = 0;
                while (begin[t + 1] <= b) ++t;
                const uint32_t got = fo::entry_of(b, coarse[b >> shift], coarse[(b >> shift) + 1], [&](uint32_t i) { ++reads; return begin[i]; });
                wrong += got != t;
                over += reads > most;
                ++looked;
            }
        }
    }
    std::printf("%u %u %u\\n", looked, wrong, over);
    """)
    looked, wrong, over = (int(x) for x in out[0].split())
    assert looked > 1000000 and wrong == 0 and over == 0


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="needs the HIP headers")
def test_conversions_of_every_accepted_size_have_tiles_enough(tmp_path):
    # a tensor may have up to 2^40 - 1 elements, and a launch's tiles are numbered with 31 bits
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text("""#include <cstdio>
#include "flashoptim_device.h"
int main() {
    for (int k = 0; k <= 40; ++k)
        for (long long d : {-1, 0, 1}) {
            const long long n = (1LL << k) + d;
            if (n < 1 || n >= 1LL << 40) continue;
            for (bool compress : {false, true}) {
                const long long tile = fo::convert_chunk(compress, fo::convert_through(n));
                std::printf("%lld %lld\\n", n, (n + tile - 1) / tile);
            }
        }
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2602_23349_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) > 200 and int(lines[-1].split()[0]) == 2**40 - 1
    assert all(int(line.split()[1]) <= 0x7fffffff for line in lines)


@pytest.mark.parametrize("waves", [1, 2, 4, 8, 16])
def test_dealt_out_tiles_cover_every_part_once(tmp_path, waves):
    # tensors of 0 to 200 whole tiles, with and without a ragged one behind them: the parts of the whole tiles are all dealt out once,
    # the ragged tile and those of the last, incomplete group keep theirs
    out = _run(tmp_path, f"""
    const int waves = {waves};
    long long wrong = 0, spread = 0;
    for (int full = 0; full <= 200; ++full)
        for (int ragged = 0; ragged < 2; ++ragged) {{
            static int seen[201 * 16];
            for (int i = 0; i < (full + ragged) * waves; ++i) seen[i] = 0;
            for (int t = 0; t < full + ragged; ++t)
                for (int w = 0; w < waves; ++w) {{
                    const long long p = fo::wave_part(t, w, waves, full);
                    if (p < 0 || p >= (full + ragged) * waves) {{ ++wrong; continue; }}
                    ++seen[p];
                    if (t >= full - full % fo::kTileGroup) wrong += p != (long long)t * waves + w;
                    else if (w > 0) spread += p - fo::wave_part(t, w - 1, waves, full) == fo::kTileGroup;
                }}
            for (int i = 0; i < (full + ragged) * waves; ++i) wrong += seen[i] != 1;
        }}
    std::printf("%lld %lld\\n", wrong, spread);
    """)
    wrong, spread = (int(x) for x in out[0].split())
    assert wrong == 0 and (spread > 0) == (waves > 1)


def test_a_pair_of_sums_is_read_only_when_all_of_it_is_there(tmp_path):
    # the four words of a pair written in any order over those of any earlier call, read in between
    out = _run(tmp_path, """
    const uint64_t sums[] = {0, ~0ull, 0x3ff0000000000000ull, 0x00000001ffffffffull, 0xfedcba9876543210ull};
    const uint32_t tickets[] = {0, 1, 4, 6, 0xffffffff};
    long long wrong = 0, ready = 0;
    for (uint64_t a : sums)
        for (uint64_t b : sums)
            for (uint32_t before : tickets)
                for (unsigned written = 0; written < 16; ++written) {
                    uint64_t w[fo::kNmseWords];
                    for (int k = 0; k < 4; ++k) {
                        const uint64_t sum = k < 2 ? a : b, old = k < 2 ? b : a;
                        w[k] = written >> k & 1 ? fo::nmse_word((uint32_t)(k & 1 ? sum >> 32 : sum), 5)
                                                : fo::nmse_word((uint32_t)(k & 1 ? old >> 32 : old), before);
                    }
                    const bool all = fo::nmse_ready(w, 5);
                    wrong += all != (written == 15);
                    if (all) wrong += fo::nmse_sum(w, 0) != a || fo::nmse_sum(w, 1) != b;
                    ready += all;
                }
    std::printf("%lld %lld\\n", wrong, ready);
    """)
    wrong, ready = (int(x) for x in out[0].split())
    assert wrong == 0 and ready == 125


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="needs the HIP headers")
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("split,quant", [(1, 1), (1, 0), (0, 1), (0, 0)])
def test_every_part_of_a_list_is_handled_once_whatever_launch_it_is_in(tmp_path, kind, split, quant):
    # tensors of 0 to 31 tiles and a remainder ahead of a large one, so that its groups of tiles lie across the cut at 2^28 elements; the
    # last launch a few tiles, just below, at and above the size from which stores go through, or nearly whole; a third launch
    src, exe = tmp_path / "parts.cpp", tmp_path / "parts"
    src.write_text("""#include <cstdio>
#include <vector>
#include "flashoptim_device.h"
int main() {
    const int kind = %d;
    const bool split = %d, quant = %d;
    const long long limit = (fo::kThroughBytes + fo::step_array_bytes(kind, split, quant) - 1) / fo::step_array_bytes(kind, split, quant);
    long long launches = 0, wrong = 0, across = 0;
    for (long long ahead : {1LL, 4096LL, 17 * 4096LL + 1, 31 * 4096LL, 70000LL})
        for (long long behind : {1000LL, 200000LL, limit - 8192, limit, limit + 8192, (1LL << 28) - 100000, (1LL << 28) + 50000}) {
            const std::vector<long long> numel = {ahead, (1LL << 28) + behind - ahead - 77, 77};
            const fo::StepShape shape = fo::step_shape(kind, split, quant, (1LL << 28) + behind);
            const int tile_elems = fo::chunk_elems(split, quant, shape), waves = fo::step_threads(split, quant, shape) / 64;
            std::vector<std::vector<unsigned char>> seen;
            std::vector<long long> first_tile;
            long long tiles = 0;
            for (long long n : numel) {
                const long long k = (n + tile_elems - 1) / tile_elems;
                first_tile.push_back(tiles);
                seen.emplace_back(k * waves, 0);
                tiles += k;
            }
            const hipError_t e = fo::for_each_step_segment(kind, split, quant, tiles, tile_elems, [&](int64_t first, int64_t n, bool through) {
                ++launches;
                size_t t = 0;
                for (int64_t b = first; b < first + n; ++b) {
                    while (t + 1 < numel.size() && first_tile[t + 1] <= b) ++t;
                    const long long tile = b - first_tile[t], full = numel[t] / tile_elems;
                    across += b == first && first > 0 && tile %% fo::kTileGroup != 0;
                    for (int w = 0; w < waves; ++w) {
                        const long long part = fo::step_dealt(kind, split, quant, through) ? fo::wave_part(tile, w, waves, full) : tile * waves + w;
                        if (part < 0 || part >= (long long)seen[t].size()) ++wrong; else ++seen[t][part];
                    }
                }
                return hipSuccess;
            });
            wrong += e != hipSuccess;
            for (const auto& s : seen) for (unsigned char c : s) wrong += c != 1;
        }
    std::printf("%%lld %%lld %%lld\\n", launches, across, wrong);
}
""" % (kind, split, quant))
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2602_23349_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    launches, across, wrong = (int(x) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert launches == 5 * (6 * 2 + 3) and across > launches // 4 and wrong == 0


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="needs the HIP headers")
def test_which_steps_deal_their_tiles_out(tmp_path):
    # AdamW with quantised states, bound by power, is slower that way; a single wavefront has nothing to deal out
    src, exe = tmp_path / "dealt.cpp", tmp_path / "dealt"
    src.write_text("""#include <cstdio>
#include "flashoptim_device.h"
int main() {
    for (int kind = 0; kind < 3; ++kind)
        for (int k = 0; k < 4; ++k)
            if (fo::step_dealt(kind, k & 1, k & 2, true)) std::printf("%d%s%s ", kind, k & 1 ? "s" : "", k & 2 ? "q" : "");
    for (int kind = 0; kind < 3; ++kind)
        for (int k = 0; k < 4; ++k) if (fo::step_dealt(kind, k & 1, k & 2, false)) return 1;
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2602_23349_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    assert out.split() == ["0s", "1s", "1q", "1sq", "2s", "2q", "2sq"]


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="needs the HIP headers")
def test_long_tables_are_not_read_by_every_workgroup_of_a_copy(tmp_path):
    # a header of 64 bytes and 16 for each tensor, in units of 64: 252 tensors are 4096 bytes
    src, exe = tmp_path / "checked.cpp", tmp_path / "checked"
    src.write_text("""#include <cstdio>
#include "flashoptim_device.h"
int main() {
    for (long long n : {1, 252, 253, 1020})
        for (long long mb : {23, 24, 256, 257}) std::printf("%d", fo::checked_copy(mb << 20, 64 + (16 * n + 63) / 64 * 64));
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2602_23349_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout == "0110" "0110" "0000" "0000"
