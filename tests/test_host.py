"""Host-only checks: the seeded generators follow their recipe, and the
benchmark refuses more than one GPU."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2101_05031_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("n", [1, 2, 5, 25, 40, 52])
def test_kuhn_edge_count_and_uniqueness(n):
    e = synth.kuhn_edges(n)
    assert len(e) == synth.kuhn_edge_count(n)
    key = np.minimum(e[:, 0], e[:, 1]).astype(np.int64) * (n + 1) ** 3 + np.maximum(e[:, 0], e[:, 1])
    assert len(np.unique(key)) == len(e)


def test_kuhn_tets_are_covered():
    """Every tet of the Kuhn split (a path of +x, +y, +z steps through a cube)
    has its 6 edges in the edge set."""
    import itertools
    n = 2
    e = synth.kuhn_edges(n)
    s = {tuple(sorted(x)) for x in e.tolist()}
    idx = lambda i, j, k: (i * (n + 1) + j) * (n + 1) + k
    for perm in itertools.permutations(range(3)):
        v = [0, 0, 0]
        verts = [idx(*v)]
        for ax in perm:
            v[ax] += 1
            verts.append(idx(*v))
        for a, b in itertools.combinations(verts, 2):
            assert tuple(sorted((a, b))) in s


def test_bcc_counts():
    lat = synth.bcc_lattice(4, 5.0, 0.5)
    assert lat.n_nodes == 189 and lat.n_edges == 812
    L = np.linalg.norm(lat.nodes[lat.edges[:, 0]] - lat.nodes[lat.edges[:, 1]], axis=1)
    assert np.allclose(np.sort(np.unique(np.round(L, 9))), [5.0 * np.sqrt(3) / 2, 5.0])


def test_configs_are_seeded_and_shaped():
    lat, grid = synth.config("D4")
    lat2, _ = synth.config("D4")
    assert np.array_equal(lat.nodes, lat2.nodes) and np.array_equal(lat.weight, lat2.weight)
    assert lat.n_edges == 115075 and lat.nodes.dtype == np.float32
    assert grid.W == grid.H == 1024 and grid.n_slices == 64
    assert lat.R == pytest.approx(1.5)
    r = lat.radius
    assert r.min() >= 0.2 + 0.8 * 0.15 - 1e-6 and r.max() <= 1.0 + 1e-6
    # grid covers the bounding box grown by R with margin
    assert grid.x0 < lat.nodes[:, 0].min() - lat.R
    assert grid.x0 + grid.W * grid.dx > lat.nodes[:, 0].max() + lat.R


def test_blob_config_has_voids():
    lat, _ = synth.config("B3", scale=12)
    assert (lat.weight == 0).any() and (lat.weight > 0).any()
    assert lat.R == pytest.approx(0.9)


def test_weight_for_radius_rejects_out_of_range():
    with pytest.raises(ValueError):
        synth.weight_for_radius(1.5, 1.5)
    w = synth.weight_for_radius(np.array([0.2, 0.5, 0.9]), 1.5)
    assert np.all(np.diff(w) > 0)       # larger radius needs a larger weight


def test_bench_refuses_several_gpus():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in json.loads(r.stdout.strip().splitlines()[-1])["error"]


def test_launches_cover_a_grid(tmp_path):
    """csrc/grid.hpp: the launches of a grid cover its blocks once, in order,
    each within 2^32 threads."""
    src = tmp_path / "grid.cpp"
    src.write_text("""
        #include "grid.hpp"
        #include <cstdio>
        #include <initializer_list>
        int main() {
            for (uint32_t threads : {64u, 256u, 1024u})
                for (uint64_t n : {0ull, 1ull, 1000ull, (1ull << 31) / threads - 1,
                                   (1ull << 31) / threads, (1ull << 31) / threads + 1,
                                   (1ull << 32) / threads, 5 * ((1ull << 32) / threads) + 7}) {
                    uint64_t at = 0, calls = 0;
                    bool ok = true;
                    lsl::for_launches(n, threads, [&](uint64_t b0, uint32_t blocks) {
                        ok = ok && b0 == at && blocks > 0 &&
                             (uint64_t)blocks * threads <= 0xffffffffull;
                        at += blocks;
                        ++calls;
                    });
                    if (!ok || at != n || calls != lsl::launch_count(n, threads)) {
                        std::printf("%u threads, %llu blocks\\n", threads, (unsigned long long)n);
                        return 1;
                    }
                }
            return 0;
        }
    """)
    run_cpp(src)


def run_cpp(src):
    """Compiles and runs a C++ program that includes the library's host headers."""
    exe = src.with_suffix("")
    subprocess.run(["g++", "-O3", "-march=native", "-std=c++17", "-I",
                    os.path.join(ROOT, "paper_2101_05031_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_splitters_are_few_and_close(tmp_path):
    """csrc/splitters.hpp: the picks never outnumber their share of the scratch
    (all prefixes up to 2^30 segments), and along any constant stride of up to
    2^17 segments per row the walk between two picks stays short (a wave walks as
    long as its longest lane).  400 steps without a pick have a probability of
    (15/16)^400 = 6e-12 under the mixed half alone; 2^28 steps are looked at."""
    src = tmp_path / "split.cpp"
    src.write_text("""
        #include "splitters.hpp"
        #include <cstdio>
        int main() {
            int64_t count = 0, most = 0;
            for (uint32_t t = 0; t < (1u << 30); t += 4096) {      // the excess over t / 8
                uint32_t c = 0;
                for (uint32_t s = t; s < t + 4096; ++s) c += lsl::split_pick(s);
                // (within a block of 4096 the count grows by at most all of it)
                if (count + c - (int64_t)t / 8 > 64)
                    for (uint32_t s = t; s < t + 4096; ++s) {
                        count += lsl::split_pick(s);
                        most = std::max(most, count - (int64_t)(s + 1) / 8);
                    }
                else
                    count += c;
            }
            std::printf("excess %lld\\n", (long long)most);
            if (most > 64) return 1;
            uint32_t longest = 0, at = 0;
            for (uint32_t m = 1; m <= (1u << 17); ++m) {
                uint32_t s = 12345u + 7919u * m, last = 0;
                for (uint32_t k = 1; k <= 2048; ++k, s += m)
                    if (lsl::split_pick(s) || k == 2048) {
                        if (k - last > longest) longest = k - last, at = m;
                        last = k;
                    }
            }
            std::printf("longest walk %u, stride %u\\n", longest, at);
            return longest > 400;
        }
    """)
    run_cpp(src)
