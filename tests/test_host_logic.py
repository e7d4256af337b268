"""Host-side logic of the package that needs no GPU: warm-start features,
histogram sizing, the benchmark's kernel-source key, and the stored oracle
references against the generator."""
from __future__ import annotations

import importlib.util
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_geometric_features_and_voxel_classes():
    from paper_2304_14568_amd import warmstart as W
    P = synth.hn_small(3)
    X = W.geometric_features(P)
    assert X.shape == (P.n, W.GEOM_FEATURES) and np.all(np.isfinite(X))
    assert np.all((X[:, 0] >= 0) & (X[:, 0] <= 1))          # layer position within its beam
    assert np.allclose(X[:, 5:8].sum(axis=1), 1.0)           # beam one-hot
    assert np.allclose(X[:, 4], np.hypot(X[:, 2], X[:, 3]), atol=1e-6)
    vc = W.voxel_class(P)
    names = P.meta["struct_names"]
    for g, nm in enumerate(names):
        sel = np.asarray(P.struct_id) == g
        want = 1 if nm.startswith("target") else 2 if nm.startswith("oar") else 0
        assert np.all(vc[sel] == want)


def test_histogram_size_fits_lds():
    from paper_2304_14568_amd.clinical import max_bins
    for G in (1, 7, 64, 256):
        nb = max_bins(G)
        assert 12 * G + 4 * G * nb <= 65536 < 12 * G + 4 * G * (nb + 1)


def test_bench_kernel_source_key():
    spec = importlib.util.spec_from_file_location("bench_mod", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    src = os.path.join(ROOT, "paper_2304_14568_amd", "csrc", "factor.hip")
    key = bench.kernel_source_hash(src, "__global__ __launch_bounds__(256) void k_xsym(")
    assert len(key) == 16
    assert bench.kernel_source_hash(src, "no such kernel(") == ""


def _run_cpp(tmp_path, body):
    """Compile and run a program over the library's host-only headers."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cassert>\n#include <cstdio>\n#include "progress.h"\nusing namespace admmbb;\n' + body)
    csrc = os.path.join(ROOT, "paper_2304_14568_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", csrc, str(src), "-o", str(exe)],
                   check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


def test_head_count_starts_from_the_reported_words(tmp_path):
    """A run that fails after one of its heads was queued: the device has had one
    more than the host finished counting.  The next run counts from the words
    it finds, so a word that the failed run left, stop bit included, never passes
    for a head of the next one; nor does the wrap of the 31-bit count."""
    _run_cpp(tmp_path, """
int main() {
  for (uint32_t had : {0u, 7u, 0x7ffffffdu, 0x7fffffffu}) {
    uint32_t words[2] = {had << 1, (had + 3) << 1};
    HeadCount h;
    h.begin(words, 2);
    assert(!h.reached(words[0], 0, 1) && !h.reached(words[1], 1, 1));
    // the first iteration's head runs and stops patient 0; its launch then throws
    words[0] = (had + 1) << 1 | 1;
    words[1] = (had + 4) << 1;
    assert(h.reached(words[0], 0, 1) && h.reached(words[1], 1, 1) && !h.reached(words[0], 0, 2));
    HeadCount next;
    next.begin(words, 2);
    assert(!next.reached(words[0], 0, 1) && !next.reached(words[1], 1, 1));
    for (uint32_t k = 1; k <= 5; ++k) {
      const uint32_t w = (had + 1 + k) << 1;
      assert(next.reached(w, 0, k) && next.reached(w, 0, 1) && !next.reached(w, 0, k + 1));
    }
  }
}
""")


def test_host_waits_as_the_process_asked(tmp_path):
    """A report that comes after 200 ms: asleep the wait takes a few per cent of a
    core, by spinning all of it; and a stream that runs dry without the report
    ends the wait in every form."""
    out = _run_cpp(tmp_path, """
#include <atomic>
#include <ctime>
static double cpu() {
  timespec t;
  clock_gettime(CLOCK_THREAD_CPUTIME_ID, &t);
  return t.tv_sec + 1e-9 * t.tv_nsec;
}
int main() {
  for (HostWait how : {HostWait::sleep, HostWait::yield, HostWait::spin}) {
    std::atomic<int> word{0};
    std::thread dev([&] {
      std::this_thread::sleep_for(std::chrono::milliseconds(200));
      word = 1;
    });
    const double c0 = cpu();
    assert(wait_report(how, [&] { return word.load() != 0; }, [] { return false; }));
    printf("%.4f\\n", cpu() - c0);
    dev.join();
    int looks = 0;
    assert(!wait_report(how, [] { return false; }, [&] { return ++looks == 3; }));
    assert(wait_report(how, [&] { return looks > 3; }, [&] { return ++looks > 3; }));  // there when the stream is dry
  }
}
""")
    asleep, _, spinning = [float(v) for v in out.split()]
    assert asleep < 0.04 and spinning > 2 * asleep


@pytest.mark.slow
def test_stored_references_match_the_generator():
    """Every stored oracle minimum of the scenario-count study still describes
    the instance the generator produces (content digest)."""
    from tests.golden.refs import load
    P = synth.hn_full(0)
    for N in (1, 5, 12):
        rec, x = load(f"hn_full_s0_n{N}")
        assert rec is not None and rec["digest"] == P.subset(list(range(N))).digest()
        assert rec["kkt"] <= 1e-12 and x.shape == (P.n,)
    rec, _ = load("hn_full_s0")
    assert rec["digest"] == P.digest()
    # more scenarios, larger minimum
    fs = [load(f"hn_full_s0_n{N}")[0]["f_star"] for N in range(1, 13)] + [rec["f_star"]]
    assert all(a < b for a, b in zip(fs, fs[1:]))


def test_packed_tile_number_to_its_blocks():
    """The dense PGD finds the blocks (I, J), I <= J, of packed tile number t from a
    float32 square root and a correction by whole rows (t(I, I) = I nb - I (I - 1)
    / 2, J = I + t - t(I, I)): the root is within one of the row for every tile of
    up to 128 blocks, so the correction takes at most one step."""
    f = np.float32
    for nb in range(1, 129):
        first = np.array([i * nb - i * (i - 1) // 2 for i in range(nb)])
        t = np.arange(nb * (nb + 1) // 2)
        b = f(2 * nb + 1)
        root = (f(0.5) * (b - np.sqrt(np.maximum(b * b - f(8) * t.astype(f), f(0))))).astype(np.int32)
        row = np.searchsorted(first, t, side="right") - 1
        assert np.all(np.abs(np.clip(root, 0, nb - 1) - row) <= 1)
