"""Which steps of a call run one by one because they share buffers (host code, CPU only): the sweep over sorted spans against all
pairs, and the time of a call with many steps."""
import ctypes as C
import os
import subprocess
import time

from paper_2509_19836_amd import build

PROGRAM = r"""
#include <cstdio>
#include <random>
#include "spans.hpp"
using namespace burst;
int main() {
  std::mt19937 rng(7);
  int apart = 0;
  const int cases = 200000;
  for (int c = 0; c < cases; ++c) {
    const int steps = 2 + rng() % 4, range = 20 << rng() % 5;
    std::vector<Use> uses;
    for (int s = -1; s < steps; ++s)
      for (int t = 0; t < (s < 0 ? 1 : 4); ++t) {
        const uintptr_t begin = rng() % range, length = rng() % 8;
        uses.push_back(Use{Span{begin, begin + length}, s, s < 0 || t < 2});
      }
    bool pairs = true;
    for (const Use& a : uses)
      for (const Use& b : uses)
        if (a.step != b.step && a.written && a.span.begin != a.span.end && b.span.begin != b.span.end && overlap(a.span, b.span)) pairs = false;
    if (steps_apart(uses) != pairs) return printf("case %d differs\n", c), 1;
    apart += pairs;
  }
  return apart < cases / 20 || apart > cases - cases / 20;   // both answers occur
}
"""


def test_the_sweep_finds_what_all_pairs_find(tmp_path):
    src, exe = tmp_path / "spans.cpp", tmp_path / "spans"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True, timeout=60)


def test_the_checks_of_a_call_grow_with_its_steps_and_not_with_their_pairs(lib):
    """The whole call up to its first launch, which may fail here, on addresses that belong to nothing: steps that share one buffer
    with nobody.  16 times the steps take 25 times as long (37 on a busy machine); all pairs took 200."""
    if os.path.exists("/dev/kfd"):
        import pytest
        pytest.skip("on a machine with a GPU the call would launch")
    raw, ref, d = lib.raw(), C.byref, 64
    good, f32 = (lib.burst_tensor_t(4096, t, 0, 64 * 2 * d, 2 * d, d) for t in (lib.BURST_BF16, lib.BURST_F32))
    vec = lib.burst_rowvec_t(4096, 128, 64)

    def call(n):
        shapes = bytes((lib.burst_shape_t * n)(*[lib.shape(1, 2, 2, d, 64, 64, 0.125)] * n))
        masks = (lib.burst_mask_t * n)(*[lib.burst_attn_fill_contiguous_mask(0, 0, 1, 64, False)] * n)
        array = lambda base, dt: bytes((lib.burst_tensor_t * n)(*[lib.burst_tensor_t((base << 32) + (i << 16), dt, 0, 64 * 2 * d, 2 * d, d)
                                                                  for i in range(n)]))
        k, v, dk, dv = (array(1 + i, lib.BURST_F32 if i > 1 else lib.BURST_BF16) for i in range(4))
        best = 1e9
        for _ in range(5):
            t0 = time.perf_counter()
            raw.burst_attn_steps_bwd(n, shapes, masks, ref(good), k, v, ref(good), ref(vec), ref(vec), ref(f32), dk, dv, 7, None)
            best = min(best, time.perf_counter() - t0)
        return best

    call(2)
    assert call(1024) <= 100 * call(64)
