"""Sampled particles through the hash table: its home slots on the host at the
largest sizes, its results on the GPU in every form.

Bar on the host: with at most one entry in eight taken, linear probing from
evenly spread home slots looks at 1 + (1 / (1 - 1/8)^2 - 1) / 2 = 1.16 entries
for an insertion (Knuth, The Art of Computer Programming 3, 6.4); 1.5 allows
for the spread of a hash that is not random.
"""
import os
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "sample_table.h"
// inserts m keys of the given stride; prints the table's size, 4-byte words
// and the mean number of entries looked at (gives up beyond 16 a key)
int main(int argc, char** argv) {
  const uint64_t np = strtoull(argv[1], 0, 10), m = strtoull(argv[2], 0, 10),
                 stride = strtoull(argv[3], 0, 10);
  const uint32_t mask = mpc::sample_table_mask(m, np);
  if (!mask) {
    std::printf("0 0 0\n");
    return 0;
  }
  std::vector<bool> taken((size_t)mask + 1);
  uint64_t probes = 0;
  for (uint64_t k = 0; k < m && probes < 16 * m; ++k) {
    uint32_t h = mpc::sample_hash((uint32_t)(k * stride), mask);
    for (++probes; taken[h] && probes < 16 * m; ++probes) h = (h + 1) & mask;
    taken[h] = true;
  }
  std::printf("%llu %llu %.4f\n", (unsigned long long)mask + 1, 2ull * ((unsigned long long)mask + 1),
              (double)probes / (double)m);
  return 0;
}
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    d = tmp_path_factory.mktemp("table")
    src, exe = str(d / "t.cpp"), str(d / "t")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2406_15236_amd", "csrc"),
                    src, "-o", exe], check=True)

    def run(np_, m, stride):
        out = subprocess.run([exe, str(np_), str(m), str(stride)], check=True, capture_output=True,
                             text=True, timeout=300).stdout.split()
        return int(out[0]), int(out[1]), float(out[2])
    return run


@pytest.mark.parametrize("np_,m,stride", [
    (2**31 - 1, 2**26 - 1, 32),     # the largest table: more samples than 2^25
    (566_231_040, 17_694_720, 32),  # every 32nd particle of 384^3 at 10 per cell
    (2**31 - 1, 2**20, 1), (2**31 - 1, 2**20, 2048), (2**31 - 1, 2**15, 2**16),
    (10**6, 1000, 1000), (100, 1, 1), (64, 2, 31)])
def test_home_slots_are_spread(table, np_, m, stride):
    size, words, probes = table(np_, m, stride)
    assert 8 * m <= size < 16 * m or size == 8
    assert 4 * words <= 4 * np_           # no more memory than the inverse array
    assert probes < 1.5


@pytest.mark.parametrize("np_,m", [(31, 1), (10_800, 338), (566_231_040, 566_231_040 // 16)])
def test_larger_samples_use_the_inverse(table, np_, m):
    assert table(np_, m, 1)[0] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["fp64", "fp32", "split"])
def test_sampled_states_through_the_table(form):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_15236_amd as mpc
    boxes = [dict(synth.config("C1"), L=(20, 18, 17), mbs=True, seed=3),
             dict(synth.config("C1"), L=(16, 11, 9), mbs=True, seed=4)]
    states = [synth.box_state(b["L"], seed=7) for b in boxes]
    rng = np.random.default_rng(11)
    print(f"case table {form}", flush=True)
    with mpc.Sim(boxes, form=form, reorder_every=2) as sim:
        for k, (x, v) in enumerate(states):
            sim.set_state(x, v, k)
        sim.step(3)
        for k in range(2):
            xg, vg = sim.get_state(k)
            n = xg.shape[1]
            for idx in (rng.integers(0, n, size=n // 32), np.full(n // 32, n - 1),
                        np.arange(0, n, 32)[:n // 32], np.array([0]), np.array([5, 5, n - 1])):
                xs, vs = sim.get_particles(idx, k)
                np.testing.assert_array_equal(xs, xg[:, idx])
                np.testing.assert_array_equal(vs, vg[:, idx])
