"""Batches of more than 128 requests, on the CPU: every group of 128 has the kernel, the cut and so the output bits that it has in
a call of its own, also where two groups share a launch."""
import os
import subprocess

import numpy as np
import pytest

import paper_2506_15155_amd as E

DUMMY = 0x1000
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def plans(lens, n_kv, group, dim, tokens=64):
    """(kernel, cut) of the whole batch, and of each of its groups of 128 in a call of its own."""
    need = [-(-n // tokens) for n in lens]
    cb = tokens * 4 * n_kv * dim
    P = E.ellm_pool_create(None, None, cb, n_kv * group, n_kv, dim, len(lens), max(need), flags=1, device_bytes=(sum(need) + 1) * cb)
    ids = [E.ellm_tensor_create(P, s * tokens) for s in need]
    for t, s in zip(ids, need):
        E.ellm_tensor_map_chunks(P, t, 0, s)
    E.ellm_kv_append(P, ids, DUMMY, DUMMY, np.asarray(lens, np.int32), stream=0)
    seen = [(E.ellm_debug_decode_kernel(P, x), list(E.ellm_decode_plan(P, x)[0])) for x in [ids] + [ids[i:i + 128] for i in range(0, len(ids), 128)]]
    E.ellm_pool_destroy(P)
    return seen


# batches whose groups go by blocks or steps of units, which carry a weight as two bf16 values, and which as a whole would be large
# enough for tiles, which carry one: all of the batch, then what is left past the first 128; then one of tiles all through, and of units
@pytest.mark.parametrize("n,length,n_kv,dim,group,kernels", [
    (200, 200, 4, 64, 1, "block block"), (150, 250, 4, 64, 2, "block block"), (140, 60, 4, 64, 2, "block block"), (136, 200, 4, 128, 4, "block block"),
    (200, 40, 4, 128, 4, "unit unit"), (136, 1000, 8, 128, 4, "tile block"), (132, 1000, 8, 128, 1, "tile unit"), (129, 2000, 8, 128, 8, "tile unit"),
    (150, 300, 8, 128, 4, "tile block"), (160, 500, 4, 128, 4, "tile block"), (136, 1000, 8, 64, 2, "tile block"), (256, 1000, 8, 128, 4, "tile tile"),
    (256, 1000, 8, 128, 6, "unit unit")])
def test_groups_keep_their_kernels(n, length, n_kv, dim, group, kernels):
    whole, *groups = plans([length] * n, n_kv, group, dim, 512)
    assert [k for k, _ in groups] == [f"decode_{k}_kernel" for k in kernels.split()]
    assert whole == (groups[0][0], groups[0][1] + groups[1][1])


def test_random_batches_keep_their_cuts():
    rng = np.random.default_rng(17)
    for _ in range(120):
        n_kv, group, dim = int(rng.choice([1, 2, 3, 4, 7, 8])), int(rng.choice([1, 2, 4, 6, 8, 12, 16, 20])), int(rng.choice([64, 128]))
        n, mean = int(rng.integers(129, 300)), float(np.exp(rng.uniform(np.log(20), np.log(3000))))
        lens = [int(x) for x in np.maximum(1, rng.lognormal(np.log(mean), rng.choice([0.05, 0.8]), n))]
        whole, *groups = plans(lens, n_kv, group, dim, int(rng.choice([16, 24, 64, 102, 512])))
        assert whole == (groups[0][0], sum((c for _, c in groups), [])), (n, mean, n_kv, group, dim)


PROGRAM = r"""
#include "kernels.hpp"
#include <cstdio>
#include <random>
#include <vector>
// every plan's workgroups, as the kernel numbers them: the slot of each one's result lies in what its request has reserved
int main() {
  std::mt19937 rng(5);
  auto draw = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  long wrong = 0, shared = 0, uneven = 0, more = 0;
  for (int turn = 0; turn < 20000; turn++) {
    static ellm::BatchArgs a;
    const int n_kv = draw(1, 9);
    a.n_req = draw(1, ellm::MAX_LAUNCH_REQ);
    a.wg_waves = draw(0, 3) ? ellm::SHARE_WAVES : 1;
    a.merge_parts = draw(0, 3) ? 1 << 20 : 0;
    std::vector<int> n(a.n_req);
    long total = 0;
    for (int& x : n) total += x = draw(0, 9) ? draw(1, 12) : draw(1, 400);
    a.waves_per_head = (int)std::min<long>(total, draw(1, 300));
    const long W = a.waves_per_head, each = total / W, extra = total - each * W;
    auto wave_of = [&](long x) { return x < extra * (each + 1) ? x / (each + 1) : extra + (x - extra * (each + 1)) / each; };
    long at = 0, by_wave = 0;
    for (int i = 0; i < a.n_req; i++) {
      a.req[i].wave_first = (int)wave_of(at);
      a.req[i].n_part = (int)(wave_of(at + n[i] - 1) - wave_of(at) + 1);
      by_wave += a.req[i].n_part > 1 ? a.req[i].n_part : 0;
      at += n[i];
    }
    const long parts = ellm::slots_by_workgroup(a, n_kv);
    if (parts > by_wave || a.parts_per_head != parts || a.ws_slots != parts * n_kv) wrong++;
    uneven += W % ellm::SHARE_WAVES != 0;
    std::vector<int> owner(parts);
    for (int g = 0; g < n_kv; g++) {
      std::fill(owner.begin(), owner.end(), -1);
      for (int i = 0; i < a.n_req; i++) {
        const auto& r = a.req[i];
        if (r.n_part < 2) continue;
        const long w0 = g * W + r.wave_first, first = w0 / a.wg_waves, n_wg = (w0 + r.n_part - 1) / a.wg_waves - first + 1;
        if (n_wg == 1 && a.merge_parts > 0) continue;          // finished in the workgroup
        shared++;
        more += n_wg > 2;
        for (long j = 0; j < n_wg; j++) {
          const long slot = r.part0 + j;
          if (slot >= parts || owner[slot] != -1) wrong++;
          else owner[slot] = i;
        }
      }
    }
  }
  std::printf("%ld %ld %ld %ld\n", wrong, shared, uneven, more);
}
"""


def test_slots_of_two_groups_in_one_launch(tmp_path):
    """Counted by workgroup they hold every partial result, whichever way a head's waves fall into workgroups."""
    src, exe = tmp_path / "s.cpp", tmp_path / "s"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "paper_2506_15155_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    wrong, shared, uneven, more = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert wrong == 0 and min(shared, uneven, more) > 1000
