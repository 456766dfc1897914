"""The attention's stream of loads (csrc/a3_attn_stream.h), compiled for the CPU and walked as the kernel walks it: K of every tile
of every item in order and V one request later, stretches of tiles in steps alone included; no request, also not those behind the
stream's last tile, starts behind the last visible key of its descriptor, and no lane's offset passes 32 bits at the longest request
that is accepted."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "a3_attn_stream.h"
struct item { int k_begin, k_end, kv_len; };
struct request { uint32_t at, size; };
static int walk(const std::vector<item> &items, uint32_t pitch, std::mt19937 &rng) {
  const uint32_t row = 256;
  std::vector<request> want, k, v;
  for (const item &i : items)
    for (int b = i.k_begin; b < i.k_end; b += kTK) want.push_back({(uint32_t)b * pitch, attn_stream::bytes(i.kv_len, pitch, row)});
  attn_stream s = {0, 0, 0};
  size_t next = 0;                                           // item of the tile whose K comes next
  uint32_t k_size = 0, v_size = 0;
  bool same = false;
  auto enter = [&]() { s.enter(items[next].k_begin, items[next].k_end, pitch); k_size = attn_stream::bytes(items[next].kv_len, pitch, row); };
  auto step = [&]() { s.step(pitch, k_size, row); };
  auto on = [&]() {
    v_size = k_size;
    same = s.same();
    if (!same && next + 1 < items.size()) { ++next; enter(); }
    else if (!same) s.end();
  };
  auto ask_k = [&]() { k.push_back({s.at, k_size}); };
  auto ask_v = [&]() { v.push_back({s.v_at, v_size}); };
  enter();
  ask_k(); step(); on();
  for (int i = 0; i < 2; ++i) { ask_k(); ask_v(); step(); on(); }
  for (const item &i : items)
    for (int k0 = i.k_begin; k0 < i.k_end;) {
      ask_k(); ask_v(); step(); on();
      k0 += kTK;
      if (k0 >= i.k_end || !same) continue;
      const int most = s.calm((i.k_end - k0 + kTK - 1) / kTK), n = most > 0 ? (int)(rng() % (most + 1)) : 0;
      for (int c = 0; c < n; ++c) { ask_k(); ask_v(); step(); }
      s.pass(n);
      k0 += n * kTK;
    }
  for (size_t t = 0; t < want.size(); ++t)
    if (k[t].at != want[t].at || k[t].size != want[t].size || v[t].at != want[t].at || v[t].size != want[t].size)
      return std::printf("tile %zu: K %u (%u), V %u (%u), want %u (%u)\n", t, k[t].at, k[t].size, v[t].at, v[t].size, want[t].at, want[t].size), 1;
  for (const auto *r : {&k, &v})
    for (const request &x : *r) {
      if (x.at > x.size - row) return std::printf("%s: offset %u behind the last key of %u bytes\n", r == &k ? "K" : "V", x.at, x.size), 1;
      if ((unsigned long long)x.at + 63ull * pitch + row > 0xffffffffull) return std::printf("offset %u passes 32 bits\n", x.at), 1;
    }
  return 0;
}
int main() {
  std::mt19937 rng(1);
  for (int trial = 0; trial < 4000; ++trial) {
    std::vector<item> items;
    for (int n = 1 + rng() % 6; n > 0; --n) {
      const int kv = 1 + rng() % (trial % 2 ? 1500 : 150), steps = (kv + kTK - 1) / kTK, b = rng() % steps, e = b + 1 + rng() % (steps - b);
      items.push_back({b * kTK, e * kTK < kv ? e * kTK : kv, kv});
    }
    if (walk(items, 256u * (1 + rng() % 8), rng)) return 1;
  }
  // the longest request: (rows + 128) x pitch below 4 GiB
  for (unsigned heads = 1; heads <= 8; heads *= 2) {
    const uint32_t pitch = 256 * heads;
    const int rows = (int)((0xffffffffull - 128ull * pitch) / pitch);
    if (walk({{(rows - 1) / kTK * kTK - 64 * 20, rows, rows}}, pitch, rng)) return 1;
  }
  return 0;
}
"""

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")


def test_requests_stay_inside_their_descriptors(tmp_path):
    src, exe = tmp_path / "stream.cpp", tmp_path / "stream"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2511_17560_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
