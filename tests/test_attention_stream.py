"""The attention's stream of loads (csrc/a3_attn_stream.h), compiled for the CPU and walked as the kernel walks it: K of every tile
of every item in order and V one request later, stretches of tiles in steps alone included; no request, also not those behind the
stream's last tile, starts behind the last visible key of its descriptor, and no lane's offset passes 32 bits at the longest request
that is accepted.  And the kernel's phases: what a phase reads of K and V has been waited for by the waves that requested it, with a barrier
between, whatever the lengths of the items; and no request overwrites a tile that is still to be read."""
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

PHASES = r"""
#include <cstdio>
#include <deque>
#include <map>
#include <random>
#include <vector>
#include "a3_attn_stream.h"
// Group g multiplies tile u (and reads K of u, V of u - 1) in phase 2 u + g and reads V of u at the end of phase 2 u + 1 + g.
static int check(const std::vector<int> &items) {            // tiles of each
  std::vector<char> first, last;
  for (int n : items)
    for (int i = 0; i < n; ++i) { first.push_back(i == 0); last.push_back(i == n - 1); }
  const int tiles = (int)first.size();
  enum { K, V, OTHER };
  std::map<int, int> landed[2][2], asked[2][2];              // [group][K, V] of a tile: phase in which it was waited for, requested
  for (int g = 0; g < 2; ++g) {
    std::deque<std::pair<int, int>> open;                    // requests in order
    auto ask = [&](int what, int tile, int n, int phase) {
      for (int i = 0; i < n; ++i) open.push_back({what, tile});
      if (what != OTHER) asked[g][what][tile] = phase;
    };
    auto wait = [&](size_t leave, int phase) {
      for (; open.size() > leave; open.pop_front())
        if (open.front().first != OTHER) landed[g][open.front().first][open.front().second] = phase;
    };
    ask(K, 0, 2, -1); ask(K, 1, 2, -1); ask(V, 0, 2, -1); ask(OTHER, 0, 10, -1); ask(K, 2, 2, -1); ask(V, 1, 2, -1);
    wait(0, -1);
    for (int u = 0; u < tiles; ++u) {
      if (first[u]) { wait(0, 2 * u + g); ask(OTHER, 0, u ? 18 : 0, 2 * u + g); }
      ask(K, u + 3, 2, 2 * u + g); ask(V, u + 2, 2, 2 * u + g);
      if (attn_waits_behind(first[u], last[u])) wait(4, 2 * u + 1 + g);
      if (last[u]) ask(OTHER, 0, 10, 2 * u + 1 + g);
    }
  }
  for (int from = 0; from < 2; ++from)                       // group that requests, group that reads
    for (int g = 0; g < 2; ++g)
      for (int t = 0; t < tiles; ++t) {
        auto there = [&](int what, int phase) { return landed[from][what].count(t) && landed[from][what][t] < phase; };
        if (!there(K, 2 * t + g) || !there(V, 2 * t + 1 + g))
          return std::printf("tile %d of %d: the part of group %d is read by group %d before it was waited for\n", t, tiles, from, g), 1;
        if ((asked[from][K].count(t + 4) && asked[from][K][t + 4] <= 2 * t + g) || (asked[from][V].count(t + 4) && asked[from][V][t + 4] <= 2 * t + 2 + g))
          return std::printf("tile %d of %d: overwritten by group %d before group %d has read it\n", t, tiles, from, g), 1;
      }
  return 0;
}
int main() {
  std::mt19937 rng(2);
  for (int trial = 0; trial < 3000; ++trial) {
    std::vector<int> items(1 + rng() % 7);
    for (int &n : items) n = 1 + rng() % 5;
    if (check(items)) return 1;
  }
  return 0;
}
"""

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")


def _run(tmp_path, program):
    src, exe = tmp_path / "stream.cpp", tmp_path / "stream"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2511_17560_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout


def test_requests_stay_inside_their_descriptors(tmp_path):
    _run(tmp_path, PROGRAM)


def test_what_a_phase_reads_has_landed(tmp_path):
    _run(tmp_path, PHASES)
