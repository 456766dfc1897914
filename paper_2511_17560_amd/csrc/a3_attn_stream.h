// The attention's stream of loads: which tile of keys is requested next, as byte offsets from the descriptor of its request and
// head.  Integer rules only, no device code: constexpr functions serve the kernel, and compile with any C++17 compiler.
#pragma once

#include <cstdint>

constexpr int kTK = 64;                                      // keys per tile

// K of a tile is requested one tile before its V.  Offsets of a request are 32-bit byte counts, its descriptor's size too: K or V
// of a request (with 128 rows in hand; the furthest lane of a tile lies 63 rows behind the last visible key) has to stay below
// 4 GiB, which the host requires.
struct attn_stream {
  uint32_t at, v_at;                                         // the tile whose K comes next, the one before it (its V)
  int left;                                                  // tiles of the item from `at` on

  // bytes from the first row of the request to the end of the last one that the item sees: the descriptor's size
  static constexpr uint32_t bytes(int kv_len, uint32_t pitch, uint32_t row_bytes) { return (uint32_t)(kv_len - 1) * pitch + row_bytes; }
  constexpr void enter(int k_begin, int k_end, uint32_t pitch) {
    at = (uint32_t)k_begin * pitch;
    left = (k_end - k_begin + kTK - 1) / kTK;
  }
  // A position is the scalar offset of its loads, which the hardware subtracts from the descriptor's size before it compares: it
  // never lies behind the last visible key.  The stream asks for up to three tiles behind its last one (nothing reads them): they
  // start at that key, and everything behind the descriptor's end comes back as zeros.
  constexpr void step(uint32_t pitch, uint32_t size, uint32_t row_bytes) {
    const uint32_t next = at + kTK * pitch, last = size - row_bytes;
    v_at = at;
    at = next < last ? next : last;
  }
  // behind a step: whether the tile that comes next belongs to the same item
  constexpr bool same() { return --left > 0; }
  constexpr void end() { left = 1 << 30; }
  // of the next `tiles` tiles that are multiplied, how many can pass with nothing but a step each
  constexpr int calm(int tiles) const { return (tiles < left ? tiles : left) - 1; }
  constexpr void pass(int tiles) { left -= tiles; }
};

// Behind the softmax of a tile and before it requests the rows of the next item, a wave waits for all but the tile's own requests (K of
// tile u + 3 and V of tile u + 2): V of tile u + 1, which every wave reads two phases later, has then landed.  The first tile of an
// item needs no wait here: it waits for everything in its matrix phase, before its stores and its requests.
constexpr bool attn_waits_behind(bool first_of_item, bool /*last_of_item*/) { return !first_of_item; }
