// bpida_ring5.h -- the batched search's 64-node round on 5x5 boards: the
// scheme of bpida_ring.h (an entry is an expanded node with the moves it has
// left; a lane makes one move a round) with coordinates of three bits.
//
// What bounds it: the LDS, then vector issue.  The round it replaces built
// all four children of a 128-bit board at 211 vector instructions for 64
// nodes; this one takes 50, but moves 28-byte entries (14 LDS cycles to read
// 64, 28 to write two masked sets, 8 for the table: 200 of the 274 cycles a
// round takes on a SIMD, whose four waves share the LDS with three others).
// Measured, 256 states of 60-move walks: 126 ms before, 51 ms.
//
// The board is six 32-bit planes: bits 0, 1, 2 of the goal row and of the goal
// column of the tile in each cell, one bit a cell, on a ring of 32 cells with
// 6 to a board row, rotated so that the blank stands at bit 22.  (Three-bit
// fields would need a ring of 96 bits, whose rotation is three funnel shifts
// and selects; bit planes rotate in one instruction each.)  The neighbours
// are at U 16, L 21, R 23, D 28.  The four compares run bit by bit, all four
// moves at once: three select the row planes at U and D and the column planes
// at L and R, three form "smaller than the blank cell's constant".
//
// Meta word: bits 4..8 the blank's ring cell (6 * row + column), 9..15 slack
// / 2, and one bit per move still to be made at its neighbour's position, so
// the move with p leading zeros turns the ring by 9 - p.
#pragma once

#include "bpida_ring.h"

namespace bpida {

constexpr uint32_t kR5Blank = 1u << 22;
constexpr uint32_t kR5U = 1u << 16, kR5L = 1u << 21, kR5R = 1u << 23, kR5D = 1u << 28;
constexpr uint32_t kR5Moves = kR5U | kR5L | kR5R | kR5D;
constexpr uint32_t kR5Base = 0xFFFFu;
constexpr uint32_t kR5Cell = 31u << 4;
constexpr uint32_t kR5Slack1 = 1u << 9;
constexpr uint32_t kR5Entry = 28;  // bytes
constexpr int kR5Turn = 9;         // turn = 9 - leading zeros
constexpr uint32_t kR5Undo = 1u << 13;  // shifted left by the leading zeros: the undoing move
static_assert(kR5Turn - ring_lz(kR5U) == -6 && kR5Turn - ring_lz(kR5L) == -1 && kR5Turn - ring_lz(kR5R) == 1 &&
                  kR5Turn - ring_lz(kR5D) == 6,
              "rotations of the moves");
static_assert((kR5Undo << ring_lz(kR5U)) == kR5D && (kR5Undo << ring_lz(kR5L)) == kR5R &&
                  (kR5Undo << ring_lz(kR5R)) == kR5L && (kR5Undo << ring_lz(kR5D)) == kR5U,
              "undoing moves");

// Ring cell <-> board cell.
__host__ __device__ constexpr uint32_t r5_cell(uint32_t p) { return p + p / 5u; }
__host__ __device__ constexpr uint32_t r5_bit(uint32_t k, uint32_t b) { return (22u + k - b) & 31u; }

__host__ __device__ constexpr uint32_t r5_legal(uint32_t b) {
  const uint32_t r = b / 6u, c = b % 6u;
  return (r > 0 ? kR5U : 0u) | (c > 0 ? kR5L : 0u) | (c < 4 ? kR5R : 0u) | (r < 4 ? kR5D : 0u);
}
// Bit j (0..2) of the numbers the neighbours' coordinates are compared with,
// at the moves' bits.  U and L bring their tile nearer iff its goal row
// (column) is not smaller than the blank's, R and D iff it is smaller than
// the blank's plus one; off the board the compare says "away".
__host__ __device__ constexpr uint32_t r5_compare(uint32_t b, int j) {
  const uint32_t r = b / 6u, c = b % 6u, legal = r5_legal(b);
  const uint32_t u = legal & kR5U ? r : 7u, l = legal & kR5L ? c : 7u, ri = legal & kR5R ? c + 1 : 0u,
                 d = legal & kR5D ? r + 1 : 0u;
  return ((u >> j) & 1u) * kR5U | ((l >> j) & 1u) * kR5L | ((ri >> j) & 1u) * kR5R | ((d >> j) & 1u) * kR5D;
}

struct R5Planes {
  uint32_t r[3], c[3];  // bits 0, 1, 2 of the goal row and column
};
// The moves that bring their tile nearer.
__host__ __device__ constexpr uint32_t r5_nearer(const R5Planes& s, uint32_t y0, uint32_t y1, uint32_t y2) {
  constexpr uint32_t ud = kR5U | kR5D;
  const uint32_t x0 = (s.r[0] & ud) | (s.c[0] & ~ud), x1 = (s.r[1] & ud) | (s.c[1] & ~ud),
                 x2 = (s.r[2] & ud) | (s.c[2] & ~ud);
  uint32_t lt = ~x0 & y0;
  lt = (~x1 & y1) | (~(x1 ^ y1) & lt);
  lt = (~x2 & y2) | (~(x2 ^ y2) & lt);
  return (lt ^ (kR5U | kR5L)) & kR5Moves;
}

// The same on the device, one instruction for each select and compare step.
__device__ __forceinline__ uint32_t r5_nearer_bits(const R5Planes& s, uint32_t y0, uint32_t y1, uint32_t y2) {
  constexpr uint32_t ud = kR5U | kR5D;
  constexpr uint32_t kSelect = 0xCA, kLess = 0x8E, kAndNot = 0x0C;  // truth tables
  const uint32_t x0 = __builtin_amdgcn_bitop3_b32(ud, s.r[0], s.c[0], kSelect);
  const uint32_t x1 = __builtin_amdgcn_bitop3_b32(ud, s.r[1], s.c[1], kSelect);
  const uint32_t x2 = __builtin_amdgcn_bitop3_b32(ud, s.r[2], s.c[2], kSelect);
  uint32_t lt = __builtin_amdgcn_bitop3_b32(x0, y0, 0u, kAndNot);
  lt = __builtin_amdgcn_bitop3_b32(x1, y1, lt, kLess);
  lt = __builtin_amdgcn_bitop3_b32(x2, y2, lt, kLess);
  return (lt ^ (kR5U | kR5L)) & kR5Moves;
}

// Compile-time proof: "nearer" is "the tile's distance to its goal shrinks"
// for every blank cell, move and tile coordinates, whatever stands elsewhere.
constexpr bool check_r5() {
  for (uint32_t p = 0; p < 25; ++p) {
    const uint32_t b = r5_cell(p);
    const int dr[4] = {-1, 0, 0, 1}, dc[4] = {0, -1, 1, 0};
    const uint32_t bit[4] = {kR5U, kR5L, kR5R, kR5D};
    for (int a = 0; a < 4; ++a) {
      const int nr = (int)(p / 5) + dr[a], nc = (int)(p % 5) + dc[a];
      const bool on = nr >= 0 && nc >= 0 && nr < 5 && nc < 5;
      if (((r5_legal(b) & bit[a]) != 0) != on) return false;
      if (bit[a] != 1u << r5_bit(b + (uint32_t)(6 * dr[a] + dc[a]), b)) return false;
      for (uint32_t tr = 0; tr < 5; ++tr)
        for (uint32_t tc = 0; tc < 5; ++tc)
          for (int fill = 0; fill < 2; ++fill) {
            R5Planes s{};
            for (int j = 0; j < 3; ++j) {
              s.r[j] = (fill ? ~bit[a] : 0u) | ((tr >> j) & 1u) * bit[a];
              s.c[j] = (fill ? ~bit[a] : 0u) | ((tc >> j) & 1u) * bit[a];
            }
            const bool near = (r5_nearer(s, r5_compare(b, 0), r5_compare(b, 1), r5_compare(b, 2)) & bit[a]) != 0;
            const int goal = dr[a] ? (int)tr : (int)tc, from = dr[a] ? nr : nc, to = dr[a] ? (int)(p / 5) : (int)(p % 5);
            const int before = goal > from ? goal - from : from - goal, after = goal > to ? goal - to : to - goal;
            if (near != (on && after < before)) return false;
          }
    }
  }
  return true;
}
static_assert(check_r5(), "5x5 ring compares disagree with the board");

__host__ __device__ constexpr uint32_t r5_rotr(uint32_t v, uint32_t s) {
  return (v >> (s & 31u)) | (v << ((32u - s) & 31u));
}

// Planes of a packed 5x5 board (5 bits a cell) whose blank is at board cell b.
__host__ __device__ __forceinline__ constexpr R5Planes r5_planes(unsigned __int128 s, uint32_t b) {
  uint32_t r0 = 0, r1 = 0, r2 = 0, c0 = 0, c1 = 0, c2 = 0;
#pragma unroll 1
  for (uint32_t p = 0; p < 25; ++p) {
    const uint32_t t = (uint32_t)s & 31u, tr = (t * 13u) >> 6, tc = t - 5u * tr, at = p + (p * 13u >> 6);
    s >>= 5;
    r0 |= (tr & 1u) << at;
    r1 |= ((tr >> 1) & 1u) << at;
    r2 |= (tr >> 2) << at;
    c0 |= (tc & 1u) << at;
    c1 |= ((tc >> 1) & 1u) << at;
    c2 |= (tc >> 2) << at;
  }
  const uint32_t turn = r5_cell(b) - 22u;
  return {{r5_rotr(r0, turn), r5_rotr(r1, turn), r5_rotr(r2, turn)},
          {r5_rotr(c0, turn), r5_rotr(c1, turn), r5_rotr(c2, turn)}};
}
// And back; b is the blank's ring cell (its own field is read as 0).
__host__ __device__ __forceinline__ constexpr unsigned __int128 r5_board(const R5Planes& v, uint32_t b) {
  const uint32_t turn = 22u - b, rest = ~(1u << b);
  const uint32_t r0 = r5_rotr(v.r[0], turn) & rest, r1 = r5_rotr(v.r[1], turn) & rest, r2 = r5_rotr(v.r[2], turn) & rest;
  const uint32_t c0 = r5_rotr(v.c[0], turn) & rest, c1 = r5_rotr(v.c[1], turn) & rest, c2 = r5_rotr(v.c[2], turn) & rest;
  unsigned __int128 s = 0;
#pragma unroll 1
  for (uint32_t p = 25; p-- > 0;) {
    const uint32_t at = p + (p * 13u >> 6);
    const uint32_t tr = ((r0 >> at) & 1u) | (((r1 >> at) & 1u) << 1) | (((r2 >> at) & 1u) << 2);
    const uint32_t tc = ((c0 >> at) & 1u) | (((c1 >> at) & 1u) << 1) | (((c2 >> at) & 1u) << 2);
    s = (s << 5) | (5u * tr + tc);
  }
  return s;
}
constexpr bool check_r5_board() {
  for (uint32_t p = 0; p < 25; ++p) {
    if ((p * 13u) >> 6 != p / 5u) return false;
    // the goal with its blank moved to cell p along the cells' order
    unsigned __int128 s = 0;
    for (uint32_t k = 0; k < 25; ++k) s |= (unsigned __int128)(k < p ? k + 1 : k == p ? 0 : k) << (5 * k);
    if (r5_board(r5_planes(s, p), r5_cell(p)) != s) return false;
  }
  return true;
}
static_assert(check_r5_board(), "5x5 planes do not round-trip");
constexpr R5Planes kR5Goal = r5_planes(Board<5>::goal(), 0);

// Meta word <-> the 16 bits it takes in a queue chunk: blank, slack / 2, and
// the moves U, L, R, D at bits 12..15.
__host__ __device__ constexpr uint32_t r5_pack(uint32_t m) {
  return ((m >> 4) & 0xFFFu) | (((m >> 16) & 1u) << 12) | (((m >> 21) & 1u) << 13) | (((m >> 23) & 1u) << 14) |
         (((m >> 28) & 1u) << 15);
}
__host__ __device__ constexpr uint32_t r5_unpack(uint32_t v) {
  return ((v & 0xFFFu) << 4) | (((v >> 12) & 1u) << 16) | (((v >> 13) & 1u) << 21) | (((v >> 14) & 1u) << 23) |
         (((v >> 15) & 1u) << 28);
}
static_assert(r5_unpack(r5_pack(kR5Moves | 0xFFF0u)) == (kR5Moves | 0xFFF0u) &&
                  r5_unpack(r5_pack(kR5R | 0xA5A0u)) == (kR5R | 0xA5A0u),
              "meta round trip");

// A blank cell's constants, in a table of 32 in LDS (16 bytes a cell, the
// meta word's blank field is the address).
struct alignas(16) R5Cell {
  uint32_t y0, y1, y2, legal;
};
constexpr uint32_t kR5Table = 32 * sizeof(R5Cell);

// A node's meta word, with the moves it keeps (as ring_meta).
__device__ __forceinline__ uint32_t r5_meta(uint32_t base, uint32_t near, uint32_t legal, uint32_t undo) {
  return ((base >= kR5Slack1 ? legal : near) & ~undo) | base;
}

struct R5Consts {
  uint32_t top_bit, undo;  // 1 << 31, kR5Undo
  uint32_t lane;           // LDS byte address of stack entry `lane`
  uint32_t base;           // LDS byte address of the stack
};
__device__ __forceinline__ R5Consts make_r5_consts(char* stack, uint32_t table) {
  const uint32_t b = (uint32_t)lane_id() & 31u;
  R5Consts k;
  k.top_bit = opaque(1u << 31);
  k.undo = opaque(kR5Undo);
  k.base = lds_addr(stack);
  k.lane = opaque(k.base + kR5Entry * (uint32_t)lane_id());
  *(R5Cell*)(stack + table + 16u * b) = {r5_compare(b, 0), r5_compare(b, 1), r5_compare(b, 2), r5_legal(b)};
  return k;
}

__device__ __forceinline__ uint32_t r5_at(uint64_t mask, uint32_t c) {
  const uint32_t r = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
  uint32_t d;
  asm("v_mad_u32_u24 %0, %1, 28, %2" : "=v"(d) : "v"(r), "s"(c));
  return d;
}

// The lanes of `mask` store an entry at LDS address `at`, with no branch.
__device__ __forceinline__ void r5_put(uint64_t mask, uint32_t at, const R5Planes& s, uint32_t m) {
  uint64_t saved;
  asm volatile(
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, %1\n\t"
      "ds_write2_b32 %2, %3, %4 offset1:1\n\t"
      "ds_write2_b32 %2, %5, %6 offset0:2 offset1:3\n\t"
      "ds_write2_b32 %2, %7, %8 offset0:4 offset1:5\n\t"
      "ds_write_b32 %2, %9 offset:24\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "s"(mask), "v"(at), "v"(s.r[0]), "v"(s.r[1]), "v"(s.r[2]), "v"(s.c[0]), "v"(s.c[1]), "v"(s.c[2]), "v"(m)
      : "memory");
}

// The tile at `turn` from the blank moves under the blank, and the ring turns.
__device__ __forceinline__ uint32_t r5_move(uint32_t v, uint32_t turn) {
  const uint32_t v1 = __builtin_amdgcn_alignbit(v, v, turn);
  const uint32_t v2 = (v1 & kR5Blank) | (v & ~kR5Blank);
  return __builtin_amdgcn_alignbit(v2, v2, turn);
}

// One round; as ring_round.
template <uint32_t TABLE, bool FULL>
__device__ __forceinline__ uint32_t r5_round(uint32_t top, int kp, uint64_t& goal, const R5Consts& k) {
  const uint32_t low = top - (uint32_t)(FULL ? 64 : kp);
  const uint32_t at = k.lane + low * kR5Entry;
  const __attribute__((address_space(3))) uint32_t* e =
      (const __attribute__((address_space(3))) uint32_t*)(uintptr_t)at;
  R5Planes s, n;
  uint32_t m = e[6];
  for (int j = 0; j < 3; ++j) {
    s.r[j] = e[j];
    s.c[j] = e[3 + j];
  }
  if (!FULL) m &= (uint32_t)lane_id() < (uint32_t)kp ? ~0u : 0u;
  const uint32_t p = (uint32_t)__builtin_clz(FULL ? m : m | 1u);
  const uint32_t turn = (uint32_t)kR5Turn - p;
  for (int j = 0; j < 3; ++j) {
    n.r[j] = r5_move(s.r[j], turn);
    n.c[j] = r5_move(s.c[j], turn);
  }
  const uint32_t at_b = (m & kR5Base) + (turn << 4);
  const __attribute__((address_space(3))) R5Cell* cell =
      (const __attribute__((address_space(3))) R5Cell*)(uintptr_t)(k.base + TABLE + (at_b & kR5Cell));
  const uint32_t y0 = cell->y0, y1 = cell->y1, y2 = cell->y2, legal = cell->legal;
  const uint32_t near = r5_nearer_bits(n, y0, y1, y2);
  const uint32_t undo = k.undo << p;
  const uint32_t base = at_b - min(near & undo, kR5Slack1);
  const uint32_t cm = r5_meta(base, near, legal, undo);
  const uint32_t left = m ^ (k.top_bit >> p);
  const uint64_t lanes = FULL ? ~0ull : ring_uniform((kp >= 64 ? 0ull : 1ull << kp) - 1ull);
  const uint64_t kl = __builtin_amdgcn_uicmp(left, kR5Base, 34);        // moves left
  const uint64_t kc = __builtin_amdgcn_uicmp(cm, kR5Base, 34) & lanes;  // child keeps some
  // goal: 16 cells of one plane first, the rest only where they agree
  const uint64_t g16 = ring_eq16(kR5Goal.c[0], n.c[0]);
  if (g16) {
    uint32_t d = 0;
    for (int j = 0; j < 3; ++j) d |= (n.r[j] ^ kR5Goal.r[j]) | (n.c[j] ^ kR5Goal.c[j]);
    goal |= __builtin_amdgcn_ballot_w64((d & ~kR5Blank) == 0 && (base & kR5Cell) == 0) & lanes;
  }
  const uint32_t mid = low + (uint32_t)__popcll(kl);
  r5_put(kl, r5_at(kl, k.base + low * kR5Entry), s, left);
  r5_put(kc, r5_at(kc, k.base + mid * kR5Entry), n, cm);
  WAVE_SYNC();
  return mid + (uint32_t)__popcll(kc);
}

}  // namespace bpida
