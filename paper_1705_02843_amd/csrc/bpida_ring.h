// bpida_ring.h -- the batched search's 64-node round on 3x3 and 4x4 boards:
// one generated node per lane and round.
//
// What bounds it: vector issue, with the LDS close behind.  The round that
// builds all four children of a popped node (bpida_board.h, still the plain
// mode's) spends two thirds of its 63 vector instructions on move slots, of
// which a node keeps one in four.  Here a stack entry is an expanded node
// together with the set of its moves that are kept but not yet made.  A round
// pops 64 entries; every lane makes ONE of its entry's moves and works out, in
// the same instructions, which moves the child keeps.  The child goes back to
// the stack if it keeps any, and the parent if it has moves left; a child that
// keeps none (a third of all) is counted and never stored.  Every lane's work
// is a node, at 34 vector and 7 LDS instructions a round.
// Measured, 4096 uneven 4x4 states: 0.949 s before, 0.541 s with this round.
// Another such batch (the stored states), at stack option 640: 0.507 s, 139
// cycles a round and SIMD, of which 31 issue slots of 4 are vector issue and
// about 98 are LDS; with the per-cell constants from two ds_bpermute (4 more
// LDS cycles a round and wave) instead of the table below 0.584 s.
//
// Two things make the move cheap although it differs from lane to lane:
//
//   - The board is two 32-bit planes, the goal row and the goal column of the
//     tile in each of 16 cells, two bits a cell, on a ring that is kept
//     rotated so that the blank stands at bits 20..21.  The neighbours are
//     then at fixed bits (U 12, L 18, R 22, D 28), and moving the blank by
//     delta is one rotation by 2*delta to fetch the tile, one bit-field insert
//     that puts it under the blank, and one more rotation.  The blank's own
//     field holds a copy of the tile moved last; nothing reads it.  A 3x3
//     board lies in the top left corner of the same 4-wide ring.
//   - All four compares "does this move take its tile away from its goal" are
//     one addition: U and L moves away iff the tile's goal row (column) is
//     smaller than the blank's, R and D iff it is larger, so adding a
//     per-blank constant to the four two-bit fields leaves each answer in the
//     bit above its field (14, 20, 24, 30).  The constant of an edge cell
//     makes a move off the board read as "away".
//
// Entry (12 bytes): row plane, column plane, and the meta word
//   bits 0..2 zero, 3..6 the blank's ring cell (4 * row + column), 7..12
//   slack / 2, and one bit per move still to be made: U 14, L 20, R 24, D 30.
// Those four positions are spaced so that a count of leading zeros finds the
// next move and indexes, as a bit position, a constant that holds the moves'
// rotations (kRingTurn).
#pragma once

#include <stdint.h>

#include "bpida_board.h"
#include "bpida_round.h"

namespace bpida {

constexpr uint32_t kRingU = 1u << 14, kRingL = 1u << 20, kRingR = 1u << 24, kRingD = 1u << 30;
constexpr uint32_t kRingMoves = kRingU | kRingL | kRingR | kRingD;
constexpr uint32_t kRingBase = 0x1FFFu;          // blank and slack
constexpr uint32_t kRingCell = 15u << 3;         // blank
constexpr uint32_t kRingSlack1 = 1u << 7;        // one unit of slack / 2
constexpr uint32_t kRingBlank = 3u << 20;        // the blank's field of a plane
constexpr uint32_t kRingRows = (3u << 12) | (3u << 28);   // U and D neighbours, row plane
constexpr uint32_t kRingCols = (3u << 18) | (3u << 22);   // L and R neighbours, column plane
constexpr uint32_t kRingEntry = 12;              // bytes

// Rotation (2 * cell offset, 5 bits signed) of the move whose bit has p
// leading zeros, at bits p..p+4.  R's (p = 7) and L's (p = 11) fields share
// bit 11, which is 0 in both.
constexpr uint32_t kRingTurn = (0x18u << 17) | (0x1Eu << 11) | (0x02u << 7) | (0x08u << 1);

constexpr int ring_lz(uint32_t bit) {
  int p = 0;
  while (!((bit << p) >> 31)) ++p;
  return p;
}
constexpr int ring_turn(int p) {
  const int v = (int)((kRingTurn >> p) & 31u);
  return v < 16 ? v : v - 32;
}
// A move's undo is the move whose bit is 1 << (13 + leading zeros).
constexpr uint32_t kRingUndo = 1u << 13;
static_assert(ring_turn(ring_lz(kRingU)) == -8 && ring_turn(ring_lz(kRingL)) == -2 &&
                  ring_turn(ring_lz(kRingR)) == 2 && ring_turn(ring_lz(kRingD)) == 8,
              "rotations of the moves");
static_assert((kRingUndo << ring_lz(kRingU)) == kRingD && (kRingUndo << ring_lz(kRingL)) == kRingR &&
                  (kRingUndo << ring_lz(kRingR)) == kRingL && (kRingUndo << ring_lz(kRingD)) == kRingU,
              "undoing moves");

// Moves that keep a blank at ring cell b on a W-wide board.
template <int W>
__host__ __device__ constexpr uint32_t ring_legal(uint32_t b) {
  const uint32_t r = b >> 2, c = b & 3u;
  return (r > 0 ? kRingU : 0u) | (c > 0 ? kRingL : 0u) | (c + 1 < (uint32_t)W ? kRingR : 0u) |
         (r + 1 < (uint32_t)W ? kRingD : 0u);
}
// Added to the neighbours' fields: bit 14 (20) of the sum is set iff U (L)
// brings its tile nearer, bit 24 (30) is set iff R (D) takes it away; off the
// board U and L read 0, R and D read 1.
template <int W>
__host__ __device__ constexpr uint32_t ring_compare(uint32_t b) {
  const uint32_t r = b >> 2, c = b & 3u, legal = ring_legal<W>(b);
  return ((legal & kRingU ? 4 - r : 0u) << 12) | ((legal & kRingL ? 4 - c : 0u) << 18) |
         ((legal & kRingR ? 3 - c : 4u) << 22) | ((legal & kRingD ? 3 - r : 4u) << 28);
}
// The moves that bring their tile nearer, from the planes (rows, cols) and
// the blank's compare constant.
__host__ __device__ constexpr uint32_t ring_nearer(uint32_t rows, uint32_t cols, uint32_t cmp) {
  const uint32_t z = ((rows & kRingRows) | (cols & kRingCols)) + cmp;
  return (z & (kRingU | kRingL)) | (~z & (kRingR | kRingD));
}
// Bit of ring cell k's field in a plane whose blank is at ring cell b.
__host__ __device__ constexpr uint32_t ring_bit(uint32_t k, uint32_t b) { return (20u + 2u * (k - b)) & 31u; }

// Compile-time proof against the definition: for every blank cell, neighbour
// tile and legal move, "nearer" is "the tile's distance to its goal shrinks";
// off the board no move is nearer; and every field other than the four read
// is without effect.
template <int W>
constexpr bool check_ring() {
  for (uint32_t b = 0; b < 16; ++b) {
    if ((b >> 2) >= (uint32_t)W || (b & 3u) >= (uint32_t)W) continue;
    const int dr[4] = {-1, 0, 0, 1}, dc[4] = {0, -1, 1, 0};
    const uint32_t bit[4] = {kRingU, kRingL, kRingR, kRingD};
    for (int a = 0; a < 4; ++a) {
      const int nr = (int)(b >> 2) + dr[a], nc = (int)(b & 3u) + dc[a];
      const bool on = nr >= 0 && nc >= 0 && nr < W && nc < W;
      if (((ring_legal<W>(b) & bit[a]) != 0) != on) return false;
      for (uint32_t tr = 0; tr < 4; ++tr)
        for (uint32_t tc = 0; tc < 4; ++tc)
          for (int fill = 0; fill < 2; ++fill) {
            const uint32_t k = b + (uint32_t)(4 * dr[a] + dc[a]), at = ring_bit(k, b);
            const uint32_t rest = fill ? ~0u : 0u;
            const uint32_t rows = (rest & ~(3u << at)) | (tr << at), cols = (rest & ~(3u << at)) | (tc << at);
            const bool near = (ring_nearer(rows, cols, ring_compare<W>(b)) & bit[a]) != 0;
            const int goal = dr[a] ? (int)tr : (int)tc, from = dr[a] ? nr : nc, to = dr[a] ? (int)(b >> 2) : (int)(b & 3u);
            const int before = goal > from ? goal - from : from - goal, after = goal > to ? goal - to : to - goal;
            if (near != (on && after < before)) return false;
          }
    }
  }
  return true;
}
static_assert(check_ring<3>() && check_ring<4>(), "ring compares disagree with the board");

// Planes of the goal board (blank at cell 0); the blank's field is ignored.
template <int W>
__host__ __device__ constexpr uint32_t ring_goal(bool rows) {
  uint32_t v = 0;
  for (uint32_t k = 1; k < 16; ++k)
    if ((k >> 2) < (uint32_t)W && (k & 3u) < (uint32_t)W) v |= (rows ? k >> 2 : k & 3u) << ring_bit(k, 0);
  return v;
}

// Meta word <-> the 16 bits it takes in a queue chunk: blank, slack / 2, and
// the moves U, L, R, D at bits 10..13.
__host__ __device__ constexpr uint32_t ring_pack(uint32_t m) {
  return ((m >> 3) & 0x3FFu) | (((m >> 14) & 1u) << 10) | (((m >> 20) & 1u) << 11) | (((m >> 24) & 1u) << 12) |
         (((m >> 30) & 1u) << 13);
}
__host__ __device__ constexpr uint32_t ring_unpack(uint32_t v) {
  return ((v & 0x3FFu) << 3) | (((v >> 10) & 1u) << 14) | (((v >> 11) & 1u) << 20) | (((v >> 12) & 1u) << 24) |
         (((v >> 13) & 1u) << 30);
}
static_assert(ring_unpack(ring_pack(kRingMoves | 0x1FF8u)) == (kRingMoves | 0x1FF8u), "meta round trip");
static_assert(ring_unpack(ring_pack(kRingL | 0xAA8u)) == (kRingL | 0xAA8u), "meta round trip");

// Planes of a packed board (4 bits a cell, bpida_board.h) whose blank is at
// cell b of the board; *ring_b receives the blank's ring cell.
template <int W>
__host__ __device__ constexpr void ring_planes(uint64_t s, uint32_t b, uint32_t* rows, uint32_t* cols,
                                               uint32_t* ring_b) {
  const uint32_t rb = W == 4 ? b : b + b / 3u;
  uint32_t r = 0, c = 0;
  for (uint32_t p = 0; p < (uint32_t)(W * W); ++p) {
    const uint32_t t = (uint32_t)(s >> (4 * p)) & 15u, k = W == 4 ? p : p + p / 3u;
    r |= (t / (uint32_t)W) << (2 * k);
    c |= (t % (uint32_t)W) << (2 * k);
  }
  const uint32_t turn = (2 * rb - 20u) & 31u;
  *rows = (r >> turn) | (r << ((32u - turn) & 31u));
  *cols = (c >> turn) | (c << ((32u - turn) & 31u));
  *ring_b = rb;
}
template <int W>
constexpr bool check_ring_goal() {
  uint32_t r = 0, c = 0, b = 0;
  ring_planes<W>((uint64_t)Board<W>::goal(), 0, &r, &c, &b);
  return b == 0 && r == ring_goal<W>(true) && c == ring_goal<W>(false);
}
static_assert(check_ring_goal<3>() && check_ring_goal<4>(), "goal planes");

// The two constants of a blank cell, in a table of 16 in LDS behind the
// wave's stack, 8 bytes a cell: the meta word's blank field is the address
// in it, and one ds_read_b64 (16 distinct words pairs, no bank conflict)
// costs the LDS half of what two ds_bpermute cost.
struct RingCell {
  uint32_t cmp, legal;
};
constexpr uint32_t kRingTable = 16 * sizeof(RingCell);

// Per-wave constants of the round.
struct RingConsts {
  uint32_t ul;             // kRingU | kRingL
  uint32_t top_bit, undo;  // 1 << 31, kRingUndo
  uint32_t lane;           // LDS byte address of stack entry `lane`
  uint32_t base;           // LDS byte address of the stack
};

// `stack`: the wave's LDS, `table` bytes into it the blank cells' constants.
template <int W>
__device__ __forceinline__ RingConsts make_ring_consts(char* stack, uint32_t table) {
  const uint32_t b = (uint32_t)lane_id() & 15u;
  RingConsts k;
  k.ul = opaque(kRingU | kRingL);
  k.top_bit = opaque(1u << 31);
  k.undo = opaque(kRingUndo);
  k.base = lds_addr(stack);
  k.lane = opaque(k.base + kRingEntry * (uint32_t)lane_id());
  *(RingCell*)(stack + table + 8u * b) = {ring_compare<W>(b), ring_legal<W>(b)};
  return k;
}

// rank * 12 + c in one instruction.
__device__ __forceinline__ uint32_t ring_at(uint64_t mask, uint32_t c) {
  const uint32_t r = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
  uint32_t d;
  asm("v_mad_u32_u24 %0, %1, 12, %2" : "=v"(d) : "v"(r), "s"(c));
  return d;
}

// Entry writes under two lane masks, with no branch: the lanes of k0 store
// (r0, c0, m0) at a0, then the lanes of k1 store (r1, c1, m1) at a1.
__device__ __forceinline__ void ring_put2(uint64_t k0, uint32_t a0, uint32_t r0, uint32_t c0, uint32_t m0,
                                          uint64_t k1, uint32_t a1, uint32_t r1, uint32_t c1, uint32_t m1) {
  uint64_t saved;
  asm volatile(
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, %1\n\t"
      "ds_write2_b32 %2, %3, %4 offset1:1\n\t"
      "ds_write_b32 %2, %5 offset:8\n\t"
      "s_mov_b64 exec, %6\n\t"
      "ds_write2_b32 %7, %8, %9 offset1:1\n\t"
      "ds_write_b32 %7, %10 offset:8\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "s"(k0), "v"(a0), "v"(r0), "v"(c0), "v"(m0), "s"(k1), "v"(a1), "v"(r1), "v"(c1), "v"(m1)
      : "memory");
}

__device__ __forceinline__ uint32_t ring_bfi(uint32_t sel, uint32_t one, uint32_t zero) {
  uint32_t d;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(d) : "v"(sel), "v"(one), "s"(zero));
  return d;
}

// A node's meta word, with the moves it keeps: any legal one if it has slack,
// else those that bring their tile nearer; never its undo.
__device__ __forceinline__ uint32_t ring_meta(uint32_t base, uint32_t near, uint32_t legal, uint32_t undo) {
  return ((base >= kRingSlack1 ? legal : near) & ~undo) | base;
}

// Lanes whose low 16 bits of v are those of c.
__device__ __forceinline__ uint64_t ring_eq16(uint32_t c, uint32_t v) {
  uint64_t r;
  asm("v_cmp_eq_u16_e64 %0, %1, %2" : "=s"(r) : "s"(c), "v"(v));
  return r;
}

// A wave-uniform mask as the compiler may not know it to be (folds away when
// it does).
__device__ __forceinline__ uint64_t ring_uniform(uint64_t v) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

// One round: pops kp = min(64, top) entries of the stack [0, top), makes one
// move of each, counts nothing (the caller adds kp nodes) and returns the new
// top.  The caller guarantees room for 64 more entries.  FULL: kp is 64.
// `goal` collects the lanes whose new node is the goal.
template <int W, uint32_t TABLE, bool FULL>
__device__ __forceinline__ uint32_t ring_round(uint32_t top, int kp, uint64_t& goal, const RingConsts& k) {
  const uint32_t low = top - (uint32_t)(FULL ? 64 : kp);
  const uint32_t at = k.lane + low * kRingEntry;
  const __attribute__((address_space(3))) uint32_t* e =
      (const __attribute__((address_space(3))) uint32_t*)(uintptr_t)at;
  const uint32_t r = e[0], c = e[1];
  const uint32_t act = FULL ? 0u : ((uint32_t)lane_id() < (uint32_t)kp ? ~0u : 0u);
  const uint32_t m = FULL ? e[2] : e[2] & act;
  // the next move, and the rotation that brings its tile to the blank
  const uint32_t p = (uint32_t)__builtin_clz(FULL ? m : m | 1u);
  const int turn = __builtin_amdgcn_sbfe((int)kRingTurn, p, 5);
  const uint32_t r1 = __builtin_amdgcn_alignbit(r, r, (uint32_t)turn);
  const uint32_t c1 = __builtin_amdgcn_alignbit(c, c, (uint32_t)turn);
  const uint32_t r2 = (r1 & kRingBlank) | (r & ~kRingBlank);
  const uint32_t c2 = (c1 & kRingBlank) | (c & ~kRingBlank);
  const uint32_t cr = __builtin_amdgcn_alignbit(r2, r2, (uint32_t)turn);
  const uint32_t cc = __builtin_amdgcn_alignbit(c2, c2, (uint32_t)turn);
  const uint32_t at_b = (m & kRingBase) + ((uint32_t)turn << 2);
  const __attribute__((address_space(3))) RingCell* cell =
      (const __attribute__((address_space(3))) RingCell*)(uintptr_t)(k.base + TABLE + (at_b & kRingCell));
  const uint32_t cmp = cell->cmp, legal = cell->legal;
  // the child's nearer moves; if its undo is one of them the move went away
  // from the goal and cost a unit of slack
  const uint32_t z = ((cr & kRingRows) | (cc & kRingCols)) + cmp;
  const uint32_t near = ring_bfi(z, k.ul, kRingR | kRingD);
  const uint32_t undo = k.undo << p;
  const uint32_t away = near & undo;
  const uint32_t base = at_b - min(away, kRingSlack1);
  const uint32_t cm = ring_meta(base, near, legal, undo);
  const uint32_t left = m ^ (k.top_bit >> p);
  const uint64_t lanes = FULL ? ~0ull : ring_uniform((kp >= 64 ? 0ull : 1ull << kp) - 1ull);
  const uint64_t kl = __builtin_amdgcn_uicmp(left, kRingBase, 34);                    // moves left
  const uint64_t kc = __builtin_amdgcn_uicmp(cm, kRingBase, 34) & lanes;               // child keeps some
  // goal: eight cells of the row plane first, the rest only where they agree
  const uint64_t g8 = ring_eq16(ring_goal<W>(true), cr);
  if (g8) {
    const bool g = (((cr ^ ring_goal<W>(true)) | (cc ^ ring_goal<W>(false))) & ~kRingBlank) == 0 && (base & kRingCell) == 0;
    goal |= __builtin_amdgcn_ballot_w64(g) & lanes;
  }
  const uint32_t mid = low + (uint32_t)__popcll(kl);
  ring_put2(kl, ring_at(kl, k.base + low * kRingEntry), r, c, left, kc, ring_at(kc, k.base + mid * kRingEntry), cr, cc,
            cm);
  WAVE_SYNC();
  return mid + (uint32_t)__popcll(kc);
}

}  // namespace bpida
