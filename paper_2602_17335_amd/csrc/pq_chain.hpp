// pq_chain.hpp -- finding the elements of a byte-stream chain side by side.
//
// Many streams of a page are chains: each element (a Snappy element, a
// hybrid run, a DELTA block, a length-prefixed string) is found only from the
// one before it.  A workgroup of NT threads finds the elements of a segment of
// NT 32-byte pieces, staged in LDS, without walking it front to back:
//   1. thread t takes piece t and finds, for each of its bytes as if an
//      element started there, where the chain from it leaves the piece
//      (backwards, so that each byte's answer follows from a later one's);
//   2. each wave follows these exits through its region of 64 pieces, from
//      each of the region's first 64 bytes;
//   3. one lane follows the true chain from region to region;
//   4. a lane per region follows it from piece to piece, which gives every
//      piece the first element that starts in it.
// An element that leaves the segment skips the bytes it covers.
#pragma once
#include "pq_device.hpp"

namespace pqk {

constexpr uint32_t CH_PIECE = 32;
constexpr uint32_t CH_STRIDE = CH_PIECE + 2;  // exit-table entries per piece (17 dwords: no bank conflicts)
constexpr uint32_t CH_CODES = 0xfff0u;        // exits from here on are codes:
constexpr uint32_t CH_BAD = 0xffffu;          // the chain meets an invalid element
constexpr uint32_t CH_LONG = 0xfffeu;         // it leaves by an element whose end does not fit the table
constexpr uint32_t CH_ODD = 0xfffdu;          // it meets an element the grammar does not decode
constexpr uint8_t CH_NONE = 0xff;             // no element starts in the piece
// what a grammar returns in place of an element's length
constexpr uint32_t STEP_BAD = 0, STEP_ODD = ~0u;

typedef uint32_t u32x4c __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) u32x4c lds_u32x4c;

// SLACK: bytes staged after the segment (a multiple of 16, 64 or more).
template <uint32_t NT, uint32_t SLACK>
struct ChainLds {
  static constexpr uint32_t SEG = NT * CH_PIECE;
  alignas(16) uint32_t in[(SEG + SLACK) / 4];
  uint16_t exit[NT * CH_STRIDE];
  uint32_t cand[NT / 64][64];
  uint32_t rent[NT / 64];
  uint32_t link[2];
  uint8_t pent[NT];

  // eight bytes from byte y of the staged segment
  __device__ __forceinline__ void bytes8(uint32_t y, uint32_t& lo, uint32_t& hi) const {
    const uint32_t j = y >> 2, w0 = in[j], w1 = in[j + 1], w2 = in[j + 2];
    lo = __builtin_amdgcn_alignbyte(w1, w0, y & 3);
    hi = __builtin_amdgcn_alignbyte(w2, w1, y & 3);
  }
  __device__ __forceinline__ uint32_t byte(uint32_t y) const { return (in[y >> 2] >> (8 * (y & 3))) & 0xffu; }
  __device__ __forceinline__ uint32_t exit_at(uint32_t y) const { return exit[(y >> 5) * CH_STRIDE + (y & 31)]; }

  // The segment at stream position S (a multiple of the piece) of a stream
  // whose bytes end at iend, base readable up to lim (a multiple of 16); the
  // true chain enters it at ip.  g(lo, hi, left, y) is the length of the
  // element at segment byte y (lo, hi: its first eight bytes; left: stream
  // bytes from it on), STEP_BAD or STEP_ODD.  Sets pent[] and returns the
  // position where the chain leaves the segment; code: 0, or CH_BAD or CH_ODD
  // when it meets such an element instead (which starts in its piece).
  // Every thread of the workgroup calls this; the tables are readable on
  // return, pent[] by the wave of its piece.
  template <class G>
  __device__ __forceinline__ uint32_t find(const G& g, const uint8_t* base, uint32_t lim, uint32_t S, uint32_t ip,
                                           uint32_t iend, uint32_t& code) {
    exits(g, base, lim, S, iend);
    return entries(g, S, ip, iend, code);
  }
  static constexpr uint32_t REG = 64 * CH_PIECE;
  // Steps 1 and 2.
  template <class G>
  __device__ __forceinline__ void exits(const G& g, const uint8_t* base, uint32_t lim, uint32_t S, uint32_t iend) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __syncthreads();  // the previous segment's tables are done with
    for (uint32_t i = tid; i < (SEG + SLACK) / 16; i += NT) {
      u32x4c v = {0u, 0u, 0u, 0u};
      if (S + 16 * i < lim) v = *reinterpret_cast<const u32x4c*>(base + S + 16 * i);
      *(lds_u32x4c*)((lds_u32*)&in[0] + 4 * i) = v;
    }
    __syncthreads();
    const uint32_t segend = min(SEG, iend - S);  // the chain ends the segment at or after this
    {
      uint32_t w[10];
#pragma unroll
      for (int c = 0; c < 10; ++c) w[c] = in[tid * (CH_PIECE / 4) + c];
      const uint32_t q0 = tid * CH_PIECE;
      uint16_t* ex = &exit[tid * CH_STRIDE];
#pragma unroll
      for (int k = (int)CH_PIECE - 1; k >= 0; --k) {
        const uint32_t lo = (k & 3) ? __builtin_amdgcn_alignbyte(w[(k >> 2) + 1], w[k >> 2], k & 3) : w[k >> 2];
        const uint32_t hi = (k & 3) ? __builtin_amdgcn_alignbyte(w[(k >> 2) + 2], w[(k >> 2) + 1], k & 3) : w[(k >> 2) + 1];
        const uint32_t y = q0 + (uint32_t)k;
        const uint32_t left = y < iend - S ? iend - S - y : 0u;
        const uint32_t st = left ? g(lo, hi, left, y) : STEP_BAD;
        const uint32_t nx = y + st;
        uint32_t v;
        if (st == STEP_BAD) v = CH_BAD;
        else if (st == STEP_ODD) v = CH_ODD;
        else if (nx >= q0 + CH_PIECE || nx >= segend) v = nx < CH_CODES ? nx : CH_LONG;
        else v = ex[nx - q0];
        ex[k] = (uint16_t)v;
      }
    }
    pent[tid] = CH_NONE;
    __syncthreads();
    {
      const uint32_t rend = min((wave + 1) * REG, segend);
      uint32_t e = wave * REG + lane;
      while (e < rend) e = exit_at(e);
      cand[wave][lane] = e;
    }
    __syncthreads();
  }
  // Where the chain from byte e of region r leaves the region; code is set
  // when it meets a bad or odd element instead.
  template <class G>
  __device__ __forceinline__ uint32_t leave(const G& g, uint32_t r, uint32_t e, uint32_t S, uint32_t iend,
                                            uint32_t& cd) const {
    const uint32_t rend = min((r + 1) * REG, min(SEG, iend - S));
    const uint32_t c = e - r * REG;
    uint32_t x;
    if (c < 64) {
      x = cand[r][c];
    } else {
      x = e;
      while (x < rend) x = exit_at(x);
    }
    if (x == CH_LONG) {
      // the last element that starts in the region, from its piece's entry
      uint32_t y = e;
      for (uint32_t z; (z = exit_at(y)) < rend;) y = z;
      for (;;) {
        uint32_t lo, hi;
        bytes8(y, lo, hi);
        const uint32_t nx = y + g(lo, hi, iend - S - y, y);
        if (nx >= CH_CODES || nx >= rend) return nx;
        y = nx;
      }
    }
    if (x >= CH_CODES) cd = x;
    return x;
  }
  // Where the chain from segment byte e leaves the segment (~0: it does not).
  template <class G>
  __device__ __forceinline__ uint32_t follow(const G& g, uint32_t e, uint32_t S, uint32_t iend) const {
    const uint32_t segend = min(SEG, iend - S);
    uint32_t cd = 0;
    while (e < segend) {
      e = leave(g, e / REG, e, S, iend, cd);
      if (cd) return ~0u;
    }
    return e;
  }
  // Steps 3 and 4.
  template <class G>
  __device__ __forceinline__ uint32_t entries(const G& g, uint32_t S, uint32_t ip, uint32_t iend, uint32_t& code) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t segend = min(SEG, iend - S);
    if (tid == 0) {
      uint32_t e = ip - S, cd = 0;
      for (uint32_t r = 0; r < NT / 64; ++r) {
        if (cd || e >= min((r + 1) * REG, segend)) { rent[r] = ~0u; continue; }
        rent[r] = e;  // (entries ascend, so e lies in region r)
        e = leave(g, r, e, S, iend, cd);
      }
      link[0] = S + e;
      link[1] = cd;
    }
    __syncthreads();
    if (lane == 0) {
      const uint32_t rend = min((wave + 1) * REG, segend);
      uint32_t y = rent[wave];
      while (y < rend) {
        pent[y >> 5] = (uint8_t)(y & 31);
        y = exit_at(y);
      }
    }
    wave_sync();
    code = link[1];
    return link[0];
  }
  // bytes of thread tid's piece that belong to the stream
  __device__ __forceinline__ uint32_t piece_len(uint32_t S, uint32_t iend) const {
    const uint32_t q = threadIdx.x * CH_PIECE, e = min(SEG, iend - S);
    return e > q ? min(CH_PIECE, e - q) : 0u;
  }
};

}  // namespace pqk
