// fbg_device.h -- gfx950 kernels for evaluating Boolean terms on the free
// generators (Section 2.3: d_j = t(b_1j .. b_nj) for every block j, each block
// computed bitwise; 2^r processors act as one 2^(k+r)-bit processor).
//
// One wave (64 lanes) evaluates one tile of 64*W 32-bit words per step; the
// index layout and the instruction format are described in fbg_isa.h.  The
// program is read with scalar loads (it is wave-uniform), generator words are
// synthesised in registers, and all bitwise work is VALU integer logic.
//
// Kernels:
//   k_eval<LOG2W, MODE, VAR>  one program, persistent grid-stride over tiles;
//                         MODE_COUNT   popcount -> wave sum -> 64-bit atomic
//                         MODE_DNF     store the words (coalesced)
//                         MODE_TILECNT per-tile model counts (enumeration 1)
//                         MODE_ENUM    ascending model indices (enumeration 2)
//                         VAR bit 0 (GEN): programs with more than clauses
//                         VAR bit 1 (COF): the uniform-cofactor variant, bit 2 (model
//                         counts per tile): its test in a launch before (k_cofactor_masks)
//   k_dnf_scan<MODE>      the two enumeration passes over a stored DNF vector
//   k_batch<LOG2W, VAR, MODE>  many programs, persistent waves popping work
//                         items (program, tiles t0 + k step) from eight
//                         device queues, one per XCD, with stealing; counts,
//                         and with MODE_DNF the DNF vectors too
//   k_tile_sums, k_tile_list  from per-tile counts the list of the tiles that
//                         hold models and their output positions
//   k_zero_*, k_set_u64   fills (used instead of memset so that a caller may
//                         capture the launches into a graph)
//
// The kernel templates live here; each eval_*.hip / batch.hip / misc.hip
// translation unit instantiates and launches its share of them, so that the
// library builds in parallel.
#ifndef FBG_DEVICE_H
#define FBG_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fbg_asm16.h"
#include "fbg_isa.h"
#include "fbg_kernels.h"

namespace fbg {
namespace dev {

enum { MODE_COUNT = 0, MODE_DNF = 1, MODE_TILECNT = 2, MODE_ENUM = 3 };

__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uni64(uint64_t x) {
  return uni((uint32_t)x) | (uint64_t)uni((uint32_t)(x >> 32)) << 32;
}

// Truth table of v_bitop3_b32(a, b, c): the function applied to the masks
// a = 0xF0, b = 0xCC, c = 0xAA.  kTT_AND_OR(T, acc, P) = acc & (T | P).
constexpr uint32_t kTT_AND_OR = 0xCCu & (0xF0u | 0xAAu);

// Program words are wave-uniform and never written by a kernel: reading them
// through the constant address space makes every fetch a scalar load.
typedef const __attribute__((address_space(4))) uint32_t *code_ptr;
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

// Lane part of a literal set: all-ones on the lanes whose bit is set in the
// 64-bit lane mask (a VCC-style mask, so this is one v_cndmask).
__device__ __forceinline__ uint32_t lane_part(uint64_t lanemask) {
  return __builtin_amdgcn_inverse_ballot_w64(lanemask) ? ~0u : 0u;
}

// ---- the general part of a program (after the clause prefix)
//
// Every operation on cur is one v_bitop3 per word whose truth table the
// encoder chose (w0 bits 8..15): inputs cur (0xF0), T or the register (0xCC)
// and the word pattern P(i) (0xAA).  The cases below are every table the
// encoder emits; a switch on a wave-uniform value costs a few scalar
// instructions, after which each word is a single VALU instruction.
#define FBG_LIT_TABLES(X) \
  X(0xEE) X(0x11) X(0x66) X(0x99) X(0xE0) X(0x10) X(0x60) X(0xFE) X(0xF1) X(0xF6) \
  X(0x1E) X(0xE1) X(0x96) X(0x1F) X(0xEF) X(0x9F) X(0x01) X(0x0E) X(0x09) X(0x69)
#define FBG_REG_TABLES(X) \
  X(0xC0) X(0x30) X(0xFC) X(0xF3) X(0x3C) X(0xC3) X(0x3F) X(0xCF) X(0x03) X(0x0C) X(0xCC) X(0x33)

// Any truth table, bit by bit (never reached with the encoder's tables).
__device__ __forceinline__ uint32_t bitop3_any(uint32_t a, uint32_t b, uint32_t c, uint32_t tt) {
  uint32_t r = 0;
#pragma unroll
  for (uint32_t m = 0; m < 8; m++) {
    if (!((tt >> m) & 1u)) continue;
    r |= ((m & 4u) ? a : ~a) & ((m & 2u) ? b : ~b) & ((m & 1u) ? c : ~c);
  }
  return r;
}

// cur = bitop3(cur, b, c) in place: the tied operand keeps cur in the same
// registers in every case of the dispatch, so the cases merge without copies.
#define FBG_BITOP3_INPLACE(d, b, c, tt) \
  asm("v_bitop3_b32 %0, %0, %1, %2 bitop3:" #tt : "+v"(d) : "v"(b), "s"(c))
#define FBG_BITOP3_INPLACE_2(d, b, tt) asm("v_bitop3_b32 %0, %0, %1, 0 bitop3:" #tt : "+v"(d) : "v"(b))

template <int W>
__device__ __forceinline__ void lit_op(uint32_t tt, uint32_t (&cur)[W], uint32_t T, const uint32_t (&P)[W]) {
  switch (tt) {
#define FBG_CASE(x)                                                                    \
  case x:                                                                              \
    _Pragma("unroll") for (int i = 0; i < W; i++) FBG_BITOP3_INPLACE(cur[i], T, P[i], x); \
    break;
    FBG_LIT_TABLES(FBG_CASE)
#undef FBG_CASE
    default:
#pragma unroll
      for (int i = 0; i < W; i++) cur[i] = bitop3_any(cur[i], T, P[i], tt);
  }
}

// The same for a literal set without word-index literals (P = 0 on every
// word): no pattern words are loaded.
template <int W>
__device__ __forceinline__ void lit_op0(uint32_t tt, uint32_t (&cur)[W], uint32_t T) {
  switch (tt) {
#define FBG_CASE(x)                                                                    \
  case x:                                                                              \
    _Pragma("unroll") for (int i = 0; i < W; i++) FBG_BITOP3_INPLACE_2(cur[i], T, x); \
    break;
    FBG_LIT_TABLES(FBG_CASE)
#undef FBG_CASE
    default:
#pragma unroll
      for (int i = 0; i < W; i++) cur[i] = bitop3_any(cur[i], T, 0u, tt);
  }
}

template <int W>
__device__ __forceinline__ void reg_op(uint32_t tt, uint32_t (&cur)[W], const uint32_t (&R)[W]) {
  switch (tt) {
#define FBG_CASE(x)                                                                    \
  case x:                                                                              \
    _Pragma("unroll") for (int i = 0; i < W; i++) FBG_BITOP3_INPLACE_2(cur[i], R[i], x); \
    break;
    FBG_REG_TABLES(FBG_CASE)
#undef FBG_CASE
    default:
#pragma unroll
      for (int i = 0; i < W; i++) cur[i] = bitop3_any(cur[i], R[i], 0u, tt);
  }
}

// Registers 0..kVgprRegs-1 live in VGPRs (selected by a wave-uniform switch);
// higher ones in LDS, W*64 words each (the launch sizes LDS for those only).
static_assert(kVgprRegs == 4, "the register switches below name registers 0..3");

// The VGPR state of the general part: cur and the first kVgprRegs
// registers.  A kernel keeps one per wave across all its tiles and clears it
// once: every program writes cur and a register before reading them, so a
// tile needs no reset.
template <int W>
struct GenState {
  uint32_t cur[W];
  uint32_t rv[kVgprRegs][W];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < W; i++) cur[i] = 0u;
#pragma unroll
    for (uint32_t r = 0; r < kVgprRegs; r++)
#pragma unroll
      for (int i = 0; i < W; i++) rv[r][i] = 0u;
  }
};

template <int LOG2W>
__device__ __forceinline__ void run_general(code_ptr w, const code_ptr table, uint32_t nins, uint64_t U0,
                                            uint32_t lane, uint32_t (&acc)[1 << LOG2W],
                                            GenState<1 << LOG2W> &st, uint32_t *__restrict__ regs) {
  constexpr int W = 1 << LOG2W;
  uint32_t (&cur)[W] = st.cur;
  uint32_t tmp[W];
  for (uint32_t pc = 0; pc < nins; ++pc, w += FBG_INS_WORDS) {
    const u32x8 ins = *(const __attribute__((address_space(4))) u32x8 *)w;
    const uint32_t w0 = ins[0];
    const uint32_t op = w0 & 15u;
    const uint32_t tt = (w0 >> FBG_F_SHIFT) & 0xFFu;
    if (op <= FBG_OP_OPL) {  // LDL / OPL (the encoder keeps CL in the clause block)
      const uint64_t lm = (uint64_t)ins[2] | ((uint64_t)ins[3] << 32);
      const uint64_t sel = (uint64_t)ins[4] | ((uint64_t)ins[5] << 32);
      uint32_t T;
      if (!(w0 & FBG_XORSET)) {
        const uint64_t neg = (uint64_t)ins[6] | ((uint64_t)ins[7] << 32);
        const uint64_t lmq = lm | (((U0 & sel) != neg) ? ~0ull : 0ull);
        T = __builtin_amdgcn_inverse_ballot_w64(lmq) ? ~0u : ins[1];
      } else {
        const uint32_t S = ins[1] ^ ((__popcll(U0 & sel) & 1) ? ~0u : 0u);
        T = lane_part(lm) ^ S;
      }
      if (w0 & FBG_HASPAT) {
        const code_ptr Pp = table + (w0 >> FBG_ARG_SHIFT);
        uint32_t P[W];
#pragma unroll
        for (int i = 0; i < W; i++) P[i] = Pp[i];
        lit_op<W>(tt, cur, T, P);
      } else {
        lit_op0<W>(tt, cur, T);
      }
      continue;
    }
    const uint32_t r = w0 >> FBG_ARG_SHIFT;
    switch (op) {
      case FBG_OP_ST:
        switch (r) {
#define FBG_ST(k) \
  case k:         \
    _Pragma("unroll") for (int i = 0; i < W; i++) st.rv[k][i] = cur[i]; \
    break;
          FBG_ST(0) FBG_ST(1) FBG_ST(2) FBG_ST(3)
#undef FBG_ST
          default: {
            uint32_t *R = regs + (size_t)(r - kVgprRegs) * (W * 64) + lane;
#pragma unroll
            for (int i = 0; i < W; i++) R[i * 64] = cur[i];
          }
        }
        if (w0 & FBG_INVOUT) {
#pragma unroll
          for (int i = 0; i < W; i++) cur[i] = ~cur[i];
        }
        break;
      case FBG_OP_OPR:
      case FBG_OP_LDR:
        switch (r) {
          case 0: reg_op<W>(tt, cur, st.rv[0]); break;
          case 1: reg_op<W>(tt, cur, st.rv[1]); break;
          case 2: reg_op<W>(tt, cur, st.rv[2]); break;
          case 3: reg_op<W>(tt, cur, st.rv[3]); break;
          default: {
            const uint32_t *R = regs + (size_t)(r - kVgprRegs) * (W * 64) + lane;
#pragma unroll
            for (int i = 0; i < W; i++) tmp[i] = R[i * 64];
            reg_op<W>(tt, cur, tmp);
          }
        }
        break;
      case FBG_OP_ACC:
        if (w0 & FBG_INV) {
#pragma unroll
          for (int i = 0; i < W; i++) acc[i] &= ~cur[i];
        } else {
#pragma unroll
          for (int i = 0; i < W; i++) acc[i] &= cur[i];
        }
        if (w0 & FBG_INVOUT) {
#pragma unroll
          for (int i = 0; i < W; i++) cur[i] = ~cur[i];
        }
        break;
      default:  // FBG_OP_NOT; an INVOUT on it (a folded second NOT) cancels it
        if (!(w0 & FBG_INVOUT)) {
#pragma unroll
          for (int i = 0; i < W; i++) cur[i] = ~cur[i];
        }
        break;
    }
  }
}

// One chunk of the clause block: the tile tests of its clauses (lane l takes
// clause l mod 32; one compare across the wave) and U, the clauses of the
// chunk that neither a lane nor a tile literal satisfies on this lane.
__device__ __forceinline__ uint32_t chunk_tile_bits(const uint32_t *__restrict__ ch, uint32_t nc, uint64_t U0,
                                                    uint32_t lane) {
  const uint32_t c = min(lane & (FBG_CB_CHUNK - 1u), nc - 1u);
  const uint4 td = *(const uint4 *)(ch + FBG_CB_CHUNK_HDR + 64 + 4 * c);
  const uint64_t sel = (uint64_t)td.x | ((uint64_t)td.y << 32);
  const uint64_t neg = (uint64_t)td.z | ((uint64_t)td.w << 32);
  return (uint32_t)__ballot((U0 & sel) != neg);
}

// Top bits of the runs (keys) of a chunk that meet U (fbg_isa.h).
__device__ __forceinline__ uint32_t runs_false(uint32_t U, uint32_t T, uint32_t F) {
  return (((U & ~T) + F) | U) & T;
}

// G & (m | ~x): v_bitop3 over (G = 0xF0, m = 0xCC, x = 0xAA).
constexpr uint32_t kTT_KEY = 0xF0u & (0xCCu | (~0xAAu & 0xFFu));
// m | ~x over (m = 0xF0, x = 0xCC).
constexpr uint32_t kTT_ORNOT = (0xF0u | (~0xCCu & 0xFFu)) & 0xFFu;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(4))) char *code_byte_ptr;

// The clause block (fbg_isa.h): the per-lane products G_g of the static
// groups chunk by chunk, acc from them by a product tree that also applies
// the keys of the first multi chunk at their levels, then any later multi
// chunk on the W words.
//
// STOP: once the product G_0 of the clauses without word literals is zero on
// every lane, acc is zero on the whole tile, whatever the other clauses are:
// false is returned and acc left unset.  Clauses made only of tile literals
// come first, then those of group 0, so a tile without models mostly ends within
// its first chunks.  Counting uses it, and the write-out of one general program
// (posets with a special element, 2^30 bits: 49 us, 38 so); that of clause programs does
// not (it waits for the stores, which the evaluation spreads out).  One count of
// a 3-CNF system of 136 clauses over 35 letters: 398 us to the end of every
// tile, 85 so, 58 with the tiles scattered over the waves (k_eval), 47 where a
// chunk of group 0 alone does not look for keys of the other groups, 27 where the
// waves of k_eval hold the first key (FirstKey; 32 to 42 with the host's part of a
// call, over several GPUs).
template <int LOG2W, bool STOP, bool BATCH = false>
__device__ __forceinline__ bool run_clauses(const uint32_t *__restrict__ cb_g, const code_ptr table, uint64_t U0,
                                            uint32_t lane, uint32_t (&acc)[1 << LOG2W]) {
  constexpr int W = 1 << LOG2W;
  constexpr int NG = 1 + 2 * LOG2W;
  const code_ptr cb = (code_ptr)cb_g;
  const uint32_t nstat = cb[1], nmulti = cb[2];
  uint32_t G[NG];
#pragma unroll
  for (int g = 0; g < NG; g++) G[g] = ~0u;
  const uint32_t *ch = cb_g + FBG_CB_HDR;
  for (uint32_t k = 0; k < nstat; ++k) {
    const code_ptr h = (code_ptr)ch;
    const u32x16 hd = *(const __attribute__((address_space(4))) u32x16 *)h;
    const uint32_t nc = hd[0];
    const uint32_t lb = ch[FBG_CB_CHUNK_HDR + lane];
    const uint32_t S = chunk_tile_bits(ch, nc, U0, lane);
    const uint32_t A = runs_false(~(lb | S), hd[2], hd[3]);
    // keys by group; hd[5 + g] is where group g's keys end (bytes)
    const code_byte_ptr hb = (code_byte_ptr)h;
    uint32_t off = (FBG_CB_CHUNK_HDR + 64 + 4 * nc) * 4;
    auto keys = [&](int g) __attribute__((always_inline)) {
      if (!STOP && !BATCH) {
        // the whole block runs: two keys to a scalar load, the second one without
        // effect where the group ends between them (128 MiB of a 3-CNF system's
        // vector 26.8 -> 25.7 us, 32 MiB 11.0 -> 10.9; a script with a general part
        // 50.5 -> 48.7; a count that mostly stops in its first chunk loses more to
        // the second compare than it gains)
        for (; off < hd[5 + g]; off += 16) {
          u32x4 km = *(const __attribute__((address_space(4))) u32x4 *)(hb + off);
          km[3] = off + 8 < hd[5 + g] ? km[3] : ~0u;
#pragma unroll
          for (int j = 0; j < 4; j += 2) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int)A, km[j], 1u);
            G[g] = __builtin_amdgcn_bitop3_b32(G[g], km[j + 1], x, kTT_KEY);
          }
        }
        off = hd[5 + g];
        return;
      }
      if (BATCH) {
        // the batched write-out in the XCD-local layout: pairs, then the odd key by
        // itself.  More code, which costs a lone vector up to 2^29 bits a microsecond
        // (2^28: 11.0, so 11.9) and the batched one at fewer words per lane a tenth (16
        // vectors of 2^32 bits at 16 words 1523 us, 1744), but the 16 at 32 words take
        // 1282 us and not 1315
        for (; off + 16 <= hd[5 + g]; off += 16) {
          const u32x4 km = *(const __attribute__((address_space(4))) u32x4 *)(hb + off);
#pragma unroll
          for (int j = 0; j < 4; j += 2) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int)A, km[j], 1u);
            G[g] = __builtin_amdgcn_bitop3_b32(G[g], km[j + 1], x, kTT_KEY);
          }
        }
      }
      for (; off < hd[5 + g]; off += 8) {
        const u32x2 km = *(const __attribute__((address_space(4))) u32x2 *)(hb + off);
        const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int)A, km[0], 1u);
        G[g] = __builtin_amdgcn_bitop3_b32(G[g], km[1], x, kTT_KEY);
      }
    };
    keys(0);
    ch += hd[1];
    // (leaving the look out for chunks without clauses of group 0 costs tiles that end at
    // their first key more than it saves: 256 layerings of posets 1458 us, so 1539)
    if (STOP) {
      if (__ballot(G[0] != 0u) == 0ull) return false;
      if (off >= hd[5 + NG - 1]) continue;  // a chunk of group 0 alone, as the first ones are
    }
#pragma unroll
    for (int g = 1; g < NG; g++) keys(g);
  }
  // the first multi chunk: its false runs now, its keys inside the tree
  u32x16 mh = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  uint32_t Am = 0, moff = 0;
  const code_byte_ptr mb = (code_byte_ptr)ch;
  if (nmulti) {
    mh = *(const __attribute__((address_space(4))) u32x16 *)ch;
    const uint32_t lb = ch[FBG_CB_CHUNK_HDR + lane];
    Am = runs_false(~(lb | chunk_tile_bits(ch, mh[0], U0, lane)), mh[2], mh[3]);
    moff = (FBG_CB_CHUNK_HDR + 64 + 4 * mh[0]) * 4;
  }
  // level j + 1 of the tree: the 2^(j+1) products of the words' low j + 1
  // bits; a multi key of level j + 1 acts on the nodes of its half
  acc[0] = G[0];
#pragma unroll
  for (int j = 0; j < LOG2W; j++) {
#pragma unroll
    for (int v = 0; v < (1 << j); v++) {
      acc[v | (1 << j)] = acc[v] & G[2 + 2 * j];
      acc[v] = acc[v] & G[1 + 2 * j];
    }
    if (j >= 1) {
#pragma unroll
      for (int half = 0; half < 2; half++) {
        for (; moff < mh[5 + 2 * (j - 1) + half]; moff += 16) {
          const u32x4 kq = *(const __attribute__((address_space(4))) u32x4 *)(mb + moff);
          const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int)Am, kq[0], 1u);
          const uint32_t T = __builtin_amdgcn_bitop3_b32(kq[1], x, 0u, kTT_ORNOT);
          const code_ptr P = table + kq[2];
#pragma unroll
          for (int v = 0; v < (1 << j); v++)
            acc[(half << j) | v] = __builtin_amdgcn_bitop3_b32(T, acc[(half << j) | v], P[v], kTT_AND_OR);
        }
      }
    }
  }
  // later multi chunks (more than 32 multi clauses): on the W words
  if (nmulti > 1) {
    ch += mh[1];
    for (uint32_t k = 1; k < nmulti; ++k) {
      const code_ptr h = (code_ptr)ch;
      const u32x16 hd = *(const __attribute__((address_space(4))) u32x16 *)h;
      const uint32_t nc = hd[0];
      const uint32_t lb = ch[FBG_CB_CHUNK_HDR + lane];
      const uint32_t A = runs_false(~(lb | chunk_tile_bits(ch, nc, U0, lane)), hd[2], hd[3]);
      const code_byte_ptr hb = (code_byte_ptr)h;
      for (uint32_t off = (FBG_CB_CHUNK_HDR + 64 + 4 * nc) * 4; off < hd[5]; off += 16) {
        const u32x4 kq = *(const __attribute__((address_space(4))) u32x4 *)(hb + off);
        const uint32_t x = (uint32_t)__builtin_amdgcn_sbfe((int)A, kq[0], 1u);
        const uint32_t T = __builtin_amdgcn_bitop3_b32(kq[1], x, 0u, kTT_ORNOT);
        const code_ptr P = table + kq[2];
#pragma unroll
        for (int i = 0; i < W; i++) acc[i] = __builtin_amdgcn_bitop3_b32(T, acc[i], P[i], kTT_AND_OR);
      }
      ch += hd[1];
    }
  }
  return true;
}

// The first key of the clause block where it is a run of clauses without in-word
// and word literals (tile literals alone come first): false on every lane of a
// tile, they leave no model there.  A wave that visits several tiles of a
// program holds it in registers, so that such a tile costs no load (run_clauses
// waits for the chunk's header, its lane words and the key, one after the other).
// Lane l holds one half of the tile selector of clause l mod 32, the low one
// below lane 32, the high one above.
// One count of 3-CNF systems (the launch alone): 35 letters, 136 clauses 46.8 us, with
// the key held 26.6; 32 letters, 60 clauses (8 tiles a wave) 37.7, 36.6; the models over 33
// letters, 150 clauses 39.4, 34.7.  Below kFirstKeyTiles tiles a wave its own loads
// cost what they save.  Not with a general part (posets with a special element, 8
// tiles a wave: 26.0, with it 27.0), nor in batches, where the item's program
// changes (16 systems of 2^32 valuations 169, 198; 256 DAGs 322, 334).
constexpr uint32_t kFirstKeyTiles = 4;
struct FirstKey {
  uint32_t lb, sel, neg;     // per lane
  uint32_t T, F, top;        // per wave
  bool any;
};

__device__ __forceinline__ FirstKey first_key(const uint32_t *__restrict__ cb_g, uint32_t lane) {
  FirstKey f = {0, 0, 0, 0, 0, 0, false};
  if (((code_ptr)cb_g)[1] == 0) return f;
  const uint32_t *ch = cb_g + FBG_CB_HDR;
  const u32x16 hd = *(const __attribute__((address_space(4))) u32x16 *)(code_ptr)ch;
  const uint32_t nc = hd[0], k0 = FBG_CB_CHUNK_HDR + 64 + 4 * nc;
  const u32x2 km = *(const __attribute__((address_space(4))) u32x2 *)((code_ptr)ch + k0);
  f.any = hd[5] > 4 * k0 && km[1] == 0u;
  f.T = hd[2], f.F = hd[3], f.top = km[0];
  const uint32_t *td = ch + FBG_CB_CHUNK_HDR + 64 + 4 * min(lane & (FBG_CB_CHUNK - 1u), nc - 1u) + (lane >> 5);
  f.lb = ch[FBG_CB_CHUNK_HDR + lane];
  f.sel = td[0], f.neg = td[2];
  return f;
}

__device__ __forceinline__ bool first_key_false(const FirstKey &f, uint64_t U0, uint32_t lane) {
  const uint32_t half = lane < 32u ? (uint32_t)U0 : (uint32_t)(U0 >> 32);
  const uint64_t b = __ballot((half & f.sel) != f.neg);
  const uint32_t A = runs_false(~(f.lb | (uint32_t)b | (uint32_t)(b >> 32)), f.T, f.F);
  return __ballot((A >> (f.top & 31u) & 1u) == 0u) == 0ull;
}

// The uniform-cofactor test of 64 tiles, lane l's is t (Tile: 32 bits where they hold
// every tile): a bit per lane, clear where a clause made only of tile literals is
// false, which makes the program false on the whole tile (acc only loses bits after
// the clause block), and on lanes that are not `valid`.  The table at the end of the
// clause block (fbg_isa.h) is read as scalars: three instructions per clause, eight
// clauses between two looks at the result, and the end as soon as no tile is left.
template <typename Tile>
__device__ __forceinline__ uint64_t tiles_alive(const uint32_t *__restrict__ cb_g, Tile t, uint64_t valid) {
  const code_ptr cb = (code_ptr)cb_g;
  uint64_t alive = valid;
  if (cb[1] == 0) return alive;
  const uint32_t k = (cb[FBG_CB_HDR + 4] + 7) / 8 * 8;
  const code_ptr td = cb + cb[0] - FBG_CB_COF_WORDS * k;
  for (uint32_t c = 0; c < k && alive != 0ull; c += 8) {
    u32x16 e[2];
#pragma unroll
    for (uint32_t j = 0; j < 2; j++)
      e[j] = *(const __attribute__((address_space(4))) u32x16 *)(td + FBG_CB_COF_WORDS * (c + 4 * j));
#pragma unroll
    for (uint32_t j = 0; j < 8; j++) {
      const u32x16 &v = e[j >> 2];
      const uint32_t i = 4 * (j & 3);
      const Tile sel = (Tile)((uint64_t)v[i] | (uint64_t)v[i + 1] << 32);
      const Tile neg = (Tile)((uint64_t)v[i + 2] | (uint64_t)v[i + 3] << 32);
      alive &= __ballot((t & sel) != neg);
    }
  }
  return alive;
}

// The same where the valid lanes' tiles are below `end`.
__device__ __forceinline__ uint64_t tiles_alive(const uint32_t *__restrict__ cb_g, uint64_t t, uint64_t valid,
                                                uint64_t end) {
  return end <= 1ull << 32 ? tiles_alive<uint32_t>(cb_g, (uint32_t)t, valid) : tiles_alive<uint64_t>(cb_g, t, valid);
}

// A bijection of [0, n): cycle-walking over a bijection of the bits-bit
// integers (2^bits >= n > 2^(bits - 1), mask = 2^bits - 1), two rounds of an
// xor-shift (invertible for a shift >= 1) and a multiplication by an odd
// constant (invertible modulo 2^bits).  The walk from x < n ends: following
// the permutation's cycle through x returns to x.
__device__ __forceinline__ uint64_t tile_hash(uint64_t x, uint64_t n, uint32_t bits, uint64_t mask) {
  const uint32_t h = bits > 1 ? bits >> 1 : 1u;
  do {
    x = ((x ^ (x >> h)) * 0x9E3779B97F4A7C15ull) & mask;
    x = ((x ^ (x >> h)) * 0xD6E8FEB86659FD93ull) & mask;
    x ^= x >> h;
  } while (x >= n);
  return x;
}

// The same for [0, 2^bits), the tiles of a program (beyond 2^32 of them k
// itself), with fewer instructions: an xor-shift, an odd multiplier, an xor-shift.
__device__ __forceinline__ uint64_t scatter_tile(uint64_t k, uint32_t bits) {
  if (bits > 32) return k;
  const uint32_t h = (bits + 1) / 2, mask = (uint32_t)((1ull << bits) - 1);
  uint32_t x = (uint32_t)k;
  x = ((x ^ (x >> h)) * 0x9E3779B1u) & mask;
  return x ^ (x >> h);
}

// Visit the tiles of group g (64 g .. 64 g + 63) within [t0, t1) that this part
// takes: of the tiles that pass the uniform-cofactor test, or (ALL) of all
// tiles, the dead ones with alive = false (all zeros, not to be evaluated),
// those whose running number r is `part` modulo mask + 1 (a power of two).
// That many waves share the group: its surviving tiles often come many
// together.  Returns the next running number.
template <bool ALL, typename Body>
__device__ __forceinline__ uint32_t visit_group(const uint32_t *__restrict__ code, uint32_t lane, uint64_t g,
                                                uint64_t t0, uint64_t t1, uint32_t r, uint32_t part, uint32_t mask,
                                                Body &&body) {
  const uint64_t first = g * 64;
  uint64_t valid = ~0ull;
  if (first < t0) valid &= ~0ull << (t0 - first);            // t0 < first + 64
  if (first + 64 > t1) valid &= ~0ull >> (first + 64 - t1);  // first < t1
  const uint64_t alive = tiles_alive(code, first + lane, valid, t1);
  for (uint64_t todo = ALL ? valid : alive; todo; r++, todo &= todo - 1) {
    if ((r & mask) != part) continue;
    const uint32_t l = (uint32_t)__builtin_ctzll(todo);
    body(first + l, ((alive >> l) & 1ull) != 0);
  }
  return r;
}

// Interpret one program over the W words of this lane in tile group U0: the
// clause block, then (GEN) the instructions after it.
// regs: this wave's LDS registers; at 16 words per lane the registers from
// lds_bytes on (byte offsets in the jump-table form) live in global memory at
// gregs instead (a block per wave).
// Returns false (acc all zero) when the tile was seen to hold no model before
// all of the program ran: with STOP in the clause block (run_clauses), and
// before the general part whenever the clauses leave no model, since acc only
// loses bits after them.  (Posets with a special element, 138 clauses and 41
// instructions over 30 letters, models in 1577 of 32768 tiles: 67 us, 29 so.)
template <int LOG2W, bool GEN, bool STOP, bool BATCH = false>
__device__ __forceinline__ bool run_program(const uint32_t *__restrict__ code_g, uint32_t nins, uint64_t U0,
                                            uint32_t lane, uint32_t (&acc)[1 << LOG2W],
                                            GenState<1 << LOG2W> &st, uint32_t *__restrict__ regs,
                                            uint32_t lds_bytes = 0, uint32_t *gregs = nullptr,
                                            uint32_t j16_any = 0) {
  constexpr int W = 1 << LOG2W;
  const code_ptr cb = (code_ptr)code_g;
  const code_ptr ins = cb + cb[0];
  const code_ptr table = ins + FBG_TABLE_OFFSET(nins, LOG2W);
  if constexpr (!GEN) return run_clauses<LOG2W, STOP, BATCH>(code_g, table, U0, lane, acc);
  // programs without clauses (most general programs) skip the block and its
  // product tree: acc starts all-ones (wave-uniform test)
  if (cb[1] + cb[2] == 0) {
#pragma unroll
    for (int i = 0; i < W; i++) acc[i] = ~0u;
  } else {
    bool live = run_clauses<LOG2W, STOP>(code_g, table, U0, lane, acc);
    if (live) {
      uint32_t any = 0;
#pragma unroll
      for (int i = 0; i < W; i++) any |= acc[i];
      live = __ballot(any != 0u) != 0ull;
    }
    if (!live) {
#pragma unroll
      for (int i = 0; i < W; i++) acc[i] = 0u;
      return false;
    }
  }
  if constexpr (LOG2W == FBG_J16_LOG2W) {
    // the jump-table form; LDS registers at this wave's block, 64 bytes a lane
    const uint32_t lds_lane =
        (uint32_t)(uintptr_t)((__attribute__((address_space(3))) uint32_t *)regs) + lane * 64u;
    run_general_j16((const uint32_t *)(uintptr_t)ins, (const uint32_t *)(uintptr_t)table, U0, lds_lane, lds_bytes,
                    gregs, lane, acc, j16_any);
  } else {
    run_general<LOG2W>(ins, table, nins, U0, lane, acc, st, regs);
  }
  return true;
}

// Store a tile of the XCD-local layout (fbg_kernels.h): the program's
// renamed variables put the lane's words 4g .. 4g+3 side by side, so each
// group is one 16-byte store to 1 KiB unit g & 3 of the tile's piece g >> 2
// (the second piece 8 pieces, 32 KiB, after the first).  dst = the first
// piece + 4 lane words, 16-byte aligned.  (Instantiated for every W; called
// at W = 32 only.)
template <int W>
__device__ __forceinline__ void store_xcd_tile(const uint32_t (&acc)[W], uint32_t *dst) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int g = 0; g < W / 4; g++) {
    const u32x4 v = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    __builtin_nontemporal_store(v, (u32x4 *)(dst + (g >> 2) * 8192 + (g & 3) * 256));
  }
}

// Zero the words of this lane that lie beyond the valuation space.
template <int LOG2W>
__device__ __forceinline__ void mask_tail(uint32_t (&acc)[1 << LOG2W], uint64_t U0, uint32_t lane,
                                          uint64_t nslices, int n) {
  constexpr int W = 1 << LOG2W;
  if ((U0 + W) * 64 > nslices) {  // wave-uniform
    // valid words of the tile, at most 64 W: 32-bit compares per word
    const uint64_t base = U0 * 64;
    const uint32_t rem = (uint32_t)min(nslices > base ? nslices - base : 0ull, (unsigned long long)W * 64);
    // word i of this lane is valid when 64 i + lane < rem, i.e. when
    // d = rem - lane exceeds 64 i: one VGPR and an immediate per word, no
    // per-word lane constants kept across the tile loop
    const int d = (int)rem - (int)lane;
#pragma unroll
    for (int i = 0; i < W; i++) acc[i] = d > 64 * i ? acc[i] : 0u;
    if (n < FBG_SLICE_BITS) acc[0] &= (uint32_t)((1ull << (1u << n)) - 1u);
  }
}

// Wave sums.  ds_swizzle exchanges within each half of the wave with the
// lane pattern in the instruction (no address registers to keep live across
// the tile loop); the two halves meet through v_readlane.  The result is
// wave-uniform.
template <int XOR>
__device__ __forceinline__ uint32_t swz_xor(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (XOR << 10));
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  v += swz_xor<16>(v);
  v += swz_xor<8>(v);
  v += swz_xor<4>(v);
  v += swz_xor<2>(v);
  v += swz_xor<1>(v);
  return (uint32_t)__builtin_amdgcn_readlane(v, 0) + (uint32_t)__builtin_amdgcn_readlane(v, 32);
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#define FBG_SUM_STEP(x)                                                   \
  {                                                                       \
    const uint64_t t = ((uint64_t)hi << 32 | lo) +                        \
                       ((uint64_t)swz_xor<x>(hi) << 32 | swz_xor<x>(lo)); \
    lo = (uint32_t)t;                                                     \
    hi = (uint32_t)(t >> 32);                                             \
  }
  FBG_SUM_STEP(16) FBG_SUM_STEP(8) FBG_SUM_STEP(4) FBG_SUM_STEP(2) FBG_SUM_STEP(1)
#undef FBG_SUM_STEP
  // readlane returns int: widen through uint32_t, never by sign extension
  const uint64_t a = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, 0) << 32 |
                     (uint32_t)__builtin_amdgcn_readlane(lo, 0);
  const uint64_t b = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, 32) << 32 |
                     (uint32_t)__builtin_amdgcn_readlane(lo, 32);
  return a + b;
}

// The sum over a block's waves of a per-lane value, for every thread (part: a
// word pair per wave).
__device__ __forceinline__ uint64_t block_sum_u64(uint64_t v, uint64_t *part, uint32_t lane, uint32_t wib,
                                                  uint32_t wpb) {
  v = wave_sum_u64(v);
  if (lane == 0) part[wib] = v;
  __syncthreads();
  uint64_t s = 0;
  for (uint32_t w = 0; w < wpb; w++) s += part[w];
  return s;
}

// Inclusive prefix sum over the 64 lanes: four row shifts and two row
// broadcasts on the VALU (DPP), against six dependent LDS permutes of a
// __shfl_up scan.  Every lane must be active.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
#define FBG_DPP(x, ctrl, rows) (uint32_t) __builtin_amdgcn_update_dpp(0, (int)(x), ctrl, rows, 0xF, false)
  v += FBG_DPP(v, 0x111, 0xF);  // row_shr:1
  v += FBG_DPP(v, 0x112, 0xF);  // row_shr:2
  v += FBG_DPP(v, 0x114, 0xF);  // row_shr:4
  v += FBG_DPP(v, 0x118, 0xF);  // row_shr:8
  v += FBG_DPP(v, 0x142, 0xA);  // row_bcast:15 into rows 1 and 3
  v += FBG_DPP(v, 0x143, 0xC);  // row_bcast:31 into rows 2 and 3
#undef FBG_DPP
  return v;
}

// Enumeration epilogues shared by the evaluator and the stored-DNF path.  A
// unit of the two passes is 2^-shift of a tile: W >> shift rows, at least four
// of them when shift > 0.

// The model counts of a tile's units to dst[0 ..].
template <int LOG2W>
__device__ __forceinline__ void tile_count_out(const uint32_t (&acc)[1 << LOG2W], uint32_t lane, uint32_t shift,
                                               uint32_t *dst) {
  constexpr uint32_t W = 1u << LOG2W, STEP = W < 4 ? W : 4;
  const uint32_t rows = W >> shift;
  uint32_t c = 0;
#pragma unroll
  for (uint32_t i = 0; i < W; i++) {
    c += __popc(acc[i]);
    if ((i + 1) % STEP == 0 && ((i + 1) & (rows - 1)) == 0) {  // wave-uniform: the unit's last row
      const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(c), 63);
      if (lane == 0) dst[i >> (LOG2W - shift)] = sum;
      c = 0;
    }
  }
}

// LDS traffic of a wave with itself: the compiler moves nothing across (the
// words may also hold registers of the general part), and the hardware keeps a
// wave's LDS accesses in order.
__device__ __forceinline__ void wave_lds_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2), aligned(8)));

// The models of rows [r0, r0 + rows) of a tile, ascending, to out[base ..]
// (below capacity).  stage: this wave's kStageModels LDS entries.
//
// What bounds it is instruction issue and the fullest unit, then the stores.
// Words ascend with (i, lane); each row i is ranked across the lanes (by its
// ballot when no word holds two models, by a prefix sum of the popcounts
// otherwise).  Stored straight from the words, every model is a lane's 8-byte
// store at its own place; the offsets in the tile (16 bits: a tile has at most
// 2^16 valuations) are gathered in LDS instead and leave 64 consecutive indices
// (512 bytes) to a store.  Triangle-free graphs, n = 28 (32768 units of four
// rows, 3.5 M models): 17 us, with whole tiles of 16 rows 44 us (the models
// crowd into few tiles, 12,626 in one), the scattered stores took 94 us.
// Giving every lane one model a step instead (a search for the word that owns
// it) measured slower: 21 us.  Units past the capacity are left out: the
// first 10 of the 45 M models of 3 clauses over 26 letters took 68 us with all of them
// gathered, 18 so.
template <int LOG2W>
__device__ __forceinline__ void tile_compact(const uint32_t (&acc)[1 << LOG2W], uint32_t r0, uint32_t rows,
                                             uint64_t U0, uint32_t lane, uint64_t base, uint64_t *out,
                                             uint64_t capacity, uint16_t *stage) {
  const uint64_t vbase = U0 * 2048;
  uint32_t fill = 0;
  // two models a lane and step: a wave stores 1 KiB at once
  auto flush = [&]() __attribute__((always_inline)) {
    wave_lds_fence();
    const uint32_t lim = (uint32_t)min((unsigned long long)fill, capacity > base ? capacity - base : 0ull);
    uint64_t *dst = out + base;
    for (uint32_t k = 2 * lane; k < lim; k += 128) {
      const u16x2 o = *(const u16x2 *)(stage + k);
      if (k + 1 < lim)
        *(u64x2 *)(dst + k) = u64x2{vbase + o[0], vbase + o[1]};
      else
        dst[k] = vbase + o[0];
    }
    wave_lds_fence();
    base += fill;
    fill = 0;
  };
#pragma unroll
  for (int i = 0; i < (1 << LOG2W); i++) {
    if ((uint32_t)i - r0 >= rows) continue;  // wave-uniform: not a row of this unit
    uint32_t x = acc[i];
    const uint64_t any = __ballot(x != 0u);
    if (any == 0ull) continue;  // wave-uniform: no model in this word of any lane
    uint32_t before, row;       // models of the row on lower lanes; of the whole row (at most 2048)
    if (__ballot((x & (x - 1u)) != 0u) == 0ull) {
      before = __builtin_amdgcn_mbcnt_hi((uint32_t)(any >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)any, 0u));
      row = (uint32_t)__popcll(any);
    } else {
      const uint32_t c = __popc(x);
      const uint32_t incl = wave_inclusive_scan(c);
      before = incl - c;
      row = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    if (fill + row > kStageModels) flush();
    uint32_t pos = fill + before;
    while (x) {
      stage[pos++] = (uint16_t)((i * 64 + lane) * 32 + (uint32_t)__builtin_ctz(x));
      x &= x - 1u;
    }
    fill += row;
  }
  flush();
}

// Compaction passes find the output position of a unit's models in one of two
// ways (the host chooses, capi.cpp):
//  - at most a block's waves' worth of units (ENUM_ONE_BLOCK): one launch of one
//    block, a unit per wave, no counting pass and no temporaries; the waves
//    rank themselves (one_block_position).  Models of a theory over 15 letters:
//    14 us a call with the two passes, 6.6 so.
//  - few units (ENUM_DIRECT): block b takes the units [b wpb, (b + 1) wpb), one per
//    wave, and adds up the counts of all units before them itself (their sums
//    per block where the counting pass left them, a.block_sums); no scan kernel
//    runs.  The last block writes the total.
//  - many units: the waves share out the list of units that hold models, with
//    the positions k_tile_list found.
// body(u, position) for each of this wave's units that holds models.
template <typename Body>
__device__ __forceinline__ void for_model_units(const EvalArgs &a, uint32_t lane, uint32_t wib, uint32_t wpb,
                                                uint64_t *part, Body &&body) {
  // the steps this wave takes: one unit of the block, or entries of the list
  uint64_t k = (uint64_t)blockIdx.x * wpb + wib, step = (uint64_t)gridDim.x * wpb, n, at = 0;
  if (a.direct == ENUM_ONE_BLOCK) {
    n = wpb;  // also waves without a tile, for the barrier
  } else if (a.direct) {
    n = a.nunits;
    const uint32_t first = blockIdx.x * wpb;
    const uint32_t c = lane < wpb && first + lane < (uint32_t)n ? a.tile_counts[first + lane] : 0u;
    const bool last = blockIdx.x == gridDim.x - 1;
    if (__ballot(c != 0u) == 0ull && !last) return;  // the same for every wave of the block
    const uint32_t *in = a.block_sums ? a.block_sums : a.tile_counts;  // padded to 256 bytes
    const uint32_t m = a.block_sums ? blockIdx.x : first;
    uint64_t s = 0;
    for (uint32_t i = threadIdx.x * 4; i < m; i += blockDim.x * 4) {
      const uint4 v = *(const uint4 *)(in + i);
      // at most 16 x 2^16: 32 bits
      s += v.x + (i + 1 < m ? v.y : 0u) + (i + 2 < m ? v.z : 0u) + (i + 3 < m ? v.w : 0u);
    }
    s = wave_sum_u64(s);
    if (lane == 0) part[wib] = s;
    __syncthreads();
    for (uint32_t w = 0; w < wpb; w++) at += part[w];
    const uint32_t incl = wave_inclusive_scan(c);
    if (last && threadIdx.x == 0) *a.out_count = at + (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    at += (uint32_t)__builtin_amdgcn_readlane((int)(incl - c), (int)wib);
    if (at >= a.capacity || __builtin_amdgcn_readlane((int)c, (int)wib) == 0) return;
  } else {
    n = *a.nlist;
  }
  for (; k < n; k += step) {
    uint64_t u = k;  // (beyond 2^32 units in large programs at few words per lane)
    if (!a.direct) {
      const uint64_t e = uni64(a.list[k]);
      u = list_tile(e);
      at = a.list_base[u / kListBlock] + list_before(e);
      if (at >= a.capacity) return;  // the list ascends: nor do the later ones have room
    }
    body(u, at);
  }
}

// ENUM_ONE_BLOCK: the position of this wave's models among those of the block's
// waves; the first thread writes the total.
template <int LOG2W>
__device__ __forceinline__ uint64_t one_block_position(const uint32_t (&acc)[1 << LOG2W], const EvalArgs &a,
                                                       uint64_t *part, uint32_t lane, uint32_t wib, uint32_t wpb) {
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < (1 << LOG2W); i++) c += __popc(acc[i]);
  c = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(c), 63);
  if (lane == 0) part[wib] = c;
  __syncthreads();
  uint64_t at = 0, total = 0;
  for (uint32_t w = 0; w < wpb; w++) {
    if (w < wib) at += part[w];
    total += part[w];
  }
  if (threadIdx.x == 0) *a.out_count = total;
  return at;
}

// DNF write-out and count of one tile: the words past the valuation space
// are cleared (only the single tile of a program smaller than one tile has
// any), the words inside the output stored, and the models of this lane
// counted.  A whole tile's stores are issued unconditionally (streaming: the
// vector is not read back by this kernel).
template <int LOG2W>
__device__ __forceinline__ uint32_t store_count_tile(const uint32_t (&acc)[1 << LOG2W], uint64_t U0, uint32_t lane,
                                                     uint64_t nslices, int n, uint32_t *out32, uint64_t out_slices) {
  constexpr int W = 1 << LOG2W;
  uint32_t *dst = out32 + U0 * 64 + lane;
  uint32_t c = 0;
  if ((U0 + W) * 64 <= nslices) {  // wave-uniform; out_slices >= nslices
#pragma unroll
    for (int i = 0; i < W; i++) {
      __builtin_nontemporal_store(acc[i], dst + i * 64);
      c += __popc(acc[i]);
    }
  } else {
    const uint64_t base = U0 * 64;
    const uint32_t rem = (uint32_t)min(nslices > base ? nslices - base : 0ull, (unsigned long long)W * 64);
    const uint32_t rem_out = (uint32_t)min(out_slices > base ? out_slices - base : 0ull, (unsigned long long)W * 64);
    const uint32_t m0 = n < FBG_SLICE_BITS ? (uint32_t)((1ull << (1u << n)) - 1u) : ~0u;
#pragma unroll
    for (int i = 0; i < W; i++) {
      // word (i, lane) of the tile is valid when lane < rem - 64 i (a
      // wave-uniform bound: no per-word lane constants)
      uint32_t v = (int)lane < (int)rem - 64 * i ? acc[i] : 0u;
      if (i == 0) v &= m0;
      if ((int)lane < (int)rem_out - 64 * i) dst[i * 64] = v;
      c += __popc(v);
    }
  }
  return c;
}

// Store the W words of this lane; the stores of a whole tile are issued
// unconditionally (streaming: the vector is not read back by this kernel).
template <int LOG2W>
__device__ __forceinline__ void store_tile(const uint32_t (&acc)[1 << LOG2W], uint64_t U0, uint32_t lane,
                                           uint32_t *out32, uint64_t out_slices) {
  constexpr int W = 1 << LOG2W;
  uint32_t *dst = out32 + U0 * 64 + lane;
  if ((U0 + W) * 64 <= out_slices) {  // wave-uniform
#pragma unroll
    for (int i = 0; i < W; i++) __builtin_nontemporal_store(acc[i], dst + i * 64);
  } else {
#pragma unroll
    for (int i = 0; i < W; i++)
      if ((U0 + i) * 64 + lane < out_slices) dst[i * 64] = acc[i];
  }
}

// Waves per SIMD each evaluator instance is compiled for (its VGPR budget),
// as many as fit without spilling: programs made of clauses alone fit 8
// (<= 64 VGPRs), the uniform-cofactor variant 7 at W = 32; the general
// interpreter 6 at W <= 8, 4 at W = 16 (124 VGPRs: cur, acc and four
// registers per word) and 2 at W = 32 (left unconstrained it takes a few registers
// more than two waves have: posets with a special element 78 us, so 56; the batched
// write-out would spill).
constexpr int min_waves(int log2w, int var) {
  return (var & 1) ? (log2w <= 3 ? 6 : (log2w == 4 ? 4 : 2)) : ((var & 2) && log2w == 5 ? 7 : 8);
}

template <int LOG2W, int MODE, int VAR>
__global__ __launch_bounds__(256, min_waves(LOG2W, VAR)) void k_eval(EvalArgs a) {
  constexpr int W = 1 << LOG2W;
  extern __shared__ __align__(16) uint32_t lds[];  // (the static words come first)
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wib = uni(threadIdx.x) >> 6;
  const uint32_t wpb = blockDim.x >> 6;
  uint32_t *regs = lds + (size_t)wib * (MODE == MODE_ENUM ? a.lds_stride : a.nregs * (W * 64));
  const uint64_t wave = (uint64_t)blockIdx.x * wpb + wib;
  const uint64_t nwaves = (uint64_t)gridDim.x * wpb;
  uint64_t total = 0;
  GenState<W> st;
  if (VAR & 1) st.clear();
  __shared__ uint64_t part[4];
  if (MODE == MODE_ENUM) {
    // (the cofactor variant is not needed here: these tiles hold models)
    for_model_units(a, lane, wib, wpb, part, [&](uint64_t u, uint64_t at) __attribute__((always_inline)) {
      const uint64_t U0 = u >> a.unit_shift << LOG2W;
      const uint32_t rows = W >> a.unit_shift, r0 = ((uint32_t)u & ((1u << a.unit_shift) - 1u)) * rows;
      uint32_t acc[W];
      run_program<LOG2W, (VAR & 1) != 0, false>(a.code, a.nins, U0, lane, acc, st, regs, a.nregs * (W * 256u),
                                                nullptr, a.j16_any);
      mask_tail<LOG2W>(acc, U0, lane, a.nslices, a.n);
      if (a.direct == ENUM_ONE_BLOCK) at = one_block_position<LOG2W>(acc, a, part, lane, wib, wpb);
      tile_compact<LOG2W>(acc, r0, rows, U0, lane, at, a.out_idx, a.capacity, (uint16_t *)regs);
    });
    return;
  }
  // dead tiles (uniform cofactor) still write their zeros in DNF mode;
  // counting skips them, and so does the tile-count pass, whose counts the
  // host clears beforehand
  constexpr bool ALL = MODE == MODE_DNF;
  FirstKey fk = {0, 0, 0, 0, 0, 0, false};
  if constexpr (MODE != MODE_DNF && VAR == 0)
    if (a.ntiles >= kFirstKeyTiles * nwaves) fk = first_key(a.code, lane);
  auto tile = [&](uint64_t t, bool alive) __attribute__((always_inline)) {
    const uint64_t U0 = t << LOG2W;
    uint32_t acc[W];
    if (LOG2W == 5 && VAR == 0 && MODE == MODE_DNF && a.xcd_code) {
      // XCD-local layout (fbg_kernels.h): full tiles only (n >= 21), output
      // 16-byte aligned
      run_program<LOG2W, false, false>(a.xcd_code, a.nins, U0, lane, acc, st, regs);
      store_xcd_tile(acc, a.out32 + (((t >> 2) & 7) + 16 * (t & 3) + 64 * (t >> 5)) * 1024 + lane * 4);
      return;
    }
    if (alive) {
      bool live = MODE == MODE_DNF || VAR != 0 || !fk.any || !first_key_false(fk, U0, lane);
      if (live)
        live = run_program<LOG2W, (VAR & 1) != 0, MODE != MODE_DNF || (VAR & 1) != 0>(
            a.code, a.nins, U0, lane, acc, st, regs, a.nregs * (W * 256u), nullptr, a.j16_any);
      if (MODE != MODE_DNF && !live) {
        if (MODE == MODE_TILECNT && lane < (1u << a.unit_shift)) a.tile_counts[(t << a.unit_shift) + lane] = 0u;
        return;
      }
      mask_tail<LOG2W>(acc, U0, lane, a.nslices, a.n);
    } else {
#pragma unroll
      for (int i = 0; i < W; i++) acc[i] = 0u;
    }
    if (MODE == MODE_COUNT) {
      uint32_t c = 0;
#pragma unroll
      for (int i = 0; i < W; i++) c += __popc(acc[i]);
      total += c;
    } else if (MODE == MODE_DNF) {
      store_tile<LOG2W>(acc, U0, lane, a.out32, a.out_slices);
    } else {
      tile_count_out<LOG2W>(acc, lane, a.unit_shift, a.tile_counts + (t << a.unit_shift));
    }
  };
  if constexpr ((VAR & 2) != 0) {
    if constexpr ((VAR & 4) != 0) {
      // The tests are done (k_cofactor_masks).  A wave looks at 64 groups, a mask
      // per lane, and takes every 2^part_shift-th of their live
      // tiles: mostly one tile or none.  Equivalence relations on 9 elements (825
      // live tiles of 2^20, up to 12 in a group): the enumeration 40.7 us, with the test
      // in the wave, whose three evaluations in a row took 9 us each, 53.4.
      // (2^18 <= ntiles <= 2^38, a power of two)
      const uint32_t nsets = (uint32_t)(a.ntiles >> 12), sets = 31u - (uint32_t)__builtin_clz(nsets);
      const uint32_t pm = (1u << a.part_shift) - 1u;
      for (uint64_t x = wave; x < (uint64_t)nsets << a.part_shift; x += nwaves) {
        const uint32_t set = (uint32_t)x & (nsets - 1u), part_no = (uint32_t)(x >> sets);
        // live groups share index bits, high or low: scattered
        const uint32_t g = (uint32_t)scatter_tile((uint64_t)lane * nsets + set, sets + 6u);
        const uint64_t m = a.masks[g];
        uint32_t r = 0;
        for (uint64_t b = __ballot(m != 0ull); b; b &= b - 1) {
          const uint32_t l = (uint32_t)__builtin_ctzll(b);
          uint64_t todo = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, l) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), l) << 32;
          for (; todo; r++, todo &= todo - 1)
            if ((r & pm) == part_no)
              tile((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)g, l) * 64 + (uint32_t)__builtin_ctzll(todo), true);
        }
      }
    } else {
      // 64 tiles of the wave at a time, one per lane.  The k-th tile of the launch is taken
      // at a hash of k: live tiles share their low index bits, and a power-of-two stride
      // would give them all to a few waves.
      uint32_t bits = 0;
      while ((1ull << bits) < a.ntiles) bits++;
      const uint64_t hmask = (1ull << bits) - 1;
      for (uint64_t k = wave; k < a.ntiles; k += nwaves * 64) {
        const uint64_t kl = k + lane * nwaves;
        const uint64_t valid = __ballot(kl < a.ntiles);
        const uint64_t tl = kl < a.ntiles ? tile_hash(kl, a.ntiles, bits, hmask) : 0ull;
        const uint64_t alive = tiles_alive(a.code, tl, valid, a.ntiles);
        for (uint64_t todo = ALL ? valid : alive; todo; todo &= todo - 1) {
          const uint32_t l = (uint32_t)__builtin_ctzll(todo);
          const uint64_t t = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)tl, l) |
                             (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(tl >> 32), l) << 32;
          tile(t, ((alive >> l) & 1ull) != 0);
        }
      }
    }
  } else if constexpr (MODE != MODE_DNF) {
    // tiles that hold models share index bits too, and evaluating one takes
    // several times as long as stopping early (run_clauses)
    const uint32_t bits = 63u - (uint32_t)__builtin_clzll(a.ntiles | 1u);
    for (uint64_t k = wave; k < a.ntiles; k += nwaves) tile(scatter_tile(k, bits), true);
  } else {
    for (uint64_t t = wave; t < a.ntiles; t += nwaves) tile(t, true);
  }
  if (MODE == MODE_COUNT) {
    // one atomic per block: they meet at one address, 12 ns each (triangle-free
    // graphs, n = 28, 2384 of 8192 waves with models: 29 of 36 us with one per
    // wave).  A launch of one block stores its sum: nothing clears the count.
    const uint64_t s = block_sum_u64(total, part, lane, wib, wpb);
    if (threadIdx.x == 0) {
      if (gridDim.x == 1)
        *a.out_count = s;
      else if (s)
        atomicAdd((unsigned long long *)a.out_count, (unsigned long long)s);
    }
  }
}

// Enumeration over a stored DNF vector: tiles of 64 W words laid out as the
// evaluator's (a unit is a tile here); a.out32 is the DNF (read only here).
// The counting pass runs at the rate of HBM (2^30 bits: 20 us, 6.7 TB/s).  With
// a.block_sums its blocks take a tile per wave and leave their sums as well, so
// that a block of the compaction pass adds up a quarter as many numbers (16384
// tiles: 9 us of a pass of 25 us went there).
template <int LOG2W, int MODE>
__global__ __launch_bounds__(256) void k_dnf_scan(EvalArgs a) {
  constexpr int W = 1 << LOG2W;
  __shared__ uint64_t part[4];
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wib = uni(threadIdx.x) >> 6;
  const uint32_t wpb = blockDim.x >> 6;
  auto load = [&](uint64_t U0, uint32_t (&acc)[W]) __attribute__((always_inline)) {
    const uint32_t *src = a.out32 + U0 * 64 + lane;
    if ((U0 + W) * 64 <= a.nslices) {  // wave-uniform: a whole tile, every load issued at once
#pragma unroll
      for (int i = 0; i < W; i++) acc[i] = __builtin_nontemporal_load(src + i * 64);
    } else {
#pragma unroll
      for (int i = 0; i < W; i++) {
        const uint64_t s = (U0 + i) * 64 + lane;
        acc[i] = s < a.nslices ? src[i * 64] : 0u;
      }
    }
  };
  if (MODE == MODE_ENUM) {
    __shared__ __align__(4) uint16_t stage[4][kStageModels];
    for_model_units(a, lane, wib, wpb, part, [&](uint64_t u, uint64_t at) __attribute__((always_inline)) {
      uint32_t acc[W];
      const uint64_t U0 = u << LOG2W;
      load(U0, acc);
      if (a.direct == ENUM_ONE_BLOCK) at = one_block_position<LOG2W>(acc, a, part, lane, wib, wpb);
      tile_compact<LOG2W>(acc, 0u, W, U0, lane, at, a.out_idx, a.capacity, stage[wib]);
    });
    return;
  }
  const uint64_t wave = (uint64_t)blockIdx.x * wpb + wib;
  const uint64_t nwaves = (uint64_t)gridDim.x * wpb;
  uint32_t c = 0;
  for (uint64_t t = wave; t < a.ntiles; t += nwaves) {
    uint32_t acc[W];
    load(t << LOG2W, acc);
    c = 0;
#pragma unroll
    for (int i = 0; i < W; i++) c += __popc(acc[i]);
    c = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(c), 63);
    if (lane == 0) a.tile_counts[t] = c;
  }
  if (a.block_sums) {  // one tile per wave
    if (lane == 0) part[wib] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t sum = 0;
      for (uint32_t w = 0; w < wpb; w++) sum += (uint32_t)part[w];
      a.block_sums[blockIdx.x] = sum;
    }
  }
}

// ---------------------------------------------------------------- batches

// MODE_COUNT adds each program's model count into its slot; MODE_DNF also
// writes the program's DNF vector (BatchProg.out32).  The item and program
// tables are read-only during the launch: scalar loads, so tile indices and
// code pointers stay wave-uniform.
template <int LOG2W, int VAR, int MODE>
__global__ __launch_bounds__(256, (VAR & 1) && LOG2W == 5 && MODE == MODE_DNF ? 1 : min_waves(LOG2W, VAR)) void k_batch(
    BatchArgs a) {
  constexpr int W = 1 << LOG2W;
  extern __shared__ __align__(16) uint32_t lds[];  // (the static words come first)
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wib = uni(threadIdx.x) >> 6;
  const uint32_t wpb = blockDim.x >> 6;
  uint32_t *regs = lds + (size_t)wib * a.max_regs * (W * 64);
  // registers beyond the LDS block: this wave's block of global scratch
  uint32_t *gregs = a.gscratch ? a.gscratch + ((size_t)blockIdx.x * wpb + wib) * a.gstride : nullptr;
  typedef const __attribute__((address_space(4))) BatchItem *item_ptr;
  typedef const __attribute__((address_space(4))) BatchProg *prog_ptr;
  // A wave adds its count to a program's slot once per run of items of
  // that program, not once per item: same-address device atomics serialize.
  uint64_t total = 0;
  uint32_t cur_slot = ~0u;
  GenState<W> st;
  if (VAR & 1) st.clear();
  auto process = [&](uint32_t item) {
    const item_ptr it = (item_ptr)a.items + item;
    const uint64_t t0 = it->t0, t1 = it->t1;
    const uint32_t step = it->step, part = it->part;
    const uint32_t slot = it->slot;
    const prog_ptr p = (prog_ptr)a.progs + it->prog;
    if (slot != cur_slot) {  // wave-uniform
      const uint64_t s = wave_sum_u64(total);
      if (lane == 0 && s) atomicAdd((unsigned long long *)(a.counts + cur_slot), (unsigned long long)s);
      total = 0;
      cur_slot = slot;
    }
    auto tile = [&](uint64_t t, bool alive) __attribute__((always_inline)) {
      const uint64_t U0 = t << LOG2W;
      uint32_t acc[W];
      if (alive) {
        const bool live = run_program<LOG2W, (VAR & 1) != 0, MODE == MODE_COUNT>(
            p->code, p->nins, U0, lane, acc, st, regs, a.max_regs * (W * 256u), gregs, a.j16_any);
        if (MODE == MODE_COUNT && !live) return;
      } else {
#pragma unroll
        for (int i = 0; i < W; i++) acc[i] = 0u;
      }
      uint32_t c = 0;
      if (MODE == MODE_DNF) {
        c = store_count_tile<LOG2W>(acc, U0, lane, p->nslices, p->n, p->out32, p->out_slices);
      } else {
        mask_tail<LOG2W>(acc, U0, lane, p->nslices, p->n);
#pragma unroll
        for (int i = 0; i < W; i++) c += __popc(acc[i]);
      }
      total += c;
      if (MODE == MODE_DNF && p->tile_counts) {  // for a later batched enumeration
        const uint32_t tc = wave_sum_u32(c);
        if (lane == 0) p->tile_counts[t] = tc;
      }
    };
    if constexpr ((VAR & 2) != 0) {
      // the waves of the block share the item
      const uint32_t n = wpb << (part & 0xFFu), mine = (part >> 8) * wpb + wib;
      uint32_t r = 0;
      for (uint64_t g = t0 >> 6; g * 64 < t1; g += step)
        r = visit_group<MODE == MODE_DNF>(p->code, lane, g, t0, t1, r, mine, n - 1u, tile);
    } else {
      for (uint64_t t = t0; t < t1; t += step) tile(t, true);
    }
  };
  // Items come sorted by cost, largest first, dealt over kQueues queues:
  // queue q holds items q, q + kQueues, ...  A wave works on the queue of
  // its XCD (workgroups go to the XCDs round-robin), then on the others
  // until all are drained; a drained queue is seen by a plain read before
  // any atomic is spent on it.  The first items of a queue, one for each of its
  // XCD's waves, are theirs by number, and the pops start behind them: a wave that
  // popped its first item and the next one ahead left others without where there is
  // about an item a wave (200 programs of 2^12 valuations and 300 clauses: 27.4
  // us, so 17.8).
  const uint32_t q0 = blockIdx.x % kQueues;
  constexpr bool BLOCKS = (VAR & 2) != 0;  // a block takes an item, not a wave
  // items of queue q taken by number
  auto taken = [&](uint32_t q) __attribute__((always_inline)) {
    return (gridDim.x + kQueues - 1 - q) / kQueues * (BLOCKS ? 1u : wpb);
  };
  auto drained = [&](uint32_t q, uint32_t popped) __attribute__((always_inline)) {
    return q + kQueues * (taken(q) + popped) >= a.nitems;
  };
  if constexpr ((VAR & 2) != 0) {
    // Uniform cofactor: a block pops an item for all its waves, and with a.pop_ahead the
    // next one while it works on it.  The live tiles of an item come many together
    // or not at all, and a wave alone took up to 44 evaluations one after the
    // other (6 us each) where it expected five; four times as many pops, 13 ns
    // each at one address, were a quarter of the launch.  A server slice of 48
    // requests, 45,500 live tiles of 494,000: 119 us, with an item per wave 250 us (on
    // one GPU; 109 to 139 over several now).
    __shared__ uint32_t popped;
    uint32_t k = 0, q = q0;
    uint32_t item = q + kQueues * (blockIdx.x / kQueues);
    for (;;) {
      // thread 0 pops from queue q (an item past the end: it is drained)
      auto pop = [&]() __attribute__((always_inline)) {
        return drained(q, 0) ? ~0u : q + kQueues * (taken(q) + atomicAdd(a.head + q * kQueueStride, 1u));
      };
      if (item >= a.nitems) {  // the queue is drained: on to one that is not
        if (threadIdx.x == 0) {
          while (item >= a.nitems && ++k < kQueues) {
            q = (q0 + k) % kQueues;
            if (!drained(q, *(volatile uint32_t *)(a.head + q * kQueueStride))) item = pop();
          }
          popped = item;
        }
        __syncthreads();
        item = uni(popped);
        __syncthreads();
        if (item >= a.nitems) break;  // the same for the whole block
      }
      uint32_t next = 0;
      if (a.pop_ahead && threadIdx.x == 0) next = pop();
      process(item);
      if (threadIdx.x == 0) popped = a.pop_ahead ? next : pop();
      __syncthreads();
      item = uni(popped);
      __syncthreads();
    }
  } else {
    for (uint32_t k = 0; k < kQueues; ++k) {
      const uint32_t q = (q0 + k) % kQueues;
      uint32_t *head = a.head + q * kQueueStride;
      const uint32_t first = taken(q);
      const bool pops = !drained(q, 0);  // the queue has more
      if (k > 0 && (!pops || drained(q, __builtin_amdgcn_readfirstlane(*(volatile uint32_t *)head)))) continue;
      // lane 0 holds the number in the queue
      uint32_t r = blockIdx.x / kQueues * wpb + wib;
      if (k > 0 && lane == 0) r = first + atomicAdd(head, 1u);
      for (;;) {
        const uint32_t item = q + kQueues * __builtin_amdgcn_readfirstlane(r);
        if (item >= a.nitems) break;  // this queue is drained
        // a.pop_ahead: the next item is popped while this one is worked on (92
        // DAGs with n <= 28: 63 us, without 96); not where items are long, as
        // one popped early waits while other waves end (4096 DAGs: 1.3 % slower)
        if (pops && a.pop_ahead && lane == 0) r = first + atomicAdd(head, 1u);
        process(item);
        if (!pops) break;
        if (!a.pop_ahead && lane == 0) r = first + atomicAdd(head, 1u);
      }
    }
  }
  // the waves of a block mostly end in the same program: one atomic for them
  __shared__ uint64_t part[4];
  __shared__ uint32_t part_slot[4];
  const uint64_t s = wave_sum_u64(total);
  if (lane == 0) part[wib] = s, part_slot[wib] = cur_slot;
  __syncthreads();
  if (threadIdx.x < wpb) {
    const uint32_t me = threadIdx.x;
    uint64_t sum = 0;
    bool first = true;  // of the waves with this slot
    for (uint32_t w = 0; w < wpb; w++) {
      if (part_slot[w] != part_slot[me]) continue;
      sum += part[w];
      first = first && w >= me;
    }
    if (first && sum) atomicAdd((unsigned long long *)(a.counts + part_slot[me]), (unsigned long long)sum);
  }
}

// Batched DNF write-out of a plan of clause-only programs without the uniform
// cofactor, on a grid of fresh blocks whose waves take a.run consecutive
// tiles each: the blocks start in order, so the waves write the vectors in
// order together, and no wave spends a queue pop or a count atomic.  a.items
// holds the plan's programs, one entry each, with [t0, t1) its tiles in the
// plan's tile order (ascending, contiguous, a.nitems >= 1); wave w takes plan
// tiles [w run, (w + 1) run), each tile finding its own program (a run may
// cross from one program into the next).  Every program has a
// tile-count array: the tile's model count goes there, and the program's count
// is the later sum over them (k_sum_tile_counts).
template <int LOG2W>
__global__ __launch_bounds__(256, min_waves(LOG2W, 0)) void k_batch_direct(BatchArgs a) {
  constexpr int W = 1 << LOG2W;
  typedef const __attribute__((address_space(4))) BatchItem *item_ptr;
  typedef const __attribute__((address_space(4))) BatchProg *prog_ptr;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wib = uni(threadIdx.x) >> 6;
  const uint64_t g0 = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + wib) * a.run;
  const item_ptr items = (item_ptr)a.items;
  const uint64_t end = items[a.nitems - 1].t1;
  if (g0 >= end) return;
  uint32_t lo = 0, hi = a.nitems;  // the entry with t0 <= g0 < t1, found once
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (items[mid].t0 <= g0)
      lo = mid;
    else
      hi = mid;
  }
  for (uint64_t g = g0; g < g0 + a.run && g < end; ++g) {  // wave-uniform
    while (g >= items[lo].t1) lo++;  // the run crossed into the next program
    const item_ptr it = items + lo;
    if (g < it->t0) continue;  // padding in front of a program of the XCD-local layout
    const prog_ptr p = (prog_ptr)a.progs + it->prog;
    const uint64_t t = g - it->t0;
    const uint64_t U0 = t << LOG2W;
    uint32_t acc[W];
    GenState<W> st;  // unused: clause-only programs
    if (LOG2W == 5 && p->xcd_code && p->chunk_counts) {
      // XCD-local layout (fbg_kernels.h): the renamed program's tile t is
      // the pieces x + 8 h + 16 (t & 3) + 64 (t >> 5) of the vector, h = 0, 1
      // (words 0..15 and 16..31 of each lane), x = bits 2..4 of t; full tiles
      // only (n >= 21), output 16-byte aligned
      run_program<LOG2W, false, false, true>(p->xcd_code, p->nins, U0, lane, acc, st, nullptr);
      const uint64_t piece = ((t >> 2) & 7) + 16 * (t & 3) + 64 * (t >> 5);
      store_xcd_tile(acc, p->out32 + piece * 1024 + lane * 4);
      uint32_t c0 = 0, c1 = 0;
#pragma unroll
      for (int i = 0; i < W; i++) {
        if (i < 16)
          c0 += __popc(acc[i]);
        else
          c1 += __popc(acc[i]);
      }
      c0 = wave_sum_u32(c0);
      c1 = wave_sum_u32(c1);
      // the two piece counts side by side, in tile order: the four waves of a
      // block fill 32 contiguous bytes
      if (lane == 0) *(uint2 *)(p->chunk_counts + 2 * t) = make_uint2(c0, c1);
    } else {
      run_program<LOG2W, false, false>(p->code, p->nins, U0, lane, acc, st, nullptr);
      const uint32_t c = store_count_tile<LOG2W>(acc, U0, lane, p->nslices, p->n, p->out32, p->out_slices);
      const uint32_t tc = wave_sum_u32(c);
      if (lane == 0) p->tile_counts[t] = tc;
    }
  }
}

#ifdef FBG_DEVICE_BATCH_KERNELS  // defined once, in batch.hip
// Counts after k_batch_direct: block (m, y) adds its share of the tile counts
// of entry m's program into that program's count slot (zeroed before).  For a
// program of the XCD-local layout it first forms each tile count from the
// counts of the tile's two 4 KiB pieces.
__global__ __launch_bounds__(256) void k_sum_tile_counts(BatchArgs a) {
  __shared__ uint64_t part[4];
  const BatchItem &it = a.items[blockIdx.x];
  const BatchProg &p = a.progs[it.prog];
  uint64_t s = 0;
  const bool xcd = p.xcd_code && p.chunk_counts;
  for (uint64_t t = (uint64_t)blockIdx.y * blockDim.x + threadIdx.x; t < p.ntiles; t += (uint64_t)gridDim.y * blockDim.x) {
    if (xcd) {
      // tile t of the vector is pieces 2t and 2t + 1; piece c came from
      // tile (c & 7) << 2 | (c >> 4 & 3) | (c >> 6) << 5 of the renamed
      // program, its half c >> 3 & 1
      uint32_t v = 0;
      for (uint64_t c = 2 * t; c < 2 * t + 2; c++) {
        const uint64_t k = ((c & 7) << 2) | ((c >> 4) & 3) | ((c >> 6) << 5);
        v += p.chunk_counts[2 * k + ((c >> 3) & 1)];
      }
      p.tile_counts[t] = v;
      s += v;
    } else {
      s += p.tile_counts[t];
    }
  }
  s = wave_sum_u64(s);
  if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t tot = 0;
    for (uint32_t w = 0; w < (blockDim.x >> 6); w++) tot += part[w];
    if (tot) atomicAdd((unsigned long long *)(a.counts + it.slot), (unsigned long long)tot);
  }
}

#endif

// Batched enumeration from the stored DNF vectors: the waves share out the
// list of the tiles that hold models (k_tile_list; the tile counts of all
// programs concatenated in program order), skip the tiles of the other plans
// and compact a tile's models into its program's list.
template <int LOG2W>
__global__ __launch_bounds__(256) void k_batch_compact(BatchEnumArgs a) {
  __shared__ __align__(4) uint16_t stage[4][kStageModels];
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wib = uni(threadIdx.x) >> 6;
  const uint64_t wave = (uint64_t)blockIdx.x * (blockDim.x >> 6) + wib;
  const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x >> 6);
  typedef const __attribute__((address_space(4))) EnumProg *enum_ptr;
  // one tile with models per wave and step
  const uint64_t nlist = *a.nlist;
  for (uint64_t k = wave; k < nlist; k += nwaves) {
    const uint64_t e = uni64(a.list[k]);
    const uint64_t g = list_tile(e);
    // the program owning global tile g: tile0 ascends with the program index
    uint32_t lo = 0, hi = a.np;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (((enum_ptr)a.progs)[mid].tile0 <= g) lo = mid; else hi = mid;
    }
    const enum_ptr p = (enum_ptr)a.progs + lo;
    if (p->log2w != (uint32_t)LOG2W || p->capacity == 0) continue;
    const uint64_t t = g - p->tile0;
    const uint64_t U0 = t << LOG2W;
    constexpr int W = 1 << LOG2W;
    uint32_t acc[W];
    const uint32_t *src = p->dnf + U0 * 64 + lane;
#pragma unroll
    for (int i = 0; i < W; i++) {
      const uint64_t sidx = (U0 + i) * 64 + lane;
      acc[i] = sidx < p->nslices ? src[i * 64] : 0u;
    }
    const uint64_t first = a.list_base[g / kListBlock] + list_before(e) - a.prog_base[lo];
    if (first >= p->capacity) continue;
    tile_compact<LOG2W>(acc, 0u, W, U0, lane, first, p->out, p->capacity, stage[wib]);
  }
}

// ------------------------------------------------------------------- lists

constexpr int LIST_THREADS = 256;
constexpr int LIST_PER_THREAD = kListBlock / LIST_THREADS;
static_assert(LIST_PER_THREAD == 8, "two 16-byte loads a thread");

#ifdef FBG_DEVICE_MISC_KERNELS  // defined once, in misc.hip

// The uniform-cofactor test of every group of 64 tiles (ngroups of them, no tiles
// beside): the live tiles' mask, and zeros for the model counts of the group's
// tiles.  A wave per group and step: two for each wave where there are 2^20 tiles,
// which wait for the scalar loads of the table (90 clauses 7 to 9 us; with a test of 64
// tiles on the scalar unit, eight words a clause, 12).
__global__ __launch_bounds__(256) void k_cofactor_masks(const uint32_t *code, uint64_t ngroups, uint64_t *masks,
                                                        uint32_t *counts) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t wave = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (uni(threadIdx.x) >> 6);
  const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x >> 6);
  for (uint64_t g = wave; g < ngroups; g += nwaves) {
    const uint64_t alive = tiles_alive(code, g * 64 + lane, ~0ull, ngroups * 64);
    if (lane == 0) masks[g] = alive;
    counts[g * 64 + lane] = 0u;
  }
}

// The counts of a thread's eight tiles (the counts array is 256-byte aligned).
__device__ __forceinline__ void load_counts(const uint32_t *in, uint64_t n, uint64_t at, uint32_t (&c)[8]) {
  if (at + 8 <= n) {
    const uint4 v0 = *(const uint4 *)(in + at), v1 = *(const uint4 *)(in + at + 4);
    c[0] = v0.x, c[1] = v0.y, c[2] = v0.z, c[3] = v0.w;
    c[4] = v1.x, c[5] = v1.y, c[6] = v1.z, c[7] = v1.w;
  } else {
#pragma unroll
    for (int k = 0; k < 8; k++) c[k] = at + k < n ? in[at + k] : 0u;
  }
}

// Sums over the block's threads of (models, tiles that hold models).
__device__ __forceinline__ TilePair block_sum(TilePair v, TilePair *sh) {
  v.models = wave_sum_u64(v.models);
  v.tiles = wave_sum_u64(v.tiles);
  if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  TilePair s = {0, 0};
  for (int w = 0; w < LIST_THREADS / 64; w++) s.models += sh[w].models, s.tiles += sh[w].tiles;
  __syncthreads();
  return s;
}

// Per block of kListBlock tiles: its models and its tiles that hold models.
__global__ __launch_bounds__(LIST_THREADS) void k_tile_sums(TileListArgs a) {
  __shared__ TilePair sh[LIST_THREADS / 64];
  uint32_t c[8];
  load_counts(a.counts, a.n, (uint64_t)blockIdx.x * kListBlock + threadIdx.x * 8, c);
  TilePair v = {0, 0};
#pragma unroll
  for (int k = 0; k < 8; k++) v.models += c[k], v.tiles += c[k] != 0u;
  v = block_sum(v, sh);
  if (threadIdx.x == 0) a.sums[blockIdx.x] = v;
}

// One block: the exclusive scan of the block sums in place (only where there
// are too many of them for every block of k_tile_list to add up the ones
// before it itself).
__global__ __launch_bounds__(LIST_THREADS) void k_tile_sums_scan(TileListArgs a, uint64_t nb) {
  __shared__ TilePair sh[LIST_THREADS];
  TilePair carry = {0, 0};
  for (uint64_t st = 0; st < nb; st += LIST_THREADS) {
    const uint64_t i = st + threadIdx.x;
    const TilePair v = i < nb ? a.sums[i] : TilePair{0, 0};
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < LIST_THREADS; off <<= 1) {
      const TilePair o = threadIdx.x >= (uint32_t)off ? sh[threadIdx.x - off] : TilePair{0, 0};
      __syncthreads();
      sh[threadIdx.x].models += o.models;
      sh[threadIdx.x].tiles += o.tiles;
      __syncthreads();
    }
    const TilePair in = sh[threadIdx.x], tot = sh[LIST_THREADS - 1];
    if (i < nb) a.sums[i] = {carry.models + in.models - v.models, carry.tiles + in.tiles - v.tiles};
    carry.models += tot.models;
    carry.tiles += tot.tiles;
    __syncthreads();
  }
}

// The list of the tiles that hold models, ascending: entry = the tile and the
// models before it in its block of kListBlock tiles (list_entry); list_base[block] the models before the block.  A block adds up the
// sums of the blocks before it itself (SCANNED: reads their scan), so one
// launch does what a scan of the sums, their application to every tile and
// the listing of the tiles would; only tiles with models are written.  The
// last block writes the number of models and the length of the list.  With
// np > 0 (a batch) a block also writes, for each program whose first tile
// (progs[p].tile0) is one of its tiles, the models before that tile.
// 2^20 tiles: 5 + 5 us with k_tile_sums, against 5 + 4.5 + 9.5 us for the
// three kernels of a full scan.
template <bool SCANNED>
__global__ __launch_bounds__(LIST_THREADS) void k_tile_list(TileListArgs a) {
  __shared__ TilePair sh[LIST_THREADS / 64];
  __shared__ uint32_t pre[kListBlock];  // batches: models before each tile of the block
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  uint32_t c[8];
  const uint64_t at = (uint64_t)blockIdx.x * kListBlock + tid * 8;
  load_counts(a.counts, a.n, at, c);
  TilePair base;
  if (SCANNED) {
    base = a.sums[blockIdx.x];
  } else {
    base = {0, 0};
    for (uint32_t k = tid; k < blockIdx.x; k += LIST_THREADS) {
      const TilePair v = a.sums[k];
      base.models += v.models;
      base.tiles += v.tiles;
    }
    base = block_sum(base, sh);
  }
  uint32_t m = 0, l = 0;
#pragma unroll
  for (int k = 0; k < 8; k++) m += c[k], l += c[k] != 0u;
  // at most 2^27 models and 2^11 tiles a block
  const uint32_t mi = wave_inclusive_scan(m), li = wave_inclusive_scan(l);
  if (lane == 63) sh[w] = {mi, li};
  __syncthreads();
  uint32_t mb = 0, lb = 0, mt = 0, lt = 0;
  for (uint32_t k = 0; k < LIST_THREADS / 64; k++) {
    if (k < w) mb += (uint32_t)sh[k].models, lb += (uint32_t)sh[k].tiles;
    mt += (uint32_t)sh[k].models, lt += (uint32_t)sh[k].tiles;
  }
  uint32_t rel = mb + mi - m;
  uint64_t at_list = base.tiles + lb + li - l;
#pragma unroll
  for (int k = 0; k < 8; k++) {
    if (a.np) pre[tid * 8 + k] = rel;
    if (c[k]) a.list[at_list++] = list_entry(at + k, rel);
    rel += c[k];
  }
  if (tid == 0) {
    a.list_base[blockIdx.x] = base.models;
    if (blockIdx.x == gridDim.x - 1) {
      *a.nlist = base.tiles + lt;
      if (a.total) *a.total = base.models + mt;
    }
  }
  if (!a.np) return;
  __syncthreads();
  const uint64_t t0 = (uint64_t)blockIdx.x * kListBlock, t1 = min(t0 + kListBlock, a.n);
  uint32_t lo = 0, hi = a.np;  // the first program with tile0 >= t0
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (a.progs[mid].tile0 < t0) lo = mid + 1; else hi = mid;
  }
  for (uint32_t p = lo + tid; p < a.np && a.progs[p].tile0 < t1; p += LIST_THREADS)
    a.prog_base[p] = base.models + pre[a.progs[p].tile0 - t0];
}

#endif

// ------------------------------------------------------------------ fills

#ifdef FBG_DEVICE_MISC_KERNELS
// p[0..n) = 0 and head[0..nhead) = 0 (queue heads and list counters).
__global__ void k_zero_u64(uint64_t *p, uint64_t n, uint32_t *head, uint32_t nhead) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
  if (i < nhead) head[i] = 0;
}

__global__ void k_set_u64(uint64_t *p, uint64_t v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

#endif

}  // namespace dev
}  // namespace fbg

#endif
