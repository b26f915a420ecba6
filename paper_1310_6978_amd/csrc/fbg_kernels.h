// fbg_kernels.h -- kernel argument blocks and launch wrappers (host side).
#ifndef FBG_KERNELS_H
#define FBG_KERNELS_H

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "../../include/fbg.h"
#include "fbg_isa.h"

namespace fbg {

// Registers of the general part held in VGPRs; the rest live in LDS.  The
// jump-table interpreter at 16 words per lane keeps three (its fixed register
// map leaves room for no more without spilling).
constexpr uint32_t kVgprRegs = 4;
constexpr uint32_t kJ16VgprRegs = FBG_J16_VGPR_REGS;
inline uint32_t vgpr_regs_of(int log2w) { return log2w == FBG_J16_LOG2W ? kJ16VgprRegs : kVgprRegs; }

// Models a wave of a compaction pass gathers in LDS before they leave (at
// least the 2048 of a row of 64 words).
constexpr uint32_t kStageModels = 2048;

// EvalArgs.direct
enum { ENUM_LISTED = 0, ENUM_DIRECT = 1, ENUM_ONE_BLOCK = 2 };

struct EvalArgs {
  const uint32_t *code;   // encoded program: clause block, instructions, pattern table
  uint32_t nins;          // instructions after the clause block (16 words per lane: 2-word units)
  uint32_t nregs;         // registers held in LDS (beyond vgpr_regs_of(log2w))
  int32_t n;              // variables
  uint64_t nslices;       // 2^max(n-5, 0) valid 32-bit words
  uint64_t ntiles;        // ceil(nslices / (64 W))
  uint64_t *out_count;    // MODE_COUNT
  uint32_t *out32;        // MODE_DNF (written); stored-DNF scans (read)
  uint64_t out_slices;    // MODE_DNF: words written (>= nslices, >= 2)
  const uint32_t *xcd_code;  // MODE_DNF at 32 words per lane: the XCD-local encoding, or null
  uint32_t *tile_counts;  // per unit: MODE_TILECNT (out), MODE_ENUM (in)
  // MODE_TILECNT after launch_cofactor_masks: the live tiles of the groups of 64 tiles, a
  // mask each; 2^part_shift waves share 64 groups
  const uint64_t *masks;
  uint32_t part_shift;
  // Units of the enumeration passes: 2^unit_shift to a tile (fbg_device.h).
  // MODE_ENUM: with `direct` a wave takes one unit; its block finds their
  // positions from tile_counts (or block_sums), the last block writing the
  // total to out_count, or there is only one block and no tile counts.  Else the
  // list of the units that hold models (TileListArgs)
  uint32_t unit_shift;
  uint32_t direct;
  uint64_t nunits;
  uint32_t *block_sums;   // stored-DNF scans: sums of the counts of a block's units, or null
  uint32_t lds_stride;    // words of LDS per wave: its registers, at least kStageModels / 2
  const uint64_t *list;
  const uint64_t *list_base;
  const uint64_t *nlist;
  uint64_t *out_idx;      // MODE_ENUM
  uint64_t capacity;      // MODE_ENUM
  // non-zero: the jump-table interpreter (16 words per lane) runs the copy of
  // its table for code off a 64 KiB boundary (same results; for tests)
  uint32_t j16_any = 0;
};

// The XCD-local layout of the batched DNF write-out (32 words per lane, a
// program made of clauses alone, n >= kXcdMinVars, an output 16 bytes
// aligned).  The write-out kernel evaluates a second encoding of the
// program with its variables renamed (xcd_write_out_permutation), so that
// its tile t (64 lanes x 32 words) holds two whole 4 KiB pieces of the DNF
// vector, pieces p and p + 8 (32 KiB apart), p = ((t >> 2) & 7) + 16 (t & 3)
// + 64 (t >> 5), and each lane's words 4g .. 4g+3 are adjacent in memory:
// eight 16-byte stores per lane, each a whole 1 KiB of a piece.  With one
// tile per wave and four waves per block, every block writes 4 KiB pieces of
// one residue class modulo 8 (blocks go to the eight XCDs in turn), so that
// the XCDs write interleaved 4 KiB pieces of one region of the vector at a
// time; HBM takes that faster than the same bytes in plain order or in
// larger pieces per XCD.  The model counts of a tile's two pieces go to
// chunk_counts[2t], [2t + 1]; k_sum_tile_counts adds the two pieces of each
// 8 KiB tile of the vector into the tile counts the batched enumeration
// reads.
constexpr int kXcdMinVars = 21;

struct BatchProg {
  const uint32_t *code;
  uint32_t nins;
  uint32_t nregs;
  int32_t n;
  uint64_t nslices;
  uint64_t ntiles;
  uint32_t *out32;      // MODE_DNF: the program's DNF vector
  uint64_t out_slices;  // MODE_DNF: 32-bit words of out32
  uint32_t *tile_counts;  // MODE_DNF: per-tile model counts (or null)
  // the batched DNF write-out in the XCD-local layout (or null): the program
  // with variables renamed, and the per-piece model counts it writes
  const uint32_t *xcd_code;
  uint32_t *chunk_counts;
};

// One program of a batched enumeration over stored DNF vectors.
struct EnumProg {
  const uint32_t *dnf;  // the DNF vector as 32-bit words
  uint64_t nslices;     // valid 32-bit words
  uint64_t tile0;       // first global tile of the program
  uint64_t *out;        // model indices (capacity entries)
  uint64_t capacity;
  uint32_t log2w;       // tiling of the program's plan
  uint32_t pad;
};

struct BatchEnumArgs {
  const EnumProg *progs;
  uint32_t np;
  const uint64_t *list;       // the tiles holding models (TileListArgs)
  const uint64_t *list_base;
  const uint64_t *nlist;
  const uint64_t *prog_base;  // models before each program's first tile
};

// From the model counts of n tiles (n >= 1) to the list of the tiles that
// hold models and the positions of their models (k_tile_sums, k_tile_list).
// Tiles go in blocks of kListBlock, nb = tile_list_blocks(n) of them.
constexpr uint32_t kListBlock = 2048;
struct TilePair {
  uint64_t models, tiles;
};
// An entry of the list: the tile, and the models before it in its block.  Both
// fit one word whatever the program: 2^37 tiles at most (48 letters at one word
// per lane), and fewer than 2^27 models before the last tile of a block.
constexpr uint32_t kListTileBits = FBG_MAX_VARS - FBG_TILE_BASE_BIT;
static_assert(((uint64_t)(kListBlock - 1) << (FBG_TILE_BASE_BIT + 5)) >> (64 - kListTileBits) == 0,
              "a tile has at most 2^16 valuations");
constexpr uint64_t list_entry(uint64_t tile, uint32_t before) { return tile | (uint64_t)before << kListTileBits; }
constexpr uint64_t list_tile(uint64_t e) { return e & ((1ull << kListTileBits) - 1); }
constexpr uint32_t list_before(uint64_t e) { return (uint32_t)(e >> kListTileBits); }
struct TileListArgs {
  const uint32_t *counts;  // n tile counts, 256-byte aligned
  uint64_t n;
  TilePair *sums;       // nb: per block (temporary)
  uint64_t *list;       // up to n entries (list_entry)
  uint64_t *list_base;  // nb: models before each block
  uint64_t *nlist;      // length of the list
  uint64_t *total;      // number of models (or null)
  const EnumProg *progs = nullptr;  // np > 0: prog_base[p] = models before progs[p].tile0
  uint64_t *prog_base = nullptr;
  uint32_t np = 0;
};

struct BatchItem {
  uint32_t prog;    // index into the program table
  uint32_t slot;    // index into the counts array
  // tiles t0, t0 + step, t0 + 2 step, ... below t1; with the uniform cofactor
  // the tiles of [t0, t1) in the groups of 64 tiles t0 / 64, t0 / 64 + step, ...,
  // share part >> 8 of 2^(part & 255) of the live ones (a block's item: its
  // waves share it further)
  uint64_t t0, t1;
  uint32_t step;
  uint32_t part;
};

// A plan's work items are split over kQueues queues (item i in queue
// i mod kQueues), one per XCD, each with its own head counter kQueueStride
// words (64 bytes) from the next, so that the queue atomics of the eight
// XCDs do not all meet at one address.
constexpr uint32_t kQueues = 8;
constexpr uint32_t kQueueStride = 16;
constexpr uint32_t kHeadWords = kQueues * kQueueStride;

struct BatchArgs {
  const BatchProg *progs;
  const BatchItem *items;
  uint32_t nitems;
  uint32_t max_regs;      // LDS registers per wave (beyond vgpr_regs_of(log2w))
  uint32_t *head;     // kHeadWords words of queue heads, zeroed before the launch
  uint64_t *counts;   // per slot; the kernel adds to it
  uint32_t pop_ahead = 0;  // queue pops overlap the work of the item before (short items)
  uint32_t run = 1;   // k_batch_direct: consecutive tiles per wave
  // registers beyond the max_regs LDS registers (jump-table form only):
  // gstride words of global scratch per wave of the grid, or none
  uint32_t *gscratch = nullptr;
  uint64_t gstride = 0;
  uint32_t j16_any = 0;   // as in EvalArgs
};

enum { EVAL_COUNT = 0, EVAL_DNF = 1, EVAL_TILECNT = 2, EVAL_ENUM = 3 };

hipError_t launch_eval(int mode, int log2w, int var, const EvalArgs &a, int grid, int block, size_t lds,
                       hipStream_t s);
hipError_t launch_dnf_scan(int mode, int log2w, const EvalArgs &a, int grid, int block, hipStream_t s);
hipError_t launch_batch(int mode, int log2w, int var, const BatchArgs &a, int grid, int block, size_t lds,
                        hipStream_t s);
// The DNF write-out of a plan of clause-only programs without the cofactor,
// a.run consecutive tiles per wave (a.items: one entry per program, [t0, t1) its tiles in the
// plan, ascending; every program has tile counts), then the per-program sums
// of those tile counts into a.counts (sum_blocks blocks per program).
hipError_t launch_batch_direct(int log2w, const BatchArgs &a, int grid, int block, int sum_blocks, hipStream_t s);
// Resident blocks per compute unit of an evaluator or batch launch.
int eval_blocks_per_cu(int mode, int log2w, int var, int block, size_t lds);
int batch_blocks_per_cu(int mode, int log2w, int var, int block, size_t lds);
hipError_t launch_batch_compact(int log2w, const BatchEnumArgs &a, int grid, int block, hipStream_t s);
// The uniform-cofactor masks of a program's ngroups groups of 64 tiles, and
// zeros for their tiles' counts.
hipError_t launch_cofactor_masks(const uint32_t *code, uint64_t ngroups, uint64_t *masks, uint32_t *counts, int grid,
                                 hipStream_t s);
hipError_t launch_tile_list(const TileListArgs &a, hipStream_t s);
uint64_t tile_list_blocks(uint64_t n);
// p[0..n) = 0 and head[0..nhead) = 0.
hipError_t launch_zero(uint64_t *p, uint64_t n, uint32_t *head, uint32_t nhead, hipStream_t s);
hipError_t launch_set_u64(uint64_t *p, uint64_t v, hipStream_t s);

// The scratch of fbg_enumerate_noalloc (noalloc.hip): a static device array
// of kNoallocScratchBytes per device, enough for the temporaries of an
// enumeration over at most kNoallocMaxTiles tiles (4-byte tile counts,
// 8-byte offsets, block sums).
constexpr uint64_t kNoallocMaxTiles = FBG_NOALLOC_MAX_TILES;
constexpr uint64_t kNoallocScratchBytes = FBG_NOALLOC_SCRATCH_BYTES;
// Its device address on the current device (looked up once per device).
hipError_t noalloc_scratch(void **out);

}  // namespace fbg

#endif
