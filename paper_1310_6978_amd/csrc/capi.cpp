// capi.cpp -- the C ABI of include/fbg.h: program residency, launch
// geometry, work plans for batches and serving, and argument checking.
#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdlib.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/fbg.h"
#include "fbg_internal.h"
#include "fbg_kernels.h"
#include "scratch_pool.h"

namespace {

thread_local std::string g_err;
thread_local int64_t g_err_off = -1;

fbg_status fail(fbg_status st, const char *fmt, ...) {
  char buf[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  g_err_off = -1;
  return st;
}

fbg_status hip_fail(hipError_t e, const char *what) {
  return fail(FBG_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

constexpr int kMaxLog2W = 5;
constexpr int kWavesPerBlock = 4;
constexpr size_t kMaxLdsPerBlock = 64 * 1024;
// Consecutive tiles per wave of the one-wave-per-tile DNF write-out of a batch
// plan (C1, 16 x 2^32 bits at W = 32: 1.45-1.46 ms at 4, 1.48 at 1, 1.58 at 2
// and 1.59 at 8).
constexpr uint32_t kDirectRun = 4;
// LDS registers a wave of a batch plan keeps at 16 words per lane (4 KiB
// each): four waves a block then take 32 KiB, so LDS allows the four blocks
// per CU that the registers of the jump-table interpreter allow.
constexpr uint32_t kJ16LdsRegs = 2;

int g_cu_count[64];
std::once_flag g_cu_once[64];

int cu_count(int dev) {
  if (dev < 0 || dev >= 64) return 256;
  std::call_once(g_cu_once[dev], [dev] {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    g_cu_count[dev] = v;
  });
  return g_cu_count[dev];
}

uint64_t slices_of(int n) { return n >= FBG_SLICE_BITS ? (1ull << (n - FBG_SLICE_BITS)) : 1ull; }
uint64_t dnf_words_of(int n) { return n >= 6 ? (1ull << (n - 6)) : 1ull; }
uint64_t tiles_of(uint64_t nslices, int log2w) {
  const uint64_t per = 64ull << log2w;
  return (nslices + per - 1) / per;
}

// Registers beyond the first kVgprRegs live in LDS: W*64 words each per wave.
uint32_t lds_regs(uint32_t nregs, int log2w) {
  const uint32_t v = fbg::vgpr_regs_of(log2w);
  return nregs > v ? nregs - v : 0u;
}
size_t lds_per_wave(uint32_t nregs, int log2w) { return (size_t)lds_regs(nregs, log2w) * (64u << log2w) * 4u; }

// Device memory for programs: size classes of powers of two (>= 4 KiB) carved
// out of 64 MiB chunks and recycled through free lists, so that compiling a
// request costs one small copy and no hipMalloc.  One arena per device.
class CodeArena {
 public:
  static CodeArena &of(int dev) {
    static std::mutex m;
    static std::vector<CodeArena *> arenas;
    std::lock_guard<std::mutex> g(m);
    if ((size_t)dev >= arenas.size()) arenas.resize((size_t)dev + 1, nullptr);
    if (!arenas[(size_t)dev]) arenas[(size_t)dev] = new CodeArena();
    return *arenas[(size_t)dev];
  }

  hipError_t alloc(size_t bytes, void **out, int &cls) {
    std::lock_guard<std::mutex> g(mu_);
    cls = 12;
    while (((size_t)1 << cls) < bytes) cls++;
    const size_t sz = (size_t)1 << cls;
    if (sz > kChunk) {  // very large programs get their own allocation
      cls = -1;
      return hipMalloc(out, bytes);
    }
    auto &fl = free_[(size_t)cls];
    if (!fl.empty()) {
      *out = fl.back();
      fl.pop_back();
      return hipSuccess;
    }
    if (!cur_ || used_ + sz > kChunk) {
      void *c = nullptr;
      hipError_t e = hipMalloc(&c, kChunk);
      if (e != hipSuccess) return e;
      cur_ = (char *)c;
      used_ = 0;
    }
    *out = cur_ + used_;
    used_ += sz;
    return hipSuccess;
  }

  void release(void *p, int cls) {
    if (!p) return;
    if (cls < 0) {
      (void)hipFree(p);
      return;
    }
    std::lock_guard<std::mutex> g(mu_);
    free_[(size_t)cls].push_back(p);
  }

 private:
  static constexpr size_t kChunk = (size_t)64 << 20;
  std::mutex mu_;
  char *cur_ = nullptr;
  size_t used_ = 0;
  std::vector<void *> free_[64];
};

fbg_status parse_wpl(int w, int &log2w) {
  if (w < 1 || w > FBG_MAX_WORDS_PER_LANE || (w & (w - 1)))
    return fail(FBG_E_INVAL, "words_per_lane must be 1, 2, 4, 8, 16 or 32 (got %d)", w);
  log2w = __builtin_ctz((unsigned)w);
  return FBG_OK;
}

}  // namespace

struct fbg_program {
  fbg::Compiled c;
  int device = -1;  // -1: compiled without a device (host only)
  uint32_t *d_code = nullptr;
  int code_class = 0;  // size class in the device's code arena
  uint64_t code_bytes = 0;  // bytes held on the device
  std::vector<uint32_t> words[kMaxLog2W + 1];
  uint64_t dev_off[kMaxLog2W + 1] = {0, 0, 0, 0, 0, 0};
  uint32_t nins[kMaxLog2W + 1] = {0, 0, 0, 0, 0, 0};
  uint32_t tilings = FBG_COMPILE_WPL_MASK;  // bit l: encoded for 2^l words per lane
  bool has_tiling(int l) const { return (tilings >> l) & 1u; }
  // programs of clauses alone with n >= kXcdMinVars: the 32-words-per-lane
  // encoding with variables renamed for the XCD-local DNF write-out
  std::vector<uint32_t> words_xcd;
  uint64_t dev_off_xcd = 0;
  bool has_xcd = false;
  double live[kMaxLog2W + 1] = {1, 1, 1, 1, 1, 1};  // share of tiles expected to pass the uniform-cofactor test
  uint32_t multi[kMaxLog2W + 1] = {};               // clauses with two or more word literals (multi_clauses)
  double j16_cost = 0;  // per tile at 16 words per lane, from the jump-table form (0: none)
  uint32_t ncl = 0;  // leading clause instructions
  int auto_log2w = 0;
  bool tuned = false;  // auto_log2w was set by fbg_program_set_tuning
  int one_count = 0, one_list = 0;  // tilings of a count and an enumeration unless tuned (one_block_log2w)
  uint64_t nslices = 1;
  bool cofactor = false;  // default evaluation variant (fbg_program_set_tuning)
  bool general() const { return c.code.size() > ncl; }
  // kernel variant: bit 0 = general code after the clauses, bit 1 = cofactor
  int variant(const fbg_tune *tune) const {
    const bool cof = cofactor || (tune && (tune->flags & FBG_TUNE_COFACTOR));
    return (general() ? 1 : 0) | (cof ? 2 : 0);
  }
};

struct fbg_batch {
  // One persistent launch per plan: programs made only of clauses run at
  // their own (wide) tiling, general programs at a narrower one whose
  // registers fit; a batch holds one or two plans.
  struct Plan {
    int log2w = 0;
    int var = 0;
    int grid = 1, grid_dnf = 1;
    int block = 256;
    size_t lds = 0;
    uint32_t nitems = 0;
    uint32_t pop_ahead = 0;  // short items
    uint32_t max_regs = 0;  // LDS registers per wave
    fbg::BatchItem *d_items = nullptr;
    // clause-only programs without the cofactor: the DNF write-out runs one
    // wave per tile over this table (one entry per program, its tiles in the
    // plan's order) once the tile counts exist (fbg_batch_set_enum_outputs)
    fbg::BatchItem *d_direct = nullptr;
    uint32_t ndirect = 0;
    uint64_t ntiles = 0, max_prog_tiles = 0;
    uint32_t direct_run = kDirectRun;  // tiles per wave of the direct write-out
    // jump-table form (16 words per lane): registers beyond the plan's LDS
    // registers, gstride words per wave of the grid
    uint32_t *d_gscratch = nullptr;
    uint64_t gstride = 0;
  };
  int device = -1;
  int32_t np = 0;
  std::vector<Plan> plans;
  fbg::BatchProg *d_progs = nullptr;
  fbg::BatchProg *d_progs_dnf = nullptr;  // with DNF outputs (fbg_batch_set_dnf_outputs)
  std::vector<fbg::BatchProg> host_progs;
  std::vector<fbg::BatchProg> host_dnf;   // host copy of d_progs_dnf
  // batched enumeration (fbg_batch_set_enum_outputs): per-tile counts written
  // by fbg_batch_eval_dnf, their list, and the per-program output table
  std::vector<int> plan_of;               // plan index of every program
  uint64_t total_tiles = 0;
  uint32_t *d_tile_counts = nullptr;
  uint32_t *d_chunk_counts = nullptr;     // XCD-local write-out: counts per 4 KiB piece
  uint64_t *d_tile_list = nullptr;        // tiles holding models (TileListArgs)
  fbg::TilePair *d_list_sums = nullptr;
  uint64_t *d_list_base = nullptr;        // per block, then the length of the list, then per program
  fbg::EnumProg *d_enum = nullptr;
  uint32_t *d_head = nullptr;             // kHeadWords of queue heads per plan (at most 4 plans)
  // captured graph of (zero fill, persistent kernels) for one counts pointer
  hipGraph_t graph = nullptr;
  hipGraphExec_t graph_exec = nullptr;
  uint64_t *graph_counts = nullptr;
};

// Bytes of queue heads at the start of a server slot: kHeadWords words,
// rounded to whole 256-byte blocks so that the program table that follows
// starts on its own cache lines.
constexpr size_t kServerHeadBytes = (fbg::kHeadWords * sizeof(uint32_t) + 255) / 256 * 256;

struct fbg_server {
  int device = -1;
  int log2w = 0;
  int32_t max_programs = 0, max_items = 0, nbuf = 0, next = 0;
  bool cofactor = false;
  // A slot's staging (pinned) and device buffers hold, in this order, the
  // kHeadWords queue heads (zero in the staging copy), the slice's program
  // table and its pieces, so that one copy uploads the slice and clears its
  // heads.
  struct Slot {
    char *h = nullptr;  // pinned staging
    char *d = nullptr;  // device copy
    hipEvent_t done = nullptr;
    bool used = false;
  };
  std::vector<Slot> slots;
};

namespace {

// Largest words-per-lane that still gives every wave of a full grid a tile,
// within the LDS budget of the program's registers.
int pick_log2w(uint64_t nslices, uint32_t nregs, bool general, int dev) {
  const uint64_t waves = (uint64_t)cu_count(dev) * 32;  // 8 waves per SIMD
  int best = 0;
  // Programs with a general part: the jump-table interpreter at 16 words per
  // lane (four waves per SIMD) whenever every compute unit gets a few tiles;
  // below that the plain interpreter, which beyond 8 words per lane loses
  // more occupancy than it gains.
  if (general && lds_per_wave(nregs, FBG_J16_LOG2W) <= kMaxLdsPerBlock &&
      tiles_of(nslices, FBG_J16_LOG2W) >= (uint64_t)cu_count(dev) * 4)
    return FBG_J16_LOG2W;
  for (int l = general ? 3 : kMaxLog2W; l >= 0; l--) {
    if (lds_per_wave(nregs, l) > kMaxLdsPerBlock) continue;
    if (tiles_of(nslices, l) >= waves || l == 0) {
      best = l;
      break;
    }
  }
  while (best > 0 && lds_per_wave(nregs, best) > kMaxLdsPerBlock) best--;
  return best;
}

struct Geometry {
  int log2w, grid, block;
  size_t lds;
  int var;  // the kernel variant (kernel_variant)
};

fbg_status block_shape(uint32_t nregs, int l, int &wpb, size_t &lds) {
  const size_t lw = lds_per_wave(nregs, l);
  wpb = kWavesPerBlock;
  if (lw * wpb > kMaxLdsPerBlock) wpb = 1;
  if (lw * wpb > kMaxLdsPerBlock)
    return fail(FBG_E_RANGE, "program needs %u registers x %d words per lane: %zu bytes of LDS per wave (max %zu)",
                nregs, 1 << l, lw, kMaxLdsPerBlock);
  lds = lw * wpb;
  return FBG_OK;
}

// FBG_E_INVAL unless the program was encoded for 2^l words per lane.
fbg_status check_tiling(const fbg_program *p, int l) {
  if (!p->has_tiling(l))
    return fail(FBG_E_INVAL, "the program was compiled without %d words per lane (FBG_COMPILE_WPL)", 1 << l);
  return FBG_OK;
}

// Clauses with two or more word literals at 2^l words per lane (multi clauses).
uint32_t multi_clauses(const fbg_program *p, int l) {
  uint32_t multi = 0;
  for (uint32_t c = 0; c < p->ncl; c++) {
    int word = 0;
    for (const fbg::Lit &x : p->c.code[c].ls.lits) word += x.k >= FBG_TILE_BASE_BIT && x.k < FBG_TILE_BASE_BIT + l;
    multi += word >= 2;
  }
  return multi;
}

// The words per lane at which a small program is one tile for each wave of one
// block, so that a count (or with `list` an enumeration) is a single launch, or
// the program's own tiling (more, narrower tiles and two launches) where that is
// faster: only where a tile's work hardly grows with its words.  Figures: a call in
// one block, then with the program's own tiling.
//  - Clauses to 32 words (n <= 18), general parts to 8 (n <= 16).
//  - A clause with two or more word literals (multi) takes a wave 0.1 to 0.2 us, any
//    other 0.01 us.  Counts save 3 us, unless a tile ends at its first clauses all
//    the same: 90 clauses of 5 literals over 18 letters (39 multi) 10.8 and 8.6 us, 75
//    of 3 literals (13) 6.6 and 8.2; 1800 of 8 literals 324 and 32; 300 of 5 literals
//    over 15 letters (28) 12.8 and 10.9; 714 of 3 literals over 18 letters (123, but none
//    is reached) 5.4 and 8.3.
//  - Enumerations save 7 us and evaluate a tile once, not twice; up to 4 words they are
//    faster whatever the clauses (1400 of 8 literals over 14 letters 30 and 54 us, all
//    2^15 valuations 19.5 and 20.1).  Beyond, multi clauses are waited for (16 letters:
//    300 clauses of 6 literals, 91 multi, 19.5 and 22.4, 320 of 8, 160 multi, 33 and 26; 17
//    letters: 663 of 3, 80 multi, 21 and 13) and so are many models, most of them in few waves (16 letters:
//    7,714 models 12.2 and 12.0, 32,768 24 and 13; 17: 8,848 14.3 and 12.2; 18: 1,846
//    16.3 and 11.8, 177 9.6 and 12.2, 131,072 86 and 13.5).
int one_block_log2w(const fbg_program *p, bool list) {
  const int own = p->auto_log2w;
  for (int k = 0; k <= (p->general() ? 3 : kMaxLog2W); k++) {
    if (!p->has_tiling(k) || tiles_of(p->nslices, k) > (uint64_t)kWavesPerBlock ||
        lds_per_wave((uint32_t)p->c.nregs, k) * kWavesPerBlock > kMaxLdsPerBlock)
      continue;
    const uint32_t multi = p->multi[k];
    // log2 of the valuations expected to satisfy the clauses, of all (a general part
    // taken as true on half) and of a block's at one word by those without word literals
    double models = p->c.n - (p->general() ? 1.0 : 0.0), first = FBG_TILE_BASE_BIT + 2;
    for (uint32_t c = 0; c < p->ncl; c++) {
      const auto &lits = p->c.code[c].ls.lits;
      bool word = false;
      for (const fbg::Lit &x : lits) word = word || (x.k >= FBG_TILE_BASE_BIT && x.k < FBG_TILE_BASE_BIT + k);
      const double share = std::log2(1.0 - std::ldexp(1.0, -(int)std::min<size_t>(std::max<size_t>(lits.size(), 1), 50)));
      models += share;
      if (!word) first += share;
    }
    const bool one = list ? k <= 2 || (multi <= (k == 3 ? 96u : 40u) && models + k <= 16)
                          : first < 0 || multi + (p->ncl - multi) / 12 <= (k == 5 ? 24u : k == 4 ? 30u : 48u);
    return one ? k : own;
  }
  return own;
}

// The kernel variant of a launch over one program's tiles.  The uniform-cofactor test
// takes a wave 64 tiles at a time; without it a tile that holds no model mostly ends at
// its first key, so a program that asks for the test is run without it where that is
// faster (the results are the same).  Figures: without the test, then with it.
//  - Counts and enumerations from 2^18 tiles on: a 3-CNF system of 30 letters and 130
//    clauses at 8 words per lane (2^16 tiles) 10.3 us and 11.5, of 32 and 130 at 8 (2^18)
//    23.1 and 18.1, of 33 and 150 at 4 (2^20) 39.8 and 17.6; equivalence relations on 8
//    elements at 4 (2^15) 12.1 and 13.8, on 9 at 32 (2^20) 47.1 and 30.5; with a general
//    part, posets with a special element at 4 (2^17) 52.5 and 67.7, 34 letters and 120
//    clauses at 32 (2^18) 99.9 and 40.0.
//  - Of the enumerations, those where fewer than one tile in 128 is expected to live have
//    the test in a launch of its own, after which the live tiles are dealt over the
//    waves (equivalence relations on 9 elements at 32 words, test in the wave 53.4,
//    so 40.7; 3-CNF systems of 36 letters and 144 clauses at 4 words, one tile in 160,
//    135 and 124; at 16, one in 37, 71.6 and 82.5).
//  - Vectors from 13 clauses for each word per lane on, whose evaluation the stores
//    no longer hide (2^32 bits: 60 clauses at 4 words 143 and 93, at 8 words 85 and 101;
//    130 at 8 132 and 103, at 16 93 and 116; 250 at 16 115 and 108, at 32 86 and 113;
//    600 at 32 149 and 114), if they are not small (2^12 tiles 5.8 and 6.7).  With a
//    general part from 24 clauses (2^28 bits and 80 clauses at 4 words 10.5 and 12.6, 2^30
//    and 138 at 4 77 and 70) and 2^16 tiles (118 clauses over 27 letters at 4 words, 2^14
//    tiles, 14.2 and 21.0, at 1, 2^16, 24.2 and 23.5); at 32 words all (2^30 bits, 60
//    clauses 43 and 32).
int kernel_variant(const fbg_program *p, const fbg_tune *tune, int mode, int l, uint64_t ntiles) {
  const int var = p->variant(tune);
  if (!(var & 2)) return var;
  const uint32_t clauses = ((var & 1) ? 24u : 13u) << l;
  const uint64_t few = mode != fbg::EVAL_DNF ? 1ull << 18 : var == 3 && l < 5 ? 1ull << 16 : 1ull << 13;
  const bool test = ntiles >= few && (mode != fbg::EVAL_DNF || p->ncl >= clauses || (var == 3 && l == 5));
  if (!test) return var & 1;
  return mode == fbg::EVAL_TILECNT && p->live[l] <= 1.0 / 128 ? var | 4 : var;
}

// Launch shape of an evaluator kernel: a persistent grid of exactly the
// blocks that can be resident at once (more would only queue behind them and
// finish in a tail), each wave striding over the tiles.
fbg_status geometry(const fbg_program *p, const fbg_tune *tune, int mode, Geometry &g) {
  int l = mode == fbg::EVAL_DNF || p->tuned ? p->auto_log2w
          : mode == fbg::EVAL_COUNT          ? p->one_count
                                             : p->one_list;
  fbg_status st;
  if (tune && tune->words_per_lane && (st = parse_wpl(tune->words_per_lane, l))) return st;
  if ((st = check_tiling(p, l))) return st;
  int wpb;
  if ((st = block_shape((uint32_t)p->c.nregs, l, wpb, g.lds))) return st;
  const uint64_t ntiles = tiles_of(p->nslices, l);
  const uint64_t blocks = (ntiles + wpb - 1) / wpb;
  g.var = kernel_variant(p, tune, mode, l, ntiles);
  const int occ = fbg::eval_blocks_per_cu(mode, l, g.var, 64 * wpb, g.lds);
  uint64_t maxb = (uint64_t)cu_count(p->device) * (uint64_t)occ;
  // A DNF write-out without the cofactor runs one tile per wave on a grid of
  // fresh blocks: the blocks start in order, so the writes advance through
  // the vector together (a 2^32-bit vector at W = 32: 0.101 ms against 0.109
  // on a resident grid).  Counting keeps the resident grid, whose waves add
  // their counts once each; the cofactor filters 64 tiles per wave at once.
  if (mode == fbg::EVAL_DNF && !(g.var & 2)) maxb = blocks;
  if (tune && tune->grid_blocks > 0) maxb = (uint64_t)tune->grid_blocks;
  g.log2w = l;
  g.block = 64 * wpb;
  g.grid = (int)std::max<uint64_t>(1, std::min(blocks, maxb));
  return FBG_OK;
}

// FBG_J16_TABLE=any in the environment makes the jump-table interpreter run
// the copy of its table meant for code loaded off a 64 KiB boundary, so that
// tests cover it (both copies compute the same).  Read at every launch.
uint32_t j16_any() {
  const char *v = getenv("FBG_J16_TABLE");
  return (v && strcmp(v, "any") == 0) ? 1u : 0u;
}

fbg_status check_device(int want) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev != want) return fail(FBG_E_INVAL, "object lives on device %d but the current device is %d", want, dev);
  return FBG_OK;
}

fbg_status check_program(const fbg_program *p) {
  if (!p) return fail(FBG_E_INVAL, "program is NULL");
  if (p->device < 0 || !p->d_code) return fail(FBG_E_DEVICE, "program was compiled without a HIP device");
  return check_device(p->device);
}

fbg::EvalArgs base_args(const fbg_program *p, int log2w) {
  fbg::EvalArgs a;
  memset(&a, 0, sizeof a);
  a.code = p->d_code + p->dev_off[log2w];
  a.nins = p->nins[log2w];
  a.nregs = lds_regs((uint32_t)p->c.nregs, log2w);
  a.n = p->c.n;
  a.nslices = p->nslices;
  a.ntiles = tiles_of(p->nslices, log2w);
  a.j16_any = j16_any();
  return a;
}

// Share of a program's tiles expected to pass the uniform-cofactor test at
// 2^l words per lane, its tile-only clauses taken as independent.
double expected_live(const fbg_program *p, int l) {
  double live = 1.0;
  for (uint32_t k = 0; k < p->ncl; k++) {
    const auto &lits = p->c.code[k].ls.lits;
    bool tile_only = true;
    for (const fbg::Lit &x : lits) tile_only = tile_only && x.k >= FBG_TILE_BASE_BIT + l;
    if (tile_only) live *= 1.0 - std::ldexp(1.0, -(int)std::min<size_t>(lits.size(), 60));
  }
  return live;
}

// Estimated cost of one tile of a program in a batch or a server slice at 2^l
// words per lane, in steps of the interpreter: at 16 words per lane the
// general part's VALU instructions per word and half a step per dispatch of
// its jump-table form (j16_general_cost), elsewhere one step per instruction
// after the clause block in the plain form; a few more per tile; a clause
// block adds its setup, product tree and count, and one step per clause.  (On
// the C3 programs made of one to four clauses a tile takes about 12 steps.)
double tile_cost(const fbg_program *p, int l) {
  const double general = l == FBG_J16_LOG2W && p->j16_cost > 0 ? p->j16_cost : (double)(p->c.code.size() - p->ncl);
  return general + 4.0 + (p->ncl ? 8.0 + (double)p->ncl : 0.0);
}

// The same with the uniform cofactor: the test, and the tiles expected to pass
// it (at 16 words per lane 0.6 % of the tiles of a 3-CNF system over 36 letters,
// 40 % over 26, so pieces of equal tile counts would cost up to 30 times one
// another).
double cofactor_tile_cost(const fbg_program *p, int l) { return 0.5 + p->live[l] * tile_cost(p, l); }

// Cut the tiles [b, e) of a program into about K work items (at most K, with
// the cofactor 2 K), appended by add(item, tiles): interleaved runs of tiles, or with the uniform
// cofactor of groups of 64 tiles, where the stride K is odd (live groups share
// their low index bits, and an even K would give them to a few items); a range
// of fewer groups than K has the live tiles of each group dealt over several
// items.
template <typename Add>
void cut_tiles(uint32_t prog, uint32_t slot, uint64_t b, uint64_t e, uint64_t K, bool cofactor, double live,
               Add &&add) {
  fbg::BatchItem it;
  it.prog = prog;
  it.slot = slot;
  it.t1 = e;
  it.part = 0;
  K = std::max<uint64_t>(1, std::min(K, e - b));
  if (!cofactor) {
    it.step = (uint32_t)K;
    for (uint64_t k = 0; k < K; k++) {
      it.t0 = b + k;
      add(it, (double)((e - b - k + K - 1) / K));
    }
    return;
  }
  const uint64_t g0 = b / 64, groups = (e - 1) / 64 - g0 + 1;
  if (K < groups) {
    if (!(K & 1)) K++;
    it.step = (uint32_t)K;
    for (uint64_t k = 0; k < K; k++) {
      it.t0 = k == 0 ? b : (g0 + k) * 64;
      add(it, (double)((groups - k + K - 1) / K) * 64.0);
    }
    return;
  }
  // as many shares as K asks for, and once more where the live tiles of a
  // group, should they crowd four times as close as expected, would be more
  // than eight evaluations for a wave of the block
  uint32_t s = 0;
  while (s < 6 && (groups << (s + 1)) <= K) s++;
  const double crowd = 64.0 * std::min(1.0, 4.0 * live) / (double)(kWavesPerBlock << s);
  if (crowd > 8.0 && s < 6) s++;
  it.step = 1;
  for (uint64_t g = 0; g < groups; g++)
    for (uint32_t part = 0; part < (1u << s); part++) {
      it.t0 = g == 0 ? b : (g0 + g) * 64;
      it.t1 = std::min(e, (g0 + g + 1) * 64);
      it.part = part << 8 | s;
      add(it, (double)(it.t1 - it.t0) / (double)(1u << s));
    }
}

// Blocks that give each of nitems a taker, `per` of them to a block, in every queue:
// with 100 blocks for 400 items four queues had two takers too few, and the launch
// took as long as two items.
uint64_t queue_blocks(uint64_t nitems, int per) {
  const uint64_t longest = (nitems + fbg::kQueues - 1) / fbg::kQueues;
  return (longest + per - 1) / per * fbg::kQueues;
}

fbg::BatchProg batch_prog(const fbg_program *p, int l) {
  fbg::BatchProg b;
  memset(&b, 0, sizeof b);
  b.code = p->d_code + p->dev_off[l];
  b.nins = p->nins[l];
  b.nregs = lds_regs((uint32_t)p->c.nregs, l);
  b.n = p->c.n;
  b.nslices = p->nslices;
  b.ntiles = tiles_of(p->nslices, l);
  if (l == 5 && p->has_xcd && p->d_code) b.xcd_code = p->d_code + p->dev_off_xcd;
  return b;
}

// Up to this many units (fbg_device.h) an enumeration is two launches: the
// counts, then compaction blocks that add up the counts before them themselves.
// Beyond it the units that hold models are listed first (launch_tile_list, two
// small launches, about 5 us each), which also spreads them evenly over the
// waves.  A stored vector's counting pass leaves the sums of its blocks too, so
// that four times as many tiles can be added up.
constexpr uint64_t kDirectUnits = 4096;
constexpr uint64_t kDirectScanTiles = 16384;

// The enumeration temporaries for nu units, each part 256-byte aligned:
// per-unit uint32 counts and, in a direct pass, sums of wpb of them each
// (`sums`), else the list of the units that hold models (TileListArgs).
struct EnumTemp {
  size_t list = 0, sums = 0, base = 0, nlist = 0, bytes = 0;  // offsets, and the size of all
};

EnumTemp enum_temp(uint64_t nu, bool direct) {
  auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  EnumTemp t;
  t.list = t.sums = up(nu * 4);
  t.bytes = t.list + up(nu);
  if (direct) return t;
  const uint64_t nb = fbg::tile_list_blocks(nu);
  t.sums = t.list + up(nu * 8);
  t.base = t.sums + up(nb * sizeof(fbg::TilePair));
  t.nlist = t.base + up(nb * 8);
  t.bytes = t.nlist + 256;
  return t;
}

// Two-pass enumeration given the pass launcher and the temporaries `tmp`
// (enum_temp(a.nunits, a.direct).bytes of device memory): counts per unit, the
// list of the units that hold models unless direct, compaction.  Every
// temporary word is written before it is read.  pass.zero_counts (the
// uniform-cofactor passes, which write the counts of live tiles only): a fill
// kernel, or the one that makes the masks, clears the counts first, in one
// coalesced sweep instead of a scattered write per dead tile.
template <typename Pass>
hipError_t enumerate_passes(fbg::EvalArgs a, char *tmp, uint64_t *d_idx, uint64_t capacity, uint64_t *d_total,
                            hipStream_t s, const Pass &pass) {
  const EnumTemp t = enum_temp(a.nunits, a.direct);
  a.tile_counts = (uint32_t *)tmp;
  if (pass.block_sums && a.direct) a.block_sums = (uint32_t *)(tmp + t.sums);
  hipError_t e = hipSuccess;
  if (a.direct == fbg::ENUM_ONE_BLOCK) {
    a.out_idx = d_idx;
    a.capacity = capacity;
    a.out_count = d_total;
    return pass(fbg::EVAL_ENUM, a);
  }
  if (pass.masks()) {
    // the masks lie where the list comes later; a group set per 64 groups, its
    // live tiles over the waves of the device
    uint64_t *masks = (uint64_t *)(tmp + t.list);
    e = fbg::launch_cofactor_masks(a.code, a.ntiles / 64, masks, a.tile_counts, pass.fill_grid(), s);
    a.masks = masks;
    a.part_shift = 0;
    while (a.part_shift < 6 && (a.ntiles >> 12 << a.part_shift) < (uint64_t)pass.fill_grid() * kWavesPerBlock)
      a.part_shift++;
  } else if (pass.zero_counts()) {
    e = fbg::launch_zero((uint64_t *)tmp, t.list / 8, nullptr, 0, s);
  }
  if (e == hipSuccess) e = pass(fbg::EVAL_TILECNT, a);
  if (e != hipSuccess) return e;
  a.out_idx = d_idx;
  a.capacity = capacity;
  a.out_count = d_total;
  if (a.direct) return pass(fbg::EVAL_ENUM, a);
  fbg::TileListArgs l;
  l.counts = a.tile_counts;
  l.n = a.nunits;
  l.list = (uint64_t *)(tmp + t.list);
  l.sums = (fbg::TilePair *)(tmp + t.sums);
  l.list_base = (uint64_t *)(tmp + t.base);
  l.nlist = (uint64_t *)(tmp + t.nlist);
  l.total = d_total;
  e = fbg::launch_tile_list(l, s);
  if (e != hipSuccess || capacity == 0) return e;
  a.list = l.list;
  a.list_base = l.list_base;
  a.nlist = l.nlist;
  return pass(fbg::EVAL_ENUM, a);
}

// The same with a block of the device's scratch pool, or with the temporaries
// allocated on the stream and freed after.
template <typename Pass>
fbg_status enumerate_with(int dev, const fbg::EvalArgs &a, uint64_t *d_idx, uint64_t capacity, uint64_t *d_total,
                          hipStream_t s, const Pass &pass) {
  hipError_t e = hipSuccess;
  if (a.direct == fbg::ENUM_ONE_BLOCK) {  // no temporaries
    e = enumerate_passes(a, nullptr, d_idx, capacity, d_total, s, pass);
    return e == hipSuccess ? FBG_OK : hip_fail(e, "launch of an enumeration kernel");
  }
  const size_t bytes = enum_temp(a.nunits, a.direct).bytes;
  char *tmp = nullptr;
  fbg::ScratchPool &pool = fbg::ScratchPool::of(dev);
  const int block = pool.acquire(bytes, s, &tmp);
  if (block < 0) e = hipMallocAsync((void **)&tmp, bytes, s);
  if (e != hipSuccess) {
    (void)hipGetLastError();  // not an error of a later call's launches
    return fail(FBG_E_NOMEM, "hipMallocAsync of %zu bytes: %s", bytes, hipGetErrorString(e));
  }
  e = enumerate_passes(a, tmp, d_idx, capacity, d_total, s, pass);
  const hipError_t e2 = block < 0 ? hipFreeAsync(tmp, s) : pool.release(block, s);
  if (e != hipSuccess) return hip_fail(e, "launch of an enumeration kernel");
  if (e2 != hipSuccess) return hip_fail(e2, "release of the temporaries");
  return FBG_OK;
}

// The passes of enumerating a program: the counts on geometry g; the
// compaction in blocks of the same size, with LDS to gather models in.  (The
// compaction needs no cofactor variant: its tiles hold models.)
struct EvalPasses {
  static constexpr bool block_sums = false;
  const fbg_program *p;
  Geometry g;
  int var;
  hipStream_t s;
  bool masks() const { return (var & 4) != 0; }
  bool zero_counts() const { return (var & 2) != 0; }
  int fill_grid() const { return cu_count(p->device) * 8; }
  // Tiles are cut into units of at least four rows while there are fewer than
  // 32768: the models of a theory crowd into few tiles, and the fullest unit
  // is what the compaction waits for (tile_compact).
  fbg::EvalArgs args() const {
    fbg::EvalArgs a = base_args(p, g.log2w);
    while (g.log2w - (int)a.unit_shift > 2 && (a.ntiles << a.unit_shift) < 32768) a.unit_shift++;
    a.nunits = a.ntiles << a.unit_shift;
      if (a.nunits <= kDirectUnits) a.direct = fbg::ENUM_DIRECT;
    if (a.ntiles <= (uint64_t)(g.block / 64)) {
      a.direct = fbg::ENUM_ONE_BLOCK;
      a.unit_shift = 0;
      a.nunits = a.ntiles;
    }
    return a;
  }
  hipError_t operator()(int mode, fbg::EvalArgs a) const {
    if (mode != fbg::EVAL_ENUM) return fbg::launch_eval(mode, g.log2w, var, a, g.grid, g.block, g.lds, s);
    const size_t wpb = (size_t)g.block / 64;
    const size_t wave = std::max(lds_per_wave((uint32_t)p->c.nregs, g.log2w), (size_t)fbg::kStageModels * 2);
    a.lds_stride = (uint32_t)(wave / 4);
    const uint64_t blocks = (a.nunits + wpb - 1) / wpb;
    uint64_t grid = blocks;
    if (!a.direct)
      grid = std::min<uint64_t>(blocks, (uint64_t)cu_count(p->device) *
                                            (uint64_t)fbg::eval_blocks_per_cu(mode, g.log2w, var & 1, g.block, wave * wpb));
    return fbg::launch_eval(mode, g.log2w, var & 1, a, (int)grid, g.block, wave * wpb, s);
  }
};

// The passes of enumerating a stored vector: tiles of 8 KiB, of 1 KiB up to
// n = 27 so that small vectors still fill the device.
struct ScanPasses {
  static constexpr bool block_sums = true;
  int dev, log2w;
  hipStream_t s;
  bool masks() const { return false; }
  bool zero_counts() const { return false; }
  int fill_grid() const { return 1; }
  hipError_t operator()(int mode, const fbg::EvalArgs &a) const {
    const uint64_t blocks = (a.ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
    const uint64_t grid = a.direct ? blocks : std::min<uint64_t>(blocks, (uint64_t)cu_count(dev) * 8);
    return fbg::launch_dnf_scan(mode, log2w, a, (int)grid, 64 * kWavesPerBlock, s);
  }
};

}  // namespace

extern "C" {

const char *fbg_version(void) { return "fbg 0.2 (gfx950)"; }
const char *fbg_last_error(void) { return g_err.c_str(); }
int64_t fbg_last_error_offset(void) { return g_err_off; }

}  // extern "C"

namespace {

// The tiling that pick_log2w prefers, or the nearest one the program is
// encoded for (the larger of two equally near).
int nearest_tiling(uint32_t tilings, int l) {
  for (int d = 0; d <= kMaxLog2W; d++) {
    if (l + d <= kMaxLog2W && ((tilings >> (l + d)) & 1u)) return l + d;
    if (l - d >= 0 && ((tilings >> (l - d)) & 1u)) return l - d;
  }
  return l;
}

fbg_status check_flags(uint32_t flags) {
  if (flags & ~FBG_COMPILE_WPL_MASK)
    return fail(FBG_E_INVAL, "flags 0x%x: only FBG_COMPILE_WPL(0..5) bits are defined", flags);
  return FBG_OK;
}

fbg_status compile_common(const char *src, int32_t n_vars, const int32_t *subst, int32_t n_free, uint32_t flags,
                          fbg_program **out) {
  fbg_program *p = new (std::nothrow) fbg_program();
  if (!p) return fail(FBG_E_NOMEM, "out of host memory");
  p->tilings = flags & FBG_COMPILE_WPL_MASK ? flags & FBG_COMPILE_WPL_MASK : FBG_COMPILE_WPL_MASK;
  std::string msg;
  int64_t off = -1;
  int st = fbg::compile_formula(src, n_vars, p->c, msg, off, subst, n_free);
  if (st != FBG_OK) {
    delete p;
    g_err = msg;
    g_err_off = off;
    if (off >= 0) g_err += " (offset " + std::to_string(off) + ")";
    return (fbg_status)st;
  }
  p->nslices = slices_of(p->c.n);
  p->ncl = fbg::leading_clauses(p->c);
  for (int l = 0; l <= kMaxLog2W; l++) {
    if (!p->has_tiling(l)) continue;
    p->live[l] = expected_live(p, l);
    p->multi[l] = multi_clauses(p, l);
  }
  size_t total = 0;
  std::string enc_err;
  for (int l = 0; l <= kMaxLog2W; l++) {
    if (!p->has_tiling(l)) continue;  // not asked for: left empty
    p->nins[l] = fbg::encode_program(p->c, l, p->words[l], &enc_err);
    p->dev_off[l] = total;
    total += p->words[l].size();
  }
  if (!p->general() && p->c.n >= fbg::kXcdMinVars && p->has_tiling(5)) {
    const fbg::Compiled x = fbg::permute_variables(p->c, fbg::xcd_write_out_permutation(p->c.n));
    const uint32_t nx = fbg::encode_program(x, 5, p->words_xcd, &enc_err);
    if (nx != p->nins[5] && enc_err.empty()) enc_err = "internal: renamed encoding differs in length";
    p->dev_off_xcd = total;
    total += p->words_xcd.size();
    p->has_xcd = true;
  }
  if (!enc_err.empty()) {
    delete p;
    return fail(FBG_E_RANGE, "%s", enc_err.c_str());
  }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) == hipSuccess && ndev > 0) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
      delete p;
      return hip_fail(e, "hipGetDevice");
    }
    p->device = dev;
    std::vector<uint32_t> all;
    all.reserve(total + 64);
    for (int l = 0; l <= kMaxLog2W; l++) all.insert(all.end(), p->words[l].begin(), p->words[l].end());
    all.insert(all.end(), p->words_xcd.begin(), p->words_xcd.end());
    all.resize(all.size() + 64, 0);  // padding: scalar loads never run past the allocation
    e = CodeArena::of(dev).alloc(all.size() * sizeof(uint32_t), (void **)&p->d_code, p->code_class);
    p->code_bytes = p->code_class >= 0 ? (1ull << p->code_class) : all.size() * sizeof(uint32_t);
    if (e != hipSuccess) {
      delete p;
      return fail(FBG_E_NOMEM, "device memory for the program: %s", hipGetErrorString(e));
    }
    e = hipMemcpy(p->d_code, all.data(), all.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
      CodeArena::of(dev).release(p->d_code, p->code_class);
      delete p;
      return hip_fail(e, "hipMemcpy of the program");
    }
    p->auto_log2w = pick_log2w(p->nslices, (uint32_t)p->c.nregs, p->general(), dev);
  } else {
    p->auto_log2w = pick_log2w(p->nslices, (uint32_t)p->c.nregs, p->general(), -1);
  }
  p->auto_log2w = nearest_tiling(p->tilings, p->auto_log2w);
  p->one_count = one_block_log2w(p, false);
  p->one_list = one_block_log2w(p, true);
  if (p->d_code) fbg::ScratchPool::of(p->device).program_added();
  if (p->general() && p->has_tiling(FBG_J16_LOG2W))
    p->j16_cost = fbg::j16_general_cost(p->words[FBG_J16_LOG2W], p->nins[FBG_J16_LOG2W]);
  *out = p;
  return FBG_OK;
}

}  // namespace

extern "C" {

fbg_status fbg_compile(const char *src, int32_t n_vars, uint32_t flags, fbg_program **out) {
  if (!out) return fail(FBG_E_INVAL, "out is NULL");
  *out = nullptr;
  if (!src) return fail(FBG_E_INVAL, "src is NULL");
  fbg_status st = check_flags(flags);
  if (st) return st;
  if (n_vars < 0 || n_vars > FBG_MAX_VARS) return fail(FBG_E_RANGE, "n=%d out of range [0,%d]", n_vars, FBG_MAX_VARS);
  return compile_common(src, n_vars, nullptr, 0, flags, out);
}

fbg_status fbg_compile_assume(const char *src, int32_t n_vars, const int8_t *assume, uint32_t flags,
                              fbg_program **out) {
  if (!out) return fail(FBG_E_INVAL, "out is NULL");
  *out = nullptr;
  if (!src) return fail(FBG_E_INVAL, "src is NULL");
  fbg_status st = check_flags(flags);
  if (st) return st;
  if (n_vars < 0 || n_vars > FBG_MAX_TEXT_VARS)
    return fail(FBG_E_RANGE, "n=%d out of range [0,%d]", n_vars, FBG_MAX_TEXT_VARS);
  if (n_vars > 0 && !assume) return fail(FBG_E_INVAL, "assume is NULL");
  std::vector<int32_t> subst((size_t)n_vars);
  int32_t nfree = 0;
  for (int32_t k = 0; k < n_vars; k++) {
    if (assume[k] < -1 || assume[k] > 1)
      return fail(FBG_E_INVAL, "assume[%d] = %d (must be -1, 0 or 1)", k, (int)assume[k]);
    subst[(size_t)k] = assume[k] < 0 ? nfree++ : (assume[k] ? FBG_SUBST_ONE : FBG_SUBST_ZERO);
  }
  if (nfree > FBG_MAX_VARS) return fail(FBG_E_RANGE, "%d free variables (max %d)", nfree, FBG_MAX_VARS);
  return compile_common(src, n_vars, subst.data(), nfree, flags, out);
}

fbg_status fbg_compile_subst(const char *src, int32_t n_vars, const int32_t *subst, int32_t n_free, uint32_t flags,
                             fbg_program **out) {
  if (!out) return fail(FBG_E_INVAL, "out is NULL");
  *out = nullptr;
  if (!src) return fail(FBG_E_INVAL, "src is NULL");
  fbg_status st = check_flags(flags);
  if (st) return st;
  if (n_vars < 0 || n_vars > FBG_MAX_TEXT_VARS)
    return fail(FBG_E_RANGE, "n=%d out of range [0,%d]", n_vars, FBG_MAX_TEXT_VARS);
  if (n_free < 0 || n_free > FBG_MAX_VARS) return fail(FBG_E_RANGE, "n_free=%d out of range [0,%d]", n_free,
                                                       FBG_MAX_VARS);
  if (n_vars > 0 && !subst) return fail(FBG_E_INVAL, "subst is NULL");
  for (int32_t k = 0; k < n_vars; k++)
    if (subst[k] < FBG_SUBST_ONE || subst[k] >= n_free)
      return fail(FBG_E_INVAL, "subst[%d] = %d (must be -1, -2 or in [0, %d))", k, subst[k], n_free);
  return compile_common(src, n_vars, subst, n_free, flags, out);
}

void fbg_program_free(fbg_program *p) {
  if (!p) return;
  if (p->d_code) {
    CodeArena::of(p->device).release(p->d_code, p->code_class);
    fbg::ScratchPool::of(p->device).program_removed();
  }
  delete p;
}

fbg_status fbg_program_info(const fbg_program *p, struct fbg_program_info *out) {
  if (!p || !out) return fail(FBG_E_INVAL, "NULL argument");
  memset(out, 0, sizeof *out);
  out->n_vars = p->c.n;
  out->const_value = p->c.const_value;
  out->l2in = p->c.l2in;
  // clauses + instructions after them, in the plain form
  out->n_instr = (int32_t)p->c.code.size();
  out->n_regs = p->c.nregs;
  out->n_clause_instr = (int32_t)p->ncl;
  out->words_per_lane = 1 << p->auto_log2w;
  out->dnf_words = dnf_words_of(p->c.n);
  out->code_bytes = p->code_bytes;
  const int l = p->auto_log2w;
  out->l_valu = fbg::valu_per_slice(p->words[l], p->nins[l], l, (uint32_t)p->c.nregs);
  return FBG_OK;
}

fbg_status fbg_program_get_info(const fbg_program *p, struct fbg_program_info *out) {
  return fbg_program_info(p, out);
}

fbg_status fbg_program_set_tuning(fbg_program *p, const fbg_tune *tune) {
  if (!p || !tune) return fail(FBG_E_INVAL, "NULL argument");
  int l = p->auto_log2w;
  fbg_status st;
  if (tune->words_per_lane && (st = parse_wpl(tune->words_per_lane, l))) return st;
  if ((st = check_tiling(p, l))) return st;
  int wpb;
  size_t lds;
  if ((st = block_shape((uint32_t)p->c.nregs, l, wpb, lds))) return st;
  p->auto_log2w = l;
  p->tuned = p->tuned || tune->words_per_lane != 0;
  p->cofactor = (tune->flags & FBG_TUNE_COFACTOR) != 0;
  return FBG_OK;
}

uint64_t fbg_program_tiles(const fbg_program *p, int32_t words_per_lane) {
  int l;
  if (!p || parse_wpl(words_per_lane, l)) return 0;
  return tiles_of(p->nslices, l);
}

fbg_status fbg_count_tuned(const fbg_program *p, uint64_t *d_count, const fbg_tune *tune, void *stream) {
  fbg_status st = check_program(p);
  if (st) return st;
  if (!d_count) return fail(FBG_E_INVAL, "d_count is NULL");
  hipStream_t s = (hipStream_t)stream;
  hipError_t e;
  if (p->c.const_value >= 0) {
    e = fbg::launch_set_u64(d_count, p->c.const_value ? (1ull << p->c.n) : 0ull, s);
    return e == hipSuccess ? FBG_OK : hip_fail(e, "launch");
  }
  Geometry g;
  if ((st = geometry(p, tune, fbg::EVAL_COUNT, g))) return st;
  fbg::EvalArgs a = base_args(p, g.log2w);
  a.out_count = d_count;
  // (one block stores the count; more add to it)
  e = g.grid > 1 ? fbg::launch_set_u64(d_count, 0, s) : hipSuccess;
  if (e != hipSuccess) return hip_fail(e, "launch");
  e = fbg::launch_eval(fbg::EVAL_COUNT, g.log2w, g.var, a, g.grid, g.block, g.lds, s);
  return e == hipSuccess ? FBG_OK : hip_fail(e, "launch of the count kernel");
}

fbg_status fbg_count(const fbg_program *p, uint64_t *d_count, void *stream) {
  return fbg_count_tuned(p, d_count, nullptr, stream);
}

fbg_status fbg_eval_dnf_tuned(const fbg_program *p, uint64_t *d_out, uint64_t out_words, const fbg_tune *tune,
                              void *stream) {
  fbg_status st = check_program(p);
  if (st) return st;
  if (!d_out) return fail(FBG_E_INVAL, "d_out is NULL");
  if (p->c.n > FBG_MAX_DNF_VARS) return fail(FBG_E_RANGE, "n=%d above %d for a DNF vector", p->c.n, FBG_MAX_DNF_VARS);
  const uint64_t need = dnf_words_of(p->c.n);
  if (out_words < need)
    return fail(FBG_E_INVAL, "out_words=%llu < %llu", (unsigned long long)out_words, (unsigned long long)need);
  Geometry g;
  if ((st = geometry(p, tune, fbg::EVAL_DNF, g))) return st;
  fbg::EvalArgs a = base_args(p, g.log2w);
  a.out32 = (uint32_t *)d_out;
  a.out_slices = 2 * need;
  // the XCD-local layout (fbg_kernels.h) on the grid of one tile per wave
  if (g.log2w == 5 && p->has_xcd && g.var == 0 && ((uintptr_t)d_out & 15) == 0)
    a.xcd_code = p->d_code + p->dev_off_xcd;
  hipError_t e = fbg::launch_eval(fbg::EVAL_DNF, g.log2w, g.var, a, g.grid, g.block, g.lds, (hipStream_t)stream);
  return e == hipSuccess ? FBG_OK : hip_fail(e, "launch of the DNF kernel");
}

fbg_status fbg_eval_dnf(const fbg_program *p, uint64_t *d_out, uint64_t out_words, void *stream) {
  return fbg_eval_dnf_tuned(p, d_out, out_words, nullptr, stream);
}

fbg_status fbg_enumerate(const fbg_program *p, uint64_t *d_idx, uint64_t capacity, uint64_t *d_total,
                         void *stream) {
  fbg_status st = check_program(p);
  if (st) return st;
  if (!d_total) return fail(FBG_E_INVAL, "d_total is NULL");
  if (capacity > 0 && !d_idx)
    return fail(FBG_E_INVAL, "d_idx is NULL with capacity %llu", (unsigned long long)capacity);
  Geometry g;
  if ((st = geometry(p, nullptr, fbg::EVAL_TILECNT, g))) return st;
  const EvalPasses pass{p, g, g.var, (hipStream_t)stream};
  return enumerate_with(p->device, pass.args(), d_idx, capacity, d_total, pass.s, pass);
}

fbg_status fbg_enumerate_noalloc(const fbg_program *p, uint64_t *d_idx, uint64_t capacity, uint64_t *d_total,
                                 void *stream) {
  fbg_status st = check_program(p);
  if (st) return st;
  if (!d_total) return fail(FBG_E_INVAL, "d_total is NULL");
  if (capacity > 0 && !d_idx)
    return fail(FBG_E_INVAL, "d_idx is NULL with capacity %llu", (unsigned long long)capacity);
  Geometry g;
  if ((st = geometry(p, nullptr, fbg::EVAL_TILECNT, g))) return st;
  const EvalPasses pass{p, g, g.var, (hipStream_t)stream};
  const fbg::EvalArgs a = pass.args();
  const size_t bytes = enum_temp(a.nunits, a.direct).bytes;
  if (a.ntiles > fbg::kNoallocMaxTiles || bytes > fbg::kNoallocScratchBytes)
    return fail(FBG_E_RANGE,
                "fbg_enumerate_noalloc: %llu tiles at %d words per lane need %zu bytes of scratch; the static "
                "scratch holds %llu tiles (%llu bytes)",
                (unsigned long long)a.ntiles, 1 << g.log2w, bytes, (unsigned long long)fbg::kNoallocMaxTiles,
                (unsigned long long)fbg::kNoallocScratchBytes);
  void *scratch = nullptr;
  hipError_t e = fbg::noalloc_scratch(&scratch);
  if (e != hipSuccess) return hip_fail(e, "address of the static scratch");
  e = enumerate_passes(a, (char *)scratch, d_idx, capacity, d_total, pass.s, pass);
  return e == hipSuccess ? FBG_OK : hip_fail(e, "launch of an enumeration kernel");
}

fbg_status fbg_enumerate_dnf(const uint64_t *d_dnf, int32_t n_vars, uint64_t *d_idx, uint64_t capacity,
                             uint64_t *d_total, void *stream) {
  if (!d_dnf || !d_total) return fail(FBG_E_INVAL, "NULL device pointer");
  if (capacity > 0 && !d_idx)
    return fail(FBG_E_INVAL, "d_idx is NULL with capacity %llu", (unsigned long long)capacity);
  if (n_vars < 0 || n_vars > FBG_MAX_DNF_VARS) return fail(FBG_E_RANGE, "n=%d out of range", n_vars);
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  fbg::EvalArgs a;
  memset(&a, 0, sizeof a);
  a.n = n_vars;
  a.nslices = 2 * dnf_words_of(n_vars);  // bits at or above 2^n are zero in a DNF vector
  // (n <= 18: four tiles of 8 KiB, one block)
  const ScanPasses pass{dev, n_vars > 18 && n_vars <= 27 ? 2 : 5, (hipStream_t)stream};
  a.nunits = a.ntiles = tiles_of(a.nslices, pass.log2w);
  a.direct = a.nunits <= kWavesPerBlock     ? fbg::ENUM_ONE_BLOCK
             : a.nunits <= kDirectScanTiles ? fbg::ENUM_DIRECT
                                            : fbg::ENUM_LISTED;
  a.out32 = (uint32_t *)d_dnf;
  return enumerate_with(dev, a, d_idx, capacity, d_total, pass.s, pass);
}

// ------------------------------------------------------------------ batches

fbg_status fbg_batch_create(const fbg_program *const *ps, int32_t np, const fbg_tune *tune, fbg_batch **out) {
  if (!out) return fail(FBG_E_INVAL, "out is NULL");
  *out = nullptr;
  if (np <= 0 || !ps) return fail(FBG_E_INVAL, "empty batch");
  int dev = -1;
  for (int32_t i = 0; i < np; i++) {
    fbg_status st = check_program(ps[i]);
    if (st) return st;
    dev = ps[i]->device;
  }
  fbg_status st;
  int fixed_l = -1;
  if (tune && tune->words_per_lane && (st = parse_wpl(tune->words_per_lane, fixed_l))) return st;
  if (tune && (tune->direct_run < 0 || tune->direct_run > 64))
    return fail(FBG_E_INVAL, "direct_run must be 0..64 (got %d)", tune->direct_run);
  const int cus = cu_count(dev);

  fbg_batch *b = new (std::nothrow) fbg_batch();
  if (!b) return fail(FBG_E_NOMEM, "out of host memory");
  b->device = dev;
  b->np = np;
  b->host_progs.resize((size_t)np);
  b->plan_of.assign((size_t)np, 0);
  std::vector<std::vector<fbg::BatchItem>> plan_items;
  std::vector<std::vector<fbg::BatchItem>> plan_direct;  // per plan: one entry per program (clause-only plans)
  // 0: clause-only programs; 1: general programs whose registers all fit in
  // VGPRs (at every tiling); 2: up to four registers in LDS; 3: more.  The LDS a plan's widest
  // program needs per wave sets the occupancy of the whole plan, so the few
  // register-hungry programs do not slow down the rest.
  // At 16 words per lane (the jump-table form) a plan keeps at most
  // kJ16LdsRegs registers of a wave in LDS and the rest in global scratch,
  // so the register count no longer limits occupancy: when the tuning fixes
  // that tiling and some program has a general part, every program goes into
  // one plan, one persistent launch.
  bool any_general = false;
  for (int32_t i = 0; i < np; i++) any_general = any_general || ps[i]->general();
  // (the library's own choice for a batch with general programs when the
  // tuning does not fix the tiling)
  if (fixed_l < 0 && any_general) fixed_l = FBG_J16_LOG2W;
  const bool one_plan = fixed_l == FBG_J16_LOG2W && any_general;
  auto group_of = [one_plan](const fbg_program *q) {
    if (one_plan) return 1;
    if (!q->general()) return 0;
    const uint32_t r = lds_regs((uint32_t)q->c.nregs, FBG_J16_LOG2W);
    return r == 0 ? 1 : (r <= 4 ? 2 : 3);
  };
  for (int group = 0; group < 4; group++) {
    std::vector<int32_t> members;
    for (int32_t i = 0; i < np; i++)
      if (group_of(ps[i]) == group) members.push_back(i);
    if (members.empty()) continue;
    // words per lane: the tuning, else the choice for the largest program,
    // or more while the tiles of all programs together still give half the
    // waves of a full device one each (a tile costs little more at twice the
    // words: 16 systems of 2^24 valuations took 352 us to count at the one word
    // per lane that suits one of them, 36 at 32 words); not 32 where two clauses in
    // five have several word literals (16 systems of 1500 clauses of 10 literals over
    // 26 letters, 66 % of them: 1135 us at 32 words, 909 at 16; of 300 of 8 literals, 50 %:
    // 235 and 221; of 130 of 5 literals, 20 %: 88 and 104)
    int l = fixed_l;
    if (l < 0) {
      uint64_t best = 0;
      bool tuned = false;
      l = 0;
      for (int32_t i : members) {
        const uint64_t cost = ps[i]->nslices * (uint64_t)std::max<size_t>(1, ps[i]->c.code.size());
        if (cost >= best) {
          best = cost;
          l = ps[i]->auto_log2w;
          tuned = ps[i]->tuned;
        }
      }
      for (int up = kMaxLog2W; up > l && !tuned; up--) {
        uint64_t tiles = 0, clauses = 0, multi = 0;
        bool all = true;
        for (int32_t i : members) {
          tiles += tiles_of(ps[i]->nslices, up);
          all = all && ps[i]->has_tiling(up);
          if (up == kMaxLog2W) clauses += ps[i]->ncl, multi += ps[i]->multi[up];
        }
        if (all && tiles >= (uint64_t)cus * 16 && 5 * multi <= 2 * clauses) l = up;
      }
    }
    uint32_t max_regs = 0;
    int var = 0;
    for (int32_t i : members) {
      if (!ps[i]->has_tiling(l)) {
        fbg_batch_free(b);
        return fail(FBG_E_INVAL, "program %d was compiled without %d words per lane (FBG_COMPILE_WPL)", i, 1 << l);
      }
      max_regs = std::max<uint32_t>(max_regs, (uint32_t)ps[i]->c.nregs);
      var |= ps[i]->variant(tune);
    }
    if (one_plan) var |= 1;  // clause-only programs run in the general kernel too
    // registers that stay in LDS, the rest (jump-table form only) in global
    // scratch, gstride words per wave
    uint32_t lds_keep = lds_regs(max_regs, l < 0 ? 0 : l);
    uint64_t gstride = 0;
    if (l == FBG_J16_LOG2W && lds_keep > kJ16LdsRegs) {
      gstride = (uint64_t)(lds_keep - kJ16LdsRegs) * (64u << l);
      lds_keep = kJ16LdsRegs;
    }
    if (gstride == 0) {
      while (l > 0 && lds_per_wave(max_regs, l) > kMaxLdsPerBlock) l--;
      // LDS registers: keep a block of 4 waves within 32 KiB (5 blocks per CU)
      if (fixed_l < 0)
        while (l > 0 && lds_per_wave(max_regs, l) * kWavesPerBlock > kMaxLdsPerBlock / 2) l--;
      lds_keep = lds_regs(max_regs, l);
    }
    int wpb;
    size_t lds;
    if ((st = block_shape(lds_keep + fbg::vgpr_regs_of(l), l, wpb, lds))) {
      fbg_batch_free(b);
      return st;
    }
    // Without the test where it would spare less than half of the work: an item is a wave's
    // then, not a block's, and a tile whose clauses leave no model ends early anyhow (share
    // spared, us with the test, without: 40 DAGs 0, 105 and 15; 92 DAGs 0.14, 181 and 43; 60
    // larger ones 0.11, 1956 and 1685; 40 systems of 150 clauses of 5 literals 0.05, 381 and
    // 286; 14 3-CNF systems of 2 clauses a letter 0.6, 169 and 153, at 32 words 160 and
    // 117; 25 of 4 a letter 0.96, 127 and 332; scripts 0.98, 77 and 84).
    double all = 0, dead = 0;
    for (int32_t i : members) {
      const double cost = (double)tiles_of(ps[i]->nslices, l) * tile_cost(ps[i], l);
      all += cost, dead += cost * (1.0 - ps[i]->live[l]);
    }
    if (2.0 * dead < all) var &= ~2;
    const bool cofactor = (var & 2) != 0;
    auto per_tile = [&](int32_t i) { return cofactor ? cofactor_tile_cost(ps[i], l) : tile_cost(ps[i], l); };
    double total_cost = 0;
    for (int32_t i : members) {
      fbg::BatchProg &q = b->host_progs[(size_t)i];
      q = batch_prog(ps[i], l);
      total_cost += (double)q.ntiles * per_tile(i);
      b->plan_of[(size_t)i] = (int)b->plans.size();
    }
    // Items of about equal cost T, never below one tile.  Pops are atomics at
    // eight addresses, about 3 ns each over all (65,536 items: 197 us whatever
    // the work), and the queues end unevenly by about T steps of 40 to 60 ns: for
    // the S steps of a batch the sum is least near T = sqrt(S / 16) with a general
    // part, but no more than 550 (256 DAGs: T = 275 362 us, 550 318, 997 320) and no
    // finer than a sixteenth of a wave's share (1024 DAGs: T = 986 1056 us, 2009
    // 1098); a step of clauses is shorter (2.7 VALU instructions, 16 in the general
    // part, and most tiles stop early), which puts T at sqrt(S / 6) (64 systems of
    // 2^26 valuations: sqrt(S / 3) 43.5 us, so 36.9).
    // All that holds for items that are popped.  The first ones, one for each wave of a
    // full grid, are taken without a pop (k_batch): where T gives more than that, a plan
    // keeps to them while they are short: below 5,000 steps of clauses (16 systems of 2^28
    // valuations: 7,296 items of 8,192 26.9 us, 10,928 items 86; of 2^30, 4,500 steps,
    // 15,424 items 115, so 56; 30 systems of 2^20 to 2^29 77 and 38), below 1,200 with a
    // general part (92 DAGs with n <= 28: 5,566 items 61.7, so 42; 256 DAGs, 4,030 steps,
    // 314 and 382).  Longer ones leave waves without work where programs or their tiles
    // differ (13 theories, equivalence relations on 9 elements the largest, 35,000 steps:
    // 207 us, so 513; 256 layerings of posets, 200,000 steps: 1545 and 4010).
    // Items of falling size, half the work first, bring more programs at a time into
    // the scalar cache (the 1024: 5 % slower).  With the uniform cofactor an item is a
    // block's: about eight per block.  A clause program has an odd number of items, if they
    // are long enough to differ little: tiles that do not end early share low index
    // bits (16 systems of 2^30 valuations in 512 items each 92 us, in 511 56).
    // A program's items interleave, so the waves working on neighbouring items
    // at the same time write neighbouring tiles (DNF vectors), which keeps the
    // HBM writes close together.
    double target = std::sqrt(total_cost / 6.0);
    if (cofactor)
      target = std::max(1.0, total_cost / (double)(cus * 64));
    else if (var & 1)
      target = std::max(total_cost / (double)(cus * 256), std::min(std::sqrt(total_cost / 16.0), 550.0));
    auto chunk_of = [&](double w, double t) { return (uint64_t)std::max(1.0, t / w); };
    auto items_at = [&](double t) {
      uint64_t n = 0;
      for (int32_t i : members) {
        const uint64_t nt = b->host_progs[(size_t)i].ntiles, chunk = chunk_of(per_tile(i), t);
        n += (nt + chunk - 1) / chunk;
      }
      return n;
    };
    uint64_t full = (uint64_t)cus * (uint64_t)fbg::batch_blocks_per_cu(fbg::EVAL_COUNT, l, var, 64 * wpb, lds);
    if (tune && tune->grid_blocks > 0) full = (uint64_t)tune->grid_blocks;
    full *= (uint64_t)wpb;
    if (!cofactor && members.size() < full && items_at(target) > full) {
      double each = std::max(target, total_cost / (double)full);
      while (items_at(each) > full) each *= 1.02;  // (every program has one item in the end)
      if (each < ((var & 1) ? 1200.0 : 5000.0)) target = each;
    }
    std::vector<fbg::BatchItem> items;
    std::vector<double> cost;
    for (int32_t i : members) {
      const fbg::BatchProg &q = b->host_progs[(size_t)i];
      const double w = per_tile(i);
      const uint64_t chunk = chunk_of(w, target);
      uint64_t K = (q.ntiles + chunk - 1) / chunk;
      if (!(var & 1) && chunk >= 16 && K > 2 && !(K & 1)) K--;
      cut_tiles((uint32_t)i, (uint32_t)i, 0, q.ntiles, K, cofactor, ps[i]->live[l],
                [&](const fbg::BatchItem &it, double tiles) {
                  items.push_back(it);
                  cost.push_back(tiles * w);
                });
    }
    if (items.size() > 0xFFFFFFF0ull) {
      fbg_batch_free(b);
      return fail(FBG_E_RANGE, "too many work items");
    }
    // largest first, so that the queue ends on small items
    std::vector<size_t> order(items.size());
    for (size_t k = 0; k < order.size(); k++) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) { return cost[x] > cost[y]; });
    std::vector<fbg::BatchItem> sorted;
    sorted.reserve(items.size());
    for (size_t k : order) sorted.push_back(items[k]);

    fbg_batch::Plan pl;
    pl.log2w = l;
    pl.var = var;
    pl.block = 64 * wpb;
    pl.lds = lds;
    pl.nitems = (uint32_t)sorted.size();
    // popped ahead where items are short, about 100 us: one popped early waits while
    // other waves end; of clauses alone always, whose tiles mostly end early, unless a
    // quarter have several word literals (the 13 theories 302 us, so 212; 16 systems of
    // 2^35 valuations 646 and 545; systems of 2 to 7 literals, 27 %, 776 and 855)
    uint64_t clauses = 0, multi = 0;
    for (int32_t i : members) clauses += ps[i]->ncl, multi += ps[i]->multi[l];
    pl.pop_ahead = cofactor || (var & 1) ? (cofactor ? target / wpb : target) < ((var & 1) ? 1200.0 : 7200.0)
                                         : 4 * multi < clauses;
    if (tune && tune->direct_run > 0) pl.direct_run = (uint32_t)tune->direct_run;
    pl.max_regs = lds_keep;
    pl.gstride = gstride;
    const uint64_t want = queue_blocks(pl.nitems, cofactor ? 1 : wpb);
    for (int mode : {fbg::EVAL_COUNT, fbg::EVAL_DNF}) {
      uint64_t maxb = (uint64_t)cus * (uint64_t)fbg::batch_blocks_per_cu(mode, l, var, pl.block, lds);
      if (tune && tune->grid_blocks > 0) maxb = (uint64_t)tune->grid_blocks;
      (mode == fbg::EVAL_COUNT ? pl.grid : pl.grid_dnf) = (int)std::max<uint64_t>(1, std::min<uint64_t>(want, maxb));
    }
    std::vector<fbg::BatchItem> direct;
    if (var == 0 && !(tune && tune->grid_blocks > 0)) {
      bool any_xcd = false;
      for (int32_t i : members) {
        const fbg::BatchProg &q = b->host_progs[(size_t)i];
        if (q.xcd_code) {
          // the XCD-local layout: the program starts at a multiple of 32
          // tiles, so that block k of its waves runs on XCD k mod 8 (the
          // tiles in between belong to no program and are skipped)
          pl.ntiles = (pl.ntiles + 31) & ~(uint64_t)31;
          any_xcd = true;
        }
        fbg::BatchItem it;
        it.prog = (uint32_t)i;
        it.slot = (uint32_t)i;
        it.t0 = pl.ntiles;
        it.t1 = pl.ntiles + q.ntiles;
        it.step = 1;
        it.part = 0;
        direct.push_back(it);
        pl.ntiles += q.ntiles;
        pl.max_prog_tiles = std::max<uint64_t>(pl.max_prog_tiles, q.ntiles);
      }
      pl.ndirect = (uint32_t)direct.size();
      // one tile per wave, four waves per block: a block's tiles share bits
      // 2..4 of their tile index, i.e. one residue class of 4 KiB pieces
      if (any_xcd && !(tune && tune->direct_run > 0)) pl.direct_run = 1;
      // fewer tiles than that many for every wave: shorter runs, on all of the device (16
      // systems of 2^22 valuations and 1500 clauses of 10 literals, 4096 tiles: runs of four
      // 346 us, of one 111; 200 of 2^18 and 300 of 8 literals 61 and 30)
      if (!(tune && tune->direct_run > 0))
        while (pl.direct_run > 1 && pl.ntiles < (uint64_t)cus * 32 * pl.direct_run) pl.direct_run /= 2;
    }
    b->plans.push_back(pl);
    plan_items.push_back(std::move(sorted));
    plan_direct.push_back(std::move(direct));
  }
  hipError_t e = hipMalloc((void **)&b->d_progs, (size_t)np * sizeof(fbg::BatchProg));
  if (e == hipSuccess) e = hipMalloc((void **)&b->d_head, 4 * fbg::kHeadWords * sizeof(uint32_t));
  for (size_t k = 0; k < b->plans.size() && e == hipSuccess; k++) {
    fbg_batch::Plan &pl = b->plans[k];
    if (pl.gstride == 0) continue;
    const uint64_t waves_max = (uint64_t)std::max(pl.grid, pl.grid_dnf) * (uint64_t)(pl.block / 64);
    e = hipMalloc((void **)&pl.d_gscratch, waves_max * pl.gstride * sizeof(uint32_t));
  }
  for (size_t k = 0; k < b->plans.size() && e == hipSuccess; k++) {
    e = hipMalloc((void **)&b->plans[k].d_items, plan_items[k].size() * sizeof(fbg::BatchItem));
    if (e == hipSuccess)
      e = hipMemcpy(b->plans[k].d_items, plan_items[k].data(), plan_items[k].size() * sizeof(fbg::BatchItem),
                    hipMemcpyHostToDevice);
    if (e == hipSuccess && !plan_direct[k].empty()) {
      e = hipMalloc((void **)&b->plans[k].d_direct, plan_direct[k].size() * sizeof(fbg::BatchItem));
      if (e == hipSuccess)
        e = hipMemcpy(b->plans[k].d_direct, plan_direct[k].data(), plan_direct[k].size() * sizeof(fbg::BatchItem),
                      hipMemcpyHostToDevice);
    }
  }
  if (e == hipSuccess)
    e = hipMemcpy(b->d_progs, b->host_progs.data(), (size_t)np * sizeof(fbg::BatchProg), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    fbg_batch_free(b);
    return fail(FBG_E_NOMEM, "batch upload: %s", hipGetErrorString(e));
  }
  *out = b;
  return FBG_OK;
}

}  // extern "C"

namespace {

fbg_status batch_launch(fbg_batch *b, int mode, const fbg::BatchProg *d_progs, uint64_t *d_counts, hipStream_t s) {
  // zero the counts and every plan's queue head, then one persistent kernel per plan
  hipError_t e = fbg::launch_zero(d_counts, (uint64_t)b->np, b->d_head, (uint32_t)b->plans.size() * fbg::kHeadWords, s);
  if (e != hipSuccess) return hip_fail(e, "launch of the zero fill");
  for (size_t k = 0; k < b->plans.size(); k++) {
    const fbg_batch::Plan &pl = b->plans[k];
    fbg::BatchArgs a;
    a.progs = d_progs;
    a.items = pl.d_items;
    a.nitems = pl.nitems;
    a.max_regs = pl.max_regs;
    a.pop_ahead = pl.pop_ahead;
    a.head = b->d_head + k * fbg::kHeadWords;
    a.counts = d_counts;
    a.gscratch = pl.d_gscratch;
    a.gstride = pl.gstride;
    a.j16_any = j16_any();
    if (mode == fbg::EVAL_DNF && pl.d_direct && b->d_tile_counts) {
      // one wave per tile over the plan's programs in order; counts from the
      // tile counts
      a.items = pl.d_direct;
      a.nitems = pl.ndirect;
      a.run = pl.direct_run;
      const uint64_t wpb = (uint64_t)(pl.block / 64);
      const uint64_t waves = (pl.ntiles + a.run - 1) / a.run;
      const uint64_t grid = (waves + wpb - 1) / wpb;
      // about 1024 tiles per block of the count sums (C1: 64 per program)
      const int sum_blocks = (int)std::min<uint64_t>(256, std::max<uint64_t>(1, pl.max_prog_tiles / 1024));
      e = fbg::launch_batch_direct(pl.log2w, a, (int)grid, pl.block, sum_blocks, s);
      if (e != hipSuccess) return hip_fail(e, "launch of the batch kernel");
      continue;
    }
    e = fbg::launch_batch(mode, pl.log2w, pl.var, a, mode == fbg::EVAL_DNF ? pl.grid_dnf : pl.grid, pl.block, pl.lds,
                          s);
    if (e != hipSuccess) return hip_fail(e, "launch of the batch kernel");
  }
  return FBG_OK;
}

}  // namespace

extern "C" {

fbg_status fbg_batch_count(fbg_batch *b, uint64_t *d_counts, void *stream) {
  if (!b) return fail(FBG_E_INVAL, "batch is NULL");
  if (!d_counts) return fail(FBG_E_INVAL, "d_counts is NULL");
  fbg_status st = check_device(b->device);
  if (st) return st;
  return batch_launch(b, fbg::EVAL_COUNT, b->d_progs, d_counts, (hipStream_t)stream);
}

fbg_status fbg_batch_set_dnf_outputs(fbg_batch *b, uint64_t *const *d_outs, const uint64_t *out_words) {
  if (!b) return fail(FBG_E_INVAL, "batch is NULL");
  if (!d_outs || !out_words) return fail(FBG_E_INVAL, "NULL argument");
  fbg_status st = check_device(b->device);
  if (st) return st;
  std::vector<fbg::BatchProg> t = b->host_progs;
  for (int32_t i = 0; i < b->np; i++) {
    fbg::BatchProg &q = t[(size_t)i];
    if (q.n > FBG_MAX_DNF_VARS) return fail(FBG_E_RANGE, "program %d: n=%d above %d for a DNF vector", i, q.n,
                                            FBG_MAX_DNF_VARS);
    const uint64_t need = dnf_words_of(q.n);
    if (!d_outs[i]) return fail(FBG_E_INVAL, "d_outs[%d] is NULL", i);
    if (out_words[i] < need)
      return fail(FBG_E_INVAL, "out_words[%d]=%llu < %llu", i, (unsigned long long)out_words[i],
                  (unsigned long long)need);
    q.out32 = (uint32_t *)d_outs[i];
    q.out_slices = 2 * need;
    // the XCD-local layout writes 16-byte groups: other outputs take the
    // plain one
    if ((uintptr_t)q.out32 & 15) q.xcd_code = nullptr;
    if (!b->host_dnf.empty()) {
      q.tile_counts = b->host_dnf[(size_t)i].tile_counts;
      q.chunk_counts = b->host_dnf[(size_t)i].chunk_counts;
    }
  }
  hipError_t e = hipSuccess;
  if (!b->d_progs_dnf) e = hipMalloc((void **)&b->d_progs_dnf, t.size() * sizeof(fbg::BatchProg));
  if (e == hipSuccess) e = hipMemcpy(b->d_progs_dnf, t.data(), t.size() * sizeof(fbg::BatchProg), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "upload of the DNF output table");
  b->host_dnf = t;
  return FBG_OK;
}

fbg_status fbg_batch_set_enum_outputs(fbg_batch *b, uint64_t *const *d_idx, const uint64_t *capacity) {
  if (!b) return fail(FBG_E_INVAL, "batch is NULL");
  if (!d_idx || !capacity) return fail(FBG_E_INVAL, "NULL argument");
  if (b->host_dnf.empty()) return fail(FBG_E_INVAL, "set the DNF outputs first (fbg_batch_set_dnf_outputs)");
  fbg_status st = check_device(b->device);
  if (st) return st;
  for (int32_t i = 0; i < b->np; i++)
    if (capacity[i] > 0 && !d_idx[i]) return fail(FBG_E_INVAL, "d_idx[%d] is NULL with capacity %llu", i,
                                                  (unsigned long long)capacity[i]);
  // programs whose DNF write-out takes the XCD-local layout: two piece
  // counts per tile
  auto xcd_direct = [&](int32_t i) {
    return b->host_progs[(size_t)i].xcd_code && b->plans[(size_t)b->plan_of[(size_t)i]].d_direct;
  };
  hipError_t e = hipSuccess;
  if (!b->d_tile_counts) {
    uint64_t total = 0, chunks = 0;
    for (int32_t i = 0; i < b->np; i++) {
      total += b->host_progs[(size_t)i].ntiles;
      if (xcd_direct(i)) chunks += 2 * b->host_progs[(size_t)i].ntiles;
    }
    if (total >= (1ull << 32)) return fail(FBG_E_RANGE, "%llu tiles: batched enumeration lists tiles in 32 bits",
                                           (unsigned long long)total);
    b->total_tiles = total;
    const uint64_t nb = std::max<uint64_t>(fbg::tile_list_blocks(total), 1);
    e = hipMalloc((void **)&b->d_tile_counts, std::max<uint64_t>(total, 1) * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMalloc((void **)&b->d_tile_list, std::max<uint64_t>(total, 1) * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMalloc((void **)&b->d_list_sums, nb * sizeof(fbg::TilePair));
    if (e == hipSuccess) e = hipMalloc((void **)&b->d_list_base, (nb + 1 + (uint64_t)b->np) * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMalloc((void **)&b->d_enum, (size_t)b->np * sizeof(fbg::EnumProg));
    if (e == hipSuccess && chunks) e = hipMalloc((void **)&b->d_chunk_counts, chunks * sizeof(uint32_t));
    if (e != hipSuccess) return fail(FBG_E_NOMEM, "enumeration buffers: %s", hipGetErrorString(e));
  }
  std::vector<fbg::EnumProg> ep((size_t)b->np);
  uint64_t tile0 = 0, chunk0 = 0;
  for (int32_t i = 0; i < b->np; i++) {
    fbg::BatchProg &q = b->host_dnf[(size_t)i];
    q.tile_counts = b->d_tile_counts + tile0;
    q.chunk_counts = nullptr;
    if (xcd_direct(i)) {
      q.chunk_counts = b->d_chunk_counts + chunk0;
      chunk0 += 2 * q.ntiles;
    }
    fbg::EnumProg &x = ep[(size_t)i];
    memset(&x, 0, sizeof x);
    x.dnf = q.out32;
    x.nslices = q.nslices;
    x.tile0 = tile0;
    x.out = d_idx[i];
    x.capacity = capacity[i];
    x.log2w = (uint32_t)b->plans[(size_t)b->plan_of[(size_t)i]].log2w;
    tile0 += q.ntiles;
  }
  e = hipMemcpy(b->d_enum, ep.data(), ep.size() * sizeof(fbg::EnumProg), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(b->d_progs_dnf, b->host_dnf.data(), b->host_dnf.size() * sizeof(fbg::BatchProg),
                  hipMemcpyHostToDevice);
  return e == hipSuccess ? FBG_OK : hip_fail(e, "upload of the enumeration tables");
}

fbg_status fbg_batch_enumerate(fbg_batch *b, void *stream) {
  if (!b) return fail(FBG_E_INVAL, "batch is NULL");
  if (!b->d_enum) return fail(FBG_E_INVAL, "no enumeration outputs set (fbg_batch_set_enum_outputs)");
  fbg_status st = check_device(b->device);
  if (st) return st;
  hipStream_t s = (hipStream_t)stream;
  const uint64_t nb = fbg::tile_list_blocks(b->total_tiles);
  fbg::TileListArgs l;
  l.counts = b->d_tile_counts;
  l.n = b->total_tiles;
  l.sums = b->d_list_sums;
  l.list = b->d_tile_list;
  l.list_base = b->d_list_base;
  l.nlist = b->d_list_base + nb;
  l.total = nullptr;
  l.progs = b->d_enum;
  l.prog_base = b->d_list_base + nb + 1;
  l.np = (uint32_t)b->np;
  hipError_t e = fbg::launch_tile_list(l, s);
  if (e != hipSuccess) return hip_fail(e, "launch of the tile listing");
  fbg::BatchEnumArgs a;
  a.progs = b->d_enum;
  a.np = (uint32_t)b->np;
  a.list = l.list;
  a.list_base = l.list_base;
  a.nlist = l.nlist;
  a.prog_base = l.prog_base;
  const int grid = cu_count(b->device) * 8;
  for (const auto &pl : b->plans) {
    e = fbg::launch_batch_compact(pl.log2w, a, grid, 256, s);
    if (e != hipSuccess) return hip_fail(e, "launch of the compaction kernel");
  }
  return FBG_OK;
}

fbg_status fbg_batch_eval_dnf(fbg_batch *b, uint64_t *d_counts, void *stream) {
  if (!b) return fail(FBG_E_INVAL, "batch is NULL");
  if (!d_counts) return fail(FBG_E_INVAL, "d_counts is NULL");
  if (!b->d_progs_dnf) return fail(FBG_E_INVAL, "no DNF outputs set (fbg_batch_set_dnf_outputs)");
  fbg_status st = check_device(b->device);
  if (st) return st;
  return batch_launch(b, fbg::EVAL_DNF, b->d_progs_dnf, d_counts, (hipStream_t)stream);
}

fbg_status fbg_batch_count_graph(fbg_batch *b, uint64_t *d_counts, void *stream) {
  if (!b) return fail(FBG_E_INVAL, "batch is NULL");
  if (!d_counts) return fail(FBG_E_INVAL, "d_counts is NULL");
  fbg_status st = check_device(b->device);
  if (st) return st;
  hipError_t e;
  if (!b->graph_exec || b->graph_counts != d_counts) {
    if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->graph_exec = nullptr;
    b->graph = nullptr;
    hipStream_t cs;
    if ((e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking)) != hipSuccess) return hip_fail(e, "stream");
    e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      st = fbg_batch_count(b, d_counts, cs);  // kernels only: no memset node, no allocation
      hipError_t e2 = hipStreamEndCapture(cs, &b->graph);
      if (st == FBG_OK && e2 != hipSuccess) st = hip_fail(e2, "hipStreamEndCapture");
      if (st == FBG_OK && (e2 = hipGraphInstantiate(&b->graph_exec, b->graph, nullptr, nullptr, 0)) != hipSuccess)
        st = hip_fail(e2, "hipGraphInstantiate");
    } else {
      st = hip_fail(e, "hipStreamBeginCapture");
    }
    (void)hipStreamDestroy(cs);
    if (st) return st;
    b->graph_counts = d_counts;
  }
  e = hipGraphLaunch(b->graph_exec, (hipStream_t)stream);
  return e == hipSuccess ? FBG_OK : hip_fail(e, "hipGraphLaunch");
}

void fbg_batch_free(fbg_batch *b) {
  if (!b) return;
  if (b->graph_exec) (void)hipGraphExecDestroy(b->graph_exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  if (b->d_progs) (void)hipFree(b->d_progs);
  if (b->d_progs_dnf) (void)hipFree(b->d_progs_dnf);
  if (b->d_tile_counts) (void)hipFree(b->d_tile_counts);
  if (b->d_chunk_counts) (void)hipFree(b->d_chunk_counts);
  if (b->d_list_sums) (void)hipFree(b->d_list_sums);
  if (b->d_list_base) (void)hipFree(b->d_list_base);
  if (b->d_enum) (void)hipFree(b->d_enum);
  if (b->d_tile_list) (void)hipFree(b->d_tile_list);
  for (auto &pl : b->plans) {
    if (pl.d_items) (void)hipFree(pl.d_items);
    if (pl.d_direct) (void)hipFree(pl.d_direct);
    if (pl.d_gscratch) (void)hipFree(pl.d_gscratch);
  }
  if (b->d_head) (void)hipFree(b->d_head);
  delete b;
}

fbg_status fbg_count_batch(const fbg_program *const *ps, int32_t np, uint64_t *d_counts, const fbg_tune *tune,
                           void *stream) {
  fbg_batch *b = nullptr;
  fbg_status st = fbg_batch_create(ps, np, tune, &b);
  if (st) return st;
  st = fbg_batch_count(b, d_counts, stream);
  // the plan must outlive the launch
  hipError_t e = hipStreamSynchronize((hipStream_t)stream);
  fbg_batch_free(b);
  if (st) return st;
  return e == hipSuccess ? FBG_OK : hip_fail(e, "hipStreamSynchronize");
}

// ------------------------------------------------------------------ serving

fbg_status fbg_server_create(int32_t max_programs, int32_t max_items, int32_t words_per_lane, int32_t nbuf,
                             int32_t flags, fbg_server **out) {
  if (!out) return fail(FBG_E_INVAL, "out is NULL");
  *out = nullptr;
  if (max_programs <= 0 || max_items <= 0 || nbuf <= 0 || nbuf > 64) return fail(FBG_E_INVAL, "bad server sizes");
  int l;
  fbg_status st = parse_wpl(words_per_lane, l);
  if (st) return st;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  fbg_server *sv = new (std::nothrow) fbg_server();
  if (!sv) return fail(FBG_E_NOMEM, "out of host memory");
  sv->device = dev;
  sv->log2w = l;
  sv->max_programs = max_programs;
  sv->max_items = max_items;
  sv->nbuf = nbuf;
  sv->cofactor = (flags & FBG_TUNE_COFACTOR) != 0;
  sv->slots.resize((size_t)nbuf);
  const size_t bytes = kServerHeadBytes + (size_t)max_programs * sizeof(fbg::BatchProg) +
                       (size_t)max_items * sizeof(fbg::BatchItem);
  for (auto &sl : sv->slots) {
    e = hipHostMalloc((void **)&sl.h, bytes, hipHostMallocDefault);
    if (e == hipSuccess) memset(sl.h, 0, kServerHeadBytes);
    if (e == hipSuccess) e = hipMalloc((void **)&sl.d, bytes);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&sl.done, hipEventDisableTiming);
    if (e != hipSuccess) {
      fbg_server_free(sv);
      return fail(FBG_E_NOMEM, "server buffers: %s", hipGetErrorString(e));
    }
  }
  *out = sv;
  return FBG_OK;
}

fbg_status fbg_server_launch(fbg_server *sv, const fbg_program *const *ps, int32_t np, const fbg_item *items,
                             int32_t nitems, uint64_t *d_counts, int32_t ncounts, void *stream) {
  if (!sv) return fail(FBG_E_INVAL, "server is NULL");
  if (np <= 0 || np > sv->max_programs || !ps) return fail(FBG_E_INVAL, "np=%d out of range", np);
  if (nitems <= 0 || nitems > sv->max_items || !items) return fail(FBG_E_INVAL, "nitems=%d out of range", nitems);
  if (!d_counts || ncounts <= 0) return fail(FBG_E_INVAL, "no counts array");
  fbg_status st = check_device(sv->device);
  if (st) return st;
  const int l = sv->log2w;
  uint32_t max_regs = 0;
  int var = sv->cofactor ? 2 : 0;
  for (int32_t i = 0; i < np; i++) {
    if ((st = check_program(ps[i]))) return st;
    if ((st = check_tiling(ps[i], l))) return st;
    max_regs = std::max<uint32_t>(max_regs, (uint32_t)ps[i]->c.nregs);
    var |= ps[i]->variant(nullptr);
  }
  // validate every item on the host: the kernel trusts them
  for (int32_t k = 0; k < nitems; k++) {
    const fbg_item &it = items[k];
    if (it.prog < 0 || it.prog >= np) return fail(FBG_E_INVAL, "item %d: program %d out of range", k, it.prog);
    if (it.slot < 0 || it.slot >= ncounts) return fail(FBG_E_INVAL, "item %d: slot %d out of range", k, it.slot);
    const uint64_t nt = tiles_of(ps[it.prog]->nslices, l);
    if (it.tile_begin > it.tile_end || it.tile_end > nt)
      return fail(FBG_E_INVAL, "item %d: tiles [%llu,%llu) outside [0,%llu)", k, (unsigned long long)it.tile_begin,
                  (unsigned long long)it.tile_end, (unsigned long long)nt);
  }
  int wpb;
  size_t lds;
  if ((st = block_shape(max_regs, l, wpb, lds))) return st;
  const int cus = cu_count(sv->device);
  int occ = fbg::batch_blocks_per_cu(fbg::EVAL_COUNT, l, var & 1, 64 * wpb, lds);
  // Without the uniform cofactor where its test would spare less than half of the work (as in
  // a batch), items are long and the staging has room for a wave's each (60 DAGs 1164 us,
  // so 1025, 1088 and 956; 40 small ones 90 and 94).
  double all = 0, dead = 0;
  for (int32_t k = 0; k < nitems; k++) {
    const fbg_program *q = ps[items[k].prog];
    const double cost = (double)(items[k].tile_end - items[k].tile_begin) * tile_cost(q, l);
    all += cost, dead += cost * (1.0 - q->live[l]);
  }
  const int64_t waves = (int64_t)cus * occ * wpb;
  if (2.0 * dead < all && sv->max_items - (int64_t)nitems >= 2 * waves && all >= 2400.0 * (double)waves)
    var &= ~2;
  else if (var & 2)
    occ = fbg::batch_blocks_per_cu(fbg::EVAL_COUNT, l, var, 64 * wpb, lds);
  const bool cofactor = sv->cofactor && (var & 2);
  fbg_server::Slot &sl = sv->slots[(size_t)sv->next];
  sv->next = (sv->next + 1) % sv->nbuf;
  hipError_t e;
  if (sl.used && (e = hipEventSynchronize(sl.done)) != hipSuccess) return hip_fail(e, "hipEventSynchronize");
  const size_t items_at = kServerHeadBytes + (size_t)np * sizeof(fbg::BatchProg);
  fbg::BatchProg *hp = (fbg::BatchProg *)(sl.h + kServerHeadBytes);
  fbg::BatchItem *hi = (fbg::BatchItem *)(sl.h + items_at);
  for (int32_t i = 0; i < np; i++) hp[i] = batch_prog(ps[i], l);  // tilings checked above
  // Cut the items into pieces of about equal estimated cost so that every
  // resident wave (with the uniform cofactor every block) gets about four,
  // within the staging capacity: an item of c tiles at cost w each gives
  // ceil(c / ceil(T / w)) <= c w / T + 1 pieces for a target T (with the
  // cofactor up to twice as many), so want + nitems, or twice that, is within
  // max_items (checked below all the same).  (Sorting the pieces by cost as
  // the batch plans do cost more host time per slice than it saved.)
  auto per_tile = [&](int32_t i) {
    const fbg_program *q = ps[i];
    return cofactor ? cofactor_tile_cost(q, l) : tile_cost(q, l);
  };
  double total = 0;
  for (int32_t k = 0; k < nitems; k++)
    total += (double)(items[k].tile_end - items[k].tile_begin) * per_tile(items[k].prog);
  const int64_t spare = (cofactor ? sv->max_items / 2 : sv->max_items) - (int64_t)nitems;
  const uint64_t room = (uint64_t)std::max<int64_t>(0, spare);
  const uint64_t want = std::min<uint64_t>(room, (uint64_t)cus * occ * (cofactor ? 1 : wpb) * 4);
  const double target = want > 0 ? total / (double)want * (1.0 + 1e-9) : 0.0;
  int32_t npieces = 0;
  bool full = false;
  for (int32_t k = 0; k < nitems; k++) {
    const uint64_t b = items[k].tile_begin, e = items[k].tile_end;
    if (b == e) continue;
    const uint64_t chunk = want > 0 ? std::max<uint64_t>(1, (uint64_t)std::ceil(target / per_tile(items[k].prog))) : ~0ull;
    if (!cofactor) {
      for (uint64_t t = b; t < e; t += std::min(chunk, e - t)) {
        if (npieces >= sv->max_items) return fail(FBG_E_INVAL, "internal: more pieces than staging room");
        hi[npieces++] = {(uint32_t)items[k].prog, (uint32_t)items[k].slot, t, t + std::min(chunk, e - t), 1u, 0u};
      }
      continue;
    }
    const uint64_t K = chunk == ~0ull ? 1 : (e - b + chunk - 1) / chunk;
    cut_tiles((uint32_t)items[k].prog, (uint32_t)items[k].slot, b, e, K, true,
              chunk == ~0ull ? 0.0 : ps[items[k].prog]->live[l], [&](const fbg::BatchItem &it, double) {
                if (npieces < sv->max_items)
                  hi[npieces++] = it;
                else
                  full = true;
              });
  }
  if (full) return fail(FBG_E_INVAL, "internal: more pieces than staging room");
  if (npieces == 0) return FBG_OK;  // empty ranges only
  hipStream_t s = (hipStream_t)stream;
  e = hipMemcpyAsync(sl.d, sl.h, items_at + (size_t)npieces * sizeof(fbg::BatchItem), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail(e, "server upload");
  fbg::BatchArgs a;
  a.progs = (const fbg::BatchProg *)(sl.d + kServerHeadBytes);
  a.items = (const fbg::BatchItem *)(sl.d + items_at);
  a.nitems = (uint32_t)npieces;
  a.max_regs = lds_regs(max_regs, l);
  // (two to four items a wave, fewer than a batch's: popping ahead pays where they are
  // short.  Without it, then with it: 30 DAGs and 13 theories, 2,300 steps an item, 210 us
  // and 185, 60 DAGs, 3,600, 1022 and 1075; of clauses alone, as in a batch, 25 3-CNF systems,
  // 7,400, 296 and 225, 40 of 150 clauses of 5 literals 364 and 317, 60 of 300 of 8, 36 %
  // with several word literals, 1962 and 2134)
  uint64_t clauses = 0, multi = 0;
  for (int32_t i = 0; i < np; i++) clauses += ps[i]->ncl, multi += ps[i]->multi[l];
  a.pop_ahead = cofactor ? target / wpb < 1200.0 : (var & 1) ? target < 3000.0 : 4 * multi < clauses;
  a.head = (uint32_t *)sl.d;
  a.counts = d_counts;
  a.j16_any = j16_any();
  const uint64_t blocks = queue_blocks((uint64_t)npieces, (var & 2) ? 1 : wpb);
  const int grid = (int)std::max<uint64_t>(1, std::min<uint64_t>(blocks, (uint64_t)cus * (uint64_t)occ));
  e = fbg::launch_batch(fbg::EVAL_COUNT, l, var, a, grid, 64 * wpb, lds, s);
  if (e == hipSuccess) e = hipEventRecord(sl.done, s);
  sl.used = true;
  return e == hipSuccess ? FBG_OK : hip_fail(e, "launch of the server slice");
}

void fbg_server_free(fbg_server *sv) {
  if (!sv) return;
  for (auto &sl : sv->slots) {
    if (sl.used && sl.done) (void)hipEventSynchronize(sl.done);
    if (sl.done) (void)hipEventDestroy(sl.done);
    if (sl.h) (void)hipHostFree(sl.h);
    if (sl.d) (void)hipFree(sl.d);
  }
  delete sv;
}

// --------------------------------------------------------------- debugging

fbg_status fbg_program_emulate(const fbg_program *p, int32_t words_per_lane, uint64_t *h_dnf, uint64_t out_words,
                               uint64_t *h_count) {
  if (!p) return fail(FBG_E_INVAL, "program is NULL");
  if (p->c.n > 30) return fail(FBG_E_RANGE, "emulation is limited to n <= 30");
  int l;
  fbg_status st = parse_wpl(words_per_lane, l);
  if (st) return st;
  if ((st = check_tiling(p, l))) return st;
  const uint64_t need = dnf_words_of(p->c.n);
  if (h_dnf && out_words < need) return fail(FBG_E_INVAL, "out_words too small");
  std::vector<uint32_t> s32((size_t)std::max<uint64_t>(2, p->nslices), 0u);
  fbg::emulate_program(p->words[l], p->nins[l], p->c.nregs, p->c.n, l, p->cofactor, s32.data());
  if (h_dnf) memcpy(h_dnf, s32.data(), need * 8);
  if (h_count) {
    uint64_t c = 0;
    for (uint64_t i = 0; i < p->nslices; i++) c += (uint64_t)__builtin_popcount(s32[i]);
    *h_count = c;
  }
  return FBG_OK;
}

int64_t fbg_program_disasm(const fbg_program *p, int32_t words_per_lane, char *buf, int64_t cap) {
  if (!p) return -1;
  int l = p->auto_log2w;
  if (words_per_lane > 0 && parse_wpl(words_per_lane, l)) return -1;
  if (check_tiling(p, l)) return -1;
  std::string s = fbg::disasm_program(p->words[l], p->nins[l], l);
  if (buf && cap > 0) {
    size_t k = std::min<size_t>((size_t)cap - 1, s.size());
    memcpy(buf, s.data(), k);
    buf[k] = 0;
  }
  return (int64_t)s.size();
}

}  // extern "C"
