// misc.hip -- launches of the small kernels (stored-DNF scans, the lists
// of the tiles that hold models, fills) and the per-mode dispatch of the
// single-program evaluator (its kernels live in eval_*.hip).
#define FBG_DEVICE_MISC_KERNELS
#include "fbg_device.h"

#include <algorithm>

namespace fbg {

hipError_t launch_eval_count(int log2w, int var, const EvalArgs &a, int grid, int block, size_t lds, hipStream_t s);
hipError_t launch_eval_dnf(int log2w, int var, const EvalArgs &a, int grid, int block, size_t lds, hipStream_t s);
hipError_t launch_eval_enum(int mode, int log2w, int var, const EvalArgs &a, int grid, int block, size_t lds,
                            hipStream_t s);
int eval_occ_count(int log2w, int var, int block, size_t lds);
int eval_occ_dnf(int log2w, int var, int block, size_t lds);
int eval_occ_enum(int mode, int log2w, int var, int block, size_t lds);

hipError_t launch_eval(int mode, int log2w, int var, const EvalArgs &a, int grid, int block, size_t lds,
                       hipStream_t s) {
  switch (mode) {
    case dev::MODE_COUNT: return launch_eval_count(log2w, var, a, grid, block, lds, s);
    case dev::MODE_DNF: return launch_eval_dnf(log2w, var, a, grid, block, lds, s);
    case dev::MODE_TILECNT:
    case dev::MODE_ENUM: return launch_eval_enum(mode, log2w, var, a, grid, block, lds, s);
  }
  return hipErrorInvalidValue;
}

int eval_blocks_per_cu(int mode, int log2w, int var, int block, size_t lds) {
  switch (mode) {
    case dev::MODE_COUNT: return eval_occ_count(log2w, var, block, lds);
    case dev::MODE_DNF: return eval_occ_dnf(log2w, var, block, lds);
    default: return eval_occ_enum(mode, log2w, var, block, lds);
  }
}

hipError_t launch_dnf_scan(int mode, int log2w, const EvalArgs &a, int grid, int block, hipStream_t s) {
  if (mode == dev::MODE_TILECNT && log2w == 2)
    hipLaunchKernelGGL((dev::k_dnf_scan<2, dev::MODE_TILECNT>), dim3(grid), dim3(block), 0, s, a);
  else if (mode == dev::MODE_TILECNT && log2w == 5)
    hipLaunchKernelGGL((dev::k_dnf_scan<5, dev::MODE_TILECNT>), dim3(grid), dim3(block), 0, s, a);
  else if (mode == dev::MODE_ENUM && log2w == 2)
    hipLaunchKernelGGL((dev::k_dnf_scan<2, dev::MODE_ENUM>), dim3(grid), dim3(block), 0, s, a);
  else if (mode == dev::MODE_ENUM && log2w == 5)
    hipLaunchKernelGGL((dev::k_dnf_scan<5, dev::MODE_ENUM>), dim3(grid), dim3(block), 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_cofactor_masks(const uint32_t *code, uint64_t ngroups, uint64_t *masks, uint32_t *counts, int grid,
                                 hipStream_t s) {
  hipLaunchKernelGGL(dev::k_cofactor_masks, dim3(grid), dim3(256), 0, s, code, ngroups, masks, counts);
  return hipGetLastError();
}

uint64_t tile_list_blocks(uint64_t n) { return (n + kListBlock - 1) / kListBlock; }

hipError_t launch_tile_list(const TileListArgs &a, hipStream_t s) {
  const uint64_t nb = tile_list_blocks(a.n);
  hipLaunchKernelGGL(dev::k_tile_sums, dim3((unsigned)nb), dim3(dev::LIST_THREADS), 0, s, a);
  if (nb <= 1024) {
    // every block adds up the (at most 16 KiB of) sums before it
    hipLaunchKernelGGL((dev::k_tile_list<false>), dim3((unsigned)nb), dim3(dev::LIST_THREADS), 0, s, a);
  } else {
    hipLaunchKernelGGL(dev::k_tile_sums_scan, dim3(1), dim3(dev::LIST_THREADS), 0, s, a, nb);
    hipLaunchKernelGGL((dev::k_tile_list<true>), dim3((unsigned)nb), dim3(dev::LIST_THREADS), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_zero(uint64_t *p, uint64_t n, uint32_t *head, uint32_t nhead, hipStream_t s) {
  if (!head) nhead = 0;
  // (a launch has fewer than 2^32 threads)
  constexpr uint64_t kMost = 1ull << 30;
  do {
    const uint64_t k = n < kMost ? n : kMost, m = std::max<uint64_t>(std::max<uint64_t>(k, nhead), 1);
    hipLaunchKernelGGL(dev::k_zero_u64, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, p, k, head, nhead);
    p += k;
    n -= k;
    nhead = 0;
  } while (n > 0);
  return hipGetLastError();
}

hipError_t launch_set_u64(uint64_t *p, uint64_t v, hipStream_t s) {
  hipLaunchKernelGGL(dev::k_set_u64, dim3(1), dim3(64), 0, s, p, v);
  return hipGetLastError();
}

}  // namespace fbg
