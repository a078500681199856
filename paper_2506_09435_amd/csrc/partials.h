// partials.h - capacity of a context's buffer of per-block partial sums (host logic only).
//
// Every reduction in the library is deterministic: each block of a launch writes its sums to
// partial[block * sums + k], and they are added in a fixed order by a one-block kernel or by every
// block of the kernel that needs the sum (reduce.h).  One buffer per
// context serves all such launches, so it must hold the largest blocks x sums of any of them.
// partial_uses lists every kind of launch that writes partials, partial_capacity is the size
// that holds them all, and partials_fit is the check made before each launch.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace fnpf {

constexpr int kPartialVecBlocks = 1024;   // grid of the grid-stride vector kernels (FP64 data)

struct PartialUse {
  const char *what;
  int64_t blocks;
  int sums;
};

// colour_blocks: blocks of the colour-scheduled apply summed over its colours (one partial each);
// owner_blocks: blocks of the owner-computes apply's first pass, which has one partial each.
inline std::vector<PartialUse> partial_uses(int64_t colour_blocks, int64_t owner_blocks) {
  const int64_t v64 = kPartialVecBlocks, v32 = 2 * kPartialVecBlocks;
  return {
      {"norm of b (k_bnorm)", v64, 1},
      {"PCG initial residual (k_pcg_init)", v64, 2},
      {"mixed outer residual (k_resid_to32)", v64, 3},
      {"p-multigrid update and dots, FP64 grid", v64, 2},
      {"p-multigrid update and dots, FP32 grid", v32, 2},
      {"Lanczos and power-iteration dots, FP32 grid", v32, 2},
      {"line-smoother B-norm (k_line_bnorm), FP32 grid", v32, 1},
      // the update after an apply puts its own partials behind the apply's
      {"apply with dot product, colour schedule, and CG update", colour_blocks + 2 * v32, 1},
      {"apply with dot product, owner-computes, and CG update", owner_blocks + 2 * v32, 1},
  };
}

inline int64_t partial_capacity(const std::vector<PartialUse> &uses) {
  int64_t cap = 0;
  for (const auto &u : uses) cap = u.blocks * u.sums > cap ? u.blocks * u.sums : cap;
  return cap;
}

inline bool partials_fit(int64_t capacity, int64_t blocks, int sums) {
  return blocks >= 0 && sums > 0 && blocks * sums <= capacity;
}

// "" when every use fits the capacity, else the first use that does not
inline std::string partial_layout_error(const std::vector<PartialUse> &uses, int64_t capacity) {
  for (const auto &u : uses)
    if (!partials_fit(capacity, u.blocks, u.sums))
      return std::string("partial-sum buffer too small for ") + u.what;
  return "";
}

}  // namespace fnpf
