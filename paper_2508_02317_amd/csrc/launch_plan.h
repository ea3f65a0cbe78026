// Which workgroup does what: integer arithmetic that launches and kernels share, without anything of a GPU in it, so that a plain
// C++ program can enumerate it (tests/test_launch_plan.py).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace moe {

// A launch has at most 2^32 - 1 threads.
constexpr bool fits_one_launch(size_t blocks, int threads) { return blocks <= 0xFFFFFFFFu / static_cast<unsigned>(threads); }

}  // namespace moe
