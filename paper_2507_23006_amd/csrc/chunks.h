// Chunks of consecutive items, in 32-bit indices up to the last one.
#pragma once

#include <stdint.h>

namespace gs {

// the first chunk that starts at or after item i (i + chunk - 1 could pass 2^32)
constexpr uint32_t first_chunk(uint32_t i, uint32_t chunk) { return i / chunk + (i % chunk != 0u ? 1u : 0u); }

}  // namespace gs
