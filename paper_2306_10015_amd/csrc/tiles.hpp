// tiles.hpp — the tile decomposition of fp32 and bf16 tensors shared by the
// engine and the checksum: a tile is kThreads 16-byte groups (4 KiB), which a
// workgroup takes with one group per lane, or fewer lanes with more groups each
// (engine_dense.hip).
#pragma once

#include <stdint.h>

#include "records.hpp"

namespace mezo {

template <uint32_t kDtype>
struct Layout;
template <>
struct Layout<kF32> {
    static constexpr uint64_t kPerGroup = 4;  // elements per 16-byte group
};
template <>
struct Layout<kBF16> {
    static constexpr uint64_t kPerGroup = 8;
};

}  // namespace mezo
