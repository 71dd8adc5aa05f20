// Internal: how the kernels for few output blocks share out the pruned columns they clear (plain arithmetic, also built
// without HIP).  A column of C is M elements; with every weight of a layer pruned M is any int, and 4 M is not.
#pragma once
#include <stdint.h>

namespace twg {

// 16-byte chunks of a column of `bytes` bytes (at most 2^33).
constexpr int zero_chunks(int64_t bytes) { return (int)((bytes + 15) / 16); }

// Chunk number i of consecutive columns: column number, byte offset inside it.
struct ZeroChunk {
  int column;
  int64_t at;
};
constexpr ZeroChunk zero_chunk(int i, int chunks) { return {i / chunks, (int64_t)(i % chunks) * 16}; }

}  // namespace twg
