// Size rules of the launches as plain host functions, so that a host build can
// check them.
#pragma once

#include <cstdint>

namespace adapm {

// The last-level cache, shared by the whole device.
constexpr int64_t LLC_BYTES = int64_t(256) << 20;

// Whether a pull of n rows of dim floats writes its output past the caches.
// Only where the output exceeds the last-level cache and so cannot be there
// when the caller reads it.  A smaller one can, and streaming it moves more
// time into the reader than it saves in the pull.  Measured, cached and
// streamed, the pull and a sum over its output: 54 MB in rows of 64 floats 38.8
// and 44.8 us (the pull alone 20.1 and 20.7), 128 MB 67.6 and 84.3, 80 MB in
// rows of 512 48.0 and 56.4; above the line 300 MB 177.6 and 177.1 (alone 99.0
// and 90.6), 500 MB 291.6 and 284.9 (alone 160 and 147).
inline bool pull_streams(int64_t n, int64_t dim) { return n * dim * 4 > LLC_BYTES; }

}  // namespace adapm
