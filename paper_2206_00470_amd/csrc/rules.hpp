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
// Two kinds of rows write lines in parts, which costs more when they are
// streamed.  Rows stored one float per lane (`floats_per_store` 1: no multiple
// of four, or an unaligned output) and wider than a wavefront never are: 1.2 GB
// in rows of 130 floats 564 us cached and 664 streamed, of 301 498 and 594.
// Rows of 257 to 512 floats that share 64-byte pieces are up to 1 GiB, as it
// costs more the larger the output is: rows of 300 floats 0.6 GB 223 and 209
// us, 4.8 GB 1,731 and 1,906; of 500 0.6 GB 210 and 191, 4.8 GB 1,673 and 1,729;
// but of 400 4.8 GB 1,585 and 1,464, of 512 1,540 and 1,429, and narrower or
// wider rows at every size (100 floats 1.2 GB 455 and 419, 1,000 4.8 GB 2,040
// and 1,856).
inline bool pull_streams(int64_t n, int64_t dim, int floats_per_store) {
  const int64_t bytes = n * dim * 4;
  if (bytes <= LLC_BYTES) return false;
  if (floats_per_store == 1 && dim > 64) return false;
  return dim <= 256 || dim > 512 || dim % 16 == 0 || bytes <= (int64_t(1) << 30);
}

// Rows of a pull that one row group keeps in flight: four where a lane holds at
// most four floats of a row and there are more workgroups than run at once
// (eight on each of 256 compute units), else one.  Below that line four rows
// per group only leave units empty.  Measured on the device (graph replays) in
// rows of 64 floats, with one and with four: 8,000 rows (500 workgroups of one
// row per group) 3.7 and 4.6 us, 32,000 (2,000) 5.6 and 6.2, 33,600 (2,100) 6.7
// and 6.5, 96,000 (6,000) 14.5 and 12.4; the line is at the same number of
// workgroups for rows of 4 to 256 floats.
constexpr int64_t PULL_BLOCKS_AT_ONCE = 2048;

inline int pull_rows(int64_t n, int groups_per_block, int floats_per_lane) {
  const int64_t blocks = (n + groups_per_block - 1) / groups_per_block;
  return floats_per_lane <= 4 && blocks > PULL_BLOCKS_AT_ONCE ? 4 : 1;
}

// The most keys whose work ps_push_prepare does in tiles (sort.hpp, "middling
// inputs", which end at MID_KEYS_MAX in any case).  A prepare runs beside another
// push's merge, and the tiles' workgroups of 1,024 threads wait until a compute
// unit has that many free, which a merge with more workgroups than run at once
// leaves late; the kernels of 256 threads slip in.  So tiles are taken beside
// short merges: 10M floats where row groups are at most 32 lanes, 28,000 keys
// where a row of up to 256 floats takes a whole wavefront.  Wider rows' merges
// are so long that neither shows.  Measured as graph replays of pipelined pushes
// with kernels of 256 threads and with tiles: rows of 64 floats, 120,000 keys
// 87 and 81 us, 200,000 96 and 98, 300,000 110 and 118; of 128, 64,000 keys 105
// and 101, 200,000 119 and 130; of 200, 24,000 keys 80 and 74, 64,000 100 and
// 110, 200,000 162 and 180; of 384, 60,000 keys 149 and 139.  (The prepares of
// the steps run beside more than a merge and gain from tiles at every size:
// factorization at rank 64 of 108,000 keys 111 and 103, 380,000 174 and 170; CTR
// of 212,992 keys 105.0 and 104.5, 312,000 134 and 128.)
inline int64_t push_prepare_tiled_keys(int64_t dim, int row_lanes) {
  if (row_lanes < 64) return 10'000'000 / dim;
  return dim <= 256 ? 28'000 : INT64_MAX;
}

// The most keys whose work a ComplEx step does in tiles beside its own gradient
// kernel, whose waves hold half of a compute unit's registers and more: where they
// are on every unit, workgroups of 1,024 threads wait for the kernel's end.
// Measured, kernels of 256 threads and tiles: 300 x 150 in rows of 64 floats 125
// and 108 us, 1,300 x 150 153 and 149, 2,000 x 150 177 and 192, 12,000 x 20 196
// and 201, 28,000 x 4 (196,000 keys) 164 without and 173 with; rows of 256 floats
// 1,000 x 150 227 and 224, 2,400 x 150 388 and 389; of
// 512 floats 300 x 150 251 and 250, 1,000 x 150 376 and 424.  (Skip-gram's and
// CTR's gradient kernels leave room: skip-gram of 377,400 keys 175 and 166, CTR of
// 390,000 184 and 182.)
inline int64_t kge_tiled_keys(int64_t dim, int64_t triples) { return dim <= 256 && triples <= 2000 ? 200'000 : 100'000; }

// Whether a merge streams its table and gradient rows past the caches
// (non-temporal).  First, where the rows it can touch (value and accumulator rows
// of at most `keys` keys, the smaller of occurrences and table rows) exceed the
// last-level cache.  That is a bound the host knows; the distinct keys may be far
// fewer, and rows that fit the cache are then streamed too.  Measured over streams
// of new batches, cached and streamed.  Above the line: pushes of 2M keys in rows
// of 100 floats 0.837 and 0.759 ms, factorization of 1M entries at rank 100
// 1.047 and 0.954, ComplEx of 422K occurrences of 256 floats 0.565 and 0.528,
// skip-gram of 5,000 centres x 20 negatives over 1M words of 100 floats 0.397
// and 0.381; with many duplicates CTR of 32,768 samples 0.318 and 0.313, 2M
// keys over 300,000 rows of 128 floats 0.492 and 0.451, but skip-gram of 5,000
// centres over 100,000 words of 300 floats, which come back batch after batch,
// 0.261 and 0.273.  Below it: CTR of 8,192 samples 0.141 and 0.148, row-wise
// factorization of 100,003 entries at rank 50 0.148 and 0.160, skip-gram of
// 5,003 centres over 100,000 words of 100 floats 0.161 and 0.167, but
// factorization of 150,000 entries at rank 100 0.224 and 0.214.
// Second, where rows do not leave too many cache lines in parts: streamed, two
// keys' parts of one line go out separately.  Pushes of 4M keys, cached and
// streamed (us): two tables of 64 floats 949 and 918, of 100 1,775 and 1,699, of
// 200 3,022 and 2,741, but of 36 947 and 986, 50 1,157 and 1,290, 65 1,369 and
// 1,558, 130 2,195 and 2,291; the two rows of a key side by side (`together`) of
// 28 floats 751 and 728, 60 1,169 and 1,066, but of 20 643 and 655, 50 1,055 and
// 1,078, 65 1,262 and 1,386; row-wise of 20 585 and 602, 50 953 and 977, 64 880
// and 836, 130 1,538 and 1,551, 200 2,078 and 1,845, 250 2,559 and 2,288; bf16 of
// 28 719 and 771, 60 1,053 and 1,079, 64 899 and 861, 101 1,567 and 1,635, 200
// 2,502 and 2,299.  Rows of no multiple of four floats are stored one float per
// lane.
inline bool merge_streams(int64_t keys, int64_t dim, bool rowwise, bool bf16, bool together) {
  const int64_t value_bytes = (bf16 ? 2 : 4) * dim;
  const int64_t accum_bytes = rowwise ? 4 : 4 * dim;
  if (keys * (value_bytes + accum_bytes) <= LLC_BYTES) return false;
  if (dim % 4 != 0) return rowwise && dim > 128;
  if (dim >= 100) return true;
  if (rowwise) return dim >= 64;
  return value_bytes % 64 == 0 || (together && !bf16 && dim >= 28);
}

}  // namespace adapm
