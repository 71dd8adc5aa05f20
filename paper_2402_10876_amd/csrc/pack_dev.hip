// Device-side packer: (B, mask[, tile mask]) in device memory -> packed handle, without moving
// the weight through the host.
//
// Paper: Section V condenses every B tile ahead of inference and replaces the tile masks by the
// indices of the unpruned rows / columns; Algorithm 3 condenses the kept columns before cutting
// tiles of G.  Here the same canonical form as the host packer's is produced by kernels:
//   structure  one kernel finds the columns that keep anything, one the rows that keep anything in each tile of
//              G kept columns, as bit sets; positions in the ascending index lists are counted from the bits
//              wherever they are needed, so that no kernel exists only to number something;
//   plan       only counts (8 bytes for every tile and 64 rows) visit the host, where padding,
//              offsets and the launch order of the tiles are laid out exactly as for a host-packed
//              weight and the image is allocated;
//   image      one kernel writes the padded lists and the values in the register order of the
//              matrix instruction (TVW: with the 2:4 positions and the fill rule for short groups).
// The image is the only copy; the lists and values of the logical form are read back from it if
// somebody asks for them (tw_export, tw_unpack, tw_concat; tw_conv_bind: the lists).
//
// What bounds it: a chain of three launches and two waits.  The counts are written straight into pinned host
// memory, each word with the call's tag beside the number, and the host looks for the tags: 5 us after the kernel where a
// copy and a wait took 13.  Prune, pack and a first product, from Python:
// 1024 x 4096 (TVW) 139 -> 84 us, 1003 x 2491 184 -> 96, 64 x 64 118 -> 60 (before: eight launches, a copy and a wait for
// each of two visits).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "launch.h"
#include "grid.h"
#include "mk_band.h"
#include "packed.h"

namespace twg {

namespace {

constexpr int T = 256;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct __attribute__((packed, aligned(1))) Piece { u32x4 v; };       // (global loads need no alignment)

// 16 mask bytes of row k from column n0 < N on, as 0x01 where non-zero (columns past N: 0).
__device__ __forceinline__ u32x4 load_mask16(const uint8_t* S, int k, int n0, int K, int N) {
  u32x4 v = {0u, 0u, 0u, 0u};
  const uint8_t* p = S + (size_t)k * N + n0;
  const int cnt = N - n0;
  if (cnt >= 16 || k < K - 1 - 16 / N) {                             // (the last rows' ends may be the end of the buffer)
    v = ((const Piece*)p)->v;
    if (cnt < 16)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] &= (uint32_t)((1ull << (8 * min(max(cnt - 4 * j, 0), 4))) - 1ull);
  } else
    for (int c = 0; c < cnt; ++c) v[c >> 2] |= (uint32_t)p[c] << (8 * (c & 3));
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (((v[j] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v[j]) >> 7 & 0x01010101u;
  return v;
}

__device__ __forceinline__ bool any_byte(const u32x4& v) { return (v[0] | v[1] | v[2] | v[3]) != 0; }

// Bit n of slice blockIdx.y of `bits` = column n of the K x N byte mask S has a non-zero entry among the slice's rows (bits
// past N: 0).  A workgroup of 1024 threads takes 128 columns: 8 lanes of 16 columns, 128 rows at a time.  Narrow weights are cut
// into slices of `rows` rows, which the readers put together: 25088 x 64 on one CU took 42 us, in 16
// slices 4.9 (two slices of 1024 x 4096 save nothing and cost the readers a microsecond).
__global__ __launch_bounds__(1024) void column_bits(const uint8_t* S, int K, int N, int rows, uint16_t* bits) {
  __shared__ u32x4 part[16][8];
  const int tid = threadIdx.x, c = tid & 7;
  const int n0 = blockIdx.x * 128 + c * 16, k_end = min(K, ((int)blockIdx.y + 1) * rows);
  u32x4 a = {0u, 0u, 0u, 0u};
  if (n0 < N)
    for (int k0 = blockIdx.y * rows + (tid >> 3); k0 < k_end; k0 += 4 * 128) {
      u32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = load_mask16(S, min(k0 + i * 128, k_end - 1), n0, K, N);
      a |= (v[0] | v[1]) | (v[2] | v[3]);
    }
#pragma unroll
  for (int d = 8; d < 64; d <<= 1)
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] |= __shfl_xor(a[j], d);
  if ((tid & 63) < 8) part[tid >> 6][c] = a;
  __syncthreads();
  if (tid >= 8) return;
#pragma unroll
  for (int w = 0; w < 16; ++w) a |= part[w][c];
  uint32_t b = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) b |= (a[j] * 0x01020408u) >> 24 << (4 * j);          // bytes 0 / 1 -> four bits
  bits[(blockIdx.y * gridDim.x + blockIdx.x) * 8 + c] = (uint16_t)b;
}

// Position of set bit number n (from 0) of x.
__device__ __forceinline__ int nth_bit(unsigned long long x, int n) {
  int at = 0;
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) {
    const int low = __popcll((x >> at) & ((1ull << w) - 1ull));
    if (n >= low) { n -= low; at += w; }
  }
  return at;
}

// Sum of the threads' numbers in front of this one, over a workgroup of whole waves; *total: over all of them.
// `part`: an int per wave; the caller puts a barrier between two uses of the same array.
__device__ __forceinline__ int sum_before(int mine, int* part, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  int in = mine;
#pragma unroll
  for (int k = 1; k < 64; k <<= 1) { const int t = __shfl_up(in, k); in += lane >= k ? t : 0; }
  if (lane == 63) part[wave] = in;
  __syncthreads();
  int front = in - mine, all = 0;
  for (int w = 0; w < waves; ++w) {
    const int n = part[w];
    front += w < wave ? n : 0;
    all += n;
  }
  *total = all;
  return front;
}

// A word for the host: the number and, above it, the call's tag.
__device__ __forceinline__ void tell(unsigned long long* at, uint32_t tag, uint32_t number) {
  __hip_atomic_store(at, (unsigned long long)tag << 32 | number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// An infinity or NaN among the 16 weights of row k from column n0 on whose mask bytes are set (columns past N:
// not set).
__device__ __forceinline__ bool any_nonfinite(const uint16_t* B, int ldb, int k, int n0, int N, const u32x4& mask) {
  union { u32x4 v[2]; uint16_t e[16]; } x;
  const uint16_t* p = B + (size_t)k * ldb + n0;
  if (n0 + 16 <= N) { x.v[0] = ((const Piece*)p)->v; x.v[1] = ((const Piece*)(p + 8))->v; }
  else {
#pragma unroll
    for (int c = 0; c < 16; ++c) x.e[c] = p[min(c, N - 1 - n0)];
  }
  bool r = false;
#pragma unroll
  for (int c = 0; c < 16; ++c) r |= (x.e[c] & 0x7c00) == 0x7c00 && (mask[c >> 2] >> (8 * (c & 3)) & 1u);
  return r;
}

// What a workgroup of tile_rows tells the host about its tile and 64 rows.
enum { ROWS_KEPT_SHIFT = 16, OUTSIDE_BIT = 1 << 24, NONFINITE_BIT = 1 << 25 };    // (low half: entries, at most 64 * 128)

struct RowArgs {
  const uint8_t *S, *element;          // structure mask; element mask to compare with it (or null)
  const uint16_t* B;                   // weights to look at for infinities (or null)
  int ldb, K, N, lg, blocks;           // blocks of 64 rows
  const unsigned long long* col_bits;  // `slices` times `stride` words
  int slices, stride;
  int32_t *kept, *dropped;             // the two column lists
  unsigned long long* row_bits;        // [tile][block]: rows that have an entry among the tile's columns
  unsigned long long* host;            // [0]: kept columns, [1 + tile * blocks + block]: the above
  uint32_t tag, n_wgs;
};

// Word w of the column bits.
__device__ __forceinline__ unsigned long long col_word(const RowArgs& a, int w) {
  unsigned long long x = 0;
#pragma unroll 4
  for (int s = 0; s < a.slices; ++s) x |= a.col_bits[s * a.stride + w];
  return x;
}

// Workgroup (tile, block of 64 rows).  The tile's columns reach from its first kept one (tile 0: from column 0) to
// the next tile's (the last tile: to column N); which they are follows from the column bits.  16 lanes of 16 columns
// x 16 rows at a time.  The workgroups of the first block also write the column lists.
__global__ __launch_bounds__(T) void tile_rows(RowArgs a) {
  __shared__ int part[2][T / 64];
  __shared__ int range[2], entries[T / 64];
  __shared__ unsigned long long word_part[T / 64];
  __shared__ int flags[T / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t wg = blockIdx.y * gridDim.x + blockIdx.x;
  if (wg >= a.n_wgs) return;
  const int t = (int)(wg / (uint32_t)a.blocks), kb = (int)(wg - (uint32_t)t * (uint32_t)a.blocks);
  const int G = 1 << a.lg, words = (a.N + 63) / 64;
  // ---- columns ----
  const int per = (words + T - 1) / T, w0 = min(tid * per, words), w1 = min(w0 + per, words);
  int mine = 0, n_kept;
  for (int w = w0; w < w1; ++w) mine += __popcll(col_word(a, w));
  const int front = sum_before(mine, part[0], &n_kept);
#pragma unroll
  for (int e = 0; e < 2; ++e) {          // column of kept column number (t + e) G
    int n = ((t + e) << a.lg) - front;
    if (n < 0 || n >= mine) continue;
    for (int w = w0; w < w1; ++w) {
      const unsigned long long x = col_word(a, w);
      const int c = __popcll(x);
      if (n < c) { range[e] = w * 64 + nth_bit(x, n); break; }
      n -= c;
    }
  }
  __syncthreads();
  const int n_tiles = (n_kept + G - 1) >> a.lg;
  if (wg == 0 && tid == 0) tell(a.host, a.tag, (uint32_t)n_kept);
  const bool live = t < max(n_tiles, 1); // (nothing kept at all: tile 0 still lists the dropped columns and looks at `element`)
  const int lo = t == 0 ? 0 : range[0], hi = (t + 1) << a.lg < n_kept ? range[1] : a.N;
  if (kb == 0 && live) {
    int base = t << a.lg;
    for (int n0 = lo; n0 < hi; n0 += T) {
      const int n = n0 + tid;
      const bool v = n < hi && (col_word(a, n >> 6) >> (n & 63) & 1ull);
      int all;
      const int p = base + sum_before(v, part[1], &all);
      if (v) a.kept[p] = n;
      else if (n < hi) a.dropped[n - p] = n;
      base += all;
      __syncthreads();
    }
  }
  if (!live) {
    if (tid == 0) tell(a.host + 1 + wg, a.tag, 0u);
    return;
  }
  // ---- rows ----
  const int k0 = kb * 64 + (tid >> 4);
  bool any[4] = {false, false, false, false};
  bool outside = false, nonfinite = false;
  int count = 0;
  for (int n0 = (lo & ~15) + 16 * (tid & 15); n0 < hi; n0 += 256) {
    u32x4 in;                            // bytes of the tile's columns
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int x = min(max(lo - n0 - 4 * d, 0), 4), y = min(max(hi - n0 - 4 * d, 0), 4);
      in[d] = (uint32_t)((1ull << (8 * y)) - 1ull) & ~(uint32_t)((1ull << (8 * x)) - 1ull);
    }
    u32x4 v[4], e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = min(k0 + 16 * i, a.K - 1);
      v[i] = load_mask16(a.S, k, n0, a.K, a.N);
      if (a.element) e[i] = load_mask16(a.element, k, n0, a.K, a.N);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = k0 + 16 * i;
      if (k >= a.K) break;
      v[i] &= in;
      any[i] |= any_byte(v[i]);
      count += __popc(v[i][0]) + __popc(v[i][1]) + __popc(v[i][2]) + __popc(v[i][3]);
      if (a.element) outside |= any_byte(e[i] & ~v[i] & in);
      if (a.B) nonfinite |= any_nonfinite(a.B, a.ldb, k, n0, a.N, v[i]);
    }
  }
  unsigned long long word = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {          // row 16 i + 4 wave + j of the block: 16 lanes
    const unsigned long long b = __ballot(any[i]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (b >> (16 * j) & 0xffffull) word |= 1ull << (16 * i + 4 * wave + j);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) count += __shfl_xor(count, d);
  const int flag = (__any(outside) ? OUTSIDE_BIT : 0) | (__any(nonfinite) ? NONFINITE_BIT : 0);
  if (lane == 0) { word_part[wave] = word; entries[wave] = count; flags[wave] = flag; }
  __syncthreads();
  if (tid == 0) {
    word = (word_part[0] | word_part[1]) | (word_part[2] | word_part[3]);
    a.row_bits[wg] = word;
    tell(a.host + 1 + wg, a.tag,
         (uint32_t)((entries[0] + entries[1]) + (entries[2] + entries[3])) | (uint32_t)__popcll(word) << ROWS_KEPT_SHIFT |
             (uint32_t)(flags[0] | flags[1] | flags[2] | flags[3]));
  }
}

struct ImageArgs {
  const uint16_t* B;
  const uint8_t* mask;                 // TVW
  const int32_t *kept, *dropped;       // kept columns, the others
  const unsigned long long* row_bits;
  const int32_t* tables;               // host: tile_kp_off, tile_order, tile_sched, as they lie in the image
  int ldb, K, N, G, blocks, n_kept, n_zero, n_tiles, uniform_kp, stages, n_table;
  int32_t* out_tables;
  int32_t *row_idx, *col_idx, *zero_cols;
  uint16_t* vals;
  uint16_t* meta;                      // TVW
  uint8_t* valid;
  uint32_t* result;                    // host: [0]: rows that some tile keeps, [1] (zero on entry): a 2:4 group keeps more than two
};

// TVW values and position words (layout: see the host packer's build_device_values): one thread per
// (half, column block, lane) of a stage of 64 rows, i.e. four groups of 4 condensed rows of a column.
// A group stores the two lowest positions that are kept, topped up with the lowest that are not (+0
// fillers); `valid`: 2 bits per group, which of the two are kept elements.  rows: the stage's kept rows, of
// which there are `left`.  Returns whether a group keeps more than two.
__device__ __forceinline__ bool image_tvw(const ImageArgs& a, int t, size_t kp0, int stage, const int32_t* rows, int left) {
  const int i = threadIdx.x, nbt = a.G / 32;
  const int l = i & 63, nb = (i >> 6) % nbt, su = (i >> 6) / nbt;
  const int c = 32 * nb + l % 32;
  const bool live = t * a.G + c < a.n_kept;
  const int n = a.kept[live ? t * a.G + c : 0];
  union { uint16_t e[8]; u32x4 v; } x;
  x.v = u32x4{0u, 0u, 0u, 0u};
  uint32_t word = 0, vbits = 0;
  bool three = false;
  const int j0 = 32 * su + 16 * (l / 32);              // the thread's 16 condensed rows
  uint16_t val[16];
  uint8_t kept[16];
#pragma unroll
  for (int p = 0; p < 16; ++p) {                       // all loads first
    const int row = rows[j0 + p];
    val[p] = a.B[(size_t)row * a.ldb + n];
    kept[p] = a.mask[(size_t)row * a.N + n];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int g0 = j0 + 4 * j;                         // first row of the group
    uint32_t pos = 0x4;                                // positions (0, 1)
    if (live && g0 < left) {
      const uint16_t* v = val + 4 * j;
      int set = 0;
#pragma unroll
      for (int p = 0; p < 4; ++p) set |= g0 + p < left && kept[4 * j + p] != 0 ? 1 << p : 0;
      three |= __popc(set) > 2;
      int chosen = set;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (__popc(chosen) < 2) chosen |= 1 << p;
      const int p0 = __ffs(chosen) - 1, p1 = __ffs(chosen & (chosen - 1)) - 1;
      pos = (uint32_t)(p0 | p1 << 2);
      uint16_t lo = 0, hi = 0;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        if (p == p0 && (set >> p & 1)) lo = v[p];
        if (p == p1 && (set >> p & 1)) hi = v[p];
      }
      x.e[2 * j] = lo;
      x.e[2 * j + 1] = hi;
      vbits |= (uint32_t)((set >> p0 & 1) | (set >> p1 & 1) << 1) << (2 * j);
    }
    word |= pos << (4 * j);
  }
  ((u32x4*)(a.vals + kp0 / 2 * a.G))[(size_t)stage * 4 * a.G + i] = x.v;
  // position words: [stage][block][lane], 16 bits per half
  const size_t w = (kp0 / 64 + stage) * nbt * 64 + nb * 64 + l;
  a.meta[2 * w + su] = (uint16_t)word;
  a.valid[2 * w + su] = (uint8_t)vbits;
  return three;
}

// TW values (layout: see the host packer's build_device_values): 8 rows of a column per thread of a stage of 32
// rows, one 16-byte store.
__device__ __forceinline__ void image_tw(const ImageArgs& a, int t, size_t kp0, int stage, const int32_t* rows, int left) {
  const int i = threadIdx.x, j0 = i / a.G * 8, c = i % a.G;
  union { uint16_t e[8]; u32x4 v; } x;
  x.v = u32x4{0u, 0u, 0u, 0u};
  if (t * a.G + c < a.n_kept && j0 < left) {
    const int n = a.kept[t * a.G + c];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint16_t v = a.B[(size_t)rows[j0 + j] * a.ldb + n];
      x.e[j] = j0 + j < left ? v : (uint16_t)0;
    }
  }
  ((u32x4*)(a.vals + (kp0 + (size_t)stage * KSTEP_TW) * a.G))[j0 / 16 * (2 * a.G) + (c / 32) * 64 + ((j0 % 16) / 8) * 32 + c % 32] = x.v;
}

// The image, 4 G threads per workgroup.  One workgroup per tile and stage (a step of the padding): which kept rows it
// holds is counted from the tile's row bits; it writes its part of the padded row list (pads repeat the last kept row)
// and its values, the first stage the tile's columns (-1 past the last).  The last workgroup writes the rest.
template <bool TVW>
__global__ __launch_bounds__(512) void build_image(ImageArgs a) {
  constexpr int STEP = TVW ? KSTEP_TVW : KSTEP_TW;
  __shared__ int32_t rows[64];
  __shared__ int part[8];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, T4 = 4 * a.G;
  const uint32_t wg = blockIdx.y * gridDim.x + blockIdx.x;
  const int t = (int)(wg / (uint32_t)a.stages), stage = (int)(wg - (uint32_t)t * (uint32_t)a.stages);
  if (t > a.n_tiles || (t == a.n_tiles && stage > 0)) return;
  const unsigned long long* bits = a.row_bits;
  if (t == a.n_tiles) {                  // slack behind the lists and values, pruned columns, the host's tables
    const int kp_end = a.tables[a.n_tiles];
    for (int i = tid; i < ROW_IDX_SLACK; i += T4) a.row_idx[kp_end + i] = 0;
    if constexpr (!TVW)
      for (int i = tid; i < KSTEP_TW * a.G / 8; i += T4) ((u32x4*)(a.vals + (size_t)kp_end * a.G))[i] = u32x4{0u, 0u, 0u, 0u};
    for (int i = tid; i < a.n_zero; i += T4) a.zero_cols[i] = a.dropped[i];
    for (int i = tid; i < a.n_table; i += T4) a.out_tables[i] = a.tables[i];
    int some = 0;
    for (int w = tid; w < a.blocks; w += T4) {
      unsigned long long x = 0;
#pragma unroll 8
      for (int u = 0; u < a.n_tiles; ++u) x |= bits[(size_t)u * a.blocks + w];
      some += __popcll(x);
    }
    int all;
    sum_before(some, part, &all);
    if (tid == 0) __hip_atomic_store(a.result, (uint32_t)all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return;
  }
  size_t kp0;
  int kp;
  if (a.uniform_kp > 0) { kp = a.uniform_kp; kp0 = (size_t)t * kp; }
  else { kp0 = (size_t)a.tables[t]; kp = a.tables[t + 1] - (int)kp0; }
  if (stage * STEP >= kp) return;
  bits += (size_t)t * a.blocks;
  if (tid == 0) last = 0;
  const int lo = stage * STEP;           // the stage holds kept rows number lo .. lo + STEP - 1
  int kt = 0, top = 0;                   // kept rows so far; the last one this thread has seen
  for (int b0 = 0; b0 < a.blocks; b0 += T4) {
    const unsigned long long x = b0 + tid < a.blocks ? bits[b0 + tid] : 0ull;
    int all;
    const int front = kt + sum_before(__popcll(x), part, &all);
    // the words of this wave that hold rows of the stage, a few whatever K is: a lane per row
    for (unsigned long long hit = __ballot(x != 0 && front < lo + STEP && front + __popcll(x) > lo); hit; hit &= hit - 1) {
      const int i = __ffsll(hit) - 1;
      const unsigned long long w = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, i) |
                                   (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), i) << 32;
      const int p = __builtin_amdgcn_readlane(front, i) + __popcll(w & ((1ull << lane) - 1ull)) - lo;
      if ((w >> lane & 1ull) && p >= 0 && p < STEP) rows[p] = (b0 + tid - lane + i) * 64 + lane;
    }
    if (x) top = (b0 + tid) * 64 + 63 - __clzll((long long)x);
    kt += all;
    if (b0 + T4 < a.blocks) __syncthreads();           // `part` may be used again
  }
  const int left = kt - lo;              // of the stage's rows, those that are kept rows
  if (left < STEP) {                     // the rest repeat the last kept row
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) top = max(top, __shfl_xor(top, d));
    if (lane == 0) atomicMax(&last, top);
  }
  __syncthreads();
  if (tid < STEP) {
    const int row = tid < left ? rows[tid] : last;
    if (tid >= left) rows[tid] = row;
    a.row_idx[kp0 + (size_t)stage * STEP + tid] = row;
  }
  if (stage == 0 && tid < a.G) a.col_idx[t * a.G + tid] = t * a.G + tid < a.n_kept ? a.kept[t * a.G + tid] : -1;
  __syncthreads();
  if constexpr (TVW) {
    if (image_tvw(a, t, kp0, stage, rows, left)) __hip_atomic_store(a.result + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  } else image_tw(a, t, kp0, stage, rows, left);
}

struct DevBuf {               // device allocation freed on scope exit
  void* p = nullptr;
  ~DevBuf() { if (p) (void)hipFree(p); }
  hipError_t alloc(size_t n) { return hipMalloc(&p, n ? n : 1); }
};

// Pinned host memory through which the kernels and the host of one call talk: a part for numbers and tables, and a
// part that only ever holds tagged words (so that a word with this call's tag was written by this call).
// Allocating it costs more than everything else the host does here (70 us and more), so up to four blocks of the usual size
// are kept, for calls on up to four threads at once; they are given back when the process ends.  The usual size holds the counts of
// 32768 x 32768 at G = 128 and of 16384 x 16384 at G = 32; above that the kernels take ten times as long as the allocation.
constexpr size_t PIN_PLAIN = 64 << 10, PIN_WORDS = 1 << 20;
struct PinnedPool {
  std::mutex m;
  std::vector<char*> idle;
  PinnedPool() { idle.reserve(4); }
  ~PinnedPool() { for (char* p : idle) (void)hipHostFree(p); }
};
PinnedPool& pinned_pool() {
  static PinnedPool pool;     // (made after the runtime, by the first call: destroyed before it)
  return pool;
}
struct Pinned {
  char* p = nullptr;
  bool usual = false;
  unsigned long long* words = nullptr;
  hipError_t get(size_t plain, size_t n_words) {
    usual = plain <= PIN_PLAIN && n_words * 8 <= PIN_WORDS;
    PinnedPool& pool = pinned_pool();
    if (usual) {
      std::lock_guard<std::mutex> lock(pool.m);
      if (!pool.idle.empty()) { p = pool.idle.back(); pool.idle.pop_back(); }
    }
    const size_t first = usual ? PIN_PLAIN : (plain + 63) / 64 * 64, rest = usual ? PIN_WORDS : n_words * 8;
    if (!p) {
      const hipError_t e = hipHostMalloc((void**)&p, first + rest, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent);
      if (e != hipSuccess) { p = nullptr; return e; }
      std::memset(p, 0, first + rest);
    }
    words = (unsigned long long*)(p + first);
    return hipSuccess;
  }
  ~Pinned() {
    if (!p) return;
    if (usual) {
      PinnedPool& pool = pinned_pool();
      std::lock_guard<std::mutex> lock(pool.m);
      if (pool.idle.size() < 4) { pool.idle.push_back(p); return; }
    }
    (void)hipHostFree(p);
  }
};
std::atomic<uint32_t> next_tag{1};

// Waits until words [0, n) carry the tag.  The stream itself is waited for where that takes long (work of the caller in
// front of ours); a stream that has ended without them has failed.
bool wait_for_tags(const unsigned long long* words, size_t n, uint32_t tag, hipStream_t s) {
  size_t i = 0;
  auto look = [&] {
    while (i < n && (uint32_t)(__atomic_load_n(words + i, __ATOMIC_RELAXED) >> 32) == tag) ++i;
    return i == n;
  };
  for (int spin = 0; spin < 4000; ++spin) {
    if (look()) return true;
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
  }
  return hipStreamSynchronize(s) == hipSuccess && look();
}

struct Launched {             // kernels of ours may be running: nothing they use is given back before they have ended
  hipStream_t s;
  bool running = false;
  ~Launched() { if (running) (void)hipStreamSynchronize(s); }
};

size_t up(size_t x) { return (x + 255) / 256 * 256; }

#define TWG_TRY(expr) do { if ((expr) != hipSuccess) { (void)hipGetLastError(); return TW_ERR_HIP; } } while (0)
#define TWG_LAUNCH(kernel, grid, block, ...)                                  \
  do {                                                                        \
    if (launch_kernel(kernel, grid, block, s, __VA_ARGS__) != hipSuccess) return TW_ERR_HIP; \
  } while (0)

}  // namespace

tw_status pack_device(const uint16_t* B, int ldb, const uint8_t* mask, const uint8_t* tile_mask, int K, int N,
                      int G, int pattern, hipStream_t s, tw_handle_s* h) try {
  const bool tvw = pattern == TW_PATTERN_TVW;
  const uint8_t* S = (tvw && tile_mask) ? tile_mask : mask;
  h->K = K; h->N = N; h->G = G; h->pattern = pattern;
  if ((size_t)K * N / T + 1 > 0x7fffffffu) return TW_ERR_UNSUPPORTED;
  const int lg = G == 128 ? 7 : G == 64 ? 6 : 5;
  const size_t ntmax = (size_t)(N + G - 1) / G;
  const int blocks = (K + 63) / 64;
  (void)hipGetLastError();
  // A stream under capture: nothing would run before the wait below.  Asked first, because an allocation can end the
  // caller's capture.
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  TWG_TRY(hipStreamIsCapturing(s, &capturing));
  if (capturing != hipStreamCaptureStatusNone) return TW_ERR_HIP;

  // ---- structure: kept columns, kept rows per tile --------------------------------------
  DevBuf ws;
  Pinned pin;
  Launched ours{s};
  const unsigned nb = (unsigned)((N + 127) / 128);
  // column bits: a workgroup per CU at most, 1024 rows at least for each
  const int slices = std::max(1, std::min({16, 256 / (int)std::min(nb, 256u), (K + 1023) / 1024})), slice_rows = (K + slices - 1) / slices;
  const size_t o_rbits = up((size_t)nb * 16 * slices), o_kept = o_rbits + up(ntmax * blocks * 8), o_drop = o_kept + up((size_t)N * 4);
  const size_t plain = 64 + (6 * ntmax + 256) * 4;                   // two numbers, then the tables (each 256-byte aligned)
  if (ws.alloc(o_drop + (size_t)N * 4) != hipSuccess || pin.get(plain, 1 + ntmax * blocks) != hipSuccess) {
    (void)hipGetLastError();
    return TW_ERR_ALLOC;
  }
  char* w = (char*)ws.p;
  const uint32_t tag = next_tag.fetch_add(1);
  TWG_LAUNCH(column_bits, dim3(nb, (unsigned)slices), dim3(1024), S, K, N, slice_rows, (uint16_t*)w);
  ours.running = true;
  RowArgs r{};
  r.S = S;
  r.element = tvw && tile_mask ? mask : nullptr;
  // only the row-major kernel asks whether all weights are finite, of TW weights and where K takes several bands
  r.B = !tvw && K > MK_KC ? B : nullptr;
  r.ldb = ldb;
  r.K = K; r.N = N; r.lg = lg; r.blocks = blocks;
  r.col_bits = (const unsigned long long*)w;
  r.slices = slices; r.stride = (int)nb * 2;
  r.row_bits = (unsigned long long*)(w + o_rbits);
  r.kept = (int32_t*)(w + o_kept); r.dropped = (int32_t*)(w + o_drop);
  r.host = pin.words; r.tag = tag;
  r.n_wgs = (uint32_t)(ntmax * blocks);
  const Grid2 rg = grid_of(ntmax * blocks, T);
  TWG_LAUNCH(tile_rows, dim3(rg.x, rg.y), dim3(T), r);

  // ---- plan: the counts visit the host ----------------------------------------------------
  if (!wait_for_tags(pin.words, 1 + ntmax * blocks, tag, s)) { (void)hipGetLastError(); return TW_ERR_HIP; }
  h->n_kept = (int)(uint32_t)pin.words[0];
  const int n_tiles = h->n_tiles = (h->n_kept + G - 1) / G;
  h->tile_k_off.assign(n_tiles + 1, 0);
  h->tile_col_off.resize(n_tiles + 1);
  h->sum_kw = 0;
  int64_t nnz = 0;
  uint32_t flags = 0;
  for (int t = 0; t <= n_tiles; ++t) h->tile_col_off[t] = std::min(t * G, h->n_kept);
  for (int t = 0; t < std::max(n_tiles, 1); ++t) {
    int kt = 0;
    for (int b = 0; b < blocks; ++b) {
      const uint32_t x = (uint32_t)pin.words[1 + (size_t)t * blocks + b];
      nnz += x & 0xffffu;
      kt += (int)(x >> ROWS_KEPT_SHIFT & 0xffu);
      flags |= x;
    }
    if (t == n_tiles) break;             // nothing kept
    h->tile_k_off[t + 1] = h->tile_k_off[t] + kt;
    h->sum_kw += (int64_t)kt * (h->tile_col_off[t + 1] - h->tile_col_off[t]);
  }
  if (flags & OUTSIDE_BIT) return TW_ERR_MASK;
  h->sum_k = h->tile_k_off[n_tiles];
  h->nonfinite = (flags & NONFINITE_BIT) != 0;
  if (!tvw || tile_mask) {               // tile-wise: the structure mask is the union of its tiles' rows x columns
    if (nnz != h->sum_kw) return TW_ERR_MASK;
  }
  h->host_lists_ready = h->host_values_ready = false;
  plan_tiles(h);
  int dev = -1;
  TWG_TRY(hipGetDevice(&dev));
  ImageLayout L;
  layout_image(h, &L);
  void* blob = nullptr;
  if (hipMalloc(&blob, L.total) != hipSuccess) { (void)hipGetLastError(); return TW_ERR_ALLOC; }
  bind_image(h, blob, L, dev);           // (from here on tw_free releases it)
  twg::DeviceImage& d = h->img;

  // ---- image: lists and values, and the host's tables as they will lie in it ------------------------
  static_assert(IMG_TILE_KP_OFF == 0 && IMG_TILE_ORDER == 1 && IMG_TILE_SCHED == 2 && IMG_COL_IDX == 3, "the tables come first");
  char* tables = pin.p + 64;
  std::copy_n((const char*)d.tile_kp_off.data(), L.bytes[IMG_TILE_KP_OFF], tables + L.off[IMG_TILE_KP_OFF]);
  std::copy_n((const char*)d.tile_order.data(), L.bytes[IMG_TILE_ORDER], tables + L.off[IMG_TILE_ORDER]);
  std::copy_n((const char*)d.tile_sched.data(), L.bytes[IMG_TILE_SCHED], tables + L.off[IMG_TILE_SCHED]);
  volatile uint32_t* result = (volatile uint32_t*)pin.p;
  result[0] = result[1] = 0;
  const int step = tvw ? KSTEP_TVW : KSTEP_TW;
  ImageArgs m{};
  m.B = B; m.mask = mask; m.kept = r.kept; m.dropped = r.dropped; m.row_bits = r.row_bits;
  m.tables = (const int32_t*)tables; m.n_table = (int)(L.off[IMG_COL_IDX] / 4); m.out_tables = (int32_t*)blob;
  m.ldb = ldb; m.K = K; m.N = N; m.G = G; m.blocks = blocks; m.n_kept = h->n_kept; m.n_zero = d.n_zero; m.n_tiles = n_tiles;
  m.uniform_kp = d.uniform_kp; m.stages = std::max(h->max_kp / step, 1);
  m.row_idx = (int32_t*)d.d_row_idx; m.col_idx = (int32_t*)d.d_col_idx; m.zero_cols = (int32_t*)d.d_zero_cols;
  m.vals = (uint16_t*)d.d_vals; m.meta = (uint16_t*)d.d_meta; m.valid = (uint8_t*)d.d_valid;
  m.result = (uint32_t*)pin.p;
  const Grid2 ig = grid_of((uint64_t)n_tiles * (uint64_t)m.stages + 1, 4 * G);
  const dim3 grid(ig.x, ig.y), block(4 * G);
  if (tvw) TWG_LAUNCH(build_image<true>, grid, block, m);
  else TWG_LAUNCH(build_image<false>, grid, block, m);
  // The handle may be used on any stream from now on.  (The one wait for the stream: 9 us with up to seven launches
  // behind it, 20 to 30 with more, which is why a prune and a pack are three launches each; waiting for an event or
  // for a copy instead leaves the 20 to 30 us to the next hipFree.)
  TWG_TRY(hipStreamSynchronize(s));
  ours.running = false;
  h->k_union = (int32_t)result[0];
  return result[1] ? TW_ERR_MASK : TW_OK;
} catch (const std::bad_alloc&) {
  return TW_ERR_ALLOC;
}

// ---- the logical form of a device-packed handle, read back from its image on first use ------------
static std::mutex fetch_mutex;

static tw_status fetch_lists_locked(tw_handle_s* h) {
  if (h->host_lists_ready) return TW_OK;
  DeviceImage& d = h->img;
  const int G = h->G, nt = h->n_tiles;
  d.col_idx.resize((size_t)nt * G);
  d.row_idx.resize((size_t)d.tile_kp_off[nt] + ROW_IDX_SLACK);
  d.zero_cols.resize((size_t)d.n_zero);
  TWG_TRY(hipMemcpy(d.col_idx.data(), d.d_col_idx, d.col_idx.size() * 4, hipMemcpyDeviceToHost));
  TWG_TRY(hipMemcpy(d.row_idx.data(), d.d_row_idx, d.row_idx.size() * 4, hipMemcpyDeviceToHost));
  TWG_TRY(hipMemcpy(d.zero_cols.data(), d.d_zero_cols, d.zero_cols.size() * 4, hipMemcpyDeviceToHost));
  h->col_idx.assign(d.col_idx.begin(), d.col_idx.begin() + h->n_kept);     // tiles of G: only the last is narrower
  h->row_idx.clear();
  for (int t = 0; t < nt; ++t)
    h->row_idx.insert(h->row_idx.end(), d.row_idx.begin() + d.tile_kp_off[t],
                      d.row_idx.begin() + d.tile_kp_off[t] + (h->tile_k_off[t + 1] - h->tile_k_off[t]));
  derive_offsets(h);
  h->host_lists_ready = true;
  return TW_OK;
}

tw_status fetch_lists(tw_handle_s* h) try {
  std::lock_guard<std::mutex> lock(fetch_mutex);
  return fetch_lists_locked(h);
} catch (const std::bad_alloc&) {
  return TW_ERR_ALLOC;
}

tw_status fetch_logical(tw_handle_s* h) try {
  std::lock_guard<std::mutex> lock(fetch_mutex);
  const tw_status st = fetch_lists_locked(h);
  if (st != TW_OK || h->host_values_ready) return st;
  const DeviceImage& d = h->img;
  const int G = h->G, nt = h->n_tiles, nbt = G / 32;
  std::vector<uint16_t> img(d.n_vals);
  TWG_TRY(hipMemcpy(img.data(), d.d_vals, img.size() * 2, hipMemcpyDeviceToHost));
  h->values.assign((size_t)h->val_off[nt], 0);
  std::vector<uint16_t> words;
  std::vector<uint8_t> vbits;
  if (h->pattern == TW_PATTERN_TVW) {
    words.resize(d.n_meta * 2);
    vbits.resize(d.n_meta * 2);
    TWG_TRY(hipMemcpy(words.data(), d.d_meta, words.size() * 2, hipMemcpyDeviceToHost));
    TWG_TRY(hipMemcpy(vbits.data(), d.d_valid, vbits.size(), hipMemcpyDeviceToHost));
    h->meta.assign((size_t)h->meta_off[nt], 0);
    h->valid.assign((size_t)h->meta_off[nt], 0);
  }
  for (int t = 0; t < nt; ++t) {
    const int kt = h->tile_k_off[t + 1] - h->tile_k_off[t], wt = h->tile_col_off[t + 1] - h->tile_col_off[t];
    const size_t kp0 = (size_t)d.tile_kp_off[t];
    uint16_t* v = h->values.data() + h->val_off[t];
    if (h->pattern != TW_PATTERN_TVW) {
      const uint16_t* o = img.data() + kp0 * G;
      for (int j = 0; j < kt; ++j)
        for (int c = 0; c < wt; ++c)
          v[(size_t)j * wt + c] = o[(size_t)(j / 16) * G * 16 + (c / 32) * 512 + ((j % 16) / 8 * 32 + c % 32) * 8 + j % 8];
      continue;
    }
    const uint16_t* o = img.data() + kp0 / 2 * G;
    for (int g = 0; g < (kt + 3) / 4; ++g)
      for (int c = 0; c < wt; ++c) {
        const int su = g / 8, l = (g % 8) / 4 * 32 + c % 32, j = g % 4, nb = c / 32;
        const uint16_t* e = o + (((size_t)su * nbt + nb) * 64 + l) * 8;
        const size_t word = 2 * ((kp0 / 64 + su / 2) * nbt * 64 + nb * 64 + l) + (su & 1);
        v[((size_t)g * 2 + 0) * wt + c] = e[2 * j];
        v[((size_t)g * 2 + 1) * wt + c] = e[2 * j + 1];
        h->meta[h->meta_off[t] + (size_t)g * wt + c] = (uint8_t)(words[word] >> (4 * j) & 15);
        h->valid[h->meta_off[t] + (size_t)g * wt + c] = (uint8_t)(vbits[word] >> (2 * j) & 3);
      }
  }
  h->host_values_ready = true;
  return TW_OK;
} catch (const std::bad_alloc&) {
  return TW_ERR_ALLOC;
}

}  // namespace twg
