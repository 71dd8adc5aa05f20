// One-shot magnitude pruning of a device-resident weight into a TW / TVW mask
// (Algorithm 3: TW-C on whole columns, Condense, TW-R on the (1,G) row pieces of
// every tile of kept columns; TVW: then 2 of every 4 consecutive kept rows per
// column, Algorithm 2's VW with vectors of 4 and 50 %).  The importance score
// is the sum of squares (Section IV names weight magnitude as the simplest score;
// the paper's Taylor score needs gradients).
//
// Scores are exact: an fp16 value is an integer multiple of 2^-24, its square
// an integer multiple of 2^-48 below 2^80, and the sums are kept in integers of
// up to 128 bits, so the ranking does not depend on the order of summation and a
// host implementation with big integers takes the same decisions.  Ranking is
// by (score, index): the lowest n are pruned, equal scores lose the lower index
// first.
//
// What bounds it: three launches one after the other on a weight of a few MB, each of them a
// few dependent trips to memory (four for tall weights, 4096 rows and more).  Whole call, seven launches / now: 1024 x 4096 at
// 87.5 % (TVW) 39.8 / 34.0 us, 64 x 64 25.6 / 14.4, 3072 x 768 44.0 / 33.7, 4096 x 4096 66.0 / 61.2, 25088 x 512 120 / 97.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "device_common.h"
#include "prune.h"

namespace twg {

namespace {

typedef unsigned __int128 u128;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));
constexpr int SCAN_T = 1024, SCAN_WAVES = SCAN_T / 64;   // threads and waves of a workgroup that selects

__device__ __forceinline__ uint64_t magnitude24(uint16_t h) {   // |value| in units of 2^-24
  const uint32_t e = (h >> 10) & 31u, m = h & 1023u;
  return e == 0 ? (uint64_t)m : (uint64_t)(m | 1024u) << (e - 1);
}

// Sum of squares.  Values below 1 have squares below 2^48: 2^15 of them fit a 64-bit sum; larger values go
// to a 128-bit sum of their own.  Up to 32 squares of values below 1 are added in fp64 first, exactly: a
// square is a multiple of 2^-48 and their sum is below 2^5 (one full-rate instruction, where a 64-bit integer
// multiply-add runs at a quarter of the rate).
struct Sum {
  uint64_t lo = 0;
  u128 hi = 0;
  double few = 0.0;
  __device__ __forceinline__ void add_small(uint16_t h) {         // |value| < 1; flush() after 32 at the latest
    union { uint16_t b; _Float16 f; } x;
    x.b = h;
    const double v = (double)(float)x.f;
    few = __builtin_fma(v, v, few);
  }
  __device__ __forceinline__ void flush() {
    lo += (uint64_t)(few * 281474976710656.0);                     // 2^48
    few = 0.0;
  }
  __device__ __forceinline__ void add(uint16_t h) {
    const uint64_t a = magnitude24(h);
    if (a < (1u << 24)) lo += (uint64_t)(uint32_t)a * (uint32_t)a;
    else hi += (u128)a * (u128)a;
  }
  __device__ __forceinline__ void carry() { hi += lo; lo = 0; }
};
// Non-zero where one of the two halves of x is 1 or more (infinities and NaN among them).
__device__ __forceinline__ uint32_t one_or_more(uint32_t x) { return ((x & 0x7fff7fffu) + 0x44004400u) & 0x80008000u; }

// Sum over the lanes whose ids differ in the bits FROM .. TO (powers of two), in every lane.  Their sums
// in `lo` together stay below 2^64.
template <int FROM, int TO>
__device__ __forceinline__ u128 sum_over_lanes(const Sum& s) {
  unsigned long long lo = s.lo;
#pragma unroll
  for (int d = FROM; d <= TO; d <<= 1) lo += __shfl_xor(lo, d);
  u128 total = lo;
  if (__any(s.hi != 0)) {                      // three 32-bit limbs, each in a 64-bit word
    unsigned long long h0 = (uint32_t)s.hi, h1 = (uint32_t)(s.hi >> 32), h2 = (unsigned long long)(s.hi >> 64);
#pragma unroll
    for (int d = FROM; d <= TO; d <<= 1) {
      h0 += __shfl_xor(h0, d);
      h1 += __shfl_xor(h1, d);
      h2 += __shfl_xor(h2, d);
    }
    total += (u128)h0 + ((u128)h1 << 32) + ((u128)h2 << 64);
  }
  return total;
}

// TW-C scores, exact and independent of any order (integer sums).  A workgroup of 1024 threads takes CW columns:
// lanes of 4 columns, 4 loads of 8 bytes in flight per thread.  CW = 16: all rows, 256 at a time; neighbouring
// workgroups, which share the 128-byte lines, run on one XCD and meet in its L2.  One kernel, where slices of the
// rows and a second kernel to add them up took 9.8 us and a launch more for 1024 x 4096.  CW = 64, tall or wide weights: blockIdx.y is a
// slice of `slice` rows with scores of its own, which add_slices() adds up.  (With 25088 rows of 4096 columns the workgroups that share
// lines drift apart: 144 us in one piece, 91 in slices.)
template <int CW>
__global__ __launch_bounds__(1024) void column_scores(const uint16_t* B, int K, int N, int ldb, int vec, int slice, u128* score) {
  constexpr int LANES = CW / 4, ROWS = 1024 / LANES, U = 4;
  __shared__ u128 part[16][CW];
  const int tid = threadIdx.x, c4 = tid % LANES;
  const int n_block = xcd_remap(blockIdx.x, gridDim.x) * CW;
  const int n = n_block + c4 * 4;
  Sum s[4];
  int rows = 0;
  const int k_end = min(K, ((int)blockIdx.y + 1) * slice);
  for (int k0 = (int)blockIdx.y * slice + tid / LANES; k0 < k_end; k0 += U * ROWS) {
    union { uint2 v; uint16_t e[4]; } x[U];
    uint32_t big = 0;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      x[i].v = uint2{0u, 0u};
      const int k = k0 + i * ROWS;
      if (k >= k_end) continue;
      const uint16_t* p = B + (size_t)k * ldb + n;
      if (vec && n + 4 <= N) x[i].v = *(const uint2*)p;
      else
        for (int c = 0; c < 4; ++c) if (n + c < N) x[i].e[c] = p[c];
    }
#pragma unroll
    for (int i = 0; i < U; ++i) big |= one_or_more(x[i].v.x) | one_or_more(x[i].v.y);
    if (!__any(big != 0)) {
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c].add_small(x[i].e[c]);
#pragma unroll
      for (int c = 0; c < 4; ++c) s[c].flush();
    } else {
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c].add(x[i].e[c]);
    }
    if ((rows += U) >= (1 << 15)) {
      rows = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) s[c].carry();
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    if (slice > (1 << 15)) s[c].carry();       // (the lanes' 64-bit sums together would not fit)
    const u128 w = sum_over_lanes<LANES, 32>(s[c]);
    if ((tid & 63) < LANES) part[tid >> 6][c4 * 4 + c] = w;
  }
  __syncthreads();
  const int col = n_block + tid;
  if (tid >= CW || col >= N) return;
  u128 t = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) t += part[w][tid];
  score[(size_t)blockIdx.y * N + col] = t;
}
__global__ void add_slices(const u128* partial, int slices, int N, u128* score) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  u128 t = 0;
#pragma unroll 16
  for (int y = 0; y < slices; ++y) t += partial[(size_t)y * N + n];
  score[n] = t;
}

// Which entries of a segment of scores are kept: all but the n_pruned lowest in (score, index) order.  For the
// SCAN_T threads of a workgroup, R rounds of SCAN_T entries at a time; REG: one such block holds the segment and
// its scores stay in registers, else they are read again in every pass.
//   1. the bits that all scores share at the top are skipped (OR of the differences to entry 0);
//   2. the threshold is found 8 bits at a time from histograms in LDS, in windows of 32 bits of the
//      score, so that a pass compares 32-bit numbers; every wave finds the digit's value by itself.  It is settled
//      as soon as all scores with its leading bits are pruned, usually after two or three digits;
//   3. scores equal to a threshold that had to be followed to its last bit are pruned in index
//      order, and the kept entries are numbered in order: out(i, number among the kept or -1) for every entry.
// What bounds it: one CU's instruction rate (with 128-bit shifts and compares in every pass 9.7 us for 4096
// entries, now 7.5 as a kernel of its own) and the chain of barriers.
struct SelectLds {
  __attribute__((aligned(16))) int hist[4][256];
  int part[2][4 * SCAN_WAVES];
  unsigned long long diff[2 * SCAN_WAVES];
};
template <int R, bool REG, class Out>
__device__ __forceinline__ void select_entries(const u128* s, int len, int n_pruned, SelectLds& lds, Out out) {
  static_assert(R * SCAN_WAVES <= 64, "a lane per count");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int blocks = REG ? 1 : (len - 1) / (R * SCAN_T) + 1;
  u128 key[R];
  auto load = [&](int b) {
#pragma unroll
    for (int r = 0; r < R; ++r) key[r] = s[min((b * R + r) * SCAN_T + tid, len - 1)];
  };
  auto there = [&](int b, int r) { return (b * R + r) * SCAN_T + tid < len; };
  if constexpr (REG) load(0);
  auto each = [&](auto f) {                    // f(score) for this thread's entries
    for (int b = 0; b < blocks; ++b) {
      if constexpr (!REG) load(b);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (there(b, r)) f(key[r]);
    }
  };
  // Scores whose bits above `shift` equal `prefix` are still open: the lowest `need` of them go.
  u128 prefix = 0;
  int shift = 0, need = n_pruned;
  bool all_equal_go = true;
  const bool some = n_pruned > 0 && n_pruned < len;                  // (uniform over the workgroup)
  if (some) {
    const u128 first = s[0];
    unsigned long long d0 = 0, d1 = 0;
    each([&](u128 v) { const u128 d = v ^ first; d0 |= (unsigned long long)d; d1 |= (unsigned long long)(d >> 64); });
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) { d0 |= __shfl_xor(d0, k); d1 |= __shfl_xor(d1, k); }
    if (lane == 0) { lds.diff[wave] = d0; lds.diff[SCAN_WAVES + wave] = d1; }
    if (tid < 4 * 64) *(i32x4_t*)&lds.hist[0][tid * 4] = i32x4_t{0, 0, 0, 0};
    __syncthreads();
    d0 = d1 = 0;
#pragma unroll
    for (int w = 0; w < SCAN_WAVES; ++w) { d0 |= lds.diff[w]; d1 |= lds.diff[SCAN_WAVES + w]; }
    shift = d1 ? 128 - __clzll((long long)d1) : d0 ? 64 - __clzll((long long)d0) : 0;
    shift = __builtin_amdgcn_readfirstlane(shift);
    prefix = shift < 128 ? first >> shift : 0;
    all_equal_go = false;
    while (shift > 0 && !all_equal_go) {       // a window of the 32 bits below `shift`, left-aligned
      const int base = shift > 32 ? shift - 32 : 0, width = shift - base;
      uint32_t win[R];
      bool open[R];
      auto window = [&](u128 v) { return (uint32_t)(v >> base) << (32 - width); };
      auto is_open = [&](u128 v) { return shift >= 128 || v >> shift == prefix; };
      if constexpr (REG) {
#pragma unroll
        for (int r = 0; r < R; ++r) { open[r] = there(0, r) && is_open(key[r]); win[r] = window(key[r]); }
      }
      uint32_t found = 0;                      // leading bits of the threshold's window
      int done = 0;
      for (int d = 0; done < width && !all_equal_go; ++d) {
        const uint32_t lead = done ? ~0u << (32 - done) : 0u;
        auto count = [&](uint32_t x) {
          if ((x & lead) == found) atomicAdd(&lds.hist[d][(x << done) >> 24], 1);
        };
        if constexpr (REG) {
#pragma unroll
          for (int r = 0; r < R; ++r) if (open[r]) count(win[r]);
        } else each([&](u128 v) { if (is_open(v)) count(window(v)); });
        __syncthreads();
        // four bins per lane: the bin that holds entry number `need`
        const i32x4_t n = *(const i32x4_t*)&lds.hist[d][lane * 4];
        const int sum = n[0] + n[1] + n[2] + n[3];
        int before = sum;
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) { const int t = __shfl_up(before, k); before += lane >= k ? t : 0; }
        before -= sum;
        const int src = __ffsll(__ballot(before < need && need <= before + sum)) - 1;      // exactly one lane
        int bin = lane * 4, in_bin = n[0];
#pragma unroll
        for (int j = 1; j < 4; ++j)
          if (need > before + in_bin) { before += in_bin; in_bin = n[j]; ++bin; }
        found |= (uint32_t)__builtin_amdgcn_readlane(bin, src) << 24 >> done;
        need -= __builtin_amdgcn_readlane(before, src);
        done += 8;
        all_equal_go = __builtin_amdgcn_readlane(in_bin, src) == need;
      }
      done = min(done, width);
      prefix = prefix << done | found >> (32 - done);
      shift -= done;
      if (shift > 0 && !all_equal_go) {        // the next window's histograms
        __syncthreads();
        if (tid < 4 * 64) *(i32x4_t*)&lds.hist[0][tid * 4] = i32x4_t{0, 0, 0, 0};
        __syncthreads();
      }
    }
  }
  // In order: round after round, wave after wave.  Numbers of the entries of a kind in front of a wave's in each
  // round of a block come from one scan over the waves' counts.
  auto fronts = [&](const bool (&v)[R], int* p, int base, int (&front)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      front[r] = __popcll(__ballot(v[r]));
      if (lane == 0) p[r * SCAN_WAVES + wave] = front[r];
    }
    __syncthreads();
    const int mine = lane < R * SCAN_WAVES ? p[lane] : 0;
    int in = mine;
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) { const int t = __shfl_up(in, k); in += lane >= k ? t : 0; }
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < R; ++r)
      front[r] = base + __shfl(in - mine, r * SCAN_WAVES + wave) + __popcll(__ballot(v[r]) & below);
    return base + __shfl(in, 63);
  };
  int n_equal = 0, n_kept = 0;                 // in the blocks before
  for (int b = 0; b < blocks; ++b) {
    if constexpr (!REG) load(b);
    bool keep[R], equal[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const u128 top = key[r] >> shift;
      keep[r] = there(b, r) && n_pruned < len && (!some || top > prefix);
      equal[r] = there(b, r) && some && !all_equal_go && top == prefix;
    }
    int at[R];
    if (some && !all_equal_go) {
      n_equal = fronts(equal, lds.part[0], n_equal, at);
#pragma unroll
      for (int r = 0; r < R; ++r) keep[r] |= equal[r] && at[r] >= need;
    }
    n_kept = fronts(keep, lds.part[1], n_kept, at);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (there(b, r)) out((b * R + r) * SCAN_T + tid, keep[r] ? at[r] : -1);
    if (b + 1 < blocks) __syncthreads();       // `part` may be used again
  }
}

// Segments too long for registers: a kernel of their own, one workgroup per segment.
// pos[i] = number among the kept or -1, list[pos] = i.
__global__ __launch_bounds__(SCAN_T) void select_kept(const u128* scores, int len, int n_pruned, int32_t* pos, int32_t* list) {
  __shared__ SelectLds lds;
  const size_t at = (size_t)blockIdx.x * len;
  select_entries<4, false>(scores + at, len, n_pruned, lds, [&](int i, int p) {
    pos[at + i] = p;
    if (p >= 0) list[at + p] = i;
  });
}

struct PruneArgs {
  const uint16_t* B;
  int K, N, ldb, n_kept, rows_kept;
  const u128* col_score;
  u128* row_score;
  int32_t *col_pos, *kept_cols;        // number among the kept columns or -1; the kept columns
  const int32_t *row_pos, *row_list;   // K > REG_MAX: the same for the rows of each tile
  uint8_t *tiles, *element;            // masks (tiles: or null)
  int blocks, rows;                    // workgroups per tile, rows of each (a multiple of 64)
  int shares;                          // masks: workgroups that share a tile's columns
};
constexpr int REG_MAX = 4 * SCAN_T;    // longest segment that is selected in registers
// The workgroups of neighbouring tiles, which share 128-byte lines of the weight and the masks, run on one XCD: its L2
// puts the lines together.
__device__ __forceinline__ void tile_and_block(const PruneArgs& a, int& t, int& b) {
  const int lid = xcd_remap(blockIdx.x, gridDim.x), tiles = (int)gridDim.x / a.blocks;
  b = lid / tiles;
  t = lid - b * tiles;
}

// TW-R scores: tile t = kept columns [t*G, min((t+1)*G, n_kept)); 16 lanes per (tile, row), their
// columns 16 apart.  Workgroup (tile, block of rows).  R > 0: every workgroup first selects the kept columns for itself
// (the first one writes them down): as long as a kernel that selects them alone on one CU, and a launch less.
template <int G, int R>
__global__ __launch_bounds__(1024) void tile_row_scores(PruneArgs a) {
  constexpr int U = 2;                         // rows per thread and step
  __shared__ SelectLds lds;
  __shared__ int32_t list[R > 0 ? R * SCAN_T : 1];
  int t, b;
  tile_and_block(a, t, b);
  const int l = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int32_t* cols = a.kept_cols + (size_t)t * G;
  if constexpr (R > 0) {
    select_entries<R, true>(a.col_score, a.N, a.N - a.n_kept, lds, [&](int i, int p) {
      if (blockIdx.x == 0) a.col_pos[i] = p;
      if (p < 0) return;
      list[p] = i;
      if (blockIdx.x == 0) a.kept_cols[p] = i;
    });
    __syncthreads();
    cols = list + t * G;
  }
  const int w = min(G, a.n_kept - t * G);      // (nothing kept at all: one workgroup, which is done)
  if (w <= 0) return;
  int col[G / 16];
#pragma unroll
  for (int i = 0; i < G / 16; ++i) col[i] = cols[min(l + 16 * i, w - 1)];
  const int k_end = min(a.K, (b + 1) * a.rows);
  for (int k0 = b * a.rows + g; k0 < k_end; k0 += 64 * U) {
    uint16_t v[U][G / 16];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const uint16_t* row = a.B + (size_t)min(k0 + 64 * r, a.K - 1) * a.ldb;
#pragma unroll
      for (int i = 0; i < G / 16; ++i) v[r][i] = row[col[i]];
    }
    uint32_t big = 0;
#pragma unroll
    for (int r = 0; r < U; ++r)
#pragma unroll
      for (int i = 0; i < G / 16; ++i) {
        if (l + 16 * i >= w) v[r][i] = 0;
        big |= one_or_more(v[r][i]);
      }
    const bool small = !__any(big != 0);
#pragma unroll
    for (int r = 0; r < U; ++r) {
      Sum s;
      if (small) {
#pragma unroll
        for (int i = 0; i < G / 16; ++i) s.add_small(v[r][i]);
        s.flush();
      } else {
#pragma unroll
        for (int i = 0; i < G / 16; ++i) s.add(v[r][i]);
      }
      const u128 total = sum_over_lanes<1, 8>(s);
      const int k = k0 + 64 * r;
      if (k < k_end && l == 0) a.row_score[(size_t)t * a.K + k] = total;
    }
  }
}

// Bytes [from, to) of a 16-byte piece, aligned: one store, or up to four that the end leaves room for.
__device__ __forceinline__ void store_piece(uint8_t* p, const u32x4_t& v, int from, int to) {
  if (from <= 0 && to >= 16) { *(u32x4_t*)p = v; return; }
  const uint64_t q0 = v[0] | (uint64_t)v[1] << 32, q1 = v[2] | (uint64_t)v[3] << 32;
  // (arithmetic: a conditional of the two halves ends up as an indexed read of a copy in LDS)
  auto bytes = [=](int o) { return (q0 ^ ((q0 ^ q1) & (0ull - (uint64_t)(o >> 3 & 1)))) >> (8 * (o & 7)); };
  if (from > 0 && to < 16) {
    for (int o = from; o < to; ++o) p[o] = (uint8_t)bytes(o);
    return;
  }
  int o = from > 0 ? from : 0;
  const int n = from > 0 ? 16 - from : to;
  auto piece = [&](int size) {
    if (!(n & size)) return;
    if (size == 8) *(uint64_t*)(p + o) = bytes(o);
    else if (size == 4) *(uint32_t*)(p + o) = (uint32_t)bytes(o);
    else if (size == 2) *(uint16_t*)(p + o) = (uint16_t)bytes(o);
    else p[o] = (uint8_t)bytes(o);
    o += size;
  };
  if (from > 0) { piece(1); piece(2); piece(4); piece(8); }
  else { piece(8); piece(4); piece(2); piece(1); }
}

// The masks.  tiles[k][n] = column n kept and row k kept in n's tile (may be null).  TVW: element[k][n], of those,
// 2:4 along the condensed kept rows of the tile: in every group of 4 consecutive kept rows and every column
// the 2 largest |w| stay; equal magnitudes: the lower position stays.
// Workgroup (tile, block of rows, share of the columns): the tile answers for the columns from its first kept one (tile 0:
// from 0) to the next tile's (the last: to N).  R > 0: the workgroup first selects the tile's kept rows for itself.  Then a team of
// G / 8 lanes takes a row, 16 bytes of the mask each, aligned whatever N is.  TVW by rows: in a kept row a lane reads the
// weights of the group's four rows and ranks its own row among them; by groups: a team reads and ranks the four rows once.  What bounds it: the selection (4 us), then
// the number of store instructions: the pieces that two tiles share are written in up to four parts.
constexpr int COL_BITS = 65536;                // columns a tile may answer for with their bits in LDS
enum { MASKS_TW = 0, MASKS_TVW_ROWS = 1, MASKS_TVW_GROUPS = 2 };
template <int R, int MODE>
__global__ __launch_bounds__(1024) void emit_masks(PruneArgs a, int lg) {
  __shared__ SelectLds lds;
  __shared__ int32_t pos_lds[R > 0 ? R * SCAN_T : 1], list_lds[R > 0 ? R * SCAN_T : 1];
  __shared__ uint32_t bits[COL_BITS / 32 + 2];
  const int K = a.K, N = a.N, tid = threadIdx.x;
  const int lid = xcd_remap(blockIdx.x, gridDim.x), tiles = (int)gridDim.x / (a.blocks * a.shares);
  const int t = lid % tiles, share = lid / tiles % a.shares, b = lid / (tiles * a.shares);
  const int c0 = t << lg, c1 = min((t + 1) << lg, a.n_kept);
  const int lo = t == 0 ? 0 : a.kept_cols[c0], hi = c1 < a.n_kept ? a.kept_cols[c1] : N;
  const bool few = hi - lo <= COL_BITS;        // (uniform)
  if (few)
    for (int i = tid; i < (hi - lo) / 32 + 2; i += 1024) bits[i] = 0;
  __syncthreads();
  if (few && c0 + tid < c1) {
    const int at = a.kept_cols[c0 + tid] - lo;
    atomicOr(&bits[at >> 5], 1u << (at & 31));
  }
  const int32_t *pos = pos_lds, *list = list_lds;
  if constexpr (R > 0) {
    if (c0 < c1)
      select_entries<R, true>(a.row_score + (size_t)t * K, K, K - a.rows_kept, lds, [&](int i, int p) {
        pos_lds[i] = p;
        if (p >= 0) list_lds[p] = i;
      });
  } else {
    pos = a.row_pos + (size_t)t * K;
    list = a.row_list + (size_t)t * K;
  }
  __syncthreads();
  // 16 columns from n on: which of them are kept ones of the tile
  auto kept16 = [&](int n) {
    uint32_t x = 0;
    if (few) {
      const int at = n - lo;
      if (at < 0) x = bits[0] << -at;          // (n > lo - 16)
      else {
        const unsigned long long w = bits[at >> 5] | (unsigned long long)bits[(at >> 5) + 1] << 32;
        x = (uint32_t)(w >> (at & 31));
      }
    } else {
      for (int c = max(n, lo); c < min(n + 16, hi); ++c) x |= (a.col_pos[c] >= 0 ? 1u : 0u) << (c - n);
    }
    return x & 0xffffu;
  };
  struct __attribute__((packed, aligned(2))) Piece { u32x4_t v; };
  // magnitudes of 16 weights of a row, order of finite fp16; columns outside the row are not used, but may be read where
  // the matrix has them
  const int64_t last_piece = (int64_t)(K - 1) * a.ldb + N - 16;
  auto load16 = [&](int row, int n, uint32_t (&v)[8]) {
    const int64_t first = (int64_t)row * a.ldb + n;
    const uint16_t* p = a.B + first;
    if (first >= 0 && first <= last_piece) {
      const u32x4_t x = ((const Piece*)p)->v, y = ((const Piece*)(p + 8))->v;
#pragma unroll
      for (int j = 0; j < 4; ++j) { v[j] = x[j] & 0x7fff7fffu; v[4 + j] = y[j] & 0x7fff7fffu; }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = n + 2 * j;
        v[j] = (p[min(max(c, 0), N - 1) - n] | (uint32_t)p[min(max(c + 1, 0), N - 1) - n] << 16) & 0x7fff7fffu;
      }
    }
  };
  const bool same = !a.tiles || (((uintptr_t)a.tiles ^ (uintptr_t)a.element) & 15) == 0;
  const int team = lg - 3, lane = tid & ((1 << team) - 1), first_team = tid >> team, teams = 1024 >> team;
  auto expand = [](uint32_t x) {               // four bits each -> bytes 0 / 1
    u32x4_t v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = ((x >> (4 * j) & 15u) * 0x00204081u) & 0x01010101u;
    return v;
  };
  auto store = [&](int k, int n, uint32_t x, const u32x4_t& tb, const u32x4_t& eb) {
    const int from = lo - n, to = hi - n;
    store_piece(a.element + (size_t)k * N + n, eb, from, to);
    if (!a.tiles) return;
    uint8_t* other = a.tiles + (size_t)k * N + n;
    if (same) store_piece(other, tb, from, to);
    else
      for (int c = max(from, 0); c < min(to, 16); ++c) other[c] = (uint8_t)(x >> c & 1u);
  };
  // this lane's columns of a row whose mask starts `off` bytes behind a multiple of 16
  auto first_column = [&](int off) { return ((lo + off) & ~15) - off + 16 * (lane + (share << team)); };
  const int step = 16 * a.shares << team;
  auto offset = [&](int k) { return (int)((uintptr_t)(a.element + (size_t)k * N) & 15); };
  constexpr uint32_t H = 0x80008000u;          // top bits of the halves
  if constexpr (MODE == MASKS_TVW_GROUPS) {
    const int groups = c0 < c1 ? (a.rows_kept + 3) / 4 : 0;
    const int g0 = (int)((int64_t)groups * b / a.blocks), g_end = (int)((int64_t)groups * (b + 1) / a.blocks);
    // (the groups first: while some teams are at them, the others write the rows that are not kept)
    for (int g = g0 + first_team; g < g_end; g += teams) {
      const int cnt = min(4, a.rows_kept - 4 * g);
      int row[4], off[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { row[q] = list[4 * g + min(q, cnt - 1)]; off[q] = offset(row[q]); }
      const bool alike = off[0] == off[1] && off[0] == off[2] && off[0] == off[3];   // (N a multiple of 16, usually)
#pragma unroll 1
      for (int only = 0; only < (alike ? 1 : cnt); ++only) {
        const int o = only == 0 ? off[0] : only == 1 ? off[1] : only == 2 ? off[2] : off[3];
        for (int n = first_column(o); n < hi; n += step) {             // the masks of all rows from column n on, or of one of them
          const uint32_t x = kept16(n);
          const u32x4_t tb = expand(x);
          u32x4_t eb[4] = {tb, tb, tb, tb};
          if (x) {
            uint32_t v[4][8];
#pragma unroll
            for (int q = 0; q < 4; ++q) load16(row[q], n, v[q]);
#pragma unroll
            for (int q = 1; q < 4; ++q)
              if (q >= cnt)                    // past the end of the list: ahead of nobody
#pragma unroll
                for (int j = 0; j < 8; ++j) v[q][j] = 0;
            // top bit of a half: the row in front is as large or larger, so it comes ahead; a row stays unless two come ahead
            auto two = [](uint32_t p, uint32_t q, uint32_t r) { return (p & q) | (r & (p | q)); };   // of three, two at least
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              uint32_t keep[4][2];
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                auto ahead = [&](int p, int q) { return (v[p][2 * j + h] | H) - v[q][2 * j + h]; };
                const uint32_t p01 = ahead(0, 1), p02 = ahead(0, 2), p03 = ahead(0, 3), p12 = ahead(1, 2), p13 = ahead(1, 3), p23 = ahead(2, 3);
                keep[0][h] = two(p01, p02, p03);
                keep[1][h] = two(~p01, p12, p13);
                keep[2][h] = two(~p02, ~p12, p23);
                keep[3][h] = two(~p03, ~p13, ~p23);
              }
#pragma unroll
              for (int q = 0; q < 4; ++q) eb[q][j] &= __builtin_amdgcn_perm(keep[q][1], keep[q][0], 0x07050301u) >> 7;
            }
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q < cnt && (alike || q == only)) store(row[q], n, x, tb, eb[q]);
        }
      }
    }
  }
  const int k_end = min(K, (b + 1) * a.rows);
  for (int k = b * a.rows + first_team; k < k_end; k += teams) {
    const int at = c0 < c1 ? pos[k] : -1;
    if (MODE == MASKS_TVW_GROUPS && at >= 0) continue;
    for (int n = first_column(offset(k)); n < hi; n += step) {
      const uint32_t x = at >= 0 ? kept16(n) : 0u;
      const u32x4_t tb = expand(x);
      u32x4_t eb = tb;
      if constexpr (MODE == MASKS_TVW_ROWS) {
        if (x) {
          const int g = at & ~3, mine = at & 3;
          uint32_t own[8], v[4][8];
          load16(k, n, own);
#pragma unroll
          for (int q = 0; q < 4; ++q)          // past the end of the list: the row itself, which is not ahead of itself
            load16(g + q < a.rows_kept ? list[g + q] : k, n, v[q]);
          // top bit of a half: row q comes ahead, being larger, or (in front) as large
          uint32_t keep[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            uint32_t ahead[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) ahead[q] = (v[q][j] | H) - (own[j] + (q >= mine ? 0x00010001u : 0u));
            const uint32_t two = (ahead[0] & ahead[1]) | (ahead[2] & ahead[3]) | ((ahead[0] | ahead[1]) & (ahead[2] | ahead[3]));
            keep[j] = ~two & H;
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
            eb[j] &= __builtin_amdgcn_perm(keep[2 * j + 1], keep[2 * j], 0x07050301u) >> 7;
        }
      }
      store(k, n, x, tb, eb);
    }
  }
}

size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

size_t prune_workspace_bytes(int K, int N, int G) {
  const size_t nt = (size_t)(N + G - 1) / G;
  // The size is part of the interface: more than the kernels use (one spare list per column and per row, and
  // room for the column scores of `slices` slices of the rows, of which prune_device() takes fewer).
  const int blocks = (N + 255) / 256, slices = K < 512 / blocks ? K : 512 / blocks > 1 ? 512 / blocks : 1;
  return align_up((size_t)N * 16) + 3 * align_up((size_t)N * 4) +          // column score, pos, list
         align_up(nt * K * 16) + 3 * align_up(nt * K * 4) +                 // row score, pos, list
         align_up((size_t)slices * N * 16);
}

hipError_t prune_device(const uint16_t* B, int K, int N, int ldb, int G, bool tvw, int n_cols_pruned,
                        int rows_per_tile, uint8_t* mask, uint8_t* tile_mask, void* workspace,
                        hipStream_t stream) {
  const int n_kept = N - n_cols_pruned;
  const int nt = (n_kept + G - 1) / G;
  char* w = (char*)workspace;
  const size_t ntmax = (size_t)(N + G - 1) / G;
  u128* col_score = (u128*)w;            w += align_up((size_t)N * 16) + align_up((size_t)N * 4);
  int32_t* col_pos = (int32_t*)w;        w += align_up((size_t)N * 4);
  int32_t* kept_cols = (int32_t*)w;      w += align_up((size_t)N * 4);
  u128* row_score = (u128*)w;            w += align_up(ntmax * K * 16) + align_up(ntmax * K * 4);
  int32_t* row_pos = (int32_t*)w;        w += align_up(ntmax * K * 4);
  int32_t* row_list = (int32_t*)w;       w += align_up(ntmax * K * 4);
  u128* partial = (u128*)w;
  const int lg = G == 128 ? 7 : G == 64 ? 6 : 5;
  auto aligned = [](const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; };
  // a failed launch ends the call: later kernels would read workspace nobody wrote
#define TWG_LAUNCH(kernel, grid, block, ...)                                  \
  do {                                                                        \
    const hipError_t e_ = launch_kernel(kernel, grid, block, stream, __VA_ARGS__); \
    if (e_ != hipSuccess) return e_;                                          \
  } while (0)
  // From 4096 rows on: slices of at least 512, 64 columns (a line) wide, one workgroup per CU in all.  In slices / not, whole
  // call: 65536 x 64 124 / 274 us, 25088 x 512 86 / 150, 16384 x 2048 96 / 129, 25088 x 4096 246 / 302, 4096 x 1024 32 / 34,
  // 4608 x 4096 67 / 70; 2304 x 256 29 / 28, 3072 x 768 30 / 31.  Wide weights have enough workgroups of whole lines without
  // (lines / quarters of lines, the kernel alone: 272 x 34912 14 / 32 us, 4096 x 14336 41 / 58, 5120 x 13824 56 / 80).
  const int vec = (int)(ldb % 4 == 0 && aligned(B, 8)), wide_wgs = (N + 63) / 64;
  const int slices = K >= 4096 ? std::max(1, std::min(256 / wide_wgs, K / 512)) : 1;
  if (slices > 1 || wide_wgs >= 128) {
    TWG_LAUNCH(column_scores<64>, dim3((unsigned)wide_wgs, (unsigned)slices), dim3(1024), B, K, N, ldb, vec,
               (K + slices - 1) / slices, slices > 1 ? partial : col_score);
    if (slices > 1) TWG_LAUNCH(add_slices, dim3((unsigned)wide_wgs), dim3(64), partial, slices, N, col_score);
  } else {
    TWG_LAUNCH(column_scores<16>, dim3((unsigned)((N + 15) / 16)), dim3(1024), B, K, N, ldb, vec, K, col_score);
  }
  PruneArgs a{B, K, N, ldb, n_kept, rows_per_tile, col_score, row_score, col_pos, kept_cols, row_pos, row_list, tile_mask, mask, 0, 0, 1};
  // Workgroups of 1024 threads for the tiles, about one per CU: each selects for itself.
  const int tiles = nt > 0 ? nt : 1;
  a.blocks = 256 / tiles > 1 ? 256 / tiles : 1;
  a.rows = ((K + a.blocks - 1) / a.blocks + 63) / 64 * 64;
  a.blocks = (K + a.rows - 1) / a.rows;
  dim3 grid((unsigned)tiles * (unsigned)a.blocks), block(1024);
  // Columns: entries per thread of a selection in registers, or (0) a kernel that selects.
  const int rc = N <= SCAN_T ? 1 : N <= REG_MAX ? 4 : 0, rk = K <= SCAN_T ? 1 : K <= REG_MAX ? 4 : 0;
  if (!rc) TWG_LAUNCH(select_kept, dim3(1), block, col_score, N, n_cols_pruned, col_pos, kept_cols);
#define TWG_ROWS(G_)                                                             \
  do {                                                                           \
    if (rc == 1) TWG_LAUNCH((tile_row_scores<G_, 1>), grid, block, a);           \
    else if (rc == 4) TWG_LAUNCH((tile_row_scores<G_, 4>), grid, block, a);      \
    else TWG_LAUNCH((tile_row_scores<G_, 0>), grid, block, a);                   \
  } while (0)
  if (G == 128) TWG_ROWS(128);
  else if (G == 64) TWG_ROWS(64);
  else TWG_ROWS(32);
  if (!rk && nt > 0) TWG_LAUNCH(select_kept, dim3(nt), block, row_score, K, K - rows_per_tile, row_pos, row_list);
  // Many rows for each workgroup and no selection in them: more workgroups, with about 768 rows, TW 384 (25088 x 4096 TVW
  // 396 -> 371 us, TW 249 -> 240, G = 32, 11008 x 4096 251 -> 214 and 151 -> 138; shorter ones gain nothing: 14336 x 4096 TVW with
  // 1344 rows 192 -> 196, 4608 x 4096 84 -> 91).  With a selection only where one per tile leaves CUs idle, TVW (the masks alone,
  // 3904 x 13520, G = 64, 150 tiles 125 -> 106; TW 50 -> 53, and 4096 x 14336, 80 tiles of three 95 -> 101).
  const bool idle = rk && tvw && a.blocks == 1 && tiles < 256 && a.rows >= 1024;
  if (idle || (!rk && a.rows >= 1536)) {
    a.blocks = std::max(1, idle ? 512 / tiles : std::min(K / (tvw ? 768 : 384), 1024 / tiles));
    a.rows = ((K + a.blocks - 1) / a.blocks + 63) / 64 * 64;
    a.blocks = (K + a.rows - 1) / a.rows;
    grid.x = (unsigned)tiles * (unsigned)a.blocks;
  }
  // Few tiles with many columns each and few rows: their columns in shares.
  const int room = 256 / (tiles * a.blocks), wide = N / (tiles * 256);
  a.shares = std::max(1, std::min(room, wide));
  grid.x *= (unsigned)a.shares;
  // TVW, few groups of four rows for a workgroup's teams: a team per row, which reads its group and ranks itself (768 x 768
  // 25.2 us, a team per group 28.5; 4096 x 4096 78 and 68).
  const int groups = ((rows_per_tile + 3) / 4 + a.blocks - 1) / a.blocks, teams = 1024 >> (lg - 3);
  const int mode = !tvw ? MASKS_TW : 4 * groups <= teams ? MASKS_TVW_ROWS : MASKS_TVW_GROUPS;
#define TWG_MASKS(R_)                                                                                  \
  do {                                                                                                 \
    if (mode == MASKS_TW) TWG_LAUNCH((emit_masks<R_, MASKS_TW>), grid, block, a, lg);                  \
    else if (mode == MASKS_TVW_ROWS) TWG_LAUNCH((emit_masks<R_, MASKS_TVW_ROWS>), grid, block, a, lg); \
    else TWG_LAUNCH((emit_masks<R_, MASKS_TVW_GROUPS>), grid, block, a, lg);                           \
  } while (0)
  if (rk == 1) TWG_MASKS(1);
  else if (rk == 4) TWG_MASKS(4);
  else TWG_MASKS(0);
#undef TWG_MASKS
#undef TWG_ROWS
#undef TWG_LAUNCH
  return hipSuccess;
}

// ---- scratch for callers that cannot allocate -------------------------------------------
// One array per GPU, held until the process ends.  In host code its name is only a stand-in:
// the device address comes from hipGetSymbolAddress, once per device, and that pointer is what
// the kernels receive.
static __device__ __align__(256) unsigned char scratch[PRUNE_STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mutex;
void* scratch_ptr[MAX_DEVICES];     // per device: address of that device's copy of `scratch`
}  // namespace

hipError_t prune_static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    scratch_ptr[dev] = p;
  }
  *out = scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace twg
