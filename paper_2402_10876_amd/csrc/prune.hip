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
// What bounds it: seven launches (TVW) one after the other on a weight of a few MB, each of them a
// few dependent trips to memory.  1024 x 4096 at 87.5 % (TVW): 41 us of kernels, against 130 with
// ranks by counting every pair, one thread per mask byte and 128-bit sums throughout.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "prune.h"
#include "scan.h"

namespace twg {

namespace {

typedef unsigned __int128 u128;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint64_t magnitude24(uint16_t h) {   // |value| in units of 2^-24
  const uint32_t e = (h >> 10) & 31u, m = h & 1023u;
  return e == 0 ? (uint64_t)m : (uint64_t)(m | 1024u) << (e - 1);
}

// Sum of squares.  Values below 1 have squares below 2^48: 2^15 of them fit a 64-bit sum, which
// takes one multiply-add each; larger values go to a 128-bit sum of their own.
struct Sum {
  uint64_t lo = 0;
  u128 hi = 0;
  __device__ __forceinline__ void add(uint16_t h) {
    const uint64_t a = magnitude24(h);
    if (a < (1u << 24)) lo += (uint64_t)(uint32_t)a * (uint32_t)a;
    else hi += (u128)a * (u128)a;
  }
  __device__ __forceinline__ void carry() { hi += lo; lo = 0; }
  __device__ __forceinline__ u128 total() const { return hi + lo; }
};

// TW-C scores in two steps, exact and independent of any order (integer sums).  A workgroup takes
// 256 columns and the rows 4 y + sub, + 4 gridDim.y, .. : 64 lanes of 4 columns x 4 rows; the four
// rows' sums meet in LDS and the slice's sum goes to partial[y][column].
__global__ void column_partial(const uint16_t* B, int K, int N, int ldb, int vec, u128* partial) {
  __shared__ u128 part[4][256];
  const int lane = threadIdx.x & 63, sub = threadIdx.x >> 6;
  const int n = blockIdx.x * 256 + lane * 4;
  Sum s[4];
  int rows = 0;
  const int step = 4 * gridDim.y;
  for (int k0 = blockIdx.y * 4 + sub; k0 < K; k0 += 8 * step) {
    union { uint2 v; uint16_t e[4]; } x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[i].v = uint2{0u, 0u};
      const int k = k0 + i * step;
      if (k >= K) continue;
      const uint16_t* p = B + (size_t)k * ldb + n;
      if (vec && n + 4 <= N) x[i].v = *(const uint2*)p;
      else
        for (int c = 0; c < 4; ++c) if (n + c < N) x[i].e[c] = p[c];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) s[c].add(x[i].e[c]);
    if ((rows += 8) >= (1 << 15)) {
      rows = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) s[c].carry();
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) part[sub][lane * 4 + c] = s[c].total();
  __syncthreads();
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col < N)
    partial[(size_t)blockIdx.y * N + col] =
        (part[0][threadIdx.x] + part[1][threadIdx.x]) + (part[2][threadIdx.x] + part[3][threadIdx.x]);
}
__global__ void column_score_finish(const u128* partial, int slices, int N, u128* score) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  u128 s = 0;
#pragma unroll 8
  for (int y = 0; y < slices; ++y) s += partial[(size_t)y * N + n];
  score[n] = s;
}

// Which entries of a segment are kept: all but the n_pruned lowest in (score, index) order.  One
// workgroup of SCAN_T threads per segment (blockIdx.x); R > 0: the segment has at most R * SCAN_T
// entries and they stay in registers, R = 0: any length, read again in every pass.
//   1. the bits that all scores share at the top are skipped (OR of the differences to entry 0);
//   2. the threshold is found 8 bits at a time from histograms in LDS; it is settled as soon as all
//      scores with its leading bits are pruned, usually after two or three digits;
//   3. scores equal to a threshold that had to be followed to its last bit are pruned in index
//      order, and the kept entries are numbered in order:
//      pos[i] = number among the kept or -1, list[pos] = i (each may be null).
template <int R>
__global__ __launch_bounds__(SCAN_T) void select_kept(const u128* scores, int len, int n_pruned, int32_t* pos, int32_t* list) {
  __shared__ int hist[256], part[2][SCAN_WAVES];
  __shared__ unsigned long long diff_w[2 * SCAN_WAVES];
  __shared__ int found[3];                     // bin, entries in it, entries in front of it
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const u128* s = scores + (size_t)blockIdx.x * len;
  if (pos) pos += (size_t)blockIdx.x * len;
  if (list) list += (size_t)blockIdx.x * len;
  const int rounds = (len + SCAN_T - 1) / SCAN_T;
  u128 key[R > 0 ? R : 1];
  if constexpr (R > 0) {
#pragma unroll
    for (int r = 0; r < R; ++r) key[r] = r * SCAN_T + tid < len ? s[r * SCAN_T + tid] : 0;
  }
  auto each = [&](auto f) {                    // f(score, index) for this thread's entries, in order
    if constexpr (R > 0) {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r < rounds) f(key[r], r * SCAN_T + tid);
    } else {
      for (int r = 0; r < rounds; ++r) {
        const int i = r * SCAN_T + tid;
        f(i < len ? s[i] : (u128)0, i);
      }
    }
  };
  u128 prefix = 0;
  int shift = 0, need = n_pruned;              // scores whose bits above `shift` equal `prefix`: the lowest `need` go
  bool all_equal_go = true;
  if (n_pruned > 0 && n_pruned < len) {
    const u128 first = s[0];
    unsigned long long d0 = 0, d1 = 0;
    each([&](u128 v, int i) {
      if (i < len) { const u128 d = v ^ first; d0 |= (unsigned long long)d; d1 |= (unsigned long long)(d >> 64); }
    });
#pragma unroll
    for (int k = 32; k >= 1; k >>= 1) { d0 |= __shfl_xor(d0, k); d1 |= __shfl_xor(d1, k); }
    if (lane == 0) { diff_w[wave] = d0; diff_w[SCAN_WAVES + wave] = d1; }
    __syncthreads();
    d0 = d1 = 0;
#pragma unroll
    for (int w = 0; w < SCAN_WAVES; ++w) { d0 |= diff_w[w]; d1 |= diff_w[SCAN_WAVES + w]; }
    shift = d1 ? 128 - __clzll((long long)d1) : d0 ? 64 - __clzll((long long)d0) : 0;
    prefix = shift < 128 ? first >> shift : 0;
    all_equal_go = false;
    while (shift > 0) {
      const int bits = shift < 8 ? shift : 8, low = shift - bits;
      for (int i = tid; i < 256; i += SCAN_T) hist[i] = 0;
      __syncthreads();
      each([&](u128 v, int i) {
        if (i < len && (shift >= 128 || v >> shift == prefix)) atomicAdd(&hist[(int)(v >> low) & ((1 << bits) - 1)], 1);
      });
      __syncthreads();
      if (wave == 0) {                         // four bins per lane: the bin that holds entry number `need`
        int n[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { n[j] = hist[lane * 4 + j]; sum += n[j]; }
        int before = sum;
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) { const int t = __shfl_up(before, k); before += lane >= k ? t : 0; }
        before -= sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (before < need && need <= before + n[j]) { found[0] = lane * 4 + j; found[1] = n[j]; found[2] = before; }
          before += n[j];
        }
      }
      __syncthreads();
      prefix = prefix << bits | (unsigned)found[0];
      need -= found[2];
      shift = low;
      if (found[1] == need) { all_equal_go = true; break; }
    }
  }
  int n_equal = 0, n_kept = 0;                 // entries equal to the threshold / kept, in the rounds before
  each([&](u128 v, int i) {
    bool keep = i < len && n_pruned < len;
    if (n_pruned > 0 && n_pruned < len) {      // (uniform over the workgroup)
      const u128 top = v >> shift;
      const bool equal = i < len && top == prefix;
      if (all_equal_go) keep = i < len && top > prefix;
      else {
        int total;
        const int at = n_equal + count_before(equal, part[0], &total);
        n_equal += total;
        keep = i < len && (top > prefix || (equal && at >= need));
      }
    }
    int total;
    const int p = n_kept + count_before(keep, part[1], &total);
    n_kept += total;
    if (i < len) {
      if (pos) pos[i] = keep ? p : -1;
      if (list && keep) list[p] = i;
    }
    __syncthreads();                           // `part` may be used again
  });
}

// TW-R scores: tile t = kept columns [t*G, min((t+1)*G, n_kept)); 16 lanes per (tile, row), their
// columns 16 apart; the lanes' sums meet in 64 bits, unless a value of 1 or more was among them.
template <int G>
__global__ void tile_row_scores(const uint16_t* B, int K, int ldb, int n_kept, const int32_t* kept_cols, u128* score) {
  const int t = blockIdx.y, l = threadIdx.x & 15;
  const int k = blockIdx.x * (blockDim.x >> 4) + (threadIdx.x >> 4);
  const int w = min(G, n_kept - t * G);
  Sum s;
  if (k < K) {
    const uint16_t* row = B + (size_t)k * ldb;
    const int32_t* cols = kept_cols + t * G;
    uint16_t v[G / 16];
#pragma unroll
    for (int i = 0; i < G / 16; ++i) v[i] = l + 16 * i < w ? row[cols[l + 16 * i]] : 0;
#pragma unroll
    for (int i = 0; i < G / 16; ++i) s.add(v[i]);
  }
  unsigned long long lo = s.lo;
#pragma unroll
  for (int d = 8; d >= 1; d >>= 1) lo += __shfl_xor(lo, d);
  u128 total = lo;
  if (__any(s.hi != 0)) {                      // three 32-bit limbs, each in a 64-bit word
    unsigned long long h0 = (uint32_t)s.hi, h1 = (uint32_t)(s.hi >> 32), h2 = (unsigned long long)(s.hi >> 64);
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) {
      h0 += __shfl_xor(h0, d);
      h1 += __shfl_xor(h1, d);
      h2 += __shfl_xor(h2, d);
    }
    total += (u128)h0 + ((u128)h1 << 32) + ((u128)h2 << 64);
  }
  if (k < K && l == 0) score[(size_t)t * K + k] = total;
}

// out[k][n] = column n kept and row k kept in n's tile, into `a` and `b`; `zeroed` (TVW) starts as
// zeros (each may be null).  A thread writes 16 columns, which belong to two tiles at most, of
// EMIT_ROWS rows (VEC: 16-byte stores).
constexpr int EMIT_ROWS = 4;
template <bool VEC>
__global__ void emit_tile_mask(int K, int N, int lg, int nt, const int32_t* col_pos, const int32_t* row_pos, uint8_t* a,
                               uint8_t* b, uint8_t* zeroed) {
  const int n0 = (blockIdx.y * blockDim.x + threadIdx.x) * 16;
  const int k0 = blockIdx.x * EMIT_ROWS;
  if (n0 >= N) return;
  const int cnt = VEC ? 16 : min(16, N - n0);
  int tile = -1;                               // the first tile; the other is the next one
  u32x4_t first = {0u, 0u, 0u, 0u}, second = first;                  // bytes of their columns
  if (a) {
    i32x4_t pos[4];
    if constexpr (VEC) {
#pragma unroll
      for (int j = 0; j < 4; ++j) pos[j] = *(const i32x4_t*)(col_pos + n0 + 4 * j);
    } else {
#pragma unroll
      for (int c = 0; c < 16; ++c) pos[c >> 2][c & 3] = c < cnt ? col_pos[n0 + c] : -1;
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const int p = pos[c >> 2][c & 3];
      if (p < 0) continue;
      if (tile < 0) tile = p >> lg;
      if (p >> lg == tile) first[c >> 2] |= 1u << (8 * (c & 3));
      else second[c >> 2] |= 1u << (8 * (c & 3));
    }
  }
  const int t0 = max(tile, 0), t1 = min(t0 + 1, max(nt - 1, 0));
  bool keep0[EMIT_ROWS], keep1[EMIT_ROWS];
#pragma unroll
  for (int r = 0; r < EMIT_ROWS; ++r) {
    const int k = min(k0 + r, K - 1);
    keep0[r] = tile >= 0 && row_pos[(size_t)t0 * K + k] >= 0;
    keep1[r] = tile >= 0 && row_pos[(size_t)t1 * K + k] >= 0;
  }
#pragma unroll
  for (int r = 0; r < EMIT_ROWS; ++r) {
    if (k0 + r >= K) break;
    union { u32x4_t v; uint8_t e[16]; } x;
    const u32x4_t none = {0u, 0u, 0u, 0u};
    x.v = (keep0[r] ? first : none) | (keep1[r] ? second : none);
    const size_t at = (size_t)(k0 + r) * N + n0;
    if constexpr (VEC) {
      if (a) *(u32x4_t*)(a + at) = x.v;
      if (b) *(u32x4_t*)(b + at) = x.v;
      if (zeroed) *(u32x4_t*)(zeroed + at) = none;
    } else {
      for (int c = 0; c < cnt; ++c) {
        if (a) a[at + c] = x.e[c];
        if (b) b[at + c] = x.e[c];
        if (zeroed) zeroed[at + c] = 0;
      }
    }
  }
}

// 2:4 along the condensed kept rows of a tile: in every group of 4 consecutive kept rows
// and every column keep the 2 largest |w|; equal magnitudes: the lower position stays.
// Workgroup: 256 / G groups of a tile, G columns each.
__global__ void two_of_four(const uint16_t* B, int K, int N, int ldb, int lg, int n_kept, int rows_kept,
                            const int32_t* kept_cols, const int32_t* row_list, uint8_t* mask) {
  const int t = blockIdx.y, c = (t << lg) + (int)(threadIdx.x & ((1u << lg) - 1u));
  const int g = blockIdx.x * (blockDim.x >> lg) + (threadIdx.x >> lg);
  if (c >= n_kept || 4 * g >= rows_kept) return;
  const int n = kept_cols[c];
  const int32_t* rows = row_list + (size_t)t * K + 4 * g;
  const int cnt = min(4, rows_kept - 4 * g);
  int row[4];
  uint16_t v[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) row[p] = rows[p < cnt ? p : 0];
#pragma unroll
  for (int p = 0; p < 4; ++p) v[p] = B[(size_t)row[p] * ldb + n] & 0x7fffu;   // magnitude order of finite fp16
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    int larger = 0;     // positions that come first: larger magnitude, or equal and lower
#pragma unroll
    for (int q = 0; q < 4; ++q) larger += q != p && q < cnt && (v[q] > v[p] || (v[q] == v[p] && q < p));
    if (p < cnt && larger < 2) mask[(size_t)row[p] * N + n] = 1;
  }
}

size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

// Row slices of the column scores: about 512 workgroups of 256 columns in all, so at most
// 2 MiB of partial sums whatever the shape.
static int column_slices(int K, int N) {
  const int nbx = (N + 255) / 256;
  const int want = 512 / nbx > 1 ? 512 / nbx : 1;
  return K < want ? K : want;
}

size_t prune_workspace_bytes(int K, int N, int G) {
  const size_t nt = (size_t)(N + G - 1) / G;
  // (one spare list per column and per row: the size is part of the interface)
  return align_up((size_t)N * 16) + 3 * align_up((size_t)N * 4) +          // column score, pos, list
         align_up(nt * K * 16) + 3 * align_up(nt * K * 4) +                 // row score, pos, list
         align_up((size_t)column_slices(K, N) * N * 16);                    // column scores per row slice
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
  u128* col_partial = (u128*)w;
  const int T = 256, lg = G == 128 ? 7 : G == 64 ? 6 : 5;
  auto aligned = [](const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; };
  (void)hipGetLastError();   // an error left behind by an earlier call of this thread is not this call's
  // a failed launch ends the call: later kernels would read workspace nobody wrote
#define TWG_LAUNCH(kernel, grid, block, ...)                                  \
  do {                                                                        \
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);          \
    const hipError_t e_ = hipGetLastError();                                  \
    if (e_ != hipSuccess) return e_;                                          \
  } while (0)
#define TWG_SELECT(segments, scores, len, n_pruned, pos, list)                                               \
  do {                                                                                                       \
    if ((len) <= SCAN_T) TWG_LAUNCH(select_kept<1>, dim3(segments), dim3(SCAN_T), scores, len, n_pruned, pos, list);           \
    else if ((len) <= 4 * SCAN_T) TWG_LAUNCH(select_kept<4>, dim3(segments), dim3(SCAN_T), scores, len, n_pruned, pos, list);  \
    else TWG_LAUNCH(select_kept<0>, dim3(segments), dim3(SCAN_T), scores, len, n_pruned, pos, list);         \
  } while (0)
  const int ky = column_slices(K, N);
  TWG_LAUNCH(column_partial, dim3((unsigned)((N + T - 1) / T), ky), dim3(T), B, K, N, ldb,
             (int)(ldb % 4 == 0 && aligned(B, 8)), col_partial);
  TWG_LAUNCH(column_score_finish, dim3((unsigned)((N + 63) / 64)), dim3(64), col_partial, ky, N, col_score);
  TWG_SELECT(1, col_score, N, n_cols_pruned, col_pos, kept_cols);
  if (nt > 0) {
    const dim3 grid((K + 15) / 16, nt);
    if (G == 128) TWG_LAUNCH(tile_row_scores<128>, grid, dim3(T), B, K, ldb, n_kept, kept_cols, row_score);
    else if (G == 64) TWG_LAUNCH(tile_row_scores<64>, grid, dim3(T), B, K, ldb, n_kept, kept_cols, row_score);
    else TWG_LAUNCH(tile_row_scores<32>, grid, dim3(T), B, K, ldb, n_kept, kept_cols, row_score);
    TWG_SELECT(nt, row_score, K, K - rows_per_tile, row_pos, row_list);
  }
  // TVW: the tile mask (if asked for) and an all-zero element mask for the 2:4 step to fill; TW: the
  // element mask is the tile mask
  const bool vec = N % 16 == 0 && aligned(mask, 16) && (!tile_mask || aligned(tile_mask, 16));
  const unsigned ex = (unsigned)((N + 16 * T - 1) / (16 * T)), ey = (unsigned)((K + EMIT_ROWS - 1) / EMIT_ROWS);
  uint8_t *out_a = tvw ? tile_mask : mask, *out_b = tvw ? nullptr : tile_mask, *zeroed = tvw ? mask : nullptr;
  if (vec) TWG_LAUNCH(emit_tile_mask<true>, dim3(ey, ex), dim3(T), K, N, lg, nt, col_pos, row_pos, out_a, out_b, zeroed);
  else TWG_LAUNCH(emit_tile_mask<false>, dim3(ey, ex), dim3(T), K, N, lg, nt, col_pos, row_pos, out_a, out_b, zeroed);
  if (tvw && nt > 0 && rows_per_tile > 0) {
    const int groups = (rows_per_tile + 3) / 4, per = T >> lg;
    TWG_LAUNCH(two_of_four, dim3((groups + per - 1) / per, nt), dim3(T), B, K, N, ldb, lg, n_kept, rows_per_tile,
               kept_cols, row_list, mask);
  }
#undef TWG_SELECT
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
