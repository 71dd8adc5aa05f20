// Device-side packer: (B, mask[, tile mask]) in device memory -> packed handle, without moving
// the weight through the host.
//
// Paper: Section V condenses every B tile ahead of inference and replaces the tile masks by the
// indices of the unpruned rows / columns; Algorithm 3 condenses the kept columns before cutting
// tiles of G.  Here the same canonical form as the host packer's is produced by kernels:
//   structure  which columns keep anything, which rows keep anything in each tile of G kept
//              columns (one pass over the structure mask each), numbered in order into the
//              ascending index lists;
//   plan       only the kept-row counts (a few hundred bytes) visit the host, where padding,
//              offsets and the launch order of the tiles are laid out exactly as for a host-packed
//              weight and the image is allocated;
//   image      one kernel writes the padded lists, one the values in the register order of the
//              matrix instruction (TVW: with the 2:4 positions and the fill rule for short groups).
// The image is the only copy; the lists and values of the logical form are read back from it if
// somebody asks for them (tw_export, tw_unpack, tw_concat; tw_conv_bind: the lists).
//
// What bounds it: two waits for the stream (11 us each), then launches of a few microseconds; the
// masks (16 bytes per lane) and the weight are read once per pass.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "mk_band.h"
#include "packed.h"
#include "scan.h"

namespace twg {

namespace {

constexpr int T = 256;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// What the structure step leaves for the host: a fixed head, then K_t of every tile.
struct Counts {
  unsigned long long nnz;      // entries of the structure mask
  int32_t outside;             // an element is kept outside the tile mask
  int32_t three;               // a 2:4 group keeps more than two
  int32_t n_kept;
  int32_t nonfinite;           // an infinity or NaN among the weights
  int32_t k_union, pad;        // rows that some tile keeps
};

static __global__ void fill_zero(u32x4* p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = u32x4{0u, 0u, 0u, 0u};
}

// 16 mask bytes of row k from column n0 on, as 0x01 where non-zero (columns past N: 0).
template <bool VEC>
__device__ __forceinline__ u32x4 load_mask16(const uint8_t* S, int k, int n0, int N) {
  u32x4 v = {0u, 0u, 0u, 0u};
  const uint8_t* p = S + (size_t)k * N + n0;
  if constexpr (VEC) v = *(const u32x4*)p;
  else {
    const int cnt = min(16, N - n0);
    for (int c = 0; c < cnt; ++c) v[c >> 2] |= (uint32_t)p[c] << (8 * (c & 3));
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = (((v[j] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v[j]) >> 7 & 0x01010101u;
  return v;
}

// any[n] (bytes, zero on entry) = 1 if column n of the K x N byte mask S has a non-zero entry; 16
// columns per thread, rows 4 blockIdx.y + threadIdx.y, + 4 gridDim.y, .. (blockDim = 64 x 4)
template <bool VEC>
__global__ void column_any(const uint8_t* S, int K, int N, uint8_t* any) {
  __shared__ u32x4 part[4][64];
  const int n0 = (blockIdx.x * 64 + threadIdx.x) * 16;
  u32x4 a = {0u, 0u, 0u, 0u};
  if (n0 < N) {
    const int step = 4 * gridDim.y;
    for (int k0 = blockIdx.y * 4 + threadIdx.y; k0 < K; k0 += 4 * step) {
      u32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = load_mask16<VEC>(S, min(k0 + i * step, K - 1), n0, N);
      a |= (v[0] | v[1]) | (v[2] | v[3]);
    }
  }
  part[threadIdx.y][threadIdx.x] = a;
  __syncthreads();
  if (threadIdx.y || n0 >= N) return;
  a = (part[0][threadIdx.x] | part[1][threadIdx.x]) | (part[2][threadIdx.x] | part[3][threadIdx.x]);
#pragma unroll
  for (int j = 0; j < 4; ++j) {          // racing writers all store 1
    if (a[j] == 0x01010101u) ((uint32_t*)(any + n0))[j] = a[j];
    else
      for (int c = 0; c < 4; ++c) if (a[j] >> (8 * c) & 1u) any[n0 + 4 * j + c] = 1;
  }
}

// Columns in order: pos[n] = number among the kept or -1, kept[] and dropped[] the two lists.
__global__ __launch_bounds__(SCAN_T) void compact_columns(const uint8_t* any, int N, int32_t* pos, int32_t* kept,
                                                          int32_t* dropped, Counts* counts) {
  __shared__ int part[SCAN_WAVES];
  int base = 0;
  for (int n0 = 0; n0 < N; n0 += SCAN_T) {
    const int n = n0 + threadIdx.x;
    const bool v = n < N && any[n] != 0;
    int total;
    const int p = base + count_before(v, part, &total);
    if (n < N) {
      pos[n] = v ? p : -1;
      if (v) kept[p] = n;
      else dropped[n - p] = n;
    }
    base += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) counts->n_kept = base;
}

// An infinity or NaN among the 16 weights of row k from column n0 on whose mask bytes are set (columns past N:
// not set).
template <bool VEC>
__device__ __forceinline__ bool any_nonfinite(const uint16_t* B, int ldb, int vec_b, int k, int n0, int N, const u32x4& mask) {
  union { u32x4 v[2]; uint16_t e[16]; } x;
  const uint16_t* p = B + (size_t)k * ldb + n0;
  if (VEC && vec_b) { x.v[0] = *(const u32x4*)p; x.v[1] = *(const u32x4*)(p + 8); }
  else {
#pragma unroll
    for (int c = 0; c < 16; ++c) x.e[c] = p[min(c, N - 1 - n0)];
  }
  bool r = false;
#pragma unroll
  for (int c = 0; c < 16; ++c) r |= (x.e[c] & 0x7c00) == 0x7c00 && (mask[c >> 2] >> (8 * (c & 3)) & 1u);
  return r;
}

// row_any[t][k] (bytes, zero on entry) = 1 if row k has an entry among the columns of tile t; counts
// the entries of S, (element != null) notes an entry of `element` that S lacks and (B != null) an infinity
// or NaN among the weights of S.  16 columns per thread, which belong to two tiles at most.
template <bool VEC>
__global__ void tile_row_any(const uint8_t* S, const uint8_t* element, const uint16_t* B, int ldb, int vec_b, int K, int N, int lg,
                             const int32_t* col_pos, uint8_t* row_any, uint32_t* nnz_part, Counts* counts) {
  __shared__ int wave_sum[T / 64];
  const int n0 = (blockIdx.x * blockDim.x + threadIdx.x) * 16;
  int mine = 0;
  bool outside = false, nonfinite = false;
  if (n0 < N) {
    int tile = -1;                       // the first tile; the other is the next one
    u32x4 first = {0u, 0u, 0u, 0u};      // bytes of its columns
    i32x4 pos[4];
    if constexpr (VEC) {
#pragma unroll
      for (int j = 0; j < 4; ++j) pos[j] = *(const i32x4*)(col_pos + n0 + 4 * j);
    } else {
#pragma unroll
      for (int c = 0; c < 16; ++c) pos[c >> 2][c & 3] = n0 + c < N ? col_pos[n0 + c] : -1;
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const int p = pos[c >> 2][c & 3];
      if (p < 0) continue;
      if (tile < 0) tile = p >> lg;
      if (p >> lg == tile) first[c >> 2] |= 1u << (8 * (c & 3));
    }
    const int step = gridDim.y;
    for (int k0 = blockIdx.y; k0 < K; k0 += 4 * step) {
      u32x4 v[4], e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = min(k0 + i * step, K - 1);
        v[i] = load_mask16<VEC>(S, k, n0, N);
        if (element) e[i] = load_mask16<VEC>(element, k, n0, N);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = k0 + i * step;
        if (k >= K) break;
        const u32x4 a = v[i] & first, b = v[i] & ~first;
        mine += __popc(v[i][0]) + __popc(v[i][1]) + __popc(v[i][2]) + __popc(v[i][3]);
        if (a[0] | a[1] | a[2] | a[3]) row_any[(size_t)tile * K + k] = 1;
        if (b[0] | b[1] | b[2] | b[3]) row_any[(size_t)(tile + 1) * K + k] = 1;
        if (element) {
          const u32x4 o = e[i] & ~v[i];
          outside |= (o[0] | o[1] | o[2] | o[3]) != 0;
        }
        if (B) nonfinite |= any_nonfinite<VEC>(B, ldb, vec_b, k, n0, N, v[i]);
      }
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d);
  if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = mine;
  __syncthreads();
  if (threadIdx.x == 0) nnz_part[blockIdx.y * gridDim.x + blockIdx.x] = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
  if (outside) counts->outside = 1;      // racing writers all store 1
  if (nonfinite) counts->nonfinite = 1;
}

// Kept rows of tile blockIdx.x in order, and their number; the first workgroup adds up the entries, those past
// the n_lists tiles count the rows that some tile keeps, SCAN_T of them each.
__global__ __launch_bounds__(SCAN_T) void compact_rows(const uint8_t* row_any, int n_lists, int K, int32_t* row_list,
                                                       int32_t* k_t, const uint32_t* nnz_part, int n_part, Counts* counts) {
  __shared__ int part[SCAN_WAVES];
  if ((int)blockIdx.x >= n_lists) {
    const int k = ((int)blockIdx.x - n_lists) * SCAN_T + threadIdx.x;
    const uint8_t* any = row_any + min(k, K - 1);
    unsigned v = 0;
#pragma unroll 16
    for (int t = 0; t < n_lists; ++t) v |= any[(size_t)t * K];
    int total;
    count_before(k < K && v != 0, part, &total);
    if (threadIdx.x == 0) atomicAdd(&counts->k_union, total);
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    unsigned long long sum = 0;
    for (int i = threadIdx.x; i < n_part; i += 64) sum += nnz_part[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
    if (threadIdx.x == 0) counts->nnz = sum;
  }
  const uint8_t* any = row_any + (size_t)blockIdx.x * K;
  int32_t* list = row_list + (size_t)blockIdx.x * K;
  int base = 0;
  for (int k0 = 0; k0 < K; k0 += SCAN_T) {
    const int k = k0 + threadIdx.x;
    const bool v = k < K && any[k] != 0;
    int total;
    const int p = base + count_before(v, part, &total);
    if (v) list[p] = k;
    base += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) k_t[blockIdx.x] = base;
}

struct Structure {            // device pointers, filled by the kernels above
  const int32_t* kept;        // kept columns
  const int32_t* dropped;     // the others
  const int32_t* row_list;    // [t * K + j]
  const int32_t* k_t;         // kept rows per tile
  int K, n_kept, n_zero, n_tiles;
};

// The padded lists of the image: tile blockIdx.y's kept rows (pads repeat the last one) and
// columns (-1 past the last); blockIdx.y == n_tiles: the slack behind the row lists, the pruned columns.
__global__ void image_lists(Structure st, int G, const int32_t* tile_kp_off, int32_t* row_idx, int32_t* col_idx,
                            int32_t* zero_cols) {
  const int t = blockIdx.y, i = blockIdx.x * blockDim.x + threadIdx.x;
  const int kp0 = tile_kp_off[t];
  if (t == st.n_tiles) {
    if (i < ROW_IDX_SLACK) row_idx[kp0 + i] = 0;
    if (i < st.n_zero) zero_cols[i] = st.dropped[i];
    return;
  }
  const int kt = st.k_t[t];
  if (i < tile_kp_off[t + 1] - kp0) row_idx[kp0 + i] = kt ? st.row_list[(size_t)t * st.K + min(i, kt - 1)] : 0;
  if (i < G) col_idx[t * G + i] = t * G + i < st.n_kept ? st.kept[t * G + i] : -1;
}

// TW values (layout: see the host packer's build_device_values): 8 rows of a column per thread, one
// 16-byte store; blockIdx.y == n_tiles: the slack behind the last tile.
__global__ void image_tw(const uint16_t* B, int ldb, Structure st, int G, const int32_t* tile_kp_off, uint16_t* vals) {
  const int t = blockIdx.y, i = blockIdx.x * blockDim.x + threadIdx.x;
  const int kp0 = tile_kp_off[t];
  u32x4* out = (u32x4*)(vals + (size_t)kp0 * G);
  if (t == st.n_tiles) {
    if (i < KSTEP_TW * G / 8) out[i] = u32x4{0u, 0u, 0u, 0u};
    return;
  }
  const int kp = tile_kp_off[t + 1] - kp0;
  if (i >= kp / 8 * G) return;
  const int j0 = i / G * 8, c = i - j0 / 8 * G;
  const int kt = st.k_t[t];
  const int32_t* rows = st.row_list + (size_t)t * st.K;
  union { uint16_t e[8]; u32x4 v; } x;
  x.v = u32x4{0u, 0u, 0u, 0u};
  if (t * G + c < st.n_kept && j0 < kt) {
    const int n = st.kept[t * G + c];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint16_t v = B[(size_t)rows[min(j0 + j, kt - 1)] * ldb + n];
      x.e[j] = j0 + j < kt ? v : (uint16_t)0;
    }
  }
  out[j0 / 16 * (2 * G) + (c / 32) * 64 + ((j0 % 16) / 8) * 32 + c % 32] = x.v;
}

// TVW values and position words (layout: see the host packer's build_device_values): one thread per
// (tile, 64-row stage, half, column block, lane), i.e. four groups of 4 condensed rows of a column.
// A group stores the two lowest positions that are kept, topped up with the lowest that are not (+0
// fillers); `valid`: 2 bits per group, which of the two are kept elements.
__global__ void image_tvw(const uint16_t* B, int ldb, const uint8_t* mask, int N, Structure st, int G,
                          const int32_t* tile_kp_off, uint16_t* vals, uint16_t* meta, uint8_t* valid, Counts* counts) {
  const int t = blockIdx.y, i = blockIdx.x * blockDim.x + threadIdx.x;
  const int kp0 = tile_kp_off[t], kp = tile_kp_off[t + 1] - kp0;
  if (i >= kp / 32 * G * 2) return;                    // (kp / 64 stages) x 2 halves x (G / 32) blocks x 64 lanes
  const int nbt = G / 32;
  const int l = i & 63, nb = (i >> 6) % nbt, su = (i >> 6) / nbt;
  const int kt = st.k_t[t], c = 32 * nb + l % 32;
  const bool live = t * G + c < st.n_kept;
  const int n = st.kept[live ? t * G + c : 0];
  const int32_t* rows = st.row_list + (size_t)t * st.K;
  union { uint16_t e[8]; u32x4 v; } x;
  x.v = u32x4{0u, 0u, 0u, 0u};
  uint32_t word = 0, vbits = 0;
  bool three = false;
  const int j0 = 32 * su + 16 * (l / 32);              // the thread's 16 condensed rows
  uint16_t val[16];
  uint8_t kept[16];
#pragma unroll
  for (int p = 0; p < 16; ++p) {                       // all loads first
    const int row = kt > 0 ? rows[min(j0 + p, kt - 1)] : 0;
    val[p] = B[(size_t)row * ldb + n];
    kept[p] = mask[(size_t)row * N + n];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int g = 8 * su + 4 * (l / 32) + j;           // group of 4 condensed rows
    uint32_t pos = 0x4;                                // positions (0, 1)
    if (live && 4 * g < kt) {
      const uint16_t* v = val + 4 * j;
      int set = 0;
#pragma unroll
      for (int p = 0; p < 4; ++p) set |= 4 * g + p < kt && kept[4 * j + p] != 0 ? 1 << p : 0;
      three |= __popc(set) > 2;
      int chosen = set;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if (__popc(chosen) < 2) chosen |= 1 << p;
      const int p0 = __ffs(chosen) - 1, p1 = __ffs(chosen & (chosen - 1)) - 1;
      pos = (uint32_t)(p0 | p1 << 2);
      uint16_t a = 0, b = 0;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        if (p == p0 && (set >> p & 1)) a = v[p];
        if (p == p1 && (set >> p & 1)) b = v[p];
      }
      x.e[2 * j] = a;
      x.e[2 * j + 1] = b;
      vbits |= (uint32_t)((set >> p0 & 1) | (set >> p1 & 1) << 1) << (2 * j);
    }
    word |= pos << (4 * j);
  }
  if (three) counts->three = 1;                        // racing writers all store 1
  ((u32x4*)(vals + (size_t)kp0 / 2 * G))[i] = x.v;
  // position words: [stage][block][lane], 16 bits per half
  const size_t w = ((size_t)kp0 / 64 + su / 2) * nbt * 64 + nb * 64 + l;
  meta[2 * w + (su & 1)] = (uint16_t)word;
  valid[2 * w + (su & 1)] = (uint8_t)vbits;
}

struct DevBuf {               // device allocation freed on scope exit
  void* p = nullptr;
  ~DevBuf() { if (p) (void)hipFree(p); }
  hipError_t alloc(size_t n) { return hipMalloc(&p, n ? n : 1); }
};

size_t up(size_t x) { return (x + 255) / 256 * 256; }

#define TWG_TRY(expr) do { if ((expr) != hipSuccess) { (void)hipGetLastError(); return TW_ERR_HIP; } } while (0)
#define TWG_LAUNCH(kernel, grid, block, ...)                                  \
  do {                                                                        \
    hipLaunchKernelGGL(kernel, grid, block, 0, s, __VA_ARGS__);               \
    if (hipGetLastError() != hipSuccess) return TW_ERR_HIP;                   \
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
  const bool vec = N % 16 == 0 && ((uintptr_t)mask & 15) == 0 && ((uintptr_t)tile_mask & 15) == 0;
  (void)hipGetLastError();

  // ---- structure: kept columns, kept rows per tile --------------------------------------
  std::vector<char> tables;              // (copied asynchronously: outlives the workspace, whose release waits for the device)
  DevBuf ws;
  const size_t o_kt = up(sizeof(Counts)), o_any = o_kt + up(ntmax * 4), o_rany = o_any + up((size_t)N + 16);
  const size_t zeroed = o_rany + up(ntmax * K), o_pos = zeroed, o_kept = o_pos + up((size_t)N * 4);
  const size_t o_drop = o_kept + up((size_t)N * 4), o_list = o_drop + up((size_t)N * 4), o_nnz = o_list + up(ntmax * K * 4);
  const unsigned nx = (unsigned)((N + 16 * T - 1) / (16 * T)), ny = (unsigned)std::min(K, 256);
  const size_t ws_bytes = o_nnz + (size_t)nx * ny * 4;
  if (ws.alloc(ws_bytes) != hipSuccess) { (void)hipGetLastError(); return TW_ERR_ALLOC; }
  char* w = (char*)ws.p;
  Counts* counts = (Counts*)w;
  int32_t* k_t = (int32_t*)(w + o_kt);
  uint8_t *col_any = (uint8_t*)w + o_any, *row_any = (uint8_t*)w + o_rany;
  int32_t *col_pos = (int32_t*)(w + o_pos), *kept = (int32_t*)(w + o_kept), *dropped = (int32_t*)(w + o_drop);
  int32_t* row_list = (int32_t*)(w + o_list);
  uint32_t* nnz_part = (uint32_t*)(w + o_nnz);
  // (a kernel of this library clears the counters: the runtime's fill costs the host three times a launch)
  TWG_LAUNCH(fill_zero, dim3((unsigned)((zeroed / 16 + T - 1) / T)), dim3(T), (u32x4*)w, zeroed / 16);
  const dim3 any_grid((unsigned)((N + 1023) / 1024), (unsigned)std::min((K + 3) / 4, 64));
  if (vec) TWG_LAUNCH(column_any<true>, any_grid, dim3(64, 4), S, K, N, col_any);
  else TWG_LAUNCH(column_any<false>, any_grid, dim3(64, 4), S, K, N, col_any);
  TWG_LAUNCH(compact_columns, dim3(1), dim3(SCAN_T), col_any, N, col_pos, kept, dropped, counts);
  const uint8_t* element = tvw && tile_mask ? mask : nullptr;
  // only the row-major kernel asks whether all weights are finite, of TW weights and where K takes several bands
  const uint16_t* finite = !tvw && K > MK_KC ? B : nullptr;
  const int vec_b = ldb % 8 == 0 && ((uintptr_t)B & 15) == 0;
  if (vec) TWG_LAUNCH(tile_row_any<true>, dim3(nx, ny), dim3(T), S, element, finite, ldb, vec_b, K, N, lg, col_pos, row_any, nnz_part, counts);
  else TWG_LAUNCH(tile_row_any<false>, dim3(nx, ny), dim3(T), S, element, finite, ldb, vec_b, K, N, lg, col_pos, row_any, nnz_part, counts);
  TWG_LAUNCH(compact_rows, dim3((unsigned)(ntmax + (K + SCAN_T - 1) / SCAN_T)), dim3(SCAN_T), row_any, (int)ntmax, K, row_list,
             k_t, nnz_part, (int)(nx * ny), counts);

  // ---- plan: the counts visit the host ----------------------------------------------------
  std::vector<char> head(o_kt + ntmax * 4);
  TWG_TRY(hipMemcpyWithStream(head.data(), w, head.size(), hipMemcpyDeviceToHost, s));
  const Counts& c = *(const Counts*)head.data();
  const int32_t* kt_h = (const int32_t*)(head.data() + o_kt);
  if (c.outside) return TW_ERR_MASK;
  h->n_kept = c.n_kept;
  const int n_tiles = h->n_tiles = (c.n_kept + G - 1) / G;
  h->tile_k_off.assign(n_tiles + 1, 0);
  h->tile_col_off.resize(n_tiles + 1);
  h->sum_kw = 0;
  for (int t = 0; t <= n_tiles; ++t) h->tile_col_off[t] = std::min(t * G, h->n_kept);
  for (int t = 0; t < n_tiles; ++t) {
    h->tile_k_off[t + 1] = h->tile_k_off[t] + kt_h[t];
    h->sum_kw += (int64_t)kt_h[t] * (h->tile_col_off[t + 1] - h->tile_col_off[t]);
  }
  h->sum_k = h->tile_k_off[n_tiles];
  h->k_union = c.k_union;
  h->nonfinite = c.nonfinite != 0;
  if (!tvw || tile_mask) {               // tile-wise: the structure mask is the union of its tiles' rows x columns
    if ((int64_t)c.nnz != h->sum_kw) return TW_ERR_MASK;
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

  // ---- image: the host's tables, then the lists and values --------------------------------------
  tables.resize(L.off[IMG_COL_IDX]);
  std::copy_n((const char*)d.tile_kp_off.data(), L.bytes[IMG_TILE_KP_OFF], tables.data() + L.off[IMG_TILE_KP_OFF]);
  std::copy_n((const char*)d.tile_order.data(), L.bytes[IMG_TILE_ORDER], tables.data() + L.off[IMG_TILE_ORDER]);
  std::copy_n((const char*)d.tile_sched.data(), L.bytes[IMG_TILE_SCHED], tables.data() + L.off[IMG_TILE_SCHED]);
  TWG_TRY(hipMemcpyAsync(blob, tables.data(), tables.size(), hipMemcpyHostToDevice, s));
  const Structure st{kept, dropped, row_list, k_t, K, h->n_kept, d.n_zero, n_tiles};
  const int longest = std::max({h->max_kp, G, ROW_IDX_SLACK, d.n_zero});
  TWG_LAUNCH(image_lists, dim3((longest + T - 1) / T, n_tiles + 1), dim3(T), st, G, d.d_tile_kp_off, (int32_t*)d.d_row_idx,
             (int32_t*)d.d_col_idx, (int32_t*)d.d_zero_cols);
  if (!tvw) {
    const int most = std::max(h->max_kp / 8 * G, KSTEP_TW * G / 8);
    TWG_LAUNCH(image_tw, dim3((most + T - 1) / T, n_tiles + 1), dim3(T), B, ldb, st, G, d.d_tile_kp_off, (uint16_t*)d.d_vals);
    TWG_TRY(hipStreamSynchronize(s));    // the workspace goes away when this returns
    return TW_OK;
  }
  if (n_tiles > 0 && h->max_kp > 0)
    TWG_LAUNCH(image_tvw, dim3((h->max_kp / 32 * G * 2 + T - 1) / T, n_tiles), dim3(T), B, ldb, mask, N, st, G,
               d.d_tile_kp_off, (uint16_t*)d.d_vals, (uint16_t*)d.d_meta, (uint8_t*)d.d_valid, counts);
  Counts after;
  TWG_TRY(hipMemcpyWithStream(&after, counts, sizeof after, hipMemcpyDeviceToHost, s));
  return after.three ? TW_ERR_MASK : TW_OK;
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
