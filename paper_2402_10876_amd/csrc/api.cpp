// C ABI of the library (see include/twgemm.h): argument checks, upload of the
// packed image, kernel selection.  No torch types, no exceptions across.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstring>
#include <new>
#include <vector>

#include "kernels.h"
#include "packed.h"
#include "prune.h"

namespace {

std::atomic<int> opt_tile_m{0};
std::atomic<int> opt_xcd_map{1};
std::atomic<int> opt_kernel{0};   // 0 = automatic, 1 = register-staged, 2 = asynchronous copies
std::atomic<int> opt_depth{3};
std::atomic<int> opt_waves{4};
std::atomic<int> opt_ksplit{0};   // 0 = automatic, 1 = off, 2 = two K groups per workgroup
std::atomic<int> opt_wg_split{0}; // 0 / 1 = off, 2..8 = workgroups per tile (needs a workspace)
std::atomic<int> opt_tiles_per_wg{0};  // 0 = automatic, 1..8 = tiles a workgroup computes one after the other
std::atomic<int> opt_idx_route{0};// kept-row lists: 0 = automatic, 1 = scalar loads, 2 = vector loads

// What one launch runs with: the caller's tw_launch_opts, or the process defaults above
// (tw_set_option) when there is none.  Read once per call, never shared between calls.
struct Opts {
  int tile_m, xcd_map, kernel, depth, waves, ksplit, wg_split, idx_route, tiles_per_wg;
  void* ws;
  size_t ws_bytes;
};
Opts default_opts() {
  return Opts{opt_tile_m.load(), opt_xcd_map.load(), opt_kernel.load(), opt_depth.load(), opt_waves.load(),
              opt_ksplit.load(), opt_wg_split.load(), opt_idx_route.load(), opt_tiles_per_wg.load(), nullptr, 0};
}
bool opts_from(const tw_launch_opts* in, Opts* o) {
  *o = default_opts();
  if (!in) return true;
  if (in->tile_m != 0 && in->tile_m != 64 && in->tile_m != 128 && in->tile_m != 256) return false;
  if (in->kernel < 0 || in->kernel > 2 || in->ksplit < 0 || in->ksplit > 2) return false;
  if (in->depth != 0 && (in->depth < 3 || in->depth > 8)) return false;
  if (in->waves != 0 && in->waves != 4 && in->waves != 8) return false;
  if (in->xcd_map < -1 || in->xcd_map > 2 || in->wg_split < 0 || in->wg_split > 8) return false;
  if (in->idx_route < 0 || in->idx_route > 2) return false;
  if (in->tiles_per_wg < 0 || in->tiles_per_wg > 8) return false;
  if (in->workspace_dev && ((uintptr_t)in->workspace_dev & 255)) return false;
  o->tile_m = in->tile_m; o->kernel = in->kernel; o->ksplit = in->ksplit; o->wg_split = in->wg_split;
  o->idx_route = in->idx_route;
  o->tiles_per_wg = in->tiles_per_wg;
  o->depth = in->depth ? in->depth : 3;
  o->waves = in->waves ? in->waves : 4;
  o->xcd_map = in->xcd_map < 0 ? 1 : in->xcd_map;
  o->ws = in->workspace_dev; o->ws_bytes = in->workspace_dev ? in->workspace_bytes : 0;
  return true;
}

// Nothing was asked for: the library chooses the kernel and its shape.
bool automatic(const Opts& o) {
  return o.tile_m == 0 && o.kernel == 0 && o.depth == 3 && o.waves == 4 && o.ksplit == 0 && o.wg_split < 2 &&
         o.idx_route == 0 && o.tiles_per_wg < 2 && o.xcd_map == 1;
}

// Workspace of the K split across workgroups: 1024 counters, then the fp32 partial tiles.
constexpr size_t WS_COUNTER_BYTES = 4096;
constexpr int WS_MAX_PAIRS = (int)(WS_COUNTER_BYTES / 4);

bool valid_G(int G) { return G == 32 || G == 64 || G == 128; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// M-tile heuristic: the largest tile that still gives every CU (256 of them)
// about two workgroups; long K loops (matrix-core bound) accept fewer, larger
// workgroups, small problems fall back to smaller tiles.  Short K loops with one
// and a half workgroups per CU still take the larger tile (128 rows; 256 for G = 64):
// they are bound by the L2 -> LDS traffic, which is (tm + G) / (tm G) per product
// (measured on the 3 x 3 convolution 256 -> 256 at 56 x 56: 17.0 against 21.7 us).
// 256-row tiles of G = 128 (8 waves) need kept-row lists of at least 384 rows: with shorter
// ones they lose 1-6 % to 128-row tiles (1024 x 4096 at M = 8192: 30.5 against 29.5 us at 75 %, 768 x
// 4096 at 60 % 34.1 against 32.1), with longer ones they win (1024 x 4096: 43.9 against 46.5 us at 50 %)
// or, on lists of 430 to 550 rows, come within 8 % either way (768 x 4096 at 50 % 37.2 against 36.0).  `dense`: the
// dense kernel has no gather to hide and takes 256 rows from one workgroup per CU on when
// K >= 1024 (2304 x 256 at M = 25088: 41.3 against 48.5 us), 128 rows for shorter K
// (768 x 3072 at M = 4096: 23.8 against 25.5 us).
int pick_tile_m(const Opts& o, int M, int n_tiles, int G, int max_k, bool dense = false) {
  const int forced = o.tile_m;
  if (forced == 64 || forced == 128 || forced == 256) {
    if (!(G == 32 && forced == 64)) return forced;
  }
  const int cand[3] = {256, 128, 64};
  for (int tm : cand) {
    if (G == 32 && tm == 64) break;
    long need = max_k >= 768 ? 320 : 512;
    if (need == 512 && (tm == 128 || (tm == 256 && G == 64))) need = 384;
    if (tm == 256 && G == 128 && max_k < 384) continue;
    if (tm == 256 && dense) need = max_k >= 1024 ? 192 : 512;
    // one 256-row workgroup per CU: 10-20 % ahead of two 128-row ones when the lists are long
    // (4096 x 1024 at M = 8192: 40.0 against 48.0 us at 50 %, 24.4 against 27.6 at 75 %; 2304 x 256 at
    // M = 25088 and 60 %: 18.7 against 23.0; 3072 x 768 at M = 8192, 192 workgroups: 28.3 against 32.9)
    if (tm == 256 && G == 128 && !dense && max_k >= 640) need = 192;
    const long wgs = (long)((M + tm - 1) / tm) * n_tiles;
    if (wgs >= need) return tm;
  }
  return G == 32 ? 128 : 64;
}

// TVW tiles are 128 rows high, two workgroups per CU (76 KB of LDS each).  64-row tiles
// (three per CU) win where 128-row tiles would leave CUs idle or end in a thin last
// round: at most one workgroup per CU, or a remainder of at most half a round of 512.
// Measured on the configured shapes: 3-13 % on the BERT-base ones, while large grids and
// long K loops (the weight tile is re-read per workgroup) keep 128.  The 256-row instance
// (8 waves) is within 3 % of the 128-row one on those; it is taken where a few N-tiles with
// long kept-row lists meet many M-tiles (at most one round of 128-row workgroups, at least
// three quarters of a round of 256-row ones): every workgroup reads its whole weight tile, and
// 256 rows share it (from HBM, 4096 x 1024 at M = 8192: 36.6 / 23.0 / 16.4 against 38.9 / 25.9 /
// 17.3 us at 75 / 87.5 / 93.75 %; 2304 x 256 at M = 25088: 15.8 against 18.6 us).
int pick_tile_m_tvw(const Opts& o, int G, int M, int n_tiles, int max_k) {
  const int forced = o.tile_m;
  if (G != 128) return 128;
  if (forced == 64 || forced == 128 || forced == 256) return forced;
  const long wgs128 = (long)((M + 127) / 128) * n_tiles;
  if (wgs128 <= 256) return 64;
  if (wgs128 <= 512 && (long)((M + 255) / 256) * n_tiles >= 192 && max_k >= 512) return 256;
  const long tail = wgs128 % 512;
  return (wgs128 <= 1536 && tail != 0 && tail <= 256) ? 64 : 128;
}

// Kept-row indices by scalar loads instead of one vector load per stage (4-wave workgroups, three
// stages in flight).  128 x 128 tiles, where more than two and nearly up to three workgroups share a CU: their
// waves hide the scalar loads' round trip, and the vector load, one more request to the copy unit per
// stage, is not hidden.  Time by scalar over time by vector loads, same buffers, grids of 6 to 29 column tiles
// and 400 to 2000 rows: 384 to 512 workgroups 0.96 .. 1.16 (768 rows: 1.05 at 75 %, 1.13 at 50 %, 0.99 at 90 %),
// 513 to 704 0.87 .. 1.03 (0.92, 0.95, 0.99), 720 to 736 0.93 .. 1.04 (0.98, 0.97, 0.99), 748 to 768 0.91 .. 1.03 (1.02,
// 0.98, 0.99), more 1.01 .. 1.13 (1.05).  768 x 2304 at M = 4096, 75 %, 576 workgroups: 10.2 / 12.2 us.
// 256 x 64 tiles only on convolutions with long lists, whose misaligned rows keep the copy unit busy:
// nine of them 0 to 3.5 % (256 -> 256 at 56 x 56, batch 8, 16.9 / 17.5; 256 -> 512 at 28 x 28, batch 16, 16.8 / 17.3;
// 128 -> 128 at 56 x 56 and 50 % 16.6 / 17.2); short lists are even (64 -> 256 at 80 x 80 14.6 / 14.5), and a plain
// 1024 x 2048 at 60 % loses (14.0 / 12.6).
bool scalar_rows(const Opts& o, int M, int n_tiles, int G, int tm, int max_k, bool conv) {
  if (o.idx_route) return o.idx_route == 1;
  const long wgs = (long)((M + tm - 1) / tm) * n_tiles;
  if (G == 128 && tm == 128) return wgs > 512 && wgs <= 736;
  return conv && G == 64 && tm == 256 && wgs > 384 && max_k > 256;
}

// K-split inside the workgroup pays when 128-row tiles cannot give every CU a
// workgroup and the K loop is long enough to amortise the final reduction.  64-row tiles
// only where 128-row tiles would leave half of the CUs idle or more: they move half as much
// again from L2 into LDS per product and read A in 128-byte pieces (3072 x 768 at M = 4096 from
// cold HBM: 15.9 us with 64-row tiles, 13.7 with 128-row tiles; 4608 x 512 at M = 1568, 52
// tiles of 128 rows: 11.1 against 14.2 us the other way).  el: bytes per weight (0: the dense baseline).
bool use_ksplit(int M, int n_tiles, int G, int max_k, int el, int* tm) {
  const long wgs128 = (long)((M + 127) / 128) * n_tiles;
  if (max_k < 12 * 32 || wgs128 > 320) return false;
  // 64 rows as long as every workgroup has a CU to itself: it is done in about three quarters of the time of 128 rows (256 / 258
  // workgroups of 64 and half as many of 128, 64 / 128 rows: 4096 x 1024 at 50 %, G = 128, 17.5 / 22.9 and 24.6 / 23.2 us;
  // 2048 x 1024 at 80 % 7.2 / 9.0 and 9.2 / 9.1; TEW 2048 x 2048 at 60 % 17.0 / 21.3 and 23.5 / 21.5; int8 4096 x 1024 at 50 %
  // 11.3 / 14.1 and 16.5 / 14.6).  Weights of uneven tiles would gain from 64 rows further on (1003 x 2491, G = 64: 288 to 864
  // workgroups 7.8 / 8.3, 8.1 / 9.3, 8.1 / 9.5 and 9.2 / 10.1, then 11.3 / 11.1), which none of these numbers tells.
  if ((long)((M + 63) / 64) * n_tiles > 256) { *tm = 128; return true; }
  // Not with many column tiles of 128, from half a round of 128-row workgroups on: few rows of A then share a long list of
  // weights, and every 64 of them fetch it again (64 / 128 rows, 64 x 32 tiles: 4096 rows, 50 %, 22.5 / 19.2 us, 2048 rows
  // 13.3 / 12.1, TEW 4096 rows, 75 %, 30.5 / 25.8, int8 4096 rows 13.7 / 12.3, dense 4096 rows 40.1 / 32.2, 1024 rows 12.9 / 11.3;
  // 26 tiles 19.8 / 19.2 and dense 33.3 / 31.1; 22 tiles 17.8 / 19.2 and 29.1 / 31.2).  Lists of 1 KiB a column gain all the same
  // (512 rows, 32 and 64 tiles 7.3 / 8.3, 7.5 / 8.2 us; int8, 1024 rows, 8.3 / 8.4).
  const bool few_or_short = n_tiles <= 24 || (el > 0 && max_k * el <= 1024);
  *tm = wgs128 < 128 || G == 64 || few_or_short ? 64 : 128;
  return true;
}

// K split across workgroups (needs a workspace).  *tm = M-tile, *S = workgroups per pair
// (1 = do not split).  Only on request: measured on the few-tile shapes it is built for
// (3072 x 768 at M = 4096; 4608 x 512 at M = 1568) it never beat the split inside the workgroup
// (two wave groups, partial sums through LDS): 18.7 against 11.9 us and 12.6 against 10.8 us at
// best.  The partial tiles have to pass through memory that is coherent across the XCDs' L2
// caches, and that traffic (4 bytes per output element and workgroup, written and read) costs
// more than the shorter K loops save.
void pick_wg_split(const Opts& o, int M, int n_tiles, int G, int max_k, int* tm, int* S) {
  *S = 1;
  if (o.wg_split < 2) return;
  const int forced_tm = (o.tile_m == 64 || o.tile_m == 128) ? o.tile_m : 0;
  int t = forced_tm ? forced_tm : 128;
  if (G == 64) t = 128;                       // the one split instance for G = 64
  const int stages = max_k / 32;
  int s = o.wg_split;
  if (s > stages) s = stages > 0 ? stages : 1;
  (void)M; (void)n_tiles;
  *tm = t;
  *S = s;
}

// TEW: restored elements one by one behind the K loop instead of in the rows that join it.  32 joined rows cost a workgroup
// as much as 2 elements in each of its columns, plus the time of 7 elements to come to its lists (fitted to 476 launches: 17 K x N,
// 60 to 95 %, 0.02 to 2 % restored, M = 256 to 8192), where joined rows are dear: up to half a workgroup of 128 rows per CU, when the
// K loop is a chain with nothing beside it and joined rows are most of it, and with many column tiles, whose weights no
// longer fit an XCD's L2, unless two workgroups are on every CU and no more.  Joined / one by one, K x N x M, sparsity, restored:
// 4096 x 1024 x 512, 90 %, 0.5 % 16.6 / 13.1 us, x 8192 37.3 / 48.1; 2048 x 3072 x 512, 75 %, 0.5 % 14.7 / 12.1, x 1024 16.5 / 16.8;
// 2560 x 4096 x 384, 85 %, 0.6 % 16.9 / 12.8, x 1024 22.1 / 19.1, x 2048 31.1 / 33.3, x 6144 103 / 83; 4096 x 4096 x 8192, 95 %,
// 0.5 % 169 / 125, 2 % 282 / 315; 2048 x 2048, 60 %, 768 x 3072 and G = 64: 5 to 40 % for joined rows.  A's rows have to start on lines
// of 128 bytes: an element's 256 bytes are three of them otherwise (2048 x 3072 x 1957, 0.5 % 25.2 / 29.6).
bool ew_elements(const tw_handle_s* h, int M, int lda) {
  const twg::DeviceImage& d = h->img;
  if (h->G != 128 || d.join_off.empty() || h->n_tiles == 0 || lda % 64) return false;
  const long wgs128 = (long)((M + 127) / 128) * d.n_tiles;
  const double rows = (double)d.join_row.size() / d.n_tiles, kept = (double)h->sum_k / h->n_tiles;   // of a tile
  const double per_column = (double)d.ew_pairs.size() / h->N;
  if (wgs128 > 256) return d.n_tiles >= 24 && wgs128 > 640 && rows / 32 > 5 + 2.1 * per_column;
  if (wgs128 > 128) return d.n_tiles >= 24 && rows / 32 > 8 + 2.1 * per_column && rows >= 1.5 * kept;
  return rows / 32 > 7 + 1.8 * per_column && rows >= (d.n_tiles >= 24 && wgs128 > 64 ? 0.9 : 1.5) * kept;
}

}  // namespace

// A convolution geometry bound to a packed weight: the kept-row lists of the handle's device
// image turned into element offsets for that geometry.  The handle itself is not changed.
struct tw_conv_s {
  tw_handle_t h = nullptr;
  tw_conv_geom geom{};
  int64_t ldx = 0;
  int32_t* d_off = nullptr;
};

extern "C" {

const char* tw_status_str(int s) {
  switch (s) {
    case TW_OK: return "ok";
    case TW_ERR_ARG: return "invalid argument";
    case TW_ERR_MASK: return "mask is not TW/TVW conformant";
    case TW_ERR_UNSUPPORTED: return "unsupported configuration";
    case TW_ERR_ALLOC: return "allocation failed";
    case TW_ERR_HIP: return "HIP runtime error";
    case TW_ERR_STATE: return "handle not uploaded";
    case TW_ERR_TOO_LARGE: return "problem larger than the library's static scratch (use the entry point that takes a workspace)";
    default: return "unknown status";
  }
}

tw_status tw_pack_host(const uint16_t* B, const uint8_t* mask, const uint8_t* tile_mask, int K,
                       int N, int G, int pattern, tw_handle_t* out) {
  if (!out) return TW_ERR_ARG;
  *out = nullptr;
  if (!B || !mask || K < 1 || N < 1 || !valid_G(G)) return TW_ERR_ARG;
  if (pattern != TW_PATTERN_TW && pattern != TW_PATTERN_TVW && pattern != TW_PATTERN_TEW) return TW_ERR_ARG;
  if (pattern == TW_PATTERN_TEW && !tile_mask) return TW_ERR_ARG;
  if (pattern == TW_PATTERN_TEW && K > 65536) return TW_ERR_UNSUPPORTED;   // restored rows travel as 16 bits
  tw_handle_s* h = new (std::nothrow) tw_handle_s();
  if (!h) return TW_ERR_ALLOC;
  tw_status st = twg::pack_host(B, mask, tile_mask, K, N, G, pattern, h);
  if (st != TW_OK) { delete h; return st; }
  *out = h;
  return TW_OK;
}

tw_status tw_upload(tw_handle_t h) {
  if (!h) return TW_ERR_ARG;
  twg::DeviceImage& d = h->img;
  if (d.blob) return TW_OK;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return TW_ERR_HIP;
  twg::ImageLayout L;
  twg::layout_image(h, &L);
  const void* src[twg::IMG_PARTS] = {};
  src[twg::IMG_TILE_KP_OFF] = d.tile_kp_off.data(); src[twg::IMG_TILE_ORDER] = d.tile_order.data();
  src[twg::IMG_TILE_SCHED] = d.tile_sched.data(); src[twg::IMG_COL_IDX] = d.col_idx.data();
  src[twg::IMG_ROW_IDX] = d.row_idx.data(); src[twg::IMG_ZERO_COLS] = d.zero_cols.data();
  src[twg::IMG_VALS] = h->dtype == TW_DTYPE_I8 ? (const void*)d.vals8.data() : (const void*)d.vals.data();
  src[twg::IMG_META] = d.meta.data(); src[twg::IMG_EW_PTR] = d.ew_ptr.data(); src[twg::IMG_EW_PAIRS] = d.ew_pairs.data();
  void* blob = nullptr;
  if (hipMalloc(&blob, L.total) != hipSuccess) { (void)hipGetLastError(); return TW_ERR_ALLOC; }
  for (int i = 0; i < twg::IMG_PARTS; ++i) {
    if (!L.bytes[i]) continue;
    if (hipMemcpy((char*)blob + L.off[i], src[i], L.bytes[i], hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipFree(blob);
      return TW_ERR_HIP;
    }
  }
  twg::bind_image(h, blob, L, dev);
  return TW_OK;
}

tw_status tw_pack(const uint16_t* B, const uint8_t* mask, const uint8_t* tile_mask, int K, int N,
                  int G, int pattern, tw_handle_t* out) {
  tw_status st = tw_pack_host(B, mask, tile_mask, K, N, G, pattern, out);
  if (st != TW_OK) return st;
  st = tw_upload(*out);
  if (st != TW_OK) { tw_free(*out); *out = nullptr; }
  return st;
}

tw_status tw_pack_i8_host(const int8_t* B, const uint8_t* mask, const uint8_t* tile_mask, int K, int N,
                          int G, int pattern, tw_handle_t* out) {
  if (!out) return TW_ERR_ARG;
  *out = nullptr;
  if (!B || !mask || K < 1 || N < 1 || !valid_G(G)) return TW_ERR_ARG;
  if (pattern == TW_PATTERN_TEW) return TW_ERR_UNSUPPORTED;
  if (pattern != TW_PATTERN_TW && pattern != TW_PATTERN_TVW) return TW_ERR_ARG;
  tw_handle_s* h = new (std::nothrow) tw_handle_s();
  if (!h) return TW_ERR_ALLOC;
  tw_status st;
  try {
    // the packer moves 16-bit patterns around without looking at them: int8 values
    // ride through it sign-extended
    std::vector<uint16_t> wide((size_t)K * N);
    for (size_t i = 0; i < wide.size(); ++i) wide[i] = (uint16_t)(int16_t)B[i];
    h->dtype = TW_DTYPE_I8;
    st = twg::pack_host(wide.data(), mask, tile_mask, K, N, G, pattern, h);
  } catch (const std::bad_alloc&) {
    st = TW_ERR_ALLOC;
  }
  if (st != TW_OK) { delete h; return st; }
  *out = h;
  return TW_OK;
}

tw_status tw_pack_i8(const int8_t* B, const uint8_t* mask, const uint8_t* tile_mask, int K, int N, int G,
                     int pattern, tw_handle_t* out) {
  tw_status st = tw_pack_i8_host(B, mask, tile_mask, K, N, G, pattern, out);
  if (st != TW_OK) return st;
  st = tw_upload(*out);
  if (st != TW_OK) { tw_free(*out); *out = nullptr; }
  return st;
}

tw_status tw_prune_workspace_bytes(int K, int N, int G, size_t* bytes) {
  if (!bytes || K < 1 || N < 1 || !valid_G(G)) return TW_ERR_ARG;
  *bytes = twg::prune_workspace_bytes(K, N, G);
  return TW_OK;
}

tw_status tw_prune_dev(const void* B_dev, int K, int N, int ldb, int G, int pattern, int n_cols_pruned,
                       int rows_per_tile, uint8_t* mask_dev, uint8_t* tile_mask_dev, void* workspace_dev,
                       size_t workspace_bytes, void* stream) {
  if (!B_dev || !mask_dev || !workspace_dev || K < 1 || N < 1 || ldb < N || !valid_G(G)) return TW_ERR_ARG;
  if (n_cols_pruned < 0 || n_cols_pruned > N || rows_per_tile < 0 || rows_per_tile > K) return TW_ERR_ARG;
  if (pattern == TW_PATTERN_TEW) return TW_ERR_UNSUPPORTED;
  if (pattern != TW_PATTERN_TW && pattern != TW_PATTERN_TVW) return TW_ERR_ARG;
  if (((uintptr_t)workspace_dev & 15) || workspace_bytes < twg::prune_workspace_bytes(K, N, G)) return TW_ERR_ARG;
  if (((size_t)K * N + 255) / 256 > 0x7fffffffu) return TW_ERR_UNSUPPORTED;   // one thread per element, grid limit
  if ((N + G - 1) / G > 65535 || (K + 255) / 256 > 65535 || (N + 255) / 256 > 65535) return TW_ERR_UNSUPPORTED;
  hipError_t e = twg::prune_device((const uint16_t*)B_dev, K, N, ldb, G, pattern == TW_PATTERN_TVW, n_cols_pruned,
                                   rows_per_tile, mask_dev, tile_mask_dev, workspace_dev, (hipStream_t)stream);
  return e == hipSuccess ? TW_OK : TW_ERR_HIP;
}

tw_status tw_prune_dev_static(const void* B_dev, int K, int N, int ldb, int G, int pattern, int n_cols_pruned,
                              int rows_per_tile, uint8_t* mask_dev, uint8_t* tile_mask_dev, void* stream) {
  if (!B_dev || !mask_dev || K < 1 || N < 1 || ldb < N || !valid_G(G)) return TW_ERR_ARG;
  if (n_cols_pruned < 0 || n_cols_pruned > N || rows_per_tile < 0 || rows_per_tile > K) return TW_ERR_ARG;
  if (pattern == TW_PATTERN_TEW) return TW_ERR_UNSUPPORTED;
  if (pattern != TW_PATTERN_TW && pattern != TW_PATTERN_TVW) return TW_ERR_ARG;
  if (twg::prune_workspace_bytes(K, N, G) > twg::PRUNE_STATIC_SCRATCH_BYTES) return TW_ERR_TOO_LARGE;
  if (((size_t)K * N + 255) / 256 > 0x7fffffffu) return TW_ERR_TOO_LARGE;
  if ((N + G - 1) / G > 65535 || (K + 255) / 256 > 65535 || (N + 255) / 256 > 65535) return TW_ERR_TOO_LARGE;
  void* ws = nullptr;
  if (twg::prune_static_scratch(&ws) != hipSuccess) { (void)hipGetLastError(); return TW_ERR_HIP; }
  hipError_t e = twg::prune_device((const uint16_t*)B_dev, K, N, ldb, G, pattern == TW_PATTERN_TVW, n_cols_pruned,
                                   rows_per_tile, mask_dev, tile_mask_dev, ws, (hipStream_t)stream);
  return e == hipSuccess ? TW_OK : TW_ERR_HIP;
}

tw_status tw_pack_dev(const void* B_dev, int ldb, const uint8_t* mask_dev, const uint8_t* tile_mask_dev, int K,
                      int N, int G, int pattern, void* stream, tw_handle_t* out) try {
  if (!out) return TW_ERR_ARG;
  *out = nullptr;
  if (!B_dev || !mask_dev || K < 1 || N < 1 || ldb < N || !valid_G(G)) return TW_ERR_ARG;
  if (pattern != TW_PATTERN_TW && pattern != TW_PATTERN_TVW && pattern != TW_PATTERN_TEW) return TW_ERR_ARG;
  hipStream_t s = (hipStream_t)stream;
  if (pattern != TW_PATTERN_TEW) {       // packed by kernels: only the index lists visit the host
    tw_handle_s* h = new (std::nothrow) tw_handle_s();
    if (!h) return TW_ERR_ALLOC;
    const tw_status st = twg::pack_device((const uint16_t*)B_dev, ldb, mask_dev, tile_mask_dev, K, N, G, pattern, s, h);
    if (st != TW_OK) { tw_free(h); return st; }
    *out = h;
    return TW_OK;
  }
  // TEW: through the host packer
  if (!tile_mask_dev) return TW_ERR_ARG;
  std::vector<uint16_t> B((size_t)K * N);
  std::vector<uint8_t> mask((size_t)K * N), tmask((size_t)K * N);
  if (hipMemcpy2DAsync(B.data(), (size_t)N * 2, B_dev, (size_t)ldb * 2, (size_t)N * 2, K, hipMemcpyDeviceToHost, s) !=
          hipSuccess ||
      hipMemcpyAsync(mask.data(), mask_dev, mask.size(), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipMemcpyAsync(tmask.data(), tile_mask_dev, tmask.size(), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    (void)hipGetLastError();
    return TW_ERR_HIP;
  }
  return tw_pack(B.data(), mask.data(), tmask.data(), K, N, G, pattern, out);
} catch (const std::bad_alloc&) {
  return TW_ERR_ALLOC;
}

tw_status tw_concat(const tw_handle_t* parts, int n, int upload, tw_handle_t* out) {
  if (!out) return TW_ERR_ARG;
  *out = nullptr;
  if (!parts || n < 1) return TW_ERR_ARG;
  for (int i = 0; i < n; ++i) {
    if (!parts[i]) return TW_ERR_ARG;
    const tw_status sf = twg::fetch_logical(parts[i]);          // a device-packed member
    if (sf != TW_OK) return sf;
  }
  tw_handle_s* h = new (std::nothrow) tw_handle_s();
  if (!h) return TW_ERR_ALLOC;
  tw_status st = twg::concat_host(parts, n, h);
  if (st == TW_OK && upload) st = tw_upload(h);
  if (st != TW_OK) { tw_free(h); return st; }
  *out = h;
  return TW_OK;
}

// The launch behind tw_gemm and tw_conv_gemm.  conv: A is the wide input, the row list holds
// window offsets (lda = 1) and M counts the wide grid.
static tw_status gemm_launch(const Opts& o, const void* A, int M, int lda, int layout, tw_handle_t h, void* C,
                             int ldc, void* stream, const tw_conv_s* conv) {
  twg::GemmArgs g{};
  g.A = (const _Float16*)A; g.C = (_Float16*)C; g.M = M; g.lda = lda; g.ldc = ldc;
  g.vals = (const _Float16*)h->img.d_vals;
  g.row_idx = h->img.d_row_idx; g.tile_kp_off = h->img.d_tile_kp_off;
  if (conv) {
    g.row_idx = conv->d_off;
    g.conv_P = conv->geom.P; g.conv_L = conv->geom.L; g.conv_H = conv->geom.H; g.conv_W = conv->geom.W;
  }
  g.col_idx = h->img.d_col_idx; g.tile_order = h->img.d_tile_order;
  g.tile_sched = h->img.d_tile_sched; g.uniform_kp = h->img.uniform_kp;
  g.zero_cols = h->img.d_zero_cols; g.n_zero = h->img.n_zero;
  g.meta = h->img.d_meta;
  g.ew_ptr = h->img.d_ew_ptr; g.ew_pairs = h->img.d_ew_pairs;
  g.ew_last = h->img.ew_pairs.empty() ? 0 : (int)h->img.ew_pairs.size() - 1;
  const int n_tiles = h->img.n_tiles;
  g.n_tiles = n_tiles; g.K = h->K; g.N = h->N; g.xcd_map = o.xcd_map;
  g.wg_split = 1;
  g.tiles_per_wg = 1;
  if (layout == TW_LAYOUT_MK) {
    hipError_t e = twg::launch_tw_mk(h->G, h->max_kp, h->nonfinite, g, (hipStream_t)stream);
    if (e == hipErrorInvalidValue) return TW_ERR_UNSUPPORTED;
    return e == hipSuccess ? TW_OK : TW_ERR_HIP;
  }
  // the asynchronous kernel addresses A with 32-bit byte offsets
  const bool a_fits32 = conv || (unsigned long long)h->K * (unsigned long long)lda * 2ull < (1ull << 32);
  // Few output blocks.  A weight with nothing pruned adds up in the order of the dense baseline (same
  // bits), and a TEW weight without restored elements in the order of its TW twin.  (sum_kw counts a TVW
  // weight before its 2:4 step, so one that keeps every row and column stays with the pipelined kernel too.)
  const bool small = h->pattern != TW_PATTERN_TEW || (h->G != 32 && a_fits32);
  if (small && automatic(o) && h->sum_kw < (int64_t)h->K * h->N &&
      twg::small_km_pays(h->G, h->pattern == TW_PATTERN_TVW, M, n_tiles, h->max_kp)) {
    hipError_t e = twg::launch_small_km(h->G, h->pattern == TW_PATTERN_TVW, !h->img.ew_pairs.empty(), h->max_kp, g,
                                        (hipStream_t)stream);
    return e == hipSuccess ? TW_OK : TW_ERR_HIP;
  }
  if (h->pattern == TW_PATTERN_TVW) {
    const int tvw_tm = pick_tile_m_tvw(o, h->G, M, n_tiles > 0 ? n_tiles : 1, h->max_kp);
    hipError_t e = twg::launch_tvw_km(h->G, tvw_tm, o.depth > 4 ? 4 : o.depth, g, (hipStream_t)stream);
    if (e == hipErrorInvalidValue) return TW_ERR_UNSUPPORTED;
    return e == hipSuccess ? TW_OK : TW_ERR_HIP;
  }
  const bool restored = !h->img.ew_pairs.empty();
  g.ew_elements = restored && ew_elements(h, M, lda);
  const int max_kp = g.ew_elements ? h->img.max_kept_kp : h->max_kp;
  int tm = pick_tile_m(o, M, n_tiles > 0 ? n_tiles : 1, h->G, max_kp);
  // no 64 x 64 instance of the asynchronous kernel without K groups (tried: one matrix instruction per wave and
  // k-step is too little work per barrier; plain TW falls back to the register-staged kernel)
  if ((h->pattern == TW_PATTERN_TEW || conv) && h->G == 64 && tm == 64) tm = 128;
  const bool tew = h->pattern == TW_PATTERN_TEW;
  // TEW: the kernels with restored elements, three stages only; without any, the TW kernels
  // The 256-row instance of G = 128 has no register to spare for its second way to the result (768 x 3072 at M =
  // 4096, 1.5 % restored: 29.4 / 26.4 us with 256 / 128 rows; 3072 x 768: 26.4 / 26.7)
  if (restored && h->G == 128 && tm == 256 && o.tile_m != 256) tm = 128;
  hipError_t e = hipErrorInvalidValue;
  auto launch_dma = restored ? twg::launch_tew_km_dma : twg::launch_tw_km_dma;
  const int depth = tew ? 3 : o.depth;
  // K split across workgroups: few tiles, long kept-row lists, and a workspace to reduce through
  if (!tew && o.kernel != 1 && h->G != 32 && a_fits32 && o.ws && o.wg_split != 1 && n_tiles > 0) {
    int stm = 0, S = 0;
    pick_wg_split(o, M, n_tiles, h->G, max_kp, &stm, &S);
    if (S > 1) {
      const long pairs = (long)((M + stm - 1) / stm) * n_tiles;
      const size_t need = WS_COUNTER_BYTES + (size_t)pairs * S * stm * h->G * 4;
      if (pairs <= WS_MAX_PAIRS && need <= o.ws_bytes) {
        g.wg_split = S;
        g.ws_counters = (int*)o.ws;
        g.ws_partials = (float*)((char*)o.ws + WS_COUNTER_BYTES);
        hipError_t es = twg::launch_tw_km_dma_split(h->G, stm, g, (hipStream_t)stream);
        if (es != hipErrorInvalidValue) return es == hipSuccess ? TW_OK : TW_ERR_HIP;
        g.wg_split = 1;
      } else if (o.wg_split > 1) {
        return TW_ERR_ARG;          // a split was asked for and the workspace cannot hold it
      }
    }
  }
  if ((o.kernel != 1 || tew || conv) && h->G != 32 && a_fits32) {
    // long K with too few tiles to fill the chip: split K inside the workgroup
    // 256-row tiles run with 8 waves (64 x 64 per wave): half the registers per wave, two
    // workgroups per CU
    int variant = (o.waves == 8 || (tm == 256 && h->G == 128)) ? twg::DMA_WAVES8 : twg::DMA_WAVES4;
    int tmk = tm;
    const int ks = o.ksplit;
    if (ks == 2 || (ks == 0 && use_ksplit(M, n_tiles, h->G, max_kp, 2, &tmk))) variant = twg::DMA_KSPLIT2;
    if (variant == twg::DMA_KSPLIT2 && ks == 2) tmk = tm == 256 ? 128 : tm;
    if (variant == twg::DMA_KSPLIT2 && h->G == 64 && (restored || ks == 2)) tmk = 128;   // (no other instance; on request)
    const int tmu = variant == twg::DMA_KSPLIT2 ? tmk : tm;
    g.scalar_rows = !restored && variant == twg::DMA_WAVES4 && scalar_rows(o, M, n_tiles, h->G, tmu, max_kp, conv);
    // several tiles per workgroup (plain TW, 4 waves, 64- or 128-row tiles of G = 128, 3 stages): on request
    if (!tew && variant == twg::DMA_WAVES4 && o.tiles_per_wg > 1) g.tiles_per_wg = o.tiles_per_wg;
    e = launch_dma(h->G, tmu, depth, variant, g, (hipStream_t)stream);
    if (e == hipErrorInvalidValue && variant != twg::DMA_WAVES4)
      e = launch_dma(h->G, tm, depth, twg::DMA_WAVES4, g, (hipStream_t)stream);
  }
  if (e == hipErrorInvalidValue && o.kernel != 2 && !tew && !conv)
    e = twg::launch_tw_km(h->G, tm, g, (hipStream_t)stream);
  if (e == hipErrorInvalidValue) return TW_ERR_UNSUPPORTED;
  return e == hipSuccess ? TW_OK : TW_ERR_HIP;
}

tw_status tw_launch_opts_init(tw_launch_opts* opts) {
  if (!opts) return TW_ERR_ARG;
  const Opts d = default_opts();
  opts->tile_m = d.tile_m; opts->kernel = d.kernel; opts->depth = d.depth; opts->waves = d.waves;
  opts->ksplit = d.ksplit; opts->xcd_map = d.xcd_map; opts->wg_split = d.wg_split; opts->idx_route = d.idx_route; opts->tiles_per_wg = d.tiles_per_wg;
  opts->workspace_dev = nullptr; opts->workspace_bytes = 0;
  return TW_OK;
}

tw_status tw_gemm_workspace_bytes(tw_handle_t h, int M, size_t* bytes) {
  if (!h || !bytes || M < 1) return TW_ERR_ARG;
  // enough for any split the library may choose at this M: 64-row tiles, 8 workgroups per pair,
  // as long as the pairs fit the counters (beyond that no split is used)
  const long pairs64 = (long)((M + 63) / 64) * (h->n_tiles > 0 ? h->n_tiles : 1);
  const long pairs = pairs64 < WS_MAX_PAIRS ? pairs64 : WS_MAX_PAIRS;
  *bytes = WS_COUNTER_BYTES + (size_t)pairs * 8 * 64 * 128 * 4;
  return TW_OK;
}

tw_status tw_workspace_init(void* workspace_dev, size_t workspace_bytes, void* stream) {
  if (!workspace_dev || ((uintptr_t)workspace_dev & 255) || workspace_bytes < WS_COUNTER_BYTES) return TW_ERR_ARG;
  return twg::launch_zero_words((uint32_t*)workspace_dev, WS_COUNTER_BYTES / 4, (hipStream_t)stream) == hipSuccess
             ? TW_OK : TW_ERR_HIP;
}

tw_status tw_gemm_ex(const void* A, int M, int lda, int layout, tw_handle_t h, void* C, int ldc,
                     const tw_launch_opts* opts, void* stream) {
  if (!A || !C || !h || M < 1) return TW_ERR_ARG;
  if (layout != TW_LAYOUT_KM && layout != TW_LAYOUT_MK) return TW_ERR_ARG;
  if (!aligned16(A) || !aligned16(C) || lda % 8 || ldc % 8) return TW_ERR_ARG;
  if (h->dtype != TW_DTYPE_F16) return TW_ERR_ARG;
  if (!h->img.blob) return TW_ERR_STATE;
  if (layout == TW_LAYOUT_MK) {
    if (lda < h->K || ldc < h->N) return TW_ERR_ARG;
    if (h->pattern != TW_PATTERN_TW) return TW_ERR_UNSUPPORTED;   // TVW and TEW exist for K x M only
  } else if (lda < M || ldc < M) {
    return TW_ERR_ARG;
  }
  Opts o;
  if (!opts_from(opts, &o)) return TW_ERR_ARG;
  return gemm_launch(o, A, M, lda, layout, h, C, ldc, stream, nullptr);
}

tw_status tw_gemm(const void* A, int M, int lda, int layout, tw_handle_t h, void* C, int ldc,
                  void* stream) {
  return tw_gemm_ex(A, M, lda, layout, h, C, ldc, nullptr, stream);
}

tw_status tw_conv_bind(tw_handle_t h, const tw_conv_geom* cg, int64_t ldx, tw_conv_t* out) {
  if (!out) return TW_ERR_ARG;
  *out = nullptr;
  if (!h || !cg) return TW_ERR_ARG;
  if (cg->C < 1 || cg->R < 1 || cg->S < 1 || cg->B < 1 || cg->H < 1 || cg->W < 1) return TW_ERR_ARG;
  if (cg->P < cg->W + cg->S - 1 || cg->L < cg->H + cg->R - 1) return TW_ERR_ARG;
  if ((int64_t)cg->C * cg->R * cg->S != h->K) return TW_ERR_ARG;
  const int64_t Mp = (int64_t)cg->B * cg->L * cg->P;
  if (Mp > INT32_MAX - 8) return TW_ERR_ARG;
  const int chunk = h->dtype == TW_DTYPE_I8 ? 16 : 8;          // elements per 16-byte copy
  const int64_t reach = (Mp + chunk - 1) / chunk * chunk + (int64_t)(cg->R - 1) * cg->P + cg->S - 1;
  if (ldx < reach || ldx % chunk || (int64_t)cg->C * ldx >= (1ll << 31)) return TW_ERR_ARG;
  if (h->pattern == TW_PATTERN_TEW || h->G == 32) return TW_ERR_UNSUPPORTED;
  if (!h->img.blob) return TW_ERR_STATE;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return TW_ERR_HIP;
  if (dev != h->img.device) return TW_ERR_STATE;
  const tw_status sf = twg::fetch_lists(h);            // the padded kept-row lists of a device-packed weight
  if (sf != TW_OK) return sf;
  std::vector<int32_t> off;
  tw_conv_s* b = new (std::nothrow) tw_conv_s();
  if (!b) return TW_ERR_ALLOC;
  try {
    off.resize(h->img.row_idx.size());
  } catch (const std::bad_alloc&) {
    delete b;
    return TW_ERR_ALLOC;
  }
  const int RS = cg->R * cg->S;
  for (size_t i = 0; i < off.size(); ++i) {
    const int k = h->img.row_idx[i], c = k / RS, r = (k % RS) / cg->S, s = k % cg->S;
    off[i] = (int32_t)((int64_t)c * ldx + (int64_t)r * cg->P + s);
  }
  int32_t* d = nullptr;
  if (hipMalloc((void**)&d, off.size() * 4 + 4) != hipSuccess) { (void)hipGetLastError(); delete b; return TW_ERR_ALLOC; }
  if (hipMemcpy(d, off.data(), off.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipFree(d);
    delete b;
    return TW_ERR_HIP;
  }
  b->h = h; b->geom = *cg; b->ldx = ldx; b->d_off = d;
  *out = b;
  return TW_OK;
}

tw_status tw_conv_free(tw_conv_t b) {
  if (!b) return TW_OK;
  const tw_status st = (b->d_off && hipFree(b->d_off) != hipSuccess) ? TW_ERR_HIP : TW_OK;
  delete b;
  return st;
}

tw_status tw_conv_gemm(const void* X, tw_conv_t b, void* C, int ldc, void* stream) {
  if (!X || !C || !b || !b->h) return TW_ERR_ARG;
  if (b->h->dtype != TW_DTYPE_F16) return TW_ERR_ARG;
  const int Mp = b->geom.B * b->geom.L * b->geom.P;
  if (!aligned16(X) || !aligned16(C) || ldc % 8 || ldc < Mp) return TW_ERR_ARG;
  return gemm_launch(default_opts(), X, Mp, 1, TW_LAYOUT_KM, b->h, C, ldc, stream, b);
}

tw_status tw_dense_gemm(const void* A, const void* B, void* C, int M, int K, int N, int lda,
                        int ldb, int ldc, int layout, void* stream) {
  if (!A || !B || !C || M < 1 || K < 1 || N < 1) return TW_ERR_ARG;
  if (layout != TW_LAYOUT_KM && layout != TW_LAYOUT_MK) return TW_ERR_ARG;
  if (!aligned16(A) || !aligned16(B) || !aligned16(C) || lda % 8 || ldb % 8 || ldc % 8)
    return TW_ERR_ARG;
  if (ldb < N) return TW_ERR_ARG;
  if (layout == TW_LAYOUT_MK) {
    if (lda < K || ldc < N) return TW_ERR_ARG;
  } else if (lda < M || ldc < M) {
    return TW_ERR_ARG;
  }
  twg::GemmArgs g{};
  g.A = (const _Float16*)A; g.C = (_Float16*)C; g.M = M; g.lda = lda; g.ldc = ldc;
  g.vals = (const _Float16*)B; g.ldb = ldb; g.K = K; g.N = N;
  const int tn = 128;
  g.n_tiles = (N + tn - 1) / tn;
  const Opts o = default_opts();
  g.xcd_map = o.xcd_map;
  g.wg_split = 1;
  if (layout == TW_LAYOUT_MK) {
    hipError_t em = twg::launch_dense_mk(g, (hipStream_t)stream);
    return em == hipSuccess ? TW_OK : TW_ERR_HIP;
  }
  const int tm = pick_tile_m(o, M, g.n_tiles, tn, K, true);
  hipError_t e = hipErrorInvalidValue;
  const bool fits32 = (unsigned long long)K * (unsigned long long)lda * 2ull < (1ull << 32) &&
                      (unsigned long long)K * (unsigned long long)ldb * 2ull < (1ull << 32);
  if (o.kernel != 1 && K % 32 == 0 && fits32) {
    int variant = (o.waves == 8 || tm == 256) ? twg::DMA_WAVES8 : twg::DMA_WAVES4;
    int tmk = tm;
    const int ks = o.ksplit;
    if (K % 64 == 0 && (ks == 2 || (ks == 0 && use_ksplit(M, g.n_tiles, tn, K, 0, &tmk)))) variant = twg::DMA_KSPLIT2;
    if (variant == twg::DMA_KSPLIT2 && ks == 2) tmk = tm == 256 ? 128 : tm;
    e = twg::launch_dense_km_dma(tn, variant == twg::DMA_KSPLIT2 ? tmk : tm, o.depth, variant, g,
                                 (hipStream_t)stream);
    if (e == hipErrorInvalidValue && variant != twg::DMA_WAVES4)
      e = twg::launch_dense_km_dma(tn, tm, o.depth, twg::DMA_WAVES4, g, (hipStream_t)stream);
  }
  if (e == hipErrorInvalidValue && o.kernel != 2)
    e = twg::launch_dense_km(tn, tm, g, (hipStream_t)stream);
  if (e == hipErrorInvalidValue) return TW_ERR_UNSUPPORTED;
  return e == hipSuccess ? TW_OK : TW_ERR_HIP;
}

// int8 M-tile: 256 rows while that still gives every CU two workgroups, else 128.  The 64-row
// instance (G = 128) is only used on request: it measured no better than 128 rows on the small
// BERT-base launches and worse on the dense baseline.  As for fp16, 256 rows need kept-row lists of
// at least 384 rows (1024 x 4096 at M = 8192 and 87.5 %, from HBM: 17.5 against 16.3 us).
static int pick_tile_m_i8(const Opts& o, int M, int n_tiles, int G, int max_k) {
  const int forced = o.tile_m;
  if (forced == 128 || forced == 256 || (forced == 64 && G == 128)) return forced;
  return (max_k >= 384 && (long)((M + 255) / 256) * n_tiles >= 512) ? 256 : 128;
}

// The launch behind tw_gemm_i8 and tw_conv_gemm_i8 (conv: see gemm_launch).
static tw_status gemm_i8_launch(const void* A, int M, int lda, tw_handle_t h, void* C, int ldc, int c_dtype,
                                float scale, void* stream, const tw_conv_s* conv) {
  const Opts o = default_opts();
  twg::GemmI8Args g{};
  g.A = (const int8_t*)A; g.C = C; g.M = M; g.lda = lda; g.ldc = ldc;
  g.c_i8 = c_dtype; g.scale = scale;
  g.vals = (const int8_t*)h->img.d_vals;
  g.row_idx = h->img.d_row_idx; g.col_idx = h->img.d_col_idx; g.tile_sched = h->img.d_tile_sched;
  g.uniform_kp = h->img.uniform_kp;
  if (conv) {
    g.row_idx = conv->d_off;
    g.conv_P = conv->geom.P; g.conv_L = conv->geom.L; g.conv_H = conv->geom.H; g.conv_W = conv->geom.W;
  }
  g.zero_cols = h->img.d_zero_cols; g.n_zero = h->img.n_zero;
  g.n_tiles = h->n_tiles; g.K = h->K; g.N = h->N; g.xcd_map = o.xcd_map ? 1 : 0;
  g.meta = h->img.d_meta;
  hipError_t e;
  if (automatic(o) && twg::small_i8_pays(h->G, h->pattern == TW_PATTERN_TVW, M, h->n_tiles, h->max_kp)) {
    e = twg::launch_small_i8(h->G, h->pattern == TW_PATTERN_TVW, h->max_kp, g, (hipStream_t)stream);
    return e == hipSuccess ? TW_OK : TW_ERR_HIP;
  }
  if (h->pattern == TW_PATTERN_TVW) {
    // 64-row tiles where 128-row tiles would not give every CU a workgroup
    const int forced = o.tile_m;
    const long wgs128 = (long)((M + 127) / 128) * (h->n_tiles > 0 ? h->n_tiles : 1);
    const int tm = h->G != 128 ? 128 : (forced == 64 || forced == 128) ? forced : (wgs128 <= 256 ? 64 : 128);
    e = twg::launch_tvw_i8(h->G, tm, g, (hipStream_t)stream);
  } else {
    // long K with too few tiles to fill the chip: split K inside the workgroup (as the fp16 path)
    const int tm = pick_tile_m_i8(o, M, h->n_tiles > 0 ? h->n_tiles : 1, h->G, h->max_kp);
    const int ks = o.ksplit;
    int tmk = tm;
    e = hipErrorInvalidValue;
    // (from 12 stages of 64 rows on: below that the reduction through LDS costs more than it saves)
    if (ks == 2 || (ks == 0 && h->max_kp >= 768 && use_ksplit(M, h->n_tiles, h->G, h->max_kp, 1, &tmk))) {
      if (ks == 2) tmk = tm == 256 ? 128 : tm;
      if (h->G == 64) tmk = 128;
      e = twg::launch_tw_i8(h->G, tmk, 2, g, (hipStream_t)stream);
    }
    if (e == hipErrorInvalidValue) e = twg::launch_tw_i8(h->G, tm, 1, g, (hipStream_t)stream);
  }
  if (e == hipErrorInvalidValue) return TW_ERR_UNSUPPORTED;
  return e == hipSuccess ? TW_OK : TW_ERR_HIP;
}

tw_status tw_gemm_i8(const void* A, int M, int lda, tw_handle_t h, void* C, int ldc, int c_dtype,
                     float scale, void* stream) {
  if (!A || !C || !h || M < 1 || (c_dtype != 0 && c_dtype != 1)) return TW_ERR_ARG;
  if (!aligned16(A) || !aligned16(C) || lda % 16 || ldc % 16 || lda < M || ldc < M) return TW_ERR_ARG;
  if (h->dtype != TW_DTYPE_I8) return TW_ERR_ARG;
  if (!h->img.blob) return TW_ERR_STATE;
  if (h->G == 32 || h->K > 131071) return TW_ERR_UNSUPPORTED;
  if ((unsigned long long)h->K * (unsigned long long)lda >= (1ull << 32)) return TW_ERR_UNSUPPORTED;
  return gemm_i8_launch(A, M, lda, h, C, ldc, c_dtype, scale, stream, nullptr);
}

tw_status tw_conv_gemm_i8(const void* X, tw_conv_t b, void* C, int ldc, int c_dtype, float scale,
                          void* stream) {
  if (!X || !C || !b || !b->h || (c_dtype != 0 && c_dtype != 1)) return TW_ERR_ARG;
  if (b->h->dtype != TW_DTYPE_I8) return TW_ERR_ARG;
  const int Mp = b->geom.B * b->geom.L * b->geom.P;
  if (!aligned16(X) || !aligned16(C) || ldc % 16 || ldc < Mp) return TW_ERR_ARG;
  if (b->h->K > 131071) return TW_ERR_UNSUPPORTED;
  return gemm_i8_launch(X, Mp, 1, b->h, C, ldc, c_dtype, scale, stream, b);
}

tw_status tw_dense_gemm_i8(const void* A, const void* B, void* C, int M, int K, int N, int lda, int ldb,
                           int ldc, int c_dtype, float scale, void* stream) {
  if (!A || !B || !C || M < 1 || K < 1 || N < 1 || (c_dtype != 0 && c_dtype != 1)) return TW_ERR_ARG;
  if (!aligned16(A) || !aligned16(B) || !aligned16(C) || lda % 16 || ldb % 16 || ldc % 16) return TW_ERR_ARG;
  if (ldb < N || lda < M || ldc < M) return TW_ERR_ARG;
  if (K % 64 || K > 131071) return TW_ERR_UNSUPPORTED;
  if ((unsigned long long)K * (unsigned long long)lda >= (1ull << 32) ||
      (unsigned long long)K * (unsigned long long)ldb >= (1ull << 32))
    return TW_ERR_UNSUPPORTED;
  twg::GemmI8Args g{};
  g.A = (const int8_t*)A; g.C = C; g.M = M; g.lda = lda; g.ldc = ldc;
  g.c_i8 = c_dtype; g.scale = scale;
  g.vals = (const int8_t*)B; g.ldb = ldb; g.K = K; g.N = N;
  const int tn = 128;
  g.n_tiles = (N + tn - 1) / tn;
  const Opts o = default_opts();
  g.xcd_map = o.xcd_map ? 1 : 0;
  hipError_t e = twg::launch_dense_i8(tn, pick_tile_m_i8(o, M, g.n_tiles, tn, K), g, (hipStream_t)stream);
  if (e == hipErrorInvalidValue) return TW_ERR_UNSUPPORTED;
  return e == hipSuccess ? TW_OK : TW_ERR_HIP;
}

tw_status tw_export(tw_handle_t h, tw_packed_view* out) {
  if (!h || !out) return TW_ERR_ARG;
  std::memset(out, 0, sizeof(*out));
  const tw_status sf = twg::fetch_logical(h);          // device-packed: lists and values come over now
  if (sf != TW_OK) return sf;
  out->K = h->K; out->N = h->N; out->G = h->G; out->pattern = h->pattern;
  out->n_kept = h->n_kept; out->n_tiles = h->n_tiles; out->dtype = h->dtype;
  out->col_idx = h->col_idx.data(); out->cto_n = h->cto_n.data();
  out->tile_k_off = h->tile_k_off.data(); out->row_idx = h->row_idx.data();
  out->cto_k = h->cto_k.data(); out->val_off = h->val_off.data(); out->values = h->values.data();
  out->tile_col_off = h->tile_col_off.data();
  if (h->pattern == TW_PATTERN_TEW) {
    out->ew_nnz = (int64_t)h->ew_row.size();
    out->ew_col_ptr = h->ew_col_ptr.data(); out->ew_row = h->ew_row.data(); out->ew_val = h->ew_val.data();
  }
  if (h->pattern == TW_PATTERN_TVW) {
    out->meta_off = h->meta_off.data(); out->meta = h->meta.data(); out->valid = h->valid.data();
  }
  return TW_OK;
}

tw_status tw_unpack(tw_handle_t h, uint16_t* Bm, uint8_t* mask) {
  if (!h) return TW_ERR_ARG;
  const tw_status sf = twg::fetch_logical(h);
  if (sf != TW_OK) return sf;
  return twg::unpack_host(h, Bm, mask);
}

tw_status tw_free(tw_handle_t h) {
  if (!h) return TW_OK;
  tw_status st = TW_OK;
  if (h->img.blob && hipFree(h->img.blob) != hipSuccess) st = TW_ERR_HIP;
  delete h;
  return st;
}

tw_status tw_set_option(const char* name, int value) {
  if (!name) return TW_ERR_ARG;
  if (!std::strcmp(name, "tile_m")) { opt_tile_m.store(value); return TW_OK; }
  if (!std::strcmp(name, "xcd_map")) { opt_xcd_map.store(value < 0 || value > 2 ? 1 : value); return TW_OK; }
  if (!std::strcmp(name, "kernel")) { opt_kernel.store(value); return TW_OK; }
  if (!std::strcmp(name, "waves")) { opt_waves.store(value == 8 ? 8 : 4); return TW_OK; }
  if (!std::strcmp(name, "ksplit")) { opt_ksplit.store(value); return TW_OK; }
  if (!std::strcmp(name, "tiles_per_wg")) { opt_tiles_per_wg.store(value < 0 || value > 8 ? 0 : value); return TW_OK; }
  if (!std::strcmp(name, "idx_route")) { opt_idx_route.store(value < 0 || value > 2 ? 0 : value); return TW_OK; }
  if (!std::strcmp(name, "wg_split")) { opt_wg_split.store(value < 0 || value > 8 ? 0 : value); return TW_OK; }
  if (!std::strcmp(name, "tile_order")) { twg::longest_first.store(value != 0); return TW_OK; }
  if (!std::strcmp(name, "depth")) { opt_depth.store(value >= 3 && value <= 8 ? value : 3); return TW_OK; }
  return TW_ERR_ARG;
}

tw_status tw_flop_counts(tw_handle_t h, int64_t* sum_kw, int64_t* sum_k, int64_t* k_union) {
  if (!h) return TW_ERR_ARG;
  if (sum_kw) *sum_kw = h->sum_kw;
  if (sum_k) *sum_k = h->sum_k;
  if (k_union) *k_union = h->k_union;
  return TW_OK;
}

}  // extern "C"
