// TW, TVW and TEW products with few output blocks (one sequence, decoding, small layers): bound by latency.
//
// The pipelined kernels give a workgroup a whole N-tile; a launch of a few dozen such workgroups
// walks its kept rows stage by stage on a quarter of the chip, one barrier and one wait per stage.
// Here a workgroup owns 32 columns of a tile x 32 rows of A, its waves deal the k-steps of the
// kept-row list among themselves, and every wave has all of its loads under way at once:
//   weights : straight into registers (both images are in the register order of the matrix
//             instruction, 1 KiB per k-step and column block);
//   A rows  : 32 elements of each kept row, by asynchronous copies into an LDS area of the wave's own
//             (a k-step is one 1 KiB copy, two with 2:4), read back with the transposing LDS read;
//             32-element rows need no swizzle: a half-wave's read is one whole bank period.
// There is no barrier before the partial sums of the waves meet in LDS; they are added in wave order.
// One round trip for the row list, one for everything else, one barrier: a launch costs about the
// same whatever its K, until the waves hold more than U k-steps each.
//
// Microseconds per launch in a stream of launches, pipelined kernels against this one, K x N:
//   TW 75 %,    M = 128: 768 x 2304 4.1 / 3.2, 768 x 768 4.0 / 2.7, 768 x 3072 4.4 / 3.3, 3072 x 768 7.2 / 4.1
//   TVW 87.5 %, M = 128: 768 x 2304 3.9 / 3.0, 3072 x 768 7.4 / 3.6, 1024 x 4096 4.3 / 3.4
//   TEW 1 ... 1.5 %: 3784 x 1257 at 88 %, M = 11 23.8 / 8.5; 2048 x 512 at 90 %, M = 200 21 / 5.0; 320 x 64, G = 64, M = 59 8.6 / 2.9
//   3 x 3 convolution 512 -> 512 at 14 x 14, one image, TW 75 %, G = 64: 10.8 / 4.7
// 64 rows of A per workgroup (half the weight reads) gained at most 8 %, only next to the line where
// the pipelined kernels take over, and lost up to 30 % elsewhere; 16 waves lost 20 % on short lists.
#include <type_traits>

#include "device_common.h"

namespace twg {

namespace {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef _Float16 half16 __attribute__((ext_vector_type(16)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

template <int OFF>
__device__ __forceinline__ int2v tr_read(uint32_t addr) {
  int2v v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}

}  // namespace

// C^T[col][m] of a TEW weight term by term: the kept rows (row list and weights of the tile from kp0 on, column c), if the
// column is a kept one, and the column's restored elements.  For results that came out infinite or NaN: there the zeros
// of the joined rows must not count.
__device__ __forceinline__ float ew_term_by_term(const GemmArgs& g, int G, int kp0, int kept, int c, int col, int m) {
  float s = 0.f;
  const _Float16* w = g.vals + (size_t)kp0 * G + (c / 32) * 512 + (c % 32) * 8;
#pragma unroll 1
  for (int j = 0; j < kept; ++j)
    s = __builtin_fmaf((float)g.A[(size_t)g.row_idx[kp0 + j] * g.lda + m],
                       (float)w[(size_t)(j / 16) * G * 16 + (j % 16) / 8 * 256 + j % 8], s);
#pragma unroll 1
  for (int e = g.ew_ptr[col]; e < g.ew_ptr[col + 1]; ++e) {
    union { uint16_t b; _Float16 h; } v;
    v.b = (uint16_t)g.ew_pairs[e];
    s = __builtin_fmaf((float)g.A[(size_t)(g.ew_pairs[e] >> 16) * g.lda + m], (float)v.h, s);
  }
  return s;
}

// SP: 2:4 inside the kept rows (TVW).  NW: waves.  U: k-steps of a wave in flight.  EW: restored elements (TEW).
template <bool SP, int NW, int U, bool EW>
__global__ __launch_bounds__(NW * 64) void tw_gemm_small_kernel(GemmArgs g, int G, int n_blocks, int zero_cols_per_wg) {
  constexpr int NT = NW * 64;
  constexpr int KR = SP ? 32 : 16;                  // condensed rows per k-step
  constexpr int NJ = KR / 16;                       // copies per k-step
  constexpr int NQ = SP ? 4 : 2;                    // transposing reads per operand
  constexpr int PITCH = 36;                         // staged partial sums: [n][m] floats
  constexpr int AREA_A = U * NJ * 1024, AREA_P = 32 * PITCH * 4;
  constexpr int AREA = ((AREA_A > AREA_P ? AREA_A : AREA_P) + 1023) / 1024 * 1024;   // LDS of one wave
  __shared__ __attribute__((aligned(1024))) char lds[NW * AREA];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bid = blockIdx.x, n_gemm = n_blocks * g.n_mtiles;
  if (bid >= n_gemm) {                              // +0 into zero_cols_per_wg pruned columns
    const int chunks = (g.M + 7) / 8, z0 = (bid - n_gemm) * zero_cols_per_wg;
    const int n = min(zero_cols_per_wg, g.n_zero - z0) * chunks;
    for (int i = tid; i < n; i += NT) {
      const int z = i / chunks, m = (i - z * chunks) * 8;
      _Float16* dst = g.C + (size_t)g.zero_cols[z0 + z] * g.ldc + m;
      if (m + 8 <= g.M) *(u32x4*)dst = u32x4{0u, 0u, 0u, 0u};
      else for (int e = 0; m + e < g.M; ++e) dst[e] = (_Float16)0.f;
    }
    return;
  }
  // The M-tiles of a column block are 8 ids apart: the same XCD, whose L2 then holds its weights.  With more M-tiles than
  // column blocks, and for the last few of these, an XCD takes a range of M-tiles and all column blocks: A, of which a line
  // of memory serves two M-tiles, then comes once (TVW 75 %, 2304 x 128, M = 3520: 13.3 / 6.7 us; TW 75 %, M = 1600 4.7 / 3.6).
  int nb, mt;
  {
    const int whole = g.n_mtiles > n_blocks ? 0 : n_blocks / 8 * 8, rem = n_blocks - whole;
    if (bid < whole * g.n_mtiles) {
      const int r = bid >> 3, grp = r / g.n_mtiles;
      mt = r - grp * g.n_mtiles;
      nb = grp * 8 + (bid & 7);
    } else {
      const int r = xcd_remap(bid - whole * g.n_mtiles, rem * g.n_mtiles);
      mt = r / rem;
      nb = whole + r - mt * rem;
    }
  }
  const int CB = G / 32;
  int t = nb / CB, kp0, kp, kept = 0;
  const int cb = nb - t * CB;
  if (g.uniform_kp > 0) { kp0 = t * g.uniform_kp; kp = g.uniform_kp; }
  else {
    const int4v rec = *(const int4v*)(g.tile_sched + 4 * t);
    t = rec[0]; kp0 = rec[1]; kp = rec[2]; kept = rec[3];
  }
  const int m0 = mt * 32;
  const int nk = kp / KR;

  constexpr int NI = 512 / NT;      // pairs of results per thread
  int cols[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    cols[i] = g.col_idx[t * G + cb * 32 + (tid + i * NT) / 16];
  }

  const char* Bt = (const char*)g.vals + ((size_t)(kp0 / KR) * CB + cb) * 1024 + lane * 16;
  const uint32_t* It = SP ? g.meta + ((size_t)(kp0 / 64) * CB + cb) * 64 + lane : nullptr;
  const int* rows = g.row_idx + kp0 + (lane >> 2);
  int el = m0 + (lane & 3) * 8;
  if (el >= g.M) el = m0;                           // past M: any chunk (those lanes are never stored)
  const _Float16* Am = g.A + el;
  char* area = lds + wave * AREA;
  const int p = lane & 15, q = lane >> 4;
  const uint32_t fa = (uint32_t)(uintptr_t)LDS_PTR(char, area) + (8 * (q >> 1) + (p >> 2)) * 64 + (16 * (q & 1) + 4 * (p & 3)) * 2;

  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

  // k-steps s0, s0 + NW, .. (CNT of them): loads, one wait, products
  auto chunk = [&](int s0, auto CNT_) {
    constexpr int CNT = decltype(CNT_)::value;
    int r[CNT][NJ];
    int4v b[CNT];
    uint32_t w[CNT];
#pragma unroll
    for (int u = 0; u < CNT; ++u)
#pragma unroll
      for (int j = 0; j < NJ; ++j) r[u][j] = rows[(s0 + u * NW) * KR + j * 16];
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      const int s = s0 + u * NW;
      b[u] = *(const int4v*)(Bt + (size_t)s * (CB * 1024));
      if constexpr (SP) w[u] = It[(size_t)(s >> 1) * (CB * 64)] >> (16 * (s & 1));
    }
#pragma unroll
    for (int u = 0; u < CNT; ++u)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        __builtin_amdgcn_global_load_lds(GLOBAL_PTR(Am + (size_t)(uint32_t)r[u][j] * (uint32_t)g.lda),
                                         LDS_PTR(void, area + (u * NJ + j) * 1024), 16, 0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int2v f[CNT][NQ];
    auto read = [&](auto U_) {
      constexpr int u = decltype(U_)::value;
      if constexpr (u < CNT) {
        constexpr int at = u * NJ * 1024;
        f[u][0] = tr_read<at>(fa);
        f[u][1] = tr_read<at + 4 * 64>(fa);
        if constexpr (SP) {
          f[u][2] = tr_read<at + 16 * 64>(fa);
          f[u][3] = tr_read<at + 20 * 64>(fa);
        }
      }
    };
    read(std::integral_constant<int, 0>{}); read(std::integral_constant<int, 1>{});
    read(std::integral_constant<int, 2>{}); read(std::integral_constant<int, 3>{});
    read(std::integral_constant<int, 4>{}); read(std::integral_constant<int, 5>{});
    read(std::integral_constant<int, 6>{}); read(std::integral_constant<int, 7>{});
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int u = 0; u < CNT; ++u)
#pragma unroll
      for (int k = 0; k < NQ; ++k) asm volatile("" : "+v"(f[u][k]));     // no use above the wait
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      union { int4v i; half8 h; } bv;
      bv.i = b[u];
      if constexpr (SP) {
        union { int2v s[4]; half16 h; } av;
#pragma unroll
        for (int k = 0; k < 4; ++k) av.s[k] = f[u][k];
        acc = __builtin_amdgcn_smfmac_f32_32x32x32_f16(bv.h, av.h, acc, (int)w[u], 0, 0);
      } else {
        union { int2v s[2]; half8 h; } av;
        av.s[0] = f[u][0]; av.s[1] = f[u][1];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(av.h, bv.h, acc, 0, 0, 0);
      }
    }
  };
  int s = wave;
  for (; s + (U - 1) * NW < nk; s += U * NW) chunk(s, std::integral_constant<int, U>{});
  const int left = s < nk ? (nk - s + NW - 1) / NW : 0;           // < U
  auto rest = [&](auto C_) {
    constexpr int C = decltype(C_)::value;
    if constexpr (C < U) { if (left == C) chunk(s, C_); }
  };
  rest(std::integral_constant<int, 1>{}); rest(std::integral_constant<int, 2>{});
  rest(std::integral_constant<int, 3>{}); rest(std::integral_constant<int, 4>{});
  rest(std::integral_constant<int, 5>{}); rest(std::integral_constant<int, 6>{});
  rest(std::integral_constant<int, 7>{});

  // ---- partial sums, [n][m] in the wave's own area.  TW: acc[r] is (m, n) = (8 (r / 4) + 4 (lane / 32)
  // + r % 4, lane % 32) of the block; TVW, whose product is formed transposed, the other way round.
  float* mine = (float*)area;
#pragma unroll
  for (int rq = 0; rq < 4; ++rq) {
    const int x = 8 * rq + 4 * (lane >> 5), y = lane & 31;
    if constexpr (SP) {
#pragma unroll
      for (int k = 0; k < 4; ++k) mine[(x + k) * PITCH + y] = acc[rq * 4 + k];
    } else {
      floatx4 v;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = acc[rq * 4 + k];
      *(floatx4*)(mine + y * PITCH + x) = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int it = tid + i * NT;
    const int n = it / 16, m = m0 + (it % 16) * 2;
    if (cols[i] < 0 || m >= g.M) continue;
    const char* at = lds + (n * PITCH + m - m0) * 4;
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float2v v = *(const float2v*)(at + w * AREA);
      s0 += v[0];
      s1 += v[1];
    }
    if (g.conv_P) {                                 // implicit img2col: the padding lanes of the wide grid are +0
      const uint32_t P = (uint32_t)g.conv_P, L = (uint32_t)g.conv_L, line = (uint32_t)m / P;
      uint32_t x = (uint32_t)m - line * P, y = line % L;
      if (x >= (uint32_t)g.conv_W || y >= (uint32_t)g.conv_H) s0 = 0.f;
      if (++x == P) { x = 0; if (++y == L) y = 0; }
      if (x >= (uint32_t)g.conv_W || y >= (uint32_t)g.conv_H) s1 = 0.f;
    }
    if constexpr (EW) {
      const bool bad0 = !(s0 * 0.f == 0.f), bad1 = m + 1 < g.M && !(s1 * 0.f == 0.f);      // infinite or NaN, and stored
      if (bad0 || bad1) {
        const int c = cb * 32 + n, rows_kept = c < (int)((uint32_t)kept >> 24) ? kept & 0xffffff : 0;
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
          if (!(h ? bad1 : bad0)) continue;
          const float x = ew_term_by_term(g, G, kp0, rows_kept, c, cols[i], m + h);
          if (h == 0) s0 = x;
          else s1 = x;
        }
      }
    }
    _Float16* dst = g.C + (size_t)cols[i] * g.ldc + m;
    if (m + 1 < g.M) *(half2v*)dst = half2v{(_Float16)s0, (_Float16)s1};
    else *dst = (_Float16)s0;
  }
}

template <bool SP, int NW, int U, bool EW = false>
static hipError_t launch_small(int G, GemmArgs& g, hipStream_t stream) {
  g.n_mtiles = (int)(((long)g.M + 31) / 32);
  const int n_blocks = g.n_tiles * (G / 32);
  const int chunks = (g.M + 7) / 8;
  const int zper = chunks < NW * 64 ? NW * 64 / chunks : 1;       // pruned columns per workgroup that clears them
  const int grid = n_blocks * g.n_mtiles + (g.n_zero + zper - 1) / zper;
  if (grid <= 0) return hipSuccess;
  return launch_kernel(tw_gemm_small_kernel<SP, NW, U, EW>, dim3(grid), dim3(NW * 64), stream, g, G, n_blocks, zper);
}

// Waves and k-steps in flight.  TW: 8 waves; 8 k-steps where the lists are longer than 8 x 4 of them
// (3072 x 768 at M = 128: 4.1 against 4.4 us), else 4, which take half the LDS (768 x 3072 at M = 256:
// 4.1 against 4.9).  TVW, k-steps of twice the rows: 4 waves for short lists and for more than two
// workgroups per CU (768 x 3072 at M = 256: 3.5 against 4.6), else 8 (3072 x 768 at M = 128: 3.6
// against 4.4).
hipError_t launch_small_km(int G, bool sparse, bool restored, int max_kp, GemmArgs g, hipStream_t stream) {
  const long blocks = (long)g.n_tiles * (G / 32) * ((g.M + 31) / 32);
  if (sparse) {
    if (max_kp <= 12 * 32 || blocks > 512) return launch_small<true, 4, 4>(G, g, stream);
    return launch_small<true, 8, 4>(G, g, stream);
  }
  if (restored) return max_kp > 8 * 4 * 16 ? launch_small<false, 8, 8, true>(G, g, stream) : launch_small<false, 8, 4, true>(G, g, stream);
  if (max_kp > 8 * 4 * 16) return launch_small<false, 8, 8>(G, g, stream);
  return launch_small<false, 8, 4>(G, g, stream);
}

// Where it beats the pipelined kernels, by the number of 32 x 32 blocks of C and the length of the lists (sweeps over M at some
// forty K x N, G and sparsities, TW and TVW, and eleven convolutions).  TW, this kernel / pipelined.  Short lists, G = 64, whose
// pipelined launches have twice the workgroups: 256 x 256 at 50 %, 256 blocks 3.0 / 3.3 us, 480 blocks 3.5 / 3.4; G = 128:
// 768 x 768 at 87.5 %, 480 blocks 3.4 / 3.8, 648 blocks 3.9 / 3.8.  Medium ones: 768 x 768 at 75 %, 672 blocks 4.0 / 4.4,
// 792 blocks 4.4 / 4.4; 2048 x 1024 at 80 %, 672 blocks 5.6 / 6.1, 800 blocks 6.7 / 6.1.  Long ones, bound by the LDS reads and
// copies again: 3072 x 768, 432 blocks 6.7 / 7.9, 552 blocks 9.1 / 8.2; 4096 x 1024 at 50 %, 448 blocks 12.3 / 15.2, 576 blocks
// 16.7 / 15.4.  TVW: 768 x 768 at 87.5 %, 720 blocks 3.9 / 4.4; 1024 x 1024 at 80 %, 704 blocks 5.1 / 5.7, 800 blocks 5.6 / 5.7;
// 4096 x 1024 at 75 %, 672 blocks 14.7 / 14.6, 800 blocks 18.6 / 14.5.
bool small_km_pays(int G, bool sparse, int M, int n_tiles, int max_kp) {
  const long blocks = (long)n_tiles * (G / 32) * (((long)M + 31) / 32);
  if (sparse && G == 32) return false;              // TVW is not offered for this width at any size
  if (sparse) return blocks <= 704;
  if (max_kp < 12 * 16) return blocks <= (G == 128 ? 480 : 256);
  if (max_kp <= 32 * 16) return blocks <= (G == 128 ? 704 : 576);
  return blocks <= 464;
}

}  // namespace twg
