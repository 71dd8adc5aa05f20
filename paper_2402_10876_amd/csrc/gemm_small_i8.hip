// Int8 TW and TVW products with few output blocks (one sequence, decoding, small layers): bound by latency.
//
// The counterpart of the fp16 kernel for few blocks: a workgroup owns 32 columns of a tile x 32 rows of A, its waves
// deal the k-steps of the kept-row list among themselves, every wave has its loads under way at once, and the int32 sums,
// which are exact in any order, meet in LDS behind the only barrier.
//   A rows  : 32 bytes of each kept row by asynchronous copies into an LDS area of the wave's own (1 KiB = 32 rows: one
//             k-step of TW, half of one with 2:4), read back with the transposing byte read; a half-wave of it reads 8 rows,
//             one whole bank period, so 32-byte rows need no swizzle.
//   weights : TW, stored k-major: copied like A's rows; TVW, in register order: straight into registers.
//
// Microseconds per launch in a stream of launches, pipelined kernels against this one, K x N:
//   TW 75 %,  M = 1: 768 x 2304 6.1 / 2.9, 3072 x 768 5.8 / 3.3;  M = 128: 768 x 2304 5.2 / 3.2, 768 x 768 5.1 / 2.9, 3072 x 768 5.9 / 3.6
//   TVW 75 %, M = 1: 768 x 2304 5.3 / 3.0, 3072 x 768 8.3 / 3.5;  M = 128: 768 x 2304 4.6 / 3.4, 768 x 768 4.5 / 3.0, 3072 x 768 7.5 / 3.9
//   3 x 3 convolutions of one 14 x 14 image, TW 75 %: 256 -> 256 6.8 / 3.6, 512 -> 512, G = 64 8.5 / 4.5
#include <type_traits>

#include "device_common.h"
#include "i8_common.h"
#include "zero_cols.h"

namespace twg {

namespace {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int8v __attribute__((ext_vector_type(8)));

template <int OFF>
__device__ __forceinline__ int2v tr8_read(uint32_t addr) {
  int2v v;
  asm volatile("ds_read_b64_tr_b8 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}

}  // namespace

// SP: 2:4 inside the kept rows (TVW).  NW: waves.  U: k-steps of a wave in flight.  OUT8: requantised output.
template <bool SP, int NW, int U, bool OUT8>
__global__ __launch_bounds__(NW * 64) void tw_gemm_small_i8_kernel(GemmI8Args g, int G, int n_blocks, int zero_cols_per_wg) {
  constexpr int NT = NW * 64;
  constexpr int KR = SP ? 64 : 32;                  // condensed rows per k-step
  constexpr int NJ = KR / 32;                       // copies of A's rows per k-step
  constexpr int NC = SP ? NJ : 2;                   // copies per k-step
  constexpr int NQ = 4;                             // transposing reads per k-step
  constexpr int PITCH = 36;                         // staged partial sums: [n][m] ints
  constexpr int AREA_A = U * NC * 1024, AREA_P = 32 * PITCH * 4;
  constexpr int AREA = ((AREA_A > AREA_P ? AREA_A : AREA_P) + 1023) / 1024 * 1024;   // LDS of one wave
  constexpr int ES = OUT8 ? 1 : 4;
  __shared__ __attribute__((aligned(1024))) char lds[NW * AREA];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bid = blockIdx.x, n_gemm = n_blocks * g.n_mtiles;
  if (bid >= n_gemm) {                              // 0 into zero_cols_per_wg pruned columns
    const int64_t bytes = (int64_t)g.M * ES;
    const int chunks = zero_chunks(bytes), z0 = (bid - n_gemm) * zero_cols_per_wg;
    const int n = min(zero_cols_per_wg, g.n_zero - z0) * chunks;      // (several columns: at most NT chunks)
    for (int i = tid; i < n; i += NT) {
      const ZeroChunk x = zero_chunk(i, chunks);
      char* row = (char*)g.C + (size_t)g.zero_cols[z0 + x.column] * g.ldc * ES;
      if (x.at + 16 <= bytes) *(u32x4*)(row + x.at) = u32x4{0u, 0u, 0u, 0u};
      else for (int64_t e = x.at; e < bytes; ++e) row[e] = 0;
    }
    return;
  }
  // The M-tiles of a column block are 8 ids apart: the same XCD, whose L2 then holds its weights.  With more M-tiles than
  // column blocks, and for the last few of these, an XCD takes a range of M-tiles and all column blocks: A, of which a line
  // of memory serves four M-tiles, then comes once (2000 x 64, G = 64, M = 5120: 7.5 / 4.0 us; 2304 x 128, M = 3520: 6.2 / 5.1).
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
  int t = nb / CB, kp0, kp;
  const int cb = nb - t * CB;
  if (g.uniform_kp > 0) { kp0 = t * g.uniform_kp; kp = g.uniform_kp; }
  else {
    const int4v rec = *(const int4v*)(g.tile_sched + 4 * t);
    t = rec[0]; kp0 = rec[1]; kp = rec[2];
  }
  const int m0 = mt * 32;
  const int nk = kp / KR;

  constexpr int NI = 512 / NT;      // pairs of results per thread
  int cols[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) cols[i] = g.col_idx[t * G + cb * 32 + (tid + i * NT) / 16];

  // TVW: 1 KiB of values, 256 bytes of position words per k-step and column block
  const char* Bt = SP ? (const char*)g.vals + ((size_t)(kp0 / 64) * CB + cb) * 1024 + lane * 16
                      : (const char*)g.vals + ((size_t)kp0 + (lane >> 1)) * G + cb * 32 + (lane & 1) * 16;
  const uint32_t* It = SP ? g.meta + ((size_t)(kp0 / 64) * CB + cb) * 64 + lane : nullptr;
  const int* rows = g.row_idx + kp0 + (lane >> 1);
  int el = m0 + (lane & 1) * 16;
  if (el >= g.M) el = m0;                           // past M: any chunk (those lanes are never stored)
  const int8_t* Am = g.A + el;
  char* area = lds + wave * AREA;
  const int p = lane & 15, q = lane >> 4;
  const uint32_t fa = (uint32_t)(uintptr_t)LDS_PTR(char, area) + (16 * (q >> 1) + (p >> 1)) * 32 + 16 * (q & 1) + 8 * (p & 1);

  intx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0;

  // k-steps s0, s0 + NW, .. (CNT of them): loads, one wait, products
  auto chunk = [&](int s0, auto CNT_) {
    constexpr int CNT = decltype(CNT_)::value;
    int r[CNT][NJ];
    int4v b[CNT];
    int w[CNT];
#pragma unroll
    for (int u = 0; u < CNT; ++u)
#pragma unroll
      for (int j = 0; j < NJ; ++j) r[u][j] = rows[(s0 + u * NW) * KR + j * 32];
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      const int s = s0 + u * NW;
      if constexpr (SP) {
        b[u] = *(const int4v*)(Bt + (size_t)s * (CB * 1024));
        w[u] = (int)It[(size_t)s * (CB * 64)];
      } else {
        __builtin_amdgcn_global_load_lds(GLOBAL_PTR(Bt + (size_t)s * (32 * G)), LDS_PTR(void, area + (2 * u + 1) * 1024), 16, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < CNT; ++u)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        __builtin_amdgcn_global_load_lds(GLOBAL_PTR(Am + (size_t)(uint32_t)r[u][j] * (uint32_t)g.lda),
                                         LDS_PTR(void, area + (2 * u + j) * 1024), 16, 0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int2v f[CNT][NQ];
    auto read = [&](auto U_) {
      constexpr int u = decltype(U_)::value;
      if constexpr (u < CNT) {
        constexpr int at = u * 2048;
        f[u][0] = tr8_read<at>(fa);
        f[u][1] = tr8_read<at + 8 * 32>(fa);
        f[u][2] = tr8_read<at + 1024>(fa);          // (TVW: rows 32 on; TW: the weights)
        f[u][3] = tr8_read<at + 1024 + 8 * 32>(fa);
      }
    };
    read(std::integral_constant<int, 0>{}); read(std::integral_constant<int, 1>{});
    read(std::integral_constant<int, 2>{}); read(std::integral_constant<int, 3>{});
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int u = 0; u < CNT; ++u)
#pragma unroll
      for (int k = 0; k < NQ; ++k) asm volatile("" : "+v"(f[u][k]));     // no use above the wait
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      if constexpr (SP) {
        union { int2v s[4]; int8v h; } av;
#pragma unroll
        for (int k = 0; k < 4; ++k) av.s[k] = f[u][k];
        acc = __builtin_amdgcn_smfmac_i32_32x32x64_i8(b[u], av.h, acc, w[u], 0, 0);
      } else {
        union { int2v s[2]; int4v h; } av, bv;
        av.s[0] = f[u][0]; av.s[1] = f[u][1];
        bv.s[0] = f[u][2]; bv.s[1] = f[u][3];
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(av.h, bv.h, acc, 0, 0, 0);
      }
    }
  };
  static_assert(U == 4, "");
  int s = wave;
  for (; s + (U - 1) * NW < nk; s += U * NW) chunk(s, std::integral_constant<int, U>{});
  const int left = s < nk ? (nk - s + NW - 1) / NW : 0;           // < U
  if (left == 1) chunk(s, std::integral_constant<int, 1>{});
  if (left == 2) chunk(s, std::integral_constant<int, 2>{});
  if (left == 3) chunk(s, std::integral_constant<int, 3>{});

  // ---- partial sums, [n][m] in the wave's own area.  TW: acc[r] is (m, n) = (8 (r / 4) + 4 (lane / 32)
  // + r % 4, lane % 32) of the block; TVW, whose product is formed transposed, the other way round.
  int* mine = (int*)area;
#pragma unroll
  for (int rq = 0; rq < 4; ++rq) {
    const int x = 8 * rq + 4 * (lane >> 5), y = lane & 31;
    if constexpr (SP) {
#pragma unroll
      for (int k = 0; k < 4; ++k) mine[(x + k) * PITCH + y] = acc[rq * 4 + k];
    } else {
      int4v v;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = acc[rq * 4 + k];
      *(int4v*)(mine + y * PITCH + x) = v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int it = tid + i * NT;
    const int n = it / 16, m = m0 + (it % 16) * 2;
    if (cols[i] < 0 || m >= g.M) continue;
    const char* at = lds + (n * PITCH + m - m0) * 4;
    int2v v = *(const int2v*)at;
#pragma unroll
    for (int w = 1; w < NW; ++w) v += *(const int2v*)(at + w * AREA);
    if (g.conv_P) {                                 // implicit img2col: the padding lanes of the wide grid are 0
      const uint32_t P = (uint32_t)g.conv_P, L = (uint32_t)g.conv_L, line = (uint32_t)m / P;
      uint32_t x = (uint32_t)m - line * P, y = line % L;
      if (x >= (uint32_t)g.conv_W || y >= (uint32_t)g.conv_H) v[0] = 0;
      if (++x == P) { x = 0; if (++y == L) y = 0; }
      if (x >= (uint32_t)g.conv_W || y >= (uint32_t)g.conv_H) v[1] = 0;
    }
    const size_t to = (size_t)cols[i] * g.ldc + m;
    if constexpr (OUT8) {
      const int lo = requantize(v[0], g.scale), hi = requantize(v[1], g.scale);
      if (m + 1 < g.M) *(uint16_t*)((int8_t*)g.C + to) = (uint16_t)((lo & 0xff) | (hi & 0xff) << 8);
      else ((int8_t*)g.C)[to] = (int8_t)lo;
    } else {
      if (m + 1 < g.M) *(int2v*)((int*)g.C + to) = v;
      else ((int*)g.C)[to] = v[0];
    }
  }
}

template <bool SP, int NW>
static hipError_t launch_small8(int G, GemmI8Args& g, hipStream_t stream) {
  g.n_mtiles = (int)(((long)g.M + 31) / 32);
  const int n_blocks = g.n_tiles * (G / 32);
  const int chunks = zero_chunks((int64_t)g.M * (g.c_i8 ? 1 : 4));
  const int zper = chunks < NW * 64 ? NW * 64 / chunks : 1;       // pruned columns per workgroup that clears them
  const int grid = n_blocks * g.n_mtiles + (g.n_zero + zper - 1) / zper;
  if (grid <= 0) return hipSuccess;
  if (g.c_i8) return launch_kernel(tw_gemm_small_i8_kernel<SP, NW, 4, true>, dim3(grid), dim3(NW * 64), stream, g, G, n_blocks, zper);
  return launch_kernel(tw_gemm_small_i8_kernel<SP, NW, 4, false>, dim3(grid), dim3(NW * 64), stream, g, G, n_blocks, zper);
}

// Four waves hold 512 kept rows at once (TVW: 1024), eight twice that and one workgroup less per CU: 768 x 2304, M = 256 3.8 / 4.7 us with
// four / eight (TVW 4.1 / 4.9), 3072 x 768, M = 1 3.5 / 3.3 (3.7 / 3.5); TVW lists between 512 and 1024 rows gain up to 10 % from eight.
hipError_t launch_small_i8(int G, bool sparse, int max_kp, GemmI8Args g, hipStream_t stream) {
  const bool four = max_kp <= 512;
  if (sparse) return four ? launch_small8<true, 4>(G, g, stream) : launch_small8<true, 8>(G, g, stream);
  return four ? launch_small8<false, 4>(G, g, stream) : launch_small8<false, 8>(G, g, stream);
}

// Where it beats the pipelined kernels, by the number of 32 x 32 blocks of C and the length of the lists (sweeps over M at
// seventeen K x N, G and sparsities, TW and TVW).  TW, this kernel / pipelined: up to 512 rows 768 x 768 at 75 %, 768
// blocks 4.3 / 5.3 us, 2048 x 1024 at 80 %, 672 blocks 5.6 / 6.3, 800 blocks 6.2 / 6.2, 768 x 2304, 1088 blocks 5.3 / 4.6; up to
// 768 rows 4096 x 4096 at 87.5 %, 464 blocks 5.4 / 6.5, 1024 x 512 at 50 %, G = 64, 560 blocks 5.7 / 5.4; up to 1024 rows
// 3840 x 576 at 80 %, 320 blocks 5.1 / 5.6, 640 blocks 9.0 / 6.0; longer 4096 x 1024 at 50 %, 192 blocks 7.3 / 9.5, 320 blocks
// 11.2 / 10.1.  TVW, half the weights per row: up to 512 rows 768 x 1536 at 80 %, 660 blocks 4.1 / 4.3, 792 blocks 4.3 / 4.3;
// longer 1024 x 1024 at 75 %, 448 blocks 4.1 / 4.8, 576 blocks 5.3 / 4.9, 4096 x 1024, 448 blocks 8.4 / 9.5, 576 blocks 11.6 / 9.7.
bool small_i8_pays(int G, bool sparse, int M, int n_tiles, int max_kp) {
  const long blocks = (long)n_tiles * (G / 32) * (((long)M + 31) / 32);
  if (max_kp <= 512) return blocks <= 704;
  if (sparse || max_kp <= 768) return blocks <= 480;
  return blocks <= (max_kp <= 1024 ? 352 : 256);
}

}  // namespace twg
