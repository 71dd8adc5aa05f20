// Grouped TW kernel for row-major activations and outputs (TW_LAYOUT_MK): A is M x K, C is M x N.
//
// In this layout a kept row of a tile is a column of A: gathering it from memory would take 2-byte
// accesses.  So a workgroup copies a band of A (64 or 32 rows x up to 768 columns) as it lies, 16 bytes
// per lane, turns it round on the way into LDS (8 x 8 blocks, in registers), and gathers from
// there: the band is stored k-major, 128 (64) bytes per k, and the transposing LDS read takes an
// address per lane, so that the four k rows a 16-lane group reads are any four rows of the band.
// The band is read from memory once per workgroup and serves all N-tiles of that workgroup.
//
//   slots   : 8 waves of 64 (32) x 32 (m x n) each; G / 32 waves make a slot that owns one N-tile, so
//             2 (G = 128), 4 (64) or 8 (32) tiles run side by side on the same band.
//   weights : every wave loads its own 32 columns straight into registers (the packed image is in
//             the register order of the matrix instruction), PF k-steps ahead and on into the next
//             tile: the K loop has no barrier, and 64 KiB or more per CU are in flight.
//   long K  : bands of 512 (768) columns one after the other, the next one's loads in flight while this
//             one is multiplied; the k-steps around the end of a band run in both, with the other
//             band's rows pointing at a row of zeros (CAREFUL: and their weights set to zero, for 0 x Inf is not 0).
//   output  : staged in LDS over the range of original columns that the tiles side by side answer
//             for, pruned ones as +0, and stored in whole 16-byte pieces of C's rows; a piece at
//             the end of the range that belongs to two workgroups is stored element by element.
//
// What bounds it: with one workgroup of 8 waves per CU the phases of a group do not overlap.  768 x 2304 at M = 4096, 75 %,
// by timestamps: the first band 3.8 us, then per group of two tiles the K loop 2.0 to 2.6 us (1.3 to 1.7 without the next
// tile's loads, which share the CU's 64 bytes a clock), 0.3 to 0.9 waiting for the slowest wave, staging 0.45, stores 0.55 to
// 0.85.  75 %, M = 4096, K x N: 768 x 2304 17.2 us, 768 x 768 8.8, 768 x 3072 18.7, 3072 x 768 20.2.
// Tried on that and not kept: staging condensed columns and reading them back with the transposing read (17.4, fewer LDS
// instructions, no faster), stores through a buffer descriptor whose number the compiler can count (18.6 with it), reads of
// the rows two k-steps ahead (17.3), 12 k-steps of weights in flight for a long K (3072 x 768 21.9), two bands on their
// way (26.3).
#include <type_traits>

#include "device_common.h"
#include "mk_band.h"

namespace twg {

namespace {

constexpr uint32_t MK_ZERO = MK_KC;    // row of zeros behind the band
constexpr int MK_NW = 8, MK_NT = MK_NW * 64;

// LDS offset of row k of the band: rows of TM * 2 bytes, and 16 bytes more after every 8 of them.  The 8 x 8 blocks are
// written with k = 8 kc + j, one j at a time for consecutive kc, which the 16 bytes spread evenly over the banks; the
// rows that a read gathers are any rows, so no order would help it.  Two instructions, for the K loop was bound by
// their number: with rows and chunks permuted by exclusive-or (eleven, 21 of vector arithmetic per k-step in all) 75 %, M =
// 4096 took 18.5 us for 768 x 2304, now 17.2; 768 x 768 9.4, 8.8; 768 x 3072 20.0, 18.7; 3072 x 768 22.2, 20.2.
template <int TM>
constexpr __device__ __forceinline__ uint32_t mk_row(uint32_t k) { return ((k & 0xffffffu) * (TM * 2 + 2)) & ~15u; }   // (24-bit multiply)

__device__ __forceinline__ half8 mk_operand(const char* lo, const char* hi) {
  union { short4v s[2]; half8 h; } u;
  u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4v, lo));
  u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4v, hi));
  return u.h;
}

}  // namespace

// LONG: K in several bands.  One band needs no registers for the next one, and PF = 14 k-steps hold
// a whole tile of 75 % sparsity at K = 768: its products then wait for no load, and the stores of the
// tiles before drain meanwhile.  CAREFUL: for rows of A too far apart for 32-bit offsets and for weights with
// infinities (or NaN) among them.  In every instance the wider sums and the masked weights would cost 5 to 14 %
// of the launches with several bands (3072 x 768 at M = 4096 24.5 / 25.6 us, at M = 1000 16.9 / 19.3).
template <int G, bool LONG, int TM, bool CAREFUL>
__global__ __launch_bounds__(MK_NT, TM == 32 ? 4 : 2) void tw_gemm_mk_kernel(GemmArgs g, int groups, int parts, int per_part, int kc_max) {
  constexpr int SW = G / 32;                        // waves per slot
  constexpr int SLOTS = MK_NW / SW;
  constexpr int NM = TM / 32;                       // blocks of 32 rows
  constexpr int KB = MK_KB<TM>;                     // columns of A a wave turns round at a time
  constexpr int A_BYTES = (int)mk_row<TM>(MK_ZERO) + TM * 2;        // LDS bytes of the band, the row of zeros the last
  constexpr int RW = TM / MK_NW;                    // rows of C a wave stores
  constexpr int PF = TM == 32 ? 6 : LONG ? 8 : 14;                 // k-steps of weights and kept rows in flight
  // output staging: 64 rows of 368 columns (256 kept ones and the pruned ones between them, usually);
  // 4 rows further on is half a bank period, so that the two halves of a wave do not collide
  constexpr int SEG = 368, PITCH = SEG * 2;
  __shared__ __attribute__((aligned(1024))) char lds[A_BYTES + TM * PITCH];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slot = wave / SW, sw = wave % SW;       // slot, wave inside the slot
  const int total = g.n_mtiles * parts;
  const int lid = g.xcd_map ? xcd_remap(blockIdx.x, total) : (int)blockIdx.x;
  const int mt = lid / parts, part = lid - mt * parts;
  const int m0 = mt * TM;
  const int gr0 = part * per_part, gr_n = min(groups - gr0, per_part);
  const int bands = LONG ? (g.K + kc_max - 1) / kc_max : 1;
  // the bands of an XCD start on different groups: weights come from memory once per XCD, and
  // workgroups in step on the same group would all wait for the same few of them
  auto group_of = [&](int i) { return gr0 + (i + mt) % gr_n; };

  // ---- band of A: global rows as they lie -> k-major LDS rows ----------------------------------
  // lane = (m block mg of 8 rows, chunk kc of 8 columns); a wave turns TM x KB round per step
  // (wave-uniform base, byte offset per lane)
  const int kc = lane % (KB / 8), mg = lane / (KB / 8);
  const char* A_band = (const char*)(g.A + (size_t)m0 * g.lda);
  const int m_last = min(TM, g.M - m0) - 1;
  auto load_block = [&](int k0, int kb, u32x4 (&v)[8]) {
    const int kg = mk_chunk<TM>(k0, kb, kc, g.K);   // (never past K, whatever lda is: A may be a slice of wider rows)
#pragma unroll
    for (int i = 0; i < 8; ++i)                     // rows past M: never stored
      v[i] = *(const u32x4*)(A_band + mk_offset<CAREFUL>(min(mg * 8 + i, m_last), g.lda, kg));
  };
  auto store_block = [&](int kb, const u32x4 (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
      u32x4 w;
#pragma unroll
      for (int d = 0; d < 4; ++d) w[d] = __builtin_amdgcn_perm(v[2 * d + 1][j >> 1], v[2 * d][j >> 1], sel);
      *(u32x4*)(lds + mk_row<TM>((uint32_t)(kb * KB + kc * 8)) + mg * 16 + j * (TM * 2)) = w;
    }
  };
  char* stg = lds + A_BYTES;

  // ---- this wave's operands --------------------------------------------------------------------
  const int p = lane & 15, q = lane >> 4;
  const int frow = 8 * (q >> 1) + (p >> 2);
  const uint32_t xa = (uint32_t)(16 * (q & 1) + 4 * (p & 3)) * 2;             // byte inside a band row, block 0

  half8 b[PF];
  int r[PF];
  // lanes 2i and 2i+1 of a group of four need the same two kept rows, frow and frow + 4: each
  // loads one of them and they swap
  const uint32_t b_lane = (uint32_t)(sw * 64 + lane) * 16u, r_lane = (uint32_t)(frow + 4 * (p & 1)) * 4u;
  struct Tile {                                     // (wave-uniform)
    const char* B;                                  // weights
    const int* rows;                                // kept rows
    int nk;                                         // k-steps
    int c_lo, c_hi;                                 // original columns its group answers for
  };
  auto fetch = [&](const Tile& t, int s, int u) {   // k-step s (clamped by the caller) -> set u
    b[u] = *(const half8*)(t.B + (size_t)s * (G * 32) + b_lane);
    r[u] = *(const int*)((const char*)(t.rows + s * 16) + r_lane);
  };
  // Offsets and first columns of the tiles of a group, a lane each (the lane behind the last slot
  // has the next group's first tile), by vector loads: scalar loads return out of order, so the K
  // loop's first wait for LDS would wait for them too.  Two groups ahead of their use.
  int hv_kp, hv_c;
  auto load_head = [&](int gr) {
    const int t = min(gr * SLOTS + lane, g.n_tiles);
    hv_kp = g.tile_kp_off[t];
    hv_c = g.col_idx[min(t, g.n_tiles - 1) * G];
  };
  // a group's columns reach from its first kept one (the first group: from column 0) to the next
  // group's (the last group: to column N)
  auto tile_of = [&](int gr) {
    Tile t;
    const int kp0 = __builtin_amdgcn_readlane(hv_kp, slot), kp1 = __builtin_amdgcn_readlane(hv_kp, slot + 1);
    t.nk = (kp1 - kp0) / 16;                        // (0 past the last tile)
    t.B = (const char*)(g.vals + (size_t)kp0 * G);
    t.rows = g.row_idx + kp0;                       // (readable past the last tile's list)
    t.c_lo = gr == 0 ? 0 : __builtin_amdgcn_readlane(hv_c, 0);
    t.c_hi = (gr + 1) * SLOTS < g.n_tiles ? __builtin_amdgcn_readlane(hv_c, SLOTS) : g.N;
    return t;
  };
  auto load_col = [&](int gr) {                     // the kept column of this lane
    const int t = gr * SLOTS + slot;
    const int c = g.col_idx[min(t, g.n_tiles - 1) * G + sw * 32 + (lane & 31)];
    return t < g.n_tiles ? c : -1;
  };
  constexpr int NFIRST = LONG ? 4 : 1;              // first rows of the k-steps, for the ends of the bands
  int first[NFIRST];
  auto load_first = [&](const Tile& t) {
    if constexpr (LONG) {
#pragma unroll
      for (int i = 0; i < NFIRST; ++i) first[i] = t.rows[max(0, min(64 * i + lane, t.nk - 1)) * 16];
    }
  };

  floatx16 acc[NM];
  u32x4 v0[8];
  load_head(group_of(0));
  load_block(0, wave, v0);
  Tile cur;
  int col;
  {
    u32x4 v1[8];
    const bool two = TM == 64 && !LONG && g.K > 512 + wave * 64;
    if (two) load_block(0, wave + 8, v1);
    cur = tile_of(group_of(0));
    load_first(cur);
    col = load_col(group_of(0));
#pragma unroll
    for (int u = 0; u < PF; ++u) fetch(cur, u < cur.nk ? u : 0, u);
    load_head(group_of(gr_n > 1 ? 1 : 0));
    for (int i = tid; i < TM * PITCH / 16; i += MK_NT) *(u32x4*)(stg + i * 16) = u32x4{0u, 0u, 0u, 0u};
    if (tid < TM / 8) *(u32x4*)(lds + mk_row<TM>(MK_ZERO) + tid * 16) = u32x4{0u, 0u, 0u, 0u};
    if (wave * KB < (LONG ? kc_max : MK_KC)) store_block(wave, v0);
    if (two) store_block(wave + 8, v1);
  }
  __syncthreads();

  for (int i = 0; i < gr_n; ++i) {
    const bool has_next = !LONG && i + 1 < gr_n;    // (LONG: one group per workgroup)
    const int gr_next = group_of(has_next ? i + 1 : i);
    const Tile next = tile_of(gr_next);
#pragma unroll
    for (int j = 0; j < NM; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[j][k] = 0.f;

    // a k-step belongs to the band if its first row lies below the band's end; set u holds k-step
    // s + u throughout, so the last round of a band is the first of the next
    int s = 0;
    u32x4 left = {0u, 0u, 0u, 0u};
    for (int band = 0; band < bands; ++band) {
      const int k0 = LONG ? band * kc_max : 0, kn = LONG ? min(g.K - k0, kc_max) : g.K;
      const bool more = LONG && band + 1 < bands;
      int s1 = cur.nk;
      if constexpr (LONG) {
        if (more) load_block(k0 + kc_max, wave, v0);
        s1 = 0;
#pragma unroll
        for (int j = 0; j < NFIRST; ++j) s1 += __popcll(__ballot(64 * j + lane < cur.nk && first[j] < k0 + kn));
        for (int b0 = NFIRST * 64; b0 < cur.nk; b0 += 64) {
          const int ss = b0 + lane;
          s1 += __popcll(__ballot(ss < cur.nk && cur.rows[min(ss, cur.nk - 1) * 16] < k0 + kn));
        }
        s1 = __builtin_amdgcn_readfirstlane(s1);
      }
      // operands of a k-step: rows of the other bands read the row of zeros
      auto operands = [&](int u, half8 (&a)[NM]) {
        const uint32_t k = (uint32_t)(r[u] - k0);
        const int row = (int)mk_row<TM>(!LONG || k < (uint32_t)kn ? k : MK_ZERO);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp(row, 0xA0, 0xf, 0xf, false) + xa;   // lanes 0,0,2,2 of each four
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp(row, 0xF5, 0xf, 0xf, false) + xa;   // lanes 1,1,3,3
        a[0] = mk_operand(lds + lo, lds + hi);
        if constexpr (NM == 2) a[1] = mk_operand(lds + lo + 64, lds + hi + 64);
      };
      auto multiply = [&](int u, const half8 (&a)[NM]) {
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[u], acc[0], 0, 0, 0);
        if constexpr (NM == 2) acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[u], acc[1], 0, 0, 0);
      };
      // The reads of k-step u+1 are issued ahead of the products of k-step u.  Whole rounds of PF
      // refill the sets as they go; the tile's last (shorter) round fills them with the next tile's.
      half8 a[2][NM];
      if (s < s1) operands(0, a[0]);
      for (; s + PF < s1; s += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          operands((u + 1) % PF, a[(u + 1) & 1]);
          multiply(u, a[u & 1]);
          fetch(cur, min(s + u + PF, cur.nk - 1), u);
        }
      }
      // CAREFUL: the band's last k-step, which its end may cut: its 16 rows ascend, and the weights of those past
      // the band, a suffix, are left for the bands behind it
      auto cut_weights = [&](int u) {
        constexpr unsigned long long ONCE = 0x0000333300003333ull;     // lanes that hold each of the rows once
        const int ours = __popcll(__ballot(r[u] < k0 + kn) & ONCE) - 8 * (lane >> 5);   // (of the lane's 8 weights)
        union { half8 h; u32x4 w; } x;
        x.h = b[u];
        left = x.w;
#pragma unroll
        for (int d = 0; d < 4; ++d)
          x.w[d] &= (2 * d < ours ? 0x0000ffffu : 0u) | (2 * d + 1 < ours ? 0xffff0000u : 0u);
        left ^= x.w;
        b[u] = x.h;
      };
      auto last_round = [&](auto FILL) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          if (s + u < s1) {
            const bool end = LONG && CAREFUL && s + u == s1 - 1;
            if (end) cut_weights(u);
            if (u + 1 < PF) operands(u + 1, a[(u + 1) & 1]);
            multiply(u, a[u & 1]);
            if constexpr (LONG && CAREFUL) {        // what the next band, which runs this round again, may count
              union { half8 h; u32x4 w; } x;
#pragma unroll
              for (int d = 0; d < 4; ++d) x.w[d] = end ? left[d] : 0u;
              b[u] = x.h;
            }
          }
          if constexpr (decltype(FILL)::value) fetch(next, u < next.nk ? u : 0, u);
        }
      };
      if (has_next && band + 1 == bands) last_round(std::true_type{});
      else last_round(std::false_type{});
      if constexpr (LONG) {
        __syncthreads();                            // everybody is done with the band
        if (more && wave * KB < kc_max) store_block(wave, v0);
        __syncthreads();
      }
    }
    // ---- epilogue: acc[i][r] is C[m0 + 32 i + 8 (r / 4) + 4 (lane / 32) + r % 4][col] ------------
    const int lo0 = cur.c_lo, hi0 = cur.c_hi, my_col = col;
    cur = next;
    if (has_next) {
      col = load_col(gr_next);
      load_head(group_of(i + 2 < gr_n ? i + 2 : i + 1));
    }
    for (int c0 = lo0 & ~7; c0 < hi0; c0 += SEG) {
      __syncthreads();                              // the staging area has been read and is zero again
      const int cl = my_col - c0;
      if (my_col >= 0 && cl >= 0 && cl < SEG) {
#pragma unroll
        for (int i = 0; i < NM; ++i)
#pragma unroll
          for (int k = 0; k < 16; ++k) {
            const int mm = i * 32 + 8 * (k >> 2) + 4 * (lane >> 5) + (k & 3);
            *(_Float16*)(stg + mm * PITCH + cl * 2) = (_Float16)acc[i][k];
          }
      }
      __syncthreads();
      // the next group's loads land ahead of the stores, whose acknowledgements the first k-steps
      // would otherwise wait for (one in-order counter)
      if constexpr (!LONG) {
#pragma unroll
        for (int u = 0; u < PF; ++u) asm volatile("" : "+v"(b[u]), "+v"(r[u]));
        asm volatile("" : "+v"(col), "+v"(hv_kp), "+v"(hv_c));
      }
      const int lo = max(lo0, c0), hi = min(hi0, c0 + SEG);           // columns of this segment that are ours
      const int f0 = (lo + 7) & ~7, f1 = max(hi & ~7, f0);            // its whole 16-byte pieces
      const int ch = (f0 - c0) / 8 + lane;
      const u32x4 zero = {0u, 0u, 0u, 0u};
      if (f0 + lane * 8 < f1) {                     // a wave stores RW rows, one at a time
        u32x4 v[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) v[i] = *(const u32x4*)(stg + (wave * RW + i) * PITCH + ch * 16);
#pragma unroll
        for (int i = 0; i < RW; ++i) *(u32x4*)(stg + (wave * RW + i) * PITCH + ch * 16) = zero;
        _Float16* dst = g.C + (size_t)(m0 + wave * RW) * g.ldc + c0 + ch * 8;
#pragma unroll
        for (int i = 0; i < RW; ++i)
          if (m0 + wave * RW + i < g.M) *(u32x4*)(dst + (size_t)i * g.ldc) = v[i];
      }
      // the ends: wave 0 the piece that lo cuts, wave 1 the piece that hi cuts, a lane per row
      if (wave < 2) {
        const int cc = wave == 0 ? lo & ~7 : hi & ~7;
        const bool cut = wave == 0 ? (lo & 7) != 0 : (hi & 7) != 0 && (hi & ~7) >= f0;
        if (cut && lane < TM) {
          u32x4* at = (u32x4*)(stg + lane * PITCH + (cc - c0) * 2);
          const u32x4 v = *at;
          *at = zero;
          uint16_t* dst = (uint16_t*)(g.C + (size_t)(m0 + lane) * g.ldc + cc);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (m0 + lane < g.M && cc + e >= lo && cc + e < hi) dst[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
      }
    }
  }
}

// A weight without a single kept column: C is all +0.
static __global__ void zero_mk(_Float16* C, int M, int N, int ldc) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  for (int m = blockIdx.y; m < M; m += gridDim.y) C[(size_t)m * ldc + n] = (_Float16)0.f;
}

template <int G, int TM, bool CAREFUL = false>
static hipError_t launch_mk(GemmArgs& g, hipStream_t stream) {
  constexpr int SLOTS = MK_NW / (G / 32);
  constexpr int RESIDENT = TM == 32 ? 512 : 256;         // workgroups the chip holds at once
  g.n_mtiles = (g.M + TM - 1) / TM;
  const int groups = (g.n_tiles + SLOTS - 1) / SLOTS;    // SLOTS tiles side by side
  int parts = (RESIDENT + g.n_mtiles - 1) / g.n_mtiles;
  if (g.K > MK_KC || parts > groups) parts = groups;     // (K in several bands: a group each)
  const int per = (groups + parts - 1) / parts;
  parts = (groups + per - 1) / per;
  const dim3 grid((unsigned)(g.n_mtiles * parts));
  if (g.K > MK_KC)
    return launch_kernel(tw_gemm_mk_kernel<G, true, TM, CAREFUL>, grid, dim3(MK_NT), stream, g, groups, parts, per, MK_KC_LONG<TM>);
  return launch_kernel(tw_gemm_mk_kernel<G, false, TM, CAREFUL>, grid, dim3(MK_NT), stream, g, groups, parts, per, MK_KC);
}

// Rows of a band.  32: twice the workgroups, two per CU, which overlap their phases and give few blocks
// a CU each, but read every weight twice as often.  They win where 64-row bands would leave half of
// the CUs idle, and where the lists are short (band 64 / 32): 768 x 768 at 75 %, 128 of the larger blocks 10.6 / 8.5 us, 256
// 12.3 / 14.1; 768 x 2304, 120 blocks 10.8 / 8.7, 160 11.1 / 12.8; 3072 x 768, 128 blocks 25.1 / 24.2, 256 27.6 / 41.0; 2000 x
// 1500 with G = 64, 96 blocks 20.1 / 18.7, 144 20.4 / 29.9; lists of 96 rows: 768 x 3072, 640 blocks 18.2 / 16.6, 768 x 2304 with
// G = 64, 256 blocks 9.5 / 8.9; of 128 rows 18.5 / 20.1, 640 blocks.  Where the rule is wrong: two bands of K and many column
// groups (1024 x 4096 at 50 %, 48 blocks 13.4 / 16.0), a last round that is nearly empty (768 x 3072, 288 blocks 20.2 / 17.9).
template <int G>
static hipError_t launch_mk_rows(int max_kp, bool nonfinite, GemmArgs& g, hipStream_t stream) {
  constexpr int SLOTS = MK_NW / (G / 32);
  const long blocks64 = (long)((g.M + 63) / 64) * ((g.n_tiles + SLOTS - 1) / SLOTS);
  if (g.lda > MK_LDA_32 || (nonfinite && g.K > MK_KC)) return launch_mk<G, 32, true>(g, stream);
  if (blocks64 <= 128 || (g.K <= MK_KC && max_kp <= 96)) return launch_mk<G, 32>(g, stream);
  return launch_mk<G, 64>(g, stream);
}

hipError_t launch_tw_mk(int G, int max_kp, bool nonfinite, GemmArgs g, hipStream_t stream) {
  if (g.n_tiles == 0)
    return launch_kernel(zero_mk, dim3((g.N + 255) / 256, g.M < 1024 ? g.M : 1024), dim3(256), stream, g.C, g.M, g.N, g.ldc);
  if (G == 128) return launch_mk_rows<128>(max_kp, nonfinite, g, stream);
  if (G == 64) return launch_mk_rows<64>(max_kp, nonfinite, g, stream);
  if (G == 32) return launch_mk_rows<32>(max_kp, nonfinite, g, stream);
  return hipErrorInvalidValue;
}

}  // namespace twg
