// Grouped TW kernel / dense baseline, asynchronous-copy pipeline for gfx950.
//
// Same decomposition and layouts as the register-staged kernel (one workgroup
// per (M-tile, N-tile) pair, Listing 1; A is K x M and C is N x M, Section V
// "Memory Accesses Coalesce"), but the stage copies never pass through
// registers: every wave issues global_load_lds_dwordx4, which moves 64 x 16
// bytes from per-lane global addresses straight into 1 KiB of LDS.  D stages
// of 32 condensed rows are in flight per workgroup; the only synchronisation
// per stage is one vmcnt wait and one s_barrier.
//
//   gather  : lane l of a copy instruction fetches one 16-byte chunk of row
//             row_idx[...] of A (Listing 1: CTO_k).
//   LDS     : k-major tiles of A (and of the dense baseline's B), 64-byte units
//             XOR-swizzled (see swz_mask); the swizzle is applied on the global
//             side, the LDS side of a copy instruction is always 1 KiB contiguous.
//             A packed weight is stored in the register order of the matrix
//             instruction (see the packer) and copied as it lies: one 16-byte
//             LDS read per operand instead of two transposing ones (1-2 % of
//             every TW launch: 8192 x 1024 x 4096 and 8192 x 4096 x 1024 at 50 %
//             together 91.0 -> 89.4 us, a BERT-base layer at 75 % 39.0 -> 38.4).
//   MFMA    : operands come from ds_read_b64_tr_b16 issued from inline
//             assembly.  The compiler orders every LDS read it knows about
//             behind all earlier asynchronous copies (vmcnt(0)), which would
//             serialise the pipeline; reads it cannot see are ordered by the
//             explicit waits written here instead.
//   overlap : the MFMAs of the second half of stage s are issued after the
//             barrier and the operand reads of stage s+1, so LDS latency is
//             hidden behind matrix-core work.
#include <type_traits>

#include "device_common.h"

namespace twg {

namespace {

typedef int int4v __attribute__((ext_vector_type(4)));

template <int OFF>
__device__ __forceinline__ int2v tr_read(uint32_t addr) {
  int2v v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}

// One matrix-core operand (32 x-values x 16 k) = two transposed 64-bit reads.
struct Frag { int2v lo, hi; };

__device__ __forceinline__ half8 as_half8(const Frag& f) {
  union { int2v s[2]; half8 h; } u;
  u.s[0] = f.lo; u.s[1] = f.hi;
  return u.h;
}
// The same operand where the tile is stored in the matrix core's register order.
template <int OFF>
__device__ __forceinline__ int4v read128(uint32_t addr) {
  int4v v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
__device__ __forceinline__ half8 as_half8(const int4v& f) {
  union { int4v s; half8 h; } u;
  u.s = f;
  return u.h;
}

// s_waitcnt tied to the fragments so that no use can be moved above it: MB blocks of A, NB of B.
__device__ __forceinline__ void tie(Frag& f) { asm volatile("" : "+v"(f.lo), "+v"(f.hi)); }
__device__ __forceinline__ void tie(int4v& f) { asm volatile("" : "+v"(f)); }
template <int MB, int NB, class FB>
__device__ __forceinline__ void wait_lds(Frag* a, FB* b) {
  asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
  for (int i = 0; i < MB; ++i) tie(a[i]);
#pragma unroll
  for (int j = 0; j < NB; ++j) tie(b[j]);
}

// Wave-uniform 16-byte record through the scalar cache, complete on return.
__device__ __forceinline__ int4v scalar_load4(const void* p) {
  int4v r;
  asm volatile("s_load_dwordx4 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(p));
  return r;
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// row * lda in 32 bits.  OPAQUE: as an instruction of its own: the compiler's 64-bit multiply-add takes
// a register pair as addend whose unused half may be one that a load is on its way to, which the
// check of the split loads would have to tell from a real use.
template <bool OPAQUE>
__device__ __forceinline__ uint32_t row_offset(int row, uint32_t lda) {
  if constexpr (!OPAQUE) return (uint32_t)row * lda;
  uint32_t r;
  asm("v_mul_lo_u32 %0, %1, %2" : "=v"(r) : "v"(row), "s"(lda));
  return r;
}

// Waits until at most `newer` stages of NPS copies each are outstanding (newer <= MAXN; in the
// steady state newer == MAXN and the first comparison decides).
template <int NPS, int MAXN>
__device__ __forceinline__ void wait_stage(int newer) {
  if constexpr (MAXN == 0) wait_vm<0>();
  else {
    if (newer >= MAXN) wait_vm<MAXN * NPS>();
    else wait_stage<NPS, MAXN - 1>(newer);
  }
}

}  // namespace

// KSPLIT = 2: the workgroup has two groups of waves that own the same output
// tile; a pipeline stage then holds 64 condensed rows, group g multiplies rows
// 32g..32g+31 of it, and the two partial accumulators are added through LDS
// (in fp32, before the single rounding).  It gives a tile two waves per SIMD,
// which long-K problems with few tiles need to keep the matrix cores busy.

// ---- TEW: restored elements (Section III-A "TEW").  The rows that hold any in a tile's columns have joined the tile's
// list (see the packer) and are multiplied by the matrix cores with the rest: 1.5 % restored elements are in 85 % of the
// rows of a 128-column tile, 1.9 in a row, and reading those rows once through the pipeline costs half of what the
// elements cost one by one (256 bytes of A each, lists of different length side by side).  From HBM, M = 4096, 75 %:
// 768 x 3072 with 0.5 / 1.5 / 3 % restored 23.8 / 34.8 / 49.8 -> 19.3 / 23.3 / 24.1 us, 3072 x 768 22.4 / 34.6 / 52.3 ->
// 21.6 / 27.0 / 28.0.  What bounds it now: what bounds a TW launch of that many rows.
// A zero of a joined row is not a term of the product, though, and an infinity of A would make it one: a workgroup whose
// sums are not all finite starts again with the kept rows alone and adds the restored elements one by one, as the CSC part
// has them, to the fp32 sums of the thread that stores the 8 values C^T[col][m .. m+8): for every restored (k, v) of the
// column, s += v * A^T[k][m .. m+8).  EW_ELEMENTS does that at once, for lists of many joined rows with few elements each (the
// host's rule has the figures).  Pairs travel as k << 16 | fp16 bits; the list is padded in registers with (row 0, +0).  A rows
// are lda >= round-up-8(M) halves long, so the 16-byte read at m < M stays inside the row.
// P columns at a time (P times the loads in flight per round trip), U elements of each; the next ones are fetched meanwhile.
// Every load is unconditional (index clamped to the list, value selected afterwards): one under a branch would be waited
// for on its own.
template <int P, int U>
__device__ __forceinline__ void ew_accumulate(const GemmArgs& g, const int (&lo)[P], const int (&hi)[P],
                                              const _Float16* A_m, float (&s)[P][8]) {
  int e[P];
  uint32_t nx[P][U];
  bool more = false;
  auto fetch = [&](int p) {
    more |= e[p] < hi[p];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t w = g.ew_pairs[min(e[p] + u, g.ew_last)];
      nx[p][u] = e[p] + u < hi[p] ? w : 0u;
    }
  };
#pragma unroll
  for (int p = 0; p < P; ++p) { e[p] = lo[p]; fetch(p); }
  while (more) {
    uint32_t w[P][U];
    half8 a[P][U];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        w[p][u] = nx[p][u];
        a[p][u] = *(const half8*)(A_m + (size_t)(w[p][u] >> 16) * g.lda);
      }
    more = false;
#pragma unroll
    for (int p = 0; p < P; ++p) { e[p] += U; fetch(p); }
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        union { uint16_t b; _Float16 h; } cv;
        cv.b = (uint16_t)(w[p][u] & 0xffffu);
        const float v = (float)cv.h;
#pragma unroll
        for (int q = 0; q < 8; ++q) s[p][q] = __builtin_fmaf(v, (float)a[p][u][q], s[p][q]);
      }
  }
}

__device__ __forceinline__ void store_row_chunk(const GemmArgs& g, _Float16* dst, int m, const float (&s)[8]) {
  half8 h;
#pragma unroll
  for (int q = 0; q < 8; ++q) h[q] = (_Float16)s[q];
  if (m + 8 <= g.M) __builtin_nontemporal_store(h, (half8*)dst);
  else for (int q = 0; m + q < g.M; ++q) dst[q] = h[q];
}

// SPLIT: K split across workgroups.  g.wg_split workgroups own the same (M-tile, N-tile) pair,
// each a contiguous share of the tile's stages; every one writes its fp32 partial tile to the
// workspace and takes a ticket at the pair's counter; the one that arrives last adds all partial
// tiles in split order (so the sum does not depend on who was last), runs the epilogue and puts
// the counter back to zero.  Nobody waits for anybody: a workgroup that is not last is done.
// MULTI: a workgroup computes g.tiles_per_wg jobs one after the other (job ids blockIdx.x,
// + gridDim.x, ..; gridDim.x is a multiple of 8, so every job keeps the workgroup's XCD).  The
// next job's first copies are issued as soon as every wave has read its staged chunks: the
// stores of the finished tile drain while the next one loads (the copies' waits count the
// stores as older operations, which only makes them wait longer).  Per job the kernel
// arguments are read again through a pointer the compiler cannot see through and the lane id is
// made opaque, so that nothing derived from them stays in registers across jobs.
template <int TM, int TN, int WAVES_M, int D, bool DENSE, int NWAVES = 4, int KSPLIT = 1, int EW = EW_NONE,
          bool SPLIT = false, bool MULTI = false, bool SCALAR = false>
// (TEW's second way to the result, the loop over jobs and the rows in flight must not cost an instance a wave per
// SIMD: the second launch-bound asks the compiler to keep the register count within that occupancy)
__global__ __launch_bounds__(NWAVES * 64, ((MULTI && TM * TN <= 64 * 128) || (!DENSE && KSPLIT == 1 && NWAVES == 8 && TM == 256)) ? 4 : ((EW || MULTI) && TM <= 128 && TN <= 128 && NWAVES == 4) ? 3 : 1)
void tw_gemm_km_dma_kernel(GemmArgs g_arg) {
  constexpr bool LIDX = D > 3;             // how the kept-row list reaches the lanes (see fetch_rows)
  static_assert(!SCALAR || (!LIDX && !DENSE && KSPLIT == 1), "");
  // The products of a stage's two k-steps under a branch that is always taken: it keeps the compiler from
  // mixing them into the operand reads, which two to three workgroups per CU prefer (768 x 3072 at M =
  // 4096 13.9 -> 11.8 us, 1500 x 3000 at 80 % 14.5 -> 14.1, 768 x 2304 in a stream of layers 10.8 -> 10.2); not the
  // 256 x 64 tiles of convolutions (16.6 / 16.9).
  constexpr bool BRANCH = SCALAR && TM == 128;
  constexpr int NT = NWAVES * 64;          // threads of the workgroup
  constexpr int WPG = NWAVES / KSPLIT;     // waves per group
  constexpr int KSS = KS * KSPLIT;         // condensed rows per pipeline stage
  constexpr int WAVES_N = WPG / WAVES_M;
  constexpr int WM = TM / WAVES_M, WN = TN / WAVES_N;
  constexpr int MB = WM / 32, NB = WN / 32;
  static_assert(MB >= 1 && NB >= 1, "wave tile must hold a 32x32 block");
  constexpr int RBA = TM * 2, RBB = TN * 2;            // LDS row bytes
  constexpr int STAGE_A = KSS * RBA, STAGE_B = KSS * RBB, STAGE = STAGE_A + STAGE_B;
  static_assert(STAGE_A % 4096 == 0 && STAGE_B % 4096 == 0, "a stage is a whole number of 1 KiB copies per wave");
  static_assert(STAGE_A % (1024 * NWAVES) == 0 && STAGE_B % (1024 * NWAVES) == 0, "");
  constexpr int NIA = STAGE_A / (1024 * NWAVES), NIB = STAGE_B / (1024 * NWAVES);   // copy instructions per wave and stage
  constexpr int RPIA = 1024 / RBA, RPIB = 1024 / RBB;         // tile rows per copy instruction
  static_assert((RPIA == 2 || RPIA == 4 || RPIA == 8) && (NIA == 1 || NIA == 2 || NIA == 4), "");
  static_assert(D >= 3 && D <= 8, "stages in flight");
  constexpr int NPS = NIA + NIB;
  constexpr int CA = TM / 8;
  // epilogue row bytes: fp16, 66 dwords mod 64 banks = 2; with restored elements to add one by one the
  // tile is staged in fp32, half at a time, so that their products join the sum before the one rounding
  constexpr int CS = (TM + 4) * 2, CS32 = (TM + 4) * 4;
  static_assert(!(EW && DENSE), "");
  constexpr int PIPE_BYTES = D * STAGE, EPI_BYTES = TN * CS;
  static_assert(!EW || TN / 2 * CS32 <= EPI_BYTES, "");
  constexpr int RED_BYTES = KSPLIT > 1 ? TM * TN * 4 : 0;      // partial accumulators of group 1
  static_assert(RED_BYTES <= PIPE_BYTES, "the reduction reuses the pipeline buffers");
  // kept-row lists travel through LDS as well: a ring of two chunks of 8 stages' indices behind
  // the pipeline buffers (the epilogue staging reuses the pipeline buffers only)
  constexpr int CH = 8 * KSS;                              // indices per chunk
  constexpr int NCI = CH * 4 / 1024;                       // 1 KiB copy instructions per chunk
  static_assert(NCI >= 1 && NCI <= NWAVES && CH * 4 % 1024 == 0, "");
  constexpr int MAIN_BYTES = PIPE_BYTES > EPI_BYTES ? PIPE_BYTES : EPI_BYTES;
  constexpr int IDX_OFF = (MAIN_BYTES + 1023) / 1024 * 1024;
  constexpr int LDS_BYTES = IDX_OFF + ((DENSE || !LIDX) ? 0 : 2 * CH * 4);
  __shared__ __attribute__((aligned(1024))) char lds[LDS_BYTES];

  static_assert(!SPLIT || (!DENSE && !EW && KSPLIT == 1), "the split across workgroups exists for plain TW");
  static_assert(!MULTI || (!DENSE && !EW && !SPLIT && KSPLIT == 1), "several jobs per workgroup exist for plain TW");
  auto job = [&](const GemmArgs& g, const int bid, const int tid) {
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = SPLIT ? g.wg_split : 1;
  const int n_gemm = g.n_mtiles * g.n_tiles * S;
  if (bid >= n_gemm) {
    zero_fill_column(g, bid - n_gemm);
    return;
  }
  int mt, t;                             // t: launch position of the tile, then the tile itself
  int pair = 0, split = 0;
  if constexpr (SPLIT) {
    // the workgroups of a pair are neighbours in the XCD's contiguous range of logical ids:
    // they run on the same XCD at about the same time, and their partial tiles meet in its L2
    const int lid = g.xcd_map ? xcd_remap(bid, n_gemm) : bid;
    pair = lid / S;
    split = lid - pair * S;
    mt = pair / g.n_tiles;
    t = pair - mt * g.n_tiles;
  } else {
    tile_of_workgroup(g, bid, n_gemm, mt, t);
  }
  const int m0 = mt * TM;

  int kp0, ns32;                                       // ns32: stages of 32 rows
  int ns32_kept = 0, w_kept = 0;                       // TEW: of these, stages of kept rows (joined rows follow); kept columns
  if constexpr (DENSE) { kp0 = 0; ns32 = g.K / KS; }   // host guarantees K % (32 KSPLIT) == 0
  else {
    // equal tiles in column order (the usual per-tile pruning recipe): the record follows from
    // the launch position, which saves the first of the kernel's dependent round trips
    if (g.uniform_kp > 0) { kp0 = t * g.uniform_kp; ns32 = ns32_kept = g.uniform_kp / KS; }
    else {
      const int4v rec = scalar_load4(g.tile_sched + 4 * t);
      t = rec[0]; kp0 = rec[1]; ns32 = rec[2] / KS;
      ns32_kept = (rec[3] & 0xffffff) / KS;
      w_kept = (int)((uint32_t)rec[3] >> 24);
      if constexpr (EW == EW_ELEMENTS) ns32 = ns32_kept;
    }
  }
  if constexpr (SPLIT) {                               // this workgroup's share of the stages
    const int first = ns32 * split / S, last = ns32 * (split + 1) / S;
    kp0 += first * KS;
    ns32 = last - first;
  }
  int ns = (ns32 + KSPLIT - 1) / KSPLIT;               // pipeline stages of KSS rows
  const _Float16* Bt = DENSE ? g.vals + (size_t)t * TN : g.vals + (size_t)kp0 * TN;
  const int ldb = DENSE ? g.ldb : TN;

  // kept-column indices of the rows of C^T this thread will store (CTO_n)
  constexpr int ROWS_PER_PASS = NT / CA;
  constexpr int NPASS = TN / ROWS_PER_PASS;
  const int c = tid % CA, r0 = tid / CA;
  int cols[NPASS];
#pragma unroll
  for (int i = 0; i < NPASS; ++i) {
    const int n = r0 + i * ROWS_PER_PASS;
    if constexpr (DENSE) { cols[i] = t * TN + n; if (cols[i] >= g.N) cols[i] = -1; }
    else cols[i] = g.col_idx[t * TN + n];
  }
  // ---- geometry of the asynchronous copies --------------------------------
  // Copy instruction j of this wave fills LDS bytes [(wave*NI + j) KiB, +1 KiB)
  // of the stage; lane l owns the 16 bytes at l*16, i.e. tile row
  // (wave*NI + j)*RPI + l*16/RB at physical byte (l*16) % RB, which holds the
  // logical bytes physical ^ swz_mask(row).
  const int lb = lane * 16;
  const int a_rloc = lb / RBA, b_rloc = lb / RBB;
  int a_el[NIA], b_el[NIB];
#pragma unroll
  for (int j = 0; j < NIA; ++j) {
    const int row = (wave * NIA + j) * RPIA + a_rloc;
    a_el[j] = ((lb % RBA) ^ swz_mask<RBA>(row)) / 2;
    if (m0 + a_el[j] >= g.M) a_el[j] = 0;   // past M: re-read chunk 0 (those lanes are never stored)
  }
#pragma unroll
  for (int j = 0; j < NIB; ++j) {
    const int row = (wave * NIB + j) * RPIB + b_rloc;
    b_el[j] = ((lb % RBB) ^ swz_mask<RBB>(row)) / 2;
    if constexpr (DENSE) { if (t * TN + b_el[j] >= g.N) b_el[j] = 0; }
    else b_el[j] = (lb % RBB) / 2;            // the packed image is copied as it lies
  }
  // Addresses are a wave-uniform base plus an unsigned 32-bit byte offset per
  // lane (the host checks that A fits): one multiply-add per copy instruction.
  const char* Abase = (const char*)(g.A + m0);
  const char* Bbase = (const char*)Bt;
  const uint32_t lda2 = (uint32_t)g.lda * 2u, ldb2 = (uint32_t)ldb * 2u;
  uint32_t b_off[NIB];
#pragma unroll
  for (int j = 0; j < NIB; ++j)
    b_off[j] = (uint32_t)((wave * NIB + j) * RPIB + b_rloc) * ldb2 + (uint32_t)b_el[j] * 2u;

  // Row indices (Listing 1: CTO_k), one per lane and copy instruction, three ways:
  // LIDX: through LDS.  Chunk c of a tile's kept-row list (8 stages' worth) is copied into
  //   half c % 2 of a small ring by the same asynchronous copies as the operand tiles, so it
  //   is tracked by the same in-order counter and has landed, at no extra wait, long before
  //   its first stage is issued; every lane then picks the index of the row it copies with
  //   one ds_read_b32 per copy instruction, waited for with the first operand reads.
  // SCALAR: by scalar loads of the RPIA consecutive entries a copy instruction covers, the lane
  //   selects its own; waited for with the first operand reads of the stage.
  // else (three stages in flight): by one vector load per stage, two iterations ahead of its use
  //   and right ahead of the copies of the stage before: the wait for those copies, by the
  //   in-order counter, has it in at no extra cost.  The four lanes of a quad copy from the same
  //   row; lane j of the quad loads the index for copy instruction j and the quad shares it.
  //   Measured against the LDS ring (few workgroups per CU) and scalar loads (many): 8192 x 4096 x
  //   1024 44.8 -> 40.2 us at 50 %, 2048 x 768 x 3072 at 60 % 9.5 -> 8.5, 4096 x 1024 x 2048 with 64-wide
  //   tiles 14.5 -> 12.6.  Where two to three 128 x 128 workgroups share a CU and all are resident,
  //   their waves hide the scalar loads' round trip and the vector load, one more request to the
  //   copy unit per stage, costs more than it saves (the host's rule has the figures).
  typedef int sidx_t __attribute__((ext_vector_type(RPIA)));
  struct Rows { std::conditional_t<SCALAR, sidx_t, int> r[NIA]; };
  static_assert(LIDX || D == 3 || DENSE, "a deeper pipeline would wait for its index loads");
  const uint32_t idx_lds0 = (uint32_t)(uintptr_t)LDS_PTR(char, lds) + IDX_OFF;
  const uint32_t idx_lane = (uint32_t)((wave * NIA + (lane & (NIA - 1))) * RPIA + a_rloc) * 4u;
  auto issue_chunk = [&](int c) {        // waves 0 .. NCI-1: 1 KiB of the list each
    if constexpr (!DENSE && LIDX) {
      if (wave < NCI)
        __builtin_amdgcn_global_load_lds(GLOBAL_PTR((const char*)(g.row_idx + kp0) + ((size_t)c * CH * 4 + wave * 1024 + lb)),
                                         LDS_PTR(void, lds + IDX_OFF + (c & 1) * (CH * 4) + wave * 1024), 16, 0, 0);
    }
  };
  auto fetch_rows = [&](int s, Rows& dst) {      // LIDX, SCALAR: rows of stage s; valid after the next lgkmcnt(0) wait
    if constexpr (SCALAR) {
#pragma unroll
      for (int j = 0; j < NIA; ++j) {
        const int* rp = g.row_idx + kp0 + s * KSS + (wave * NIA + j) * RPIA;
        if constexpr (RPIA == 2) asm volatile("s_load_dwordx2 %0, %1, 0x0" : "=s"(dst.r[j]) : "s"(rp));
        else if constexpr (RPIA == 4) asm volatile("s_load_dwordx4 %0, %1, 0x0" : "=s"(dst.r[j]) : "s"(rp));
        else asm volatile("s_load_dwordx8 %0, %1, 0x0" : "=s"(dst.r[j]) : "s"(rp));
      }
    } else if constexpr (!DENSE && LIDX) {
#pragma unroll
      for (int j = 0; j < NIA; ++j) {
        const uint32_t pos = (uint32_t)(s * KSS + (wave * NIA + j) * RPIA + a_rloc) & (2 * CH - 1);
        asm volatile("ds_read_b32 %0, %1" : "=v"(dst.r[j]) : "v"(idx_lds0 + pos * 4));
      }
    }
  };
  // (the address must not come from a vector instruction within five wait states: a spilled one would; the build checks it)
  auto fetch_quad = [&](int s, int& dst) {       // else: of the quad; valid once the load has been waited for
    if constexpr (!DENSE && !LIDX && !SCALAR)
      asm volatile("global_load_dword %0, %1, %2" : "=v"(dst) : "v"(idx_lane), "s"(g.row_idx + kp0 + s * KSS));
  };
  auto share_quad = [&](int& src, Rows& dst) {   // (instructions of their own, behind the wait for the load)
    if constexpr (!SCALAR) {
    asm volatile("s_nop 1\n\tv_mov_b32_dpp %0, %1 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf" : "=v"(dst.r[0]) : "v"(src));
    if constexpr (NIA > 1) asm volatile("v_mov_b32_dpp %0, %1 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf" : "=v"(dst.r[1]) : "v"(src));
    if constexpr (NIA > 2) asm volatile("v_mov_b32_dpp %0, %1 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf" : "=v"(dst.r[2]) : "v"(src));
    if constexpr (NIA > 2) asm volatile("v_mov_b32_dpp %0, %1 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf" : "=v"(dst.r[3]) : "v"(src));
    }
  };
  auto tie_rows = [&](Rows& x) {      // after a wait: no use of x may be moved above this point
    if constexpr (SCALAR) {
#pragma unroll
      for (int j = 0; j < NIA; ++j) asm volatile("" : "+s"(x.r[j]));
    } else if constexpr (!DENSE) {
#pragma unroll
      for (int j = 0; j < NIA; ++j) asm volatile("" : "+v"(x.r[j]));
    }
  };
  auto issue = [&](int s, const Rows& rows) {     // copies of stage s; rows = its kept-row indices
    char* dstA = lds + (s % D) * STAGE;
    char* dstB = dstA + STAGE_A;
    const uint32_t bs = (uint32_t)s * (uint32_t)KSS * ldb2;
#pragma unroll
    for (int j = 0; j < NIB; ++j)
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(Bbase + (bs + b_off[j])),
                                       LDS_PTR(void, dstB + (wave * NIB + j) * 1024), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < NIA; ++j) {
      int row;
      if constexpr (DENSE) row = s * KSS + (wave * NIA + j) * RPIA + a_rloc;
      else if constexpr (SCALAR) {
        row = rows.r[j][0];
#pragma unroll
        for (int q = 1; q < RPIA; ++q) row = (a_rloc == q) ? rows.r[j][q] : row;
      } else row = rows.r[j];
      __builtin_amdgcn_global_load_lds(GLOBAL_PTR(Abase + (row_offset<!DENSE && !LIDX && !SCALAR>(row, lda2) + (uint32_t)a_el[j] * 2u)),
                                       LDS_PTR(void, dstA + (wave * NIA + j) * 1024), 16, 0, 0);
    }
  };

  floatx16 acc[MB][NB];
  const int grp = wave / WPG, wl = wave % WPG;         // K-split group, wave inside the group
  const int wm = wl % WAVES_M, wn = wl / WAVES_M;
  // per-lane LDS byte address of each operand block at stage buffer 0, k-step 0
  const uint32_t lds0 = (uint32_t)(uintptr_t)LDS_PTR(char, lds);
  const int p = lane & 15, q = lane >> 4;
  const int frow = 8 * (q >> 1) + (p >> 2);
  uint32_t fa[MB], fb[NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
    fa[i] = lds0 + grp * (KS * RBA) + swz<RBA>(frow, (wm * WM + i * 32 + 16 * (q & 1) + 4 * (p & 3)) * 2);
#pragma unroll
  for (int j = 0; j < NB; ++j)
    fb[j] = lds0 + STAGE_A + grp * (KS * RBB) +
            (DENSE ? swz<RBB>(frow, (wn * WN + j * 32 + 16 * (q & 1) + 4 * (p & 3)) * 2) : (wn * NB + j) * 1024 + lane * 16);

  // operands of k-steps 0 and 1 of a stage; a packed weight is stored in register order (one
  // 16-byte read per lane), the dense baseline's B needs the transposing reads
  struct Ops { Frag a[MB]; std::conditional_t<DENSE, Frag, int4v> b[NB]; };
  Ops f0, f1;
  auto read_step = [&](uint32_t boff, auto KK_, Ops& f) {
    constexpr int KK = decltype(KK_)::value;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      f.a[i].lo = tr_read<KK * RBA>(fa[i] + boff);
      f.a[i].hi = tr_read<(KK + 4) * RBA>(fa[i] + boff);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if constexpr (DENSE) {
        f.b[j].lo = tr_read<KK * RBB>(fb[j] + boff);
        f.b[j].hi = tr_read<(KK + 4) * RBB>(fb[j] + boff);
      } else {
        f.b[j] = read128<KK * RBB>(fb[j] + boff);
      }
    }
  };
  auto mfma_step = [&](const Ops& f) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_half8(f.a[i]), as_half8(f.b[j]), acc[i][j], 0, 0, 0);
  };
  using K0 = std::integral_constant<int, 0>;
  using K16 = std::integral_constant<int, 16>;

  // EW_JOINED: once with the joined rows, and, if that came out infinite or NaN anywhere in the tile, again with the kept rows
  // alone and the restored elements one by one: a zero of a joined row times an infinity of A is no part of the product.
  bool joined = EW == EW_JOINED;
  for (;;) {
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  bool live_prev = false;
  // What an iteration does once stage s is in LDS: `cur` are the rows of stage s+D-1.
  auto consume = [&](int s, const Rows& cur, auto after_first_reads) {
    const uint32_t boff = (uint32_t)((s % D) * STAGE);
    read_step(boff, K0{}, f0);
    if (KSPLIT == 1 && !BRANCH ? s > 0 : live_prev) mfma_step(f1);   // second k-step of the previous stage
    // false only for group 1 on an odd tail (BRANCH: always true, and a branch all the same)
    const bool live = (KSPLIT == 1 && !BRANCH) || s * KSPLIT + grp < ns32;
    wait_lds<MB, NB>(f0.a, f0.b);
    after_first_reads();
    // the copies of stage sn = s+D-1 go into the buffer of stage s-1, which every wave has
    // finished reading; LIDX: when sn opens chunk c >= 1 of the list, chunk c+1 follows it into the
    // half of the ring whose last reader (stage 8c-1, two iterations ago) is behind this barrier
    const int sn = s + D - 1;
    if (sn < ns) {
      issue(sn, cur);
      if (LIDX && (sn & 7) == 0 && sn >= 8 && sn + 8 < ns) issue_chunk((sn >> 3) + 1);
    }
    read_step(boff, K16{}, f1);
    if (live) mfma_step(f0);
    live_prev = live;
    wait_lds<MB, NB>(f1.a, f1.b);
  };
  if constexpr (LIDX || DENSE || SCALAR) {
    Rows rows_cur, rows_next;            // of the next stage to copy and of the one after
    if (ns > 0) {
      // (LIDX: the first two chunks of the kept-row list,) the indices of the first D stages in
      // one round trip, then the copies of D-1 stages
      issue_chunk(0);
      if (ns > 8) issue_chunk(1);
      Rows pro[D];
      if constexpr (!DENSE && LIDX) {
        wait_vm<0>();
        asm volatile("s_barrier" ::: "memory");
      }
#pragma unroll
      for (int d = 0; d < D; ++d) fetch_rows(d < ns ? d : ns - 1, pro[d]);
      if constexpr (!DENSE) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int d = 0; d < D; ++d) tie_rows(pro[d]);
#pragma unroll
      for (int d = 0; d < D - 1; ++d)
        if (d < ns) issue(d, pro[d]);
      rows_cur = pro[D - 1];
    }
    for (int s = 0; s < ns; ++s) {
      // own copies of stage s have landed: at most the copies of the newer stages remain
      // (a wave that also copies list chunks waits for one copy more at times: harmless)
      int newer = ns - 1 - s;
      if (newer > D - 2) newer = D - 2;
      wait_stage<NPS, D - 2>(newer);
      // everybody's copies of stage s have landed, everybody is done reading stage s-1
      asm volatile("s_barrier" ::: "memory");
      // rows of stage s+D: needed by the next iteration, so that the addresses of its copies
      // can be formed ahead of the wait that completes this fetch
      fetch_rows(s + D < ns ? s + D : ns - 1, rows_next);
      consume(s, rows_cur, [&] { tie_rows(rows_next); });      // (the full wait has the index fetch in)
      rows_cur = rows_next;
    }
  } else {
    // Two row fetches in flight, in two registers by turns (iterations in pairs, a single one last if
    // their number is odd), because no register may be copied while its load is under way.
    static_assert(LIDX || DENSE || D == 3, "");
    int even, odd;
    auto iteration = [&](int s, int& q, auto LAST) {   // q: rows of stage s+2; receives those of stage s+4
      constexpr bool last = decltype(LAST)::value;     // the tile's last stage
      // own copies of stage s and the rows of stage s+2, issued ahead of them, have landed: newer are
      // the rows of stage s+3 and the copies of stage s+1
      if (!last && s + 3 < ns) wait_vm<NPS + 1>();
      else if (!last && s + 1 < ns) wait_vm<NPS>();
      else wait_vm<0>();
      Rows cur;
      if constexpr (!last) share_quad(q, cur);
      // everybody's copies of stage s have landed, everybody is done reading stage s-1
      asm volatile("s_barrier" ::: "memory");
      // (behind the operand reads: a copy unit with its queue full would hold them up)
      consume(s, cur, [&] { if (!last && s + 4 < ns) fetch_quad(s + 4, q); });
    };
    if (ns > 0) {
      int q0, q1;
      fetch_quad(0, q0);
      fetch_quad(ns > 1 ? 1 : 0, q1);
      fetch_quad(ns > 2 ? 2 : 0, even);
      wait_vm<0>();
      Rows r0, r1;
      share_quad(q0, r0);
      share_quad(q1, r1);
      issue(0, r0);
      if (ns > 1) {                        // (a single stage has no use for them: nothing may be under way then)
        fetch_quad(ns > 3 ? 3 : 0, odd);
        issue(1, r1);
      }
      int s = 0;
      for (; s + 1 < ns; s += 2) {
        iteration(s, even, std::false_type{});
        iteration(s + 1, odd, std::false_type{});
      }
      wait_vm<0>();                      // (nothing is under way, or the copies of the last stage, needed next)
      if (s < ns) iteration(s, even, std::true_type{});
    }
    wait_vm<0>();                        // (nothing is outstanding: every copy has been waited for)
  }
  if (KSPLIT == 1 && !BRANCH ? ns > 0 : live_prev) mfma_step(f1);
  if constexpr (EW == EW_JOINED) {
    if (joined) {                                      // (uniform over the workgroup)
      // NaN unless everything that is stored is finite (rows past M come from the padding of A, which may hold anything)
      float z = 0.f;
      int m_lane = m0 + wm * WM + 4 * (lane >> 5);
      // (otherwise the comparisons move to the kernel's start and their masks push the scalar registers of the K loop out)
      asm volatile("" : "+v"(m_lane));
      auto look = [&](auto WHOLE) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            if (!decltype(WHOLE)::value && m_lane + i * 32 + 8 * (r / 4) + r % 4 >= g.M) continue;
#pragma unroll
            for (int j = 0; j < NB; ++j) z = __builtin_fmaf(acc[i][j][r], 0.f, z);
          }
      };
      if (m0 + TM <= g.M) look(std::true_type{});
      else look(std::false_type{});
      const bool bad = __any(!(z == 0.f));
      __syncthreads();                                 // everybody is done with the pipeline buffers
      if (lane == 0) ((int*)lds)[wave] = bad;
      __syncthreads();
      int any = 0;
#pragma unroll
      for (int w = 0; w < NWAVES; ++w) any |= ((const int*)lds)[w];
      if (any) {
        joined = false;
        ns32 = ns32_kept;
        ns = (ns32 + KSPLIT - 1) / KSPLIT;
        __syncthreads();                               // everybody has read the flags
        continue;
      }
    }
  }
  break;
  }

  if constexpr (SPLIT) {
    if (S > 1) {
      __shared__ int ticket;
      constexpr int TILE = TM * TN;                       // floats per partial tile
      // partial tile as [wave][block][register][lane]: every store instruction of a wave is 256
      // contiguous bytes
      float* tile0 = g.ws_partials + (size_t)pair * S * TILE + wave * (MB * NB * 16 * 64) + lane;
      float* mine = tile0 + (size_t)split * TILE;
      // Partial tiles travel as device-scope relaxed atomic stores and loads: each access is
      // performed at the level that is coherent across the XCDs' L2 caches, so no cache-wide
      // write-back or invalidate is needed (a device-scope fence costs one of each per
      // workgroup and made the launch several times slower).  Order: own stores complete
      // (vmcnt), the workgroup's waves meet, then the ticket; the last arriver loads after it
      // has seen every ticket taken.
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            __hip_atomic_store(mine + ((i * NB + j) * 16 + r) * 64, acc[i][j][r], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
      wait_vm<0>();
      __syncthreads();
      if (tid == 0)
        ticket = __hip_atomic_fetch_add(g.ws_counters + pair, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      if (ticket != S - 1) return;                        // not the last one: done
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
      for (int q = 0; q < S; ++q) {                       // fixed order: the result does not depend on who is last
        const float* part = tile0 + (size_t)q * TILE;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              acc[i][j][r] += __hip_atomic_load(part + ((i * NB + j) * 16 + r) * 64, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
      }
      if (tid == 0)                                       // ready for the next launch
        __hip_atomic_store(g.ws_counters + pair, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // ---- epilogue: fp32 -> fp16 (RNE), stage as [n][m], store rows of C^T ----
  const int m = m0 + c * 8;
  long long dst_off[NPASS];
#pragma unroll
  for (int i = 0; i < NPASS; ++i)
    dst_off[i] = (cols[i] < 0 || m >= g.M) ? -1 : (long long)cols[i] * g.ldc + m;
  __syncthreads();
  if constexpr (KSPLIT > 1) {
    // group 1 hands its fp32 partial sums to group 0: [wave in group][register][lane]
    float* red = (float*)lds + wl * (MB * NB * 16 * 64) + lane;
    if (grp == 1) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) red[((i * NB + j) * 16 + r) * 64] = acc[i][j][r];
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] += red[((i * NB + j) * 16 + r) * 64];
    }
    __syncthreads();
  }
  if (EW && !joined) {
    if constexpr (EW) {
    // fp32 staging, half of the tile's columns at a time (the staging area then fits the
    // pipeline buffers and does not cost occupancy); every thread finishes its
    // (column, 8 x m) pieces: restored elements added, one rounding, streaming store
    static_assert(NPASS % 2 == 0 && (TN / 2) % 32 == 0, "");
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h) __syncthreads();
      if (grp == 0) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const int nblk = wn * WN + j * 32;                 // wave-uniform
            if (nblk / (TN / 2) != h) continue;
            const int n = nblk - h * (TN / 2) + (lane & 31);
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
              const int mm = wm * WM + i * 32 + 8 * rq + 4 * (lane >> 5);
              floatx4 v;
#pragma unroll
              for (int r = 0; r < 4; ++r) v[r] = acc[i][j][rq * 4 + r];
              *(floatx4*)(lds + n * CS32 + mm * 4) = v;
            }
          }
      }
      __syncthreads();
      constexpr int P = EW == EW_ELEMENTS && (NPASS / 2) % 2 == 0 ? 2 : 1;       // columns finished together
#pragma unroll
      for (int i = h * (NPASS / 2); i < (h + 1) * (NPASS / 2); i += P) {
        float sum[P][8];
        int lo[P], hi[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const int n = r0 + (i + p) * ROWS_PER_PASS - h * (TN / 2);
          const floatx4 lo4 = *(const floatx4*)(lds + n * CS32 + c * 32);
          const floatx4 hi4 = *(const floatx4*)(lds + n * CS32 + c * 32 + 16);
          // a dropped column: not even zeros of the kept rows
          const bool dropped = g.uniform_kp == 0 && r0 + (i + p) * ROWS_PER_PASS >= w_kept;
#pragma unroll
          for (int q = 0; q < 4; ++q) { sum[p][q] = dropped ? 0.f : lo4[q]; sum[p][4 + q] = dropped ? 0.f : hi4[q]; }
          const bool live = dst_off[i + p] >= 0;
          const int col = live ? cols[i + p] : 0;
          const int p0 = g.ew_ptr[col], p1 = g.ew_ptr[col + 1];
          lo[p] = live ? p0 : 0;
          hi[p] = live ? p1 : 0;
        }
        ew_accumulate<P, EW == EW_ELEMENTS ? 8 / P : 4>(g, lo, hi, g.A + (m < g.M ? m : 0), sum);
#pragma unroll
        for (int p = 0; p < P; ++p)
          if (dst_off[i + p] >= 0) store_row_chunk(g, g.C + dst_off[i + p], m, sum[p]);
      }
    }
    }
  } else {
    if (grp == 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int n = wn * WN + j * 32 + (lane & 31);
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            const int mm = wm * WM + i * 32 + 8 * rq + 4 * (lane >> 5);
            half4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (_Float16)acc[i][j][rq * 4 + r];
            *(half4*)(lds + n * CS + mm * 2) = v;
          }
        }
    }
    __syncthreads();
      // all staged chunks into registers first, then the stores back to back; C is
    // written once and not read again here: streaming (non-temporal) stores keep it
    // from lingering dirty in L2 until the end-of-kernel write-back
    union Chunk { uint2 h[2]; u32x4 v; };   // staging rows are 8-byte aligned only
    Chunk ck[NPASS];
#pragma unroll
    for (int i = 0; i < NPASS; ++i) {
      const int n = r0 + i * ROWS_PER_PASS;
      ck[i].h[0] = *(const uint2*)(lds + n * CS + c * 16);
      ck[i].h[1] = *(const uint2*)(lds + n * CS + c * 16 + 8);
    }
    // implicit img2col: the padding lanes of the wide grid are written as +0 (uniform branch)
    u32x4 vm = {~0u, ~0u, ~0u, ~0u};
    if (g.conv_P) vm = conv_valid_mask(g, m);
#pragma unroll
    for (int i = 0; i < NPASS; ++i) {
      if (dst_off[i] < 0) continue;
      _Float16* dst = g.C + dst_off[i];
      if (m + 8 <= g.M) __builtin_nontemporal_store(ck[i].v & vm, (u32x4*)dst);
      else {
        const int n = r0 + i * ROWS_PER_PASS;
        const uint16_t* e = (const uint16_t*)(lds + n * CS + c * 16);
#pragma unroll
        for (int qq = 0; qq < 8; ++qq)
          if (m + qq < g.M) ((uint16_t*)dst)[qq] = e[qq] & (uint16_t)(vm[qq >> 1] >> (16 * (qq & 1)));
      }
    }
  }
  };   // job
  if constexpr (!MULTI) {
    job(g_arg, (int)blockIdx.x, (int)threadIdx.x);
  } else {
    typedef const GemmArgs __attribute__((address_space(4)))* karg_ptr;
    const int total_jobs = g_arg.n_mtiles * g_arg.n_tiles + g_arg.n_zero;
    for (int r = 0; r < g_arg.tiles_per_wg; ++r) {
      const int bid = (int)blockIdx.x + r * (int)gridDim.x;
      if (bid >= total_jobs) break;
      if (r) {                 // every wave has read its chunks of the staging area: it may be overwritten
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
      }
      karg_ptr gp = (karg_ptr)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(gp));
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      job(*(const GemmArgs*)gp, bid, tid);
    }
  }
}

template <int TM, int TN, int WAVES_M, int D, bool DENSE, int NWAVES = 4, int KSPLIT = 1, int EW = EW_NONE,
          bool SPLIT = false, bool MULTI = false, bool SCALAR = false>
static hipError_t launch(const GemmArgs& g, hipStream_t stream) {
  const int jobs = g.n_mtiles * g.n_tiles * (SPLIT ? g.wg_split : 1) + g.n_zero;
  if (jobs <= 0) return hipSuccess;
  const int tpw = MULTI && g.tiles_per_wg > 1 ? g.tiles_per_wg : 1;
  const int grid = MULTI ? ((jobs + tpw - 1) / tpw + 7) / 8 * 8 : jobs;
  return launch_kernel(tw_gemm_km_dma_kernel<TM, TN, WAVES_M, D, DENSE, NWAVES, KSPLIT, EW, SPLIT, MULTI, SCALAR>, dim3(grid),
                       dim3(NWAVES * 64), stream, g);
}

// TEW instances: three stages in flight only.
template <int EW>
static hipError_t dispatch_ew(int G, int tm, int variant, GemmArgs& g, hipStream_t stream) {
  g.n_mtiles = (g.M + tm - 1) / tm;
  if (variant == DMA_KSPLIT2) {
    if (G == 128 && tm == 128) return launch<128, 128, 2, 3, false, 8, 2, EW>(g, stream);
    if (G == 128 && tm == 64) return launch<64, 128, 1, 3, false, 8, 2, EW>(g, stream);
    return hipErrorInvalidValue;
  }
  if (variant == DMA_WAVES8) {
    if (G == 128 && tm == 256) return launch<256, 128, 4, 3, false, 8, 1, EW_JOINED>(g, stream);   // (no registers left for elements)
    return hipErrorInvalidValue;
  }
  if (G == 128 && tm == 64) return launch<64, 128, 1, 3, false, 4, 1, EW>(g, stream);
  if (G == 128 && tm == 128) return launch<128, 128, 2, 3, false, 4, 1, EW>(g, stream);
  if (G == 64 && tm == 128) return launch<128, 64, 2, 3, false, 4, 1, EW_JOINED>(g, stream);     // (never faster one by one)
  if (G == 64 && tm == 256) return launch<256, 64, 4, 3, false, 4, 1, EW_JOINED>(g, stream);
  return hipErrorInvalidValue;
}

// The instances that can compute several tiles per workgroup, and the others.
template <int TM, int TN, int WAVES_M, int D, bool DENSE, int NWAVES = 4>
static hipError_t launch_multi(const GemmArgs& g, hipStream_t stream) {
  if constexpr (!DENSE) {
    if (g.tiles_per_wg > 1) return launch<TM, TN, WAVES_M, D, false, NWAVES, 1, EW_NONE, false, true>(g, stream);
  }
  return launch<TM, TN, WAVES_M, D, DENSE, NWAVES>(g, stream);
}

template <bool DENSE>
static hipError_t dispatch(int G, int tm, int depth, int variant, GemmArgs& g, hipStream_t stream) {
  g.n_mtiles = (g.M + tm - 1) / tm;
  if (variant == DMA_KSPLIT2) {   // two K-split groups of four waves
    if (G == 128 && tm == 128 && depth == 3) return launch<128, 128, 2, 3, DENSE, 8, 2>(g, stream);
    if (G == 128 && tm == 64 && depth == 3) return launch<64, 128, 1, 3, DENSE, 8, 2>(g, stream);
    if (G == 128 && tm == 64 && depth == 4) return launch<64, 128, 1, 4, DENSE, 8, 2>(g, stream);
    if (G == 64 && tm == 128 && depth == 3) return launch<128, 64, 2, 3, DENSE, 8, 2>(g, stream);
    // One 32 x 32 block per wave and k-step is little work per barrier, but twice the workgroups where half of the chip
    // is idle: 64 / 128 rows, 3072 x 768 at 75 %, M = 1403, 242 workgroups of 64 7.5 / 8.8 us; 4608 x 512, M = 1915 9.3 / 10.7;
    // 3 x 3 convolutions 512 -> 512 of eight 14 x 14 images 9.9 / 11.8, 256 -> 256 of four 28 x 28 6.6 / 7.9; short lists even
    // (768 x 768 at 40 %, M = 1019 6.3 / 6.4).  (More workgroups than CUs: 3072 x 768, M = 1531 9.0 / 8.7.)
    if constexpr (!DENSE) {
      if (G == 64 && tm == 64 && depth == 3) return launch<64, 64, 2, 3, false, 8, 2>(g, stream);
    }
    return hipErrorInvalidValue;
  }
  if (variant == DMA_WAVES8) {    // 512-thread workgroups: 64 x 32 (m x n) per wave
    if (G == 128 && tm == 128 && depth == 3) return launch<128, 128, 2, 3, DENSE, 8>(g, stream);
    if (G == 128 && tm == 128 && depth == 4) return launch<128, 128, 2, 4, DENSE, 8>(g, stream);
    if (G == 128 && tm == 256 && depth == 3) return launch<256, 128, 4, 3, DENSE, 8>(g, stream);
    return hipErrorInvalidValue;
  }
  if constexpr (!DENSE) {
    if (g.scalar_rows && depth == 3 && g.tiles_per_wg <= 1) {
      if (G == 128 && tm == 128) return launch<128, 128, 2, 3, false, 4, 1, EW_NONE, false, false, true>(g, stream);
      if (G == 64 && tm == 256) return launch<256, 64, 4, 3, false, 4, 1, EW_NONE, false, false, true>(g, stream);
    }
  }
#define TWG_CASE(TM_, TN_, WM_, D_) \
  if (G == TN_ && tm == TM_ && depth == D_) return launch<TM_, TN_, WM_, D_, DENSE>(g, stream);
  if (G == 128 && tm == 64 && depth == 3) return launch_multi<64, 128, 1, 3, DENSE>(g, stream);
  if (G == 128 && tm == 128 && depth == 3) return launch_multi<128, 128, 2, 3, DENSE>(g, stream);
  TWG_CASE(256, 128, 2, 3)
  TWG_CASE(64, 128, 1, 4) TWG_CASE(128, 128, 2, 4) TWG_CASE(256, 128, 2, 4)
  TWG_CASE(128, 64, 2, 3) TWG_CASE(256, 64, 4, 3)
  TWG_CASE(128, 64, 2, 4) TWG_CASE(256, 64, 4, 4)
  // deep pipelines for launches with about one workgroup per CU
  TWG_CASE(64, 128, 1, 6) TWG_CASE(128, 128, 2, 6) TWG_CASE(128, 64, 2, 6)
  TWG_CASE(64, 128, 1, 8) TWG_CASE(128, 128, 2, 8) TWG_CASE(128, 64, 2, 8)
#undef TWG_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_tw_km_dma(int G, int tm, int depth, int variant, GemmArgs g, hipStream_t stream) {
  return dispatch<false>(G, tm, depth, variant, g, stream);
}

static __global__ void zero_words(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}
hipError_t launch_zero_words(uint32_t* p, int n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  return launch_kernel(zero_words, dim3((n + 255) / 256), dim3(256), stream, p, n);
}

hipError_t launch_tw_km_dma_split(int G, int tm, GemmArgs g, hipStream_t stream) {
  if (g.wg_split < 1 || !g.ws_partials || !g.ws_counters) return hipErrorInvalidValue;
  g.n_mtiles = (g.M + tm - 1) / tm;
  if (G == 128 && tm == 128) return launch<128, 128, 2, 3, false, 4, 1, EW_NONE, true>(g, stream);
  if (G == 128 && tm == 64) return launch<64, 128, 1, 3, false, 4, 1, EW_NONE, true>(g, stream);
  if (G == 64 && tm == 128) return launch<128, 64, 2, 3, false, 4, 1, EW_NONE, true>(g, stream);
  return hipErrorInvalidValue;
}
hipError_t launch_tew_km_dma(int G, int tm, int depth, int variant, GemmArgs g, hipStream_t stream) {
  if (depth != 3) return hipErrorInvalidValue;
  return g.ew_elements ? dispatch_ew<EW_ELEMENTS>(G, tm, variant, g, stream) : dispatch_ew<EW_JOINED>(G, tm, variant, g, stream);
}
hipError_t launch_dense_km_dma(int tn, int tm, int depth, int variant, GemmArgs g, hipStream_t stream) {
  return dispatch<true>(tn, tm, depth, variant, g, stream);
}

}  // namespace twg
