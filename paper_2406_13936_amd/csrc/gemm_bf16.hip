// Replica-batched ("grouped") bf16 GEMM on the gfx950 matrix cores.
//
//   C[g][m][n] = sum_k A[g][m][k] * B[g][n][k],   g = replica
//
// covers the contractions of one local step (Alg. 1 of the paper, "compute the local batch
// gradient"): forward  a W^T, backward-data  delta W, weight gradient  delta^T a, and the extra
// contraction  a Gbar^T  of the inner-product statistics.  Either operand may be stored
// k-contiguous (memory [row][k]) or row-contiguous (memory [k][row]).
//
// Data path (no operand ever passes through vector registers on its way to LDS):
//   * global -> LDS with `buffer_load_dwordx4 ... lds` (16 bytes per lane, written by the
//     memory pipeline at M0 + 16*lane), NS stage buffers in a ring; out-of-range chunks come
//     back as zeros through the buffer descriptor's range check, so ragged m / n / k need no
//     branches.  A stage's loads are spread over the MFMA groups of the previous stage so that
//     a wavefront never sits in the memory-issue queue while the matrix pipe idles.
//   * k-contiguous tiles are kept as [row][BK] with the 16-byte chunk index XOR-swizzled by the
//     row (the permutation is applied on the global-address side, since the LDS side of a
//     direct load is linear in the lane id); an MFMA fragment is one ds_read_b128.
//   * row-contiguous tiles are kept as [k][rows] and read with ds_read_b64_tr_b16, the LDS
//     transpose read: inside each group of 16 lanes, lane i receives element (i % 4) of the
//     8-byte vectors addressed by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12 -- i.e. four
//     consecutive k for its own row when lane j addresses (k = j / 4, rows 4 (j % 4) ..+3).
//   * one s_barrier per k-tile; s_waitcnt vmcnt(n) lets the younger stages stay in flight.
//   * the 256 x 256 tile has a main loop of its own (see the note above the kernel).
//
// Tiling: BM x BN x BK block tile, WM x WN wavefronts of 64 lanes, each a grid of 32x32x16
// (256 x 256 tile: 16x16x32) bf16 MFMAs with fp32 accumulators.  Work-group ids are remapped so that each XCD (ids are
// dealt round-robin to the 8 XCDs) works on a contiguous range of tiles and its L2 sees one
// replica's operands at a time.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <utility>
#include "abs_internal.h"
#include "device_utils.h"
#include "gather.h"
#include "step_tail.h"

namespace absk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

namespace {

// Epilogue outputs and the elementwise operand are touched once per launch: non-temporal accesses
// keep them from displacing the operand tiles that other work-groups of the launch re-read from L2.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef f32x4 f32x4_t;
__device__ __forceinline__ uint4 ld_once(const bf16_t *p) {
  const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_once(bf16_t *p, uint4 v) {
  const u32x4_t w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, reinterpret_cast<u32x4_t *>(p));
}
__device__ __forceinline__ void st_once(bf16_t *p, uint2 v) {
  const u32x2_t w = {v.x, v.y};
  __builtin_nontemporal_store(w, reinterpret_cast<u32x2_t *>(p));
}
__device__ __forceinline__ float4 ld_once(const float *p) {
  const f32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_once(float *p, float4 v) {
  const f32x4_t w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, reinterpret_cast<f32x4_t *>(p));
}

// EPI_IPDOT instances whose activation slot holds this also leave the squared norms of E's rows (GemmP::part2)
constexpr int IPDOT_NORMS = 1;

constexpr uint32_t OOB = 0x80000000u;   // byte offset beyond any operand (operands are < 2 GiB)

// XOR on the 16-byte chunk index of k-row k in a row-contiguous tile.  A 32-lane half of a transpose read meets four values of
// k x 4 chunks (KR = 16: 32 rows) or eight values of k, 0 .. 3 and 8 .. 11 of the step, x 2 chunks (KR = 32: 16 rows); either
// way the 16 chunks spread over all 64 banks (conflicts: 1 % of a weight gradient's LDS cycles, with either).  The same for k and k + 4, the fragment's second read, and for every k-step.
template <int KR> __device__ __forceinline__ int tr_swizzle(int k) { return KR == 16 ? 4 * (k & 3) : 2 * (k & 3) + (k & 8); }

template <int N> __device__ __forceinline__ void wait_vmcnt() {
  // s_waitcnt immediate on gfx9: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// ---- one operand's stage: addressing of the direct loads and of the fragment reads ---------
// ROWS = tile extent along m (or n); TRANS = memory is [k][row]; KR: k per MFMA (which k-rows a transpose read meets).
template <int ROWS, int BK, bool TRANS, int NW, int KR = 16>
struct Operand {
  static constexpr int ELEMS = ROWS * BK;                 // bf16 elements per stage
  static constexpr int NI = ELEMS / 8 / 64 / NW;          // load instructions per wave per stage
  static_assert(ELEMS % (8 * 64 * NW) == 0 && NI >= 1, "tile too small for the wave count");
  static constexpr int CPR = BK / 8;                      // k-contiguous: chunks per row
  static constexpr int SWS = CPR >= 8 ? 1 : 2;
  static constexpr int CH = ROWS / 8;                     // row-contiguous: chunks per k-row
  static_assert(!TRANS || CH >= 8, "transposed tiles need at least 64 rows");

  uint32_t voff[NI];     // per-lane byte offset of its chunk at k0 = 0 (OOB if the row is outside)
  int kofs[NI];          // k (relative to k0) of the chunk, for the ragged last k-tile

  // SPREAD (k-contiguous only): stage row u holds matrix row row0 + 64 (u / 32) + u % 32, i.e. every second group of 32
  template <bool SPREAD = false>
  __device__ __forceinline__ void init(int wave, int lane, int row0, int rows, int ld) {
    static_assert(!(SPREAD && TRANS), "row-contiguous stages keep their rows in order");
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = (wave * NI + i) * 64 + lane;          // linear 16-byte chunk index in the stage
      if (!TRANS) {
        const int row = c / CPR, kc = (c % CPR) ^ ((row >> SWS) & (CPR - 1));
        const int mrow = row0 + (SPREAD ? (row >> 5) * 64 + (row & 31) : row);
        kofs[i] = kc * 8;
        voff[i] = (mrow < rows) ? (uint32_t)(mrow * ld + kc * 8) * 2u : OOB;
      } else {
        const int kq = c / CH, ch = (c % CH) ^ (tr_swizzle<KR>(kq) & (CH - 1));
        kofs[i] = kq;
        voff[i] = (row0 + ch * 8 < rows) ? (uint32_t)(kq * ld + row0 + ch * 8) * 2u : OOB;
      }
    }
  }
  // rows from elsewhere: matrix row r at row_of(r) of the operand (k-contiguous)
  template <class F>
  __device__ __forceinline__ void init_rows(int wave, int lane, int row0, int rows, int ld, F row_of) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int mrow = row0 + ((wave * NI + i) * 64 + lane) / CPR;
      if (mrow < rows) voff[i] = ((uint32_t)row_of(mrow) * (uint32_t)ld + (uint32_t)kofs[i]) * 2u;
    }
  }
  // byte offset added for k-tile kt (scalar)
  static __device__ __forceinline__ uint32_t soff(int kt, int ld) {
    return TRANS ? (uint32_t)kt * BK * ld * 2u : (uint32_t)kt * BK * 2u;
  }
  // i is a compile-time constant after unrolling (voff / kofs live in registers)
  __device__ __forceinline__ void load(int i, __amdgpu_buffer_rsrc_t rsrc, bf16_t *stage, int wave, int kt,
                                       int K, int ld, bool full) const {
    uint32_t v = voff[i];
    if (!full && kt * BK + kofs[i] >= K) v = OOB;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)(stage + (wave * NI + i) * 512), 16, v,
                                             soff(kt, ld), 0, 0);
  }
  // The whole stage from k = kbeg on, for callers that keep the number of loads in flight constant: chunks at or
  // beyond K come back as zeros, also where the stage lies wholly beyond it (then ksafe, a multiple of BK below K,
  // takes the place of kbeg in the scalar offset, which the range check subtracts from the operand's extent).
  __device__ __forceinline__ void load_all(__amdgpu_buffer_rsrc_t rsrc, bf16_t *stage, int wave, int kbeg, int ksafe, int K,
                                           int ld) const {
    const uint32_t so = (uint32_t)(kbeg < K ? kbeg : ksafe) * (TRANS ? (uint32_t)ld * 2u : 2u);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t v = kofs[i] < K - kbeg ? voff[i] : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)(stage + (wave * NI + i) * 512), 16, v, so, 0, 0);
    }
  }
};

// fragment of rows [r0, r0+32) for k-step kk of a stage
template <int ROWS, int BK, bool TRANS>
struct Frag {
  static constexpr int CPR = BK / 8, SWS = CPR >= 8 ? 1 : 2, CH = ROWS / 8;
  int base, swz;         // !TRANS: element offset of the row, and its swizzle
  int tbase[2];          // TRANS: element offsets for the two transpose reads at kk = 0
  __device__ __forceinline__ void init(int r0, int lane) {
    if (!TRANS) {
      const int r = r0 + (lane & 31);
      base = r * BK;
      swz = (r >> SWS) & (CPR - 1);
    } else {
      const int i16 = lane & 15, g16 = lane >> 4;
      const int rr = r0 + (g16 & 1) * 16 + 4 * (i16 & 3);     // first of this lane's 4 rows
      const int kq = (g16 >> 1) * 8 + (i16 >> 2);             // k within the 16-wide step
      const int ch = (rr >> 3) ^ (tr_swizzle<16>(kq) & (CH - 1));
      tbase[0] = kq * ROWS + ch * 8 + (rr & 7);
      tbase[1] = tbase[0] + 4 * ROWS;
    }
  }
  __device__ __forceinline__ bf16x8 read(const bf16_t *stage, int kk) const {
    if (!TRANS) {
      const int kc = kk * 2 + (threadIdx.x >> 5 & 1);
      return *reinterpret_cast<const bf16x8 *>(stage + base + ((kc ^ swz) << 3));
    } else {
      // Issued as inline assembly: through the builtin the compiler cannot tell that this read
      // does not alias the direct-to-LDS loads in flight (they fill the other stage buffer) and
      // puts s_waitcnt vmcnt(0) in front of every group of reads, which serialises the pipeline.
      // The price is that the compiler no longer counts these reads in lgkmcnt: the main loop
      // waits for them itself (wait_frags) before the MFMAs that use them.
      const uint32_t a0 = (uint32_t)(uintptr_t)(lds_void *)(stage + tbase[0] + kk * 16 * ROWS);
      const uint32_t a1 = (uint32_t)(uintptr_t)(lds_void *)(stage + tbase[1] + kk * 16 * ROWS);
      s16x4 lo, hi;
      asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(lo) : "v"(a0) : "memory");
      asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(hi) : "v"(a1) : "memory");
      const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8, v);
    }
  }
};

// LDS fragment reads with the stage, row-tile and k-step as an immediate offset (inline assembly for the reason
// given in Frag::read; the caller waits for them itself)
template <int OFF> __device__ __forceinline__ bf16x8 lds_read_rows(uint32_t addr) {
  bf16x8 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF, int NEXT4> __device__ __forceinline__ bf16x8 lds_read_cols(uint32_t addr) {
  s16x4 lo, hi;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(OFF) : "memory");
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(OFF + NEXT4) : "memory");
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
template <int V> struct Const { static constexpr int value = V; };
template <int... I, class F> __device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F &&f) {
  (f(Const<I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, static_cast<F &&>(f));
}

// Wait until at most N LDS operations of this wave are outstanding, and make the fragments that
// the following MFMAs read depend on that wait (needed where fragment reads are inline assembly).
template <int N, int MI, int NI>
__device__ __forceinline__ void wait_frags(bf16x8 (&a)[MI], bf16x8 (&b)[NI]) {
  static_assert(N >= 0 && N <= 15, "lgkmcnt range");
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));          // vmcnt, expcnt: no wait; lgkmcnt = N
#pragma unroll
  for (int i = 0; i < MI; ++i) asm volatile("" : "+v"(a[i]));
#pragma unroll
  for (int j = 0; j < NI; ++j) asm volatile("" : "+v"(b[j]));
}

// 32 tiles of 256 x 256 run side by side on an XCD; they fetch one operand panel per row and one per column of their arrangement
// into its L2.  Rows of more than BAND tiles are cut into bands of at most BAND columns, so that the 32 tiles stand 4 x 8 or
// nearly so (12 panels) and not 2 x 16 (18).
constexpr int BAND = 8;

// Ragged groups with extents of their own along m: tile lb of those that exist, group by group, is tile t of group g.  Numbering
// the tiles of the largest extent for every group instead, an XCD's share of whole groups is what its groups happen to have: 16
// workers of 1024 to 8192 rows, the largest paired with the smallest, gave one XCD a third more than the mean.  3072-2048-2048-2048-100:
// forward 587 -> 526 us, inner products 505 -> 464, backward-data 501 -> 464, logits 94 -> 63, the step 6750 -> 6299.
// One lane per group, a scan, 64 groups at a time; uniform over the wavefront.  The lookup stands in front of the first operand load:
// one load and a scan on DPP.  us per step with shuffles through LDS and the count loaded again -> this (grids of the largest
// extent, without a lookup): 784-336-336-336-100, 9 replicas of up to 1123 samples, 212.7 -> 207.5 (211.2); 784-128-128-100,
// 8 replicas of up to 1498, 106.8 -> 105.1 (105.5).
__device__ __forceinline__ int wave_scan(int v) {              // inclusive
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8: inside 16 lanes
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);      // row_bcast:15 into lanes 16 .. 31 and 48 .. 63
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);      // row_bcast:31 into lanes 32 .. 63
  return v;
}
template <int BM>
__device__ __forceinline__ void ragged_tile(const int *__restrict__ rows, int groups, int tilesN, int lb, int &g, int &t, int &rows_g) {
  const int lane = threadIdx.x & 63;
  t = lb;
  for (int g0 = 0;; g0 += 64) {
    const int r = g0 + lane < groups ? rows[g0 + lane] : 0, own = (r + BM - 1) / BM * tilesN, sum = wave_scan(own);
    const int before = __popcll(__ballot(sum <= t));           // groups that end in front of the tile
    if (before < 64 || g0 + 64 >= groups) {                    // (the grid has the groups' tiles: in the last 64 one holds it)
      g = g0 + before;
      t -= __builtin_amdgcn_readlane(sum - own, before);
      rows_g = __builtin_amdgcn_readlane(r, before);
      return;
    }
    t -= __builtin_amdgcn_readlane(sum, 63);
  }
}

// ---- the kernel --------------------------------------------------------------------------
//
// Main loop of the 256 x 256 tile.  64 KB of operands per k-tile of 64 and 256 x 256 outputs is what a CU has to take in
// every 2048 matrix-core cycles; a fifth of it misses the XCD's L2 and comes back after 1000 to 1600 cycles, so a load that
// is issued during the k-tile before it is needed arrives late (two 64 KB stages with one wait per k-tile: the waves
// stood at that wait for a third of their time).  Here LDS holds the same 128 KB as eight units of 16 KB (A rows in two
// halves h, B in two halves c, two k-tiles), each with its own life: a k-tile is four phases (h, c) of sixteen MFMAs per wave,
// a phase reads one unit's fragments and refills, for the k-tile after the next, the unit that the phase before read, so every
// load has seven phases (3500 cycles) to arrive and six units stay in flight at each wait.
// The four waves with wm = 1 (one per SIMD) run one barrier behind those with wm = 0: while one wave of a SIMD issues its
// MFMAs the other one reads fragments and issues loads.
//   phase        0 (0,0)     1 (0,1)     2 (1,0)     3 (1,1)
//   reads        A0          B1          A1          B0 of the next k-tile
//   refills      B0          A0          B1          A1            (of k-tile + 2)
// Why a refill cannot overtake a read: a wave waits for its own reads (lgkmcnt) before the barrier that ends its memory
// half, and the refill is issued at the earliest one barrier after the later group's reads.  Why a read finds its data: the
// wait in phase f covers the unit of phase f + 1, and a barrier of all waves lies between.
// B halves: k-contiguous operands split by columns (unit c holds columns 64 j + 32 c .. + 31 of every wave column j, so that
// a wave still owns 64 consecutive columns), row-contiguous ones by k (unit c = 32 of the 64 k: 512 bytes of a memory row).
// Measured, 16 replicas, 8192 x 2048 x 2048, two-stage loop -> this one with 32x32x16 MFMAs -> with 16x16x32: inner products 1017 ->
// 850 -> 843 us (1.30 PFLOP/s), forward 1160 -> 1043 -> 1035, backward-data 1110 -> 922 -> 932, weight gradient with the step in
// its epilogue 1178 -> 993 -> 1019, launch by launch on different boxes; side by side the step at 16 replicas went from 13.22 to
// 12.65 ms with the last change: at the power limit the clock rises with what an MFMA saves.
// (the work of one work-group: tile lb of the tilesM x tilesN x groups of a launch)
// MODE, a kernel of its own each, since what the short launches do not need costs them up to 0.7 of 11 us in front of their first
// load: ROWS_OWN: ragged groups (not the weight gradients); ROWS_DATASET: the rows of A are rows of the dataset (GemmP::aidx).
enum { ROWS_PLAIN = 0, ROWS_OWN = 1, ROWS_DATASET = 2 };
template <int BM, int BN, int BK, int WM, int WN, int NS, bool PP, bool AT, bool BT, int EPI, int ACT, int MODE = ROWS_PLAIN>
__device__ __forceinline__ void gemm_bf16_tile(const GemmP &pin, const int tilesM, const int tilesN, const int lb) {
  constexpr int NW = WM * WN, NT = NW * 64;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr bool IS_WGRAD = EPI == EPI_WGRAD || EPI == EPI_WGRAD_UPD;   // _UPD: ACT carries the optimizer
  constexpr int MI = TM / 32, NI = TN / 32;
  constexpr int STAGE = (BM + BN) * BK;                 // bf16 elements per stage
  constexpr int NPART = BK / 16;                        // MFMA groups per k-tile
  static_assert(TM % 32 == 0 && TN % 32 == 0 && BK % 16 == 0 && NS >= 2, "tile shape");
  static_assert(MODE == ROWS_PLAIN || !IS_WGRAD, "weight gradients read p.rows");
  typedef Operand<BM, BK, AT, NW> OpA;
  typedef Operand<BN, BK, BT, NW> OpB;
  constexpr int NL = OpA::NI + OpB::NI;                 // load instructions per wave per stage
  static_assert((NS - 2) * NL <= 63, "vmcnt range");
  static_assert(!PP || (BM == 256 && BN == 256 && BK == 64 && WM == 2 && WN == 4 && NS == 2), "the pipelined main loop");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t *smem = reinterpret_cast<bf16_t *>(smem_raw);

  int g, t, ksl = 0, rowsM = tilesM, own = 0;     // group, tile of the group, k-slice, the group's rows of tiles and its own extent
  const int ksplit = (EPI == EPI_WGRAD && pin.ksplit > 1) ? pin.ksplit : 1;   // (no split with the step fused)
  if constexpr (MODE == ROWS_OWN) {               // only the tiles that ragged groups have are numbered (ragged_blocks)
    ragged_tile<BM>(pin.rows, pin.groups, tilesN, lb, g, t, own);
    rowsM = (own + BM - 1) / BM;
  } else {
    const int per_g = tilesM * tilesN;
    const int vg = lb / per_g;                    // group, or (group, k-slice) pair of a split reduction
    t = lb - vg * per_g;
    const int gv = vg / ksplit;
    ksl = vg - gv * ksplit;
    g = IS_WGRAD && pin.gperm ? pin.gperm[gv] : gv;   // position in the launch order -> group
  }
  int tm, tn;
  if (BM == 256 && tilesN > BAND) {               // bands of columns (see BAND), row by row inside a band
    const int nb = (tilesN + BAND - 1) / BAND, bw = (tilesN + nb - 1) / nb, b = t / (bw * rowsM);
    const int w = min(bw, tilesN - b * bw), r = t - b * bw * rowsM;
    tm = r / w; tn = b * bw + r - tm * w;
  } else {
    tm = t / tilesN; tn = t - tm * tilesN;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  GemmP p = pin;
  if (MODE == ROWS_OWN || (IS_WGRAD && p.rows)) { // ragged groups: this group's own extent
    if (IS_WGRAD) { p.Kd = p.rows[g]; p.alpha = 1.0f / (float)p.Kd; } else p.Md = own;
  }
  long long kofsA = 0, kofsB = 0;                 // element offsets of this block's k-slice
  if (EPI == EPI_WGRAD && ksplit > 1) {
    const int k0 = ksl * p.kchunk;
    int kd = p.Kd - k0;
    kd = kd < 0 ? 0 : (kd > p.kchunk ? p.kchunk : kd);
    p.Kd = kd;                                    // an empty slice runs no k-tile and writes zeros
    kofsA = AT ? (long long)k0 * p.lda : k0;
    kofsB = BT ? (long long)k0 * p.ldb : k0;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  const bf16_t *A = static_cast<const bf16_t *>(p.A) + (long long)g * p.sAg + kofsA;
  const bf16_t *B = static_cast<const bf16_t *>(p.B) + (long long)g * p.sBg + kofsB;
  // range = the operand's extent in memory: rows*ld (k-contiguous) or K*ld (row-contiguous)
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t *>(A), 0, (int)((long long)(AT ? p.Kd : MODE == ROWS_DATASET ? p.aN : p.Md) * p.lda * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t *>(B), 0, (int)((long long)(BT ? p.Kd : p.Nd) * p.ldb * 2), 0x00020000);

  // accumulators: 32 x 32 tiles (32x32x16 MFMAs), or 16 x 16 ones in the pipelined loop (16x16x32)
  constexpr int RT = PP ? 16 : 32;
  f32x16 acc[PP ? 1 : MI][PP ? 1 : NI];
  f32x4 acc16[PP ? TM / 16 : 1][PP ? TN / 16 : 1];
  if constexpr (PP) {
#pragma unroll
    for (int i = 0; i < TM / 16; ++i)
#pragma unroll
      for (int j = 0; j < TN / 16; ++j) acc16[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  } else {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  }

  // first row of row slice i (32 rows) of this wave, relative to the tile
  auto slice_row = [&](int i) -> int { return PP ? (i >> 1) * 128 + wm * 64 + (i & 1) * 32 : wm * TM + i * 32; };

  // Fused optimizer step (EPI_WGRAD_UPD): the epilogue walks this wave's slices (32 rows x TN columns) in batches of
  // UHB 16-byte chunks per lane, and the loads of batch k + 1 (parameters and optimizer state) are issued before
  // batch k is processed, so that a wave always has a batch of loads in flight while it computes and stores.
  // (Four chunks for the 128 x 128 and 64 x 256 tiles: config 3 at b = 64 2.4 % faster than with two, b = 256
  // unchanged; the 256 x 256 tile has no registers to spare for more than two.)
  constexpr bool UPD = EPI == EPI_WGRAD_UPD;
  constexpr int UFCPR = TN / 4;                             // float4 chunks per slice row
  constexpr int UFIT = 32 * UFCPR / 64;                     // chunks per lane per slice
  constexpr int UHBW = ((BM == 128 && BN == 128) || BM == 64) ? 4 : 2;
  constexpr int UHB = UFIT < UHBW ? UFIT : UHBW;
  constexpr int UBPS = UFIT / UHB;
  static_assert(!UPD || UFIT % UHB == 0, "chunk batches");
  // The 128 x 128 and 64 x 256 tiles (short batches: a launch is all epilogue) issue the first batch before the operand loads of
  // the reduction, so that its latency passes behind the main loop; being older than every operand load, these
  // loads do not disturb the counting of the main loop's waits (loads return in order).
  constexpr bool UPD_EARLY = UPD && ((BM == 128 && BN == 128) || BM == 64);
  float4 xq[2][UPD ? UHB : 1], vq[2][UPD ? UHB : 1], mq[2][UPD ? UHB : 1];
  const long long ugoff = UPD ? (long long)g * p.sCg : 0;
  auto upd_where = [&](int bi, int u, int &m, int &n, int &row, int &cc) {
    const int c = ((bi % UBPS) * UHB + u) * 64 + lane;
    row = c / UFCPR; cc = c % UFCPR;
    m = m0 + slice_row(bi / UBPS) + row;
    n = n0 + wn * TN + cc * 4;
  };
  auto upd_prefetch = [&](int bi) {
    if constexpr (UPD) {
#pragma unroll
      for (int u = 0; u < UHB; ++u) {
        int m, n, row, cc;
        upd_where(bi, u, m, n, row, cc);
        xq[bi & 1][u] = vq[bi & 1][u] = mq[bi & 1][u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (m < p.Md && n < p.Nd) {                          // Nd is a multiple of 4 (checked by the launcher)
          const long long o = ugoff + (long long)m * p.ldc + n;
          xq[bi & 1][u] = ld_once(p.upd_x + o);
          if (ACT != OPT_SGD) vq[bi & 1][u] = ld_once(p.upd_v + o);       // (the optimizer travels in the activation slot)
          if (ACT == OPT_ADAMW) mq[bi & 1][u] = ld_once(p.upd_m + o);
        }
      }
    }
  };
  if constexpr (UPD_EARLY) upd_prefetch(0);

  const int KT = (p.Kd + BK - 1) / BK;
  if constexpr (PP) {
    // ---- pipelined main loop of the 256 x 256 tile (see the note above the kernel) -----------------------------
    typedef Operand<128, 64, AT, NW, 32> UA;                 // A unit h: rows 128 h .. 128 h + 127 of the tile, 64 k
    typedef Operand<BT ? 256 : 128, BT ? 32 : 64, BT, NW, 32> UB;   // B unit c: k 32 c .. (BT), or columns 64 j + 32 c ..
    constexpr int UNIT = 8192;                               // elements of a unit (16 KB)
    UA ua[2];
    UB ub[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      ua[h].init(wave, lane, m0 + h * 128, p.Md, p.lda);
      if constexpr (BT) ub[h].init(wave, lane, n0, p.Nd, p.ldb);
      else ub[h].template init<true>(wave, lane, n0 + h * 32, p.Nd, p.ldb);
    }
    auto load_a = [&](int kt, int slot, int h) {
      ua[h].load_all(ra, smem + (slot * 2 + h) * UNIT, wave, kt * 64, 0, p.Kd, p.lda);
    };
    auto load_b = [&](int kt, int slot, int c) {
      ub[c].load_all(rb, smem + (4 + slot * 2 + c) * UNIT, wave, kt * 64 + (BT ? c * 32 : 0), 0, p.Kd, p.ldb);
    };
    // LDS byte addresses of this lane's fragments (16 rows x 32 k: lane l holds row l % 16, eight k from 8 (l / 16)) in unit 0;
    // everything else is an immediate offset
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
    const int i16 = lane & 15, g16 = lane >> 4;
    const int kq = g16 * 8 + (i16 >> 2);                     // transpose reads: k within the 32-wide step
    uint32_t aaddr[AT ? 4 : 2], baddr[BT ? 4 : 2];           // (transpose reads: by row tile; else by k-step)
    if constexpr (AT) {
#pragma unroll
      for (int ii = 0; ii < 4; ++ii) {
        const int rr = wm * 64 + ii * 16 + 4 * (i16 & 3);
        aaddr[ii] = lds0 + 2u * (uint32_t)(kq * 128 + ((rr >> 3) ^ tr_swizzle<32>(kq)) * 8 + (rr & 7));
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        aaddr[kk] = lds0 + (uint32_t)((wm * 64 + i16) * 128 + (((kk * 4 + g16) ^ (i16 >> 1)) << 4));
    }
    if constexpr (BT) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int rr = wn * 64 + j * 16 + 4 * (i16 & 3);
        baddr[j] = lds0 + 65536u + 2u * (uint32_t)(kq * 256 + ((rr >> 3) ^ tr_swizzle<32>(kq)) * 8 + (rr & 7));
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        baddr[kk] = lds0 + 65536u + (uint32_t)((wn * 32 + i16) * 128 + (((kk * 4 + g16) ^ (i16 >> 1)) << 4));
    }
    bf16x8 fa[4][2], fb[2][4];                               // fa[row tile][k-step]; fb[unit][BT: column tile, else 2 column tile + k-step]
    auto read_a = [&](auto SLOT, auto H) {
      constexpr int U = (decltype(SLOT)::value * 2 + decltype(H)::value) * UNIT * 2;
      static_for<8>([&](auto I) {
        constexpr int kk = decltype(I)::value >> 2, ii = decltype(I)::value & 3;
        if constexpr (AT) fa[ii][kk] = lds_read_cols<U + kk * 8192, 1024>(aaddr[ii]);
        else fa[ii][kk] = lds_read_rows<U + ii * 2048>(aaddr[kk]);
      });
    };
    auto read_b = [&](auto SLOT, auto C) {
      constexpr int c = decltype(C)::value, U = (decltype(SLOT)::value * 2 + c) * UNIT * 2;
      static_for<4>([&](auto I) {
        constexpr int q = decltype(I)::value;
        if constexpr (BT) fb[c][q] = lds_read_cols<U, 2048>(baddr[q]);
        else fb[c][q] = lds_read_rows<U + (q >> 1) * 2048>(baddr[q & 1]);
      });
    };
    auto close_reads = [&]() {                               // this wave's fragment reads are done
      __builtin_amdgcn_s_waitcnt(0xC07F);
#pragma unroll
      for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(fa[q][0]), "+v"(fa[q][1]), "+v"(fb[0][q]), "+v"(fb[1][q]));
    };
    auto phase = [&](auto SLOT, auto F, int kt) {
      constexpr int f = decltype(F)::value, h = f >> 1, c = f & 1;
      // memory half: this phase's fragments, and the unit two k-tiles ahead that takes the place read last phase
      if constexpr (f == 0) { read_a(SLOT, Const<0>{}); load_b(kt + 2, SLOT.value, 0); }
      if constexpr (f == 1) { read_b(SLOT, Const<1>{}); load_a(kt + 2, SLOT.value, 0); }
      if constexpr (f == 2) { read_a(SLOT, Const<1>{}); load_b(kt + 2, SLOT.value, 1); }
      if constexpr (f == 3) { read_b(Const<1 - decltype(SLOT)::value>{}, Const<0>{}); load_a(kt + 2, SLOT.value, 1); }
      wait_vmcnt<12>();                                      // the unit read next phase has landed; six more stay in flight
      close_reads();
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
      static_for<16>([&](auto I) {                           // (operands swapped as below: a lane owns one row of C)
        constexpr int q = decltype(I)::value;
        if constexpr (BT) {
          constexpr int ii = q >> 2, j = q & 3;
          acc16[4 * h + ii][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[c][j], fa[ii][c], acc16[4 * h + ii][j], 0, 0, 0);
        } else {
          constexpr int kk = q >> 3, ii = (q >> 1) & 3, j = q & 1;
          acc16[4 * h + ii][2 * c + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[c][2 * j + kk], fa[ii][kk], acc16[4 * h + ii][2 * c + j], 0, 0, 0);
        }
      });
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
    };
    auto ktile = [&](auto SLOT, int kt) { static_for<4>([&](auto F) { phase(SLOT, F, kt); }); };
#pragma unroll
    for (int s = 0; s < 2; ++s) { load_b(s, s, 0); load_a(s, s, 0); load_b(s, s, 1); load_a(s, s, 1); }
    wait_vmcnt<12>();
    __builtin_amdgcn_s_barrier();
    read_b(Const<0>{}, Const<0>{});
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    if (wm == 1) __builtin_amdgcn_s_barrier();               // these four waves run half a phase behind
    for (int kt = 0; kt < KT; kt += 2) {
      ktile(Const<0>{}, kt);
      if (kt + 1 < KT) ktile(Const<1>{}, kt + 1);
    }
    if (wm == 0) __builtin_amdgcn_s_barrier();
    wait_vmcnt<0>();                                         // (zeros beyond K still on their way to LDS)
  } else {
    OpA oa;
    OpB ob;
    oa.init(wave, lane, m0, p.Md, p.lda);
    ob.init(wave, lane, n0, p.Nd, p.ldb);
    if constexpr (MODE == ROWS_DATASET) oa.init_rows(wave, lane, m0, p.Md, p.lda, [&](int row) { return dataset_row(p, g, row); });

    // issue the loads of stage-slot `buf` for k-tile kt whose index l satisfies l % NPART == part
    auto issue = [&](int kt, int buf, int part) {
      bf16_t *sa = smem + buf * STAGE, *sb = sa + BM * BK;
      const bool full = (kt + 1) * BK <= p.Kd;
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        if (l % NPART != part) continue;
        if (l < OpA::NI) oa.load(l, ra, sa, wave, kt, p.Kd, p.lda, full);
        else ob.load(l - OpA::NI, rb, sb, wave, kt, p.Kd, p.ldb, full);
      }
    };

    Frag<BM, BK, AT> fa[MI];
    Frag<BN, BK, BT> fb[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[i].init(wm * TM + i * 32, lane);
#pragma unroll
    for (int j = 0; j < NI; ++j) fb[j].init(wn * TN + j * 32, lane);

#pragma unroll
    for (int s = 0; s < NS - 1; ++s) {
      if (s < KT) {
#pragma unroll
        for (int q = 0; q < NPART; ++q) issue(s, s, q);
      }
    }

    for (int kt = 0; kt < KT; ++kt) {
      // k-tile kt has landed once only the loads of the younger in-flight stages are outstanding
      if (kt + NS - 1 <= KT) wait_vmcnt<(NS - 2) * NL>(); else wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();      // all waves' loads of kt visible; everyone is done with kt-1
      const bool more = kt + NS - 1 < KT;
      const bf16_t *S = smem + (kt % NS) * STAGE;
      // fragments are double-buffered in registers: the LDS reads of MFMA group kk+1 and this
      // group's share of the next stage's global loads are issued before the MFMAs of group kk,
      // which then run as one raised-priority cluster
      bf16x8 af[2][MI], bfr[2][NI];
      // transpose reads (untracked by the compiler's lgkmcnt accounting) go first, so that the
      // newest outstanding reads are always the ones the compiler counts
      if (BT && !AT) {
#pragma unroll
        for (int j = 0; j < NI; ++j) bfr[0][j] = fb[j].read(S + BM * BK, 0);
      }
#pragma unroll
      for (int i = 0; i < MI; ++i) af[0][i] = fa[i].read(S, 0);
      if (!(BT && !AT)) {
#pragma unroll
        for (int j = 0; j < NI; ++j) bfr[0][j] = fb[j].read(S + BM * BK, 0);
      }
#pragma unroll
      for (int kk = 0; kk < NPART; ++kk) {
        const int cur = kk & 1, nxt = cur ^ 1;
        if (kk + 1 < NPART) {
          if (BT && !AT) {
#pragma unroll
            for (int j = 0; j < NI; ++j) bfr[nxt][j] = fb[j].read(S + BM * BK, kk + 1);
          }
#pragma unroll
          for (int i = 0; i < MI; ++i) af[nxt][i] = fa[i].read(S, kk + 1);
          if (!(BT && !AT)) {
#pragma unroll
            for (int j = 0; j < NI; ++j) bfr[nxt][j] = fb[j].read(S + BM * BK, kk + 1);
          }
        }
        if (more) issue(kt + NS - 1, (kt + NS - 1) % NS, kk);
        if (AT || BT) {
          // LDS reads issued per MFMA group (transpose reads count two per fragment); the reads of
          // group kk + 1, if any, are the newest ones and may stay outstanding
          constexpr int RD = (AT ? 2 : 1) * MI + (BT ? 2 : 1) * NI;
          if (kk + 1 < NPART) wait_frags<RD>(af[cur], bfr[cur]); else wait_frags<0>(af[cur], bfr[cur]);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            // operands swapped: the accumulator tile is C^T, so a lane owns one row m of C and
            // groups of four consecutive columns n (see the epilogue)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[cur][j], af[cur][i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- epilogue.  With the operands swapped in the MFMA, a lane holds groups of four consecutive columns of one row.  Of slice
  // i (32 rows x TN columns) it holds, e = 0 .. 3 (tile-relative):
  //   32 x 32 tiles: row lane % 32,        group c: col 32 (c / 4) + 8 (c % 4) + 4 (lane / 32) + e = acc[i][c / 4][4 (c % 4) + e]
  //   16 x 16 tiles: row 16 h + lane % 16, group c: col 16 c + 4 (lane / 16) + e                   = acc16[2 i + h][c][e]
  // bf16 outputs and the elementwise operand E
  // go through a per-wave LDS staging slice of 32 rows x TN columns, so that every global access
  // of the epilogue is a 16-byte vector, 8 lanes to a 128-byte row segment.
  constexpr int NH = 32 / RT, NC = TN / (4 * (64 / RT));    // rows and column groups of a lane per slice
  const int lrow = lane & (RT - 1), lq = lane / RT;
  auto gcol = [&](int c) -> int { return RT == 32 ? (c >> 2) * 32 + (c & 3) * 8 + lq * 4 : c * 16 + lq * 4; };
  auto val = [&](int i, int h, int c, int e) -> float {
    if constexpr (PP) return acc16[2 * i + h][c][e];
    else return acc[i][c >> 2][4 * (c & 3) + e];
  };
  auto row_total = [&](float v) -> float {                  // over the lanes that share a row
    if (RT == 16) v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
  };
  const float *bias = p.bias ? p.bias + (long long)g * p.sBiasg : nullptr;
  constexpr int SLD = TN + 8;                               // staging row stride (elements)
  bf16_t *stg = smem + wave * (32 * SLD);
  constexpr int CPRW = TN / 8;                              // 16-byte chunks per staged row
  constexpr int SIT = 32 * CPRW / 64;                       // chunks per lane per slice
  static_assert(32 * CPRW % 64 == 0, "staging slice");
  const int nw0 = n0 + wn * TN;                             // first column of this wave
  const bool nfull = n0 + BN <= p.Nd;                       // no ragged columns in this tile (uniform)
  // this lane's 4-column groups of the bias vector, loaded once for all row slices
  float bv[NC][4];
  if (EPI == EPI_FWD_ACT || EPI == EPI_IPDOT || EPI == EPI_LOGITS) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int n = nw0 + gcol(c);
      if (bias && nfull) {
        const float4 b4 = *reinterpret_cast<const float4 *>(bias + n);
        bv[c][0] = b4.x; bv[c][1] = b4.y; bv[c][2] = b4.z; bv[c][3] = b4.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[c][e] = (bias && n + e < p.Nd) ? bias[n + e] : 0.0f;
      }
    }
  }

  // rows [mrow0, mrow0+32) x this wave's TN columns of a bf16 matrix: global -> registers (so the
  // next slice can be in flight while the current one is processed), registers -> staging
  auto load_slice = [&](const bf16_t *src, int ld, int mrow0, int ncols, uint4 (&r)[SIT]) {
#pragma unroll
    for (int it = 0; it < SIT; ++it) {
      const int c = it * 64 + lane, row = c / CPRW, cc = c % CPRW;
      r[it] = make_uint4(0, 0, 0, 0);
      if (mrow0 + row < p.Md && nw0 + cc * 8 < ncols)
        r[it] = ld_once(src + (long long)(mrow0 + row) * ld + nw0 + cc * 8);
    }
  };
  auto put_slice = [&](const uint4 (&r)[SIT]) {
#pragma unroll
    for (int it = 0; it < SIT; ++it) {
      const int c = it * 64 + lane, row = c / CPRW, cc = c % CPRW;
      *reinterpret_cast<uint4 *>(stg + row * SLD + cc * 8) = r[it];
    }
  };
  uint4 ereg[2][SIT];
  const bf16_t *Eg = p.E ? static_cast<const bf16_t *>(p.E) + (long long)g * p.sEg : nullptr;
  constexpr bool USES_E = EPI == EPI_IPDOT || (EPI == EPI_BWD && ACT != ACT_NONE);
  if (USES_E) load_slice(Eg, p.lde, m0 + slice_row(0), p.Nd, ereg[0]);
  // staging -> global
  auto stage_out = [&](bf16_t *dst, int ld, int mrow0, int ncols) {
#pragma unroll
    for (int it = 0; it < SIT; ++it) {
      const int c = it * 64 + lane, row = c / CPRW, cc = c % CPRW;
      const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * SLD + cc * 8);
      if (mrow0 + row < p.Md && nw0 + cc * 8 < ncols)
        st_once(dst + (long long)(mrow0 + row) * ld + nw0 + cc * 8, v);
    }
  };
  auto piece = [&](int h, int c) -> bf16_t * { return stg + (h * RT + lrow) * SLD + gcol(c); };

  if (EPI == EPI_FWD_ACT || EPI == EPI_BWD || EPI == EPI_IPDOT) __syncthreads();   // stages are dead
  static_assert(32 * (TN / 4) % 64 == 0, "fp32 staging slice");

  float *red = reinterpret_cast<float *>(smem + NW * 32 * SLD);   // [WN][BM] row partials of the waves
  // add the WN waves' row partials in wave order and write part[g][tn][m]
  auto finish_rows_to = [&](const float *src, float *dst) {
    float *part = dst + (long long)g * p.sPartg + (long long)tn * p.sPartTile;
    for (int r = tid; r < BM; r += NT) {
      float v = 0.0f;
#pragma unroll
      for (int w = 0; w < WN; ++w) v += src[w * BM + r];
      if (m0 + r < p.Md) part[m0 + r] = v;
    }
  };
  auto finish_rows = [&]() {
    __syncthreads();
    finish_rows_to(red, p.part);
  };
  // squares of the four bf16 values packed in pk
  auto sq4 = [](uint2 pk) -> float {
    const float a = __uint_as_float(pk.x << 16), b = __uint_as_float(pk.x & 0xffff0000u);
    const float c = __uint_as_float(pk.y << 16), d = __uint_as_float(pk.y & 0xffff0000u);
    return fmaf(a, a, fmaf(b, b, fmaf(c, c, d * d)));
  };

  if (EPI == EPI_IPDOT) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int mrow0 = m0 + slice_row(i);
      if (i + 1 < MI) load_slice(Eg, p.lde, m0 + slice_row(i + 1), p.Nd, ereg[(i + 1) & 1]);
      put_slice(ereg[i & 1]);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        float rs = 0.0f, es = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const uint2 ev = *reinterpret_cast<const uint2 *>(piece(h, c));
          if (ACT == IPDOT_NORMS) es += sq4(ev);
          const float e4[4] = {__uint_as_float(ev.x << 16), __uint_as_float(ev.x & 0xffff0000u),
                               __uint_as_float(ev.y << 16), __uint_as_float(ev.y & 0xffff0000u)};
#pragma unroll
          for (int e = 0; e < 4; ++e) rs = fmaf(e4[e], val(i, h, c, e) + bv[c][e], rs);   // E is zero outside the matrix
        }
        rs = row_total(rs);
        if (lq == 0) red[wn * BM + slice_row(i) + h * RT + lrow] = rs;
        if (ACT == IPDOT_NORMS) {
          es = row_total(es);
          if (lq == 0) red[(WN + wn) * BM + slice_row(i) + h * RT + lrow] = es;
        }
      }
    }
    finish_rows();
    if (ACT == IPDOT_NORMS) finish_rows_to(red + WN * BM, p.part2);
    return;
  }

  if (EPI == EPI_FWD_ACT) {
    bf16_t *C = static_cast<bf16_t *>(p.C) + (long long)g * p.sCg;
    bf16_t *C2 = p.C2 ? static_cast<bf16_t *>(p.C2) + (long long)g * p.sC2g : nullptr;
    const int ncols = p.pad_to_ld ? p.ldc : p.Nd;           // pad columns are written as zeros
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int mrow0 = m0 + slice_row(i);
      uint2 dpk[NH][NC];
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        float rs = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          float a4[4], d4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            // columns beyond Nd: accumulator and bias are both zero there (operand rows past the
            // matrix read as zeros), so phi(0) = 0 is what the pad columns of C receive
            act_fwd<ACT>(val(i, h, c, e) + bv[c][e], a4[e], d4[e]);
          }
          uint2 apk;
          apk.x = pack2bf(a4[0], a4[1]); apk.y = pack2bf(a4[2], a4[3]);
          dpk[h][c].x = pack2bf(d4[0], d4[1]); dpk[h][c].y = pack2bf(d4[2], d4[3]);
          *reinterpret_cast<uint2 *>(piece(h, c)) = apk;
          rs += sq4(apk);
        }
        if (p.part) {
          rs = row_total(rs);
          if (lq == 0) red[wn * BM + slice_row(i) + h * RT + lrow] = rs;
        }
      }
      stage_out(C, p.ldc, mrow0, ncols);
      if (ACT == ACT_GELU && C2) {
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
          for (int c = 0; c < NC; ++c) *reinterpret_cast<uint2 *>(piece(h, c)) = dpk[h][c];
        stage_out(C2, p.ldc2, mrow0, ncols);
      }
    }
    if (p.part) finish_rows();
    return;
  }

  if (EPI == EPI_BWD) {
    bf16_t *C = static_cast<bf16_t *>(p.C) + (long long)g * p.sCg;
    const int ncols = p.pad_to_ld ? p.ldc : p.Nd;
    static_assert(TN % 64 == 0 || TN == 32, "column sums: lanes map to columns");
    float cs[(TN + 63) / 64];                            // column sums over this wave's rows, one column per lane
#pragma unroll
    for (int c = 0; c < (TN + 63) / 64; ++c) cs[c] = 0.0f;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int mrow0 = m0 + slice_row(i);
      if (ACT != ACT_NONE) {
        if (i + 1 < MI) load_slice(Eg, p.lde, m0 + slice_row(i + 1), p.Nd, ereg[(i + 1) & 1]);
        put_slice(ereg[i & 1]);
      }
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        float rs = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          float e4[4] = {1.0f, 1.0f, 1.0f, 1.0f};
          if (ACT != ACT_NONE) {
            const uint2 ev = *reinterpret_cast<const uint2 *>(piece(h, c));
            e4[0] = __uint_as_float(ev.x << 16); e4[1] = __uint_as_float(ev.x & 0xffff0000u);
            e4[2] = __uint_as_float(ev.y << 16); e4[3] = __uint_as_float(ev.y & 0xffff0000u);
          }
          float o4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = val(i, h, c, e);
            o4[e] = (ACT == ACT_RELU) ? (e4[e] > 0.0f ? v : 0.0f) : (ACT == ACT_GELU ? v * e4[e] : v);
            if (!nfull && nw0 + gcol(c) + e >= p.Nd) o4[e] = 0.0f;
          }
          uint2 opk;
          opk.x = pack2bf(o4[0], o4[1]); opk.y = pack2bf(o4[2], o4[3]);
          *reinterpret_cast<uint2 *>(piece(h, c)) = opk;      // each lane overwrites the piece it read
          rs += sq4(opk);
        }
        if (p.part) {
          rs = row_total(rs);
          if (lq == 0) red[wn * BM + slice_row(i) + h * RT + lrow] = rs;
        }
      }
      stage_out(C, p.ldc, mrow0, ncols);
      if (p.cpart) {
        // bias-gradient partials: a lane adds its column of the staged slice, rows in order (rows
        // past the batch were computed from zero operands and hold zeros)
#pragma unroll
        for (int c = 0; c < (TN + 63) / 64; ++c) {
          const int col = c * 64 + lane;
          if (col < TN) {
#pragma unroll
            for (int r = 0; r < 32; ++r) cs[c] += bf2f(stg[r * SLD + col]);
          }
        }
      }
    }
    if (p.cpart) {
      float *cp = p.cpart + (long long)g * p.sCpartg + (long long)(tm * WM + wm) * p.Nd;
#pragma unroll
      for (int c = 0; c < (TN + 63) / 64; ++c) {
        const int n = nw0 + c * 64 + lane;
        if (c * 64 + lane < TN && n < p.Nd) cp[n] = cs[c];
      }
    }
    if (p.part) finish_rows();
    return;
  }

  // fp32 outputs (weight gradient, logits).  A lane holds one row and groups of four columns, so
  // direct stores would scatter 16-byte pieces over 32 rows per instruction; instead each wave
  // passes its 32 x TN slice through an fp32 staging area in LDS and writes whole row segments
  // (16 lanes x 16 bytes = 256 contiguous bytes per row).
  constexpr int FLD = TN + 4;                               // staging row stride (floats)
  constexpr int FCPR = TN / 4;                              // float4 chunks per staged row
  constexpr int FIT = 32 * FCPR / 64;                       // chunks per lane per slice
  float *stf = reinterpret_cast<float *>(smem) + wave * (32 * FLD);
  float *Cg = p.C ? static_cast<float *>(p.C) + (long long)g * p.sCg : nullptr;   // (null: EPI_WGRAD for C2 and sq64 alone)
  bf16_t *C2g = (IS_WGRAD && p.C2) ? static_cast<bf16_t *>(p.C2) + (long long)g * p.sC2g : nullptr;
  bool accumulate = EPI == EPI_WGRAD && p.accumulate;        // micro-batch accumulation: C += alpha * acc
  if (EPI == EPI_WGRAD && ksplit > 1) {                      // raw partial product of this k-slice
    Cg = p.kpart + ((long long)g * ksplit + ksl) * p.Md * p.Nd;
    p.ldc = p.Nd; p.alpha = 1.0f;
    C2g = nullptr; accumulate = false;
  }
  const bool vec_ok = (p.ldc & 3) == 0 && (!C2g || (p.ldc2 & 3) == 0);
  double sq64 = 0.0;                                        // EPI_WGRAD: squared entries of this wave's part of Gbar
  __syncthreads();                                          // stages are dead
  if constexpr (EPI == EPI_WGRAD_UPD) {
    // The optimizer step in place of the gradient store: a lane's staged float4 holds four consecutive entries
    // of one row of Gbar_l; the parameters, their state and their bf16 shadow sit at the same offsets.
    const long long goff = (long long)g * p.sCg;
    float *X = p.upd_x + goff;                               // (loaded through upd_prefetch, stored through these)
    float *V = p.upd_v ? p.upd_v + goff : nullptr;
    float *Mo = p.upd_m ? p.upd_m + goff : nullptr;
    bf16_t *__restrict__ SH = p.upd_shadow ? p.upd_shadow + goff : nullptr;
    OptHyper h = {p.upd_lr, p.upd_momentum, p.upd_beta1, p.upd_beta2, p.upd_eps, p.upd_wd, p.upd_c1, p.upd_c2};
    if (p.upd_scal) { h.lr = p.upd_scal[0]; h.c1 = p.upd_scal[1]; h.c2 = p.upd_scal[2]; }     // uniform loads
    constexpr int opt = ACT;                                 // the optimizer travels in the activation slot
    float sq = 0.0f;
    constexpr int HB = UHB, BPS = UBPS, NBATCH = MI * BPS;
    auto &where = upd_where;
    auto &prefetch = upd_prefetch;
    if constexpr (!UPD_EARLY) prefetch(0);
#pragma unroll
    for (int bi = 0; bi < NBATCH; ++bi) {
      if (bi % BPS == 0) {                                   // a new slice: accumulators -> staging
        const int i = bi / BPS;
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
          for (int c = 0; c < NC; ++c)
            *reinterpret_cast<float4 *>(stf + (h * RT + lrow) * FLD + gcol(c)) =
                make_float4(val(i, h, c, 0) * p.alpha, val(i, h, c, 1) * p.alpha, val(i, h, c, 2) * p.alpha, val(i, h, c, 3) * p.alpha);
      }
      if (bi + 1 < NBATCH) prefetch(bi + 1);
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        int m, n, row, cc;
        where(bi, u, m, n, row, cc);
        if (m >= p.Md || n >= p.Nd) continue;
        const long long o = (long long)m * p.ldc + n;
        const float4 gv = *reinterpret_cast<const float4 *>(stf + row * FLD + cc * 4);
        const float gs[4] = {gv.x, gv.y, gv.z, gv.w};
        float xs[4] = {xq[bi & 1][u].x, xq[bi & 1][u].y, xq[bi & 1][u].z, xq[bi & 1][u].w};
        float vs[4] = {vq[bi & 1][u].x, vq[bi & 1][u].y, vq[bi & 1][u].z, vq[bi & 1][u].w};
        float ms[4] = {mq[bi & 1][u].x, mq[bi & 1][u].y, mq[bi & 1][u].z, mq[bi & 1][u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) opt_step_elem<opt>(xs[e], gs[e], vs[e], ms[e], h);
        sq = fmaf(gs[0], gs[0], fmaf(gs[1], gs[1], fmaf(gs[2], gs[2], fmaf(gs[3], gs[3], sq))));
        st_once(X + o, make_float4(xs[0], xs[1], xs[2], xs[3]));
        if (opt != OPT_SGD) st_once(V + o, make_float4(vs[0], vs[1], vs[2], vs[3]));
        if (opt == OPT_ADAMW) st_once(Mo + o, make_float4(ms[0], ms[1], ms[2], ms[3]));
        if (SH) {
          uint2 w;
          w.x = pack2bf(xs[0], xs[1]); w.y = pack2bf(xs[2], xs[3]);
          st_once(SH + o, w);
        }
        if (C2g) {
          uint2 w;
          w.x = pack2bf(gs[0], gs[1]); w.y = pack2bf(gs[2], gs[3]);
          st_once(C2g + (long long)m * p.ldc2 + n, w);
        }
      }
    }
    sq = wave_sum(sq);
    if (lane == 0) p.upd_sq[(long long)g * p.upd_sSqg + p.upd_slot0 + (long long)(tm * tilesN + tn) * NW + wave] = sq;
    return;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int mrow0 = m0 + slice_row(i);
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        float4 o;
        if (IS_WGRAD) {
          o = make_float4(val(i, h, c, 0) * p.alpha, val(i, h, c, 1) * p.alpha, val(i, h, c, 2) * p.alpha, val(i, h, c, 3) * p.alpha);
        } else {
          o = make_float4(val(i, h, c, 0) + bv[c][0], val(i, h, c, 1) + bv[c][1], val(i, h, c, 2) + bv[c][2], val(i, h, c, 3) + bv[c][3]);
        }
        *reinterpret_cast<float4 *>(stf + (h * RT + lrow) * FLD + gcol(c)) = o;
      }
#pragma unroll
    for (int it = 0; it < FIT; ++it) {
      const int c = it * 64 + lane, row = c / FCPR, cc = c % FCPR;
      const int m = mrow0 + row, n = nw0 + cc * 4;
      if (m >= p.Md || n >= p.Nd) continue;
      float4 v = *reinterpret_cast<const float4 *>(stf + row * FLD + cc * 4);
      float *crow = Cg + (long long)m * p.ldc + n;
      if (n + 4 <= p.Nd && vec_ok) {
        if (accumulate) {
          const float4 old = *reinterpret_cast<const float4 *>(crow);
          v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w;
        }
        if (Cg) st_once(crow, v);
        if (EPI == EPI_WGRAD) sq64 += (double)fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, v.w * v.w)));
        if (C2g) {
          uint2 o;
          o.x = pack2bf(v.x, v.y); o.y = pack2bf(v.z, v.w);
          st_once(C2g + (long long)m * p.ldc2 + n, o);
        }
      } else {
        const float v4[4] = {v.x, v.y, v.z, v.w};
        for (int e = 0; e < 4; ++e) {
          if (n + e >= p.Nd) break;
          const float r = accumulate ? v4[e] + crow[e] : v4[e];
          if (Cg) crow[e] = r;
          if (EPI == EPI_WGRAD) sq64 += (double)(r * r);
          if (C2g) C2g[(long long)m * p.ldc2 + n + e] = f2bf(r);
        }
      }
    }
  }
  if (EPI == EPI_WGRAD && p.sq64) {                         // uniform
    sq64 = wave_sum(sq64);
    if (lane == 0) p.sq64[(long long)g * p.sSq64g + (long long)(tm * tilesN + tn) * NW + wave] = sq64;
  }
}

template <int BM, int BN, int BK, int WM, int WN, int NS, bool PP, bool AT, bool BT, int EPI, int ACT, int MODE>
__global__ void __launch_bounds__(WM * WN * 64)
gemm_bf16_kernel(const GemmP pin, const int tilesM, const int tilesN, const int nblk, const int chunk) {
  // XCD-aware remap of the flat work-group id
  const int bid = blockIdx.x;
  const int lb = (bid & 7) * chunk + (bid >> 3);
  if (lb >= nblk) return;
  gemm_bf16_tile<BM, BN, BK, WM, WN, NS, PP, AT, BT, EPI, ACT, MODE>(pin, tilesM, tilesN, lb);
}

// Weight gradients of several layers in one launch (64 x 256 x 32 tiles of short batches, two-stage 128 x 128 or 64 x 128
// tiles of narrow nets and medium batches): what separate launches add is their starts, their nearly empty last waves and, where a
// layer alone has fewer tiles than the chip has places, idle CUs.  The tiles of the layers lie one behind the other;
// a work-group picks its layer by the tile number.
// In front of them go the blocks of a step's end that need nothing but the signals (StepTail): launches of their own cost their
// starts and a gap each.
struct WgradMany {
  enum { MAXN = 8 };
  struct Layer {
    const void *A, *B;
    long long sAg, sBg;
    int lda, ldb, Md, Nd;
    void *C, *C2;
    int ldc, ldc2;
    float *upd_x, *upd_v, *upd_m;
    bf16_t *upd_shadow;
    int upd_slot0, ksplit, kchunk;
    float *kpart;
    double *sq64;
  };
  int n, nblk, chunk;
  int end[MAXN], tilesM[MAXN], tilesN[MAXN];
  int Kd, groups, accumulate;                     // of every layer
  long long sCg, sC2g;
  float alpha;
  const int *rows, *gperm;
  float upd_lr, upd_momentum, upd_beta1, upd_beta2, upd_eps, upd_wd, upd_c1, upd_c2;
  const float *upd_scal;
  float *upd_sq; long long upd_sSqg, sSq64g;
  Layer p[MAXN];
};
static_assert(sizeof(WgradMany) + sizeof(StepTail) <= 4096, "kernel arguments");

template <int OPT>
__device__ __forceinline__ void step_tail_block(const StepTail &t, int id) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int ncf = t.cf_x * t.cf.n * t.groups;
  if (id < ncf) {
    const int bx = id % t.cf_x, l = id / t.cf_x % t.cf.n, g = id / (t.cf_x * t.cf.n);
    col_finish_block<OPT>(t.cf, bx, t.cf_x, l, g, reinterpret_cast<float *>(smem_raw));
    return;
  }
  id -= ncf;
  const int nb = t.st.nb_done;
  if (id >= nb * t.groups) return;
  const int g = id / nb, blk = id - g * nb;
  StatsSums o = {{0.0, 0.0, 0.0, 0.0, 0.0}};
  stats_samples<256>(t.st, g, blk, nb, o, reinterpret_cast<float *>(smem_raw));
  const double r = stats_block_sums<256>(o, reinterpret_cast<double *>(smem_raw + 4096));
  if (threadIdx.x < 5 && threadIdx.x != 1) t.st.partials[((long long)g * 5 + threadIdx.x) * STATS_PBLK + blk] = r;
}

template <int BM, int BN, int BK, int WM, int WN, bool PP, int EPI, int ACT>
__device__ __forceinline__ void wgrad_many_tile(const WgradMany &q, const int bid) {
  int lb = (bid & 7) * q.chunk + (bid >> 3);
  if (lb >= q.nblk) return;
  int l = 0;
  while (lb >= q.end[l]) ++l;                     // uniform; end[n - 1] == nblk
  if (l > 0) lb -= q.end[l - 1];
  const WgradMany::Layer &y = q.p[l];
  GemmP p = {};
  p.A = y.A; p.B = y.B; p.sAg = y.sAg; p.sBg = y.sBg; p.lda = y.lda; p.ldb = y.ldb; p.a_trans = p.b_trans = 1;
  p.Md = y.Md; p.Nd = y.Nd; p.Kd = q.Kd; p.groups = q.groups;
  p.C = y.C; p.sCg = q.sCg; p.ldc = y.ldc; p.C2 = y.C2; p.sC2g = q.sC2g; p.ldc2 = y.ldc2;
  p.alpha = q.alpha; p.accumulate = q.accumulate; p.rows = q.rows; p.rows_is_k = 1; p.gperm = q.gperm;
  p.ksplit = y.ksplit; p.kchunk = y.kchunk; p.kpart = y.kpart;
  p.upd_x = y.upd_x; p.upd_v = y.upd_v; p.upd_m = y.upd_m; p.upd_shadow = y.upd_shadow;
  p.upd_lr = q.upd_lr; p.upd_momentum = q.upd_momentum; p.upd_beta1 = q.upd_beta1; p.upd_beta2 = q.upd_beta2;
  p.upd_eps = q.upd_eps; p.upd_wd = q.upd_wd; p.upd_c1 = q.upd_c1; p.upd_c2 = q.upd_c2; p.upd_scal = q.upd_scal;
  p.upd_sq = q.upd_sq; p.upd_sSqg = q.upd_sSqg; p.upd_slot0 = y.upd_slot0;
  p.sq64 = y.sq64; p.sSq64g = q.sSq64g;
  gemm_bf16_tile<BM, BN, BK, WM, WN, 2, PP, true, true, EPI, ACT>(p, q.tilesM[l], q.tilesN[l], lb);
}
template <int BM, int BN, int BK, int WM, int WN, int EPI, int ACT>
__global__ void __launch_bounds__(256) wgrad_many_kernel(const WgradMany q, const StepTail t) {
  if ((int)blockIdx.x < t.blocks) { step_tail_block<EPI == EPI_WGRAD_UPD ? ACT : -1>(t, blockIdx.x); return; }
  // (t.blocks is a multiple of 8: the XCDs stay where they were)
  wgrad_many_tile<BM, BN, BK, WM, WN, false, EPI, ACT>(q, blockIdx.x - t.blocks);
}
// Slices of the layers' reductions on 256 x 256 tiles (GemmP::fine == 2): 64 KB of operands into a CU for 8.4 MFLOP, where 64 x 128 tiles
// take 24 KB for 1.  A k-tile takes 1.5 us, of which its MFMAs are 1.1 at the 1.95 PFLOP/s of a stream from registers; three 64 x 128
// tiles to a CU take 1.47 for 3.1 MFLOP and 72 KB.
__global__ void __launch_bounds__(512, 2) wgrad_slices_kernel(const WgradMany q) {
  wgrad_many_tile<256, 256, 64, 2, 4, true, EPI_WGRAD, ACT_NONE>(q, blockIdx.x);
}

// Tiles that ragged groups have (ragged_tile)
long long ragged_blocks(const GemmP &p, int bm, int tilesN) {
  long long n = 0;
  for (int g = 0; g < p.groups; ++g) n += (long long)((p.rows_host[g] + bm - 1) / bm) * tilesN;
  return n;
}

template <int BM, int BN, int BK, int WM, int WN, int NS, bool PP, bool AT, bool BT, int EPI, int ACT, int MODE>
hipError_t launch_mode(const GemmP &p, hipStream_t s) {
  constexpr int NT = WM * WN * 64;
  constexpr size_t tile_bytes = (size_t)NS * (BM + BN) * BK * sizeof(bf16_t);
  constexpr size_t epi_bf16 = (size_t)WM * WN * 32 * (BN / WN + 8) * sizeof(bf16_t) + (size_t)(EPI == EPI_IPDOT ? 2 : 1) * WN * BM * sizeof(float);
  constexpr size_t epi_f32 = (size_t)WM * WN * 32 * (BN / WN + 4) * sizeof(float);
  constexpr size_t epi_bytes = epi_bf16 > epi_f32 ? epi_bf16 : epi_f32;
  constexpr size_t lds = tile_bytes > epi_bytes ? tile_bytes : epi_bytes;
  static_assert(lds <= 160 * 1024, "LDS budget");
  auto kern = gemm_bf16_kernel<BM, BN, BK, WM, WN, NS, PP, AT, BT, EPI, ACT, MODE>;
  // once per kernel variant, also when several host threads (each with a context of its own) launch it first together
  static std::once_flag attr_once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [&] {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr_err != hipSuccess) return attr_err;
  const int tilesM = (p.Md + BM - 1) / BM, tilesN = (p.Nd + BN - 1) / BN;
  long long nblk = (long long)tilesM * tilesN * p.groups * ((EPI == EPI_WGRAD && p.ksplit > 1) ? p.ksplit : 1);
  if (nblk <= 0) return hipSuccess;
  if (nblk > 0x3fffffff) return hipErrorInvalidValue;
  if (MODE == ROWS_OWN) nblk = ragged_blocks(p, BM, tilesN);
  const int chunk = (int)((nblk + 7) / 8);
  hipLaunchKernelGGL(kern, dim3(chunk * 8), dim3(NT), lds, s, p, tilesM, tilesN, (int)nblk, chunk);
  return hipGetLastError();
}

template <int BM, int BN, int BK, int WM, int WN, int NS, bool PP, bool AT, bool BT, int EPI, int ACT>
hipError_t launch_cfg(const GemmP &p, hipStream_t s) {
  if constexpr (EPI != EPI_WGRAD && EPI != EPI_WGRAD_UPD) {
    if (p.rows) return p.aidx ? hipErrorInvalidValue : launch_mode<BM, BN, BK, WM, WN, NS, PP, AT, BT, EPI, ACT, ROWS_OWN>(p, s);
    if constexpr (EPI == EPI_FWD_ACT && BM == 64)
      if (p.aidx) return launch_mode<BM, BN, BK, WM, WN, NS, PP, AT, BT, EPI, ACT, ROWS_DATASET>(p, s);
  }
  return p.aidx ? hipErrorInvalidValue : launch_mode<BM, BN, BK, WM, WN, NS, PP, AT, BT, EPI, ACT, ROWS_PLAIN>(p, s);
}

int tiled_shape(int Md, int Nd, int groups, const int *rows_host);
// Reductions up to this length keep the two-stage loop in 256 x 256 tiles: the pipelined loop fetches two k-tiles beyond the
// last one and starts later, which a handful of k-tiles does not pay back (784-512-512-10, 8 replicas, b = 4096, one tile
// per CU: 285.7 us per step with the pipelined loop everywhere, 281.9 with this line at 512, 283.0 at 1024; 1024-wide
// layers, K = 1024, b = 4096: 2184 us with the two-stage loop, 2006 with the pipelined one).
constexpr int PIPE_MIN_K = 512;

// Tile shape by problem size: the large shape where its rounds of work-groups take less time (tiled_shape, gemm_bf16_wgrad_shape),
// otherwise a 128x128 (or 128x64 for narrow outputs, 64x128 for outputs of at most 64 rows) tile.
template <bool AT, bool BT, int EPI, int ACT>
hipError_t launch_shape(const GemmP &p, hipStream_t s) {
  constexpr bool IS_WGRAD = EPI == EPI_WGRAD || EPI == EPI_WGRAD_UPD;
  switch (IS_WGRAD ? gemm_bf16_wgrad_shape(p.Md, p.Nd, p.Kd, p.groups, p.upd_x != nullptr, p.rows_host)
                   : tiled_shape(p.Md, p.Nd, p.groups, p.rows_host)) {
    case 0: return launch_cfg<128, 64, 64, 4, 1, 3, false, AT, BT, EPI, ACT>(p, s);
    case 3: return hipErrorInvalidValue;         // (launch_wgrad_many)
    case 2:
      if constexpr (!IS_WGRAD) if (p.Kd <= PIPE_MIN_K) return launch_cfg<256, 256, 64, 2, 4, 2, false, AT, BT, EPI, ACT>(p, s);
      return launch_cfg<256, 256, 64, 2, 4, 2, true, AT, BT, EPI, ACT>(p, s);
    case 4:
      if constexpr (!IS_WGRAD) return launch_cfg<64, 128, 64, 2, 2, 6, false, AT, BT, EPI, ACT>(p, s);
      else return hipErrorInvalidValue;
    case 5:
      if constexpr (EPI == EPI_WGRAD_UPD) return launch_cfg<128, 256, 32, 2, 4, 3, false, AT, BT, EPI, ACT>(p, s);
      else return hipErrorInvalidValue;
    default: {
      // Two stages (64 KB) let two work-groups share a CU; a deeper ring keeps one work-group fed through a long
      // reduction.  Two when the reduction is short or the launch has more blocks than CUs (measured: 2048-wide
      // layers at b = 256, 512 blocks: 43 against 62 us; 1024 blocks of a 100-wide output: 145 against 163 us;
      // 256 blocks: the deeper ring wins); four stages (128 KB, still one work-group per CU, three k-tiles in
      // flight: such launches are bound by the latency of their operand stream) otherwise.
      const long long nblk = (long long)((p.Md + 127) / 128) * ((p.Nd + 127) / 128) * p.groups *
                             ((EPI == EPI_WGRAD && p.ksplit > 1) ? p.ksplit : 1);
      if (p.Kd <= 1024 || nblk > 256) return launch_cfg<128, 128, 64, 2, 2, 2, false, AT, BT, EPI, ACT>(p, s);
      return launch_cfg<128, 128, 64, 2, 2, 4, false, AT, BT, EPI, ACT>(p, s);
    }
  }
}

template <bool AT, bool BT, int EPI>
hipError_t launch_act(const GemmP &p, hipStream_t s) {
  if constexpr (EPI == EPI_WGRAD_UPD) {          // the optimizer is a compile-time constant of the fused epilogue
    switch (p.upd_opt) {
      case OPT_SGD: return launch_shape<AT, BT, EPI, OPT_SGD>(p, s);
      case OPT_SHB: return launch_shape<AT, BT, EPI, OPT_SHB>(p, s);
      case OPT_ADAMW: return launch_shape<AT, BT, EPI, OPT_ADAMW>(p, s);
      case OPT_ADAGRAD: return launch_shape<AT, BT, EPI, OPT_ADAGRAD>(p, s);
      default: return hipErrorInvalidValue;
    }
  }
  if constexpr (EPI == EPI_FWD_ACT || EPI == EPI_BWD) {
    switch (p.act) {
      case ACT_RELU: return launch_shape<AT, BT, EPI, ACT_RELU>(p, s);
      case ACT_GELU: return launch_shape<AT, BT, EPI, ACT_GELU>(p, s);
      default: return launch_shape<AT, BT, EPI, ACT_NONE>(p, s);
    }
  }
  if constexpr (EPI == EPI_IPDOT) if (p.part2) return launch_shape<AT, BT, EPI, IPDOT_NORMS>(p, s);
  return launch_shape<AT, BT, EPI, ACT_NONE>(p, s);
}

constexpr long long FEW_TILES = 128;

// Time of `blocks` 128 x 128 tiles per k-tile: full rounds of two work-groups to a CU and the last one
double rounds_128(long long blocks) {
  const long long full = blocks / 512, rem = blocks - full * 512;
  const double last = rem > 256 ? 1.42 : rem == 0 ? 0.0 : full == 0 ? 1.13 : 1.13 + 0.29 * (double)rem / 256;
  return 1.42 * (double)full + last;
}

// Tiles of e x e that ragged groups make of an output Nd wide
long long tile_count(int Nd, int groups, const int *rows_host, int e) {
  long long tm = 0;
  for (int g = 0; g < groups; ++g) tm += (rows_host[g] + e - 1) / e;
  return tm * ((Nd + e - 1) / e);
}

int tiled_shape(int Md, int Nd, int groups, const int *rows_host) {
  if (Nd <= 64) return 0;
  // up to 64 rows (the first local batch sizes): the launch streams its B operand (the weights) once and is bound by
  // that stream; a 64-row tile leaves LDS for a ring of six stages, five k-tiles of B in flight per work-group
  // (config 3 at b = 64 against the 128 x 128 tile with four stages: forward 4.1 -> 4.3 TB/s of weight bytes,
  // backward-data 4.5 -> 5.0-5.1, the step 1.17 -> 1.155 ms)
  if (Md <= 64) return 4;
  // 256 x 256 tiles or 128 x 128: whichever takes less time by rounds of work-groups.  Per k-tile of 64 a round of large tiles, one
  // to a CU, takes as long as 1.5 us against 1.13 for 128 x 128 tiles alone on their CUs and 1.42 for two to a CU (fitted to steps;
  // padding counts, since it is computed).  us per step, 128 x 128 -> 256 x 256 where the line now lies beyond them, or the other
  // way round: 16 replicas, 3072-2048-2048-100 b = 257 1252 -> 1058, b = 900 (256 x 256 either way) 1657; 3072-1024-1024-100
  // b = 700 827 -> 683, b = 512 (128 x 128) 600, 615 with large tiles; 4 replicas, b = 1024 368 with large tiles -> 282 (with the
  // weight gradients); 784-512-512-10, 8 replicas, b = 3000 232 -> 214, b = 2048 (128 x 128) 169, 188 with large tiles;
  // 784-200-10, 16 replicas, b = 4096 283 -> 259
  const long long t256 = (long long)((Md + 255) / 256) * ((Nd + 255) / 256) * groups;
  const long long t128 = (long long)((Md + 127) / 128) * ((Nd + 127) / 128) * groups;
  if (Md > 128 && Nd > 128 && 1.5 * (double)((t256 + 255) / 256) <= rounds_128(t128)) {
    if (!rows_host) return 2;
    // Workers with batches of their own make fewer tiles, and the large ones soon leave most CUs idle: the largest worker's shape
    // goes where 128 x 128 tiles cost a tenth less (less than that the model does not tell); second places that a single round
    // does not fill count as far as it does.  us per step, always 256 x 256 -> this line (tiles of 256, of 128): 16 replicas,
    // 784-384-384-10 one of 2048 samples beside fifteen of 257 (76, 183) 159 -> 135; 784-768-768-768-100, 1024 beside 130
    // (57, 228) 269 -> 233; 784-432-432-432-10, 2 to 1221 samples (82, 300) 336 -> 284; 10 replicas, 784-496-496-496-10, 2717 beside 169
    // (40, 160) 334 -> 251.  Long reductions at more than 256 tiles of 128 gain nothing: 3072-1168-1168-1168-100 (115, 310) 910, 932
    const long long r256 = tile_count(Nd, groups, rows_host, 256), r128 = tile_count(Nd, groups, rows_host, 128);
    const double c128 = r128 > 256 && r128 < 512 ? 1.13 + 0.29 * (double)(r128 - 256) / 256 : rounds_128(r128);
    return 1.5 * (double)((r256 + 255) / 256) <= 1.1 * c128 ? 2 : 1;
  }
  // 128 x 128 tiles for half of the CUs or fewer: twice as many 64 x 128 ones with a deeper ring (784-512-512-10, 8 replicas:
  // b = 501, 128 tiles, a step 124 -> 107.5 us, forward 16.9 -> 11.7; b = 768, 192 tiles, would go from 128 to 140)
  return t128 <= FEW_TILES ? 4 : 1;
}

// Launches of at most this many 32 x 32 tiles go to gemm_small.hip: a latency chain instead of a nearly empty chip.  Past two
// work-groups per CU their re-reads of both operands cost more than the tiled family's empty places: forward and logits of 512
// tiles; of 384 where more than 32 classes leave the head to a launch of its own; backward-data, whose work-groups hold two
// tiles, of 1024, unless those are one row of 32768 columns, whose weights the ring streams faster.  One launch, tiled -> small, us:
//   forward 512 x 512: 16 replicas, b = 32 (256 tiles) 12.7 -> 9.6; 8 replicas, b = 128 (512) 12.7 -> 11.5, b = 256 (1024)
//     13.6 -> 16.3; 2048 x 2048, 16 replicas, b = 32 (1024) 34 -> 53
//   backward 512 x 512, 8 replicas: b = 256 (1024) 13.1 -> 11.3, b = 501 (2048) 13.1 -> 17.3; 2048 x 2048, 16 replicas, b = 32
//     27.6 -> 31.1; 1024 x 1024, 32 replicas, b = 32 17.8 -> 19.3
//   logits and head 512 -> 10, 8 replicas, b = 32 9.8 -> 5.0; 512 -> 100, 8 replicas, b = 512 (512) 17.3 -> 18.0, b = 1024
//     (1024) 19.1 -> 23.2
//   3072-1024-1024-100, 1 replica, b = 1024 (1024 tiles of the 64 x 128 ring's 128): the step 189 on the ring, 218 small
constexpr long long SMALL_TILES = 1024;
long long small_limit(int epi, int Md, int Nd, int groups) {
  if (epi == EPI_BWD) return (long long)Nd * groups < 32768 ? SMALL_TILES : SMALL_TILES / 2;
  return epi == EPI_LOGITS && Nd > 32 ? 384 : 512;
}
long long small_tiles(int Md, int Nd, int groups) { return (long long)((Md + 31) / 32) * ((Nd + 31) / 32) * groups; }

template <int BM, int BN, int BK, int WM, int WN, int EPI, int ACT>
hipError_t launch_many_cfg(const WgradMany &q, const StepTail &t, hipStream_t s) {
  // dynamic LDS: two stages, or the epilogue's fp32 staging slices
  constexpr size_t lds = std::max<size_t>((size_t)2 * (BM + BN) * BK * sizeof(bf16_t), (size_t)4 * 32 * (BN / WN + 4) * sizeof(float));
  static_assert(lds <= 64 * 1024 && lds >= 8192 && WM * WN == 4, "no attribute needed; room for a StepTail block");
  hipLaunchKernelGGL((wgrad_many_kernel<BM, BN, BK, WM, WN, EPI, ACT>), dim3(t.blocks + q.chunk * 8), dim3(256), lds, s, q, t);
  return hipGetLastError();
}
template <int EPI, int ACT>
hipError_t launch_many(const WgradMany &q, const StepTail &t, int shape, int fine, hipStream_t s) {
  if (shape == 1 && fine) return launch_many_cfg<64, 128, 64, 2, 2, EPI, ACT>(q, t, s);
  return shape == 3 ? launch_many_cfg<64, 256, 32, 1, 4, EPI, ACT>(q, t, s) : launch_many_cfg<128, 128, 64, 2, 2, EPI, ACT>(q, t, s);
}

hipError_t launch_wgrad_slices(const WgradMany &q, hipStream_t s) {
  constexpr size_t lds = std::max<size_t>((size_t)2 * 512 * 64 * sizeof(bf16_t), (size_t)8 * 32 * (64 + 4) * sizeof(float));
  static std::once_flag attr_once;                 // (as in launch_mode)
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [&] {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void *>(wgrad_slices_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL(wgrad_slices_kernel, dim3(q.chunk * 8), dim3(512), lds, s, q);
  return hipGetLastError();
}

// operand checks that every launch relies on: 16-byte aligned rows, operands below 2 GiB per replica
bool operands_ok(const GemmP &p, int epi) {
  if (p.head.y && !(epi == EPI_LOGITS && gemm_head_fits(1, p.Md, p.Nd, p.groups))) return false;
  if ((p.lda & 7) || (p.ldb & 7)) return false;
  if ((reinterpret_cast<uintptr_t>(p.A) & 15) || (reinterpret_cast<uintptr_t>(p.B) & 15)) return false;
  if ((p.sAg & 7) || (p.sBg & 7)) return false;
  if (!p.a_trans && (p.Kd > p.lda)) return false;
  if (!p.b_trans && (p.Kd > p.ldb)) return false;
  if (p.a_trans && (p.Md > p.lda)) return false;
  if (p.b_trans && (p.Nd > p.ldb)) return false;
  const long long abytes = (long long)(p.a_trans ? p.Kd : p.Md) * p.lda * 2;
  const long long bbytes = (long long)(p.b_trans ? p.Kd : p.Nd) * p.ldb * 2;
  if (abytes >= (1LL << 31) || bbytes >= (1LL << 31)) return false;
  if (p.ksplit > 1 && (epi != EPI_WGRAD || !p.kpart || p.kchunk <= 0 || (p.kchunk & 63) ||
                       (long long)p.kchunk * p.ksplit < p.Kd || (p.Nd & 3)))
    return false;
  if ((p.rows_host && !p.rows) || (p.rows && p.rows_is_k != (epi == EPI_WGRAD)) || (p.rows && !p.rows_host && epi != EPI_WGRAD)) return false;
  if (p.rows_host)                                // the grid has exactly the tiles that these counts make
    for (int g = 0; g < p.groups; ++g) if (p.rows_host[g] < 1 || p.rows_host[g] > (p.rows_is_k ? p.Kd : p.Md)) return false;
  if (p.sq64 && (epi != EPI_WGRAD || p.ksplit > 1 || p.upd_x)) return false;
  if (epi == EPI_WGRAD && !p.C && (!p.C2 || p.accumulate || p.ksplit > 1 || p.upd_x)) return false;
  if (p.part2 && epi != EPI_IPDOT) return false;
  if (p.gather || p.aidx) {
    const int sh = epi == EPI_FWD_ACT || epi == EPI_LOGITS ? gemm_bf16_tile_shape(epi, p.Md, p.Nd, p.groups, p.rows_host) : -1;
    if (p.gather && sh != 5) return false;
    if (p.aidx && ((sh != 5 && !(sh == 4 && epi == EPI_FWD_ACT)) || p.aN < 1 || p.aldi < p.Md || p.sAg || (long long)p.aN * p.lda * 2 >= (1LL << 31)))
      return false;
  }
  if (p.upd_x && (epi != EPI_WGRAD || p.ksplit > 1 || p.accumulate || !p.upd_sq || (p.ldc & 3) || (p.Nd & 3) ||
                  (p.sCg & 3) || (reinterpret_cast<uintptr_t>(p.upd_x) & 15) || (p.C2 && ((p.ldc2 & 3) || p.ldc2 != p.ldc)) ||
                  (p.upd_opt != OPT_SGD && !p.upd_v) || (p.upd_opt == OPT_ADAMW && !p.upd_m)))
    return false;
  return true;
}

}  // namespace

bool gemm_bf16_operands_ok(const GemmP &p, int epi) { return operands_ok(p, epi); }

int gemm_bf16_tile_shape(int epi, int Md, int Nd, int groups, const int *rows_host) {
  if ((epi == EPI_FWD_ACT || epi == EPI_LOGITS || epi == EPI_BWD) && small_tiles(Md, Nd, groups) <= small_limit(epi, Md, Nd, groups))
    return 5;
  return tiled_shape(Md, Nd, groups, rows_host);
}

// (bf16: the 32-row tiles hold 32 columns; fp32: the smallest tile holds 16)
bool gemm_head_fits(int is_bf16, int Md, int Nd, int groups) {
  return is_bf16 ? Nd <= 32 && gemm_bf16_tile_shape(EPI_LOGITS, Md, Nd, groups, nullptr) == 5 : Nd <= 16;
}

// The gather rides with a launch that is a chain of latencies, as long as its blocks find a place beside the tiles (four to a CU):
// its own launch cost 3 to 8 us and a gap.  us per step: 256-10 in fp32, 4 replicas, b = 16 31.9 -> 28.6, b = 512 39.8 -> 36.6;
// 784-512-512-10, 8 replicas, b = 32 66 -> 63, b = 501 87 -> 82; 784-144-4, 9 replicas, b = 61 64.4 -> 61.4.  A first layer on
// 64 x 128 tiles, one work-group to a CU, leaves it to small logits (nothing before the weight gradients needs it).
// bf16: 32-bit byte offsets into the dataset (its rows are whole 16-byte chunks: widths are multiples of 8).
int gather_rides(int is_bf16, int L, int b, const int *dims, int groups, long long N, const int *rows_host) {
  if ((long long)((b + 3) / 4) * groups > GATHER_RIDES) return 0;
  if (!is_bf16) return 1;
  if (N * dims[0] * 2 >= (1LL << 31)) return 0;
  const int first = gemm_bf16_tile_shape(L == 1 ? EPI_LOGITS : EPI_FWD_ACT, b, dims[1], groups, rows_host);
  if (first == 5) return 1;
  return first == 4 && !rows_host && L > 1 && gemm_bf16_tile_shape(EPI_LOGITS, b, dims[L], groups, nullptr) == 5 ? 2 : 0;
}

// Weight gradients reduce over the local batch (Kd = b).  While the batch is short the launch is all epilogue
// (one or a few k-tiles, then 4 to 20 bytes of stores and loads per output entry): a 64 x 256 x 32 tile with two
// 20 KB stages lets several work-groups share a CU, which keeps far more memory requests in flight than one
// 256 x 256 work-group does; its four wavefronts sit side by side, so a work-group touches 1 KB of consecutive
// bytes in each of its 64 rows (measured against a 128 x 128 tile, 512 bytes in each of 128 rows, on config 3 at
// b = 64: 2 to 2.5 % faster with the optimizer step in the epilogue, equal at b = 256).
int gemm_bf16_wgrad_shape(int Md, int Nd, int Kd, int groups, int fused, const int *rows_host) {
  // Large tiles or 128 x 128 (narrow outputs: 128 x 64).  A launch of large tiles on a part of the CUs pays only when the reduction
  // is long: the smaller ones share a launch with other layers and fill the chip.  us per step, large -> 128-wide tiles: 4 replicas
  // of 3072-1024-1024-100 (64 large tiles), AdamW, b = 1024 368 -> 282, b = 3000 434 -> 421, b = 6000 709 (large), 731;
  // 5 replicas of 3072-1536-1536-100 (180) b = 1024 579 -> 553, b = 4096 1140 (large), 1187.  128-wide -> large: 784-512-512-10,
  // 16 replicas, b = 4096 489 -> 471; 784-768-768-768-100 (192 and 144) b = 4096 1018 -> 987, b = 1500 544 (128-wide), 566;
  // 784-640-640-10, 12 replicas, whose large tiles are 36 % padding, b = 4096 509 (128-wide), 528
  int sh = Nd <= 64 ? 0 : 1;
  if (Md >= 256 && Nd >= 512) {
    const long long tm = (Md + 255) / 256, tn = (Nd + 255) / 256, tiles = tm * tn * groups;
    long long K = Kd;                        // ragged groups: on average (the largest: 16 replicas, us per step, -> this:
    if (rows_host) {                         //   784-768-768-768-100, two of 4096 samples beside fourteen of 256, 547 -> 407;
      K = 0;                                 //   784-656-656-100, 1258 and 2517, 603 -> 570)
      for (int g = 0; g < groups; ++g) K += rows_host[g];
      K = (K + groups - 1) / groups;
    }
    if (Md >= 1024 && Nd >= 1024) { if (tiles >= (Kd > 4096 ? 1 : Kd > 2048 ? 128 : 192)) sh = 2; }
    else if (K > 2048 ? tiles >= 128 && 10LL * Md * Nd >= 7LL * tm * tn * 65536 : tiles >= 256 && 10LL * Md >= 7LL * tm * 256) sh = 2;
  }
  if (sh != 0 && Kd <= 256) return 3;        // (measured on config 3: at b = 384 and above the large tiles are faster)
  // with the optimizer step in the epilogue a medium batch is still mostly epilogue: two or three 128 x 128
  // work-groups per CU stream it better than one 256 x 256 work-group (config 3: b = 384 1.92 -> 1.87 ms per step,
  // b = 512 2.02 -> 2.00)
  if (fused && sh == 2 && Kd <= 512) return 1;
  // up to 1536 two 128 x 256 work-groups of eight wavefronts share a CU where there are tiles for two: sixteen waves keep more of
  // the epilogue's memory requests in flight than eight (3072-2048-2048-2048-100, 16 replicas, heavy ball, the three wide layers:
  // b = 600 1107 -> 1020 us, b = 1001 1196 -> 1145, b = 2048 1514 -> 1536; four wavefronts of 64 x 128 1290 / 1530 / 2170)
  if (fused && sh == 2 && Kd <= 1536 && (long long)((Md + 255) / 256) * ((Nd + 255) / 256) * groups >= 256) return 5;
  return sh;
}

int gemm_bf16_upd_slots(int Md, int Nd, int Kd, int groups, int fused, int fine, const int *rows_host) {
  const int bm[6] = {128, 128, 256, 64, 64, 128}, bn[6] = {64, 128, 256, 256, 128, 256}, nw[6] = {4, 4, 8, 4, 4, 8};
  const int sh = gemm_bf16_wgrad_tile(gemm_bf16_wgrad_shape(Md, Nd, Kd, groups, fused, rows_host), fine);
  return ((Md + bm[sh] - 1) / bm[sh]) * ((Nd + bn[sh] - 1) / bn[sh]) * nw[sh];
}

int gemm_bf16_row_parts(int epi, int Md, int Nd, int groups, const int *rows_host) {
  const int bn[6] = {64, 128, 256, 0, 128, epi == EPI_BWD ? 64 : 32};
  const int sh = gemm_bf16_tile_shape(epi, Md, Nd, groups, rows_host);
  return (Nd + bn[sh] - 1) / bn[sh];
}

void gemm_bf16_col_part_shape(int epi, int Md, int Nd, int groups, const int *rows_host, int *tile_m, int *parts_per_tile) {
  const int bm[6] = {128, 128, 256, 0, 64, 32}, wm[6] = {4, 2, 2, 0, 2, 1};
  const int sh = gemm_bf16_tile_shape(epi, Md, Nd, groups, rows_host);
  *tile_m = bm[sh];
  *parts_per_tile = wm[sh];
}

int gemm_bf16_col_parts(int epi, int Md, int Nd, int groups, const int *rows_host) {
  int bm, wm;
  gemm_bf16_col_part_shape(epi, Md, Nd, groups, rows_host, &bm, &wm);
  return (Md + bm - 1) / bm * wm;
}

size_t gemm_bf16_row_part_floats(int Nd, int groups, int cap) {
  const size_t rows = ((size_t)cap + 63) / 64 * 64;
  const size_t tiled = rows * gemm_bf16_ipdot_parts(Nd);
  // a launch of gemm_small.hip has at most SMALL_TILES tiles over all groups: 32 rows each, partials 64-rounded rows apart
  const size_t small = std::min(rows * (size_t)((Nd + 31) / 32), (size_t)(SMALL_TILES * 64 / groups));
  return std::max(tiled, small);
}

int gemm_bf16_ipdot_parts(int Nd) {
  if (Nd <= 64) return 1;
  // upper bound over the tile shapes launch_shape may pick (128-wide tiles)
  return (Nd + 127) / 128;
}

hipError_t launch_wgrad_many(const GemmP *p, int n, int shape, hipStream_t s, const StepTail *tail) {
  if (shape != 1 && shape != 3) return hipErrorInvalidValue;
  if (n < 1) return tail ? hipErrorInvalidValue : hipSuccess;
  const GemmP &c0 = p[0];
  const bool slices = shape == 1 && c0.fine == 2;
  const int bm = slices ? 256 : shape == 3 || c0.fine ? 64 : 128, bn = slices || shape == 3 ? 256 : 128;
  const bool upd = c0.upd_x != nullptr;
  if (slices && (tail || upd)) return hipErrorInvalidValue;
  StepTail t;
  std::memset(&t, 0, sizeof(t));
  if (tail) {
    t = *tail;
    // the bias gradients take their step exactly if the weights do
    if (t.groups != c0.groups || (t.cf.n > 0 && ((t.cf.upd_x != nullptr) != upd || (upd && (t.cf.upd_opt != c0.upd_opt || !t.cf.sq)) ||
                                                 (upd && t.cf.accumulate) || t.cf.n > ColFinishMany::MAXN || t.cf_x < 1 || (t.cf.cb != 64 && t.cf.cb != 256))) ||
        (t.st.nb_done > 0 && (!t.st.do_n || t.st.do_q || !t.st.partials || t.st.nb_done > STATS_PBLK)))
      return hipErrorInvalidValue;
    t.blocks = (t.groups * (t.cf_x * t.cf.n + t.st.nb_done) + 7) / 8 * 8;
  }
  for (int at = 0; at < n;) {
    WgradMany q;
    std::memset(&q, 0, sizeof(q));
    long long blocks = 0;
    for (; at < n && q.n < WgradMany::MAXN; ++at) {
      const GemmP &c = p[at];
      // one kernel variant for all: every layer carries the same optimizer step, or none
      if (!operands_ok(c, EPI_WGRAD) || !c.a_trans || !c.b_trans || (c.upd_x != nullptr) != upd ||
          (upd && c.upd_opt != c0.upd_opt) || (shape == 3 && c.ksplit > 1) || (slices && c.ksplit < 2) || c.fine != c0.fine ||
          gemm_bf16_wgrad_shape(c.Md, c.Nd, c.Kd, c.groups, upd, c.rows_host) != shape)
        return hipErrorInvalidValue;
      // and the fields that the launch holds once
      if (c.Kd != c0.Kd || c.groups != c0.groups || c.accumulate != c0.accumulate || c.sCg != c0.sCg || (c.C2 && c.sC2g != c0.sC2g) ||
          (c.C2 != nullptr) != (c0.C2 != nullptr) || c.alpha != c0.alpha || c.rows != c0.rows || (c.rows && !c.rows_is_k) ||
          c.gperm != c0.gperm || c.upd_scal != c0.upd_scal || c.upd_sq != c0.upd_sq || c.upd_sSqg != c0.upd_sSqg || c.sSq64g != c0.sSq64g)
        return hipErrorInvalidValue;
      q.tilesM[q.n] = (c.Md + bm - 1) / bm; q.tilesN[q.n] = (c.Nd + bn - 1) / bn;
      blocks += (long long)q.tilesM[q.n] * q.tilesN[q.n] * c.groups * (c.ksplit > 1 ? c.ksplit : 1);
      if (blocks > 0x3fffffff) return hipErrorInvalidValue;
      q.end[q.n] = (int)blocks;
      WgradMany::Layer &y = q.p[q.n++];
      y.A = c.A; y.B = c.B; y.sAg = c.sAg; y.sBg = c.sBg; y.lda = c.lda; y.ldb = c.ldb; y.Md = c.Md; y.Nd = c.Nd;
      y.C = c.C; y.C2 = c.C2; y.ldc = c.ldc; y.ldc2 = c.ldc2;
      y.upd_x = c.upd_x; y.upd_v = c.upd_v; y.upd_m = c.upd_m; y.upd_shadow = c.upd_shadow; y.upd_slot0 = c.upd_slot0;
      y.ksplit = c.ksplit; y.kchunk = c.kchunk; y.kpart = c.kpart; y.sq64 = c.sq64;
    }
    q.Kd = c0.Kd; q.groups = c0.groups; q.accumulate = c0.accumulate; q.sCg = c0.sCg; q.sC2g = c0.sC2g; q.alpha = c0.alpha;
    q.rows = c0.rows; q.gperm = c0.gperm;
    q.upd_lr = c0.upd_lr; q.upd_momentum = c0.upd_momentum; q.upd_beta1 = c0.upd_beta1; q.upd_beta2 = c0.upd_beta2;
    q.upd_eps = c0.upd_eps; q.upd_wd = c0.upd_wd; q.upd_c1 = c0.upd_c1; q.upd_c2 = c0.upd_c2; q.upd_scal = c0.upd_scal;
    q.upd_sq = c0.upd_sq; q.upd_sSqg = c0.upd_sSqg; q.sSq64g = c0.sSq64g;
    if (blocks <= 0 && t.blocks == 0) continue;
    q.nblk = (int)blocks;
    q.chunk = (q.nblk + 7) / 8;
    hipError_t e;
    if (slices) e = launch_wgrad_slices(q, s);
    else if (!upd) e = launch_many<EPI_WGRAD, ACT_NONE>(q, t, shape, c0.fine, s);
    else if (c0.upd_opt == OPT_SGD) e = launch_many<EPI_WGRAD_UPD, OPT_SGD>(q, t, shape, c0.fine, s);
    else if (c0.upd_opt == OPT_SHB) e = launch_many<EPI_WGRAD_UPD, OPT_SHB>(q, t, shape, c0.fine, s);
    else if (c0.upd_opt == OPT_ADAMW) e = launch_many<EPI_WGRAD_UPD, OPT_ADAMW>(q, t, shape, c0.fine, s);
    else if (c0.upd_opt == OPT_ADAGRAD) e = launch_many<EPI_WGRAD_UPD, OPT_ADAGRAD>(q, t, shape, c0.fine, s);
    else return hipErrorInvalidValue;
    if (e != hipSuccess) return e;
    std::memset(&t, 0, sizeof(t));                 // (the first launch took it along)
  }
  return hipSuccess;
}

hipError_t launch_gemm_bf16(const GemmP &p, int epi, hipStream_t s) {
  if (!operands_ok(p, epi)) return hipErrorInvalidValue;
  if (epi == EPI_WGRAD && gemm_bf16_wgrad_shape(p.Md, p.Nd, p.Kd, p.groups, p.upd_x != nullptr, p.rows_host) == 3)
    return launch_wgrad_many(&p, 1, 3, s);
  if (epi == EPI_WGRAD && p.fine) return launch_wgrad_many(&p, 1, 1, s);
  if (epi != EPI_WGRAD && gemm_bf16_tile_shape(epi, p.Md, p.Nd, p.groups, p.rows_host) == 5) return launch_gemm_small(p, epi, s);
  if (!p.a_trans && !p.b_trans) {
    if (epi == EPI_FWD_ACT) return launch_act<false, false, EPI_FWD_ACT>(p, s);
    if (epi == EPI_LOGITS) return launch_act<false, false, EPI_LOGITS>(p, s);
    if (epi == EPI_IPDOT) return launch_act<false, false, EPI_IPDOT>(p, s);
  } else if (!p.a_trans && p.b_trans) {
    if (epi == EPI_BWD) return launch_act<false, true, EPI_BWD>(p, s);
  } else if (p.a_trans && p.b_trans) {
    if (epi == EPI_WGRAD) return p.upd_x ? launch_act<true, true, EPI_WGRAD_UPD>(p, s) : launch_act<true, true, EPI_WGRAD>(p, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace absk
