// Main loops of the bf16 MFMA GEMMs for gfx950:  acc[M,N] += A . B over k (binary32 accumulate).
//
//   mainloop       both operands K-major (dWq = dY^T X): 256 x 256 macro tile, 2 x 2 wavefronts
//   mainloop_wide  both K-contiguous (Y = X Wq^T, dX = dY Wq): 2 x 2 or 2 x 4 wavefronts (two per SIMD)
//
// Each wavefront owns a (BM/2) x (BN/WAVES_N) block of 32 x 32 accumulator tiles fed by v_mfma_f32_32x32x16_bf16.
//
// Operand path.  Tiles travel HBM/L2 -> LDS with buffer_load_dwordx4 ... lds (no VGPR staging): one wave instruction fills
// 1 KiB of LDS, lane l writing bytes [16 l, 16 l + 16).  What lies past the matrix edge is given an out-of-range buffer
// offset, for which the hardware returns zeros, so the loops have no branches.  LDS holds rings of stages; loads run
// stages ahead of the MFMAs and are waited for with a partial s_waitcnt vmcnt(), so HBM latency is covered by several
// stages of matrix work.
//
// Operand order.  The MFMA is issued as D = Bfrag . Afrag^T, i.e. the accumulator tile holds
// C^T: lane l owns column m = l % 32 of C^T (a row of C) and its 16 registers hold
// n = 8 (e / 4) + 4 (l / 32) + (e % 4).  Four consecutive registers are four consecutive
// n (contiguous in memory for row-major C), which gives 8/16-byte stores and, for the weight
// gradient, makes a lane the owner of one weight row.
#pragma once

#include <type_traits>

#include "l4q_device.h"

namespace l4q {
namespace gemm {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int NUM_XCD = 8;
constexpr int GROUP_M = 4;
// Operands are below 1 GiB.  A row outside the matrix gets OOB_OFFSET; a stage past the end of K adds
// PAST_END_OFFSET.  Either one, or both together, lands beyond num_records without wrapping 32 bits.
constexpr unsigned OOB_OFFSET = 0x80000000u;
constexpr unsigned PAST_END_OFFSET = 0x40000000u;

// gfx9 s_waitcnt immediate for "vmcnt(n)" only
constexpr int waitcnt_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }
constexpr int waitcnt_lgkm0() { return 15 | (3 << 14) | (7 << 4) | (0 << 8); }

// Hardware workgroup id -> tile.  Ids go round-robin over the 8 XCDs; XCD x gets the x-th
// contiguous band of tile ids, and ids walk GROUP_M tile rows at a time.
__device__ __forceinline__ void tile_of_block(int pid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n;
  const int xcd = pid % NUM_XCD;
  const int local = pid / NUM_XCD;
  const int per = (total + NUM_XCD - 1) / NUM_XCD;
  const int tall = total % NUM_XCD;
  int id;
  if (tall == 0 || xcd < tall) id = xcd * per + local;
  else id = tall * per + (xcd - tall) * (per - 1) + local;
  const int in_group = GROUP_M * tiles_n;
  const int group = id / in_group;
  const int first_m = group * GROUP_M;
  const int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
  const int rem = id - group * in_group;
  tm = first_m + rem % gsz;
  tn = rem / gsz;
}

// Tile of the loop for K-major operands: BK k-values a stage, ring of NS stages.  USED < 256: operand A has no more columns
// than that (a rank), and the waves multiply no others; its place in LDS stays 256 wide.
template <int BM_, int BN_, int BK_, int NS_, int USED_ = BM_>
struct Tile {
  static constexpr bool WIDE = false;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, NS = NS_, USED = USED_;
  static constexpr int WAVES_M = USED == BM ? 2 : 1, WAVES_N = 4 / WAVES_M;
  static constexpr int NW = WAVES_M * WAVES_N;
  static constexpr int NT = 64 * NW;
  static constexpr int WTM = USED / WAVES_M, WTN = BN / WAVES_N;  // wave tile
  static constexpr int TM = WTM / 32, TN = WTN / 32;  // 32 x 32 accumulator tiles per wave
  static constexpr int RPI = 2;                       // LDS rows (one k each) filled by one wave-wide load
  static constexpr int A_INSTR = BK / RPI / NW;       // loads per wave per stage, operand A
  static constexpr int B_INSTR = BK / RPI / NW;
  static constexpr int A_BYTES = BK * BM * 2, B_BYTES = BK * BN * 2;
  static constexpr int STAGE = A_BYTES + B_BYTES;
  static constexpr int KK = BK / 16;                  // MFMA k-steps per stage
  static constexpr int D = NS - 1;                    // prefetch distance in stages
  static constexpr int LDS_BYTES = NS * STAGE;
  static_assert(BM == 256 && BN == 256 && BK == 32, "rows of 512 bytes, four loads of either operand per wave and stage");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
  static_assert(NS >= 3, "the last part of a stage's loads is issued after the wait for the next stage");
};

template <class T>
struct Accum {
  f32x16_t v[T::TM][T::TN];
};

// Runs the whole K loop for the tile (m0, n0) and leaves C^T tiles in `acc`.  Operands P[k, ld] with the tile's 256 rows
// along the contiguous axis (dY and X in dWq = dY^T X).
// The MFMA wants, per lane, 8 consecutive k of one row.  A stage is BK LDS rows of 512 B exactly as they lie in
// memory (each wave-wide load brings two full 512 B rows), and the transposition happens on
// the way to the registers with ds_read_b64_tr_b16: within 16 lanes, lane j supplies the address of
// 4 consecutive elements of row k0 + j / 4 at column 4 (j % 4), and receives column j of rows
// k0 .. k0 + 3.  Two such reads fill the 8 k-slots of a lane.  The 16-byte chunk c of LDS row k sits
// at chunk position c ^ 4 (k % 4), which puts the 4 x 32 B a 16-lane group reads, and the two
// groups of a half-wave, on all 64 banks once.
// Ranges.  M, N: columns of the operands.  K: number of k values.  Anything outside reads as zero (num_records ends the
// matrix in k; out-of-range columns get an out-of-bounds offset).
// On return every wave has passed a barrier after its last LDS read, so LDS may be reused.
//
// Tail loads.  The loop keeps issuing loads for the D stages past the end of K so that its wait
// arithmetic stays uniform; by default they carry an out-of-range offset and move nothing.  A caller whose epilogue
// needs a block of memory right after the loop can have those D x (A_INSTR + B_INSTR) loads per wave fetch it
// instead: tail stage q = 0 .. D - 1 lands in ring slot (nk + q) % NS, load c of the A part at byte
// (wave A_INSTR + c) 1024 + 16 lane of the slot, load c of the B part A_BYTES further on, each lane reading 16 bytes
// at byte offset voff_a[c] / voff_b[c] + q * stage_bytes of the buffer (out-of-range offsets read as zero).
struct NoTailLoads {
  static constexpr bool ENABLED = false;
};
template <int NA, int NB>
struct TailLoads {
  static constexpr bool ENABLED = true;
  const void* base;                 // the buffer the tail loads read: base address and size in bytes (< 2 GiB)
  int bytes;
  unsigned voff_a[NA], voff_b[NB];  // per lane
  unsigned stage_bytes;             // added once per tail stage
};

template <class T, class Tail = NoTailLoads>
__device__ __forceinline__ void mainloop(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ B,
                                         int64_t ldb, int M, int N, int K, int m0, int n0, unsigned char* lds,
                                         Accum<T>& acc, const Tail& tail = Tail()) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the declaration
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_ptr_t;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps LDS bases in SGPRs
  const int wm = wave / T::WAVES_N, wn = wave % T::WAVES_N;

  const __amdgpu_buffer_rsrc_t rsrcA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, (int)((int64_t)K * lda * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(B), 0, (int)((int64_t)K * ldb * 2), 0x00020000);

  // per-lane source offsets (bytes) of the loads this wave issues each stage
  unsigned voffA[T::A_INSTR], voffB[T::B_INSTR];
  auto setup_voff = [&](unsigned* voff, int ninstr, int64_t ld, int origin, int extent) {
#pragma unroll
    for (int c = 0; c < ninstr; ++c) {
      const int kr = (wave * ninstr + c) * T::RPI + (lane >> 5);  // LDS row = k within the stage
      const int col = origin + (((lane & 31) ^ (4 * (kr & 3))) << 3);
      voff[c] = col < extent ? (unsigned)(((int64_t)kr * ld + col) * 2) : OOB_OFFSET;
    }
  };
  setup_voff(voffA, T::A_INSTR, lda, m0, M);
  setup_voff(voffB, T::B_INSTR, ldb, n0, N);
  const unsigned stage_bytes_a = (unsigned)(T::BK * lda * 2), stage_bytes_b = (unsigned)(T::BK * ldb * 2);

  // per-lane LDS offsets of the MFMA fragments: one per 32-column block; k-steps and the second half add constants
  unsigned km_off_a[T::TM], km_off_b[T::TN];
  auto setup_km = [&](unsigned* off, int nblk, int wave_col0) {
    const int j = lane & 15, g16 = lane >> 4;
    const int kr = 8 * (lane >> 5) + (j >> 2);
#pragma unroll
    for (int blk = 0; blk < nblk; ++blk) {
      const int chunk = (wave_col0 + blk * 32) / 8 + 2 * (g16 & 1) + ((j & 3) >> 1);
      off[blk] = kr * 512 + ((chunk ^ (4 * (j >> 2))) << 4) + ((j & 1) << 3);
    }
  };
  setup_km(km_off_a, T::TM, wm * T::WTM);
  setup_km(km_off_b, T::TN, wn * T::WTN);

  const int nk = (K + T::BK - 1) / T::BK;

  // part `part` of `nparts` of the loads of stage `stage` < nk into ring slot `slot`
  auto issue_loads = [&](int stage, int slot, int part, int nparts) {
    const unsigned ka = (unsigned)stage * stage_bytes_a, kb = (unsigned)stage * stage_bytes_b;
    unsigned char* base = lds + slot * T::STAGE;
#pragma unroll
    for (int c = 0; c < T::A_INSTR; ++c)
      if (c * nparts / T::A_INSTR == part)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcA, (lds_ptr_t)(base + (wave * T::A_INSTR + c) * 1024), 16,
                                                 voffA[c] + ka, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < T::B_INSTR; ++c)
      if (c * nparts / T::B_INSTR == part)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsrcB, (lds_ptr_t)(base + T::A_BYTES + (wave * T::B_INSTR + c) * 1024), 16, voffB[c] + kb, 0, 0, 0);
  };
  // the same number of loads for tail stage q (stage nk + q): the caller's block, or nothing (out-of-range offsets)
  auto issue_tail = [&](int q, int slot, int part, int nparts) {
    unsigned char* base = lds + slot * T::STAGE;
    __amdgpu_buffer_rsrc_t rt = rsrcA;
    unsigned kq = PAST_END_OFFSET;
    if constexpr (Tail::ENABLED) {
      rt = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(tail.base), 0, tail.bytes, 0x00020000);
      kq = (unsigned)q * tail.stage_bytes;
    }
#pragma unroll
    for (int c = 0; c < T::A_INSTR; ++c)
      if (c * nparts / T::A_INSTR == part) {
        unsigned v = voffA[c];
        if constexpr (Tail::ENABLED) v = tail.voff_a[c];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rt, (lds_ptr_t)(base + (wave * T::A_INSTR + c) * 1024), 16, v + kq,
                                                 0, 0, 0);
      }
#pragma unroll
    for (int c = 0; c < T::B_INSTR; ++c)
      if (c * nparts / T::B_INSTR == part) {
        unsigned v = voffB[c];
        if constexpr (Tail::ENABLED) v = tail.voff_b[c];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rt, (lds_ptr_t)(base + T::A_BYTES + (wave * T::B_INSTR + c) * 1024),
                                                 16, v + kq, 0, 0, 0);
      }
  };

  bf16x8_t fa[2][T::TM], fb[2][T::TN];
  auto read_km = [&](const unsigned char* region, unsigned off, int kk) -> bf16x8_t {
    const unsigned char* p0 = region + off + kk * (16 * 512);
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr_t)p0);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr_t)(p0 + 4 * 512));
    typedef short s16x8_t __attribute__((ext_vector_type(8)));
    const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8_t, v);
  };
  auto read_frags_a = [&](int slot, int kk, int set) {
    const unsigned char* region = lds + slot * T::STAGE;
#pragma unroll
    for (int a = 0; a < T::TM; ++a) fa[set][a] = read_km(region, km_off_a[a], kk);
  };
  auto read_frags_b = [&](int slot, int kk, int set) {
    const unsigned char* region = lds + slot * T::STAGE + T::A_BYTES;
#pragma unroll
    for (int b = 0; b < T::TN; ++b) fb[set][b] = read_km(region, km_off_b[b], kk);
  };
  auto mfma_block = [&](int set) {
#pragma unroll
    for (int a = 0; a < T::TM; ++a)
#pragma unroll
      for (int b = 0; b < T::TN; ++b)
        acc.v[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][b], fa[set][a], acc.v[a][b], 0, 0, 0);
  };

  constexpr int LOADS = T::A_INSTR + T::B_INSTR;
  static_assert(T::A_INSTR % T::KK == 0 && T::B_INSTR % T::KK == 0, "loads are spread evenly over the k-steps");
  constexpr int LPK = LOADS / T::KK;                 // loads issued per k-step
  constexpr int NDA = 2 * T::TM, NDB = 2 * T::TN;     // LDS read instructions per k-step
  constexpr int NMF = T::TM * T::TN;
  // with few matrix ops there is nothing to hide the other two kinds behind: the order is the compiler's
  constexpr bool DEALT = NMF == 16;
  constexpr int EXTRA = NDA + NDB + LPK > NMF ? NDA + NDB + LPK - NMF : 0;  // reads that share a matrix op
  static_assert(!DEALT || 2 * EXTRA <= NDA + NDB, "too many LDS reads per matrix op");
#pragma unroll
  for (int s = 0; s < T::D; ++s) {
    if (s < nk) issue_loads(s, s, 0, 1);
    else issue_tail(s - nk, s, 0, 1);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __builtin_amdgcn_s_barrier();
  read_frags_a(0, 0, 0);
  read_frags_b(0, 0, 0);

  // Steady state.  Per k-step: the LDS reads of the next k-step, 1/KK of the global loads for stage
  // s + D (stages past the end get an out-of-range offset: no memory traffic, and the vmcnt arithmetic
  // stays uniform), and TM x TN matrix ops, interleaved so that the other two kinds issue in the
  // shadow of the matrix pipeline and the global loads of the four waves do not arrive in one burst.
  // The LDS reads come first and the matrix ops left over come last, so that the wait for the reads
  // at the next stage boundary finds them complete.  Program order is reads, then DMA loads: the DMA
  // loads write LDS and the compiler keeps them behind the reads before them.
  constexpr int REST = NMF - (NDA + NDB - EXTRA + LPK);
  static_assert(!DEALT || REST >= 0, "more LDS reads and loads than matrix ops to hide them behind");
  int slot = 0;
  // one stage; `load_part(kk)` issues part kk of the loads of stage s + D into the slot stage s - 1 has left
  auto stage = [&](auto&& load_part) {
    int pslot = slot + T::D;
    if (pslot >= T::NS) pslot -= T::NS;
    int nslot = slot + 1;
    if (nslot == T::NS) nslot = 0;
#pragma unroll
    for (int kk = 0; kk < T::KK; ++kk) {
      const bool last = kk + 1 == T::KK;
      if (last) {
        // Stage s + 1 must have landed for every wave: all but the loads of stages s + 2 .. s + D issued
        // so far, i.e. (D - 2) whole stages plus this stage's first KK - 1 parts, may still be in flight.
        // All of this wave's LDS reads have returned, so the slot refilled next is free once every wave is here.
        __builtin_amdgcn_sched_barrier(0);  // the matrix ops of the previous k-step are issued before the wait
        __builtin_amdgcn_s_waitcnt(waitcnt_vm((T::D - 2) * LOADS + (T::KK - 1) * LPK));
        __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());
        __builtin_amdgcn_s_barrier();
      }
      // after the last stage the reads below fetch stale LDS; the values are never used
      read_frags_a(last ? nslot : slot, last ? 0 : kk + 1, (kk + 1) & 1);
      read_frags_b(last ? nslot : slot, last ? 0 : kk + 1, (kk + 1) & 1);
      load_part(pslot, kk);
      mfma_block(kk & 1);
      if constexpr (DEALT) {
#pragma unroll
        for (int q = 0; q < EXTRA; ++q) {  // where reads outnumber matrix ops, two reads per matrix op
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
#pragma unroll
        for (int q = 0; q < NDA + NDB - 2 * EXTRA; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int q = 0; q < LPK; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        }
        if constexpr (REST > 0) __builtin_amdgcn_sched_group_barrier(0x008, REST, 0);
      }
    }
    slot = nslot;
  };
  // The stages whose look-ahead stage still lies inside K, then the last D whose loads are the tail loads: two
  // copies of the same straight-line body, no selection inside it.
  const int n_inside = nk > T::D ? nk - T::D : 0;
  int s = 0;
  for (; s < n_inside; ++s) stage([&](int pslot, int kk) { issue_loads(s + T::D, pslot, kk, T::KK); });
  for (; s < nk; ++s) stage([&](int pslot, int kk) { issue_tail(s + T::D - nk, pslot, kk, T::KK); });
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());
  __builtin_amdgcn_s_barrier();
#endif
}

// Tile of the wide-row loop (mainloop_wide): operand A in units of 64 k-values, ring of NA of them; operand B in stages of
// 32, ring of NB.
template <int BM_, int BN_, int NA_, int NB_, int WAVES_N_>
struct WideTile {
  static constexpr bool WIDE = true;
  static constexpr int BM = BM_, BN = BN_, NA = NA_, NB = NB_, BK = 32;
  static constexpr int WAVES_M = 2, WAVES_N = WAVES_N_;
  static constexpr int NW = WAVES_M * WAVES_N, NT = 64 * NW;
  static constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  static constexpr int TM = WTM / 32, TN = WTN / 32;
  static constexpr int A_UNIT = BM * 128, B_STAGE = BN * 64;  // bytes
  static constexpr int A_INSTR = BM / 8 / NW / 2;             // loads per wave and stage: half a unit of A,
  static constexpr int B_INSTR = BN / 16 / NW;                // a stage of B
  static constexpr int DA = NA - 1, DB = NB - 1;              // units / stages ahead
  static constexpr int LDS_BYTES = NA * A_UNIT + NB * B_STAGE;
  static_assert(WTM % 32 == 0 && WTN % 32 == 0 && BM % (16 * NW) == 0 && BN % (16 * NW) == 0, "tile");
  static_assert(DB >= 2 && DB <= 2 * DA - 1, "the wait for a stage of B covers the unit of A that was requested before it");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// The loop for a K-contiguous operand A that lies in memory as the caller's rows do.  A wave-wide load fetches 8 rows of 128
// bytes, whole cache lines, instead of 16 rows of 64: a load of half lines takes the compute unit's cache three times as
// long (measured, all units reading one 512 KB array out of the L2s: 16 rows x 64 bytes a load, 15.4 us; 8 x 128, 5.8; 2 x
// 512, 5.8), also where the load of the other halves follows at once.  So A goes to LDS in units of 64 k-values (rows of
// 128 bytes, chunk c of row r at position c ^ (r / 2) % 8), two stages of B each; during a stage half a unit of A and a
// stage of B are requested, DA units and DB stages ahead, and the waits count them together (loads return in order).
// B row-major (ldb), or, B_BLK, in blocks of 32 k-values: B[k / 32][row][k % 32] with all N rows of a k-block contiguous, so
// that a stage of the tile is one run of BN x 64 bytes and the merge + quantize pass, which writes Wq and Wq^T this way,
// stores whole 1 KiB / 4 KiB runs; B is zero for K_a <= k < K.  In LDS chunk c of a 64-byte row r is at c ^ (r / 4) % 4.
// Both row pitches put the DMA writes (consecutive lanes = consecutive positions of a row) and the fragment reads
// (consecutive lanes = consecutive rows, same logical chunk) on all 64 banks once per 16 lanes.  K_a: end of A's rows, a multiple of 8, in the last 32 k-values;
// MASK_A_K: K_a is no multiple of 64, and the chunks of the last unit past it read as zero (what follows a row in memory is
// the next row: a NaN or Inf there must not reach this one through 0 x Inf, and after the last row there may be nothing).
// On return every wave has passed a barrier after its last LDS read, so LDS may be reused.
template <class T, bool MASK_A_K, bool B_BLK>
__device__ __forceinline__ void mainloop_wide(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ B,
                                              int64_t ldb, int M, int N, int K, int m0, int n0, unsigned char* lds,
                                              Accum<T>& acc, int K_a) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / T::WAVES_N, wn = wave % T::WAVES_N;
  const __amdgpu_buffer_rsrc_t rsrcA =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, (int)((int64_t)M * lda * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcB = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(B), 0, (int)((int64_t)N * (B_BLK ? (int64_t)K : ldb) * 2), 0x00020000);
  const int nk = (K + 31) / 32, nu = (nk + 1) / 2;

  // load c of half h of a unit: rows ((h A_INSTR + c) NW + wave) 8 + lane / 8
  unsigned voffA[2][T::A_INSTR], voffA_last[2][MASK_A_K ? T::A_INSTR : 1], voffB[T::B_INSTR];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < T::A_INSTR; ++c) {
      const int row = ((h * T::A_INSTR + c) * T::NW + wave) * 8 + (lane >> 3);
      const int ch = (lane & 7) ^ ((row >> 1) & 7);
      voffA[h][c] = m0 + row < M ? (unsigned)(((int64_t)(m0 + row) * lda + ch * 8) * 2) : OOB_OFFSET;
      if constexpr (MASK_A_K) voffA_last[h][c] = (nu - 1) * 64 + ch * 8 < K_a ? voffA[h][c] : OOB_OFFSET;
    }
#pragma unroll
  for (int c = 0; c < T::B_INSTR; ++c) {
    const int row = (wave * T::B_INSTR + c) * 16 + (lane >> 2);
    const int ch = (lane & 3) ^ ((row >> 2) & 3);
    voffB[c] = n0 + row < N ? (unsigned)(((int64_t)(n0 + row) * (B_BLK ? 32 : ldb) + ch * 8) * 2) : OOB_OFFSET;
  }
  const unsigned stage_bytes_b = B_BLK ? (unsigned)N * 64u : 64u;
  unsigned char* const ldsB = lds + T::NA * T::A_UNIT;

  auto load_a = [&](int unit, int slot, int h, int c) {
    unsigned v = voffA[h][c];
    if constexpr (MASK_A_K) v = unit == nu - 1 ? voffA_last[h][c] : v;
    const unsigned k = unit < nu ? (unsigned)unit * 128u : PAST_END_OFFSET;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rsrcA, (lds_ptr_t)(lds + slot * T::A_UNIT + ((h * T::A_INSTR + c) * T::NW + wave) * 1024), 16, v + k, 0, 0, 0);
  };
  auto load_b = [&](int stage, int slot, int c) {
    const unsigned k = stage < nk ? (unsigned)stage * stage_bytes_b : PAST_END_OFFSET;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcB, (lds_ptr_t)(ldsB + slot * T::B_STAGE + (wave * T::B_INSTR + c) * 1024), 16,
                                             voffB[c] + k, 0, 0, 0);
  };

  // fragments: k-step q of a unit (0 .. 3) of A, of a stage (0, 1) of B; row lane % 32, 8 k-values by lane / 32
  const int r = lane & 31, lh = lane >> 5;
  unsigned offA[4], offB[2];
#pragma unroll
  for (int q = 0; q < 4; ++q) offA[q] = r * 128 + (((q * 2 + lh) ^ ((r >> 1) & 7)) << 4);
#pragma unroll
  for (int q = 0; q < 2; ++q) offB[q] = r * 64 + (((q * 2 + lh) ^ ((r >> 2) & 3)) << 4);
  bf16x8_t fa[2][T::TM], fb[2][T::TN];
  auto read_a = [&](int slot, int q, int set) {
    const unsigned char* p = lds + slot * T::A_UNIT + wm * T::WTM * 128 + offA[q];
#pragma unroll
    for (int a = 0; a < T::TM; ++a) fa[set][a] = *reinterpret_cast<const bf16x8_t*>(p + a * 32 * 128);
  };
  auto read_b = [&](int slot, int q, int set) {
    const unsigned char* p = ldsB + slot * T::B_STAGE + wn * T::WTN * 64 + offB[q];
#pragma unroll
    for (int b = 0; b < T::TN; ++b) fb[set][b] = *reinterpret_cast<const bf16x8_t*>(p + b * 32 * 64);
  };
  auto mfma_block = [&](int set) {
#pragma unroll
    for (int a = 0; a < T::TM; ++a)
#pragma unroll
      for (int b = 0; b < T::TN; ++b)
        acc.v[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][b], fa[set][a], acc.v[a][b], 0, 0, 0);
  };

  constexpr int LOADS = T::A_INSTR + T::B_INSTR;
  static_assert(T::A_INSTR % 2 == 0 && T::B_INSTR % 2 == 0, "loads are spread evenly over the two k-steps of a stage");
  constexpr int LPK = LOADS / 2, NR = T::TM + T::TN, NMF = T::TM * T::TN;
  constexpr int EXTRA = NR + LPK > NMF ? NR + LPK - NMF : 0;  // reads that share a matrix op
  static_assert(2 * EXTRA <= NR, "too many LDS reads per matrix op");
  constexpr int REST = NMF - (NR - EXTRA + LPK);
  static_assert(REST >= 0, "more LDS reads and loads than matrix ops to hide them behind");

  // in the order of the steady state: during stage s, half s % 2 of unit s / 2 + DA and stage s + DB
#pragma unroll
  for (int s = -2 * T::DA; s < 0; ++s) {
#pragma unroll
    for (int c = 0; c < T::A_INSTR; ++c) load_a((s >> 1) + T::DA, (s >> 1) + T::DA, s & 1, c);
    if (s + T::DB >= 0) {
#pragma unroll
      for (int c = 0; c < T::B_INSTR; ++c) load_b(s + T::DB, s + T::DB, c);
    }
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm((T::DB - 1) * LOADS));  // unit 0 and stage 0 have landed
  __builtin_amdgcn_s_barrier();
  read_a(0, 0, 0);
  read_b(0, 0, 0);
  int sa = 0, sb = 0;  // slots of the current unit and stage
  auto stage = [&](auto half, int s) {
    constexpr int H = decltype(half)::value;
    const int pa = sa == 0 ? T::NA - 1 : sa - 1, pb = sb == 0 ? T::NB - 1 : sb - 1;  // the slots left last
    const int na = sa + 1 == T::NA ? 0 : sa + 1, nb = sb + 1 == T::NB ? 0 : sb + 1;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (kk == 1) {
        // Stage s + 1 of B (and the unit of A it starts) must have landed for every wave: all but the loads of the DB - 2
        // stages before this one and the first half of this one's may be in flight.  All of this wave's reads have returned:
        // the slots of this stage (and unit) are free once every wave is here.
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm((T::DB - 2) * LOADS + LPK));
        __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());
        __builtin_amdgcn_s_barrier();
      }
      // (after the last stage the reads fetch what is not used)
      if (kk == 0) { read_a(sa, 2 * H + 1, 1); read_b(sb, 1, 1); }
      else { read_a(H == 0 ? sa : na, H == 0 ? 2 : 0, 0); read_b(nb, 0, 0); }
#pragma unroll
      for (int c = kk * T::A_INSTR / 2; c < (kk + 1) * T::A_INSTR / 2; ++c) load_a((s >> 1) + T::DA, pa, H, c);
#pragma unroll
      for (int c = kk * T::B_INSTR / 2; c < (kk + 1) * T::B_INSTR / 2; ++c) load_b(s + T::DB, pb, c);
      mfma_block(kk);
#pragma unroll
      for (int q = 0; q < EXTRA; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
#pragma unroll
      for (int q = 0; q < NR - 2 * EXTRA; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
#pragma unroll
      for (int q = 0; q < LPK; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      if constexpr (REST > 0) __builtin_amdgcn_sched_group_barrier(0x008, REST, 0);
    }
    if (H == 1) sa = na;
    sb = nb;
  };
  int s = 0;
  for (; s + 1 < nk; s += 2) {
    stage(std::integral_constant<int, 0>(), s);
    stage(std::integral_constant<int, 1>(), s + 1);
  }
  if (s < nk) stage(std::integral_constant<int, 0>(), s);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());
  __builtin_amdgcn_s_barrier();
#endif
}

// Row m and first column n of the 4 consecutive outputs held in registers 4 eg .. 4 eg + 3 of
// accumulator tile (a, b), relative to the macro tile origin.
template <class T>
__device__ __forceinline__ void acc_coords(int a, int b, int eg, int& m, int& n) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  m = (wave / T::WAVES_N) * T::WTM + a * 32 + (lane & 31);
  n = (wave % T::WAVES_N) * T::WTN + b * 32 + 8 * eg + 4 * (lane >> 5);
}

}  // namespace gemm
}  // namespace l4q
