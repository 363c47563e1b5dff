// bf16 MFMA tile engine for gfx950: C[M,N] += A[M,K] * B[N,K]^T with both operands K-contiguous.
//
// A workgroup owns a BM x BN tile of C and walks K in steps of 64; each wavefront owns a
// (BM/WM) x (BN/WN) sub-tile as a grid of 16x16 blocks of v_mfma_f32_16x16x32_bf16 with float
// accumulators (on random operands a register-only loop of this instruction sustains 2.0 PFLOP/s on this
// part, one of the 32x32x16 form 1.77: the chip runs into its power limit later).  The main loops fill the
// LDS straight from global memory.
//
// Operand layout of one block (lane l): row (or column) l % 16, k = 8 (l / 16) .. 8 (l / 16) + 7.
// Accumulator layout of one 16x16 block (register r of lane l):
//   row (A side, "M")  = 4*(l/16) + r
//   col (B side, "N")  = l%16
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace umas {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

template <int BM_, int BN_, int WM_, int WN_>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int BK = 64;
  static constexpr int T = 64 * WM * WN;               // threads per workgroup
  static constexpr int WTM = BM / WM, WTN = BN / WN;   // wavefront sub-tile
  static constexpr int MI = WTM / 16, NI = WTN / 16;   // 16x16 blocks per wavefront
  static_assert(BM % (32 * WM) == 0 && BN % (16 * WN) == 0, "sub-tiles are grids of 16x16 blocks, an even number along M");
};

// The thread's number as a value that the compiler takes for a new one every time: what a tile derives from it (addresses of
// loads and fragments, dozens of registers for each kind of tile) is then not kept over a loop of tiles.
__device__ __forceinline__ int tile_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xFFFFFFFF, 0x00020000);
}

// ---------------------------------------------------------------------------------------------
// Main loop for K-contiguous operands, K a multiple of 8.
//
// K is walked in steps of 64: 128 bytes per row, the line size of the vector caches, so every line is
// fetched once.  Tiles go from global memory straight into LDS stages of 256 rows x 128 bytes per operand
// (buffer_load_dwordx4 ... lds: no staging registers, no ds_write); one wavefront-wide load fills 8
// consecutive rows (1 KB).  Operands are addressed as raw buffers: a wave-uniform base (the caller picks it
// so that every byte offset of the tile fits 32 bits) plus one 32-bit byte offset per load slot.  The 16-byte chunk c of row r sits in slot
// c ^ ((r >> 1) & 7), which keeps the fragment reads of 16 consecutive rows on distinct banks.
// Operand A has three stages and is loaded two steps ahead, operand B two stages, one step ahead (the callers
// put the operand that comes from farther away in A).  Per step j: the loads of B for step j+1 and of A for step
// j+2 go out right away (everybody left those stages before the barrier of the previous step); phases 0..2 run;
// then the wavefront waits for its LDS reads and for all loads but the youngest ones (A of step j+2: loads into
// LDS return in the order they were issued), the workgroup meets at the barrier, and phase 3 runs while the first
// fragments of the next step are read.
// A_POLICY is the cache policy of operand A's loads: kCached, or kStream for an operand that is read once.
// With TAIL the last step holds fewer than 64 k: the chunks of a row past its end repeat the row's last chunk, and the threads that
// loaded them clear them in LDS, in both operands (a product with a value that is not finite would not be 0 otherwise), in front
// of the barrier behind which the step is read.  (A loop with registers and a second LDS pitch in place of this one: 2500 rows of
// 1544 against 50 001 532 us, now 391; 700 rows of 3000 against 80 001 466 us, now 340; 5000 rows kept 3.95 ms, now 2.66.)
constexpr int kCached = 0, kStream = 2;
template <class C>
struct Ring2Cfg {
  static constexpr int BK = 64;
  static constexpr int ROWB = 128;
  static constexpr int ASTAGE = C::BM * ROWB, BSTAGE = C::BN * ROWB;   // bytes of one stage of an operand
  static constexpr int BBASE = 3 * ASTAGE;                             // three stages of A, then two of B
  static constexpr int LDS_BYTES = BBASE + 2 * BSTAGE;
  static constexpr int NA = C::BM * 8 / C::T, NB = C::BN * 8 / C::T;   // 16-byte loads per thread per step
  static constexpr int ROWS_PER_PASS = C::T / 8;
  static_assert(C::T % 64 == 0 && (C::BM * 8) % C::T == 0 && (C::BN * 8) % C::T == 0, "load slots divide evenly");
};
template <class C>
__device__ __forceinline__ int ring2_row(int i, int t = threadIdx.x) { return i * (C::T / 8) + (t >> 3); }
// K offset (elements) of the chunk this lane fetches: slot (tid & 7) of row ring2_row holds chunk slot ^ ((row >> 1) & 7);
// rows per pass and wavefront row offsets are multiples of 8, so (row >> 1) & 7 = ((tid >> 3) >> 1) & 7 with tid >> 3 < 64
__device__ __forceinline__ int ring2_kofs(int t = threadIdx.x) {
  return 8 * ((t & 7) ^ (((t >> 3) >> 1) & 7));
}

template <class C, bool TAIL, int A_POLICY>
__device__ __forceinline__ void mfma_mainloop_ring2(__amdgpu_buffer_rsrc_t ra, const uint32_t (&oa)[Ring2Cfg<C>::NA],
                                                    __amdgpu_buffer_rsrc_t rb, const uint32_t (&ob)[Ring2Cfg<C>::NB],
                                                    int K, uint16_t* lds, floatx4 (&acc)[C::MI][C::NI]) {
  using R = Ring2Cfg<C>;
  constexpr int HA = C::MI / 2;                      // A blocks of one half of the wavefront's sub-tile
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  char* base = reinterpret_cast<char*>(lds);
  const int nsub = (K + R::BK - 1) / R::BK;
  // the last step's chunk of this thread when it lies past the end of the row: how far in front of it the row's last one is
  const int k_last = (nsub - 1) * R::BK + ring2_kofs();
  const bool past = TAIL && k_last >= K;
  const uint32_t back = past ? static_cast<uint32_t>(k_last - (K - 8)) * 2u : 0u;

  static_assert(R::NA < 16, "the wait before the barrier leaves the loads of A outstanding");
  auto gload_a = [&](int sub, int ia) {
    const int kbytes = sub * R::BK * 2;
    char* sa = base + ia * R::ASTAGE + wave * 8 * R::ROWB;
    const uint32_t cut = TAIL && sub == nsub - 1 ? back : 0u;
#pragma unroll
    for (int i = 0; i < R::NA; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, reinterpret_cast<uint32_t*>(sa + i * R::ROWS_PER_PASS * R::ROWB), 16,
                                               TAIL ? oa[i] - cut : oa[i], kbytes, 0, A_POLICY);
  };
  auto gload_b = [&](int sub, int ib) {
    const int kbytes = sub * R::BK * 2;
    char* sb = base + R::BBASE + ib * R::BSTAGE + wave * 8 * R::ROWB;
    const uint32_t cut = TAIL && sub == nsub - 1 ? back : 0u;
#pragma unroll
    for (int i = 0; i < R::NB; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, reinterpret_cast<uint32_t*>(sb + i * R::ROWS_PER_PASS * R::ROWB), 16,
                                               TAIL ? ob[i] - cut : ob[i], kbytes, 0, 0);
  };
  auto clear_past = [&](int ia, int ib) {            // the last step's stages, once this thread's loads of it have landed
    if (past) {
      char* sa = base + ia * R::ASTAGE + wave * 8 * R::ROWB + lane * 16;
      char* sb = base + R::BBASE + ib * R::BSTAGE + wave * 8 * R::ROWB + lane * 16;
#pragma unroll
      for (int i = 0; i < R::NA; ++i) *reinterpret_cast<uint4*>(sa + i * R::ROWS_PER_PASS * R::ROWB) = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int i = 0; i < R::NB; ++i) *reinterpret_cast<uint4*>(sb + i * R::ROWS_PER_PASS * R::ROWB) = make_uint4(0u, 0u, 0u, 0u);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0)
  };
  // Operand of a 16x16x32 block: lane l holds row l % 16, k = 8 (l / 16) .. + 7 of the 32-wide slice, i.e. chunk
  // 4 s + l / 16 of the row.  A step is four phases of 16 MFMAs: (slice 0, upper half of the A rows), (slice 0,
  // lower half), (slice 1, upper), (slice 1, lower); the B fragments of a slice serve both of its phases.
  const int sw = (lane >> 1) & 7;                    // (row >> 1) & 7 of this lane's fragment rows
  const int arow = (wm * C::WTM + (lane & 15)) * R::ROWB;
  const int brow = R::BBASE + (wn * C::WTN + (lane & 15)) * R::ROWB;
  bf16x8 af[2][HA], bfr[2][C::NI];
  auto fload_a = [&](int buf, int ia, int s, int h) {
    const int coff = ((4 * s + (lane >> 4)) ^ sw) * 16;
    const char* sa = base + ia * R::ASTAGE + arow + coff + h * HA * 16 * R::ROWB;
#pragma unroll
    for (int i = 0; i < HA; ++i) af[buf][i] = *reinterpret_cast<const bf16x8*>(sa + i * 16 * R::ROWB);
  };
  auto fload_b = [&](int buf, int ib, int s) {
    const int coff = ((4 * s + (lane >> 4)) ^ sw) * 16;
    const char* sb = base + ib * R::BSTAGE + brow + coff;
#pragma unroll
    for (int j = 0; j < C::NI; ++j) bfr[buf][j] = *reinterpret_cast<const bf16x8*>(sb + j * 16 * R::ROWB);
  };
  auto mfmas = [&](int abuf, int bbuf, int h) {
#pragma unroll
    for (int i = 0; i < HA; ++i)
#pragma unroll
      for (int jj = 0; jj < C::NI; ++jj) {
        const int j = i & 1 ? C::NI - 1 - jj : jj;
        acc[h * HA + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[abuf][i], bfr[bbuf][j], acc[h * HA + i][j], 0, 0, 0);
      }
  };
  auto interleave = [&](int n_ds, int n_vm) {
#pragma unroll
    for (int i = 0; i < HA * C::NI; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i < n_ds) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (i < n_vm) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
  };

  auto clamp_sub = [&](int sub) { return sub < nsub ? sub : nsub - 1; };   // past the end of K the loads repeat the last step (nobody reads them)
  gload_a(0, 0);
  gload_b(0, 0);
  gload_a(clamp_sub(1), 1);
  __builtin_amdgcn_s_waitcnt(0x0070);
  if (TAIL && nsub == 1) clear_past(0, 0);
  __builtin_amdgcn_s_barrier();
  fload_b(0, 0, 0);
  fload_a(0, 0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  int ia = 0;                                        // A stage of the current step
  for (int j = 0; j < nsub; ++j) {
    const int ib = j & 1;
    const int ia1 = ia == 2 ? 0 : ia + 1, ia2 = ia1 == 2 ? 0 : ia1 + 1;
    gload_b(clamp_sub(j + 1), ib ^ 1);
    gload_a(clamp_sub(j + 2), ia2);
    fload_a(1, ia, 0, 1);
    mfmas(0, 0, 0);
    interleave(HA, R::NA + R::NB);
    __builtin_amdgcn_sched_barrier(0);
    fload_b(1, ib, 1);
    fload_a(0, ia, 1, 0);
    mfmas(1, 0, 1);
    interleave(HA + C::NI, 0);
    __builtin_amdgcn_sched_barrier(0);
    fload_a(1, ia, 1, 1);
    mfmas(0, 1, 0);
    interleave(HA, 0);
    __builtin_amdgcn_sched_barrier(0);
    // own reads of this step done, own loads for the next step landed (the youngest, A of the step after
    // next, may still be on their way); then everybody's
    __builtin_amdgcn_s_waitcnt(0x0070 | R::NA);      // vmcnt(NA) and lgkmcnt(0), expcnt untouched (gfx9 encoding)
    if (TAIL && j == nsub - 2) clear_past(ia1, ib ^ 1);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    fload_b(0, ib ^ 1, 0);
    fload_a(0, ia1, 0, 0);
    mfmas(1, 1, 1);
    interleave(HA + C::NI, 0);
    __builtin_amdgcn_sched_barrier(0);
    ia = ia1;
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_s_barrier();
}

// ---------------------------------------------------------------------------------------------
// The same loop for operands that are not K-contiguous in memory.
//
// An operand stored K-major (row k holds the 256 tile entries of that k next to each other, 512 bytes) is
// brought into LDS as it lies: a stage holds 64 k-rows of 512 bytes, one wavefront-wide load fills two of
// them.  Fragments come out through ds_read_b64_tr_b16, which transposes on the way: in a group of 16
// lanes, lane l receives element l % 4 of the 8-byte chunks addressed by lanes l / 4, l / 4 + 4, l / 4 + 8
// and l / 4 + 12.  Lane i = q + 4 j of a group therefore points at k-row kbase + j, entries 4 q .. 4 q + 3
// of the block's 16, and lane l ends up with entry l of the 16 for the four k of the read; two reads give
// the eight k of a 16x16x32 operand, group g of the wavefront taking k-rows 8 g .. 8 g + 7 of the slice.
// The 16-byte unit u of k-row k sits in slot u ^ (4 (k & 3)) ^ (2 ((k >> 3) & 1)), which keeps the 32 lanes
// served in one cycle (two groups, four k-rows each) on distinct banks.
typedef short short4v __attribute__((ext_vector_type(4)));

template <class C>
struct MixedLdsBytes {          // LDS of mfma_mainloop_mixed: three A stages and two B stages of 32 KB, like the ring's
  static constexpr int value = Ring2Cfg<C>::LDS_BYTES;
};
struct KMajor {                 // an operand tile stored K-major
  const char* base;             // byte address of (k-row 0, first entry of the tile)
  int64_t ld_bytes;             // bytes between consecutive k-rows
  int64_t hi_bytes;             // added once more per 256 k-rows (an operand stored in blocks of 256 rows), else 0
  int k_rows;                   // k-rows that exist; later ones read the last one (the other operand is zero there)
  int n_units;                  // 16-byte units of a k-row that exist from base on (<= 32); later ones read the last one
};
struct KContig {                // an operand tile stored K-contiguous: per-slot byte offsets from a base
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t off[4];
  uint32_t hi_bytes;            // added once more per 256 k (an operand stored in blocks of 256 columns), else 0
};

// B_STREAM: operand B is read once, past the caches.  CUT: only m_rows rows of the tile are looked at; a wavefront whose sub-tile has none of
// them loads for the others and multiplies nothing.
template <class C, bool ATR, bool BTR, int AHEAD, bool B_STREAM = false, bool CUT = false>
__device__ __forceinline__ void mfma_mainloop_mixed(const KContig& ca, const KMajor& ka, const KContig& cb, const KMajor& kb,
                                                    int K, uint16_t* lds, floatx4 (&acc)[C::MI][C::NI], int m_rows = C::BM) {
  using R = Ring2Cfg<C>;
  static_assert(C::BM == 256 && C::BN == 256 && C::T == 512 && R::NA == 4 && R::NB == 4, "written for 256x256 tiles, 8 wavefronts");
  constexpr int HA = C::MI / 2;                      // A blocks of one half of the wavefront's sub-tile
  const int tid = tile_thread();
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  char* base = reinterpret_cast<char*>(lds);
  const int nsub = K / R::BK;
  // LDS: five stages of 32 KB.  One operand (AHEAD = 1: A, AHEAD = 2: B) has three of them and is loaded two steps
  // ahead, the other two, one step ahead; the callers give the third stage to the operand that comes from farther
  // away.
  static_assert(AHEAD == 1 || AHEAD == 2, "which operand is loaded two steps ahead");
  constexpr int kAStage = C::BM * R::ROWB, kBStage = C::BN * R::ROWB;
  constexpr int kABase = AHEAD == 2 ? 3 * kBStage : 0, kBBase = AHEAD == 2 ? 0 : 3 * kAStage;
  static_assert(3 * kAStage + 2 * kBStage <= MixedLdsBytes<C>::value && kAStage == kBStage, "LDS of the mixed loop");

  // K-major loads: pass p covers k-rows 16 p .. 16 p + 15, this wavefront rows 16 p + 2 wave, + 1; lane l fills slot
  // l & 31 of row k = 16 p + 2 wave + (l >> 5) and fetches unit slot ^ 4 (k & 3) ^ 2 ((k >> 3) & 1)
  const int tr_krow = 2 * wave + (lane >> 5);        // + 16 p
  const int tr_slot_unit = (lane & 31) ^ (4 * (tr_krow & 3)) ^ (2 * ((tr_krow >> 3) & 1));
  auto kmajor_units = [&](const KMajor& k) { return static_cast<uint32_t>(min(tr_slot_unit, k.n_units - 1)) * 16u; };
  auto kmajor_step = [&](const KMajor& k, int sub) { return min(sub * R::BK, ((k.k_rows - 1) / R::BK) * R::BK); };   // first k-row of the (clamped) step
  auto kmajor_rsrc = [&](const KMajor& k, int k0) { return make_rsrc(k.base + static_cast<int64_t>(k0) * k.ld_bytes + (k0 >> 8) * k.hi_bytes); };
  auto kmajor_offset = [&](const KMajor& k, int k0, int p) {
    return static_cast<uint32_t>(min(16 * p + tr_krow, k.k_rows - 1 - k0)) * static_cast<uint32_t>(k.ld_bytes);
  };
  auto gload_kmajor = [&](const KMajor& k, int sub, char* region) {
    const uint32_t ubytes = kmajor_units(k);
    const int k0 = kmajor_step(k, sub);
    const __amdgpu_buffer_rsrc_t r = kmajor_rsrc(k, k0);
#pragma unroll
    for (int p = 0; p < 4; ++p)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, reinterpret_cast<uint32_t*>(region + (16 * p + 2 * wave) * 512), 16,
                                               kmajor_offset(k, k0, p) + ubytes, 0, 0, kCached);
  };
  auto gload_kmajor_stream = [&](const KMajor& k, int sub, char* region) {     // the policy is part of the instruction
    const uint32_t ubytes = kmajor_units(k);
    const int k0 = kmajor_step(k, sub);
    const __amdgpu_buffer_rsrc_t r = kmajor_rsrc(k, k0);
#pragma unroll
    for (int p = 0; p < 4; ++p)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, reinterpret_cast<uint32_t*>(region + (16 * p + 2 * wave) * 512), 16,
                                               kmajor_offset(k, k0, p) + ubytes, 0, 0, kStream);
  };
  auto gload_kcontig = [&](const KContig& c, int sub, char* region) {
    const int kbytes = sub * R::BK * 2 + (sub >> 2) * static_cast<int>(c.hi_bytes);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(c.rsrc, reinterpret_cast<uint32_t*>(region + (i * R::ROWS_PER_PASS + wave * 8) * R::ROWB), 16,
                                               c.off[i], kbytes, 0, 0);
  };
  auto gload_a = [&](int sub, int ia) {
    char* sa = base + kABase + ia * kAStage;
    if (ATR) gload_kmajor(ka, sub, sa); else gload_kcontig(ca, sub, sa);
  };
  auto gload_b = [&](int sub, int ib) {
    char* sb = base + kBBase + ib * kBStage;
    if (BTR && B_STREAM) gload_kmajor_stream(kb, sub, sb); else if (BTR) gload_kmajor(kb, sub, sb); else gload_kcontig(cb, sub, sb);
  };

  // fragment addresses (K-contiguous operands as in mfma_mainloop_ring2)
  const int sw = (lane >> 1) & 7;
  const int arow = (wm * C::WTM + (lane & 15)) * R::ROWB;
  const int brow = (wn * C::WTN + (lane & 15)) * R::ROWB;
  const int tq = lane & 3, tj = (lane >> 2) & 3;     // position q + 4 j inside the group of 16 lanes
  const int tg = lane >> 4;                          // the group: k-rows 8 g .. 8 g + 7 of a slice
  // The transposing reads are issued as inline assembly: the compiler cannot tell that they do not touch the stage
  // the LDS-filling loads are writing and would wait for those loads before every one of them.  Their results are
  // therefore handed over by an explicit wait (tr_wait_*) that also names the registers, so that no use moves above it.
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) char*)(base)));
  // LDS byte address of this lane's chunk for block t (16 entries = two units) of an operand whose sub-tile starts at
  // unit u0: k-row 8 g + j, 8-byte half of the unit, unit slot; stage, region, slice and the + 4 k-rows of the second
  // read are added as offsets
  auto tr_addr = [&](int u0, int t) -> uint32_t {
    const int unit = u0 + t * 2 + (tq >> 1);
    return lds0 + (tg * 8 + tj) * 512 + (tq & 1) * 8 + ((unit ^ (4 * tj) ^ (2 * (tg & 1))) * 16);
  };
  uint32_t tra[C::MI], trb[C::NI];
#pragma unroll
  for (int i = 0; i < C::MI; ++i) tra[i] = tr_addr(wm * (C::WTM / 8), i);
#pragma unroll
  for (int j = 0; j < C::NI; ++j) trb[j] = tr_addr(wn * (C::WTN / 8), j);
  typedef short short8v __attribute__((ext_vector_type(8)));
  bf16x8 af[2][HA], bfr[2][C::NI];
  auto fload_a = [&](int buf, int ia, auto s_c, auto h_c) {
    constexpr int s = decltype(s_c)::value, h = decltype(h_c)::value;
    const uint32_t stoff = kABase + static_cast<uint32_t>(ia) * kAStage;
#pragma unroll
    for (int i = 0; i < HA; ++i) {
      if (ATR) {
        short4v lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(tra[h * HA + i] + stoff), "n"(s * 32 * 512));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(tra[h * HA + i] + stoff), "n"(s * 32 * 512 + 4 * 512));
        const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        af[buf][i] = __builtin_bit_cast(bf16x8, v);
      } else {
        const int coff = ((4 * s + (lane >> 4)) ^ sw) * 16;
        af[buf][i] = *reinterpret_cast<const bf16x8*>(base + stoff + arow + coff + (h * HA + i) * 16 * R::ROWB);
      }
    }
  };
  auto fload_b = [&](int buf, int ib, auto s_c) {
    constexpr int s = decltype(s_c)::value;
    const uint32_t stoff = kBBase + static_cast<uint32_t>(ib) * kBStage;
#pragma unroll
    for (int j = 0; j < C::NI; ++j) {
      if (BTR) {
        short4v lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(trb[j] + stoff), "n"(s * 32 * 512));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(trb[j] + stoff), "n"(s * 32 * 512 + 4 * 512));
        const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        bfr[buf][j] = __builtin_bit_cast(bf16x8, v);
      } else {
        const int coff = ((4 * s + (lane >> 4)) ^ sw) * 16;
        bfr[buf][j] = *reinterpret_cast<const bf16x8*>(base + stoff + brow + coff + j * 16 * R::ROWB);
      }
    }
  };
  // every LDS read issued so far has returned; the named fragments may be used from here on
  auto tr_wait_a = [&](int buf) {
    if (ATR) {
#pragma unroll
      for (int i = 0; i < HA; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(af[buf][i]));
    }
  };
  auto tr_wait_b = [&](int buf) {
    if (BTR) {
#pragma unroll
      for (int j = 0; j < C::NI; ++j) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bfr[buf][j]));
    }
  };
  auto mfmas = [&](int abuf, int bbuf, int h) {
#pragma unroll
    for (int i = 0; i < HA; ++i)
#pragma unroll
      for (int jj = 0; jj < C::NI; ++jj) {
        const int j = i & 1 ? C::NI - 1 - jj : jj;
        acc[h * HA + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[abuf][i], bfr[bbuf][j], acc[h * HA + i][j], 0, 0, 0);
      }
  };

  constexpr int kDsA = (ATR ? 2 : 1) * HA, kDsB = (BTR ? 2 : 1) * C::NI;   // LDS reads of an A half, of a slice of B
  auto interleave = [&](int n_ds, int n_vm) {
#pragma unroll
    for (int i = 0; i < HA * C::NI; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i < n_ds) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (i < n_vm) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto clamp_sub = [&](int sub) { return sub < nsub ? sub : nsub - 1; };   // past the end the last step is loaded again (nobody reads it)
  gload_a(0, 0);
  gload_b(0, 0);
  if (AHEAD == 1) gload_a(clamp_sub(1), 1);
  if (AHEAD == 2) gload_b(clamp_sub(1), 1);
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_s_barrier();
  auto next3 = [](int i) { return i == 2 ? 0 : i + 1; };
  int ia = 0, ib = 0;                                // stages of the current step
  if (CUT && wm * C::WTM >= m_rows) {                // the loads and barriers of the loop below
    for (int j = 0; j < nsub; ++j) {
      const int ia1 = AHEAD == 1 ? next3(ia) : (ia ^ 1), ib1 = AHEAD == 2 ? next3(ib) : (ib ^ 1);
      if (AHEAD == 1) {
        gload_b(clamp_sub(j + 1), ib1);
        gload_a(clamp_sub(j + 2), next3(ia1));
      } else {
        gload_a(clamp_sub(j + 1), ia1);
        gload_b(clamp_sub(j + 2), next3(ib1));
      }
      __builtin_amdgcn_s_waitcnt(0x0074);
      __builtin_amdgcn_s_barrier();
      ia = ia1;
      ib = ib1;
    }
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    return;
  }
  fload_b(0, 0, I0{});
  fload_a(0, 0, I0{}, I0{});
  for (int j = 0; j < nsub; ++j) {
    const int ia1 = AHEAD == 1 ? next3(ia) : (ia ^ 1);              // stages of the next step
    const int ib1 = AHEAD == 2 ? next3(ib) : (ib ^ 1);
    tr_wait_a(0);
    tr_wait_b(0);
    if (AHEAD == 1) {                                // the loads that may stay outstanding go out last
      gload_b(clamp_sub(j + 1), ib1);
      gload_a(clamp_sub(j + 2), next3(ia1));
    } else {
      gload_a(clamp_sub(j + 1), ia1);
      gload_b(clamp_sub(j + 2), next3(ib1));
    }
    fload_a(1, ia, I0{}, I1{});
    mfmas(0, 0, 0);
    interleave(kDsA, 8);
    __builtin_amdgcn_sched_barrier(0);
    tr_wait_a(1);
    fload_b(1, ib, I1{});
    fload_a(0, ia, I1{}, I0{});
    mfmas(1, 0, 1);
    interleave(kDsA + kDsB, 0);
    __builtin_amdgcn_sched_barrier(0);
    tr_wait_a(0);
    tr_wait_b(1);
    fload_a(1, ia, I1{}, I1{});
    mfmas(0, 1, 0);
    interleave(kDsA, 0);
    __builtin_amdgcn_sched_barrier(0);
    // own LDS reads of this step done and own loads for the next step landed: with three A stages the four
    // youngest loads (A of the step after next) may still be on their way; then everybody's
    __builtin_amdgcn_s_waitcnt(0x0074);              // vmcnt(4), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    tr_wait_a(1);
    fload_b(0, ib1, I0{});
    fload_a(0, ia1, I0{}, I0{});
    mfmas(1, 1, 1);
    interleave(kDsA + kDsB, 0);
    __builtin_amdgcn_sched_barrier(0);
    ia = ia1;
    ib = ib1;
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_s_barrier();
}

// Column of the accumulators of blocks (., j) inside the workgroup tile: l % 16 of the block.
template <class C>
__device__ __forceinline__ int acc_col(int j) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave % C::WN) * C::WTN + j * 16 + (lane & 15);
}

// Workgroups are handed to the 8 XCDs round-robin; give every XCD a contiguous range of the
// logical tile order, and order tiles in groups of GM x GN so that the workgroups resident on
// one XCD share operand rows through its L2.  A workgroup handles `per_wg` tiles one after the other:
// the tile with the same place in `per_wg` consecutive groups, so that the workgroups of an XCD keep
// working on one group at a time.  With at most GN column tiles the tiles themselves are numbered, column tiles of a row
// tile next to each other, one to a workgroup: the same sharing, and the few rounds there are come out even (groups
// half or more empty left 96 of 256 compute units idle with one column tile).
// More column tiles than `panel` (a multiple of GN) are worked through a panel of them after the other, all XCDs in the same
// panel: the B operand of a panel is read again for every GM row tiles, from the memory-side cache if it fits there.
// Returns false when iteration `it` of this workgroup has no tile.
template <int GM, int GN>
__device__ __forceinline__ bool tile_coords(int tiles_m, int tiles_n, int panel, int* tm, int* tn, int it, int per_wg) {
  const int xcd = static_cast<int>(blockIdx.x & 7), w = static_cast<int>(blockIdx.x >> 3);   // w: workgroup number inside its XCD
  if (tiles_n <= GN) {
    const int per_xcd = (tiles_m * tiles_n + 7) / 8, t = xcd * per_xcd + w;
    *tm = t / tiles_n;
    *tn = t % tiles_n;
    return it == 0 && w < per_xcd && *tm < tiles_m;
  }
  const int groups_m = (tiles_m + GM - 1) / GM;
  const int full = (groups_m * (panel / GN) + 7) / 8;                      // groups of a whole panel per XCD
  const int grp_in_seq = w / (GM * GN) * per_wg + it, within = w % (GM * GN);
  const int p = min(grp_in_seq / full, (tiles_n - 1) / panel), n0 = p * panel;
  const int groups_n = (min(panel, tiles_n - n0) + GN - 1) / GN, groups = groups_m * groups_n;
  const int groups_per_xcd = (groups + 7) / 8;                             // contiguous range of the panel's groups per XCD
  const int grp_in_xcd = grp_in_seq - p * full, grp = xcd * groups_per_xcd + grp_in_xcd;
  if (grp_in_xcd >= groups_per_xcd || grp >= groups) return false;
  const int gm = grp / groups_n;
  *tm = gm * GM + within % GM;
  *tn = n0 + (grp - gm * groups_n) * GN + within / GM;
  return *tm < tiles_m && *tn < tiles_n;
}
// Shares of a sequence of tiles per XCD: XCD x owns tiles first[x] .. first[x + 1] - 1.
struct XcdShares {
  int first[9];
};
// Tile number t of tiles_m x tiles_n, numbered group of GM x GN after group (row of groups after row of groups; the groups at
// the edges are smaller), so that any run of GM GN numbers shares operand rows.
template <int GM, int GN>
__device__ __forceinline__ void tile_of_groups(int t, int tiles_m, int tiles_n, int* tm, int* tn) {
  const int gm = t / (GM * tiles_n), in_row = t - gm * (GM * tiles_n), rows = min(GM, tiles_m - gm * GM);
  const int gn = in_row / (rows * GN), in_group = in_row - gn * (rows * GN), c = in_group / rows;
  *tm = gm * GM + in_group - c * rows;
  *tn = gn * GN + c;
}
template <int GM, int GN>
inline unsigned tile_grid(int tiles_m, int tiles_n, int panel, int per_wg) {   // workgroups tile_coords needs
  if (tiles_n <= GN) return static_cast<unsigned>((static_cast<long long>(tiles_m) * tiles_n + 7) / 8 * 8);
  const long long groups_m = (tiles_m + GM - 1) / GM, panels = (tiles_n - 1) / panel;                  // whole panels in front of the last
  const long long last = (tiles_n - panels * panel + GN - 1) / GN;
  const long long groups_per_xcd = panels * ((groups_m * (panel / GN) + 7) / 8) + (groups_m * last + 7) / 8;
  const long long wg_groups = (groups_per_xcd + per_wg - 1) / per_wg;       // groups of workgroups per XCD
  return static_cast<unsigned>(wg_groups * (GM * GN) * 8);
}

}  // namespace umas
