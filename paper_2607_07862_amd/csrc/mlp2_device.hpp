// Device building blocks of the tile-pipelined two-layer MLP on gfx950.
//
//   * an LDS double-buffered bf16 MFMA tile mainloop (v_mfma_f32_16x16x32_bf16),
//     with the row-major weight tile read transposed out of LDS by
//     ds_read_b64_tr_b16;
//   * the fused epilogues: activation + bf16 store + ready signal for GEMM1,
//     bf16 store for GEMM2, and a deterministic split-K reduction;
//   * the flag primitives: increment of a ready counter by the
//     producer, bounded acquire-spin by the consumer (Sec. III-A: the
//     producer fences its data before it signals; the consumer polls before
//     it reads).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlp2 {

template <class A, class B>
struct is_same_type {
  static constexpr bool value = false;
};
template <class A>
struct is_same_type<A, A> {
  static constexpr bool value = true;
};
template <bool V>
struct bool_constant {
  static constexpr bool value = V;
};
template <int V>
struct int_constant {
  static constexpr int value = V;
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4_t;

constexpr int kBK = 64;        // K granularity of the plans (split-K ranges); a plan whose tiles take
                               // 128-deep stages keeps its K ranges multiples of 128

// Words per 128-byte line.  Every counter that work-groups update with device-
// scope atomics sits on a line of its own: such atomics are performed at the
// memory side of the device, one at a time per line, so counters sharing a
// line would queue behind each other's traffic.
constexpr int kLine = 32;

// Control words of a plan (device memory, zero at plan creation), one per line.
enum {
  CTRL_EPOCH = 0,                  // runs completed; read at kernel start, bumped by the run's last work-group
  CTRL_ERROR = 1 * kLine,          // nonzero once a bounded flag wait gave up
  CTRL_DONE_ALL = 2 * kLine,       // claim lists of the current kernel whose work-groups have all finished
  CTRL_TICKET = 3 * kLine,         // CTRL_TICKET + l * kLine: next ticket of claim list l (up to 16 lists:
                                   // 8 per role when the pipelined launch splits the grid into roles)
  CTRL_DONE = 19 * kLine,          // CTRL_DONE + l * kLine: finished work-groups of claim list l
  CTRL_QHEAD = 35 * kLine,         // workqueue mode: CTRL_QHEAD + l * kLine: queue slots that consumers of
                                   // claim list l have claimed (8 lists)
  CTRL_QTAIL = 43 * kLine,         // workqueue mode: next queue slot a producer fills
  CTRL_EPOCH_WQ = 44 * kLine,      // workqueue runs completed (the scoreboards advance in those only)
  CTRL_EPOCH_SN = 45 * kLine,      // sentinel runs completed (their parity picks the intermediate buffer)
  CTRL_WORDS = 46 * kLine
};
__device__ __forceinline__ int ctrl_ticket(int l) { return CTRL_TICKET + l * kLine; }
__device__ __forceinline__ int ctrl_done(int l) { return CTRL_DONE + l * kLine; }

enum { ACT_IDENTITY = 0, ACT_GELU_TANH = 1, ACT_SWIGLU = 2 };

struct Args {
  const uint16_t* X;   // [M, H]
  const uint16_t* W1;  // [H, F]  (SwiGLU: [2, H, F])
  const uint16_t* W2;  // [F, H]
  uint16_t* Y;         // [M, H]
  uint16_t* Z;         // [Mpad, F]
  uint16_t* Zs;        // sentinel mode: two intermediates of [Mpad, F] each, zs_elems apart; sentinel runs
                       // alternate between them (the other one is refilled with sentinels meanwhile)
  long zs_elems;
  uint16_t* Zr;        // inside a sentinel run: the intermediate the next sentinel run uses (refilled with
                       // sentinels tile by tile); null otherwise
  float* part1;        // GEMM1 split-K partials (fragment-native), or null
  float* part2;        // GEMM2 split-K partials, or null
  uint32_t* cnt1;      // split-K arrival counters of GEMM1: tile t at word t * kLine
  uint32_t* cnt2;      // split-K arrival counters of GEMM2: tile t at word t * kLine
  uint32_t* ready;     // ready counters: tile (mb, nb1) at word (nb1 * Mb + mb) * kLine
  uint32_t* board;     // workqueue mode: scoreboard of GEMM2 unit q at word q * kLine
  uint32_t* queue;     // workqueue mode: ring of ready GEMM2 units, items2 + 1 slots (one per unit and
                       // run, and a spare)
  uint32_t* ctrl;      // CTRL_* words
  const uint32_t* order1;  // GEMM1 item per rank of the GEMM1 kernel, length items1
  const uint32_t* order2;  // GEMM2 item per rank of the GEMM2 kernel, length items2 + items_red
                           // (bit 30 set: reduction item)
  const uint32_t* orderp;  // item per rank of the pipelined kernel, length items1 + items2 + items_red
                           // (bit 31 set: GEMM2 item, bits 31 and 30: reduction item; else GEMM1 item id)
  int M, H, F, act;
  int Mb, Nb1, Nb2;        // row blocks; GEMM1 / GEMM2 column blocks
  int S1, S2;              // split-K factors
  int kc1, kc2;            // K per split (multiples of kBK)
  int items1, items2;      // GEMM1 / GEMM2 work items (tiles x split-K parts)
  int bn1;                 // GEMM1 column-block width (ready-counter granularity along GEMM2's K)
  uint32_t spin_limit;
  int drop_signal;         // GEMM1 tile whose signal is skipped (failure injection), -1 = none
  uint64_t* trace;         // per-work-group timing records (trace builds only), or null
  int trace_cap;           // records per work-group
  int trace_groups;        // work-groups per trace section (the largest grid of the plan)
  int lists;               // claim lists of the launch (1 or 8; work-group g claims from list g % lists)
  int first_static;        // work-groups g < first_static take rank g as their first item without a
                           // ticket (ranks below it are items that never wait); the others claim
  int p1;                  // pipelined launch: 0 = shared roles; else work-groups with g % 64 < p1 take
                           // GEMM1 items only (from order1) and the others GEMM2 items only (order2)
  int lists2;              // claim lists of the GEMM2 role (role split only; `lists` is the GEMM1 role's)
  int red2;                // GEMM2 split-K: 0 = the part that arrives last sums the tile; else the tile is
                           // summed by red2 reduction items (slices of its units), ranked after every GEMM2 item
  int items_red;           // reduction items of the launch (tiles2 * red2, or 0)
};

// ------------------------------------------------------------------ optional timing trace
//
// Built with -DMLP2_TRACE, thread 0 of every work-group records per item:
// {rank, start, mainloop end, split-K arrival released, siblings arrived, end,
// ring-wait ticks, flag-wait ticks} on the 100 MHz real-time counter.  Ring waits are the mainloop's waits for its own
// loads plus the stage barrier; flag waits are ready-counter and sibling waits.
// Without the macro every hook compiles to nothing.
#ifdef MLP2_TRACE
constexpr bool kTrace = true;
#else
constexpr bool kTrace = false;
#endif
constexpr int kTraceWords = 8;

struct TraceAcc {
  uint64_t ring = 0, flag = 0, t_main = 0, t_rel = 0, t_wait = 0;
  uint64_t c_start = 0;  // shader-clock counter at the item's start
};

__device__ __forceinline__ uint64_t trace_now() {
  if constexpr (kTrace) return __builtin_amdgcn_s_memrealtime();
  return 0;
}

// Shader-clock counter (core clock cycles): beside the real-time counter it
// gives the clock an item ran at.
__device__ __forceinline__ uint64_t trace_clock() {
  if constexpr (kTrace) return __builtin_amdgcn_s_memtime();
  return 0;
}

// ------------------------------------------------------------------ scalars

__device__ __forceinline__ uint32_t ld_relaxed(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A value every lane of the wave holds (read from LDS after a barrier, or
// loaded from a wave-uniform address), moved to a scalar register so that
// branches on it are scalar branches.  Every branch that has a barrier on
// either side must be taken this way: the compiler cannot prove uniformity
// of an LDS or memory value by itself and would otherwise lay the code out as
// an exec-masked divergent region, in which waves can execute different
// numbers of s_barrier and deadlock the work-group.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// The thread's index through an empty asm, for what an item derives from it
// alone: otherwise the compiler computes all of that before the persistent
// item loop and, in the 256-row kernels, keeps it in scratch memory.
__device__ __forceinline__ int thread_here() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// Every wave waits until its own outstanding memory operations are complete
// (stores acknowledged), so that a later count by one lane of
// the work-group covers the data of all waves.
__device__ __forceinline__ void wait_all_mem() { __builtin_amdgcn_s_waitcnt(0); }

// e^{-t} through the hardware base-2 exponential.
__device__ __forceinline__ float exp_neg(float t) { return __builtin_amdgcn_exp2f(-1.4426950408889634f * t); }

// GELU (tanh form): 0.5 z (1 + tanh(y)) with y = sqrt(2/pi)(z + 0.044715 z^3).
// Uses the identity 0.5 (1 + tanh(y)) = 1 / (1 + e^{-2y}).
__device__ __forceinline__ float gelu_tanh(float z) {
  const float y = 0.7978845608028654f * (z + 0.044715f * z * z * z);
  return z / (1.0f + exp_neg(2.0f * y));
}

// SiLU: g / (1 + e^{-g}).
__device__ __forceinline__ float silu(float g) { return g / (1.0f + exp_neg(g)); }

__device__ __forceinline__ u32x4 pack_bf16x8(const float (&v)[8]) {
  bf16x8 b;
#pragma unroll
  for (int i = 0; i < 8; ++i) b[i] = (__bf16)v[i];  // round to nearest even
  return __builtin_bit_cast(u32x4, b);
}

// ------------------------------------------------------------------ tile geometry

// A work-group tile of BM rows (the M side: X or Z rows) by BN columns (the N
// side: W columns), staged through an NS-deep ring of LDS buffers of kBK rows
// of K each.  Four or eight 64-wide waves in a WM x WN grid; each wave owns a
// (BM/WM) x (BN/WN) sub-tile made of 16x16 MFMA blocks.  Eight waves let a
// large tile (256 x 256: a quarter of the operand bytes per flop of 128 x 128)
// keep two waves per SIMD, so that one wave's LDS reads overlap the other's
// products.
//
// The MFMA is issued with the *weight* fragment as its A operand and the
// activation fragment as its B operand, so each lane ends up holding output
// row (lane % 16) and, for a pair of adjacent blocks, 8 consecutive output
// columns: the epilogue stores 16 contiguous bytes per lane.
//
// LDS stage layout (bytes), both parts unpadded and XOR-swizzled in 16-byte
// chunks, because the direct-to-LDS loads write each wave's 1 KB contiguously
// (lane i -> bytes 16 i):
//   activation tile [BM][BK] bf16, rows of BK * 2 bytes, XOR-swizzled per
//     chunk (swz_a) so that the 16 rows read by one ds_read_b128 group land
//     in 16 distinct 4-bank groups;
//   weight tile [BK][BN] bf16 per operand: chunk c of row k at c ^ swzB(k),
//     which puts the 4 rows read by one ds_read_b64_tr_b16 group in
//     different banks.
template <int BM_, int BN_, int WM_, int WN_, int NS_, int BK_ = kBK, bool WNT_ = false>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_;
  // Weight loads with the non-temporal hint (plans whose weights exceed the
  // last-level cache): the streamed weights then stop displacing the lines
  // that the activation loads reuse.
  static constexpr bool WNT = WNT_;
  // K depth of one stage: 64; 32 (half the bytes per stage, so a ring of the
  // same LDS holds twice the stages); or 128 (twice the products per stage
  // for the same per-stage costs: the wait, the barrier, the DMA issue and
  // the first fragment reads, which a small tile with one wave per SIMD pays
  // in series).  The activation tile's rows are BK * 2 bytes.
  static constexpr int BK = BK_;
  static_assert(BK == 128 || BK == 64 || BK == 32, "stage depth");
  static constexpr int ROW_BYTES = BK * 2;      // activation tile row pitch in LDS
  static constexpr int CHUNKS = BK / 8;         // 16-byte chunks per activation row
  static constexpr int NWAVES = WM * WN;
  static constexpr int THREADS = 64 * NWAVES;
  static_assert(NWAVES == 4 || NWAVES == 8, "four or eight waves");
  static_assert(BN == 64 || BN == 128 || BN == 256, "weight tile width");
  static_assert(NS >= 2, "at least double buffered");
  static constexpr int MW = BM / WM;  // rows per wave
  static constexpr int NW = BN / WN;  // columns per wave
  static constexpr int TM = MW / 16;
  static constexpr int TN = NW / 16;
  // The quadrant tile: 256 rows over eight waves with a two-stage ring runs
  // the ping-pong mainloop (below), whose waves own 64 x 32 blocks of the four
  // 128 x 128 quadrants instead of one contiguous block.
  static constexpr bool QUAD = BM == 256 && WM == 2 && WN == 4 && NS == 2 && BK_ == 64 && (BN == 128 || BN == 256);
  // The pair tile: 256 x 128 with a three-stage ring, the same loop over two
  // 128 x 128 halves (for products with too few 256 x 256 tiles).
  static constexpr bool PAIR = BM == 256 && WM == 2 && WN == 4 && NS == 3 && BK_ == 64 && BN == 128;
  static constexpr bool HALVES = QUAD || PAIR;  // waves own 64-row blocks of both row halves
  // First row of row block tm, and first column of block pair tp, of the wave at (wm, wn).
  __device__ static constexpr int row_of(int wm, int tm) {
    return HALVES ? 64 * wm + 16 * (tm & 3) + 128 * (tm >> 2) : wm * MW + 16 * tm;
  }
  __device__ static constexpr int col_of(int wn, int tp) { return HALVES ? 32 * wn + 128 * tp : wn * NW + 32 * tp; }
  static_assert(TM >= 1 && TN >= 2 && TN % 2 == 0, "wave tile shape");
  static constexpr int A_BYTES = BM * BK * 2;
  static constexpr int B_BYTES = BK * BN * 2;
  static constexpr int A_DMA = A_BYTES / 1024 / NWAVES;  // 1 KB wave loads per wave and stage
  static constexpr int B_DMA = B_BYTES / 1024 / NWAVES;
  static_assert(A_DMA >= 1 && B_DMA >= 1 && A_BYTES % (1024 * NWAVES) == 0 && B_BYTES % (1024 * NWAVES) == 0,
                "every wave loads whole 1 KB pieces of both operands");
  template <int NB>
  static constexpr int stage_bytes() { return A_BYTES + NB * B_BYTES; }
  template <int NB>
  static constexpr int lds_bytes() { return NS * stage_bytes<NB>(); }
  template <int NB>
  static constexpr int dma_per_stage() { return A_DMA + NB * B_DMA; }
};

// Activation tile swizzle: 256-byte rows (BK = 128), one to a bank period,
// put chunk c of row r at c ^ (r & 15); 128-byte rows (BK = 64) at
// c ^ ((r >> 1) & 7); 64-byte rows (BK = 32), four to a bank period, at
// c ^ ((r >> 2) & 3).  Either way the 16 rows one ds_read_b128 group reads
// land in 16 distinct 4-bank groups.
template <int BK = kBK>
__device__ __forceinline__ int swz_a(int row) {
  return BK == 128 ? row & 15 : BK == 64 ? (row >> 1) & 7 : (row >> 2) & 3;
}
template <int BN>
__device__ __forceinline__ int swz_b(int k) {
  return BN >= 128 ? 4 * (k & 3) : 4 * ((k >> 1) & 1);
}

// One 16-byte-per-lane direct-to-LDS load: lane i reads 16 bytes at
// base + voff and writes them to LDS at lds_addr + 16 i.  Issued through
// inline assembly so that the compiler does not serialise every LDS read
// behind it (it cannot tell the ring's stages apart); completion is tracked
// explicitly with s_waitcnt vmcnt.  M0 carries the LDS address: it is an
// operand of the asm ("{m0}" constraint), so the compiler itself writes it and
// knows the register holds that value, and never has a value of its own there.
// The base goes through a scalar move of the asm's own: a vector-memory
// instruction must not read a scalar register within five wait states of a
// vector instruction that wrote it (a spilled scalar comes back by
// v_readlane), which the compiler keeps for its own instructions but not for
// the ones in here; the move also stands between the write of M0 and its use.
#define MLP2_DMA16(FLAGS)                                                                              \
  const void* b;                                                                                       \
  asm volatile("s_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0" FLAGS                              \
               : "=&s"(b)                                                                              \
               : "v"(voff), "s"(base), "{m0}"(lds_addr)                                                \
               : "memory")
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds_addr) { MLP2_DMA16(""); }

// The same load with the non-temporal hint (a streamed operand read once).
__device__ __forceinline__ void dma16_nt(const void* base, uint32_t voff, uint32_t lds_addr) {
  MLP2_DMA16(" nt");
}

// The same load at device scope (sc1, the scope bit of the compiler's own
// agent-scope atomic loads): it reads the device's point of coherence rather
// than a line the consumer's XCD L2 may hold.  The sentinel mode's consumers
// read the intermediate this way, since no release and acquire order it.
__device__ __forceinline__ void dma16_coherent(const void* base, uint32_t voff, uint32_t lds_addr) {
  MLP2_DMA16(" sc1");
}
#undef MLP2_DMA16

// ------------------------------------------------------------------ sentinel synchronisation
//
// Sec. V-A of the paper: instead of a fence and a flag per tile, the
// intermediate buffer holds a sentinel value before its producer writes it,
// and the consumer re-reads until no sentinel is left.  The sentinel is the
// bf16 pattern 0xFFFF (a NaN with every payload bit set).  The GEMM1 epilogue
// never writes it (canonicalize_z turns it into the canonical NaN 0x7FC0, in
// every mode, so the modes stay bit-identical), so an element still holding
// 0xFFFF has not been written yet; the check is per element, so a load that
// sees part of a 16-byte piece before the rest was written is caught too.
constexpr uint16_t kSentinel = 0xFFFF;

__device__ __forceinline__ bool has_sentinel(u32x4 v) {
  bool any = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) any |= (v[i] & 0xFFFFu) == 0xFFFFu || (v[i] >> 16) == 0xFFFFu;
  return any;
}

__device__ __forceinline__ u32x4 canonicalize_z(u32x4 v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if ((v[i] & 0xFFFFu) == 0xFFFFu) v[i] = (v[i] & 0xFFFF0000u) | 0x7FC0u;
    if ((v[i] >> 16) == 0xFFFFu) v[i] = (v[i] & 0xFFFFu) | 0x7FC00000u;
  }
  return v;
}

// A 16-byte piece of the intermediate stored at device scope without any
// fence: two 8-byte agent-scope relaxed atomic stores (each single-copy atomic).
__device__ __forceinline__ void store_coherent16(uint16_t* p, u32x4 v) {
  uint64_t* q = reinterpret_cast<uint64_t*>(p);
  __hip_atomic_store(q, (uint64_t)v[0] | ((uint64_t)v[1] << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(q + 1, (uint64_t)v[2] | ((uint64_t)v[3] << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 16 bytes stored through to the device's point of coherence (the sc1 bit of
// the compiler's own agent-scope atomic stores): once the store is
// acknowledged (vmcnt), every XCD can read it.  Data published inside a
// launch (Z tiles, split-K partials) is stored this way, so publishing needs
// only that wait and a relaxed atomic.  An agent-scope release instead writes
// back the XCD's whole L2, once per work-group and item, in turn: at 32 rows
// and less that was a third to half of the run (figures at release_add).
// `base` is the same in every lane; `off` is in bytes, below 4 GiB.
__device__ __forceinline__ void store_through16(void* base, uint32_t off, u32x4 v, int step = 0) {
  constexpr int kSc1 = 16;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000);
  __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, (int)off, step, kSc1);
}

// Wait until at most n of this wave's vector-memory operations are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Wait until this wave's loads of the current stage are complete while the
// `after` (<= A) stages issued behind it stay in flight.  `after` is uniform.
template <int PER, int A>
__device__ __forceinline__ void wait_stages_behind(int after) {
  if constexpr (A <= 0) {
    wait_vm<0>();
  } else {
    static_assert(A * PER <= 63, "vmcnt holds at most 63 outstanding loads");
    if (after >= A) wait_vm<A * PER>();
    else wait_stages_behind<PER, A - 1>(after);
  }
}

// ------------------------------------------------------------------ mainloop

// acc[b][tn][tm] = sum over k in [kbeg, kend) of W_b[k][n] * A[m][k] for the
// tile at (m0, n0[b]).  A rows past `mlast` are clamped to `mlast`, and
// columns past the last 8 of W's `ldb` to those (the results of either are
// never stored).  `wait(k)` runs, in every wave, before the activation
// operand of the stage starting at k is requested (after its weight loads).
//
// Pipeline: stages k0, k0 + BK, ... are loaded NS - 1 ahead of use.  At
// iteration it a wave waits for its own loads of stage it, a barrier makes
// every wave's loads of stage it visible and retires every wave's reads of
// stage it - 1, then the loads of stage it + NS - 1 go into that freed buffer
// and stage it is multiplied.  Four-wave tiles with three or more stages read
// one stage ahead into registers instead (below), and keep NS stages loading.
// A stage check that does nothing (every mode but the sentinel mode).
struct NoCheck {
  static constexpr bool kCoherentA = false;
  template <class... X>
  __device__ __forceinline__ void operator()(X...) {}
};

// The mainloop of the quadrant tile (Tile::QUAD): 256 rows by two column halves
// of 128 (one 256-column operand, or two 128-column ones), eight waves, two
// waves to a SIMD.
//
// What bounds it: a 64-deep stage is 2048 cycles of MFMA per SIMD, and its
// fragment reads and direct-to-LDS writes keep the LDS busy about three
// quarters of that time.  With every wave reading its fragments after one barrier and the
// whole next stage requested only then, neither side overlapped: 3700 cycles
// a stage.  Here the two waves of a SIMD alternate instead (waves 0-3 run half
// a phase ahead of waves 4-7): while one multiplies, the other reads the
// fragments of its next products and requests loads.
//
// A stage is four phases, one output quadrant (rows half a, columns half b)
// of 64 x 32 per wave and 16 products each, in the order
//   phase 0: (A0, B0)   1: (A0, B1)   2: (A1, B1)   3: (A1, B0)
// and a phase is a memory slot and a product slot, each ended by a barrier:
//   memory slot 0 of stage it: request A1 of stage it + 1, read B0 of stage it
//               1:             request A0 of it + 2,       read B1 of it
//               2:             request B0 of it + 2,       read A1 of it
//               3:             request B1 of it + 2,       read A0 of it + 1
// Each half tile is requested six phases before it is read, so five half
// tiles (80 KB of the 128 KB ring) stay in flight and no wait drains them.
//   * Visibility: a wave waits for its own pieces of a half tile at the end
//     of the memory slot before the one that reads it.  The trailing waves
//     reach that wait one slot before the leading waves read, and a barrier
//     lies between.
//   * Reuse: a half tile read in memory slot p is complete in registers at
//     product slot p (lgkmcnt(0)), and its ring slot is requested again in
//     memory slot p + 2.  The trailing waves' product slot p ends, with a
//     barrier, before the leading waves' memory slot p + 2 begins.
// An item that may have to wait for its activation rows: wave 0 waits in
// memory slot 0 for the rows of stage it + 2, which no wave requests before
// the barrier that ends the slot, so that barrier is the broadcast.
//
// Measured against the plain two-stage loop (pipelined mode): 8192 rows
// through 8192 x 8192 weights 1682 -> 1528 us (1.31 -> 1.44 PFLOP/s),
// 2048 x 4096 x 14336 429 -> 396 us, gated 256 x 8192 x 28672 374 -> 339 us.
//
// The products of one output run in the same order as in the plain mainloop.
template <class T, int NB, class Wait>
__device__ __forceinline__ void mainloop_quad(const uint16_t* __restrict__ A, long lda, int m0, int mlast,
                                              const uint16_t* const (&Bp)[NB], const int (&n0)[NB], long ldb, int kbeg,
                                              int kend, f32x4 (&acc)[NB][T::TN][T::TM], char* lds, Wait& wait, TraceAcc& tr) {
  static_assert(T::QUAD && NB * T::BN == 256 && T::TM == 8 && NB * T::TN == 4 && T::NWAVES == 8, "quadrant tile");
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // per-lane offsets are derived per call, as in the plain mainloop
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wm = wave % T::WM, wn = wave / T::WM;
  const bool trailing = wave >= 4;

#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < T::TN; ++i)
#pragma unroll
      for (int j = 0; j < T::TM; ++j) acc[b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nk = (kend - kbeg) / 64;
  if (nk <= 0) return;

  constexpr uint32_t kHalf = 16384, kB = 2 * kHalf, kStage = 4 * kHalf;  // LDS: A0, A1, B0, B1 per stage
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;

  // Load sources: per-lane offsets from a per-stage uniform base.  A half: 128
  // rows of 128 bytes, 8 to a 1 KB piece; B half: 64 rows of 256 bytes, 4 to a piece.
  uint32_t a_off[4], b_off[2][2];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = 8 * (wave + 8 * j) + lane / 8;
    int gr = m0 + row;
    gr = gr > mlast ? mlast : gr;
    a_off[j] = (uint32_t)(((long)gr * lda + 8 * ((lane & 7) ^ swz_a<64>(row))) * 2);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = 4 * (wave + 8 * j) + lane / 16;
      const int col = (NB == 2 ? n0[h % NB] : n0[0] + 128 * h) + 8 * ((lane & 15) ^ swz_b<128>(row));
      b_off[h][j] = (uint32_t)(((long)row * ldb + min(col, (int)ldb - 8)) * 2);
    }
  const uint16_t* pa = A + kbeg;
  const uint16_t* pb[2] = {Bp[0] + (long)kbeg * ldb, Bp[NB - 1] + (long)kbeg * ldb};

  auto load_a = [&](int half, int st) {
    const uint32_t dst = lds_base + (uint32_t)(st & 1) * kStage + (uint32_t)half * kHalf + (uint32_t)wave * 1024u;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16(pa + (long)st * 64, a_off[2 * half + j], uniform(dst + 8192u * j));
  };
  auto load_b = [&](int half, int st) {
    const uint32_t dst = lds_base + (uint32_t)(st & 1) * kStage + kB + (uint32_t)half * kHalf + (uint32_t)wave * 1024u;
    const uint16_t* src = pb[half] + (long)st * 64 * ldb;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (T::WNT) dma16_nt(src, b_off[half][j], uniform(dst + 8192u * j));
      else dma16(src, b_off[half][j], uniform(dst + 8192u * j));
    }
  };

  // Fragment addresses inside a stage (the plain mainloop's, per half tile).
  const int arow = T::row_of(wm, 0) + (lane & 15);
  uint32_t a_frag[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) a_frag[ks] = (uint32_t)(arow * 128 + (((4 * ks + (lane >> 4)) ^ swz_a<64>(arow)) << 4));
  const int brow = 8 * (lane >> 4) + ((lane & 15) >> 2);
  const uint32_t b_frag = kB + (uint32_t)(brow * 256 + (((4 * wn + (lane & 3)) ^ swz_b<128>(brow)) << 4));

  bf16x8 xa[2][4], xb[2][4], w0[2][2], w1[2][2];
  auto read_a = [&](bf16x8 (&x)[2][4], int half, int st) {
    const char* base = lds + (st & 1) * kStage + half * kHalf;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int tm = 0; tm < 4; ++tm) x[ks][tm] = *reinterpret_cast<const bf16x8*>(base + a_frag[ks] + tm * 2048);
  };
  auto read_b = [&](bf16x8 (&w)[2][2], int half, int st) {
    const char* base = lds + (st & 1) * kStage + half * kHalf;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const char* p = base + b_frag + ks * 8192 + i * 8;
        bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p));
        bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p + 1024));
        w[ks][i] = (bf16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
  };
  auto mma = [&](const bf16x8 (&w)[2][2], const bf16x8 (&x)[2][4], auto bh, auto ah) {
    constexpr int b = decltype(bh)::value ? 1 : 0, a = decltype(ah)::value ? 4 : 0;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int tm = 0; tm < 4; ++tm) {
          f32x4& c = acc[NB == 2 ? b : 0][NB == 2 ? i : 2 * b + i][a + tm];
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][i], x[ks][tm], c, 0, 0, 0);
        }
  };
  using Lo = bool_constant<false>;
  using Hi = bool_constant<true>;

  auto slot_end = [&]() {  // a barrier that neither the compiler's memory operations nor its products cross
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto vm_traced = [&](auto n) {
    const uint64_t t0 = trace_now();
    wait_vm<decltype(n)::value>();
    if constexpr (kTrace) tr.ring += trace_now() - t0;
  };
  auto products_begin = [&]() {  // this wave's fragment reads are complete
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
  };
  auto products_end = [&]() {
    __builtin_amdgcn_s_setprio(0);
    slot_end();
  };

  // One stage.  LEFT: stages after it, counted up to 2 (fewer loads to request
  // and to leave in flight).
  auto stage = [&](int it, auto left_) {
    constexpr int LEFT = decltype(left_)::value;
    if constexpr (LEFT >= 1) load_a(1, it + 1);
    read_b(w0, 0, it);
    if constexpr (LEFT >= 2) {
      const int k = kbeg + (it + 2) * 64;
      if (Wait::kBlocks && wave == 0) wait.leader(k);
      wait.known(k);
    }
    vm_traced(int_constant<LEFT >= 1 ? 10 : 2>());  // B1 of this stage
    slot_end();
    products_begin();
    mma(w0, xa, Lo(), Lo());
    products_end();

    if constexpr (LEFT >= 2) load_a(0, it + 2);
    read_b(w1, 1, it);
    vm_traced(int_constant<LEFT >= 2 ? 10 : LEFT == 1 ? 8 : 0>());  // A1 of this stage
    slot_end();
    products_begin();
    mma(w1, xa, Hi(), Lo());
    products_end();

    if constexpr (LEFT >= 2) load_b(0, it + 2);
    read_a(xb, 1, it);
    if constexpr (LEFT >= 1) vm_traced(int_constant<LEFT >= 2 ? 10 : 6>());  // A0 of the next stage
    slot_end();
    products_begin();
    mma(w1, xb, Hi(), Hi());
    products_end();

    if constexpr (LEFT >= 2) load_b(1, it + 2);
    if constexpr (LEFT >= 1) {
      read_a(xa, 0, it + 1);
      vm_traced(int_constant<LEFT >= 2 ? 10 : 4>());  // B0 of the next stage
    }
    slot_end();
    products_begin();
    mma(w0, xb, Lo(), Hi());
    products_end();
  };

  // Prologue: the first stage and all of the second but A1.
  const bool two = nk > 1;
  if constexpr (Wait::kBlocks) {  // the weights stream while the item waits for its rows
    load_b(0, 0);
    load_b(1, 0);
    if (two) {
      load_b(0, 1);
      load_b(1, 1);
    }
    if (wave == 0) {
      wait.leader(kbeg);
      if (two) wait.leader(kbeg + 64);
    }
    slot_end();
    load_a(0, 0);
    load_a(1, 0);
    if (two) load_a(0, 1);
    wait_vm<0>();  // requested out of the stage order, so nothing less covers it
  } else {
    load_a(0, 0);
    load_b(0, 0);
    load_b(1, 0);
    load_a(1, 0);
    if (two) {
      load_a(0, 1);
      load_b(0, 1);
      load_b(1, 1);
      wait_vm<10>();  // A0, B0
    } else {
      wait_vm<4>();
    }
  }
  wait.known(kbeg);
  if (two) wait.known(kbeg + 64);
  slot_end();
  read_a(xa, 0, 0);
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)

  if (trailing) slot_end();
  for (int it = 0; it < nk - 2; ++it) stage(it, int_constant<2>());
  if (two) stage(nk - 2, int_constant<1>());
  stage(nk - 1, int_constant<0>());
  if (!trailing) slot_end();
  __syncthreads();  // every wave is done reading the ring before it is reused
}

// The mainloop of the pair tile (Tile::PAIR): 256 rows by 128 columns, as the
// quadrant tile's with one column half and so two phases a stage:
//   memory slot 0 of stage it: read B of stage it;             request B of it + 2
//               1:             read A1 of it and A0 of it + 1; request A1 of it + 2, A0 of it + 3
// Three stages of 48 KB (144 KB): every half tile is requested four phases
// before it is read, and two phases after its ring slot was; the waits and
// barriers are placed as in the quadrant tile's loop, whose visibility and
// reuse arguments hold unchanged.
template <class T, class Wait>
__device__ __forceinline__ void mainloop_pair(const uint16_t* __restrict__ A, long lda, int m0, int mlast,
                                              const uint16_t* B, int n0, long ldb, int kbeg, int kend,
                                              f32x4 (&acc)[T::TN][T::TM], char* lds, Wait& wait, TraceAcc& tr) {
  static_assert(T::PAIR && T::TM == 8 && T::TN == 2 && T::NWAVES == 8, "pair tile");
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // per-lane offsets are derived per call, as in the plain mainloop
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int wm = wave % T::WM, wn = wave / T::WM;
  const bool trailing = wave >= 4;

#pragma unroll
  for (int i = 0; i < T::TN; ++i)
#pragma unroll
    for (int j = 0; j < T::TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nk = (kend - kbeg) / 64;
  if (nk <= 0) return;

  constexpr uint32_t kHalf = 16384, kA1 = 3 * kHalf, kB = 6 * kHalf;  // LDS: A0, A1 and B, three stages each
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
  uint32_t a_off[4], b_off[2];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = 8 * (wave + 8 * j) + lane / 8;
    int gr = m0 + row;
    gr = gr > mlast ? mlast : gr;
    a_off[j] = (uint32_t)(((long)gr * lda + 8 * ((lane & 7) ^ swz_a<64>(row))) * 2);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = 4 * (wave + 8 * j) + lane / 16;
    const int col = n0 + 8 * ((lane & 15) ^ swz_b<128>(row));
    b_off[j] = (uint32_t)(((long)row * ldb + min(col, (int)ldb - 8)) * 2);
  }
  const uint16_t* pa = A + kbeg;
  const uint16_t* pb = B + (long)kbeg * ldb;
  auto load_a = [&](int half, int st, int slot) {
    const uint32_t dst = lds_base + (half ? kA1 : 0u) + (uint32_t)slot * kHalf + (uint32_t)wave * 1024u;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16(pa + (long)st * 64, a_off[2 * half + j], uniform(dst + 8192u * j));
  };
  auto load_b = [&](int st, int slot) {
    const uint32_t dst = lds_base + kB + (uint32_t)slot * kHalf + (uint32_t)wave * 1024u;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16(pb + (long)st * 64 * ldb, b_off[j], uniform(dst + 8192u * j));
  };

  // Fragment addresses inside a half tile.
  const int arow = T::row_of(wm, 0) + (lane & 15);
  uint32_t a_frag[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) a_frag[ks] = (uint32_t)(arow * 128 + (((4 * ks + (lane >> 4)) ^ swz_a<64>(arow)) << 4));
  const int brow = 8 * (lane >> 4) + ((lane & 15) >> 2);
  const uint32_t b_frag = kB + (uint32_t)(brow * 256 + (((4 * wn + (lane & 3)) ^ swz_b<128>(brow)) << 4));

  bf16x8 x0[2][4], x1[2][4], w[2][2];
  auto read_a = [&](bf16x8 (&x)[2][4], int half, int slot) {
    const char* base = lds + (half ? kA1 : 0u) + slot * kHalf;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int tm = 0; tm < 4; ++tm) x[ks][tm] = *reinterpret_cast<const bf16x8*>(base + a_frag[ks] + tm * 2048);
  };
  auto read_b = [&](int slot) {
    const char* base = lds + slot * kHalf;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const char* p = base + b_frag + ks * 8192 + i * 8;
        bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p));
        bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p + 1024));
        w[ks][i] = (bf16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
  };
  auto mma = [&](const bf16x8 (&x)[2][4], auto half) {
    constexpr int a = decltype(half)::value * 4;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int tm = 0; tm < 4; ++tm)
          acc[i][a + tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][i], x[ks][tm], acc[i][a + tm], 0, 0, 0);
  };
  auto slot_end = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto vm_traced = [&](auto n) {
    const uint64_t t0 = trace_now();
    wait_vm<decltype(n)::value>();
    if constexpr (kTrace) tr.ring += trace_now() - t0;
  };
  auto products = [&](const bf16x8 (&x)[2][4], auto half) {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's fragment reads are complete
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    mma(x, half);
    __builtin_amdgcn_s_setprio(0);
    slot_end();
  };

  // One stage.  LEFT: stages after it, counted up to 3; r: its ring slot.
  int r = 0;
  auto stage = [&](int it, auto left_) {
    constexpr int LEFT = decltype(left_)::value;
    const int r1 = r == 2 ? 0 : r + 1, r2 = r == 0 ? 2 : r - 1;  // (r + 1, r + 2) % 3
    if constexpr (LEFT >= 2) load_b(it + 2, r2);
    read_b(r);
    if constexpr (LEFT >= 3) {
      const int k = kbeg + (it + 3) * 64;
      if (Wait::kBlocks && wave == 0) wait.leader(k);
      wait.known(k);
    }
    vm_traced(int_constant<LEFT >= 2 ? 8 : LEFT == 1 ? 4 : 0>());  // A1 of this stage, A0 of the next
    slot_end();
    products(x0, int_constant<0>());

    if constexpr (LEFT >= 2) load_a(1, it + 2, r2);
    if constexpr (LEFT >= 3) load_a(0, it + 3, r);
    read_a(x1, 1, r);
    if constexpr (LEFT >= 1) {
      read_a(x0, 0, r1);
      vm_traced(int_constant<LEFT >= 3 ? 10 : LEFT == 2 ? 8 : 2>());  // B of the next stage
    }
    slot_end();
    products(x1, int_constant<1>());
    r = r1;
  };

  // Prologue: the first two stages, and A0 of the third.
  if constexpr (Wait::kBlocks) {  // the weights stream while the item waits for its rows
    load_b(0, 0);
    if (nk > 1) load_b(1, 1);
    if (wave == 0) {
      wait.leader(kbeg);
      if (nk > 1) wait.leader(kbeg + 64);
      if (nk > 2) wait.leader(kbeg + 128);
    }
    slot_end();
    load_a(0, 0, 0);
    load_a(1, 0, 0);
    if (nk > 1) {
      load_a(0, 1, 1);
      load_a(1, 1, 1);
    }
    if (nk > 2) load_a(0, 2, 2);
    wait_vm<0>();  // requested out of the stage order, so nothing less covers it
  } else {
    load_a(0, 0, 0);
    load_b(0, 0);
    load_a(1, 0, 0);
    if (nk > 1) {
      load_a(0, 1, 1);
      load_b(1, 1);
      load_a(1, 1, 1);
    }
    if (nk > 2) {
      load_a(0, 2, 2);
      wait_vm<10>();  // A0, B
    } else if (nk == 2) {
      wait_vm<8>();
    } else {
      wait_vm<2>();
    }
  }
  wait.known(kbeg);
  if (nk > 1) wait.known(kbeg + 64);
  if (nk > 2) wait.known(kbeg + 128);
  slot_end();
  read_a(x0, 0, 0);
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)

  if (trailing) slot_end();
  for (int it = 0; it < nk - 3; ++it) stage(it, int_constant<3>());
  if (nk > 2) stage(nk - 3, int_constant<2>());
  if (nk > 1) stage(nk - 2, int_constant<1>());
  stage(nk - 1, int_constant<0>());
  if (!trailing) slot_end();
  __syncthreads();  // every wave is done reading the ring before it is reused
}

template <class T, int NB, class Wait, class Check = NoCheck>
__device__ __forceinline__ void mainloop(const uint16_t* __restrict__ A, long lda, int m0, int mlast,
                                         const uint16_t* const (&Bp)[NB], const int (&n0)[NB], long ldb, int kbeg,
                                         int kend, f32x4 (&acc)[NB][T::TN][T::TM], char* lds, Wait& wait, TraceAcc& tr,
                                         Check check = Check()) {
  if constexpr (T::QUAD && NB * T::BN == 256 && is_same_type<Check, NoCheck>::value) {
    mainloop_quad<T, NB>(A, lda, m0, mlast, Bp, n0, ldb, kbeg, kend, acc, lds, wait, tr);
    return;
  }
  if constexpr (T::PAIR && NB == 1 && is_same_type<Check, NoCheck>::value) {
    mainloop_pair<T>(A, lda, m0, mlast, Bp[0], n0[0], ldb, kbeg, kend, acc[0], lds, wait, tr);
    return;
  }
  // The thread index passes through an empty asm, so the compiler derives
  // this call's per-lane offsets here instead of hoisting them out of the
  // persistent item loop: in the pipelined kernel, whose items take one of
  // two tile shapes, hoisted offsets of both shapes would stay live across
  // the whole kernel and push the mainloop's accumulators out of registers.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % T::WM;
  const int wn = wave / T::WM;

#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < T::TN; ++i)
#pragma unroll
      for (int j = 0; j < T::TM; ++j) acc[b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = (kend - kbeg) / T::BK;
  if (nk <= 0) return;

  const uint32_t lds_base = (uint32_t)(uintptr_t)lds;
  constexpr int SB = T::template stage_bytes<NB>();
  constexpr int PER_STAGE = T::template dma_per_stage<NB>();

  // DMA source offsets (bytes, relative to the tensor bases) at k = 0.
  uint32_t a_off[T::A_DMA];
#pragma unroll
  for (int j = 0; j < T::A_DMA; ++j) {
    const int ch = wave + T::NWAVES * j;  // 1 KB chunk = 8 rows of 128 B (4 of 256 B, 16 of 64 B)
    const int row = (1024 / T::ROW_BYTES) * ch + lane / T::CHUNKS;
    const int lc = (lane % T::CHUNKS) ^ swz_a<T::BK>(row);
    int gr = m0 + row;
    gr = gr > mlast ? mlast : gr;
    a_off[j] = (uint32_t)(((long)gr * lda + 8 * lc) * 2);
  }
  constexpr int CPR = T::BN / 8;      // 16-byte chunks per weight row
  constexpr int RPC = 64 / CPR;       // weight rows per 1 KB chunk
  uint32_t b_off[NB][T::B_DMA];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int j = 0; j < T::B_DMA; ++j) {
      const int ch = wave + T::NWAVES * j;
      const int row = RPC * ch + lane / CPR;
      const int lc = (lane % CPR) ^ swz_b<T::BN>(row);
      b_off[b][j] = (uint32_t)(((long)row * ldb + min(n0[b] + 8 * lc, (int)ldb - 8)) * 2);
    }

  // A stage's loads: the activation rows first (measured on the gated GEMM1
  // operand stream without math, 256 activation rows and two 128-column
  // weight stripes per stage: 216 -> 202 us), except while a GEMM2 item may
  // still have to wait for its activation rows: then the weights first, so
  // they stream during the wait.  The order is fixed per loop, not chosen
  // per stage: in the plain stage loop (every tile but the four-wave tiles
  // with three or more stages, below) an item that waits runs its stages
  // in the weights-first loop until its wait has seen every producer of its K
  // range complete, then in the activation-first loop (pipelined, with the
  // 256-row tiles in this loop, before they had one of their own: gated 396
  // -> 388 us, prefill 440 -> 421; a choice per stage inside one loop made the
  // one-launch kernels much slower: decode 74 -> 113 us).
  auto issue = [&](int st, auto weights_first) {
    const int k = kbeg + st * T::BK;
    const uint32_t sbase = lds_base + (uint32_t)((st % T::NS) * SB);
    auto weights = [&]() {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int j = 0; j < T::B_DMA; ++j) {
          const uint32_t dst = uniform(sbase + (uint32_t)(T::A_BYTES + b * T::B_BYTES + (wave + T::NWAVES * j) * 1024));
          if constexpr (T::WNT)
            dma16_nt(Bp[b], b_off[b][j] + (uint32_t)((long)k * ldb * 2), dst);
          else
            dma16(Bp[b], b_off[b][j] + (uint32_t)((long)k * ldb * 2), dst);
        }
    };
    auto activations = [&]() {
#pragma unroll
      for (int j = 0; j < T::A_DMA; ++j) {
        if constexpr (Check::kCoherentA)
          dma16_coherent(A, a_off[j] + (uint32_t)(k * 2), uniform(sbase + (uint32_t)((wave + T::NWAVES * j) * 1024)));
        else
          dma16(A, a_off[j] + (uint32_t)(k * 2), uniform(sbase + (uint32_t)((wave + T::NWAVES * j) * 1024)));
      }
    };
    if constexpr (decltype(weights_first)::value) {
      weights();
      wait(k);  // covers the stage's columns [k, k + BK)
      activations();
    } else {
      activations();
      wait(k);  // returns at once (takes the next ticket at the last stage)
      weights();
    }
  };
  using WaitFirst = bool_constant<Wait::kBlocks>;  // weights first where the item may wait
  using ActFirst = bool_constant<false>;

  // Fragment addressing (bytes inside a stage).
  //   activation (MFMA B operand): lane holds A[row = l%16][k = 8(l/16) .. +7]  -> ds_read_b128
  //   weight (MFMA A operand): ds_read_b64_tr_b16 over 4 rows x 4 chunks per 16-lane group;
  //     lane 4r+c of group g addresses row 8g+r (+4 for the upper half), columns 8c + 4*t2 .. +3,
  //     and receives column (8*(i/4) + 4*t2 + i%4) of those 4 rows, i = lane % 16.
  const int arow = T::row_of(wm, 0) + (lane & 15);
  int a_frag[T::BK / 32];  // K half ks: chunk 4 ks + lane / 16 of the row
#pragma unroll
  for (int ks = 0; ks < T::BK / 32; ++ks)
    a_frag[ks] = arow * T::ROW_BYTES + (((4 * ks + (lane >> 4)) ^ swz_a<T::BK>(arow)) << 4);
  const int g = lane >> 4, r4 = (lane & 15) >> 2, c4 = lane & 3;
  const int brow = 8 * g + r4;
  int b_frag[T::TN / 2];
#pragma unroll
  for (int tp = 0; tp < T::TN / 2; ++tp) {
    const int q = (T::col_of(wn, tp) >> 3) + c4;
    b_frag[tp] = T::A_BYTES + brow * (2 * T::BN) + ((q ^ swz_b<T::BN>(brow)) << 4);
  }

  // K slices of 32 per stage (BK / 32 of them).  With a two-stage ring every fragment of
  // the stage is read before its first product: the reads of the second
  // half and of the later column pairs then overlap the first products in
  // whatever code the mainloop is inlined into (the one-launch kernels' item
  // loop otherwise schedules one read pair ahead of its four products).
  // Deeper rings keep each half's reads next to its products.  Both orders
  // accumulate every output in the same sequence (first half, then second).
  auto weight_frag = [&](const char* base, int ks, int b, int i) {
    const char* p = base + b * T::B_BYTES + b_frag[i / 2] + ks * 32 * (2 * T::BN) + (i % 2) * 8;
    bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p));
    bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p + 4 * (2 * T::BN)));
    return (bf16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto act_frag = [&](const char* base, int ks, int tm) {
    return *reinterpret_cast<const bf16x8*>(base + a_frag[ks] + T::row_of(0, tm) * T::ROW_BYTES);
  };
  auto compute = [&](int st) {
    const char* base = lds + (st % T::NS) * SB;
    if constexpr (T::NS == 2) {
      bf16x8 xf[T::BK / 32][T::TM];
      bf16x8 wf[T::BK / 32][NB][T::TN];
#pragma unroll
      for (int ks = 0; ks < T::BK / 32; ++ks) {
#pragma unroll
        for (int tm = 0; tm < T::TM; ++tm) xf[ks][tm] = act_frag(base, ks, tm);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < T::TN; ++i) wf[ks][b][i] = weight_frag(base, ks, b, i);
      }
#pragma unroll
      for (int ks = 0; ks < T::BK / 32; ++ks)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < T::TN; ++i)
#pragma unroll
            for (int tm = 0; tm < T::TM; ++tm)
              acc[b][i][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][b][i], xf[ks][tm], acc[b][i][tm], 0, 0, 0);
    } else {
#pragma unroll
      for (int ks = 0; ks < T::BK / 32; ++ks) {
        bf16x8 xf[T::TM];
#pragma unroll
        for (int tm = 0; tm < T::TM; ++tm) xf[tm] = act_frag(base, ks, tm);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < T::TN; ++i) {
            const bf16x8 wf = weight_frag(base, ks, b, i);
#pragma unroll
            for (int tm = 0; tm < T::TM; ++tm)
              acc[b][i][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf[tm], acc[b][i][tm], 0, 0, 0);
          }
      }
    }
  };

  // Own loads of stage st complete (the stages issued after it may stay in
  // flight), then every wave's: the barrier also retires every wave's reads
  // of the stages before st.
  auto resident = [&](int st) {
    const uint64_t t0 = trace_now();
    wait_stages_behind<PER_STAGE, T::NS - 2>(min(T::NS - 2, nk - 1 - st));
    if constexpr (!is_same_type<Check, NoCheck>::value) {
      // The stage's activation pieces this wave loaded are in LDS: check them
      // (and reload any piece that still holds a sentinel) before the barrier
      // hands the stage to the other waves.
      const int k = kbeg + st * T::BK;
      const uint32_t sbase = lds_base + (uint32_t)((st % T::NS) * SB);
      check.template operator()<T>(A, a_off, k, sbase, lds + (st % T::NS) * SB, wave, lane);
    }
    __syncthreads();
    if constexpr (kTrace) tr.ring += trace_now() - t0;
  };

  // Prologue: NS - 1 stages in flight.
#pragma unroll
  for (int st = 0; st < T::NS - 1; ++st)
    if (st < nk) issue(st, WaitFirst());

  if constexpr (T::NWAVES == 4 && T::NS >= 3) {
    // One wave per SIMD: nothing else on the SIMD hides a stage's LDS read
    // latency, so the fragments of stage it + 1 are read into a second set
    // of registers while stage it is multiplied.  Stage it's slot is free
    // once every wave holds its fragments (the barrier of stage it + 1), and
    // takes the loads of stage it + NS.  Same products in the same order.
    struct Frags {
      bf16x8 x[T::BK / 32][T::TM];
      bf16x8 w[T::BK / 32][NB][T::TN];
    };
    auto read = [&](Frags& f, int st) {
      const char* base = lds + (st % T::NS) * SB;
#pragma unroll
      for (int ks = 0; ks < T::BK / 32; ++ks) {
#pragma unroll
        for (int tm = 0; tm < T::TM; ++tm) f.x[ks][tm] = act_frag(base, ks, tm);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < T::TN; ++i) f.w[ks][b][i] = weight_frag(base, ks, b, i);
      }
    };
    auto mma = [&](const Frags& f) {
#pragma unroll
      for (int ks = 0; ks < T::BK / 32; ++ks)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < T::TN; ++i)
#pragma unroll
            for (int tm = 0; tm < T::TM; ++tm)
              acc[b][i][tm] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[ks][b][i], f.x[ks][tm], acc[b][i][tm], 0, 0, 0);
    };
    // Stage it is multiplied while stage it + 1 (< nk) is read.
    auto advance = [&](int it, Frags& cur, Frags& nxt, auto order) {
      resident(it + 1);
      if (it + T::NS < nk) issue(it + T::NS, order);
      read(nxt, it + 1);
      mma(cur);
    };
    resident(0);
    if (T::NS - 1 < nk) issue(T::NS - 1, WaitFirst());
    Frags fa, fb;
    read(fa, 0);
    // Two stages per trip, the fragment sets swapping roles; every trip reads
    // a next stage, so both sets keep their registers (no conditional read
    // merges into the products' control flow).
    // (One loop: a waiting item keeps the weights-first order throughout; a
    // second, activation-first loop after the item's producers were all seen
    // complete made these kernels slower: decode 76 -> 88 us.)
    int it = 0;
    for (; it + 2 < nk; it += 2) {
      advance(it, fa, fb, WaitFirst());
      advance(it + 1, fb, fa, WaitFirst());
    }
    if (it + 1 < nk) {  // two stages left
      advance(it, fa, fb, WaitFirst());
      mma(fb);
    } else {            // one stage left
      mma(fa);
    }
    __syncthreads();  // every wave is done reading the ring before it is reused
    return;
  }

  int it = 0;
  if constexpr (Wait::kBlocks) {
    for (; it < nk && !wait.all_known(); ++it) {
      resident(it);
      if (it + T::NS - 1 < nk) issue(it + T::NS - 1, WaitFirst());
      compute(it);
    }
  }
  for (; it < nk; ++it) {
    resident(it);
    if (it + T::NS - 1 < nk) issue(it + T::NS - 1, ActFirst());
    compute(it);
  }
  __syncthreads();  // every wave is done reading the ring before it is reused
}

// The sentinel mode's stage check (the consumer side of Sec. V-A): each wave
// reads back the activation pieces it loaded for the stage (16 bytes per lane
// per 1 KB piece), and reloads a piece, at device scope, while any lane still
// sees a sentinel element in it, sleeping between tries.  After spin_limit
// tries, or once another wait gave up, it latches CTRL_ERROR (bit 2) and
// stops; the kernel still exits and mlp2_check reports the timeout.
struct SentinelCheck {
  static constexpr bool kCoherentA = true;
  uint32_t* err;  // CTRL_ERROR word
  uint32_t spin_limit;
  TraceAcc* tr;   // re-read time is counted as flag-wait time (trace builds)
  template <class T>
  __device__ __forceinline__ void operator()(const uint16_t* A, const uint32_t (&a_off)[T::A_DMA], int k,
                                             uint32_t sbase, const char* stage, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < T::A_DMA; ++j) {
      const int piece = (wave + T::NWAVES * j) * 1024;
      const uint64_t t0 = trace_now();
      for (uint32_t tries = 0;; ++tries) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(stage + piece + 16 * lane);
        if (__builtin_amdgcn_ballot_w64(has_sentinel(v)) == 0) {  // the same in every lane
          if constexpr (kTrace) {
            if (tries) tr->flag += trace_now() - t0;
          }
          break;
        }
        if (tries >= spin_limit || ((tries & 63u) == 63u && uniform(ld_relaxed(err)) != 0u)) {
          if (lane == 0) __hip_atomic_fetch_or(err, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(2);
        dma16_coherent(A, a_off[j] + (uint32_t)(k * 2), uniform(sbase + (uint32_t)piece));
        wait_vm<0>();
      }
    }
  }
};

// ------------------------------------------------------------------ fragment <-> tile coordinates

// Output coordinates held by this lane for block pair tp and row block tm.
template <class T>
struct FragPos {
  int row0, col0, block0;
  __device__ FragPos(int m0, int n0) {
    const int tid = thread_here(), lane = tid & 63, wave = uniform(tid >> 6);
    row0 = m0 + T::row_of(wave % T::WM, 0) + (lane & 15);
    block0 = n0 + T::col_of(wave / T::WM, 0);
    col0 = block0 + 8 * (lane >> 4);
  }
  __device__ int row(int tm) const { return row0 + T::row_of(0, tm); }
  __device__ int col(int tp) const { return col0 + T::col_of(0, tp); }
  // first of the wave's 32 columns of block pair tp, a scalar
  __device__ int block(int tp) const { return block0 + T::col_of(0, tp); }
};

template <class T>
__device__ __forceinline__ void pair_values(const f32x4 (&a)[T::TN][T::TM], int tp, int tm, float (&v)[8]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    v[r] = a[2 * tp][tm][r];
    v[4 + r] = a[2 * tp + 1][tm][r];
  }
}

// ------------------------------------------------------------------ split-K partials
//
// With split-K, a tile's K range is cut into S parts computed by separate
// work items.  Each part stores its fp32 accumulators "fragment-native": lane
// l of wave w writes its f32x4 of block i at ((tile*S + s)*PER_ITEM +
// (w*PER_WAVE + i)*64 + l), so writes and reads are fully coalesced 1 KB runs.
// Each part then counts its arrival on the tile's counter; the part that
// arrives last (it reads the count just below the run's target) adds up the
// tile in "units" (a wave's pair of adjacent 16x16 blocks in one row block,
// for every weight operand) in the fixed order s = 0, 1, ..., S-1 and runs the
// tile's epilogue; the other parts go straight on to their next item.  No part
// ever waits for a sibling, and the order of the adds never depends on which
// part finished last, so every run and mode gives the same bits.

template <class T, int NB>
struct Partial {
  static constexpr int PER_WAVE = NB * T::TN * T::TM;  // f32x4 per lane
  static constexpr long PER_ITEM = (long)T::NWAVES * PER_WAVE * 64;  // f32x4 per (tile, split)
  static constexpr int UNITS = T::NWAVES * T::TM * (T::TN / 2); // (wave, tm, tp) triples per tile
  __device__ static long block_index(long tile, int S, int s, int w, int b, int tn, int tm) {
    return (tile * S + s) * PER_ITEM + ((long)w * PER_WAVE + ((b * T::TN + tn) * T::TM + tm)) * 64;
  }
};

template <class T, int NB>
__device__ __forceinline__ void store_partial(float* base, long tile, int S, int s, const f32x4 (&acc)[NB][T::TN][T::TM]) {
  float* item = base + Partial<T, NB>::block_index(tile, S, s, 0, 0, 0, 0) * 4;
  const uint32_t tid = (uint32_t)thread_here();
  const uint32_t off = ((tid >> 6) * Partial<T, NB>::PER_WAVE * 64 + (tid & 63)) * 16;
  int i = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int tn = 0; tn < T::TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < T::TM; ++tm, ++i) store_through16(item, off, __builtin_bit_cast(u32x4, acc[b][tn][tm]), i * 1024);
}

// A reduction unit: wave w's blocks (2 tp, tm) and (2 tp + 1, tm).
template <class T>
struct Unit {
  int w, tm, tp;
  __device__ Unit() = default;
  __device__ explicit Unit(int u) {
    constexpr int per_wave = T::TM * (T::TN / 2);
    w = u / per_wave;
    const int r = u - w * per_wave;
    tm = r / (T::TN / 2);
    tp = r - tm * (T::TN / 2);
  }
  // Output row and first of the 8 consecutive columns held by `lane` of this unit.
  __device__ int row(int m0, int lane) const { return m0 + T::row_of(w % T::WM, tm) + (lane & 15); }
  __device__ int block(int n0) const { return n0 + T::col_of(w / T::WM, tp); }  // the unit's first column
  __device__ int col(int n0, int lane) const { return block(n0) + 8 * (lane >> 4); }
};

// v[g][b][0..7] = sum over s = 0 .. S-1 (in that order) of the 8 values of
// unit ug[g] for weight operand b, as held by `lane` (the layout pair_values
// produces).  G units at a time and R parts per round keep 2*G*NB*R loads of
// one wave in flight together; slots past the last part load part S - 1
// again (in bounds) and are not added.
template <class T, int NB, int G, int R>
__device__ __forceinline__ void reduce_units(const float* base, long tile, int S, const Unit<T> (&ug)[G], int lane,
                                             float (&v)[G][NB][8]) {
  const f32x4* p = reinterpret_cast<const f32x4*>(base);
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 8; ++i) v[g][b][i] = 0.f;
  for (int s = 0; s < S; s += R) {
    f32x4 q[R][G][NB][2];
#pragma unroll
    for (int h = 0; h < R; ++h) {
      const int sh = min(s + h, S - 1);
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int t2 = 0; t2 < 2; ++t2)
            q[h][g][b][t2] = p[Partial<T, NB>::block_index(tile, S, sh, ug[g].w, b, 2 * ug[g].tp + t2, ug[g].tm) + lane];
    }
#pragma unroll
    for (int h = 0; h < R; ++h) {
      if (s + h >= S) break;  // uniform
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[g][b][r] += q[h][g][b][0][r];
            v[g][b][4 + r] += q[h][g][b][1][r];
          }
    }
  }
}

// The parts a round loads: no more than the tile has, up to 8 (two parts in
// rounds of eight read part 1 seven times: 2048 x 4096 x 14336 in the workqueue
// mode, when the last part to arrive still summed the 512 KB of a tile alone,
// 433 -> 390 us).  `f` is called with the count as a constant.
template <class F>
__device__ __forceinline__ void with_round(int S, F&& f) {
  if (S <= 2) f(int_constant<2>());
  else if (S <= 4) f(int_constant<4>());
  else f(int_constant<8>());
}

// Increment of a counter after every wave's stores through to the point of
// coherence are acknowledged (used for split-K arrivals and for the producer's
// ready signal): the stores are visible to the device before the count is.
// Against an agent-scope release per increment and acquire-release exits
// (pipelined mode): 1 x 4096 x 14336 gated 109 -> 82 us, 32 x 8192 x 3584
// 51 -> 40, 128 x 4096 x 14336 92 -> 77, 64 x 512 x 2048 14.1 -> 12.1, a
// chain of four 8192 x 8192 at 128 rows 222 -> 195.
__device__ __forceinline__ void release_add(uint32_t* cnt) {
  wait_vm<0>();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A split-K part's arrival: store the partial, then one increment of the
// tile's counter (after every wave's stores are acknowledged).
// Returns true (uniformly) on the part that arrives last in this run, i.e.
// that reads `target - 1`; that part then reads the others' partials after a
// barrier and a work-group-scope acquire.  No agent-scope acquire is needed,
// for the reason given for Z with the ready waits below: each tile's
// partials (whole 1 KB runs, never sharing a line with another tile's) are
// read once per launch, only by the completing part, after every part has
// stored them through.
template <class T, int NB>
__device__ __forceinline__ bool arrive_split(float* part, uint32_t* cnt, long tile, int S, int s, uint32_t target,
                                             const f32x4 (&acc)[NB][T::TN][T::TM], int* s_slot, TraceAcc& tr) {
  store_partial<T, NB>(part, tile, S, s, acc);
  wait_vm<0>();
  __syncthreads();
  if constexpr (kTrace) tr.t_rel = trace_now();
  if (threadIdx.x == 0) {
    const uint32_t old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_slot = old == target - 1u;
  }
  __syncthreads();
  const bool last = uniform(*s_slot) != 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  __syncthreads();  // *s_slot may be rewritten
  if constexpr (kTrace) tr.t_wait = trace_now();
  return last;
}

// ------------------------------------------------------------------ claiming items

// The next item of a persistent work-group.  Claim list l = blockIdx % lists
// hands out the ranks l, l + lists, l + 2 lists, ... in increasing order: the
// first `skip` of them without a ticket (first items of the list's
// work-groups below Args::first_static), the rest through the list's ticket
// word.  Taking a ticket is a device-scope
// atomic whose result comes back from the memory side after a long round
// trip, so `issue` sends it as early as the protocol allows (thread 0 keeps
// the ticket in a register while the item runs) and `park` writes the rank
// to LDS at the end of the item, where the next iteration reads it after a
// barrier.  Every item calls `issue` exactly once, then `park`.
struct Claim {
  uint32_t* ticket;
  int base, stride, skip;
  uint32_t t;
  __device__ __forceinline__ void issue() {
    if (threadIdx.x == 0) t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void park(int* s_next) const {
    if (threadIdx.x == 0) *s_next = base + stride * ((int)t + skip);
  }
};

// The mainloop hook of every item: the item's own wait for the stage at K
// offset k (if any), then, when the loads of the item's last stage are
// issued, the ticket for the work-group's next item.  The last stage's wait
// is the item's last wait, so the claim never precedes a wait of its item.
// The atomic's round trip overlaps the last stages and the epilogue, while
// the choice of the next item is still made late: a work-group that
// committed to its next item a whole item ahead would keep it from a
// work-group that frees up sooner, and lengthen the launch's tail.
struct NoWait {
  static constexpr bool kBlocks = false;  // never waits
  __device__ __forceinline__ bool all_known() const { return true; }
  __device__ __forceinline__ void leader(int) {}
  __device__ __forceinline__ void operator()(int) {}
};

template <class Wait, class C = Claim>
struct ClaimAtLastStage {
  static constexpr bool kBlocks = Wait::kBlocks;
  Wait& wait;
  C* next;
  int k_last;  // K offset of the item's last stage
  __device__ __forceinline__ bool all_known() const { return wait.all_known(); }
  __device__ __forceinline__ void operator()(int k) {
    wait(k);
    known(k);
  }
  // The wait by wave 0 alone (ReadyWait::leader), and the claim.
  __device__ __forceinline__ void leader(int k) { wait.leader(k); }
  __device__ __forceinline__ void known(int k) {
    if (k == k_last) next->issue();
  }
};

// The claim of an item whose successor comes from somewhere else (a
// workqueue consumer pops its next unit after the item).
struct NoClaim {
  __device__ __forceinline__ void issue() {}
  __device__ __forceinline__ void park(int*) const {}
};

// ------------------------------------------------------------------ ready flags

// Producer side (Sec. III-A: the producer fences its output, then signals):
// every wave's Z stores are through to the point of coherence, then one lane
// increments the tile's ready counter.
__device__ __forceinline__ void signal_ready(uint32_t* flag) { release_add(flag); }

// Consumer side: before loading Z columns [k, k + span) of row block mb (one
// stage), every GEMM1 tile (mb, kb) whose columns they overlap must have
// signalled in this run (once per tile and run), i.e. its counter must have
// reached epoch + 1 (compared wrap-safe).  A stage deeper than a GEMM1 tile
// is wide (128-deep stages over 64-column tiles) can need two tiles; the
// wait then repeats from the first tile still unknown.
//
// Wave 0 polls the first counter it needs; once that is ready it reads up to
// 64 consecutive counters of the item's K range in one vector load and takes
// the longest ready prefix (a ballot).  Between polls the wave sleeps; after
// spin_limit polls it gives up, latches CTRL_ERROR and stops waiting for the
// rest of the run.  The result reaches the other waves
// through LDS and a work-group barrier.  Every call is made by all waves with
// the same k.
//
// Visibility of Z.  The producer's Z lines are stored through its XCD's L2,
// and acknowledged, before the counter moves.  The consumer needs no
// agent-scope acquire (on this chip an invalidation of its XCD's whole L2,
// which throws away the lines every other work-group of the XCD is
// streaming, and measured several percent of a run where consumers wait
// often): a cache can only return a stale Z line if it already held that
// line, and none can.  Every launch starts with the caches invalidated, and
// within a launch a line of Z (128 bytes of one row in one 64-column block;
// rows and blocks are 128-byte aligned) is read only after the counter of
// the tile that writes it has been seen complete, by the work-group whose
// wait returned or by another that waited for it the same way.  The
// observing load is an atomic, so it reads the counter at the device's
// point of coherence; the Z loads are issued after it, in program order,
// and a work-group-scope acquire orders them for the compiler.
struct ReadyWait {
  static constexpr bool kBlocks = true;  // waits on ready counters before the activation loads
  const uint32_t* ready;
  uint32_t* err;  // CTRL_ERROR word
  int mb, Mb, bn1;
  int kb_last;    // last column block of this item's K range
  uint32_t target;
  uint32_t spin_limit;
  int* s_known;   // LDS broadcast slot
  int k_ready;    // K offsets below this are in column blocks this work-group has acquired (uniform)
  TraceAcc* tr;
  int span;       // K depth of one stage
  // Every producer of the item's K range was seen complete (uniform).
  __device__ __forceinline__ bool all_known() const { return k_ready == 0x7fffffff; }
  __device__ __forceinline__ void operator()(int k) {
    const int k_hi = k + span - 1;  // the stage's last column
    if (k_hi < k_ready) return;     // one compare per stage; the division below only on a miss
    const uint64_t t0 = trace_now();
    // Each round acquires at least the first unknown column block, or gives up
    // (k_ready then covers everything), so the loop ends.
    do acquire((k > k_ready ? k : k_ready) / bn1);
    while (k_hi >= k_ready);
    if constexpr (kTrace) tr->flag += trace_now() - t0;
  }
  // For a loop whose barriers already order the waves: wave 0 alone calls
  // this before a barrier that every wave passes before it requests the
  // stage's activation rows.  The barrier tells the others; k_ready is then
  // wave 0's own.
  __device__ __forceinline__ void leader(int k) {
    const int k_hi = k + span - 1;
    if (k_hi < k_ready) return;
    const uint64_t t0 = trace_now();
    do {
      const int hi = poll((k > k_ready ? k : k_ready) / bn1);
      k_ready = hi < 0 || hi >= kb_last ? 0x7fffffff : (hi + 1) * bn1;
    } while (k_hi >= k_ready);
    if constexpr (kTrace) tr->flag += trace_now() - t0;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
  // One poll-and-gather round from column block kb, by one wave: the last
  // block of the ready prefix, or -1 when the wait gave up.
  __device__ __forceinline__ int poll(int kb) const {
    const int lane = threadIdx.x & 63;
    const int j = kb + lane;
    int hi = -1;
    if (uniform(ld_relaxed(err)) == 0u) {
      // Poll the first counter needed, every lane at the same address (one
      // request per poll: a long wait must not flood the memory side that
      // the running producers stream from); scalar loop, uniform exits.
      const uint32_t* first = ready + ((long)kb * Mb + mb) * kLine;
      uint64_t m = 0;
      for (uint32_t polls = 0;; ++polls) {
        const uint32_t v = ld_relaxed(first);
        m = __builtin_amdgcn_ballot_w64((int32_t)(v - target) >= 0);
        if ((m & 1u) || polls >= spin_limit) break;
        __builtin_amdgcn_s_sleep(2);
      }
      if (m & 1u) {
        // then the longest ready prefix of up to 64 counters in one gather
        // (counters only grow during a run, so the first is still ready)
        const uint32_t v = ld_relaxed(ready + ((long)(j <= kb_last ? j : kb_last) * Mb + mb) * kLine);
        m = __builtin_amdgcn_ballot_w64((j <= kb_last) & ((int32_t)(v - target) >= 0));
        // ~m == 0 (all 64 ready) must be taken apart: a count of trailing
        // zeros of 0 is undefined, and the scalar find-first-one the
        // compiler emits for it returns -1.
        hi = ~m ? kb + (int)__builtin_ctzll(~m) - 1 : kb + 63;
      } else if (lane == 0) {
        __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    return hi;
  }
  // The round for every wave: wave 0 polls and broadcasts; updates k_ready.
  __device__ __forceinline__ void acquire(int kb) {
    if (uniform((int)(threadIdx.x >> 6)) == 0) {  // wave 0, as a scalar branch
      const int hi = poll(kb);
      if ((threadIdx.x & 63) == 0) *s_known = hi >= 0 ? hi : 0x7fffffff;
    }
    __syncthreads();
    const int known = uniform(*s_known);
    k_ready = known >= kb_last ? 0x7fffffff : (known + 1) * bn1;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    // Every wave has read *s_known before wave 0 may write it again: the
    // pipeline prologue calls this back to back, with no other barrier between.
    __syncthreads();
  }
};

// ------------------------------------------------------------------ workqueue mode
//
// The paper's own consumer scheduling (Sec. III-A.2-3): a scoreboard per
// consumer unit counts its finished producers, and the producer that
// completes a unit's count pushes the unit onto a ring-buffer workqueue from
// which consumer work-groups pop whole units.  Here a unit is a GEMM2 item
// (tile, split-K part) and its producers are the GEMM1 tiles of its row
// block whose Z columns overlap its K range (a closed form, so no dependency
// array is stored).  Counts only grow, and only in workqueue runs: with w
// the number of earlier workqueue runs (CTRL_EPOCH_WQ), a unit with n
// producers reaches (w + 1) * n in this run.  (The producers also signal
// their ready counters, which thus advance once per run in every mode.)  A
// queue entry carries the low 8 bits of w + 1 above the unit id, so a
// consumer never takes a slot filled by an earlier run (every slot below
// the run's unit count is rewritten in every workqueue run).  Every unit has at least one producer (the plan
// makes S2 = ceil(F / kc2) parts, none of them empty), so every unit is
// pushed exactly once per run.

__device__ __forceinline__ uint32_t queue_tag(uint32_t wq_epoch) { return ((wq_epoch + 1u) & 0xffu) << 24; }

// Producer side: every wave's Z stores of the tile are through to the point of
// coherence, then wave 0 increments the scoreboard of each unit that reads the
// tile, one unit per lane.  The units whose count this completes are pushed together:
// lane 0 reserves as many queue slots as the ballot has bits with one atomic
// (a tile that completes a whole split's units would otherwise pay one
// round trip per unit, one after the other), and each completing lane
// publishes its unit in its slot.  The queue has one spare slot
// past the run's unit count; a reservation beyond it (impossible: each unit
// completes once per run) would land there, no consumer reads it, and the
// unit's consumer would time out and report the error.
__device__ __forceinline__ void push_ready(const Args& a, int tile, uint32_t wq_epoch) {
  wait_vm<0>();
  __syncthreads();
  if (uniform((int)(threadIdx.x >> 6)) == 0) {  // wave 0, as a scalar branch
    const int lane = threadIdx.x & 63;
    const int mb = tile % a.Mb, kb = tile / a.Mb;
    const int k0 = kb * a.bn1, k1 = min(a.F, k0 + a.bn1) - 1;  // the tile's Z columns
    const int s_lo = k0 / a.kc2, s_hi = k1 / a.kc2;            // the K ranges they fall in
    const int units = a.Nb2 * (s_hi - s_lo + 1);
    for (int i0 = 0; i0 < units; i0 += 64) {  // uniform trip count; one unit per lane
      const int i = i0 + lane;
      int q = 0;
      bool complete = false;
      if (i < units) {
        const int s = s_lo + i / a.Nb2, nb2 = i % a.Nb2;
        q = (nb2 * a.Mb + mb) * a.S2 + s;
        const int kbeg = s * a.kc2, kend = min(a.F, kbeg + a.kc2);
        const uint32_t n = (uint32_t)((kend - 1) / a.bn1 - kbeg / a.bn1 + 1);
        const uint32_t old =
            __hip_atomic_fetch_add(a.board + (long)q * kLine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        complete = old + 1u == (wq_epoch + 1u) * n;
      }
      const uint64_t m = __builtin_amdgcn_ballot_w64(complete);
      if (m) {  // a scalar branch: m is the same in every lane
        uint32_t base = 0;
        if (lane == 0)
          base = __hip_atomic_fetch_add(a.ctrl + CTRL_QTAIL, (uint32_t)__builtin_popcountll(m), __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
        base = uniform(base);
        if (complete) {
          const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          __hip_atomic_store(a.queue + min(base + below, (uint32_t)a.items2), queue_tag(wq_epoch) | (uint32_t)q,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
  }
}

// Consumer side: wave 0 claims the next queue slot of the work-group's claim
// list (list l of L has slots l, l + L, ...: hundreds of work-groups claiming
// at once from one word took turns for microseconds) and polls it (every lane
// at the same address, a scalar loop with uniform exits) until a producer of
// this run has filled it, sleeping between polls; after spin_limit polls, or
// once another wait gave up, it latches CTRL_ERROR and returns no unit.
// Returns the unit for every wave; past the run's units, items2 + r for
// reduction item r (nothing to wait for here: it waits for its tile's parts
// itself); or -1 once all are claimed.  Z visibility follows the ready counters' argument: every
// producer of the unit stored its Z lines through before its increment, the
// completing increment had returned before the entry was stored, and no L2
// holds a Z line before a consumer has seen its producers complete.
__device__ __forceinline__ int pop_ready(const Args& a, uint32_t wq_epoch, int* s_bcast) {
  if (uniform((int)(threadIdx.x >> 6)) == 0) {  // wave 0, as a scalar branch
    const int lane = threadIdx.x & 63;
    uint32_t h = 0;
    const uint32_t lists = (uint32_t)a.lists, l = (uint32_t)blockIdx.x % lists;
    if (lane == 0)
      h = __hip_atomic_fetch_add(a.ctrl + CTRL_QHEAD + l * kLine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    h = l + lists * uniform(h);
    int q = -1;
    if (h < (uint32_t)a.items2) {
      const uint32_t want = uniform(queue_tag(wq_epoch));
      for (uint32_t polls = 0;; ++polls) {
        const uint32_t v = uniform(ld_relaxed(a.queue + h));
        if ((v & 0xff000000u) == want) {
          q = (int)(v & 0x00ffffffu);
          if (q >= a.items2) {  // not an entry any producer writes: give up loudly
            if (lane == 0) __hip_atomic_fetch_or(a.ctrl + CTRL_ERROR, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            q = -1;
          }
          break;
        }
        if (polls >= a.spin_limit || ((polls & 63u) == 63u && uniform(ld_relaxed(a.ctrl + CTRL_ERROR)) != 0u)) {
          if (lane == 0) __hip_atomic_fetch_or(a.ctrl + CTRL_ERROR, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
    } else if (h < (uint32_t)(a.items2 + a.items_red)) {
      q = (int)h;
    }
    if (lane == 0) *s_bcast = q;
  }
  // No load of the item before is in flight here, and the compiler is told so:
  // the sums load parts that they may not need, and for the registers of such
  // a load it otherwise keeps a wait in every stage of the next unit's
  // mainloop, which drains the ring (2048 x 4096 x 14336: 428 -> 376 us).
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __syncthreads();
  const int q = uniform(*s_bcast);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  __syncthreads();  // every wave has read the slot before wave 0 writes it again
  return q;
}

}  // namespace mlp2
