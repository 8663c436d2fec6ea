// Step 4: grouped SwiGLU expert FFN over the local slots (App. A), forward,
// input gradient and weight gradient.
//
// bf16 path: persistent workgroups of 8 wavefronts (4 for 128-wide weight
// gradient tiles) walk a tile list built on the device from the slot offsets
// (no host sync). Operand tiles stream from
// HBM straight into LDS with range-checked buffer loads (buffer_load ... lds:
// no staging registers; rows outside the current slot read as zero and no
// load can leave its operand) through a ring of LDS stages, and are
// multiplied with v_mfma_f32_32x32x16_bf16 (fp32 accumulation). Operands
// that are contiguous along K are read with ds_read_b128; operands contiguous
// along M/N (the weights in dgrad, both operands of wgrad) stay in their
// memory layout in LDS and are read with the gfx950 transpose read
// ds_read_b64_tr_b16. The SwiGLU activation and its derivative are fused into
// the epilogues.
//
// f32 path: ffn_f32.hip.
#include <climits>
#include <type_traits>

#include "common.h"
#include "ffn_f32.h"
#include "row_units.h"

namespace foremoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Tile configurations (overridable at build time for tuning sweeps).
#ifndef FM_ROWS_NS
#define FM_ROWS_NS 2
#endif
#ifndef FM_ROWS_WGM
#define FM_ROWS_WGM 4
#endif
#ifndef FM_ROWS_WGN
#define FM_ROWS_WGN 2
#endif
#ifndef FM_WG_BK
#define FM_WG_BK 64
#endif
#ifndef FM_WG_NS
#define FM_WG_NS 2
#endif
#ifndef FM_WG_WGM
#define FM_WG_WGM 2
#endif
#ifndef FM_WG_WGN
#define FM_WG_WGN 4
#endif
// k-steps over which one stage's loads are spread (capped at the k-steps of a stage)
#ifndef FM_LOAD_SPREAD
#define FM_LOAD_SPREAD 2
#endif
// Wave priority while a k-step's MFMAs issue (0: leave it): the wave that
// is multiplying wins the SIMD's issue arbitration over the other wave on
// that SIMD, whose reads and loads then fill the gaps.
#ifndef FM_SETPRIO
#define FM_SETPRIO 1
#endif

enum Epi { kEpiStore = 0, kEpiSwigluFwd = 1, kEpiSwigluBwd = 2 };

// SiLU a / D and sigmoid 1 / D with D = 1 + exp(-a), correctly rounded in fp32.
// The hardware reciprocal alone is 1 ulp off; one Newton step on it (on the
// quotient) gives the division's bits for every fp32 number a where neither
// D nor |a| reaches 2^126 (all of them were compared), in a third of its
// instructions. Beyond, where the reciprocal flushes its subnormal result (a
// below -87.3, with SiLU near 1e-37 in bf16) or the step has infinities, the
// division itself; one check for the N values of every lane. Down input
// gradient of 8 slots of 512 rows (d = 1024, F = 512), us: reciprocal alone
// 20.9, this 21.2, divisions 22.7; Qwen3 share's gate/up forward 115.2 / 117.2
// / 119.8.
constexpr float kDivideFrom = 0x1p126f;

template <int N>
__device__ __forceinline__ void silu_n(const float* a, float* s) {
  float D[N], m = 0.f;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    D[e] = 1.0f + __expf(-a[e]);
    m = fmaxf(m, fmaxf(D[e], fabsf(a[e])));
    const float r = __builtin_amdgcn_rcpf(D[e]), q = a[e] * r;
    s[e] = copysignf(fmaf(fmaf(-q, D[e], a[e]), r, q), a[e]);  // (a zero's sign)
  }
  if (__builtin_expect(__ballot(m >= kDivideFrom) != 0, 0)) {
#pragma unroll
    for (int e = 0; e < N; ++e) s[e] = a[e] / D[e];
  }
}
template <int N>
__device__ __forceinline__ void sigmoid_n(const float* a, float* s) {
  float D[N], m = 0.f;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    D[e] = 1.0f + __expf(-a[e]);
    m = fmaxf(m, D[e]);
    const float r = __builtin_amdgcn_rcpf(D[e]);
    s[e] = fmaf(fmaf(-D[e], r, 1.0f), r, r);
  }
  if (__builtin_expect(__ballot(m >= kDivideFrom) != 0, 0)) {
#pragma unroll
    for (int e = 0; e < N; ++e) s[e] = 1.0f / D[e];
  }
}

__device__ __forceinline__ int lane64() { return threadIdx.x & 63; }
// The same, recomputed where it stands: a kernel with several tile shapes in
// one loop would otherwise keep the lane offsets of all of them in registers
// across the loop (and spill).
__device__ __forceinline__ int lane64_here() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Virtual workgroup id: workgroups are dispatched round-robin over the 8 XCDs,
// so give the workgroups of one XCD consecutive ids (they then share tiles
// that reuse the same operand rows in that XCD's L2).
#ifndef FM_XCD_MAP
#define FM_XCD_MAP 1
#endif
__device__ __forceinline__ int xcd_virtual_id() {
  const int b = blockIdx.x, n = gridDim.x;
  if (!FM_XCD_MAP || n % 8 != 0) return b;
  return (b % 8) * (n / 8) + b / 8;
}

// ---------------------------------------------------------------------------
// Range-checked buffer loads straight into LDS
// ---------------------------------------------------------------------------
// A buffer resource over [base, base + bytes): a load at an offset >= bytes
// returns zeros, so ragged tile edges read as zero and no load can leave the
// operand.
__device__ __forceinline__ i32x4 buf_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)base;
  i32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r.y = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xFFFFu));
  r.z = __builtin_amdgcn_readfirstlane((int)bytes);
  r.w = 0x00020000;
  return r;
}

// One wavefront moves 64 x 16 bytes: lane l's bytes land at LDS address
// lds_wave_base + 16 l. The load is issued asynchronously; completion is
// awaited with wait_vm() before the workgroup barrier that publishes it.
__device__ __forceinline__ void dma16(i32x4 rs, uint32_t lds_wave_base, uint32_t voff) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_wave_base);
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(m0v), "v"(voff), "s"(rs)
               : "memory");
}

// The same with lane offset voff0 + soff (soff wave-uniform): the add sits
// in the asm so that one temporary serves every load instead of one
// precomputed offset register per load.
__device__ __forceinline__ void dma16s(i32x4 rs, uint32_t lds_wave_base, uint32_t voff0, uint32_t soff) {
  const uint32_t m0v = __builtin_amdgcn_readfirstlane(lds_wave_base);
  uint32_t t;
  asm volatile(
      "v_add_u32 %0, %1, %2\n\ts_mov_b32 m0, %3\n\tbuffer_load_dwordx4 %0, %4, 0 offen lds"
      : "=&v"(t)
      : "s"(soff), "v"(voff0), "s"(m0v), "s"(rs)
      : "memory");
}

// Wait until at most N vector-memory operations of this wavefront are in flight.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(uintptr_t)p; }

// ---------------------------------------------------------------------------
// LDS operand tiles. A "K-major" tile keeps ROWS rows (m or n) of BK
// contiguous k values; a "MN-major" tile keeps BK rows (k) of ROWS contiguous
// m or n values. Both are filled by dma16 and XOR-swizzled in 16-byte chunks
// so that the MFMA fragment reads hit 16 (or 32) different LDS bank groups of
// gfx950's 64 banks.
// ---------------------------------------------------------------------------
template <int ROWS, int BK, int NW>
struct KTile {
  static constexpr int CPR = BK / 8;     // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;   // rows per wavefront load
  static constexpr int NI = ROWS / RPI;  // wavefront loads per tile
  static constexpr int PER_WAVE = NI / NW;
  static constexpr int BYTES = ROWS * BK * 2;
  static_assert(NI % NW == 0, "tile must split over the wavefronts");
  __device__ __forceinline__ static int swz(int r) {
    if constexpr (CPR == 8) return (r >> 1) & 7;
    else return (r >> 2) & 3;
  }
  // This lane's source offset in load i (0 <= i < PER_WAVE) of this
  // wavefront's share of the tile, relative to the stage's first k; rowoff(r)
  // is the byte offset of tile row r. Fixed for a whole tile: each stage
  // moves the buffer resource instead.
  template <class RowOff>
  __device__ __forceinline__ static uint32_t voff(int l, RowOff rowoff, int i) {
    const int w = wave_id();
    const int r = (w + NW * i) * RPI + l / CPR;
    const int c = (l % CPR) ^ swz(r);
    return rowoff(r) + (uint32_t)c * 16u;
  }
  __device__ __forceinline__ static void issue(i32x4 rs, uint32_t lds, uint32_t voff, int i) {
    dma16(rs, lds + (wave_id() + NW * i) * 1024, voff);
  }
  // load i with lane offset voff(0) + soff_i, soff_i = voff(i) - voff(0) (the
  // same for every lane: the swizzle of a row or k row does not change by i)
  __device__ __forceinline__ static void issue_s(i32x4 rs, uint32_t lds, uint32_t voff0, uint32_t soff, int i) {
    dma16s(rs, lds + (wave_id() + NW * i) * 1024, voff0, soff);
  }
  // MFMA operand for rows mn0..mn0+31 of the tile, k-step kk (16 k values):
  // lane l gets row mn0 + l % 32, k = 16 kk + 8 (l / 32) + 0..7. The swizzle
  // only depends on l % 32 (mn0 is a multiple of 32), so the address splits
  // into a per-block lane offset and a per-k-step lane offset.
  __device__ __forceinline__ static uint32_t lane_off(int l, int mn0) {
    return (uint32_t)(mn0 + (l & 31)) * (BK * 2);
  }
  __device__ __forceinline__ static uint32_t kstep_off(int l, int kk) {
    return (uint32_t)(((2 * kk + (l >> 5)) ^ swz(l & 31)) * 16);
  }
  __device__ __forceinline__ static bf16x8 frag(const char* lds, uint32_t off, const uint32_t* koff, int kk) {
    return *reinterpret_cast<const bf16x8*>(lds + off + koff[kk]);
  }
};

template <int ROWS, int BK, int NW>
struct MTile {
  static constexpr int RB = ROWS * 2;    // bytes per k row
  static constexpr int KPI = 1024 / RB;  // k rows per wavefront load
  static constexpr int NI = BK / KPI;
  static constexpr int PER_WAVE = NI / NW;
  static constexpr int BYTES = ROWS * BK * 2;
  static_assert(NI % NW == 0 && KPI >= 1, "tile must split over the wavefronts");
  __device__ __forceinline__ static int swz(int k) { return 4 * (k & 3); }
  // This lane's source offset in load i (0 <= i < PER_WAVE) of this
  // wavefront's share of the tile; koff(k) is the byte offset of the tile's
  // k-row k (relative to the stage's first k row) at the tile's first m/n.
  template <class KOff>
  __device__ __forceinline__ static uint32_t voff(int l, KOff koff, int i) {
    const int w = wave_id();
    const int k = (w + NW * i) * KPI + (l * 16) / RB;
    const int c = ((l * 16) % RB) / 16 ^ swz(k);
    return koff(k) + (uint32_t)c * 16u;
  }
  __device__ __forceinline__ static void issue(i32x4 rs, uint32_t lds, uint32_t voff, int i) {
    dma16(rs, lds + (wave_id() + NW * i) * 1024, voff);
  }
  // load i with lane offset voff(0) + soff_i, soff_i = voff(i) - voff(0) (the
  // same for every lane: the swizzle of a row or k row does not change by i)
  __device__ __forceinline__ static void issue_s(i32x4 rs, uint32_t lds, uint32_t voff0, uint32_t soff, int i) {
    dma16s(rs, lds + (wave_id() + NW * i) * 1024, voff0, soff);
  }
  // Same operand layout as KTile::frag, assembled from two transpose reads:
  // in each 16-lane group g, lane i addresses 4 consecutive m/n of one k row
  // and lane j receives one m/n at 4 consecutive k. The k row's low two bits
  // (which pick the swizzle) come from the lane alone, so the address is a
  // per-block lane offset plus an immediate (16 kk + 4 h) * RB.
  __device__ __forceinline__ static uint32_t lane_off(int l, int mn0) {
    const int g = l >> 4, j = l & 15;
    const int krow = 8 * (g >> 1) + (j >> 2);
    const int mn = mn0 + 16 * (g & 1) + 4 * (j & 3);
    return (uint32_t)(krow * RB + (((mn >> 3) ^ swz(krow)) << 4) + (mn & 7) * 2);
  }
  __device__ __forceinline__ static uint32_t kstep_off(int, int) { return 0; }
  __device__ __forceinline__ static bf16x8 frag(const char* lds, uint32_t off, const uint32_t*, int kk) {
    s16x4 v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
      v[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds + off + (kk * 16 + 4 * h) * RB));
    const s16x8 t = __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, t);
  }
};

// ---------------------------------------------------------------------------
// MFMA tile core: WGM x WGN wavefronts, each owning (BM/WGM) x (BN/WGN) of
// the output as 32x32 blocks. The MFMA is fed the B rows as its first
// operand, so each lane ends up with 4 consecutive output columns of one
// output row: block (i, j), register q of lane l holds row
// wm*WM + 32 i + l % 32 and column bcol(j) + 8 (q / 4) + 4 (l / 32) + q % 4.
// ---------------------------------------------------------------------------
template <int BM, int BN, int WGM, int WGN, bool SWIGLU_COLS>
struct Core {
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int MB = WM / 32, NB = WN / 32;
  static constexpr int GW = BN / 2 / WGN;  // SwiGLU: gate (or up) columns per wave
  static_assert(MB >= 1 && NB >= 1 && (!SWIGLU_COLS || NB % 2 == 0), "wave tile");
  f32x16 acc[MB][NB];

  // LDS row of the B tile that wave column wn's block j starts at.
  __device__ __forceinline__ static int bcol(int wn, int j) {
    if constexpr (SWIGLU_COLS) {
      // gate rows live in [0, BN/2), up rows in [BN/2, BN); the wave keeps the
      // gate block j and the up block j + NB/2 of the same output columns
      constexpr int H = NB / 2;
      return j < H ? wn * GW + j * 32 : BN / 2 + wn * GW + (j - H) * 32;
    } else {
      return wn * WN + j * 32;
    }
  }

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  }

  // Per-lane LDS offsets of every 32-row block this wave reads (fixed for
  // the whole kernel) and of every k-step.
  template <class AT, class BT, int BK>
  struct Offsets {
    uint32_t a[MB], b[NB], ka[BK / 16], kb[BK / 16];
    __device__ __forceinline__ Offsets(int lane, int wm, int wn) {
#pragma unroll
      for (int i = 0; i < MB; ++i) a[i] = AT::lane_off(lane, wm * WM + i * 32);
#pragma unroll
      for (int j = 0; j < NB; ++j) b[j] = BT::lane_off(lane, bcol(wn, j));
#pragma unroll
      for (int kk = 0; kk < BK / 16; ++kk) {
        ka[kk] = AT::kstep_off(lane, kk);
        kb[kk] = BT::kstep_off(lane, kk);
      }
    }
  };

  // Operand fragments of FS k-steps in registers (the one being multiplied
  // and the ones being read ahead).
  template <int FS>
  struct Frags {
    bf16x8 a[FS][MB], b[FS][NB];
  };

  template <class AT, class BT, int BK, class FragsT>
  __device__ __forceinline__ static void load_frags(FragsT& f, int set, const char* As, const char* Bs,
                                                    const Offsets<AT, BT, BK>& o, int kk) {
#pragma unroll
    for (int i = 0; i < MB; ++i) f.a[set][i] = AT::frag(As, o.a[i], o.ka, kk);
#pragma unroll
    for (int j = 0; j < NB; ++j) f.b[set][j] = BT::frag(Bs, o.b[j], o.kb, kk);
  }

  // The MFMAs of one k-step from register set CUR, with the LDS reads of a
  // later k-step's fragments (k-step nkk of the stage at nAs/nBs, into set
  // NXT) interleaved: one read (two in the smallest wave tiles) after each of the
  // first MFMAs, so the reads complete under the matrix work. extra(q), q < NX, runs right after
  // MFMA s when q < (s + 1) NX / (MB NB) and q >= s NX / (MB NB), evenly
  // over the k-step: the loads of a later stage, spread over the k-step so
  // that the address unit drains them while the matrix cores keep working.
  template <class AT, class BT, int BK, int NX, int CUR, int NXT, class FragsT, class Extra>
  __device__ __forceinline__ void mfma_step(FragsT& f, const char* nAs, const char* nBs, const Offsets<AT, BT, BK>& o,
                                            int nkk, Extra&& extra) {
    constexpr int NM = MB * NB;
    constexpr int RPM = (MB + NB + NM - 1) / NM;  // reads after each MFMA: one, or two in the smallest wave tiles
    static_assert(NX >= 0 && NX <= NM, "loads per k-step");
    static_assert(CUR != NXT, "the fragments being read go to another set");
    if constexpr (FM_SETPRIO > 0) __builtin_amdgcn_s_setprio(FM_SETPRIO);
#pragma unroll
    for (int s = 0; s < NM; ++s) {
      const int i = s / NB, j = s % NB;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[CUR][j], f.a[CUR][i], acc[i][j], 0, 0, 0);
      if (FM_SETPRIO > 0 && s == NM - 1) __builtin_amdgcn_s_setprio(0);
#pragma unroll
      for (int t = s * RPM; t < (s + 1) * RPM && t < MB + NB; ++t) {
        if (t < MB) f.a[NXT][t] = AT::frag(nAs, o.a[t], o.ka, nkk);
        else f.b[NXT][t - MB] = BT::frag(nBs, o.b[t - MB], o.kb, nkk);
      }
      if constexpr (NX > 0) {
#pragma unroll
        for (int q = s * NX / NM; q < (s + 1) * NX / NM; ++q) extra(q);
      }
    }
#pragma unroll
    for (int s = 0; s < NM; ++s) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
      if (s * RPM < MB + NB) __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);  // its LDS reads
    }
  }
};

// Wait for the loads of the stage about to be computed: `ahead` younger
// stages (of PER loads each) may stay in flight.
template <int NS, int PER>
__device__ __forceinline__ void wait_stage(int ahead) {
  static_assert(NS >= 2 && NS <= 4 && (NS - 1) * PER < 64, "stages");
  if constexpr (NS >= 4) {
    if (ahead >= 3) {
      wait_vm<3 * PER>();
      return;
    }
  }
  if constexpr (NS >= 3) {
    if (ahead >= 2) {
      wait_vm<2 * PER>();
      return;
    }
  }
  if (ahead >= 1) {
    wait_vm<PER>();
    return;
  }
  wait_vm<0>();
}

// ---------------------------------------------------------------------------
// Software-pipelined K loop over an LDS ring of NS >= 2 stages.
//
// Stage kt's first fragments are already in registers when iteration kt
// starts, and every later k-step's fragments are read one k-step ahead. So
// when the last k-step of stage kt begins, every read of stage kt's buffer
// has been issued: each wavefront waits for its own loads of stage kt+1, and
// the workgroup barrier (which also retires all LDS reads) both publishes
// stage kt+1 and frees stage kt's buffer. The loads of stage kt+NS go into
// that buffer, spread over the MFMAs of the last k-step of stage kt and the
// first k-steps of stage kt+1 (issued in one burst, they would stall every
// wavefront behind the address unit at once). issue(s, p) issues load p
// (0 <= p < PER) of stage s, in increasing s, each stage whole before the
// next. Stages s >= KT must issue loads of nothing (zero-size buffer
// resources, which still write zeros to their LDS stage): every iteration
// then issues the same loads, with no branch among the MFMAs, and the
// counter waits stay exact.
// ---------------------------------------------------------------------------
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Fragment read distance: 2 in the row GEMMs' 256-row tiles (gate/up forward
// 2% faster than with 1, the others the same), 1 in their smaller tiles and
// in the weight gradients (a third register set makes those spill).
#ifndef FM_FRAG_DIST
#define FM_FRAG_DIST 1
#endif
#ifndef FM_FRAG_DIST_ROWS
#define FM_FRAG_DIST_ROWS 2
#endif

// Fragments read one k-step ahead (two register sets).
template <class CoreT, class AT, class BT, int BK, int NS, class Issue, class Started>
__device__ __forceinline__ void pipelined_k_loop_d1(CoreT& core, char* lds, int KT,
                                                    const typename CoreT::template Offsets<AT, BT, BK>& o,
                                                    Issue&& issue, bool drain, Started&& started) {
  static_assert(BK % 32 == 0, "the last k-step's fragments must be read before the barrier");
  constexpr int KK = BK / 16;
  constexpr int STAGE = AT::BYTES + BT::BYTES;
  constexpr int PER = AT::PER_WAVE + BT::PER_WAVE;
  // the loads of a stage ride on SPREAD k-steps: the last one of the stage
  // before and the first SPREAD - 1 of the next; load p goes with k-step
  // j when lo(j) <= p < lo(j + 1)
  // (and no k-step carries more loads than it has MFMAs)
  constexpr int MIN_SPREAD = (PER + CoreT::MB * CoreT::NB - 1) / (CoreT::MB * CoreT::NB);
  constexpr int WANT = FM_LOAD_SPREAD > MIN_SPREAD ? FM_LOAD_SPREAD : MIN_SPREAD;
  constexpr int SPREAD = WANT < KK ? WANT : KK;
  static_assert(SPREAD >= MIN_SPREAD, "load spread");
  auto lo = [](int j) constexpr { return j * PER / SPREAD; };
  typename CoreT::template Frags<2> f;
  // stages 0 .. NS-2 whole, and the part of stage NS-1 that a previous
  // iteration's last k-step would have carried
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int p = 0; p < (s < NS - 1 ? PER : lo(1)); ++p) issue(s, p);
  }
  if (drain) wait_vm<0>();
  else wait_vm<(NS - 2) * PER + lo(1)>();
  __syncthreads();
  started();
  CoreT::template load_frags<AT, BT, BK>(f, 0, lds, lds + AT::BYTES, o, 0);
  for (int kt = 0; kt < KT; ++kt) {
    const char* st = lds + (kt % NS) * STAGE;
    static_for<0, KK>([&](auto kkc) {
      constexpr int kk = decltype(kkc)::value;
      constexpr int set = kk & 1;
      if constexpr (kk < KK - 1) {
        constexpr int j = kk + 1;  // position in the load window of stage kt - 1 + NS
        core.template mfma_step<AT, BT, BK, (j < SPREAD ? lo(j + 1) - lo(j) : 0), set, set ^ 1>(
            f, st, st + AT::BYTES, o, kk + 1, [&](int q) { issue(kt - 1 + NS, lo(j) + q); });
      } else {
        wait_stage<NS, PER>(NS - 2);  // stage kt+1 (past the last: empty) has landed
        __syncthreads();
        const char* nst = lds + ((kt + 1) % NS) * STAGE;
        // (after the last stage this reads a stale buffer: harmless, and no
        // branch among the MFMAs)
        core.template mfma_step<AT, BT, BK, lo(1), set, set ^ 1>(f, nst, nst + AT::BYTES, o, 0,
                                                                 [&](int q) { issue(kt + NS, q); });
      }
    });
  }
  wait_vm<0>();  // the (empty) loads of stages past the last have landed too
}

// Fragments read D k-steps ahead (D + 1 register sets), so that each LDS read
// has D k-steps of matrix work to complete under. The barrier then comes at
// k-step KK - D of stage kt, the first whose reads reach into stage kt+1: by
// then every read of stage kt's buffer has been issued, and the loads of
// stage kt+NS go into it during k-steps KK - D .. KK - D + SPREAD - 1. The
// set of global k-step g is g % (D + 1); the stage loop is unrolled U times
// so that every set index is a compile-time constant.
template <class CoreT, class AT, class BT, int BK, int NS, int D, class Issue, class Started>
__device__ __forceinline__ void pipelined_k_loop_deep(CoreT& core, char* lds, int KT,
                                                      const typename CoreT::template Offsets<AT, BT, BK>& o,
                                                      Issue&& issue, bool drain, Started&& started) {
  constexpr int KK = BK / 16;
  constexpr int FS = D + 1;
  constexpr int STAGE = AT::BYTES + BT::BYTES;
  constexpr int PER = AT::PER_WAVE + BT::PER_WAVE;
  constexpr int SPREAD = FM_LOAD_SPREAD < D ? FM_LOAD_SPREAD : D;
  static_assert(D >= 2 && KK >= D, "read distance");
  static_assert(SPREAD >= 1, "load spread");
  auto lo = [](int j) constexpr { return j * PER / SPREAD; };
  constexpr int U = [] {
    int u = 1;
    while ((u * KK) % FS) ++u;
    return u;
  }();
  typename CoreT::template Frags<FS> f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int p = 0; p < PER; ++p) issue(s, p);
  }
  wait_stage<NS, PER>(drain ? 0 : NS - 1);  // stage 0 has landed
  __syncthreads();
  started();
  static_for<0, D>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    CoreT::template load_frags<AT, BT, BK>(f, k, lds, lds + AT::BYTES, o, k);
  });
  int kt = 0;
  while (kt < KT) {  // kt advances inside the unrolled stage loop
    static_for<0, U>([&](auto phc) {
      constexpr int ph = decltype(phc)::value;
      if (kt >= KT) return;
      const char* st = lds + (kt % NS) * STAGE;
      const char* nst = lds + ((kt + 1) % NS) * STAGE;
      static_for<0, KK>([&](auto kkc) {
        constexpr int kk = decltype(kkc)::value;
        constexpr int g = ph * KK + kk;
        constexpr int cur = g % FS, nxt = (g + D) % FS;
        constexpr int j = kk - (KK - D);  // position in the load window of stage kt + NS
        constexpr int nx = (j >= 0 && j < SPREAD) ? lo(j + 1) - lo(j) : 0;
        if constexpr (j == 0) {
          wait_stage<NS, PER>(NS - 2);  // stage kt+1 (past the last: empty) has landed
          __syncthreads();
        }
        // reads of k-step kk + D: in this stage's buffer, or in the next's
        // (after the last stage a stale buffer: harmless, and no branch among
        // the MFMAs)
        const char* rs = kk + D < KK ? st : nst;
        constexpr int rk = (kk + D) % KK;
        core.template mfma_step<AT, BT, BK, nx, cur, nxt>(f, rs, rs + AT::BYTES, o, rk, [&](int q) {
          if constexpr (j >= 0) issue(kt + NS, lo(j) + q);
        });
      });
      ++kt;
    });
  }
  wait_vm<0>();  // the (empty) loads of stages past the last have landed too
}

// drain: the first wait is for every vector-memory operation of the
// wavefront, older stores included. started() runs after the first barrier.
template <class CoreT, class AT, class BT, int BK, int NS, int D, class Issue, class Started>
__device__ __forceinline__ void pipelined_k_loop(CoreT& core, char* lds, int KT,
                                                 const typename CoreT::template Offsets<AT, BT, BK>& o,
                                                 Issue&& issue, bool drain, Started&& started) {
  if constexpr (D >= 2 && BK / 16 >= D)
    pipelined_k_loop_deep<CoreT, AT, BT, BK, NS, D>(core, lds, KT, o, issue, drain, started);
  else
    pipelined_k_loop_d1<CoreT, AT, BT, BK, NS>(core, lds, KT, o, issue, drain, started);
}

// ---------------------------------------------------------------------------
// Row-grouped GEMM: for each slot j, rows [off_j, off_{j+1}) (clamped to
// n_cap) times the slot's weight matrix.
// ---------------------------------------------------------------------------
struct RowsArgs {
  const uint16_t* A;  // [n_cap, K]
  int64_t lda;
  const uint16_t* B;  // weights; matrix w starts at B + w * wstride
  int64_t ldb;
  int64_t wstride;
  int K;
  int N;   // output columns of the tile grid (2F for the fused gate/up)
  int F;   // SwiGLU width
  uint16_t* C;  // main output
  int64_t ldc;
  uint16_t* C2;  // forward: saved [A | U] or NULL
  int64_t ldc2;
  const uint16_t* AU;  // input gradient: saved [A | U]
  int64_t ldau;
};

// One launch: one GEMM, or two with the second consuming the first's rows.
struct FfnArgs {
  RowsArgs p[2];  // gate/up then down forward, or down then gate/up input gradient
  int phases;     // bit i: run p[i]
  int W;
  const int32_t* slot_offset;
  const int32_t* slot_widx;
  int S;
  int64_t n_cap;
  float* part;         // workspace: partial tiles of tiles cut along K, or NULL
  unsigned* arrived;   // workspace: arrival count per (half) tile cut along K
  unsigned* queue;     // workspace: kQueues counters per GEMM, then the finished workgroups
  unsigned* row_done;  // workspace: halves of column tiles done per row tile of the first GEMM
};

constexpr int kQueues = 8;       // one per XCD
// Queue counters are 256 bytes apart: in one line, the atomics of all
// workgroups (they end their tiles together) would queue up behind each other.
constexpr int kQueueStride = 64;

// Row tiles of a launch (slot_tiles), built by every workgroup from the slot
// offsets. They are numbered: the 256-row ones slot by slot, then the short
// ones, then the thin ones.
struct RowTiles {
  int full[FOREMOE_MAX_SLOTS + 1];  // 256-row tiles of the slots before
  uint16_t tail[FOREMOE_MAX_SLOTS];  // slots of the short tiles from the front, of the thin ones from the back
  int off[FOREMOE_MAX_SLOTS + 1];    // the slots' row offsets, clamped to the buffer
  int widx[FOREMOE_MAX_SLOTS];
  int n_short, n_thin;
};

__device__ __forceinline__ int64_t clamp_row(int32_t v, int64_t n_cap) {
  return v < 0 ? 0 : (v > n_cap ? n_cap : v);
}

// Up to 64 slots: one wavefront does it all and no barrier but the last is
// needed (every launch starts with this).
__device__ void build_row_tiles(const int32_t* __restrict__ off, const int32_t* __restrict__ widx, int S,
                                int64_t n_cap, RowTiles& R, int* s_tmp) {
  const bool one_wave = S <= 64;
  const int nthreads = one_wave ? 64 : (int)blockDim.x;
  int full0 = 0, tail0 = 0;  // tail0: short tiles in the low half, thin ones in the high half
  if (!one_wave || threadIdx.x < 64) {
    for (int j0 = 0; j0 < S; j0 += nthreads) {
      const int j = j0 + threadIdx.x, lane = lane64();
      int full = 0, tail = 0;
      if (j < S) {
        const int beg = (int)clamp_row(off[j], n_cap), end = (int)clamp_row(off[j + 1], n_cap), rows = end - beg;
        R.off[j] = beg;
        if (j == S - 1) R.off[S] = end;
        R.widx[j] = widx[j];
        if (rows > 0) {
          const SlotTiles t = slot_tiles(rows);
          full = t.full;
          tail = t.is_short | t.is_thin << 16;
        }
      }
      int fi = full, ti = tail;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int f = __shfl_up(fi, o, 64), t = __shfl_up(ti, o, 64);
        if (lane >= o) {
          fi += f;
          ti += t;
        }
      }
      int full_all = __shfl(fi, 63, 64), tail_all = __shfl(ti, 63, 64);
      if (!one_wave) {
        const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
        if (lane == 63) {
          s_tmp[w] = fi;
          s_tmp[8 + w] = ti;
        }
        __syncthreads();
        full_all = tail_all = 0;
        for (int i = 0; i < nw; ++i) {
          if (i < w) {
            fi += s_tmp[i];
            ti += s_tmp[8 + i];
          }
          full_all += s_tmp[i];
          tail_all += s_tmp[8 + i];
        }
        __syncthreads();
      }
      if (j < S) R.full[j] = full0 + fi - full;
      const int before = tail0 + ti - tail;
      if (tail == 1) R.tail[before & 0xFFFF] = (uint16_t)j;
      if (tail == 1 << 16) R.tail[FOREMOE_MAX_SLOTS - 1 - (before >> 16)] = (uint16_t)j;
      full0 += full_all;
      tail0 += tail_all;
    }
    if (threadIdx.x == 0) {
      R.full[S] = full0;
      R.n_short = tail0 & 0xFFFF;
      R.n_thin = tail0 >> 16;
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Row-GEMM epilogue through LDS. The MFMA leaves each lane with 4-column
// pieces of 32 different rows; stored directly, every store instruction
// would touch 32 partly written lines. Instead each wavefront converts one
// 32-row block at a time to bf16 in its own LDS region and reads it back as
// whole row segments, 16 bytes per lane with consecutive lanes along a row,
// so each store instruction writes complete 128-byte lines. The staged rows
// are XOR-swizzled in 16-byte chunks so that the 8-byte writes of 32 rows
// spread over the LDS banks.
// ---------------------------------------------------------------------------
template <int RB>  // bytes per staged row
struct StagedRows {
  static constexpr int CPR = RB / 16;                   // 16-byte chunks per row
  static constexpr int RPB = RB >= 256 ? 1 : 256 / RB;  // rows per 256-byte bank cycle
  static constexpr int RPI = 64 / CPR;                  // rows per wavefront instruction
  static constexpr int NI = 32 / RPI;                   // instructions per 32-row block
  static constexpr int BYTES = 32 * RB;
  static_assert(CPR >= 1 && CPR <= 64 && 32 % RPI == 0, "staged row width");
  __device__ __forceinline__ static uint32_t chunk(int r, int c) {
    return (uint32_t)(r * RB + ((c ^ ((r / RPB) % CPR)) << 4));
  }
  // 4 consecutive values at column col (a multiple of 4) of row r
  __device__ __forceinline__ static void put4(char* base, int r, int col, float v0, float v1, float v2, float v3) {
    *reinterpret_cast<uint2*>(base + chunk(r, col >> 3) + ((col & 4) << 1)) =
        make_uint2(pack_bf2(v0, v1), pack_bf2(v2, v3));
  }
  // the 16-byte chunk lane l reads back in instruction it: row, chunk index
  __device__ __forceinline__ static int row_of(int lane, int it) { return it * RPI + lane / CPR; }
  __device__ __forceinline__ static int col_of(int lane) { return lane % CPR; }
  __device__ __forceinline__ static uint4 get(const char* base, int r, int c) {
    return *reinterpret_cast<const uint4*>(base + chunk(r, c));
  }
};

// fp32 staging (the SwiGLU backward keeps dH in fp32): RB bytes per row,
// 16-byte chunks of 4 floats; lane l reads back 8 consecutive floats.
template <int RB>
struct StagedRowsF32 {
  static constexpr int CPR = RB / 16;
  static constexpr int LPR = CPR / 2;  // lanes per row in the read-back
  static constexpr int RPI = 64 / LPR;
  static constexpr int NI = 32 / RPI;
  static constexpr int BYTES = 32 * RB;
  static_assert(RB % 256 == 0 && LPR >= 1 && LPR <= 64 && 32 % RPI == 0, "staged row width");
  __device__ __forceinline__ static uint32_t chunk(int r, int c) { return (uint32_t)(r * RB + ((c ^ (r % 16)) << 4)); }
  __device__ __forceinline__ static void put4(char* base, int r, int col, float v0, float v1, float v2, float v3) {
    *reinterpret_cast<float4*>(base + chunk(r, col >> 2)) = make_float4(v0, v1, v2, v3);
  }
  __device__ __forceinline__ static int row_of(int lane, int it) { return it * RPI + lane / LPR; }
  __device__ __forceinline__ static int col_of(int lane) { return lane % LPR; }  // in units of 8 values
  __device__ __forceinline__ static void get8(const char* base, int r, int c8, float* f) {
    const float4 lo = *reinterpret_cast<const float4*>(base + chunk(r, 2 * c8));
    const float4 hi = *reinterpret_cast<const float4*>(base + chunk(r, 2 * c8 + 1));
    f[0] = lo.x; f[1] = lo.y; f[2] = lo.z; f[3] = lo.w;
    f[4] = hi.x; f[5] = hi.y; f[6] = hi.z; f[7] = hi.w;
  }
};

template <class CoreT, int EPI>
struct EpiBytes {
  // SwiGLU forward stages H, A and U (GW bf16 columns each), the backward
  // WN fp32 columns, the plain store WN bf16 columns
  static constexpr int PER_WAVE = EPI == kEpiSwigluFwd   ? 3 * StagedRows<CoreT::GW * 2>::BYTES
                                  : EPI == kEpiSwigluBwd ? StagedRowsF32<CoreT::WN * 4>::BYTES
                                                         : StagedRows<CoreT::WN * 2>::BYTES;
};

__device__ __forceinline__ void unpack8(uint4 v, float* f) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = bf2f(w[i] & 0xFFFFu);
    f[2 * i + 1] = bf2f(w[i] >> 16);
  }
}

__device__ __forceinline__ uint4 pack8(const float* f) {
  return make_uint4(pack_bf2(f[0], f[1]), pack_bf2(f[2], f[3]), pack_bf2(f[4], f[5]), pack_bf2(f[6], f[7]));
}

template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T*)(((uint64_t)hi << 32) | lo);
}

// 16-byte buffer accesses. kCoherentDevice (the SC1 cache-policy bit) writes
// through to memory, so that a workgroup of another XCD can read the bytes
// in the same launch.
constexpr int kCoherentDevice = 16;
template <int AUX>
__device__ __forceinline__ void buffer_store16(__amdgpu_buffer_rsrc_t rs, uint32_t off, uint4 v) {
  i32x4 t;
  t.x = (int)v.x;
  t.y = (int)v.y;
  t.z = (int)v.z;
  t.w = (int)v.w;
  __builtin_amdgcn_raw_buffer_store_b128(t, rs, off, 0, AUX);
}
__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Writes this wave's output block: rows wrow0 .. wrow0 + WM - 1 (those below
// rend), output columns n0 + wn * WN .. (SwiGLU forward: H columns
// f0 + wn * GW ..). `ep` is the wave's private LDS region.
// Columns past the output's width (the last tile of a width that is no
// multiple of 256) are not stored.
template <class CoreT, int EPI>
__device__ __forceinline__ void rows_epilogue(const RowsArgs& a, const CoreT& core, char* ep, int64_t wrow0,
                                              int64_t rend, int n0, int f0, int wn) {
  const int lane = lane64_here();
  const int l32 = lane & 31, c4 = (lane >> 5) * 4;
  // Buffer resources over this wave's rows: those past the slot, and columns
  // past the width (moved past the resource's end), fall outside and are
  // neither loaded nor stored. No access is behind a branch, so the compiler
  // can count them.
  const int64_t left = rend - wrow0;
  const int64_t nrow = left <= 0 ? 0 : (left < CoreT::WM ? left : CoreT::WM);
  const uint32_t ldc2 = (uint32_t)a.ldc * 2u;
  auto rows_of = [&](const uint16_t* p, int64_t ld) {
    return __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(const_cast<uint16_t*>(p) + (nrow ? wrow0 * ld : 0)), (short)0,
                                             __builtin_amdgcn_readfirstlane((int)(nrow * ld * 2)), 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t cs = rows_of(a.C, a.ldc);
  constexpr uint32_t kOutside = 0x80000000u;
#pragma unroll
  for (int i = 0; i < CoreT::MB; ++i) {
    if constexpr (EPI == kEpiSwigluFwd) {
      using SR = StagedRows<CoreT::GW * 2>;
      constexpr int H = CoreT::NB / 2;
      char* sh = ep;
      char* sa = ep + SR::BYTES;
      char* su = ep + 2 * SR::BYTES;
#pragma unroll
      for (int jj = 0; jj < H; ++jj)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int col = jj * 32 + g * 8 + c4;
          float hv[4], av[4], uv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            av[e] = core.acc[i][jj][g * 4 + e];
            uv[e] = core.acc[i][jj + H][g * 4 + e];
          }
          silu_n<4>(av, hv);
#pragma unroll
          for (int e = 0; e < 4; ++e) hv[e] *= uv[e];
          SR::put4(sh, l32, col, hv[0], hv[1], hv[2], hv[3]);
          SR::put4(sa, l32, col, av[0], av[1], av[2], av[3]);
          SR::put4(su, l32, col, uv[0], uv[1], uv[2], uv[3]);
        }
      const int fc = f0 + wn * CoreT::GW + SR::col_of(lane) * 8;
      const __amdgpu_buffer_rsrc_t cs2 = rows_of(a.C2, a.C2 ? a.ldc2 : 0);  // ldc2 = 2 ldc
#pragma unroll
      for (int it = 0; it < SR::NI; ++it) {
        const int r = SR::row_of(lane, it);
        const uint4 vh = SR::get(sh, r, SR::col_of(lane));
        const uint4 va = SR::get(sa, r, SR::col_of(lane));
        const uint4 vu = SR::get(su, r, SR::col_of(lane));
        buffer_store16<kCoherentDevice>(cs, (uint32_t)(i * 32 + r) * ldc2 + (uint32_t)fc * 2u, vh);
        // (a NULL save_au: an empty resource)
        const uint32_t o2 = (uint32_t)(i * 32 + r) * (2u * ldc2) + (uint32_t)fc * 2u;
        buffer_store16<0>(cs2, o2, va);
        buffer_store16<0>(cs2, o2 + ldc2, vu);
      }
    } else if constexpr (EPI == kEpiSwigluBwd) {
      using SR = StagedRowsF32<CoreT::WN * 4>;
      const __amdgpu_buffer_rsrc_t aus = rows_of(a.AU, a.ldau);  // ldau = ldc
      const int nc = n0 + wn * CoreT::WN + SR::col_of(lane) * 8;
      const uint32_t outside = nc < a.N ? 0u : kOutside;
#pragma unroll
      for (int jj = 0; jj < CoreT::NB; ++jj)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int q = g * 4;
          SR::put4(ep, l32, jj * 32 + g * 8 + c4, core.acc[i][jj][q], core.acc[i][jj][q + 1], core.acc[i][jj][q + 2],
                   core.acc[i][jj][q + 3]);
        }
      // saved A and U of the rows this lane stores, loaded once this block's
      // accumulators are staged (their registers are free again; loaded
      // before the staging, they made the kernel spill), overlapping the
      // read-back of the staged dH
      uint4 xa[SR::NI], xu[SR::NI];
#pragma unroll
      for (int it = 0; it < SR::NI; ++it) {
        const uint32_t o = outside | ((uint32_t)(i * 32 + SR::row_of(lane, it)) * ldc2 + (uint32_t)nc * 2u);
        xa[it] = buffer_load16(aus, o);
        xu[it] = buffer_load16(aus, o + 2u * (uint32_t)a.F);
      }
#pragma unroll
      for (int it = 0; it < SR::NI; ++it) {
        const int r = SR::row_of(lane, it);
        // dH at columns nc .. nc + 7; saved A in [0, F), U in [F, 2F)
        float dh[8], A8[8], U8[8], sg8[8], da[8], du[8];
        SR::get8(ep, r, SR::col_of(lane), dh);
        unpack8(xa[it], A8);
        unpack8(xu[it], U8);
        sigmoid_n<8>(A8, sg8);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float sg = sg8[e];
          da[e] = dh[e] * U8[e] * (sg + A8[e] * sg * (1.0f - sg));
          du[e] = dh[e] * A8[e] * sg;
        }
        const uint32_t o = outside | ((uint32_t)(i * 32 + r) * ldc2 + (uint32_t)nc * 2u);
        buffer_store16<kCoherentDevice>(cs, o, pack8(da));
        buffer_store16<kCoherentDevice>(cs, o + 2u * (uint32_t)a.F, pack8(du));
      }
    } else {
      using SR = StagedRows<CoreT::WN * 2>;
      const int nc = n0 + wn * CoreT::WN + SR::col_of(lane) * 8;
      const uint32_t outside = nc < a.N ? 0u : kOutside;
#pragma unroll
      for (int jj = 0; jj < CoreT::NB; ++jj)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int q = g * 4;
          SR::put4(ep, l32, jj * 32 + g * 8 + c4, core.acc[i][jj][q], core.acc[i][jj][q + 1], core.acc[i][jj][q + 2],
                   core.acc[i][jj][q + 3]);
        }
#pragma unroll
      for (int it = 0; it < SR::NI; ++it) {
        const int r = SR::row_of(lane, it);
        const uint4 v = SR::get(ep, r, SR::col_of(lane));
        buffer_store16<0>(cs, outside | ((uint32_t)(i * 32 + r) * ldc2 + (uint32_t)nc * 2u), v);
      }
    }
  }
}

// Tiles cut along K: the partial sums of a piece stay in the MFMA register
// layout, one workspace slot per piece, then per wave, then per float4 index
// with the 64 lanes consecutive, so every store and load moves a whole 1 KiB.
//
// The pieces of a tile may run on different XCDs, whose L2 caches are not
// coherent with each other. The partial sums are therefore stored and loaded
// with device-scope coherence (the SC1 cache-policy bit: the store writes
// through to memory, the load does not take a stale L2 line), and a store is
// complete once the wave's vector-memory counter has drained. No device-wide
// fence is needed: such a fence would write back and invalidate the whole
// L2 of the XCD, evicting the operand tiles that every other workgroup there
// is using.
#ifndef FM_SPLIT_REGION_KIB
#define FM_SPLIT_REGION_KIB 16
#endif
constexpr int kSplitRegionKiB = FM_SPLIT_REGION_KIB;  // LDS per wave for the pieces in flight

// Byte offset of float4 group e of this wavefront in piece pc's slot.
template <class CoreT, int NW>
__device__ __forceinline__ uint32_t split_offset(int lane, int pc, int wave, int e) {
  constexpr int PER_WAVE = CoreT::MB * CoreT::NB * 4 * 64;  // float4 per wave
  static_assert(NW * PER_WAVE * 16 <= kPieceBytes, "a piece fits its slot");
  return (uint32_t)(pc * kPieceBytes + (wave * PER_WAVE + e * 64 + lane) * 16);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t split_rsrc(float* part, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(part, (short)0, (int)bytes, 0x00020000);
}

// One wavefront moves 64 x 16 bytes of the split workspace into LDS (lane l
// to lds_wave_base + 16 l), device-coherently.
__device__ __forceinline__ void split_dma16(__amdgpu_buffer_rsrc_t rs, uint32_t lds_wave_base, uint32_t voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(uintptr_t)lds_wave_base, 16,
                                           voff, 0, 0, kCoherentDevice);
}

template <class CoreT, int NW>
__device__ __forceinline__ void split_store(__amdgpu_buffer_rsrc_t rs, int pc, int wave, const CoreT& core) {
  const int lane = lane64_here();
#pragma unroll
  for (int i = 0; i < CoreT::MB; ++i)
#pragma unroll
    for (int j = 0; j < CoreT::NB; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        i32x4 v;
        v.x = __float_as_int(core.acc[i][j][4 * c]);
        v.y = __float_as_int(core.acc[i][j][4 * c + 1]);
        v.z = __float_as_int(core.acc[i][j][4 * c + 2]);
        v.w = __float_as_int(core.acc[i][j][4 * c + 3]);
        __builtin_amdgcn_raw_buffer_store_b128(v, rs, split_offset<CoreT, NW>(lane, pc, wave, (i * CoreT::NB + j) * 4 + c),
                                               0, kCoherentDevice);
      }
}

// acc = piece 0 + piece 1 + ... + piece SPLIT-1, added in this order for
// every element, all read back from the workspace (this workgroup's own
// piece included), so the result does not depend on which piece arrived
// last. The pieces travel workspace -> LDS by asynchronous loads that need
// no registers (up to 16 KiB per wave in flight, in the wave's own part of
// the free operand ring), then LDS -> registers for the additions. (Taking
// the own piece from the registers instead saves one read but makes the
// compiler spill the accumulators.) `rs` covers the tile's SPLIT slots;
// `wl` is the wave's LDS region.
template <int NW, int SPLIT, class CoreT>
__device__ __forceinline__ void split_sum(__amdgpu_buffer_rsrc_t rs, int wave, char* wl, CoreT& core) {
  constexpr int NE = CoreT::MB * CoreT::NB * 4;  // float4 groups per lane
  constexpr int GR = kSplitRegionKiB / SPLIT;    // groups per round
  const uint32_t wbase = lds_addr(wl);
  const int lane = lane64_here();
  static_for<0, (NE + GR - 1) / GR>([&](auto rc) {
    constexpr int e0 = decltype(rc)::value * GR;
    constexpr int ne = NE - e0 < GR ? NE - e0 : GR;
#pragma unroll
    for (int g = 0; g < ne; ++g)
#pragma unroll
      for (int pc = 0; pc < SPLIT; ++pc)
        split_dma16(rs, wbase + (pc * GR + g) * 1024, split_offset<CoreT, NW>(lane, pc, wave, e0 + g));
    wait_vm<0>();  // this wave's loads have landed in its LDS region
#pragma unroll
    for (int g = 0; g < ne; ++g) {
      const int e = e0 + g, c = e % 4, j = (e / 4) % CoreT::NB, i = e / 4 / CoreT::NB;
      float4 t = *reinterpret_cast<const float4*>(wl + g * 1024 + lane * 16);
#pragma unroll
      for (int pc = 1; pc < SPLIT; ++pc) {
        const float4 x = *reinterpret_cast<const float4*>(wl + (pc * GR + g) * 1024 + lane * 16);
        t.x += x.x;
        t.y += x.y;
        t.z += x.z;
        t.w += x.w;
      }
      core.acc[i][j][4 * c] = t.x;
      core.acc[i][j][4 * c + 1] = t.y;
      core.acc[i][j][4 * c + 2] = t.z;
      core.acc[i][j][4 * c + 3] = t.w;
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): LDS reads done before the region is refilled
  });
}

// Queue of XCD x: the units it takes, in order. Whole rounds of G units are
// dealt in blocks of G / nq consecutive units (which share operand tiles in
// that XCD's L2), a last partial round in nq nearly equal blocks, so that it
// is spread over all XCDs.
struct Queues {
  int G, nq, c;  // c = G / nq
  __device__ __forceinline__ int rounds(int total) const { return G == 256 ? total >> 8 : total / G; }
  __device__ __forceinline__ int part(int rest, int x) const { return nq == kQueues ? x * rest / kQueues : x * rest; }
  __device__ __forceinline__ int length(int total, int x) const {
    const int r = rounds(total), rest = total - r * G;
    return r * c + part(rest, x + 1) - part(rest, x);
  }
  __device__ __forceinline__ int unit(int total, int x, int k) const {
    const int r = rounds(total), rest = total - r * G, q = c == 32 ? k >> 5 : k / c;
    return q < r ? q * G + x * c + k - q * c : r * G + part(rest, x) + k - r * c;
  }
};

// Order of a slot's 256-row tiles: column tiles first, or on wide outputs in
// groups of 8 row tiles (which share every weight tile), row tile by row tile
// within each column tile of the group. An XCD's 32 units in flight share its
// L2: column tiles first, they span 32 / nt row tiles x nt column tiles, few
// operand tiles while nt is small, but 1 x 32 on a wide output (33 operand
// tiles for 32 products, against 8 x 4 with groups: 12). Measured, column
// tiles first -> groups (us): nt = 112 (Mixtral-8x7B gate/up) 2055 -> 1848,
// nt = 28 (DeepSeek-V3 gate/up input gradient) 563 -> 524, nt = 16 923 -> 907;
// nt = 6 (Qwen3 gate/up) 113 -> 120, nt = 3 71 -> 75. Between them, over down
// forward and gate/up input gradient (F = 2048) of 16284 uneven, 8 x 1024,
// 8192 and 16 x 2048 rows: nt = 8 to 11 groups 0.97 to 1.02 of the speed, 12 to
// 15 0.98 to 1.04, on average 1.01.
#ifndef FM_ROW_GROUP_MIN_NT
#define FM_ROW_GROUP_MIN_NT 12
#endif

// Tile shapes: rows x columns, wavefronts along each, LDS stages. The ring
// of every shape fits kRingBytes.
template <int BM_, int BN_, int WGM_, int WGN_, int NS_>
struct TileShape {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, NS = NS_;
};
using FullTile = TileShape<256, 256, FM_ROWS_WGM, FM_ROWS_WGN, FM_ROWS_NS>;
using HalfTile = TileShape<256, 128, FM_ROWS_WGM, FM_ROWS_WGN, 3>;
using ShortTile = TileShape<128, 256, 4, 2, 3>;
using ThinTile = TileShape<64, 256, 2, 4, 3>;
constexpr int kRingBytes = 147456;

// One unit: tile (slot j, rows from mrel, row tile number mt, column tile
// nt), half h of it, piece q.
constexpr int kNone = -1;       // no unit left
constexpr int kElsewhere = -2;  // the queue is empty, others may not be
struct RowUnit {
  int ph;   // which GEMM, kNone or kElsewhere
  int cls;  // 0: 256 rows, 1: 128, 2: 64
  int rbeg, rend, w;  // the slot's rows and weight index
  int mrel, mt, nt;
  int halved;
  int h, q, cut;  // cut: index of this unit among the cut ones
};

__device__ __forceinline__ RowUnit decode_unit(const PhaseUnits& u, const RowTiles& R, int S, int nfull, int idx) {
  RowUnit r;
  r.halved = 0;
  r.h = r.q = 0;
  int t = idx, j;
  r.cut = idx - u.plain;
  if (r.cut >= 0) {
    int c = r.cut;
    const int per = u.h * u.s;
    if (c < u.full_cut * per) {
      t = u.plain + c / per;
      r.halved = u.h == 2;
      r.h = c % per / u.s;
      r.q = c % u.s;
    } else {
      c -= u.full_cut * per;
      t = u.plain + u.full_cut + c / u.s;
      r.q = c % u.s;
    }
  }
  if (t < nfull * u.nt) {
    int lo = 0, hi = S - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (R.full[mid] * u.nt <= t) lo = mid;
      else hi = mid - 1;
    }
    j = __builtin_amdgcn_readfirstlane(lo);
    const int first = __builtin_amdgcn_readfirstlane(R.full[j]);
    const int mf = __builtin_amdgcn_readfirstlane(R.full[j + 1]) - first;
    const int local = t - first * u.nt;
    int m = local / u.nt;
    r.nt = local - m * u.nt;
    if (u.nt >= FM_ROW_GROUP_MIN_NT) {
      const int g = m >> 3, rem = local - 8 * g * u.nt, left = mf - 8 * g;
      if (left >= 8) {
        r.nt = rem >> 3;
        m = 8 * g + (rem & 7);
      } else {
        r.nt = rem / left;
        m = 8 * g + rem - r.nt * left;
      }
    }
    r.cls = 0;
    r.mrel = m * 256;
    r.mt = first + m;
  } else {
    t -= nfull * u.nt;
    const int i = t / u.nt;
    r.nt = t % u.nt;
    const int n_short = __builtin_amdgcn_readfirstlane(R.n_short);
    r.cls = i < n_short ? 1 : 2;
    j = __builtin_amdgcn_readfirstlane(R.tail[i < n_short ? i : FOREMOE_MAX_SLOTS - 1 - (i - n_short)]);
    r.mrel = (__builtin_amdgcn_readfirstlane(R.full[j + 1]) - __builtin_amdgcn_readfirstlane(R.full[j])) * 256;
    r.mt = nfull + i;
  }
  r.rbeg = __builtin_amdgcn_readfirstlane(R.off[j]);
  r.rend = __builtin_amdgcn_readfirstlane(R.off[j + 1]);
  r.w = __builtin_amdgcn_readfirstlane(R.widx[j]);
  return r;
}

__device__ __forceinline__ unsigned load_agent(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The hand-over of rows between two GEMMs of one launch. A row tile counts
// its column tiles in halves (2 for a whole one, 1 for each half of a halved
// one) in fa.row_done, and the queue word kDoneTotal counts all of them.
//
// A workgroup may count a tile once all its wavefronts' stores of it have
// reached memory. Waiting for that right after the epilogue would leave the
// CU idle while the stores drain, so the count is kept pending: the next
// unit's first stage loads are issued, and its first wait covers the stores
// too.
constexpr int kFinished = 2 * kQueues;       // queue word: workgroups finished
constexpr int kDoneTotal = 2 * kQueues + 1;  // queue word: halves done
constexpr int kQueueWords = 2 * kQueues + 2;
// Looks at the counters before a wait is given up: seconds, against the
// milliseconds of the longest unit. Looks are counted, not time, so that a
// process that is not running does not run out of it.
constexpr int kMaxPolls = 1 << 23;

struct HandOver {
  int tile;       // row tile of the unit whose count is pending, or -1
  unsigned count;
  bool all_done;  // no wait is needed any more: every tile of the first GEMM is done (thread 0)
};

__device__ __forceinline__ void count_done(const FfnArgs& fa, HandOver& ho) {
  // (clamped: slots that overlap, which is not valid, could make more row
  // tiles than there are counters)
  if (threadIdx.x == 0) {
    const int t = ho.tile < kMaxRowTiles ? ho.tile : kMaxRowTiles - 1;
    __hip_atomic_fetch_add(&fa.row_done[t], ho.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&fa.queue[kDoneTotal * kQueueStride], ho.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  ho.tile = -1;
}
// Counts a pending tile now.
__device__ __forceinline__ void flush_done(const FfnArgs& fa, HandOver& ho) {
  if (ho.tile < 0) return;
  wait_vm<0>();
  __syncthreads();
  count_done(fa, ho);
}

// Computes unit r of GEMM fa.p[PH]. take() starts taking the next unit once
// the k-loop's loads are done; taken() publishes it after the epilogue's
// stores have been issued, so that its latency hides under the epilogue.
// done_all: halves of the whole first GEMM.
template <class TS, bool B_KMAJ, int EPI, int PH, class Take, class Taken>
__device__ __forceinline__ void run_unit(const FfnArgs& fa, const PhaseUnits& u, const RowUnit& r, char* lds,
                                         int* s_flag, HandOver& ho, unsigned done_tile, unsigned done_all,
                                         Take&& take, Taken&& taken) {
  constexpr int BM = TS::BM, BN = TS::BN, BK = FM_ROWS_BK, NS = TS::NS, WGM = TS::WGM, WGN = TS::WGN;
  constexpr bool SW = (EPI == kEpiSwigluFwd);
  constexpr int NW = WGM * WGN;
  using CoreT = Core<BM, BN, WGM, WGN, SW>;
  using AT = KTile<BM, BK, NW>;
  using BT = typename std::conditional<B_KMAJ, KTile<BN, BK, NW>, MTile<BN, BK, NW>>::type;
  constexpr int STAGE = AT::BYTES + BT::BYTES;
  static_assert(NS * STAGE <= kRingBytes, "the ring fits");
  static_assert(NW == 8, "eight wavefronts");
  const RowsArgs& a = fa.p[PH];
  const int lane = lane64_here(), wave = wave_id();
  const int wm = wave / WGN, wn = wave % WGN;
  const uint32_t lds0 = lds_addr(lds);
  const bool pair = fa.phases == 3;
  if (PH == 1 && pair) {
    // Every unit of the first GEMM has been taken by a running workgroup
    // (units of the second are only handed out after that), those never
    // wait, and this one's pending count is done first: the rows come, within
    // the time of one unit. They do not if the counters were not zero when
    // the call began, or another call changes them meanwhile: after
    // kMaxPolls looks the workgroup goes on, and waits no more.
    flush_done(fa, ho);
    if (threadIdx.x == 0 && !ho.all_done) {
      const unsigned* done = fa.row_done + (r.mt < kMaxRowTiles ? r.mt : kMaxRowTiles - 1);
      for (int polls = 0;; ++polls) {
        const unsigned here = load_agent(done), all = load_agent(&fa.queue[kDoneTotal * kQueueStride]);
        ho.all_done = all >= done_all || polls == kMaxPolls;
        if (ho.all_done || here >= done_tile) break;
        __builtin_amdgcn_s_sleep(16);  // about half a microsecond
      }
    }
    __syncthreads();
  }
  // rows of this unit are done (stores issued)
  auto unit_done = [&]() {
    if (PH == 0 && pair) {
      flush_done(fa, ho);  // (a pending count is normally done by now)
      ho.tile = r.mt;
      ho.count = r.halved ? 1u : 2u;
    }
  };
  const int64_t rbeg = r.rbeg, rend = r.rend;
  const int64_t m0 = rbeg + r.mrel;
  const int w = r.w;
  const int n0 = r.nt * 256 + r.h * 128;         // first output column of the tile grid
  const int f0 = r.nt * 128 + r.h * 64;          // SwiGLU: first H column
  // an invalid weight index leaves the rows unwritten (every piece skips);
  // the second half of a column tile that is only 128 wide has no columns
  if (w < 0 || w >= fa.W || n0 >= a.N) {
    if (r.q == 0) unit_done();
    take();
    __syncthreads();  // every wave has read the current unit
    taken();
    return;
  }
  const int kb = r.q * u.kt / u.s, nk = (r.q + 1) * u.kt / u.s - kb;
  const int pieces = r.cut >= 0 ? u.s : 1;
  const int kb_ = pieces > 1 ? kb : 0, nk_ = pieces > 1 ? nk : u.kt;

  // operand A: the slot's rows only (rows past the slot read as zero);
  // operand B: weight matrix w. Lane offsets are fixed for the tile; each
  // stage moves the start of the buffer resource to its first k, so the
  // range check still ends at the slot's last row.
  const uint32_t lda2 = (uint32_t)(a.lda * 2), ldb2 = (uint32_t)(a.ldb * 2);
  const uint16_t* abase = a.A + rbeg * a.lda;
  const uint32_t abytes = (uint32_t)((rend - rbeg) * a.lda * 2);
  const uint16_t* bbase = a.B + (int64_t)w * a.wstride;
  const uint32_t bbytes = (uint32_t)(a.wstride * 2);
  auto arow = [&](int i) -> uint32_t { return (uint32_t)(r.mrel + i) * lda2; };
  auto brow = [&](int i) -> uint32_t {
    if constexpr (B_KMAJ) {
      int wr;
      if constexpr (SW) wr = i < BN / 2 ? f0 + i : a.F + f0 + (i - BN / 2);
      else wr = n0 + i;
      return (uint32_t)wr * ldb2;
    } else {
      // K-major weights: element (n, k) at (k * ldb + n) * 2
      return (uint32_t)i * ldb2 + (uint32_t)n0 * 2u;
    }
  };
  const uint32_t va0 = AT::voff(lane, arow, 0), vb0 = BT::voff(lane, brow, 0);
  uint32_t sa_[AT::PER_WAVE], sb_[BT::PER_WAVE];
#pragma unroll
  for (int i = 0; i < AT::PER_WAVE; ++i) sa_[i] = __builtin_amdgcn_readfirstlane(AT::voff(lane, arow, i) - va0);
#pragma unroll
  for (int i = 0; i < BT::PER_WAVE; ++i) sb_[i] = __builtin_amdgcn_readfirstlane(BT::voff(lane, brow, i) - vb0);
  auto issue = [&](int kt, int p) {
    // stages past the last load nothing (zero-size resources)
    const bool live = kt < nk_;
    const uint32_t sa = lds0 + (uint32_t)((kt % NS) * STAGE);
    const uint32_t k0 = live ? (uint32_t)((kb_ + kt) * BK) : 0u;
    if (p < AT::PER_WAVE) {
      AT::issue_s(buf_rsrc(abase + k0, live ? abytes - 2u * k0 : 0u), sa, va0, sa_[p], p);
    } else if constexpr (B_KMAJ) {
      BT::issue_s(buf_rsrc(bbase + k0, live ? bbytes - 2u * k0 : 0u), sa + AT::BYTES, vb0, sb_[p - AT::PER_WAVE],
                  p - AT::PER_WAVE);
    } else {
      BT::issue_s(buf_rsrc(bbase + (int64_t)k0 * a.ldb, live ? bbytes - k0 * ldb2 : 0u), sa + AT::BYTES, vb0,
                  sb_[p - AT::PER_WAVE], p - AT::PER_WAVE);
    }
  };

  CoreT core;
  const typename CoreT::template Offsets<AT, BT, BK> offs(lane, wm, wn);
  core.zero();
  constexpr int D = BM == 256 ? FM_FRAG_DIST_ROWS : FM_FRAG_DIST;
  const bool drain = PH == 0 && ho.tile >= 0;
  pipelined_k_loop<CoreT, AT, BT, BK, NS, D>(core, lds, nk_, offs, issue, drain, [&] {
    if (drain) count_done(fa, ho);
  });
  take();

  if constexpr (BM * BN * 4 <= kPieceBytes) {
    if (pieces > 1) {
      // the partial sums go to the workspace; the last piece of the (half)
      // tile to arrive adds all of them in piece order
      const int base = PH * cut_units((int)gridDim.x), first = base + r.cut - r.q;  // slot of piece 0
      const __amdgpu_buffer_rsrc_t rs =
          split_rsrc(fa.part + (size_t)first * (kPieceBytes / 4), (uint32_t)pieces * kPieceBytes);
      split_store<CoreT, NW>(rs, r.q, wave, core);
      wait_vm<0>();  // this wave's partial sums have reached memory
      __syncthreads();
      unsigned* count = fa.arrived + base + r.cut / pieces;
      if (threadIdx.x == 0) *s_flag = atomicAdd(count, 1u) == (unsigned)(pieces - 1);
      __syncthreads();
      if (!*s_flag) {
        taken();
        return;
      }
      static_assert(NW * kSplitRegionKiB * 1024 <= kRingBytes, "split pieces must fit in the ring");
      char* wl = lds + wave * (kSplitRegionKiB * 1024);
      if (pieces == 2) split_sum<NW, 2>(rs, wave, wl, core);
      else if (pieces == 3) split_sum<NW, 3>(rs, wave, wl, core);
      else split_sum<NW, 4>(rs, wave, wl, core);
      if (threadIdx.x == 0) atomicExch(count, 0u);  // ready for the next call
    }
  }
  static_assert(NW * EpiBytes<CoreT, EPI>::PER_WAVE <= kRingBytes, "epilogue staging must fit in the ring");
  __syncthreads();  // every wave is done reading the ring: it now stages the epilogue
  rows_epilogue<CoreT, EPI>(a, core, lds + wave * EpiBytes<CoreT, EPI>::PER_WAVE, m0 + wm * CoreT::WM, rend, n0, f0,
                            wn);
  unit_done();
  taken();
}

// The row GEMMs of one direction (FWD: gate/up with SwiGLU, then down; else
// the down input gradient with SwiGLU', then gate/up's): persistent
// workgroups, one per CU, compute units until none is left. One GEMM alone:
// every workgroup has a fixed share of its XCD's queue. Both in one launch
// (fa.phases == 3, which needs the workspace): the queues have counters; a
// workgroup takes from its own XCD's queue, then from the others', and takes
// units of the second GEMM only when the first has none left, so that the
// second fills the CUs that the first's last round leaves idle. A unit of
// the second starts once its row tile is done (fa.row_done). The next unit is
// taken and looked up while the current one's rows are being stored.
//
// What bounds it. A 256 x 256 tile's k-step of 64 takes 2700 cycles against
// 2048 of matrix work; around the k-loop a tile pays about 5000 cycles for
// its first stage and 10000 (plain) to 15000 (SwiGLU) for its epilogue, when
// all CUs store at once. On the Qwen3 EP=8 share (16278 rows in 10 slots, 5
// to 5586 each; K = 2048, 768) the launches are 1.6 and 2.1 rounds of tiles
// long, so idle CUs in the last round cost most. Measured on one box, before
// -> now (us):
//   Qwen3 forward, both GEMMs       197 -> 171   (114 + 68 -> 111 + 65 apart)
//   Qwen3 input gradients           194 -> 183   (73 + 113 -> 68 + 112 apart)
//   Mixtral-8x7B forward           2992 -> 2829  (row groups, tile heights)
//   DeepSeek-V3 input gradients     896 -> 831
//   12 slots of 26 rows, d = 2048, F = 768: gate/up 31.0 -> 23.9 (64-row
//   tiles with three stages in flight, 64 weight rows per CU and k-step at
//   5 TB/s), down 16.4 -> 14.1
// before: 256-row tiles only, a GEMM per launch, a fixed share of tiles, and
// bf16 rounding in integer arithmetic in the epilogues (15000-23000 cycles).
// One GEMM alone from the counters instead of the fixed share: 2-3 us slower
// per launch, and the policy update no faster.
template <bool FWD>
__global__ __launch_bounds__(512) void gemm_rows_kernel(FfnArgs fa) {
  __shared__ __attribute__((aligned(1024))) char lds[kRingBytes];
  __shared__ RowTiles R;
  __shared__ int s_tmp[16];
  __shared__ int s_flag;
  __shared__ int s_claim;
  __shared__ __attribute__((aligned(16))) RowUnit s_unit;

  const int tid = threadIdx.x;
  const int G = gridDim.x, nq = G % kQueues == 0 ? kQueues : 1;
  const Queues Q{G, nq, G / nq};
  const int x0 = nq == kQueues ? blockIdx.x % kQueues : 0;  // workgroups go to the XCDs in turn
  const bool pair = fa.phases == 3;
  // Of two GEMMs even the first unit is taken from the queue, since a
  // workgroup waiting for rows relies on every unit of the first GEMM being
  // held by a running workgroup (and not by one that still waits for its CU).
  int first = nq == kQueues ? blockIdx.x / kQueues : blockIdx.x;
  if (pair && tid == 0) first = (int)atomicAdd(&fa.queue[x0 * kQueueStride], 1u);
  build_row_tiles(fa.slot_offset, fa.slot_widx, fa.S, fa.n_cap, R, s_tmp);
  if (tid == 0) s_claim = first;
  const int nfull = __builtin_amdgcn_readfirstlane(R.full[fa.S]);
  const int nsmall = __builtin_amdgcn_readfirstlane(R.n_short + R.n_thin);
  const LaunchUnits lu =
      launch_units(nfull, nsmall, fa.p[0].N, fa.p[0].K, fa.p[1].N, fa.p[1].K, fa.phases, G, fa.part != nullptr);
  const PhaseUnits &u0 = lu.u0, &u1 = lu.u1;
  HandOver ho{-1, 0u, false};
  const unsigned done_tile = 2u * (unsigned)u0.nt, done_all = done_tile * (unsigned)(nfull + nsmall);

  // Wavefront 0 keeps the place in the queues: GEMM ph, queue x, position
  // s_claim. publish() looks the unit up and leaves it in s_unit; it runs
  // while the other wavefronts still store their rows. Where the queue is
  // empty, take_elsewhere() follows, after a pending tile has been counted
  // (a workgroup of the second GEMM may be waiting for it).
  int ph = (fa.phases & 1) ? 0 : 1, x = x0, step = 0;
  auto publish = [&]() __attribute__((always_inline)) {
    const int k = __builtin_amdgcn_readfirstlane(s_claim);
    const int total = ph == 0 ? u0.total : u1.total;
    if ((unsigned)k >= (unsigned)Q.length(total, x)) {  // (unsigned: whatever a counter held)
      if (tid == 0) s_unit.ph = pair ? kElsewhere : kNone;
      return;
    }
    step = k;
    RowUnit r = decode_unit(ph == 0 ? u0 : u1, R, fa.S, nfull, Q.unit(total, x, k));
    r.ph = ph;
    if (tid == 0) s_unit = r;
  };
  // Looks at all counters at once and takes from the first queue with units
  // left (own XCD first, first GEMM first).
  auto take_elsewhere = [&]() __attribute__((always_inline)) {
    const int lane = lane64();
    const int qp = (lane >> 3) & 1, qx = ((lane & 7) + x0) % kQueues;
    const int len = lane < 2 * kQueues && qx < nq ? Q.length(qp == 0 ? u0.total : u1.total, qx) : 0;
    unsigned* c = &fa.queue[(qp * kQueues + qx) * kQueueStride];
    bool open = lane < 2 * kQueues && load_agent(c) < (unsigned)len;
    int got = 0;
    uint64_t found;
    while ((found = __ballot(open)) != 0) {
      const int from = __builtin_ctzll(found);
      if (lane == from) {
        got = (int)atomicAdd(c, 1u);
        open = (unsigned)got < (unsigned)len;
      }
      if ((__ballot(open) >> from) & 1) {
        ph = from >> 3;
        x = ((from & 7) + x0) % kQueues;
        const int k = __builtin_amdgcn_readlane(got, from);
        if (tid == 0) s_claim = k;
        publish();
        return;
      }
    }
    if (tid == 0) s_unit.ph = kNone;
  };

  if (wave_id() == 0) publish();
  for (;;) {
    __syncthreads();  // the unit is known; staging reads done before its loads overwrite the ring
    if (__builtin_amdgcn_readfirstlane(s_unit.ph) == kElsewhere) {
      flush_done(fa, ho);
      __syncthreads();  // every wave has read s_unit
      if (wave_id() == 0) take_elsewhere();
      __syncthreads();
    }
    RowUnit r;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(RowUnit) / 4); ++i)
      reinterpret_cast<int*>(&r)[i] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(&s_unit)[i]);
    if (r.ph == kNone) break;
    auto go = [&](auto phc) __attribute__((always_inline)) {
      constexpr int PH = decltype(phc)::value;
      constexpr int EPI = PH == 1 ? kEpiStore : (FWD ? kEpiSwigluFwd : kEpiSwigluBwd);
      const PhaseUnits& up = PH == 0 ? u0 : u1;
      int next = 0;
      auto take = [&]() __attribute__((always_inline)) {
        next = pair ? INT_MAX : step + Q.c;
        if (pair && x == x0 && tid == 0)
          next = (int)atomicAdd(&fa.queue[(PH * kQueues + x0) * kQueueStride], 1u);
      };
      auto taken = [&]() __attribute__((always_inline)) {
        if (tid == 0) s_claim = next;
      };
      // a last column tile of 128 columns is a half tile too
      if (r.cls == 0 && (r.halved || r.nt * 256 + 128 >= fa.p[PH].N))
        run_unit<HalfTile, FWD, EPI, PH>(fa, up, r, lds, &s_flag, ho, done_tile, done_all, take, taken);
      else if (r.cls == 0)
        run_unit<FullTile, FWD, EPI, PH>(fa, up, r, lds, &s_flag, ho, done_tile, done_all, take, taken);
      else if (r.cls == 1)
        run_unit<ShortTile, FWD, EPI, PH>(fa, up, r, lds, &s_flag, ho, done_tile, done_all, take, taken);
      else
        run_unit<ThinTile, FWD, EPI, PH>(fa, up, r, lds, &s_flag, ho, done_tile, done_all, take, taken);
    };
    if (r.ph == 0) go(std::integral_constant<int, 0>{});
    else go(std::integral_constant<int, 1>{});
    if (wave_id() == 0) publish();
  }
  if (!pair) return;
  flush_done(fa, ho);

  // the last workgroup to finish leaves every counter at zero
  if (tid == 0) s_flag = atomicAdd(&fa.queue[kFinished * kQueueStride], 1u) == (unsigned)(G - 1);
  __syncthreads();
  if (!s_flag) return;
  if (tid < kQueueWords) store_agent(&fa.queue[tid * kQueueStride], 0u);
  for (int i = tid; i < nfull + nsmall && i < kMaxRowTiles; i += blockDim.x) store_agent(&fa.row_done[i], 0u);
}

// ---------------------------------------------------------------------------
// Weight gradient: dW[g] (M x N, fp32) += sum over the rows of every slot
// with gradient index g of A[row, :]^T B[row, :].
//
// Work split: the row sequence of a group (the concatenated row ranges of
// its slots, in slot order) is cut into chunks of CH rows when the caller's
// workspace allows, so that one hot expert spreads over many CUs. Chunk 0 of
// a group adds its result straight into dW; chunks 1.. write fp32 partial
// tiles to the workspace, and wgrad_reduce_kernel (launched next on the same
// stream) adds them in chunk order. Every output element therefore has one
// fixed summation order: deterministic, no atomics on floats.
// ---------------------------------------------------------------------------
// One micro-step's operands of a weight-gradient call: rows [0, n_cap) of A
// and B, and its slot table.
struct WgradStep {
  const uint16_t* A;  // [n_cap, M]
  const uint16_t* B;  // [n_cap, N]
  const int32_t* slot_offset;
  const int32_t* slot_gidx;
  int S;
  int vbase;  // first virtual slot of this step (prefix of S over the steps before)
  int64_t n_cap;
};

struct WgradArgs {
  WgradStep step[FOREMOE_MAX_WGRAD_STEPS];
  int n_steps;
  int V;  // virtual slots: every step's slots, steps in order
  int64_t lda, ldb;
  int M, N;
  int G;
  float* C;  // dW[g] at C + g * gstride, row-major [M, N]
  int64_t ldc;
  int64_t gstride;
  float* part;  // partial tiles [p_max][BM * BN]
  int p_max;
  // with partial tiles: the plan the reduce kernel needs, written by
  // workgroup 0 of the main kernel: {groups with rows, chunk rows, then per
  // ordered group: gradient index, rows, first partial tile}
  int* plan_out;
  // work counters {next item, finished workgroups} (zero on entry, zeroed
  // again by the last workgroup), or NULL for a static item order
  unsigned* sched;
  // output tiles of this call: tile index t of a group's dW (row-major over
  // the BM x BN tiles) with t % tparts == tpart
  int tpart, tparts;
};

// Tiles of one group's dW that a call computes, and the index of the i-th.
// M and N are multiples of 128: a last row or column of 256-wide tiles may be
// half empty.
__device__ __forceinline__ int wgrad_call_tiles(const WgradArgs& a, int BM, int BN) {
  return (((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN) - a.tpart + a.tparts - 1) / a.tparts;
}
__device__ __forceinline__ int wgrad_tile(const WgradArgs& a, int i) { return a.tpart + i * a.tparts; }

// The row sequence of gradient group g is the rows of every virtual slot v
// (step m's slot j, v = vbase_m + j) with gradient index g, in v order: the
// micro-steps in order, each one's slots in order.
struct WgradPlan {
  int beg[FOREMOE_MAX_SLOTS];        // clamped row range [beg, end) of virtual slot v in its step's rows
  int end[FOREMOE_MAX_SLOTS];
  uint16_t gs[FOREMOE_MAX_SLOTS];    // step << 10 | gradient index, kNoSlot for empty/invalid slots
  uint16_t next[FOREMOE_MAX_SLOTS];  // next virtual slot of the same group, kNoSlot after the last
  uint16_t first[FOREMOE_MAX_SLOTS];  // first virtual slot of each group
  int rows[FOREMOE_MAX_SLOTS];       // rows per group
  uint16_t order[FOREMOE_MAX_SLOTS];  // groups by descending rows
  uint16_t rem[FOREMOE_MAX_SLOTS];   // ordered groups with a last, partial chunk, by its descending size
  int ibase[FOREMOE_MAX_SLOTS + 1];  // prefix over ordered groups of their whole chunks
  int pbase[FOREMOE_MAX_SLOTS + 1];  // partial-tile prefix over ordered groups
  const uint16_t* A[FOREMOE_MAX_WGRAD_STEPS];  // operands of each step
  const uint16_t* B[FOREMOE_MAX_WGRAD_STEPS];
  unsigned long long total;          // rows of all groups
  int nne;                           // non-empty groups
  int nrem;                          // groups with a partial chunk
  int ch;                            // chunk rows (INT_MAX: no split)
  static constexpr int kNoSlot = 0xFFFF;
  __device__ __forceinline__ int gidx(int v) const { return gs[v] & 1023; }
  __device__ __forceinline__ int step(int v) const { return gs[v] >> 10; }
};
static_assert(FOREMOE_MAX_SLOTS <= 1024 && FOREMOE_MAX_WGRAD_STEPS <= 32, "gs fields");

// Every workgroup builds the plan, so it has to be quick: a slot finds its
// group's next one once here (walked through at every item and every slot
// change, 80 to 160 virtual slots cost each item thousands of cycles), and
// one wavefront does the prefix sums and the ranking of the partial chunks.
template <int BM, int BN, int BK>
__device__ void build_wgrad_plan(const WgradArgs& a, WgradPlan& P) {
  const int tid = threadIdx.x;
  const int G = a.G, V = a.V;
  const int tpg = wgrad_call_tiles(a, BM, BN);
  const int nt = blockDim.x;
  if (tid == 0) {
    P.nne = P.nrem = 0;
    P.total = 0;
  }
  // the step table into LDS with compile-time indices (a kernel argument
  // indexed at run time would be copied to scratch)
#pragma unroll
  for (int m = 0; m < FOREMOE_MAX_WGRAD_STEPS; ++m) {
    if (tid == m && m < a.n_steps) {
      P.A[m] = a.step[m].A;
      P.B[m] = a.step[m].B;
    }
  }
  int* first = P.ibase;  // (free until the prefix sums)
  for (int g = tid; g < G; g += nt) {
    P.rows[g] = 0;
    first[g] = INT_MAX;
  }
  for (int v = tid; v < V; v += nt) {
    int m = 0;
#pragma unroll
    for (int q = 1; q < FOREMOE_MAX_WGRAD_STEPS; ++q)
      if (q < a.n_steps && v >= a.step[q].vbase) m = q;
    const int32_t* off = nullptr;
    const int32_t* gi = nullptr;
    int64_t n_cap = 0;
    int j = 0;
#pragma unroll
    for (int q = 0; q < FOREMOE_MAX_WGRAD_STEPS; ++q)
      if (q == m) {
        off = a.step[q].slot_offset;
        gi = a.step[q].slot_gidx;
        n_cap = a.step[q].n_cap;
        j = v - a.step[q].vbase;
      }
    const int lo = (int)clamp_row(off[j], n_cap), hi = (int)clamp_row(off[j + 1], n_cap);
    const int g = gi[j];
    const bool ok = g >= 0 && g < G && hi > lo;
    P.beg[v] = lo;
    P.end[v] = ok ? hi : lo;
    P.gs[v] = (uint16_t)(ok ? (m << 10 | g) : WgradPlan::kNoSlot);
  }
  __syncthreads();
  for (int v = tid; v < V; v += nt) {
    const int gs = P.gs[v];
    if (gs == WgradPlan::kNoSlot) continue;
    const int g = gs & 1023, n = P.end[v] - P.beg[v];
    atomicAdd(&P.rows[g], n);
    atomicMin(&first[g], v);
    atomicAdd(&P.total, (unsigned long long)n);
    int w = v + 1;
    while (w < V && (P.gs[w] == WgradPlan::kNoSlot || (P.gs[w] & 1023) != g)) ++w;
    P.next[v] = (uint16_t)(w < V ? w : WgradPlan::kNoSlot);
  }
  __syncthreads();
  for (int g = tid; g < G; g += nt) {
    const int rg = P.rows[g];
    if (rg <= 0) continue;
    P.first[g] = (uint16_t)first[g];
    int rank = 0;
    for (int h = 0; h < G; ++h) {
      const int rh = P.rows[h];
      rank += (rh > rg) || (rh == rg && h < g);
    }
    P.order[rank] = (uint16_t)g;
    atomicAdd(&P.nne, 1);
  }
  __syncthreads();
  if (tid < 64) {
    const int nne = __builtin_amdgcn_readfirstlane(P.nne), lane = lane64();
    int ch = INT_MAX;
    if (a.p_max > 0 && nne > 0) {
      unsigned long long c = (P.total * (unsigned)tpg + (unsigned)a.p_max - 1) / (unsigned)a.p_max;
      c = (c + BK - 1) / BK * BK;
      ch = c > INT_MAX ? INT_MAX : (int)c;
    }
    int ib = 0, pb = 0, nrem = 0;
    for (int i0 = 0; i0 < nne; i0 += 64) {
      const int i = i0 + lane;
      const int rg = i < nne ? P.rows[P.order[i]] : 0;
      const int whole = ch == INT_MAX ? 0 : rg / ch, ri = rg - whole * (ch == INT_MAX ? 0 : ch);
      const int wt = whole * tpg, pt = rg > 0 ? (whole + (ri > 0) - 1) * tpg : 0;
      int wi = wt, pi = pt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int w = __shfl_up(wi, o, 64), p = __shfl_up(pi, o, 64);
        if (lane >= o) {
          wi += w;
          pi += p;
        }
      }
      if (i < nne) {
        P.ibase[i] = ib + wi - wt;
        P.pbase[i] = pb + pi - pt;
      }
      ib += __shfl(wi, 63, 64);
      pb += __shfl(pi, 63, 64);
      // ranked within these 64 groups (all there are, but for huge tables)
      int rank = nrem;
      const int n = nne - i0 < 64 ? nne - i0 : 64;
      for (int h = 0; h < n; ++h) {
        const int rh = __builtin_amdgcn_readlane(ri, h);
        rank += (rh > ri) || (rh == ri && h < lane);
      }
      if (ri > 0) P.rem[rank] = (uint16_t)i;
      nrem += __popcll(__ballot(ri > 0));
    }
    if (lane == 0) {
      P.ibase[nne] = ib;
      P.pbase[nne] = pb;
      P.nrem = nrem;
      P.ch = ch;
    }
  }
  __syncthreads();
}

// Walks the k-tiles of one chunk [s0, s1) of a group's row sequence: each
// k-tile lies inside one virtual slot's row range [lo, hi).
struct KCursor {
  int j, pos, lo, hi, k;  // virtual slot, sequence position of slot start, segment rows, tile start
  bool done;
  const uint16_t* pa;  // operands of slot j's micro-step (wave-uniform: scalar registers)
  const uint16_t* pb;
};

__device__ __forceinline__ void cursor_slot(const WgradPlan& P, int s0, int s1, KCursor& c) {
  const int beg = __builtin_amdgcn_readfirstlane(P.beg[c.j]), end = __builtin_amdgcn_readfirstlane(P.end[c.j]);
  const int n = end - beg, skip = s0 > c.pos ? s0 - c.pos : 0;
  c.lo = beg + skip;
  c.hi = beg + (n < s1 - c.pos ? n : s1 - c.pos);
  c.k = c.lo;
  const int m = __builtin_amdgcn_readfirstlane(P.step(c.j));
  c.pa = uniform_ptr(P.A[m]);
  c.pb = uniform_ptr(P.B[m]);
}

__device__ __forceinline__ void cursor_next_slot(const WgradPlan& P, int s1, KCursor& c) {
  const int next = __builtin_amdgcn_readfirstlane(P.next[c.j]);
  c.pos += __builtin_amdgcn_readfirstlane(P.end[c.j]) - __builtin_amdgcn_readfirstlane(P.beg[c.j]);
  if (next == WgradPlan::kNoSlot || c.pos >= s1) {
    c.done = true;
    return;
  }
  c.j = next;
  cursor_slot(P, 0, s1, c);
}

// [s0, s1) is not empty and lies inside the group's rows.
__device__ __forceinline__ KCursor cursor_begin(const WgradPlan& P, int g, int s0, int s1) {
  KCursor c;
  c.done = false;
  c.pos = 0;
  c.j = __builtin_amdgcn_readfirstlane(P.first[g]);
  for (;;) {
    const int n = __builtin_amdgcn_readfirstlane(P.end[c.j]) - __builtin_amdgcn_readfirstlane(P.beg[c.j]);
    const int next = __builtin_amdgcn_readfirstlane(P.next[c.j]);
    if (c.pos + n > s0 || next == WgradPlan::kNoSlot) break;
    c.pos += n;
    c.j = next;
  }
  cursor_slot(P, s0, s1, c);
  return c;
}

template <int BK>
__device__ __forceinline__ void cursor_advance(const WgradPlan& P, int s1, KCursor& c) {
  c.k += BK;
  if (c.k >= c.hi) cursor_next_slot(P, s1, c);
}

template <int BM, int BN, int BK, int NS, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_wgrad_kernel(WgradArgs a) {
  constexpr int NW = WGM * WGN;
  using CoreT = Core<BM, BN, WGM, WGN, false>;
  using AT = MTile<BM, BK, NW>;
  using BT = MTile<BN, BK, NW>;
  constexpr int STAGE = AT::BYTES + BT::BYTES;
  __shared__ __attribute__((aligned(1024))) char lds[NS * STAGE];
  __shared__ WgradPlan P;

  build_wgrad_plan<BM, BN, BK>(a, P);
  if (a.plan_out && blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      a.plan_out[0] = P.nne;
      a.plan_out[1] = P.ch;
    }
    for (int i = threadIdx.x; i < P.nne; i += blockDim.x) {
      a.plan_out[2 + 3 * i] = P.order[i];
      a.plan_out[3 + 3 * i] = P.rows[P.order[i]];
      a.plan_out[4 + 3 * i] = P.pbase[i];
    }
  }
  const int nt_n = (a.N + BN - 1) / BN, tpg = wgrad_call_tiles(a, BM, BN);
  const int whole = __builtin_amdgcn_readfirstlane(P.ibase[P.nne]);
  const int total = whole + __builtin_amdgcn_readfirstlane(P.nrem) * tpg;
  const int lane = lane64(), wave = wave_id();
  const int wm = wave / WGN, wn = wave % WGN;
  const uint32_t lds0 = lds_addr(lds);
  const uint32_t lda2 = (uint32_t)(a.lda * 2), ldb2 = (uint32_t)(a.ldb * 2);
  CoreT core;
  const typename CoreT::template Offsets<AT, BT, BK> offs(lane, wm, wn);

  // Items (output tile x row chunk) come in descending size: the whole chunks
  // of all groups, then the groups' last, partial ones. (Group by group, a
  // large group's small rest ran before the next group's whole chunks, which
  // then ended late: 4 micro-steps of the Qwen3 share, down 0.84 of that time
  // in a simulation of the item sizes.) With work counters each workgroup
  // takes the next item when it is free, which balances the very uneven
  // sizes; without, a fixed stride (XCD-aware).
  __shared__ int s_item;
  auto next_item = [&](int prev) -> int {
    if (!a.sched) return prev < 0 ? xcd_virtual_id() : prev + (int)gridDim.x;
    if (threadIdx.x == 0) s_item = (int)atomicAdd(&a.sched[0], 1u);
    __syncthreads();
    return s_item;
  };
  for (int t = next_item(-1); t < total; t = next_item(t)) {
    int lo, local, c;  // ordered group, item within its whole (partial) chunks, chunk
    if (t < whole) {
      lo = 0;
      int hi = P.nne - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (P.ibase[mid] <= t) lo = mid;
        else hi = mid - 1;
      }
      lo = __builtin_amdgcn_readfirstlane(lo);
      local = t - P.ibase[lo];
      c = local / tpg;
    } else {
      local = t - whole;
      lo = __builtin_amdgcn_readfirstlane(P.rem[local / tpg]);
      c = P.ch == INT_MAX ? 0 : P.rows[P.order[lo]] / P.ch;
    }
    const int gi = lo, g = __builtin_amdgcn_readfirstlane(P.order[gi]);
    const int tile_l = local % tpg, tile = wgrad_tile(a, tile_l);
    const int m0 = (tile / nt_n) * BM, n0 = (tile % nt_n) * BN;
    const int rg = P.rows[g];
    const int s0 = P.ch == INT_MAX ? 0 : c * P.ch;
    const int s1 = P.ch == INT_MAX ? rg : (s0 + P.ch < rg ? s0 + P.ch : rg);

    // number of k-tiles of this chunk (each k-tile stays inside one slot)
    int KT = 0;
    for (KCursor cc = cursor_begin(P, g, s0, s1); !cc.done; cursor_next_slot(P, s1, cc))
      KT += (cc.hi - cc.lo + BK - 1) / BK;
    KCursor ic = cursor_begin(P, g, s0, s1);
    auto koa = [&](int k) -> uint32_t { return (uint32_t)k * lda2 + (uint32_t)m0 * 2u; };
    auto kob = [&](int k) -> uint32_t { return (uint32_t)k * ldb2 + (uint32_t)n0 * 2u; };
    const uint32_t va0 = AT::voff(lane, koa, 0), vb0 = BT::voff(lane, kob, 0);
    uint32_t sa_[AT::PER_WAVE], sb_[BT::PER_WAVE];
#pragma unroll
    for (int i = 0; i < AT::PER_WAVE; ++i) sa_[i] = __builtin_amdgcn_readfirstlane(AT::voff(lane, koa, i) - va0);
#pragma unroll
    for (int i = 0; i < BT::PER_WAVE; ++i) sb_[i] = __builtin_amdgcn_readfirstlane(BT::voff(lane, kob, i) - vb0);
    auto issue = [&](int kt, int p) {
      // the loads of one k-tile are issued in order p = 0 .. PER-1, k-tiles
      // in order: load the cursor's k-tile, advance after its last load. The
      // resource starts at the k-tile's first row and ends at the segment's
      // last, so rows past the segment read as zero; once the cursor is
      // done, the stages past the last load nothing.
      const bool live = !ic.done;
      const uint32_t sa = lds0 + (uint32_t)((kt % NS) * STAGE);
      const int k = live ? ic.k : 0;
      const uint32_t nrow = live ? (uint32_t)(ic.hi - ic.k) : 0u;
      if (p < AT::PER_WAVE) {
        AT::issue_s(buf_rsrc(ic.pa + (int64_t)k * a.lda, nrow * lda2), sa, va0, sa_[p], p);
      } else {
        BT::issue_s(buf_rsrc(ic.pb + (int64_t)k * a.ldb, nrow * ldb2), sa + AT::BYTES, vb0, sb_[p - AT::PER_WAVE],
                    p - AT::PER_WAVE);
      }
      if (p == AT::PER_WAVE + BT::PER_WAVE - 1 && live) cursor_advance<BK>(P, s1, ic);
    };

    core.zero();
    pipelined_k_loop<CoreT, AT, BT, BK, NS, FM_FRAG_DIST>(core, lds, KT, offs, issue, false, [] {});
    __syncthreads();

    const int l32 = lane & 31, c4 = (lane >> 5) * 4;
    // a wave past the last row or column of dW (both multiples of 128) has
    // nothing to add
    static_assert(128 % CoreT::WM == 0 && 128 % CoreT::WN == 0, "waves are wholly inside or outside");
    const bool inside = m0 + wm * CoreT::WM < a.M && n0 + wn * CoreT::WN < a.N;
    if (!inside) {
      // (falls through to the barrier below)
    } else if (c == 0) {
      // dW += acc. The current dW values of this wave's output are brought
      // into LDS with asynchronous buffer loads (two 32-row blocks at a time,
      // all loads in flight together; each wave uses its own LDS region, so
      // no barrier is needed), then added to the accumulators and stored.
      float* Cg = a.C + (int64_t)g * a.gstride;
      constexpr int RB = CoreT::WN * 4;  // bytes of one output row of this wave
      constexpr int CH = RB / 16;        // 16-byte chunks per row
      constexpr int REGION = 2 * 32 * RB;
      static_assert(NW * REGION <= NS * STAGE, "epilogue staging must fit the LDS stages");
      static_assert(CH >= 16 && (CH & (CH - 1)) == 0, "row chunks");
      const i32x4 rsc = buf_rsrc(Cg, (uint32_t)((int64_t)a.M * a.N * 4));
      char* wl = lds + wave * REGION;
      const int nb = n0 + wn * CoreT::WN;
#pragma unroll
      for (int ph = 0; ph < (CoreT::MB + 1) / 2; ++ph) {
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
          const int i = ph * 2 + ii;
          if (i >= CoreT::MB) break;
          const int mb = m0 + wm * CoreT::WM + i * 32;
#pragma unroll
          for (int q = 0; q < 32 * RB / 1024; ++q) {
            const int r = q * (1024 / RB) + (lane * 16) / RB;
            const int pc = ((lane * 16) % RB) / 16;
            const int lc = pc ^ (r & (CH - 1));
            dma16(rsc, lds_addr(wl + ii * (32 * RB) + q * 1024),
                  (uint32_t)(((int64_t)(mb + r) * a.ldc + nb) * 4) + (uint32_t)lc * 16u);
          }
        }
        wait_vm<0>();
        // add the accumulators in place (LDS row r, chunk pc holds the
        // global chunk pc ^ (r % CH) of row r)...
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
          const int i = ph * 2 + ii;
          if (i >= CoreT::MB) break;
#pragma unroll
          for (int jj = 0; jj < CoreT::NB; ++jj) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int nl = jj * 32 + q * 8 + c4;
              const int pc = (nl / 4) ^ (l32 & (CH - 1));
              float4* lp = reinterpret_cast<float4*>(wl + ii * (32 * RB) + l32 * RB + pc * 16);
              float4 o = *lp;
              o.x += core.acc[i][jj][q * 4 + 0];
              o.y += core.acc[i][jj][q * 4 + 1];
              o.z += core.acc[i][jj][q * 4 + 2];
              o.w += core.acc[i][jj][q * 4 + 3];
              *lp = o;
            }
          }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the sums are in LDS
        // ...then store them from the lanes that loaded them: each store
        // instruction writes whole row segments (full 128-byte lines)
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
          const int i = ph * 2 + ii;
          if (i >= CoreT::MB) break;
          const int mb = m0 + wm * CoreT::WM + i * 32;
#pragma unroll
          for (int q = 0; q < 32 * RB / 1024; ++q) {
            const int r = q * (1024 / RB) + (lane * 16) / RB;
            const int pc = ((lane * 16) % RB) / 16;
            const int lc = pc ^ (r & (CH - 1));
            const float4 o = *reinterpret_cast<const float4*>(wl + ii * (32 * RB) + q * 1024 + lane * 16);
            *reinterpret_cast<float4*>(Cg + (int64_t)(mb + r) * a.ldc + nb + lc * 4) = o;
          }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): LDS reads done before the region is refilled
      }
    } else {
      float* Pt = a.part + (int64_t)(P.pbase[gi] + (c - 1) * tpg + tile_l) * (BM * BN);
#pragma unroll
      for (int i = 0; i < CoreT::MB; ++i) {
        const int m = wm * CoreT::WM + i * 32 + l32;
#pragma unroll
        for (int jj = 0; jj < CoreT::NB; ++jj) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = wn * CoreT::WN + jj * 32 + q * 8 + c4;
            *reinterpret_cast<float4*>(Pt + m * BN + n) =
                make_float4(core.acc[i][jj][q * 4 + 0], core.acc[i][jj][q * 4 + 1], core.acc[i][jj][q * 4 + 2],
                            core.acc[i][jj][q * 4 + 3]);
          }
        }
      }
    }
    __syncthreads();  // the epilogue's LDS staging is done before the next item's loads
  }
  if (a.sched && threadIdx.x == 0) {
    // each workgroup counts itself finished after its last take returned, so
    // the last one to finish can zero the counters for the next call
    if (atomicAdd(&a.sched[1], 1u) == gridDim.x - 1) {
      atomicExch(&a.sched[0], 0u);
      atomicExch(&a.sched[1], 0u);
    }
  }
}

// dW[g] tile += partials of chunks 1.. in chunk order. Each tile is cut into
// kReduceParts row bands, one workgroup per band, so that all CUs stream.
constexpr int kReduceParts = 16;

template <int BM, int BN, int BK>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(WgradArgs a) {
  // the main kernel's plan (its split groups come first: largest rows)
  const int* pl = a.plan_out;
  const int nne = pl[0], ch = pl[1];
  if (ch == INT_MAX) return;
  const int nt_n = (a.N + BN - 1) / BN, tpg = wgrad_call_tiles(a, BM, BN);
  int nsplit = 0;
  while (nsplit < nne && (pl[3 + 3 * nsplit] + ch - 1) / ch > 1) ++nsplit;
  const int total = nsplit * tpg * kReduceParts;
  constexpr int BAND = BM * BN / kReduceParts;  // elements per band
  constexpr int V = BAND / 1024 < 4 ? BAND / 1024 : 4;  // float4 per thread per pass
  static_assert(V >= 1 && BAND % (256 * 4 * V) == 0, "band split");
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    const int part = t % kReduceParts, tt = t / kReduceParts;
    const int gi = tt / tpg, tile_l = tt % tpg, tile = wgrad_tile(a, tile_l);
    const int g = pl[2 + 3 * gi];
    const int cg = (pl[3 + 3 * gi] + ch - 1) / ch;
    const int m0 = (tile / nt_n) * BM, n0 = (tile % nt_n) * BN;
    float* Cg = a.C + (int64_t)g * a.gstride;
    const float* P0 = a.part + (int64_t)(pl[4 + 3 * gi] + tile_l) * (BM * BN);
    const int64_t cstride = (int64_t)tpg * (BM * BN);
    for (int e0 = part * BAND + threadIdx.x * 4; e0 < (part + 1) * BAND; e0 += 256 * 4 * V) {
      float4 s[V];
#pragma unroll
      for (int v = 0; v < V; ++v) s[v] = *reinterpret_cast<const float4*>(P0 + e0 + v * 1024);
      for (int c = 2; c < cg; ++c) {
        float4 x[V];
#pragma unroll
        for (int v = 0; v < V; ++v) x[v] = *reinterpret_cast<const float4*>(P0 + (c - 1) * cstride + e0 + v * 1024);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          s[v].x += x[v].x;
          s[v].y += x[v].y;
          s[v].z += x[v].z;
          s[v].w += x[v].w;
        }
      }
      float4 o[V];
      // (rows and columns of the tile past dW's are left alone)
      auto in_dw = [&](int e) { return m0 + e / BN < a.M && n0 + e % BN < a.N; };
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int e = e0 + v * 1024;
        if (in_dw(e)) o[v] = *reinterpret_cast<const float4*>(Cg + (int64_t)(m0 + e / BN) * a.ldc + n0 + e % BN);
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int e = e0 + v * 1024;
        if (!in_dw(e)) continue;
        o[v].x += s[v].x;
        o[v].y += s[v].y;
        o[v].z += s[v].z;
        o[v].w += s[v].w;
        *reinterpret_cast<float4*>(Cg + (int64_t)(m0 + e / BN) * a.ldc + n0 + e % BN) = o[v];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
int persistent_grid() { return num_cus(); }

// Launches the row GEMMs set in a.phases. e0, e1: optional timing events set
// when the kernel starts and ends (they ride on the dispatch itself, so no
// event command sits in the stream).
template <bool FWD>
void launch_rows(FfnArgs a, void* ws, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const int G = persistent_grid();
  if (ws && rows_workspace_fits(G)) {
    a.arrived = (unsigned*)((char*)ws + kRowsArrivedOff);
    a.queue = (unsigned*)((char*)ws + kRowsQueueOff);
    a.row_done = (unsigned*)((char*)ws + kRowsDoneOff);
    a.part = (float*)((char*)ws + kRowsPartOff);
  }
  // both GEMMs in one launch: the counters must hold every row tile, and two
  // row tiles must not share a 128-byte line of the rows handed over (a
  // workgroup that read one row tile would keep a stale copy of the next
  // one's first bytes)
  const bool pair = a.queue && a.n_cap / 256 + a.S <= kMaxRowTiles && ((uintptr_t)a.p[0].C & 127) == 0;
  if (a.phases == 3 && !pair) {
    FfnArgs b = a;
    b.phases = 1;
    hipExtLaunchKernelGGL(gemm_rows_kernel<FWD>, dim3(G), dim3(512), 0, st, e0, nullptr, 0, b);
    a.phases = 2;
    e0 = nullptr;
  }
  hipExtLaunchKernelGGL(gemm_rows_kernel<FWD>, dim3(G), dim3(512), 0, st, e0, e1, 0, a);
}

// Weight-gradient workspace: a 256-byte header of work counters, then the
// partial-tile budget of the split (tiles of 256 x 256 fp32).
constexpr size_t kWgradHeaderBytes = 256;
constexpr size_t kWgradPlanBytes = 16384;  // the exported plan: 2 + 3 * FOREMOE_MAX_SLOTS ints
constexpr size_t kWgradPartialTiles = 256;
constexpr size_t kWgradWorkspaceBytes = kWgradHeaderBytes + kWgradPlanBytes + kWgradPartialTiles * 256 * 256 * 4;
static_assert((2 + 3 * FOREMOE_MAX_SLOTS) * 4 <= kWgradPlanBytes, "plan export region");

}  // namespace
}  // namespace foremoe

using namespace foremoe;

#define REQUIRE(cond, ...)                                      \
  do {                                                          \
    if (!(cond)) return set_error(FOREMOE_EINVAL, __VA_ARGS__); \
  } while (0)

static int check_ffn(const char* who, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S, int64_t n_cap,
                     const int32_t* slot_offset) {
  REQUIRE(dtype == FOREMOE_F32 || dtype == FOREMOE_BF16, "%s: bad dtype", who);
  REQUIRE(d >= 1 && F >= 1, "%s: d and F must be positive", who);
  REQUIRE(S >= 0 && S <= FOREMOE_MAX_SLOTS, "%s: S=%d out of range", who, S);
  REQUIRE(n_cap >= 0 && n_cap < (int64_t)INT_MAX, "%s: n_cap out of range", who);
  REQUIRE(slot_offset, "%s: slot_offset is NULL", who);
  if (dtype == FOREMOE_BF16 && (d % 128 != 0 || F % 128 != 0))
    return set_error(FOREMOE_EUNSUPPORTED, "%s: bf16 needs d %% 128 == 0 and F %% 128 == 0 (d=%d, F=%d)", who, d, F);
  // 32-bit buffer offsets: (rows of one slot + one tile) * row bytes must fit
  if (dtype == FOREMOE_BF16 && (n_cap + 256) * (int64_t)(d > 2 * F ? d : 2 * F) * 2 >= ((int64_t)1 << 32))
    return set_error(FOREMOE_EUNSUPPORTED, "%s: (n_cap + 256) * row bytes must stay below 4 GiB", who);
  return FOREMOE_OK;
}

static int check_rows_ws(const char* who, const void* workspace, size_t ws_bytes) {
  if (!workspace) return FOREMOE_OK;
  REQUIRE(((uintptr_t)workspace & 255) == 0, "%s: workspace must be 256-byte aligned", who);
  const size_t need = rows_workspace_bytes(persistent_grid());
  REQUIRE(ws_bytes >= need, "%s: workspace of %zu bytes, %zu needed", who, ws_bytes, need);
  return FOREMOE_OK;
}

// A timed call that launches nothing still sets its events, back to back on
// the stream, so that their elapsed time reads as zero.
static int no_launch(hipEvent_t e0, hipEvent_t e1, void* stream) {
  if (!e0 && !e1) return FOREMOE_OK;
  if (e0 && hipEventRecord(e0, (hipStream_t)stream) != hipSuccess)
    return set_error(FOREMOE_EHIP, "row GEMM: recording the start event failed");
  if (e1 && hipEventRecord(e1, (hipStream_t)stream) != hipSuccess)
    return set_error(FOREMOE_EHIP, "row GEMM: recording the stop event failed");
  return FOREMOE_OK;
}

extern "C" {

// The checks and the arguments of each row GEMM. `who` names the call;
// returns OK with *run = false when there is nothing to do.
struct RowsCall {
  foremoe_dtype dtype;
  int32_t d, F, S;
  const int32_t* slot_offset;
  const int32_t* slot_widx;
  int32_t W;
  int64_t n_cap;
  void* workspace;
  size_t ws_bytes;
};

static int check_rows(const char* who, const RowsCall& c, bool* run) {
  int rc = check_ffn(who, c.dtype, c.d, c.F, c.S, c.n_cap, c.slot_offset);
  if (rc) return rc;
  rc = check_rows_ws(who, c.workspace, c.ws_bytes);
  if (rc) return rc;
  *run = c.S != 0 && c.n_cap != 0;
  return FOREMOE_OK;
}

static FfnArgs ffn_args(const RowsCall& c, int phases) {
  FfnArgs a{};
  a.phases = phases;
  a.W = c.W;
  a.slot_offset = c.slot_offset;
  a.slot_widx = c.slot_widx;
  a.S = c.S;
  a.n_cap = c.n_cap;
  return a;
}

static F32RowsArgs f32_args(const RowsCall& c, const void* A, const void* W, const void* AU, void* C, void* C2) {
  return {(const float*)A, (const float*)W, (const float*)AU, c.d, c.F, c.W, c.slot_offset, c.slot_widx, c.S, c.n_cap,
          (float*)C, (float*)C2};
}

static RowsArgs gate_up_fwd_args(const RowsCall& c, const void* x_perm, const void* w_gate_up, void* h,
                                 void* save_au) {
  RowsArgs a{};
  a.A = (const uint16_t*)x_perm;
  a.lda = c.d;
  a.B = (const uint16_t*)w_gate_up;
  a.ldb = c.d;
  a.wstride = (int64_t)2 * c.F * c.d;
  a.K = c.d;
  a.N = 2 * c.F;
  a.F = c.F;
  a.C = (uint16_t*)h;
  a.ldc = c.F;
  a.C2 = (uint16_t*)save_au;
  a.ldc2 = 2 * (int64_t)c.F;
  return a;
}

static RowsArgs down_fwd_args(const RowsCall& c, const void* h, const void* w_down, void* y_perm) {
  RowsArgs a{};
  a.A = (const uint16_t*)h;
  a.lda = c.F;
  a.B = (const uint16_t*)w_down;
  a.ldb = c.F;
  a.wstride = (int64_t)c.d * c.F;
  a.K = c.F;
  a.N = c.d;
  a.F = c.F;
  a.C = (uint16_t*)y_perm;
  a.ldc = c.d;
  return a;
}

static RowsArgs down_dgrad_args(const RowsCall& c, const void* dy_perm, const void* save_au, const void* w_down,
                                void* d_au) {
  RowsArgs a{};
  a.A = (const uint16_t*)dy_perm;
  a.lda = c.d;
  a.B = (const uint16_t*)w_down;  // [d, F]: K-major for this product
  a.ldb = c.F;
  a.wstride = (int64_t)c.d * c.F;
  a.K = c.d;
  a.N = c.F;
  a.F = c.F;
  a.C = (uint16_t*)d_au;
  a.ldc = 2 * (int64_t)c.F;
  a.AU = (const uint16_t*)save_au;
  a.ldau = 2 * (int64_t)c.F;
  return a;
}

static RowsArgs gate_up_dgrad_args(const RowsCall& c, const void* d_au, const void* w_gate_up, void* dx_perm) {
  RowsArgs a{};
  a.A = (const uint16_t*)d_au;
  a.lda = 2 * (int64_t)c.F;
  a.B = (const uint16_t*)w_gate_up;  // [2F, d]: K-major for this product
  a.ldb = c.d;
  a.wstride = (int64_t)2 * c.F * c.d;
  a.K = 2 * c.F;
  a.N = c.d;
  a.F = c.F;
  a.C = (uint16_t*)dx_perm;
  a.ldc = c.d;
  return a;
}

static int ffn_gate_up_fwd_impl(const void* x_perm, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                                const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                                const void* w_gate_up, int64_t n_cap, void* h, void* save_au, void* workspace,
                                size_t ws_bytes, void* stream, hipEvent_t e0, hipEvent_t e1) {
  const RowsCall c{dtype, d, F, S, slot_offset, slot_widx, W, n_cap, workspace, ws_bytes};
  bool run = false;
  const int rc = check_rows("gate_up_fwd", c, &run);
  if (rc) return rc;
  if (!run) return no_launch(e0, e1, stream);
  REQUIRE(x_perm && slot_widx && w_gate_up && h && W >= 1, "gate_up_fwd: NULL buffer or W < 1");
  if (dtype == FOREMOE_BF16) {
    FfnArgs a = ffn_args(c, 1);
    a.p[0] = gate_up_fwd_args(c, x_perm, w_gate_up, h, save_au);
    launch_rows<true>(a, workspace, (hipStream_t)stream, e0, e1);
  } else {
    launch_f32_rows(kF32GateUpFwd, f32_args(c, x_perm, w_gate_up, nullptr, h, save_au), (hipStream_t)stream, e0, e1);
  }
  return check_launch("foremoe_ffn_gate_up_fwd");
}

static int ffn_down_fwd_impl(const void* h, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                             const int32_t* slot_offset, const int32_t* slot_widx, int32_t W, const void* w_down,
                             int64_t n_cap, void* y_perm, void* workspace, size_t ws_bytes, void* stream,
                             hipEvent_t e0, hipEvent_t e1) {
  const RowsCall c{dtype, d, F, S, slot_offset, slot_widx, W, n_cap, workspace, ws_bytes};
  bool run = false;
  const int rc = check_rows("down_fwd", c, &run);
  if (rc) return rc;
  if (!run) return no_launch(e0, e1, stream);
  REQUIRE(h && slot_widx && w_down && y_perm && W >= 1, "down_fwd: NULL buffer or W < 1");
  if (dtype == FOREMOE_BF16) {
    FfnArgs a = ffn_args(c, 2);
    a.p[1] = down_fwd_args(c, h, w_down, y_perm);
    launch_rows<true>(a, workspace, (hipStream_t)stream, e0, e1);
  } else {
    launch_f32_rows(kF32DownFwd, f32_args(c, h, w_down, nullptr, y_perm, nullptr), (hipStream_t)stream, e0, e1);
  }
  return check_launch("foremoe_ffn_down_fwd");
}

int foremoe_grouped_ffn_fwd(const void* x_perm, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                            const int32_t* slot_offset, const int32_t* slot_widx, int32_t W, const void* w_gate_up,
                            const void* w_down, int64_t n_cap, void* h, void* y_perm, void* save_au, void* workspace,
                            size_t ws_bytes, void* stream) {
  const RowsCall c{dtype, d, F, S, slot_offset, slot_widx, W, n_cap, workspace, ws_bytes};
  bool run = false;
  const int rc = check_rows("grouped_ffn_fwd", c, &run);
  if (rc || !run) return rc;
  REQUIRE(x_perm && slot_widx && w_gate_up && w_down && h && y_perm && W >= 1,
          "grouped_ffn_fwd: NULL buffer or W < 1");
  if (dtype == FOREMOE_BF16) {
    FfnArgs a = ffn_args(c, 3);
    a.p[0] = gate_up_fwd_args(c, x_perm, w_gate_up, h, save_au);
    a.p[1] = down_fwd_args(c, h, w_down, y_perm);
    launch_rows<true>(a, workspace, (hipStream_t)stream, nullptr, nullptr);
  } else {
    const hipStream_t st = (hipStream_t)stream;
    launch_f32_rows(kF32GateUpFwd, f32_args(c, x_perm, w_gate_up, nullptr, h, save_au), st, nullptr, nullptr);
    launch_f32_rows(kF32DownFwd, f32_args(c, h, w_down, nullptr, y_perm, nullptr), st, nullptr, nullptr);
  }
  return check_launch("foremoe_grouped_ffn_fwd");
}

static int ffn_down_dgrad_impl(const void* dy_perm, const void* save_au, foremoe_dtype dtype, int32_t d, int32_t F,
                               int32_t S, const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                               const void* w_down, int64_t n_cap, void* d_au, void* workspace, size_t ws_bytes,
                               void* stream, hipEvent_t e0, hipEvent_t e1) {
  const RowsCall c{dtype, d, F, S, slot_offset, slot_widx, W, n_cap, workspace, ws_bytes};
  bool run = false;
  const int rc = check_rows("down_dgrad", c, &run);
  if (rc) return rc;
  if (!run) return no_launch(e0, e1, stream);
  REQUIRE(dy_perm && save_au && slot_widx && w_down && d_au && W >= 1, "down_dgrad: NULL buffer or W < 1");
  if (dtype == FOREMOE_BF16) {
    FfnArgs a = ffn_args(c, 1);
    a.p[0] = down_dgrad_args(c, dy_perm, save_au, w_down, d_au);
    launch_rows<false>(a, workspace, (hipStream_t)stream, e0, e1);
  } else {
    launch_f32_rows(kF32DownDgrad, f32_args(c, dy_perm, w_down, save_au, d_au, nullptr), (hipStream_t)stream, e0, e1);
  }
  return check_launch("foremoe_ffn_down_dgrad");
}

static int ffn_gate_up_dgrad_impl(const void* d_au, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                                  const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                                  const void* w_gate_up, int64_t n_cap, void* dx_perm, void* workspace,
                                  size_t ws_bytes, void* stream, hipEvent_t e0, hipEvent_t e1) {
  const RowsCall c{dtype, d, F, S, slot_offset, slot_widx, W, n_cap, workspace, ws_bytes};
  bool run = false;
  const int rc = check_rows("gate_up_dgrad", c, &run);
  if (rc) return rc;
  if (!run) return no_launch(e0, e1, stream);
  REQUIRE(d_au && slot_widx && w_gate_up && dx_perm && W >= 1, "gate_up_dgrad: NULL buffer or W < 1");
  if (dtype == FOREMOE_BF16) {
    FfnArgs a = ffn_args(c, 2);
    a.p[1] = gate_up_dgrad_args(c, d_au, w_gate_up, dx_perm);
    launch_rows<false>(a, workspace, (hipStream_t)stream, e0, e1);
  } else {
    launch_f32_rows(kF32GateUpDgrad, f32_args(c, d_au, w_gate_up, nullptr, dx_perm, nullptr), (hipStream_t)stream, e0,
                    e1);
  }
  return check_launch("foremoe_ffn_gate_up_dgrad");
}

int foremoe_ffn_gate_up_fwd(const void* x_perm, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                            const int32_t* slot_offset, const int32_t* slot_widx, int32_t W, const void* w_gate_up,
                            int64_t n_cap, void* h, void* save_au, void* workspace, size_t ws_bytes, void* stream) {
  return ffn_gate_up_fwd_impl(x_perm, dtype, d, F, S, slot_offset, slot_widx, W, w_gate_up, n_cap, h, save_au,
                              workspace, ws_bytes, stream, nullptr, nullptr);
}

int foremoe_ffn_gate_up_fwd_timed(const void* x_perm, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                                  const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                                  const void* w_gate_up, int64_t n_cap, void* h, void* save_au, void* workspace,
                                  size_t ws_bytes, void* stream, void* start_event, void* stop_event) {
  return ffn_gate_up_fwd_impl(x_perm, dtype, d, F, S, slot_offset, slot_widx, W, w_gate_up, n_cap, h, save_au,
                              workspace, ws_bytes, stream, (hipEvent_t)start_event, (hipEvent_t)stop_event);
}

int foremoe_ffn_down_fwd(const void* h, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                         const int32_t* slot_offset, const int32_t* slot_widx, int32_t W, const void* w_down,
                         int64_t n_cap, void* y_perm, void* workspace, size_t ws_bytes, void* stream) {
  return ffn_down_fwd_impl(h, dtype, d, F, S, slot_offset, slot_widx, W, w_down, n_cap, y_perm, workspace, ws_bytes,
                           stream, nullptr, nullptr);
}

int foremoe_ffn_down_fwd_timed(const void* h, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                               const int32_t* slot_offset, const int32_t* slot_widx, int32_t W, const void* w_down,
                               int64_t n_cap, void* y_perm, void* workspace, size_t ws_bytes, void* stream,
                               void* start_event, void* stop_event) {
  return ffn_down_fwd_impl(h, dtype, d, F, S, slot_offset, slot_widx, W, w_down, n_cap, y_perm, workspace, ws_bytes,
                           stream, (hipEvent_t)start_event, (hipEvent_t)stop_event);
}

int foremoe_ffn_down_dgrad(const void* dy_perm, const void* save_au, foremoe_dtype dtype, int32_t d, int32_t F,
                           int32_t S, const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                           const void* w_down, int64_t n_cap, void* d_au, void* workspace, size_t ws_bytes,
                           void* stream) {
  return ffn_down_dgrad_impl(dy_perm, save_au, dtype, d, F, S, slot_offset, slot_widx, W, w_down, n_cap, d_au,
                             workspace, ws_bytes, stream, nullptr, nullptr);
}

int foremoe_ffn_down_dgrad_timed(const void* dy_perm, const void* save_au, foremoe_dtype dtype, int32_t d, int32_t F,
                                 int32_t S, const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                                 const void* w_down, int64_t n_cap, void* d_au, void* workspace, size_t ws_bytes,
                                 void* stream, void* start_event, void* stop_event) {
  return ffn_down_dgrad_impl(dy_perm, save_au, dtype, d, F, S, slot_offset, slot_widx, W, w_down, n_cap, d_au,
                             workspace, ws_bytes, stream, (hipEvent_t)start_event, (hipEvent_t)stop_event);
}

int foremoe_ffn_gate_up_dgrad(const void* d_au, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                              const int32_t* slot_offset, const int32_t* slot_widx, int32_t W, const void* w_gate_up,
                              int64_t n_cap, void* dx_perm, void* workspace, size_t ws_bytes, void* stream) {
  return ffn_gate_up_dgrad_impl(d_au, dtype, d, F, S, slot_offset, slot_widx, W, w_gate_up, n_cap, dx_perm,
                                workspace, ws_bytes, stream, nullptr, nullptr);
}

int foremoe_ffn_gate_up_dgrad_timed(const void* d_au, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                                    const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                                    const void* w_gate_up, int64_t n_cap, void* dx_perm, void* workspace,
                                    size_t ws_bytes, void* stream, void* start_event, void* stop_event) {
  return ffn_gate_up_dgrad_impl(d_au, dtype, d, F, S, slot_offset, slot_widx, W, w_gate_up, n_cap, dx_perm,
                                workspace, ws_bytes, stream, (hipEvent_t)start_event, (hipEvent_t)stop_event);
}

int foremoe_grouped_ffn_dgrad(const void* dy_perm, const void* save_au, foremoe_dtype dtype, int32_t d, int32_t F,
                              int32_t S, const int32_t* slot_offset, const int32_t* slot_widx, int32_t W,
                              const void* w_gate_up, const void* w_down, int64_t n_cap, void* d_au, void* dx_perm,
                              void* workspace, size_t ws_bytes, void* stream) {
  const RowsCall c{dtype, d, F, S, slot_offset, slot_widx, W, n_cap, workspace, ws_bytes};
  bool run = false;
  const int rc = check_rows("grouped_ffn_dgrad", c, &run);
  if (rc || !run) return rc;
  REQUIRE(dy_perm && save_au && slot_widx && w_down && w_gate_up && d_au && dx_perm && W >= 1,
          "grouped_ffn_dgrad: NULL buffer or W < 1");
  if (dtype == FOREMOE_BF16) {
    FfnArgs a = ffn_args(c, 3);
    a.p[0] = down_dgrad_args(c, dy_perm, save_au, w_down, d_au);
    a.p[1] = gate_up_dgrad_args(c, d_au, w_gate_up, dx_perm);
    launch_rows<false>(a, workspace, (hipStream_t)stream, nullptr, nullptr);
  } else {
    const hipStream_t st = (hipStream_t)stream;
    launch_f32_rows(kF32DownDgrad, f32_args(c, dy_perm, w_down, save_au, d_au, nullptr), st, nullptr, nullptr);
    launch_f32_rows(kF32GateUpDgrad, f32_args(c, d_au, w_gate_up, nullptr, dx_perm, nullptr), st, nullptr, nullptr);
  }
  return check_launch("foremoe_grouped_ffn_dgrad");
}

// One weight-gradient GEMM over n steps' rows (every step: A [n_cap, M],
// B [n_cap, N], slot table), accumulated into dw [G, M, N].
static int wgrad_common(const char* who, const foremoe_wgrad_step* steps, int32_t n, int lda, int ldb, int M, int N,
                        foremoe_dtype dtype, int32_t G, int32_t part, int32_t parts, float* dw, void* ws,
                        size_t ws_bytes, void* stream) {
  REQUIRE(G >= 1 && G <= FOREMOE_MAX_SLOTS, "%s: G=%d out of range", who, G);
  REQUIRE(parts >= 1 && parts <= FOREMOE_MAX_WGRAD_STEPS && part >= 0 && part < parts,
          "%s: part %d of %d out of range", who, part, parts);
  REQUIRE(ws || ws_bytes == 0, "%s: ws is NULL but ws_bytes > 0", who);
  REQUIRE(n >= 0 && n <= FOREMOE_MAX_WGRAD_STEPS, "%s: n_steps=%d out of range", who, n);
  REQUIRE(n == 0 || steps, "%s: steps is NULL", who);
  int V = 0;
  bool any = false;
  for (int m = 0; m < n; ++m) {
    const foremoe_wgrad_step& t = steps[m];
    REQUIRE(t.S >= 0 && t.S <= FOREMOE_MAX_SLOTS, "%s: step %d: S=%d out of range", who, m, t.S);
    REQUIRE(t.n_cap >= 0 && t.n_cap < (int64_t)INT_MAX, "%s: step %d: n_cap out of range", who, m);
    if (t.S == 0 || t.n_cap == 0) continue;
    REQUIRE(t.a && t.b && t.slot_offset && t.slot_gidx, "%s: step %d: NULL buffer", who, m);
    if (dtype == FOREMOE_BF16 && (t.n_cap + 256) * (int64_t)(M > N ? M : N) * 2 >= ((int64_t)1 << 32))
      return set_error(FOREMOE_EUNSUPPORTED, "%s: step %d: (n_cap + 256) * row bytes must stay below 4 GiB", who, m);
    V += t.S;
    any = true;
  }
  REQUIRE(V <= FOREMOE_MAX_SLOTS, "%s: %d slots over all steps, at most %d", who, V, FOREMOE_MAX_SLOTS);
  if (!any) return FOREMOE_OK;
  REQUIRE(dw, "%s: NULL buffer", who);
  hipStream_t st = (hipStream_t)stream;
  if (dtype == FOREMOE_BF16) {
    WgradArgs a{};
    int v = 0;
    int64_t rows = 0;  // at most
    for (int m = 0; m < n; ++m) {
      const foremoe_wgrad_step& t = steps[m];
      if (t.S == 0 || t.n_cap == 0) continue;  // contributes nothing
      WgradStep& q = a.step[a.n_steps++];
      q.A = (const uint16_t*)t.a;
      q.B = (const uint16_t*)t.b;
      q.slot_offset = t.slot_offset;
      q.slot_gidx = t.slot_gidx;
      q.S = t.S;
      q.vbase = v;
      q.n_cap = t.n_cap;
      rows += t.n_cap;
      v += t.S;
    }
    a.V = v;
    a.tpart = part;
    a.tparts = parts;
    a.lda = lda;
    a.ldb = ldb;
    a.M = M;
    a.N = N;
    a.G = G;
    a.C = dw;
    a.ldc = N;
    a.gstride = (int64_t)M * N;
    // the workspace header holds the work counters; the rest partial tiles
    const bool has_ws = ws && ws_bytes >= kWgradHeaderBytes;
    const bool has_part = has_ws && ws_bytes >= kWgradHeaderBytes + kWgradPlanBytes;
    a.sched = has_ws ? (unsigned*)ws : nullptr;
    a.plan_out = has_part ? (int*)((char*)ws + kWgradHeaderBytes) : nullptr;
    a.part = has_part ? (float*)((char*)ws + kWgradHeaderBytes + kWgradPlanBytes) : nullptr;
    const size_t part_bytes = has_part ? ws_bytes - kWgradHeaderBytes - kWgradPlanBytes : 0;
    const dim3 grid(persistent_grid()), block(256);
    // 256 x 256 tiles. Where a dimension is an odd multiple of 128, too, with
    // half-empty last ones, if these make the work at most 1.6 times as much
    // and there is enough of it: 128 -> 256 tiles, both products, 12 groups of
    // 200 / 2000 / 16000 rows in all (us): d = 1152, F = 896 110 -> 94 /
    // 151 -> 122 / 291 -> 227; d = 640, F = 384 56 -> 62 / 94 -> 76 /
    // 135 -> 112; d = 384, F = 128 45 -> 47 / 58 -> 63 / 127 -> 130; d = F =
    // 128 (twice and four times the work) 41 -> 51 / 51 -> 64 / 126 -> 151. A
    // call for one part of several keeps the tile numbering of the interface,
    // which has 128 x 128 tiles there.
    const int64_t area = (int64_t)M * N, padded = (int64_t)((M + 255) / 256) * ((N + 255) / 256) * 65536;
    const bool odd_ok = parts == 1 && 5 * padded <= 8 * area && area >= 131072 && (area >= 1048576 || rows >= 1024);
    if ((M % 256 == 0 && N % 256 == 0) || odd_ok) {
      constexpr int WGM = FM_WG_WGM, WGN = FM_WG_WGN;
      a.p_max = (int)(part_bytes / (256 * 256 * 4));
      hipLaunchKernelGGL((gemm_wgrad_kernel<256, 256, FM_WG_BK, FM_WG_NS, WGM, WGN>), grid, dim3(64 * WGM * WGN), 0,
                         st, a);
      if (a.p_max > 0) hipLaunchKernelGGL((wgrad_reduce_kernel<256, 256, FM_WG_BK>), dim3(persistent_grid() * 4), block, 0, st, a);
    } else {
      a.p_max = (int)(part_bytes / (128 * 128 * 4));
      hipLaunchKernelGGL((gemm_wgrad_kernel<128, 128, 64, 3, 2, 2>), grid, block, 0, st, a);
      if (a.p_max > 0) hipLaunchKernelGGL((wgrad_reduce_kernel<128, 128, 64>), dim3(persistent_grid() * 4), block, 0, st, a);
    }
  } else {
    // fp32 path: one launch per step, in step order (each adds into dw);
    // a part is the rows m of dw with m % parts == part
    for (int m = 0; m < n; ++m) {
      const foremoe_wgrad_step& t = steps[m];
      if (t.S == 0 || t.n_cap == 0) continue;
      launch_f32_wgrad((const float*)t.a, lda, (const float*)t.b, ldb, M, N, t.slot_offset, t.slot_gidx, t.S, G,
                       t.n_cap, part, parts, dw, st);
    }
  }
  return check_launch(who);
}

static int check_wgrad_shape(const char* who, foremoe_dtype dtype, int32_t d, int32_t F) {
  REQUIRE(dtype == FOREMOE_F32 || dtype == FOREMOE_BF16, "%s: bad dtype", who);
  REQUIRE(d >= 1 && F >= 1, "%s: d and F must be positive", who);
  if (dtype == FOREMOE_BF16 && (d % 128 != 0 || F % 128 != 0))
    return set_error(FOREMOE_EUNSUPPORTED, "%s: bf16 needs d %% 128 == 0 and F %% 128 == 0 (d=%d, F=%d)", who, d, F);
  return FOREMOE_OK;
}

size_t foremoe_ffn_workspace_size(void) { return rows_workspace_bytes(persistent_grid()); }

size_t foremoe_wgrad_workspace_size(int32_t d, int32_t F) {
  if (d < 1 || F < 1) return 0;
  return kWgradWorkspaceBytes;
}

int foremoe_ffn_gate_up_wgrad_steps(const foremoe_wgrad_step* steps, int32_t n_steps, foremoe_dtype dtype,
                                    int32_t d, int32_t F, int32_t G, int32_t part, int32_t parts, float* dw_gate_up,
                                    void* ws, size_t ws_bytes, void* stream) {
  int rc = check_wgrad_shape("gate_up_wgrad", dtype, d, F);
  if (rc) return rc;
  return wgrad_common("foremoe_ffn_gate_up_wgrad", steps, n_steps, 2 * F, d, 2 * F, d, dtype, G, part, parts,
                      dw_gate_up, ws, ws_bytes, stream);
}

int foremoe_ffn_down_wgrad_steps(const foremoe_wgrad_step* steps, int32_t n_steps, foremoe_dtype dtype, int32_t d,
                                 int32_t F, int32_t G, int32_t part, int32_t parts, float* dw_down, void* ws,
                                 size_t ws_bytes, void* stream) {
  int rc = check_wgrad_shape("down_wgrad", dtype, d, F);
  if (rc) return rc;
  return wgrad_common("foremoe_ffn_down_wgrad", steps, n_steps, d, F, d, F, dtype, G, part, parts, dw_down, ws,
                      ws_bytes, stream);
}

int foremoe_ffn_gate_up_wgrad(const void* d_au, const void* x_perm, foremoe_dtype dtype, int32_t d, int32_t F,
                              int32_t S, const int32_t* slot_offset, const int32_t* slot_gidx, int32_t G,
                              int64_t n_cap, float* dw_gate_up, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_ffn("gate_up_wgrad", dtype, d, F, S, n_cap, slot_offset);
  if (rc) return rc;
  const foremoe_wgrad_step one = {d_au, x_perm, slot_offset, slot_gidx, S, n_cap};
  return foremoe_ffn_gate_up_wgrad_steps(&one, 1, dtype, d, F, G, 0, 1, dw_gate_up, ws, ws_bytes, stream);
}

int foremoe_ffn_down_wgrad(const void* dy_perm, const void* h, foremoe_dtype dtype, int32_t d, int32_t F, int32_t S,
                           const int32_t* slot_offset, const int32_t* slot_gidx, int32_t G, int64_t n_cap,
                           float* dw_down, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_ffn("down_wgrad", dtype, d, F, S, n_cap, slot_offset);
  if (rc) return rc;
  const foremoe_wgrad_step one = {dy_perm, h, slot_offset, slot_gidx, S, n_cap};
  return foremoe_ffn_down_wgrad_steps(&one, 1, dtype, d, F, G, 0, 1, dw_down, ws, ws_bytes, stream);
}

int foremoe_grouped_ffn_wgrad(const void* x_perm, const void* h, const void* dy_perm, const void* d_au,
                              foremoe_dtype dtype, int32_t d, int32_t F, int32_t S, const int32_t* slot_offset,
                              const int32_t* slot_gidx, int32_t G, int64_t n_cap, float* dw_gate_up, float* dw_down,
                              void* ws, size_t ws_bytes, void* stream) {
  int rc = foremoe_ffn_gate_up_wgrad(d_au, x_perm, dtype, d, F, S, slot_offset, slot_gidx, G, n_cap, dw_gate_up, ws,
                                     ws_bytes, stream);
  if (rc) return rc;
  return foremoe_ffn_down_wgrad(dy_perm, h, dtype, d, F, S, slot_offset, slot_gidx, G, n_cap, dw_down, ws, ws_bytes,
                                stream);
}

}  // extern "C"
