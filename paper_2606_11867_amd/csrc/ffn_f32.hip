// Step 4 in fp32: the grouped SwiGLU FFN on fp32 tensors of any width (no
// divisibility, 4-byte alignment). Every product runs on the fp32 matrix
// cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation) in 32 x 32
// output tiles. A workgroup's four wavefronts split every 64-deep K slice
// between them (16 k each) and their partial sums meet in LDS in wavefront
// order; two slices are in flight in registers and two buffers in LDS.
//
// What bounds it: these shapes are small (tens of rows per slot, widths of a
// few hundred), so a launch is a handful of dependent K slices per tile, and
// their latency counts, not the fp32 matrix rate. Splitting K over the
// wavefronts quarters a tile's serial chain of matrix instructions; 64 x 64
// tiles with a quarter per wavefront and one slice in flight took 15-25 us
// where these take 8-12, and were no faster at the largest sizes measured
// (2048 tokens, widths of 500). One thread per output element, which this
// replaces, walked K alone through uncoalesced loads. Measured on 270 rows
// over 6 slots, d = 128, F = 256 (us, before -> now): gate/up forward
// 60 -> 9.5, down forward 34 -> 7.6, down dgrad 16 -> 8.0, gate/up dgrad
// 64 -> 12, both weight gradients 50 -> 18; a whole layer forward and
// backward of 2048 tokens, d = 256, F = 300: 2148 -> 184.
#include "ffn_f32.h"

#include <hip/hip_ext.h>

namespace foremoe {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;  // four wavefronts

constexpr int kTile = 32;      // output rows and columns per workgroup
constexpr int kDeep = 64;      // K slice: 16 k per wavefront
constexpr int kLd = kTile + 1;  // odd LDS row length: transposed stores hit all banks
constexpr int kPer = kTile * kDeep / kThreads;   // elements per thread and operand slice
constexpr int kSlice = kDeep * kLd;              // floats of a slice in LDS
constexpr int kOut = kTile * kTile / kThreads;   // outputs per thread

// One operand slice: kTile rows or columns x kDeep k values, held in LDS as
// [k][row]. KC: memory is contiguous along k (element (r, k) at r * ld + k),
// else along the row index (k * ld + r * rs). Elements outside
// [0, nr) x [0, nk) read as zero.
template <bool KC>
__device__ __forceinline__ void slice_load(const float* __restrict__ p, int64_t ld, int nr, int nk, float* v,
                                           int rs = 1) {
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int idx = threadIdx.x + kThreads * i;
    const int r = KC ? idx / kDeep : idx % kTile, k = KC ? idx % kDeep : idx / kTile;
    v[i] = (r < nr && k < nk) ? p[KC ? r * ld + k : k * ld + r * rs] : 0.f;
  }
}

template <bool KC>
__device__ __forceinline__ void slice_store(float* s, const float* v) {
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int idx = threadIdx.x + kThreads * i;
    const int r = KC ? idx / kDeep : idx % kTile, k = KC ? idx % kDeep : idx / kTile;
    s[k * kLd + r] = v[i];
  }
}

// acc += A B^T over this wavefront's 16 k of one slice: lane l feeds row
// (column) l % 32 of the tile at k + l / 32. Output register q of lane l is
// row 8 (q / 4) + 4 (l / 32) + q % 4, column l % 32.
__device__ __forceinline__ void slice_mfma(const float* sa, const float* sb, f32x16& acc) {
  const int l = threadIdx.x & 63, k0 = (threadIdx.x >> 6) * 16 + (l >> 5);
  const float* a = sa + k0 * kLd + (l & 31);
  const float* b = sb + k0 * kLd + (l & 31);
#pragma unroll
  for (int kk = 0; kk < 16; kk += 2)
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[kk * kLd], b[kk * kLd], acc, 0, 0, 0);
}

// This thread's outputs (rows out_row(i), column out_col() of the tile): the
// four wavefronts' partial sums added in wavefront order, through `red`.
__device__ __forceinline__ int out_row(int i) { return (int)(threadIdx.x >> 5) + 8 * i; }
__device__ __forceinline__ int out_col() { return (int)(threadIdx.x & 31); }
__device__ __forceinline__ void outputs(const f32x16& acc, float* red, float* out) {
  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();  // the slices (or an earlier sum) are no longer read
#pragma unroll
  for (int q = 0; q < 16; ++q)
    red[wave * 1024 + (8 * (q >> 2) + 4 * (l >> 5) + (q & 3)) * 32 + (l & 31)] = acc[q];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kOut; ++i) {
    const float* r = red + out_row(i) * 32 + out_col();
    out[i] = ((r[0] + r[1024]) + r[2048]) + r[3072];
  }
}

// The K slices of one tile: load(set) issues the next slice's loads into
// register set `set` and returns false past the last; store(set, buf) writes
// a set to LDS buffer buf; mul(buf) multiplies it. Two slices are in flight
// in registers and two buffers in LDS, so each slice costs one barrier and
// its loads have two slices' time to arrive.
template <class Load, class Store, class Mul>
__device__ __forceinline__ void k_slices(Load&& load, Store&& store, Mul&& mul) {
  bool v0 = load(0), v1 = v0 && load(1);
  while (v0) {
    store(0);
    v0 = v1 && load(0);
    __syncthreads();
    mul(0);
    if (!v1) break;
    store(1);
    v1 = v0 && load(1);
    __syncthreads();
    mul(1);
  }
}

__device__ __forceinline__ int64_t clamp_row(int32_t v, int64_t n_cap) {
  return v < 0 ? 0 : (v > n_cap ? n_cap : v);
}

// The slot and first row (relative to the slot) of row tile y; false past
// the last. All threads call it together.
__device__ bool find_row_tile(const int32_t* __restrict__ off, int S, int64_t n_cap, int y, int* s_tmp, int& slot,
                              int& row0) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int carry = 0;
  for (int j0 = 0; j0 < S; j0 += kThreads) {
    const int j = j0 + threadIdx.x;
    int n = 0;
    if (j < S) {
      const int64_t rows = clamp_row(off[j + 1], n_cap) - clamp_row(off[j], n_cap);
      n = rows > 0 ? (int)((rows + kTile - 1) / kTile) : 0;
    }
    int incl = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    if (lane == 63) s_tmp[w] = incl;
    __syncthreads();
    int before = carry, total = carry;
#pragma unroll
    for (int i = 0; i < kThreads / 64; ++i) {
      if (i < w) before += s_tmp[i];
      total += s_tmp[i];
    }
    const int first = before + incl - n;
    if (y >= first && y < first + n) {
      s_tmp[4] = j;
      s_tmp[5] = (y - first) * kTile;
    }
    __syncthreads();
    if (y < total) {
      slot = s_tmp[4];
      row0 = s_tmp[5];
      return true;
    }
    carry = total;
  }
  return false;
}

template <int OP>
__global__ __launch_bounds__(kThreads) void f32_rows_kernel(F32RowsArgs a) {
  constexpr bool kTwo = OP == kF32GateUpFwd;  // gate and up columns side by side
  constexpr bool kBKC = OP == kF32GateUpFwd || OP == kF32DownFwd;
  constexpr int kBuf = (kTwo ? 3 : 2) * kSlice;  // operand slices of one LDS buffer
  __shared__ float s_op[2 * kBuf];
  static_assert(2 * kBuf >= 4 * 1024, "the partial sums fit in the slices");
  __shared__ int s_tmp[6];
  const int d = a.d, F = a.F;
  const int K = OP == kF32DownFwd ? F : (OP == kF32GateUpDgrad ? 2 * F : d);
  const int ncols = (OP == kF32GateUpFwd || OP == kF32DownDgrad) ? F : d;
  const int64_t lda = K, ldb = kBKC ? K : ncols;
  const int n0 = blockIdx.x * kTile;
  for (int y = blockIdx.y;; y += gridDim.y) {
    int j, row0;
    if (!find_row_tile(a.off, a.S, a.n_cap, y, s_tmp, j, row0)) return;
    __syncthreads();  // s_tmp is free again, and so are the slices of the tile before
    const int w = a.widx[j];
    if (w < 0 || w >= a.W) continue;
    const int64_t r0 = clamp_row(a.off[j], a.n_cap) + row0;
    const int64_t left = clamp_row(a.off[j + 1], a.n_cap) - r0;
    const int nr = left < kTile ? (int)left : kTile;
    const int nc = ncols - n0 < kTile ? ncols - n0 : kTile;
    const float* A = a.A + r0 * lda;
    const float* B = a.Wt + (int64_t)w * ((OP == kF32GateUpFwd || OP == kF32GateUpDgrad) ? 2 : 1) * F * d +
                     (kBKC ? (int64_t)n0 * ldb : (int64_t)n0);
    const float* B2 = B + (int64_t)F * d;
    f32x16 acc = {}, acc2 = {};
    float va[2][kPer], vb[2][kPer], vb2[2][kTwo ? kPer : 1];
    int k0 = 0;
    k_slices(
        [&](int set) {
          if (k0 >= K) return false;
          slice_load<true>(A + k0, lda, nr, K - k0, va[set]);
          slice_load<kBKC>(B + (kBKC ? (int64_t)k0 : k0 * ldb), ldb, nc, K - k0, vb[set]);
          if constexpr (kTwo) slice_load<true>(B2 + k0, ldb, nc, K - k0, vb2[set]);
          k0 += kDeep;
          return true;
        },
        [&](int set) {
          float* s = s_op + set * kBuf;
          slice_store<true>(s, va[set]);
          slice_store<kBKC>(s + kSlice, vb[set]);
          if constexpr (kTwo) slice_store<true>(s + 2 * kSlice, vb2[set]);
        },
        [&](int set) {
          const float* s = s_op + set * kBuf;
          slice_mfma(s, s + kSlice, acc);
          if constexpr (kTwo) slice_mfma(s, s + 2 * kSlice, acc2);
        });
    float out[kOut], out2[kTwo ? kOut : 1];
    outputs(acc, s_op, out);
    if constexpr (kTwo) outputs(acc2, s_op, out2);
    const int col = n0 + out_col();
    if (col >= ncols) continue;
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
      const int r = out_row(i);
      if (r >= nr) continue;
      const int64_t row = r0 + r;
      if constexpr (OP == kF32GateUpFwd) {
        const float av = out[i], uv = out2[i];
        a.C[row * F + col] = av / (1.0f + __expf(-av)) * uv;
        if (a.C2) {
          a.C2[row * 2 * F + col] = av;
          a.C2[row * 2 * F + F + col] = uv;
        }
      } else if constexpr (OP == kF32DownDgrad) {
        const float av = a.AU[row * 2 * F + col], uv = a.AU[row * 2 * F + F + col];
        const float s = 1.0f / (1.0f + __expf(-av));
        a.C[row * 2 * F + col] = out[i] * uv * (s + av * s * (1.0f - s));
        a.C[row * 2 * F + F + col] = out[i] * av * s;
      } else {
        a.C[row * d + col] = out[i];
      }
    }
  }
}

// The K slices of one gradient group: the rows of every slot with index g,
// slots in order, kDeep rows at a time (a slice stays inside one slot).
// Wave-uniform; 64 slots' indices are compared at once.
struct GroupRows {
  const int32_t* off;
  const int32_t* gidx;
  int S, g;
  int64_t n_cap;
  int j0;         // first slot of the 64 in `match`
  uint64_t match;  // slots of this 64 not yet taken
  int64_t row, end;
  __device__ __forceinline__ void scan() {
    const int j = j0 + (threadIdx.x & 63);
    match = __ballot(j < S && gidx[j < S ? j : 0] == g);
  }
  __device__ __forceinline__ bool advance() {
    row += kDeep;
    while (row >= end) {
      while (!match) {
        j0 += 64;
        if (j0 >= S) return false;
        scan();
      }
      const int j = j0 + __builtin_ctzll(match);
      match &= match - 1;
      row = clamp_row(off[j], n_cap);
      end = clamp_row(off[j + 1], n_cap);
    }
    return true;
  }
  __device__ __forceinline__ int rows() const { return end - row < kDeep ? (int)(end - row) : kDeep; }
};

// dW[g][m][n] += sum over the group's rows r of A[r][m] B[r][n]; only the
// rows m with m % parts == part, row part + parts * i being the i-th of the
// tiles. Tiles of all rows, most of them dropped at the store, would do the
// whole product in each part. Both products in 16 parts, one after another:
// 64 groups, 4096 rows, d = 512, F = 768 5.9 -> 0.96 ms (undivided 0.51); one
// group of 2000 rows, d = F = 512, where a part is 32 tiles for 256 CUs,
// 1.26 -> 1.80.
__global__ __launch_bounds__(kThreads) void f32_wgrad_kernel(const float* __restrict__ A, int lda,
                                                             const float* __restrict__ B, int ldb, int M, int N,
                                                             const int32_t* __restrict__ off,
                                                             const int32_t* __restrict__ gidx, int S, int64_t n_cap,
                                                             int part, int parts, float* __restrict__ C) {
  constexpr int kBuf = 2 * kSlice;
  __shared__ float s_op[2 * kBuf];
  static_assert(2 * kBuf >= 4 * 1024, "the partial sums fit in the slices");
  const int n0 = blockIdx.x * kTile, m0 = blockIdx.y * kTile, g = blockIdx.z;
  const int n_rows = (M - part + parts - 1) / parts;  // of this part
  GroupRows it{off, gidx, S, g, n_cap, 0, 0, -kDeep, 0};
  it.scan();
  f32x16 acc = {};
  float va[2][kPer], vb[2][kPer];
  bool any = false;
  k_slices(
      [&](int set) {
        if (!it.advance()) return false;
        any = true;
        slice_load<false>(A + it.row * lda + part + (int64_t)m0 * parts, lda, n_rows - m0, it.rows(), va[set], parts);
        slice_load<false>(B + it.row * ldb + n0, ldb, N - n0, it.rows(), vb[set]);
        return true;
      },
      [&](int set) {
        slice_store<false>(s_op + set * kBuf, va[set]);
        slice_store<false>(s_op + set * kBuf + kSlice, vb[set]);
      },
      [&](int set) { slice_mfma(s_op + set * kBuf, s_op + set * kBuf + kSlice, acc); });
  if (!any) return;  // no rows: dW[g] stays as it is
  float out[kOut];
  outputs(acc, s_op, out);
  const int n = n0 + out_col();
  if (n >= N) return;
#pragma unroll
  for (int i = 0; i < kOut; ++i) {
    const int i_row = m0 + out_row(i);
    if (i_row < n_rows) C[((int64_t)g * M + part + (int64_t)i_row * parts) * N + n] += out[i];
  }
}

}  // namespace

void launch_f32_rows(int op, const F32RowsArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const int ncols = (op == kF32GateUpFwd || op == kF32DownDgrad) ? a.F : a.d;
  // every slot adds at most one ragged tile; the tile count is only known on
  // the device, so workgroups past the last tile leave at once
  int64_t tiles = a.n_cap / kTile + a.S;
  if (tiles > 65535) tiles = 65535;
  const dim3 grid((unsigned)((ncols + kTile - 1) / kTile), (unsigned)tiles), block(kThreads);
  switch (op) {
    case kF32GateUpFwd:
      hipExtLaunchKernelGGL(f32_rows_kernel<kF32GateUpFwd>, grid, block, 0, st, e0, e1, 0, a);
      break;
    case kF32DownFwd:
      hipExtLaunchKernelGGL(f32_rows_kernel<kF32DownFwd>, grid, block, 0, st, e0, e1, 0, a);
      break;
    case kF32DownDgrad:
      hipExtLaunchKernelGGL(f32_rows_kernel<kF32DownDgrad>, grid, block, 0, st, e0, e1, 0, a);
      break;
    default:
      hipExtLaunchKernelGGL(f32_rows_kernel<kF32GateUpDgrad>, grid, block, 0, st, e0, e1, 0, a);
  }
}

void launch_f32_wgrad(const float* A, int lda, const float* B, int ldb, int M, int N, const int32_t* off,
                      const int32_t* gidx, int S, int G, int64_t n_cap, int part, int parts, float* C,
                      hipStream_t st) {
  const int n_rows = M > part ? (M - part + parts - 1) / parts : 0;
  if (n_rows == 0) return;
  hipLaunchKernelGGL(f32_wgrad_kernel, dim3((N + kTile - 1) / kTile, (n_rows + kTile - 1) / kTile, G), dim3(kThreads),
                     0, st, A, lda, B, ldb, M, N, off, gidx, S, n_cap, part, parts, C);
}

}  // namespace foremoe
