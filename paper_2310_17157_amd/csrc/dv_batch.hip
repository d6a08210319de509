// Batched decode, B <= 32 sequences with one token each (Section 5.2, Appendix C.1).
//
// With 32 tokens the gathered products become real dense contractions: every weight
// row fetched from HBM is used by all B tokens, so the work is done on the matrix
// cores (16x16x32 fp16 MFMA, fp32 accumulation) with the token batch as the N
// dimension, padded to NB = 16 or 32 with zero rows. The row sets are the union of
// the per-sequence sets (the union is what turns B sparse GEMVs into one sparse
// GEMM); each fetched row is read from HBM once per call.
//
//   k_union_*     union of B ascending index sets (chunked bitmaps, then ranks), and
//                 per-row membership bits of the sequences.
//   k_ln_cast     x-hat = LN(x) (or x) as fp16 in k-steps, zero padded.
//   k_rows        sum_k W[row(r)][k] x-hat[b][k]: gathered rows whose contraction index
//                 is contiguous in memory (fc1, Q/K/V, predictor factors). A workgroup's
//                 wavefronts split k, keep their part of x-hat in registers and apply
//                 the epilogue (bias, sigma, masks, cache writes) to the summed tiles.
//   k_mfma_cols   P2[s][b][n] = sum_{u in split s} C(b, u) M[row(u)][n]: gathered rows
//                 contracted over the row index (fc2, out-projection). Row tiles are
//                 written to a per-wavefront LDS tile (XOR-swizzled) and read back
//                 column-wise with the LDS transpose read into the B operand.
//   finishers     sum the split partials of k_mfma_cols in a fixed order with bias and
//                 residual; combine split-KV partials.
#include <math.h>

#include <type_traits>

#include "dv_internal.hpp"

namespace dv {

__device__ __forceinline__ f32x4 mfma16x16x32(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

typedef short v4s_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));

// gfx950 LDS transpose read of four 16-bit elements (p: 8-byte aligned LDS address).
__device__ __forceinline__ v4s_t ds_read_tr16(const _Float16* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (v4s_t __attribute__((address_space(3)))*)(const_cast<_Float16*>(p)));
}

// ------------------------------------------------------------------ union
// Union of B ascending sets sets[b][0..k) in [0, n) in one launch, one workgroup per
// chunk of kUnionChunk indices. Every workgroup reads all B * k entries (they stay
// in L2) and marks a byte per index below its chunk's end in LDS (plain stores, so
// entries shared by many sets do not contend); the members below the chunk give
// its offset, the marks inside it the ranks. U[offset + rank] = the members in
// ascending order, *count = their number (last chunk), and optionally
// mask[offset + rank] = the member's sets as bits (bit b: set b holds it), gathered
// by LDS atomics on one word per index of the chunk. Optionally also slot[b][i] = i's place
// in set b, or -1 (each workgroup for its chunk).
constexpr int kUnionChunk = 2048;
constexpr int kUnionNT = 1024;
static_assert(kUnionChunk == 2 * kUnionNT, "two indices of the chunk per thread");

// Calls fn(e, v) for every entry e of sets[0..total) with value v. The entries are
// read as aligned int4 with all of a thread's loads in flight (one round trip for up
// to PER * 4 * kUnionNT entries; rounds of loads past the end are not issued). sets
// need only be 4-byte aligned: the quads start at its 16-byte block, so the first and
// the last quad may reach up to 12 bytes outside [sets, sets + total). Those bytes share
// an aligned 16-byte block with an entry, and such a block never crosses a page (GPU
// pages are at least 4 KB), so they are readable; their values are skipped.
template <class Fn>
__device__ __forceinline__ void union_scan(const int32_t* __restrict__ sets, int total, Fn fn) {
  constexpr int PER = 16;
  if (total <= 0) return;
  const int shift = (int)(((uintptr_t)sets & 15u) >> 2);
  const int4* base = reinterpret_cast<const int4*>((uintptr_t)sets & ~(uintptr_t)15u);
  const int n4 = (total + shift + 3) >> 2;
  for (int q0 = 0; q0 < n4; q0 += PER * kUnionNT) {
    const int nu = min(PER, (n4 - q0 + kUnionNT - 1) / kUnionNT);   // rounds of quads left (workgroup-uniform)
    int4 v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u)
      v[u] = u < nu ? base[min(q0 + u * kUnionNT + (int)threadIdx.x, n4 - 1)] : make_int4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < PER; ++u) {   // quads of rounds not loaded have e >= total
      const int e = 4 * (q0 + u * kUnionNT + (int)threadIdx.x) - shift;
      if (e + 0 >= 0 && e + 0 < total) fn(e + 0, v[u].x);
      if (e + 1 >= 0 && e + 1 < total) fn(e + 1, v[u].y);
      if (e + 2 >= 0 && e + 2 < total) fn(e + 2, v[u].z);
      if (e + 3 >= 0 && e + 3 < total) fn(e + 3, v[u].w);
    }
  }
}

// Sum of four 0/1 bytes.
__device__ __forceinline__ int byte_flags(uint32_t w) { return (int)((w * 0x01010101u) >> 24); }

// Chunk c of nc; ush: dynamic LDS, marks [round_up(n, 16)] bytes, then (mask and slot only)
// kUnionChunk words.
template <bool MASK, bool SLOT>
__device__ __forceinline__ void union_chunk(const int32_t* __restrict__ sets, int B, int k, int n,
                                            int32_t* __restrict__ U, int32_t* __restrict__ count,
                                            uint32_t* __restrict__ mask, int32_t* __restrict__ slot, int c, int nc,
                                            uint32_t* ush) {
  __shared__ int red[kUnionNT / 64 + 1];
  const int tid = threadIdx.x;
  const int lo = c * kUnionChunk, hi = min(n, lo + kUnionChunk);
  const int n16 = (n + 15) & ~15;
  uint8_t* mk = reinterpret_cast<uint8_t*>(ush);
  uint32_t* mw = ush + n16 / 4;
  const int nq = ((hi + 15) & ~15) / 16;   // marks read below: [0, round_up(hi, 16))
  for (int q = tid; q < nq; q += kUnionNT) reinterpret_cast<uint4*>(mk)[q] = make_uint4(0u, 0u, 0u, 0u);
  constexpr bool words = MASK || SLOT;
  if (words)
    for (int i = tid; i < kUnionChunk; i += kUnionNT) mw[i] = 0u;
  __syncthreads();
  union_scan(sets, B * k, [&](int e, int v) {
    if ((unsigned)v < (unsigned)hi) {
      mk[v] = 1;
      if (words && v >= lo) {
        const int b = e / k;
        atomicOr(&mw[v - lo], 1u << b);
        if (SLOT) slot[(size_t)b * n + v] = e - b * k;
      }
    }
  });
  __syncthreads();
  // members before the chunk (lo is a multiple of 16)
  int part = 0;
  for (int q = tid; q < lo / 16; q += kUnionNT) {
    const uint4 w = reinterpret_cast<const uint4*>(mk)[q];
    part += byte_flags(w.x) + byte_flags(w.y) + byte_flags(w.z) + byte_flags(w.w);
  }
  int before = 0;
  (void)block_excl_scan<kUnionNT>(part, red, &before);
  // thread t ranks indices lo + 2t and lo + 2t + 1
  const int i0 = lo + 2 * tid;
  const int f0 = i0 < hi ? mk[i0] : 0, f1 = i0 + 1 < hi ? mk[i0 + 1] : 0;
  int in_chunk = 0;
  const int r = before + block_excl_scan<kUnionNT>(f0 + f1, red, &in_chunk);
  if (f0) {
    U[r] = i0;
    if (MASK) mask[r] = mw[i0 - lo];
  }
  if (f1) {
    U[r + f0] = i0 + 1;
    if (MASK) mask[r + f0] = mw[i0 + 1 - lo];
  }
  if (c == nc - 1 && tid == 0) *count = before + in_chunk;
  // the chunk's places that no entry has written, every thread some (each entry clearing the gap before
  // its own is a serial chain: 10.5 us for the launch at 32 sets of 2 of 96 heads against 7.2)
  if (SLOT)
    for (int e = tid; e < B * (hi - lo); e += kUnionNT) {
      const int b = e / (hi - lo), i = e - b * (hi - lo);
      if (!((mw[i] >> b) & 1u)) slot[(size_t)b * n + lo + i] = -1;
    }
}

template <bool MASK, bool SLOT>
__global__ void __launch_bounds__(kUnionNT) k_union(const int32_t* __restrict__ sets, int B, int k, int n,
                                                    int32_t* __restrict__ U, int32_t* __restrict__ count,
                                                    uint32_t* __restrict__ mask, int32_t* __restrict__ slot) {
  extern __shared__ __attribute__((aligned(16))) uint32_t ush[];
  union_chunk<MASK, SLOT>(sets, B, k, n, U, count, mask, slot, blockIdx.x, gridDim.x, ush);
}

// The kernel of a union without mask and slot, with mask, or with slot. (Chosen inside, the scan
// of 32 sets of 2457 without either took 2 us longer.)
template <class K>
static K union_form(const uint32_t* mask, const int32_t* slot, K none, K masked, K slotted) {
  return mask != nullptr ? masked : (slot != nullptr ? slotted : none);
}

size_t union_lds_bytes(int n) { return (size_t)((n + 15) & ~15) + (size_t)kUnionChunk * 4; }

hipError_t launch_union(const int32_t* sets, int B, int k, int n, int32_t* U, int32_t* count, uint32_t* mask,
                        int32_t* slot, hipStream_t st) {
  const int nc = (n + kUnionChunk - 1) / kUnionChunk;
  const size_t lds = union_lds_bytes(n);
  if (mask != nullptr && slot != nullptr) return hipErrorInvalidValue;
  const auto kern = union_form(mask, slot, k_union<false, false>, k_union<true, false>, k_union<false, true>);
  const hipError_t e = ensure_dyn_lds(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  launch_k(kern, dim3(nc), dim3(kUnionNT), lds, st, sets, B, k, n, U, count, mask, slot);
  return hipGetLastError();
}

// --------------------------------------------------------------- x-hat cast
// X16(b, 0..Kpad) = fp16(LN(x[b])) (g == NULL: x[b]) for b < B; zero for b >= B
// and for k >= d, in the layout of coef_index (a wavefront's B operand of one k-step is then
// contiguous). One workgroup per row b of NB; d % 4 == 0, so rows move as float4.
__device__ __forceinline__ void ln_cast_row(const float* __restrict__ x, int B, int d, int Kpad,
                                            const float* __restrict__ g, const float* __restrict__ be, float eps,
                                            _Float16* __restrict__ X16, int b, int NB) {
  __shared__ float red[16];
  const int n4 = d >> 2;
  if (b >= B) {
    for (int k = threadIdx.x; k < Kpad; k += 1024) X16[coef_index(b, k, NB)] = (_Float16)0.f;
    return;
  }
  const f32x4* xr = reinterpret_cast<const f32x4*>(x + (size_t)b * d);
  float mean = 0.f, rstd = 1.f;
  if (g != nullptr) {
    float sum = 0.f;
    for (int i = threadIdx.x; i < n4; i += 1024) {
      const f32x4 v = xr[i];
      sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
    mean = block_sum<1024>(sum, red) / (float)d;
    float q = 0.f;
    for (int i = threadIdx.x; i < n4; i += 1024) {
      const f32x4 v = xr[i];
      const float a0 = v[0] - mean, a1 = v[1] - mean, a2 = v[2] - mean, a3 = v[3] - mean;
      q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
    }
    rstd = 1.0f / sqrtf(block_sum<1024>(q, red) / (float)d + eps);
  }
  for (int i = threadIdx.x; i < (Kpad >> 2); i += 1024) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (i < n4) {
      v = xr[i];
      if (g != nullptr) {
        const f32x4 gg = reinterpret_cast<const f32x4*>(g)[i];
        const f32x4 bb = be ? reinterpret_cast<const f32x4*>(be)[i] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (v[e] - mean) * rstd * gg[e] + bb[e];
      }
    }
    typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
    f16x4 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (_Float16)v[e];
    *reinterpret_cast<f16x4*>(X16 + coef_index(b, 4 * i, NB)) = h;
  }
}

__global__ void __launch_bounds__(1024) k_ln_cast(const float* __restrict__ x, int B, int d, int Kpad,
                                                  const float* __restrict__ g, const float* __restrict__ be,
                                                  float eps, _Float16* __restrict__ X16) {
  ln_cast_row(x, B, d, Kpad, g, be, eps, X16, blockIdx.x, gridDim.x);
}

// The cast and the union of the batch's sets in one launch (they are independent):
// workgroups [0, NB) cast row b, the next nc take union chunk c.
template <bool MASK, bool SLOT>
__global__ void __launch_bounds__(1024) k_cast_union(const float* __restrict__ x, int B, int d, int Kpad,
                                                     const float* __restrict__ g, const float* __restrict__ be,
                                                     float eps, _Float16* __restrict__ X16, int NB,
                                                     const int32_t* __restrict__ sets, int k, int n,
                                                     int32_t* __restrict__ U, int32_t* __restrict__ count,
                                                     uint32_t* __restrict__ mask, int32_t* __restrict__ slot, int nc) {
  extern __shared__ __attribute__((aligned(16))) uint32_t ush[];
  if ((int)blockIdx.x < NB)
    ln_cast_row(x, B, d, Kpad, g, be, eps, X16, blockIdx.x, NB);
  else
    union_chunk<MASK, SLOT>(sets, B, k, n, U, count, mask, slot, (int)blockIdx.x - NB, nc, ush);
}

hipError_t launch_ln_cast(const float* x, int B, int NB, int d, int Kpad, const float* g, const float* be, float eps,
                          _Float16* X16, hipStream_t st) {
  launch_k(k_ln_cast, dim3(NB), dim3(1024), 0, st, x, B, d, Kpad, g, be, eps, X16);
  return hipGetLastError();
}

hipError_t launch_cast_union(const float* x, int B, int NB, int d, int Kpad, const float* g, const float* be,
                             float eps, _Float16* X16, const int32_t* sets, int k, int n, int32_t* U,
                             int32_t* count, uint32_t* mask, int32_t* slot, hipStream_t st) {
  static_assert(kUnionNT == 1024, "the cast and the union share the workgroup size");
  const int nc = (n + kUnionChunk - 1) / kUnionChunk;
  const size_t lds = union_lds_bytes(n);
  if (mask != nullptr && slot != nullptr) return hipErrorInvalidValue;
  const auto kern = union_form(mask, slot, k_cast_union<false, false>, k_cast_union<true, false>, k_cast_union<false, true>);
  const hipError_t e = ensure_dyn_lds(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  launch_k(kern, dim3(NB + nc), dim3(1024), lds, st, x, B, d, Kpad, g, be, eps, X16, NB, sets, k, n, U, count, mask, slot,
           nc);
  return hipGetLastError();
}

// ----------------------------------------------------------------- k_rows
// Gathered rows times the token batch, HBM-bound (a weight byte feeds 2 * NB / 2 flops). One
// workgroup per CU takes a contiguous, even share of the rows (to one row, whatever the
// count) over their whole length: its 8 wavefronts split the contraction index, so a
// wavefront reads its part of the inputs once from L2 into registers (B operands) and uses
// it for up to MT 16-row tiles, and the 8 partial sums are added through LDS, in wavefront
// order, by the threads that apply the epilogue (bias, sigma, cache writes, casts). Nothing
// is staged ahead of the stream, no split sum goes through memory and no finishing launch
// follows. Against K splits over workgroups with the input slice in LDS, partials in
// memory and a finishing launch (batch 32, OPT-175B shapes, us): QKV 146.5 + 11.7, fc1 of
// 24950 rows 107.6 + 6.8; batch 8 at the OPT-6.7B shapes, where whole groups of workgroups had
// no rows: predictor first layer 16.9 + 6.6, scores 22.4, QKV 24.9 + 4.9, fc1 19.2 + 4.5. This
// form: QKV 158, fc1 104; first layer 8.1, scores 11.2, QKV 22.5, fc1 12.9.
//
// Per tile, each load instruction fetches whole 128-byte lines (8 rows x 8 lanes x 16
// bytes): fetching the MFMA operand layout straight from memory (16 rows x 64 bytes per
// instruction) runs at about 70% of the bandwidth of whole-line loads. Each 64-element
// block of the tile's 16 rows is re-laid through a 2 KB per-wavefront LDS tile (16-byte
// chunk c of row r stored at c ^ (r & 7), conflict-free both ways) into the A operand: lane
// (lr, lg) takes row lr, chunk 4h + lg for k-step h of the block. A tile's reads go on for up to
// four blocks (512 bytes of a row) before the next tile's.
//
// XF32: the inputs stay fp32. A superblock of a token is scaled by a power of two to below
// 2^14 and split into three fp16 terms of 11 bits, the second held times 2^11 and the third times 2^22,
// so that an element down to 2^-23 after the scaling (2^-37 of the superblock's largest) is their sum
// exactly. Their products with the fp16 weights are exact; the fp32 sums over one
// superblock, one per term, are added in fp64. Two terms would lose a bit and a half against
// fp32, one fp32 sum over all superblocks another, and three terms under one scale would lose elements
// below 2^-14 of the largest one (at 10^8 under an element that meets zero weights, 2.6e-4 of the result,
// against 1.2e-7 here and 1.6e-7 in fp32 FMAs). Where a token still has smaller elements but zero, its
// rows are computed again in fp64 from the inputs as they are (rows_dot), and so are sums that are
// not finite: a term is zero where the input is not, and an infinite weight makes that NaN.
template <int MODE>
__device__ __forceinline__ int rows_count(const RowsSrc& s) {
  if constexpr (MODE == kRowsIdentity) {
    return s.nrows;
  } else {
    const int c = s.list_count ? min(*s.list_count, s.list_max) : s.list_max;
    return MODE == kRowsList ? c : 3 * c * s.dh;
  }
}

// The weight row of contraction row r (the list lookup and the divisions, once per tile):
// its index in W0 (list), or counted through W0, W1, W2 one after the other.
template <int MODE>
__device__ __forceinline__ int rows_id(const RowsSrc& s, int r, int n) {
  if constexpr (MODE == kRowsIdentity) {
    return r;
  } else if constexpr (MODE == kRowsList) {
    return min(max(s.list[r], 0), s.list_range - 1);
  } else {
    const int per = n / 3, m = r / per, rem = r - m * per, p = rem / s.dh;
    return m * s.n0 + min(max(s.list[p], 0), s.list_range - 1) * s.dh + (rem - p * s.dh);
  }
}
template <int MODE>
__device__ __forceinline__ const char* rows_addr(const RowsSrc& s, int id) {
  const size_t rowb = (size_t)s.d * 2;
  if constexpr (MODE == kRowsList) {
    return static_cast<const char*>(s.W0) + (size_t)id * rowb;
  } else if constexpr (MODE == kRowsIdentity) {
    return id < s.n0 ? static_cast<const char*>(s.W0) + (size_t)id * rowb
                     : static_cast<const char*>(s.W1) + (size_t)(id - s.n0) * rowb;
  } else {
    const void* W = id < s.n0 ? s.W0 : (id < 2 * s.n0 ? s.W1 : s.W2);
    const int o = id < s.n0 ? 0 : (id < 2 * s.n0 ? s.n0 : 2 * s.n0);
    return static_cast<const char*>(W) + (size_t)(id - o) * rowb;
  }
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// XF32: elements [k0, k1) of weight row id times token b, in fp64.
template <int MODE>
__device__ __forceinline__ float rows_dot(const RowsArgs& a, const RowsSrc& s, int id, int b, int k0, int k1) {
  const char* w = rows_addr<MODE>(s, id);
  const float* x = static_cast<const float*>(s.X) + (size_t)b * s.d;
  double v = 0.;
#pragma unroll 1
  for (int k = k0; k < k1; k += 8) {
    const f16x8 h = __builtin_bit_cast(f16x8, ld_plain(w + (size_t)k * 2));
    for (int e = 0; e < 8; ++e) {
      float xe = x[k + e];
      for (int p = 1; p < a.XP; ++p) xe += x[(size_t)p * a.B * s.d + k + e];
      v = fma((double)h[e], (double)xe, v);
    }
  }
  return (float)v;
}

// Epilogue of one value: row r (of n), token b.
template <int EPI, int NB, typename KT>
__device__ __forceinline__ void rows_epilogue(const RowsArgs& a, const RowsSrc& s, int r, int n, int b, int sp, float v) {
  if constexpr (EPI == kEpiFc1) {
    if (a.b1) v += a.b1[min(max(s.list[r], 0), s.list_range - 1)];
    v = act_apply(v, a.act);
    if (b >= a.B || (a.mask && !((a.mask[r] >> b) & 1u))) v = 0.f;
    a.C[coef_index(b, r, NB)] = (_Float16)v;
  } else if constexpr (EPI == kEpiQkv) {
    const int g = r / s.dh, t = r - g * s.dh, nu = n / 3 / s.dh, m = g / nu;
    const int h = min(max(s.list[g - m * nu], 0), s.list_range - 1);
    if (b >= a.B) return;
    const int jj = a.slot[b * s.list_range + h];   // h's place in the sequence's set, or -1
    if (jj < 0 || jj >= a.n_heads) return;
    const float* bias = m == 0 ? a.bq : (m == 1 ? a.bk : a.bv);
    if (bias) v += bias[(size_t)h * s.dh + t];
    if (m == 0) {
      a.q[((size_t)b * a.n_heads + jj) * s.dh + t] = v;
    } else {
      KT* Cc = static_cast<KT*>(m == 1 ? a.K : a.V);
      Cc[(((size_t)b * s.list_range + h) * a.cap + a.posb[b]) * s.dh + t] = (KT)v;
    }
  } else if constexpr (EPI == kEpiCoef) {   // the rows as the next contraction's fp16 inputs
    if (r < s.n0)
      a.C[coef_index(b, r, NB)] = (_Float16)v;
    else
      a.C1[coef_index(b, r - s.n0, NB)] = (_Float16)v;
  } else {
    if (b < a.B) s.out[(size_t)(sp * a.B + b) * s.nrows + r] = v;
  }
}

constexpr int kRowsNW = 8;
// Tiles per round of the sums through LDS.
template <int MT> constexpr int kRowsRT = MT < 5 ? MT : 5;
template <int NB, bool XF32, int MT>
constexpr size_t rows_lds() {
  return (size_t)kRowsNW * (16 * 64 * 2 + kRowsRT<MT> * 16 * (NB + 1) * (XF32 ? 8 : 4));
}

// MT: tiles a wavefront accumulates in registers at a time; SB: blocks of a superblock (a power
// of two); TB: tiles whose loads are in flight together.
template <int NB, int MODE, int EPI, bool XF32, typename KT, int MT, int SB, int TB>
__global__ void __launch_bounds__(kRowsNW * 64) k_rows(RowsArgs a) {
  constexpr int NW = kRowsNW, NT = NW * 64, NBT = NB / 16;
  constexpr int RT = kRowsRT<MT>;
  using Sum = std::conditional_t<XF32, double, float>;
  extern __shared__ __attribute__((aligned(16))) _Float16 rsm[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  _Float16* at = rsm + wave * (16 * 64);         // this wavefront's re-layout tile
  Sum* red = reinterpret_cast<Sum*>(rsm + NW * 16 * 64);   // [NW][RT][16][NB + 1]
  // workgroups [0, G0) take the first source's rows, the rest the second's
  constexpr bool TWO = EPI == kEpiOut && !XF32;
  const bool sec = TWO && (int)blockIdx.x >= a.G0;
  const RowsSrc& s = TWO ? a.src[sec ? 1 : 0] : a.src[0];
  const int S = XF32 ? a.S : 1, sp = XF32 ? (int)blockIdx.x % S : 0;   // split of the contraction
  // XF32: workgroups [0, G) take tokens [0, NB), the next G (S == 1) the tokens from NB
  const int b0 = XF32 && (int)blockIdx.x >= a.G0 ? NB : 0;
  const int wg = TWO ? (int)blockIdx.x - (sec ? a.G0 : 0) : (XF32 ? (int)blockIdx.x % a.G0 : (int)blockIdx.x) / S;
  const int G = TWO ? (sec ? (int)gridDim.x - a.G0 : a.G0) : (XF32 ? a.G0 : (int)gridDim.x) / S;
  if constexpr (EPI == kEpiQkv) {
    // the attention's coefficient matrix, before it writes its part
    if (a.zero != nullptr)
      for (int i = (int)blockIdx.x * NT + tid; i < a.zero_n / 8; i += (int)gridDim.x * NT)
        reinterpret_cast<u32x4*>(a.zero)[i] = u32x4{0u, 0u, 0u, 0u};
  }
  const int n = rows_count<MODE>(s);
  const int r0 = (int)((long)wg * n / G), r1 = (int)((long)(wg + 1) * n / G);
  const int nblk = (s.d + 63) >> 6;              // 64-element blocks of a row
  // (a contiguous part each: with superblocks dealt to the wavefronts in turn, QKV at batch
  // 32 took 172 us instead of 158)
  const int sb0 = sp * nblk / S, sbn = (sp + 1) * nblk / S - sb0;
  const int kb0 = sb0 + wave * sbn / NW, kb1 = sb0 + (wave + 1) * sbn / NW;
  const int dbytes = s.d * 2;
  const int cb = (lane & 7) * 16;                // this lane's 16 bytes of a 128-byte block
  const int rl0 = lane >> 3;                     // its rows of a tile: rl0 and rl0 + 8

  for (int c0 = r0; c0 < r1; c0 += 16 * MT) {
    const int T = min(MT, (r1 - c0 + 15) >> 4);
    int id0[MT], id1[MT];                        // (past the share: its last row again)
#pragma unroll
    for (int q = 0; q < MT; ++q) {
      id0[q] = rows_id<MODE>(s, min(c0 + 16 * q + rl0, r1 - 1), n);
      id1[q] = rows_id<MODE>(s, min(c0 + 16 * q + rl0 + 8, r1 - 1), n);
    }
    Sum acc[MT][NBT][4];
#pragma unroll
    for (int q = 0; q < MT; ++q)
#pragma unroll
      for (int j = 0; j < NBT; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[q][j][i] = 0;
    bool wide[NBT] = {};                         // XF32: elements the split does not hold exactly

    auto super = [&](auto blocks, int kb) {
      constexpr int NBLK = decltype(blocks)::value;
      constexpr int TERMS = XF32 ? 3 : 1;
      f16x8 bf[2 * NBLK][NBT][TERMS];
      float inv[NBT];
      auto load_w = [&](u32x4 (&w)[2 * NBLK], int q) {
        // (opaque, so that the addresses of all tiles are not kept in registers across superblocks)
        int i0 = id0[q], i1 = id1[q];
        asm volatile("" : "+v"(i0), "+v"(i1));
        const char* p0 = rows_addr<MODE>(s, i0);
        const char* p1 = rows_addr<MODE>(s, i1);
#pragma unroll
        for (int u = 0; u < 2 * NBLK; ++u) {
          const int off = (kb + (u >> 1)) * 128 + cb;          // (past the row: its last 16 bytes, then zeroed)
          w[u] = ld_stream(((u & 1) ? p1 : p0) + min(off, dbytes - 16));
        }
      };
      // XF32: the first tiles' weights are on their way while the inputs are split
      u32x4 wf[XF32 ? TB : 1][2 * NBLK];
      if constexpr (XF32) {
        f32x4 xv[2 * NBLK][NBT][2];
#pragma unroll
        for (int ks = 0; ks < 2 * NBLK; ++ks) {
          const int k = (2 * kb + ks) * 32 + 8 * lg;
#pragma unroll
          for (int j = 0; j < NBT; ++j) {
            const float* xp = static_cast<const float*>(s.X) + (size_t)min(b0 + lr + 16 * j, a.B - 1) * s.d + min(k, s.d - 8);
            xv[ks][j][0] = *reinterpret_cast<const f32x4*>(xp);
            xv[ks][j][1] = *reinterpret_cast<const f32x4*>(xp + 4);
            for (int p = 1; p < a.XP; ++p) {     // inputs given as parts (few): their sum
              const float* pp = xp + (size_t)p * a.B * s.d;
              xv[ks][j][0] += *reinterpret_cast<const f32x4*>(pp);
              xv[ks][j][1] += *reinterpret_cast<const f32x4*>(pp + 4);
            }
          }
        }
#pragma unroll
        for (int tt = 0; tt < TB; ++tt) load_w(wf[tt], tt);
#pragma unroll
        for (int j = 0; j < NBT; ++j) {
          float m = 0.f, least = INFINITY;
#pragma unroll
          for (int ks = 0; ks < 2 * NBLK; ++ks) {
            const bool in = (2 * kb + ks) * 32 + 8 * lg < s.d;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float v = in ? xv[ks][j][e >> 2][e & 3] : 0.f;
              xv[ks][j][e >> 2][e & 3] = v;
              m = fmaxf(m, fabsf(v));
              least = fminf(least, fabsf(v));
            }
          }
          m = fmaxf(m, __shfl_xor(m, 16, kWave));
          m = fmaxf(m, __shfl_xor(m, 32, kWave));
          // 2^(13 - floor(log2 m)), at most 2^126 (zeros and subnormals), from the exponent bits
          const int e2 = min(max(140 - (int)((__float_as_uint(m) >> 23) & 255u), -126), 126);
          const float sc = __uint_as_float((uint32_t)(e2 + 127) << 23);
          inv[j] = __uint_as_float((uint32_t)(127 - e2) << 23);
          if (__any(least < 0x1p-23f * inv[j])) {                // zeros, as a rule
#pragma unroll
            for (int ks = 0; ks < 2 * NBLK; ++ks)
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const float v = xv[ks][j][e >> 2][e & 3];
                wide[j] |= v != 0.f && fabsf(v) < 0x1p-23f * inv[j];
              }
          }
#pragma unroll
          for (int ks = 0; ks < 2 * NBLK; ++ks) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float v = xv[ks][j][e >> 2][e & 3] * sc;   // (infinities and NaN make NaN of the rest)
              const _Float16 hi = (_Float16)v;
              const float rest = fmaf((float)hi, -0x1p11f, v * 0x1p11f);
              const _Float16 mid = (_Float16)rest;
              bf[ks][j][0][e] = (_Float16)fmaf((float)mid, -0x1p11f, rest * 0x1p11f);
              bf[ks][j][TERMS - 2][e] = mid;
              bf[ks][j][TERMS - 1][e] = hi;
            }
            if constexpr (MT > 1) __builtin_amdgcn_sched_barrier(0);   // (terms made ahead spill)
          }
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < 2 * NBLK; ++ks)
#pragma unroll
          for (int j = 0; j < NBT; ++j)
            bf[ks][j][0] = __builtin_bit_cast(
                f16x8, ld_plain(static_cast<const _Float16*>(s.X) + coef_index(lr + 16 * j, (2 * kb + ks) * 32 + 8 * lg, NB)));
      }
      // N tiles from q0: their loads all in flight, then each re-laid and multiplied
      auto tiles = [&](auto count, int q0) {
        constexpr int N = decltype(count)::value;
        u32x4 w[N][2 * NBLK];
#pragma unroll
        for (int tt = 0; tt < N; ++tt) {
          if (XF32 && q0 + tt < TB) {
#pragma unroll
            for (int u = 0; u < 2 * NBLK; ++u) w[tt][u] = wf[XF32 ? q0 + tt : 0][u];
          } else {
            load_w(w[tt], q0 + tt);
          }
        }
#pragma unroll
        for (int tt = 0; tt < N; ++tt) {
          const int q = q0 + tt;
          f32x4 t[NBT], tm[NBT], tl[NBT];                      // (XF32: a sum per term)
#pragma unroll
          for (int j = 0; j < NBT; ++j) {
            tm[j] = tl[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (XF32) t[j] = tl[j];
            else t[j] = f32x4{acc[q][j][0], acc[q][j][1], acc[q][j][2], acc[q][j][3]};
          }
#pragma unroll
          for (int blk = 0; blk < NBLK; ++blk) {
            const bool in = (kb + blk) * 128 + cb < dbytes;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const int r = rl0 + 8 * i, c = lane & 7;
              *reinterpret_cast<u32x4*>(at + r * 64 + ((c ^ (r & 7)) << 3)) =
                  in ? w[tt][2 * blk + i] : u32x4{0u, 0u, 0u, 0u};
            }
            wave_lds_fence();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const f16x8 av = *reinterpret_cast<const f16x8*>(at + lr * 64 + (((4 * h + lg) ^ (lr & 7)) << 3));
#pragma unroll
              for (int j = 0; j < NBT; ++j) {
                if constexpr (XF32) {
                  tl[j] = mfma16x16x32(av, bf[2 * blk + h][j][0], tl[j]);
                  tm[j] = mfma16x16x32(av, bf[2 * blk + h][j][1], tm[j]);
                }
                t[j] = mfma16x16x32(av, bf[2 * blk + h][j][TERMS - 1], t[j]);
              }
            }
            wave_lds_fence();
          }
#pragma unroll
          for (int j = 0; j < NBT; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if constexpr (XF32)
                acc[q][j][i] += ((double)t[j][i] + (double)fmaf(tl[j][i], 0x1p-11f, tm[j][i]) * 0x1p-11) * (double)inv[j];
              else acc[q][j][i] = t[j][i];
            }
        }
      };
#pragma unroll
      for (int q0 = 0; q0 < MT; q0 += TB) {
        if (q0 + TB <= T && q0 + TB <= MT) {
          tiles(std::integral_constant<int, TB>{}, q0);
        } else if constexpr (TB > 1) {
#pragma unroll
          for (int q = q0; q < q0 + TB && q < MT; ++q)
            if (q < T) tiles(std::integral_constant<int, 1>{}, q);
        }
      }
    };
    int kb = kb0;
    for (; kb + SB <= kb1; kb += SB) super(std::integral_constant<int, SB>{}, kb);
    if constexpr (SB > 4)
      if (kb + 4 <= kb1) {
        super(std::integral_constant<int, 4>{}, kb);
        kb += 4;
      }
    if constexpr (SB > 2)
      if (kb + 2 <= kb1) {
        super(std::integral_constant<int, 2>{}, kb);
        kb += 2;
      }
    for (; kb < kb1; ++kb) super(std::integral_constant<int, 1>{}, kb);

    if constexpr (XF32)
#pragma unroll
      for (int j = 0; j < NBT; ++j) {
        int w = wide[j];
        w |= __shfl_xor(w, 16, kWave);
        w |= __shfl_xor(w, 32, kWave);
        if (w)
#pragma unroll
          for (int q = 0; q < MT; ++q) acc[q][j][0] = acc[q][j][1] = acc[q][j][2] = acc[q][j][3] = NAN;
      }
    // ---- the wavefronts' sums added in order, RT tiles at a time (lane: rows 4 lg + i,
    // tokens lr + 16 j of a tile)
#pragma unroll
    for (int t0 = 0; t0 < MT; t0 += RT) {
      if (t0 >= T) continue;
      __syncthreads();
#pragma unroll
      for (int q = t0; q < t0 + RT && q < MT; ++q)
#pragma unroll
        for (int j = 0; j < NBT; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            red[((wave * RT + (q - t0)) * 16 + 4 * lg + i) * (NB + 1) + lr + 16 * j] = acc[q][j][i];
      __syncthreads();
      for (int e = tid; e < min(RT, T - t0) * 16 * NB; e += NT) {
        const int rr = e & 15, bl = (e >> 4) % NB, q = (e >> 4) / NB, b = b0 + bl;
        const int r = c0 + 16 * (t0 + q) + rr;
        if (r >= r1) continue;
        Sum v = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[((w * RT + q) * 16 + rr) * (NB + 1) + bl];
        if constexpr (XF32)
          if (b < a.B && !(fabs(v) < INFINITY)) {
            int ro = r, bo = b;                        // (opaque: nothing of it is computed ahead)
            asm volatile("" : "+v"(ro), "+v"(bo));
            v = rows_dot<MODE>(a, s, rows_id<MODE>(s, ro, n), bo, sb0 * 64, min((sb0 + sbn) * 64, s.d));
          }
        rows_epilogue<EPI, NB, KT>(a, s, r, n, b, sp, (float)v);
      }
    }
  }
  // zero rows up to the next contraction's whole k-steps (by the last workgroup)
  if constexpr (EPI == kEpiFc1) {
    if (wg == G - 1) {
      const int pad = ((n + 31) & ~31) - n;
      for (int e = tid; e < pad * NB; e += NT) a.C[coef_index(e / pad, n + e % pad, NB)] = (_Float16)0.f;
    }
  }
  if constexpr (EPI == kEpiCoef) {
    if (wg == G - 1) {
      const int n1 = n - s.n0, p0 = ((s.n0 + 63) & ~63) - s.n0, p1 = ((n1 + 63) & ~63) - n1;
      for (int e = tid; e < p0 * NB; e += NT) a.C[coef_index(e / p0, s.n0 + e % p0, NB)] = (_Float16)0.f;
      if (a.C1 != nullptr)
        for (int e = tid; e < p1 * NB; e += NT) a.C1[coef_index(e / p1, n1 + e % p1, NB)] = (_Float16)0.f;
    }
  }
}

template <int NB, int MODE, int EPI, bool XF32, typename KT, int MT, int SB, int TB>
static hipError_t launch_rows_v(const RowsArgs& a, int G, hipStream_t st) {
  constexpr size_t lds = rows_lds<NB, XF32, MT>();
  const auto kern = k_rows<NB, MODE, EPI, XF32, KT, MT, SB, TB>;
  const hipError_t e = ensure_dyn_lds(reinterpret_cast<const void*>(kern), lds);
  if (e != hipSuccess) return e;
  launch_k(kern, dim3(G), dim3(kRowsNW * 64), lds, st, a);
  return hipGetLastError();
}

// Splits of the contraction of a fp32-input launch with few rows: 16-row tiles times splits
// fill the CUs once (every workgroup splits its part of the inputs itself, so workgroups of
// a few rows over the whole length would mostly repeat that: predictor of rank 1000, width
// 9216, 16 inputs, 26.8 us).
int rows_splits(int nrows) { return min(max(device_cu_count() / ((nrows + 15) / 16), 1), kRowsMaxSplit); }

template <int NB, int MODE, int EPI, bool XF32, typename KT>
static hipError_t launch_rows_t(RowsArgs a, hipStream_t st) {
  // one workgroup per CU; two sources share them by their rows' bytes
  const int G = max(device_cu_count(), 2);
  const double w0 = (double)a.src[0].nrows * a.src[0].d, w1 = (double)a.src[1].nrows * a.src[1].d;
  a.G0 = a.src[1].W0 == nullptr ? G : min(max((int)(G * w0 / (w0 + w1) + 0.5), 1), G - 1);
  if constexpr (XF32) {
    if (a.S > 1) {
      a.G0 = (a.src[0].nrows + 15) / 16 * a.S;
      return launch_rows_v<NB, MODE, EPI, XF32, KT, 1, NB == 16 ? 4 : 2, 1>(a, a.G0, st);
    }
    // Nine tiles with two tiles' loads in flight fill the registers (ten tiles, or loads of one or three,
    // spill). 17 to 32 inputs are two workgroups of 16 for each share of the rows, the second reading
    // them from L2: with all of them in one workgroup the registers hold two tiles and superblocks of one
    // block (32 inputs at the OPT-6.7B, 66B, 175B predictors, the whole call: 56, 117, 142 us; this way 37, 68, 87).
    a.S = 1;
    const int parts = (a.B + 15) / 16;
    a.G0 = G / parts;
    return launch_rows_v<16, MODE, EPI, XF32, KT, 9, 2, 2>(a, a.G0 * parts, st);
  } else {
    // few rows (to one tile per workgroup): one tile, longer superblocks. Otherwise two tiles'
    // loads in flight with 16 tokens (four spill: QKV of the OPT-6.7B heads 29.5 against 24.4 us), one
    // with 32 (two spill)
    if constexpr (MODE == kRowsIdentity)
      if (a.src[1].W0 == nullptr && a.src[0].nrows <= 16 * G)
        return launch_rows_v<NB, MODE, EPI, XF32, KT, 1, NB == 16 ? 8 : 4, 1>(a, G, st);
    // Gathered rows, at most four tiles per workgroup by the sets' sizes: few sums are held, and the
    // loads of all tiles (with 32 tokens of two) go together. Whole calls, the general form / this one, us:
    // 16 sequences with 2 of 72 heads of width 9216 75.4 / 74.1, 17 with one 64.4 / 60.8, 2 with 4 of 32 heads
    // of width 4096 40.1 / 37.6, 8 MLPs of 100 neurons of width 9216 30.4 / 28.8. (Superblocks of eight
    // instead: 72.3, 60.8, 38.3, 30.7.)
    if constexpr (MODE != kRowsIdentity) {
      const RowsSrc& s = a.src[0];
      const long most = MODE == kRowsHeads ? 3L * min(s.list_max, a.B * a.n_heads) * s.dh : (long)s.list_max;
      if (most <= 16L * 4 * G)
        return launch_rows_v<NB, MODE, EPI, XF32, KT, 4, 4, NB == 16 ? 4 : 2>(a, G, st);
    }
    return launch_rows_v<NB, MODE, EPI, XF32, KT, 10, 4, NB == 16 ? 2 : 1>(a, G, st);
  }
}

template <int NB>
static hipError_t launch_rows_nb(int epi, int kvtype, bool xf32, const RowsArgs& a, hipStream_t st) {
  switch (epi) {
    case kEpiFc1: return launch_rows_t<NB, kRowsList, kEpiFc1, false, float>(a, st);
    case kEpiQkv:
      return kvtype == DV_F16 ? launch_rows_t<NB, kRowsHeads, kEpiQkv, false, _Float16>(a, st)
                              : launch_rows_t<NB, kRowsHeads, kEpiQkv, false, float>(a, st);
    case kEpiCoef: return launch_rows_t<NB, kRowsIdentity, kEpiCoef, false, float>(a, st);
    default:
      return xf32 ? launch_rows_t<NB, kRowsIdentity, kEpiOut, true, float>(a, st)
                  : launch_rows_t<NB, kRowsIdentity, kEpiOut, false, float>(a, st);
  }
}

hipError_t launch_rows(int NB, int epi, int kvtype, bool xf32, const RowsArgs& a, hipStream_t st) {
  return NB <= 16 ? launch_rows_nb<16>(epi, kvtype, xf32, a, st) : launch_rows_nb<32>(epi, kvtype, xf32, a, st);
}

// ------------------------------------------------------------ k_mfma_cols
// Rows of the contraction: M[list[u]] (dh == 0) or M[list[u / dh] * dh + u % dh].
__device__ __forceinline__ int cols_count(const McolsArgs& a) {
  const int c = a.list_count ? min(*a.list_count, a.list_max) : a.list_max;
  return a.dh > 0 ? c * a.dh : c;
}
__device__ __forceinline__ size_t cols_row(const McolsArgs& a, int u) {
  if (a.dh == 0) return (size_t)min(max(a.list[u], 0), a.list_range - 1);
  const int p = u / a.dh;
  return (size_t)min(max(a.list[p], 0), a.list_range - 1) * a.dh + (u - p * a.dh);
}

// Wavefront tile in LDS: 32 rows x 64 columns fp16, 16-byte chunk c of row r stored at
// chunk c ^ (2 * ((r >> 3) & 3)) so that the row-wise 16-byte writes are free of bank
// conflicts and the four 8-row groups of a transpose read land in distinct banks.
//
// Load pipeline of a wavefront: the row indices of batch k+2, the weights and
// coefficients of batch k+1 and the MFMAs of batch k are in flight together. Indices
// are always loaded one batch before the weights that need them, so no wait for an
// index ever drains the weight loads behind it.
template <int NB, int U>
struct ColsStep {
  u32x4 w[U][4];        // weights: rows (lane >> 3) + 8*i, 16-byte chunk lane & 7
  u32x4 h[U][NB / 16];  // coefficients: token lr + 16*j, rows 8*lg .. 8*lg + 7
  unsigned ok;          // bit 4u + i: weight chunk w[u][i] is wanted (else written as 0)
};

// Row of M for contraction row `row` (clamped into [0, uend) so that every load is in
// bounds; rows past uend are zeroed after the load).
template <bool HEADS, int U>
__device__ __forceinline__ void mc_index(int (&ix)[U][4], const McolsArgs& a, int q0, int qstride, int uend,
                                         int lane) {
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = min(32 * (q0 + u * qstride) + (lane >> 3) + 8 * i, uend - 1);
      if (HEADS) {
        const int p = row / a.dh;
        ix[u][i] = min(max(a.list[p], 0), a.list_range - 1) * a.dh + (row - p * a.dh);
      } else {
        ix[u][i] = min(max(a.list[row], 0), a.list_range - 1);
      }
    }
}

template <int NB, int U>
__device__ __forceinline__ void mc_load(ColsStep<NB, U>& st, const int (&ix)[U][4], const McolsArgs& a,
                                        const char* Mb, int q0, int qstride, int uend, bool col_on, int lane) {
  const int lr = lane & 15, lg = lane >> 4;
  const size_t rowb = (size_t)a.d * 2;
  st.ok = 0u;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int q = min(q0 + u * qstride, (uend - 1) >> 5);     // clamped: loads stay in bounds
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 32 * (q0 + u * qstride) + (lane >> 3) + 8 * i;
      st.ok |= (col_on && row < uend) ? (1u << (4 * u + i)) : 0u;
      st.w[u][i] = ld_stream(Mb + (size_t)ix[u][i] * rowb);
    }
#pragma unroll
    for (int j = 0; j < NB / 16; ++j) st.h[u][j] = ld_plain(a.C + coef_index(lr + 16 * j, 32 * q + 8 * lg, NB));
  }
}

// WIDE: the wavefronts of a workgroup take adjacent 64-column tiles over the same rows
// (each row is then read in NW * 128 contiguous bytes, and the coefficients are shared
// through L1), and each writes its own partial tile. Otherwise they split the rows of
// one 64-column tile and are summed in LDS.
template <int NB, int NW, int U, bool HEADS, bool WIDE>
__global__ void __launch_bounds__(NW * 64) k_mfma_cols(McolsArgs a) {
  constexpr int NBT = NB / 16;
  extern __shared__ __attribute__((aligned(16))) _Float16 csm[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, lg = lane >> 4;
  _Float16* tile = csm + wave * (32 * 64);
  float* red = reinterpret_cast<float*>(csm + NW * 32 * 64);     // [NW][NB][64] (not WIDE)
  const int n0 = WIDE ? (blockIdx.x * NW + wave) * 64 : blockIdx.x * 64;
  const int s = blockIdx.y;
  const int n = cols_count(a);
  const int us = ((n + a.S - 1) / a.S + 31) & ~31;
  const int ubeg = s * us, uend = min(n, ubeg + us);
  const int qbeg = ubeg >> 5, qend = (uend + 31) >> 5;
  const bool col_on = n0 + 8 * (lane & 7) < a.d;
  const char* Mb = static_cast<const char*>(a.M) + (size_t)(col_on ? n0 + 8 * (lane & 7) : 0) * 2;

  f32x4 acc[NBT][4];
#pragma unroll
  for (int j = 0; j < NBT; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[j][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int qstride = WIDE ? 1 : NW;
  const int bstep = qstride * U;                 // k-steps per batch of this wavefront
  int q = WIDE ? qbeg : qbeg + wave;
  if (q < qend) {
    int ix0[U][4], ix1[U][4];
    mc_index<HEADS, U>(ix0, a, q, qstride, uend, lane);
    mc_index<HEADS, U>(ix1, a, q + bstep, qstride, uend, lane);
    ColsStep<NB, U> cur;
    mc_load<NB, U>(cur, ix0, a, Mb, q, qstride, uend, col_on, lane);
  for (; q < qend; q += bstep) {
    ColsStep<NB, U> nxt;
    const bool more = q + bstep < qend;
    // issued unconditionally (clamped in-bounds past the end, then discarded) so that
    // the waits below never have to drain them
    mc_index<HEADS, U>(ix0, a, q + 2 * bstep, qstride, uend, lane);          // batch k+2
    mc_load<NB, U>(nxt, ix1, a, Mb, q + bstep, qstride, uend, col_on, lane);  // batch k+1
    __builtin_amdgcn_sched_barrier(0);          // keep the prefetch ahead of the MFMAs
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (q + u * qstride >= qend) break;
      // row-wise write of the 32 x 64 tile
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = (lane >> 3) + 8 * i;
        const int c = (lane & 7) ^ (2 * i);
        *reinterpret_cast<u32x4*>(tile + r * 64 + c * 8) =
            ((cur.ok >> (4 * u + i)) & 1u) ? cur.w[u][i] : u32x4{0u, 0u, 0u, 0u};
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      f16x8 hv[NBT];
#pragma unroll
      for (int j = 0; j < NBT; ++j) hv[j] = __builtin_bit_cast(f16x8, cur.h[u][j]);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        // Column-wise B operand (lane (n = lr, g = lg) takes rows 8g .. 8g + 7 of column
        // 16t + n) with two LDS transpose reads. Within a 16-lane group the transpose
        // read hands lane i, slot j element i % 4 of the 4 elements that lane 4j + i/4
        // addressed, so lane s addresses row 8g + s/4 (+ 4 for the second read) at
        // columns 16t + 4 (s % 4) .. + 3.
        const int col = 16 * t + 4 * (lr & 3);
        v4s_t half[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const int r = 8 * lg + (lr >> 2) + 4 * hh;
          const int pc = (col >> 3) ^ (2 * ((r >> 3) & 3));
          half[hh] = ds_read_tr16(tile + r * 64 + pc * 8 + (col & 7));
        }
        const f16x8 bv = __builtin_shufflevector(__builtin_bit_cast(f16x4_t, half[0]),
                                                 __builtin_bit_cast(f16x4_t, half[1]), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int j = 0; j < NBT; ++j) acc[j][t] = mfma16x16x32(hv[j], bv, acc[j][t]);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (!more) break;
    cur = nxt;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) ix1[u][i] = ix0[u][i];
  }
  }
  if constexpr (WIDE) {
    // lane holds tokens 16j + 4lg + i of columns n0 + 16t + lr
#pragma unroll
    for (int j = 0; j < NBT; ++j)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int b = 16 * j + 4 * lg + i, c = n0 + 16 * t + lr;
          if (b < a.B && c < a.d) a.P[((size_t)s * a.B + b) * a.d + c] = acc[j][t][i];
        }
    return;
  }
  // ---- reduce the wavefronts' partials in a fixed order
#pragma unroll
  for (int j = 0; j < NBT; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[(wave * NB + 16 * j + 4 * lg + i) * 64 + 16 * t + lr] = acc[j][t][i];
  __syncthreads();
  for (int e = tid; e < NB * 64; e += NW * 64) {
    const int b = e >> 6, c = e & 63;
    if (b < a.B && n0 + c < a.d) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) v += red[(w * NB + b) * 64 + c];
      a.P[((size_t)s * a.B + b) * a.d + n0 + c] = v;
    }
  }
}

static constexpr int kMcNW = 8, kMcU = 1;
static constexpr bool kMcWide = true;

int mcols_split(int d, int nmax) {
  // one workgroup per CU: more splits only add partial-sum traffic (each split writes a
  // full B x d partial) and, past the CU count, a second round of workgroups (measured at
  // d = 12288: 10 splits 57 + 5 us out-proj, 32 splits 71 + 9 us)
  const int tiles = kMcWide ? (d + 64 * kMcNW - 1) / (64 * kMcNW) : (d + 63) / 64;
  int s = max(1, device_cu_count() / tiles);
  const int q = (nmax + 31) / 32;                  // k-steps available
  s = max(1, min(s, max(1, kMcWide ? q / 2 : q / (2 * kMcNW))));
  return min(s, 32);
}

template <int NB>
static hipError_t launch_mcols_t(const McolsArgs& a, hipStream_t st) {
  const size_t lds = (size_t)kMcNW * 32 * 64 * 2 + (kMcWide ? 0 : (size_t)kMcNW * NB * 64 * 4);
  dim3 grid(kMcWide ? (a.d + 64 * kMcNW - 1) / (64 * kMcNW) : (a.d + 63) / 64, a.S);
  if (a.dh > 0)
    launch_k((k_mfma_cols<NB, kMcNW, kMcU, true, kMcWide>), grid, dim3(kMcNW * 64), lds, st, a);
  else
    launch_k((k_mfma_cols<NB, kMcNW, kMcU, false, kMcWide>), grid, dim3(kMcNW * 64), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_mcols(int NB, const McolsArgs& a, hipStream_t st) {
  return NB <= 16 ? launch_mcols_t<16>(a, st) : launch_mcols_t<32>(a, st);
}

// --------------------------------------------------------------- finishers
// Four consecutive elements summed over the splits in split order; every split's load is issued before the
// first add, unpredicated (split index clamped, surplus not added).
__device__ __forceinline__ f32x4 sum_splits4(const float* __restrict__ P, int S, size_t stride, size_t e) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < S; s0 += 8) {
    f32x4 t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = *reinterpret_cast<const f32x4*>(P + (size_t)min(s0 + u, S - 1) * stride + e);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (s0 + u < S) v += t[u];
  }
  return v;
}

// Sum of k_mfma_cols partials: out[b][c] = sum_s P2[s][b][c] + bias[c] + resid[b][c];
// one thread per four columns (d % 4 == 0), every split's load in flight at once.
__global__ void __launch_bounds__(256) k_cols_finish(ColsFinishArgs a) {
  const long total = (long)a.B * a.d;
  const long e = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (e >= total) return;
  const int c = (int)(e % a.d);
  f32x4 v = sum_splits4(a.P, a.S, (size_t)total, (size_t)e);
  if (a.bias) v += *reinterpret_cast<const f32x4*>(a.bias + c);
  if (a.resid) v += *reinterpret_cast<const f32x4*>(a.resid + e);
  *reinterpret_cast<f32x4*>(a.out + e) = v;
}

hipError_t launch_cols_finish(const ColsFinishArgs& a, hipStream_t st) {
  const long quads = ((long)a.B * a.d / 4 + 255) / 256;
  launch_k(k_cols_finish, dim3((unsigned)max(1L, quads)), dim3(256), 0, st, a);
  return hipGetLastError();
}

// Attention outputs as out-projection coefficients: C(b, p*dh + t) = H_h(x_b)[t] for
// the union head h = list[p] if h is in sequence b's set (combining its split-KV
// partials), else 0; rows up to ldc are covered (zero beyond the union). C is in the
// layout of coef_index with gridDim.y (the padded token count) tokens.
__global__ void __launch_bounds__(256) k_attn_finish(AttnFinishArgs a) {
  __shared__ float fac[kAttnMaxSplit];
  __shared__ int jsel;
  const int p = blockIdx.x, b = blockIdx.y;
  const int nu = *a.hcount;
  const int r0 = p * a.dh;
  if (r0 >= a.ldc) return;
  const int rows = min(a.dh, a.ldc - r0);
  if (threadIdx.x == 0) {
    int jj = -1;
    if (p < nu && b < a.B) {
      const int h = a.list[p];   // union entries are in range by construction
      const int32_t* hs = a.heads + (size_t)b * a.n_heads;
      int lo = 0, hi = a.n_heads - 1;
      while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        if (hs[mid] == h) { jj = mid; break; }
        if (hs[mid] < h) lo = mid + 1; else hi = mid - 1;
      }
    }
    jsel = jj;
    if (jj >= 0) {
      const float* P = a.part + ((size_t)b * a.n_heads + jj) * a.n_split * (a.dh + 2);
      float M = -INFINITY;
      for (int c = 0; c < a.n_split; ++c) M = fmaxf(M, P[(size_t)c * (a.dh + 2)]);
      float L = 0.f;
      for (int c = 0; c < a.n_split; ++c) {
        const float m = P[(size_t)c * (a.dh + 2)];
        const float f = m == -INFINITY ? 0.f : __expf(m - M);
        fac[c] = f;
        L += P[(size_t)c * (a.dh + 2) + 1] * f;
      }
      for (int c = 0; c < a.n_split; ++c) fac[c] /= L;
    }
  }
  __syncthreads();
  const int jj = jsel;
  for (int t = threadIdx.x; t < rows; t += 256) {
    float v = 0.f;
    if (jj >= 0 && t < a.dh) {
      const float* P = a.part + ((size_t)b * a.n_heads + jj) * a.n_split * (a.dh + 2) + 2 + t;
      for (int c = 0; c < a.n_split; ++c) v += P[(size_t)c * (a.dh + 2)] * fac[c];
    }
    a.C[coef_index(b, r0 + t, gridDim.y)] = (_Float16)v;
  }
}

hipError_t launch_attn_finish(int NB, const AttnFinishArgs& a, hipStream_t st) {
  dim3 grid((a.ldc + a.dh - 1) / a.dh, NB);
  launch_k(k_attn_finish, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace dv
