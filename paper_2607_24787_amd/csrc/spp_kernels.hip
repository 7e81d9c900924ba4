// gfx950 kernels of the offloaded-MoE decode hot path.
//
// Lane layout shared by every row-dot kernel: a row of D elements is read as
// 16-byte chunks (8 bf16 or 4 fp32); lane l of a 64-wide wave owns chunks
// l, l+64, l+128, ... so one wave-wide load instruction moves 1 KiB of
// contiguous memory.  Loads are issued into raw registers first and unpacked
// only after every load of the step is in flight.  A row's dot product is the
// sum of per-lane partial sums followed by a DPP reduction across the wave
// whose result is bit-identical in every lane.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "spp_internal.h"

namespace spp {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kBStage = 8192;  // adapter B elements staged in LDS (n * r)

template <typename T>
struct Vec;
template <>
struct Vec<float> {
  static constexpr int N = 4;
};
template <>
struct Vec<uint16_t> {
  static constexpr int N = 8;
};

// Loads through global-address-space pointers: a generic pointer (e.g. one read
// back from LDS) would otherwise become a flat load, which also counts against
// the LDS counter and serialises unrelated waits.
#if defined(__HIP_DEVICE_COMPILE__)
#define SPP_GLOBAL(T, p) ((const __attribute__((address_space(1))) T*)(p))
#else
#define SPP_GLOBAL(T, p) (reinterpret_cast<const T*>(p))
#endif

__device__ __forceinline__ uint4 ld16(const void* p) { return *SPP_GLOBAL(uint4, p); }

template <typename T>
__device__ __forceinline__ void unpack(const uint4 r, float* f);
template <>
__device__ __forceinline__ void unpack<float>(const uint4 r, float* f) {
  f[0] = __uint_as_float(r.x);
  f[1] = __uint_as_float(r.y);
  f[2] = __uint_as_float(r.z);
  f[3] = __uint_as_float(r.w);
}
template <>
__device__ __forceinline__ void unpack<uint16_t>(const uint4 r, float* f) {
  f[0] = __uint_as_float(r.x << 16);
  f[1] = __uint_as_float(r.x & 0xffff0000u);
  f[2] = __uint_as_float(r.y << 16);
  f[3] = __uint_as_float(r.y & 0xffff0000u);
  f[4] = __uint_as_float(r.z << 16);
  f[5] = __uint_as_float(r.z & 0xffff0000u);
  f[6] = __uint_as_float(r.w << 16);
  f[7] = __uint_as_float(r.w & 0xffff0000u);
}

template <typename T>
__device__ __forceinline__ float load_elem(const void* p, size_t i);
template <>
__device__ __forceinline__ float load_elem<float>(const void* p, size_t i) {
  return reinterpret_cast<const float*>(p)[i];
}
template <>
__device__ __forceinline__ float load_elem<uint16_t>(const void* p, size_t i) {
  return __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(p)[i]) << 16);
}

template <typename T>
__device__ __forceinline__ void store_elem(void* p, size_t i, float v);
template <>
__device__ __forceinline__ void store_elem<float>(void* p, size_t i, float v) {
  reinterpret_cast<float*>(p)[i] = v;
}
template <>
__device__ __forceinline__ void store_elem<uint16_t>(void* p, size_t i, float v) {
  // round to nearest, ties to even
  uint32_t b = __float_as_uint(v);
  uint16_t o;
  if ((b & 0x7fffffffu) > 0x7f800000u) {
    o = 0x7fc0;  // NaN
  } else {
    b += 0x7fffu + ((b >> 16) & 1u);
    o = static_cast<uint16_t>(b >> 16);
  }
  reinterpret_cast<uint16_t*>(p)[i] = o;
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float v) {
  uint32_t b = __float_as_uint(v);
  if ((b & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
  b += 0x7fffu + ((b >> 16) & 1u);
  return static_cast<uint16_t>(b >> 16);
}

__device__ __forceinline__ uint32_t pack2(uint16_t lo, uint16_t hi) {
  return lo | (static_cast<uint32_t>(hi) << 16);
}

// x as a bf16 pair hi + lo (to 2^-17 of x), two values per word.
__device__ __forceinline__ void split2(float a, float b, uint32_t* hi, uint32_t* lo) {
  const uint16_t ha = f32_to_bf16_rne(a), hb = f32_to_bf16_rne(b);
  *hi = pack2(ha, hb);
  *lo = pack2(f32_to_bf16_rne(a - __uint_as_float(static_cast<uint32_t>(ha) << 16)),
              f32_to_bf16_rne(b - __uint_as_float(static_cast<uint32_t>(hb) << 16)));
}

// DPP move of a float across lanes (row/bank masks all on).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Sum over the 64 lanes.  Within each 16-lane row: xor-1 and xor-2 quad
// permutes, then half-row and row mirrors (each step adds a commutative pair,
// so every lane of a row holds identical bits); then the four row sums are
// added in row order.  Every lane returns the same value.
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  return ((lane_value(v, 0) + lane_value(v, 16)) + lane_value(v, 32)) + lane_value(v, 48);
}

__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  v = fmaxf(v, dpp<0x140>(v));
  return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}

// Unsigned maximum over the 64 lanes (the same DPP steps as wave_max); every
// lane returns the same value.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max(v, dpp_u32<0xB1>(v));
  v = max(v, dpp_u32<0x4E>(v));
  v = max(v, dpp_u32<0x141>(v));
  v = max(v, dpp_u32<0x140>(v));
  const uint32_t a = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 0));
  const uint32_t b = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 16));
  const uint32_t c = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 32));
  const uint32_t d = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 48));
  return max(max(a, b), max(c, d));
}

__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// One 16-byte load; NT marks it non-temporal (streamed once, kept out of the caches' reuse set).
template <bool NT>
__device__ __forceinline__ uint4 ld_chunk(const void* row, int c) {
  if (NT) {
    const u32x4 t = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, row) + c);
    return make_uint4(t.x, t.y, t.z, t.w);
  }
  return SPP_GLOBAL(uint4, row)[c];
}

// Raw 16-byte chunks of a row in lane layout (zero past the row end).  FULL:
// the row is exactly 64*NCH chunks, so no lane needs a bounds check and the
// loaded data goes through no select (a select forces a wait for its load).
// Past the end a lane re-reads chunk 0 and keeps zero; the loads carry no
// branch.
template <int NCH, bool FULL = false, bool NT = false>
__device__ __forceinline__ void load_chunks(const void* row, int lane, int nch, uint4 (&r)[NCH]) {
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int c = lane + 64 * j;
    if (FULL) {
      r[j] = ld_chunk<NT>(row, c);
    } else {
      const bool ok = c < nch;
      const uint4 v = ld_chunk<NT>(row, ok ? c : 0);
      r[j] = ok ? v : make_uint4(0, 0, 0, 0);
    }
  }
}

// fp32 row (V values per chunk of the storage type T) in lane layout; FULL as above.
template <typename T, int NCH, bool FULL = false>
__device__ __forceinline__ void load_row_f32(const float* src, int lane, int nch, float (&xv)[NCH][Vec<T>::N]) {
  constexpr int V = Vec<T>::N;
  constexpr int Q = V / 4;  // 16-byte fp32 pieces per storage chunk
  uint4 r[NCH][Q];
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int c = lane + 64 * j;
    const bool ok = FULL || c < nch;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint4 v = ld16(src + (ok ? c : 0) * V + 4 * q);  // no branch: all loads go out together
      r[j][q] = FULL || ok ? v : make_uint4(0, 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < NCH; ++j)
#pragma unroll
    for (int q = 0; q < Q; ++q) unpack<float>(r[j][q], &xv[j][4 * q]);
}

template <typename T, int NCH, bool FULL = false>
__device__ __forceinline__ void load_row_storage(const T* src, int lane, int nch, float (&xv)[NCH][Vec<T>::N]) {
  uint4 r[NCH];
  load_chunks<NCH, FULL>(src, lane, nch, r);
#pragma unroll
  for (int j = 0; j < NCH; ++j) unpack<T>(r[j], xv[j]);
}

template <typename T, int NCH>
__device__ __forceinline__ float rms_scale(float (&xv)[NCH][Vec<T>::N], int D, float eps) {
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < NCH; ++j)
#pragma unroll
    for (int v = 0; v < Vec<T>::N; ++v) ss += xv[j][v] * xv[j][v];
  ss = wave_sum(ss);
  return 1.0f / sqrtf(ss / static_cast<float>(D) + eps);
}

constexpr int kEQ = kMaxExpertsTopK / kThreads;  // experts per thread in the tails

// Host handoff.  The host records are written with system-scope atomic stores,
// which the GPU's caches do not hold back, and cross-workgroup values with
// agent-scope atomic stores and loads.  For such stores, waiting until the
// wave's own outstanding memory operations have completed is the whole of a
// release: a store issued after the wait (a counter increment, a flag) is seen
// only after them.  This avoids the L2 write-back that a release fence adds
// for ordinary stores.
__device__ __forceinline__ void wait_own_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One host record: the launch's sequence number in the high half and the
// payload in the low half, in one 8-byte system-scope store.  The host takes
// a record as written by this launch once its high half equals seq, so no
// store has to complete before another is issued (a completion flag after
// the results cost the host one more round trip over the host link).
__device__ __forceinline__ void st_record(uint64_t* p, unsigned seq, uint32_t payload) {
  __hip_atomic_store(p, (static_cast<uint64_t>(seq) << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The same tagging between the workgroups of one launch (device memory,
// agent scope): a value whose high half is this launch's seq is this launch's,
// so a reader polls for it instead of waiting on a completion counter, which
// costs the writer a wait for its own store and then an atomic round trip.
__device__ __forceinline__ void st_tag(uint64_t* p, unsigned seq, float v) {
  __hip_atomic_store(p, (static_cast<uint64_t>(seq) << 32) | __float_as_uint(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// Bound on the polls of a router tail (each at least one device-memory round
// trip, so about a second).  One wave per kind of row waits, for workgroups
// that were dispatched before its own and wait for nothing, so the bound is
// only reached where other work keeps those off the device that long.
constexpr unsigned kPollMax = 1u << 20;

// Lane l's values p[l + 64 q] (q < Q; indices >= cnt are not waited for) once
// every one carries seq; false if `polls` polls did not see that.
template <int Q>
__device__ __forceinline__ bool poll_tags(const uint64_t* p, int cnt, int lane, unsigned seq, unsigned polls, float* v) {
  for (unsigned it = 0; it < polls; ++it) {
    bool ok = true;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = lane + 64 * q;
      const uint64_t t = __hip_atomic_load(p + min(i, cnt - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      v[q] = __uint_as_float(static_cast<uint32_t>(t));
      ok = ok && (i >= cnt || static_cast<uint32_t>(t >> 32) == seq);
    }
    if (__all(ok)) return true;
    __builtin_amdgcn_s_sleep(1);
  }
  return false;
}

// The routing that the router workgroups of this launch publish, if it appears
// within `polls` polls: lane k < K gets the slot of the k-th selected expert,
// lane 32 + k its gate.
__device__ __forceinline__ bool poll_route(const uint64_t* p, int K, int lane, unsigned seq, unsigned polls,
                                           uint32_t* word) {
  *word = 0;
  for (unsigned it = 0; it < polls; ++it) {
    const uint64_t t = __hip_atomic_load(p + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *word = static_cast<uint32_t>(t);
    if (__all((lane & 31) >= K || static_cast<uint32_t>(t >> 32) == seq)) return true;
    __builtin_amdgcn_s_sleep(1);
  }
  return false;
}

// Token b's host records from wave 0 after select_topk (lane k < K: expert
// s_isel[k], gate s_zsel[k]).
__device__ __forceinline__ void route_records(const RouterArgs& a, int b, int tid, const float* s_zsel,
                                              const int* s_isel) {
  if (a.route_rec && tid < a.K) {
    const int idx = b * a.K + tid;
    st_record(a.route_rec + idx, a.seq, static_cast<uint32_t>(s_isel[tid]));
    st_record(a.gate_rec + idx, a.seq, __float_as_uint(s_zsel[tid]));
  }
}

// Order-preserving key of (logit z, expert e): key(e') > key(e) exactly when e'
// beats e under the Top-K rule -- a larger logit, or an equal logit and a lower
// index.  -0 is folded into +0 first, so the two stay equal as in a float
// comparison.
__device__ __forceinline__ uint32_t logit_order(float z) {
  uint32_t u = __float_as_uint(z);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float order_logit(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}
__device__ __forceinline__ uint64_t topk_key(float z, int e) {
  return (static_cast<uint64_t>(logit_order(z)) << 32) | (0xFFFFFFFFu - static_cast<uint32_t>(e));
}
__device__ __forceinline__ float key_logit(uint64_t k) { return order_logit(static_cast<uint32_t>(k >> 32)); }

// Top-K of one token by rank counting over its keys (LDS, n values): expert e
// takes position rank(e) = #{e' : key(e') > key(e)} (the keys are distinct, so
// the ranks are a permutation).  With n <= 128 two threads share an expert,
// each counting over half of the candidates.  Wave 0 then forms the combine
// weights (softmax over all n renormalised over the K selected = softmax over
// the selected) and writes token b's device outputs; s_zsel[k] then holds
// gate k (for route_records).  Every thread of the workgroup calls it.
__device__ __forceinline__ void select_topk(const RouterArgs& a, const uint64_t* s_key, int b, int tid, int* s_rk,
                                            float* s_zsel, int* s_isel) {
  const int n = a.n;
  const int P = n <= kThreads / 2 ? 2 : 1;
  const int E = kThreads / P;
  const int part = tid / E, el = tid - part * E;
  const int span = (n + P - 1) / P;
  const int j0 = part * span, j1 = min(n, j0 + span);
  for (int e0 = 0; e0 < n; e0 += E) {
    const int e = e0 + el;
    const uint64_t ke = s_key[min(e, n - 1)];
    int rank = 0;
#pragma unroll 8
    for (int j = j0; j < j1; ++j) rank += s_key[j] > ke ? 1 : 0;
    if (P == 2) {  // one pass: E >= n
      s_rk[tid] = rank;
      __syncthreads();
      if (part == 0) rank += s_rk[tid + E];
    }
    if (part == 0 && e < n && rank < a.K) {
      s_isel[rank] = e;
      s_zsel[rank] = key_logit(ke);
    }
  }
  __syncthreads();
  if (tid < 64) {
    const bool on = tid < a.K;
    const float m = s_zsel[0];
    const float v = on ? expf(s_zsel[on ? tid : 0] - m) : 0.f;
    const float sum = wave_sum(v);
    if (on) {
      const int idx = b * a.K + tid;
      const int e = s_isel[tid];
      const float gk = v / sum;
      a.topk[idx] = e;
      a.gates[idx] = gk;
      if (a.slot_tab) a.sel[idx] = a.slot_tab[e];
      s_zsel[tid] = gk;  // each lane rewrites only its own entry
    }
  }
}

// One token's predicted distribution pi_hat = softmax(B a) over the n experts
// (sa: the token's r adapter hidden units in LDS; B transposed in LDS when
// staged).  Thread tid gets experts tid + kThreads*q in pi[q].
template <typename T>
__device__ __forceinline__ void adapter_token(const RouterArgs& a, const float* sa, bool staged, const float* s_B,
                                              int tid, int lane, int wave, float* s_red, float (&pi)[kEQ]) {
  const int n = a.n, r = a.r;
  float zh[kEQ];
  float mx = -INFINITY;
#pragma unroll
  for (int q = 0; q < kEQ; ++q) {
    const int e = tid + kThreads * q;
    zh[q] = -INFINITY;
    if (e < n) {
      float acc = 0.f;
      if (staged) {
#pragma unroll 8
        for (int j = 0; j < r; ++j) acc += s_B[j * n + e] * sa[j];
      } else {
        for (int j = 0; j < r; ++j) acc += load_elem<T>(a.Bm, static_cast<size_t>(e) * r + j) * sa[j];
      }
      zh[q] = acc;
      mx = fmaxf(mx, acc);
    }
  }
  mx = wave_max(mx);
  if (lane == 0) s_red[wave] = mx;
  __syncthreads();
  mx = s_red[0];
  for (int wv = 1; wv < kWaves; ++wv) mx = fmaxf(mx, s_red[wv]);
  __syncthreads();
  float part = 0.f;
#pragma unroll
  for (int q = 0; q < kEQ; ++q) {
    const int e = tid + kThreads * q;
    pi[q] = e < n ? expf(zh[q] - mx) : 0.f;
    part += pi[q];
  }
  part = wave_sum(part);
  if (lane == 0) s_red[wave] = part;
  __syncthreads();
  float sum = 0.f;
  for (int wv = 0; wv < kWaves; ++wv) sum += s_red[wv];
#pragma unroll
  for (int q = 0; q < kEQ; ++q) pi[q] /= sum;
}

// The token's input row (always a valid address).
__device__ __forceinline__ const void* input_row(const RouterArgs& a) {
  return a.u ? static_cast<const void*>(a.u) : a.h;
}

// Adapter B, transposed into LDS ([r][n]); the loads are issued early by the
// caller and stored after its first wait.  The loads carry no branch: a chunk
// past the end (or every chunk, when B is not wanted) re-reads the first 16
// bytes of B (or of the input row) and is never stored.
template <typename T>
struct BStage {
  static constexpr int VB = Vec<T>::N;
  static constexpr int kLoads = kBStage / VB / kThreads;  // 16-byte chunks per thread
  uint4 rb[kLoads];
  int nchunk = 0;
  __device__ __forceinline__ void load(const RouterArgs& a, int tid, bool want) {
    nchunk = want ? (a.n * a.r) / VB : 0;  // n*r*sizeof(T) is a multiple of 16 (checked at launch)
    const uint8_t* src = static_cast<const uint8_t*>(want ? a.Bm : input_row(a));
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int c = tid + q * kThreads;
      rb[q] = ld16(src + static_cast<size_t>(c < nchunk ? c : 0) * 16);  // store() reads only c < nchunk
    }
  }
  __device__ __forceinline__ void store(const RouterArgs& a, int tid, float* s_B) const {
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int c = tid + q * kThreads;
      if (c < nchunk) {
        float f[VB];
        unpack<T>(rb[q], f);
#pragma unroll
        for (int v = 0; v < VB; ++v) {
          const int idx = c * VB + v;
          const int e = idx / a.r, j = idx - e * a.r;
          s_B[j * a.n + e] = f[v];
        }
      }
    }
  }
};

// One token's x: the router's input, normalised unless it is x already.
template <typename T, int NCH, bool FULL>
__device__ __forceinline__ void input_x(const RouterArgs& a, int lane, int nch, float (&xv)[NCH][Vec<T>::N]) {
  if (a.u) {
    load_row_f32<T, NCH, FULL>(a.u, lane, nch, xv);
  } else {
    load_row_storage<T, NCH, FULL>(reinterpret_cast<const T*>(a.h), lane, nch, xv);
  }
  if (a.x_given) return;
  const float inv = rms_scale<T, NCH>(xv, a.D, a.eps);
#pragma unroll
  for (int j = 0; j < NCH; ++j)
#pragma unroll
    for (int v = 0; v < Vec<T>::N; ++v) xv[j][v] *= inv;
}

// A router (or adapter) row times x, summed over the wave.
template <typename T, int NCH>
__device__ __forceinline__ float row_dot(const uint4 (&w)[NCH], const float (&xv)[NCH][Vec<T>::N]) {
  float acc = 0.f;
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    float wf[Vec<T>::N];
    unpack<T>(w[j], wf);
#pragma unroll
    for (int v = 0; v < Vec<T>::N; ++v) acc += wf[v] * xv[j][v];
  }
  return wave_sum(acc);
}

// One token's routing in one wave (n <= 64 Q, K <= 32): zv[q] the logit and
// slt[q] the slot of expert lane + 64 q.  Lane k < K returns the gate of the
// k-th selected expert, with its id and slot.
template <int Q>
__device__ __forceinline__ float select_wave(const float (&zv)[Q], const int (&slt)[Q], int n, int K, int lane,
                                             int* isel_out, int* slot_out) {
  uint32_t u[Q];
  bool av[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    av[q] = lane + 64 * q < n;
    u[q] = logit_order(zv[q]);
  }
  float zsel = 0.f;
  int isel = 0;
  for (int k = 0; k < K; ++k) {
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) c = max(c, av[q] ? u[q] : 0u);
    const uint32_t m = wave_max_u32(c);
    int e = -1;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint64_t hit = __ballot(av[q] && u[q] == m);
      if (e < 0 && hit) e = 64 * q + __builtin_ctzll(hit);
    }
    if (lane == (e & 63)) {
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (q == (e >> 6)) av[q] = false;
    }
    if (lane == k) {
      zsel = order_logit(m);
      isel = e;
    }
  }
  const float m0 = lane_value(zsel, 0);
  const float v = lane < K ? expf(zsel - m0) : 0.f;
  const float sum = wave_sum(v);
  int slot = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int t = __shfl(slt[q], isel & 63);
    slot = q == (isel >> 6) ? t : slot;
  }
  *isel_out = isel;
  *slot_out = slot;
  return v / sum;
}

// The routing of select_wave as the words of RouterArgs::route_tag: lane k < K
// the slot, lane 32 + k the gate.
__device__ __forceinline__ uint32_t route_word(int slot, float gk, int lane) {
  const uint32_t gl = __float_as_uint(__shfl(gk, lane & 31));
  return lane < 32 ? static_cast<uint32_t>(slot) : gl;
}

// ---------------------------------------------------------------------------
// Router for one token, one launch.  Workgroups [0, gr) hold the router rows,
// the rest the adapter-A rows, one wave per weight row.  Each kind hands off
// in a single pass: the last router workgroup to finish selects the Top-K and
// gates, the last adapter workgroup forms the adapter distribution -- the two
// tails run at the same time on different compute units.
//
// EPL = 0: the general tails (any n up to kMaxExpertsTopK, K <= 32, any r),
// run by the whole workgroup through LDS; adapter workgroups fetch B together
// with their rows, so the scoring tail starts with B in registers.
// EPL = 1 or 2 (n <= 64 * EPL; with an adapter: bf16, r <= 64 and a multiple of 8):
// the tails run in wave 0 alone, with no barrier -- lane l holds experts
// l + 64 q (q < EPL).  Top-K: K rounds of a wave maximum over the 32-bit
// order of the available logits, the lowest index taking a tie (the same
// order as topk_key).  Adapter: the tail wave holds B's rows of its lanes'
// experts in registers; the hidden unit a_j is broadcast from lane j.  Both
// give the bits of the general tails: the same products in the same order, and
// the distribution's sum as the sum of the per-64-expert wave sums in expert
// order.  Every row's value is also stored tagged with the launch's number, and
// wave 0 of the last workgroup of each kind takes that kind's tail as soon as
// its poll sees every value tagged: the writers neither wait for their stores
// nor pass a counter (1.0 us less per launch than EPL = 0's handoff to the last
// workgroup through a completion counter, same outputs).
// ---------------------------------------------------------------------------
// `nblocks` workgroups take part; `bid` is this one's index among them.  ALONE:
// a launch of adapter rows alone, whose tail never fails (the other launches'
// missing records tell the host).
template <typename T, int NCH, bool FULL, int EPL, bool ALONE>
__device__ __forceinline__ void router_adapter_body(const RouterArgs& a, int bid, int nblocks) {
  constexpr int V = Vec<T>::N;
  constexpr int kBC = 8;  // 16-byte chunks of one B row in the fast tail (r <= 64 bf16)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int D = a.D, nch = D / V, n = a.n, r = a.r;
  const int nr = a.router_on ? n : 0;
  const int na = a.A ? r : 0;
  const int gr = (nr + kWaves - 1) / kWaves;
  const bool adapter_wg = bid >= gr;
  const int row = (adapter_wg ? bid - gr : bid) * kWaves + wave;

  __shared__ int s_last;
  __shared__ float s_zsel[32];
  __shared__ int s_isel[32];
  __shared__ float s_red[kWaves];
  __shared__ int s_rk[kThreads];
  __shared__ float s_a[256];
  __shared__ uint64_t s_key[kMaxExpertsTopK];
  __shared__ float s_B[EPL ? 1 : kBStage];  // adapter B transposed ([r][n]) when n*r fits

  // a wave past its kind's last row re-reads that row (a valid address) and drops it
  const int rows = adapter_wg ? na : nr;
  const bool has_row = row < rows;
  const T* wrow = reinterpret_cast<const T*>(adapter_wg ? a.A : a.Wr) + static_cast<size_t>(min(row, rows - 1)) * D;
  const int zcol = adapter_wg ? n + row : row;
  // A caller without launch numbers (its launches may be replays of a graph):
  // every workgroup draws a ticket, and each launch draws nblocks of them, so
  // launches in order get numbers of their own whatever became of the ones
  // before -- also after launches that overlapped and mixed their tickets.
  constexpr unsigned kLaunches = 1u << 20;  // numbers before they repeat (every launch rewrites all its tags)
  unsigned ticket = 0;
  if (ALONE && EPL && a.tickets && tid == 0) ticket = atomicInc(a.tickets, nblocks * kLaunches - 1u);
  uint4 w[NCH];
  load_chunks<NCH, FULL>(wrow, lane, has_row ? nch : 0, w);
  const bool staged = na && n * r <= kBStage;
  BStage<T> bst;
  uint4 rbf[EPL ? EPL : 1][kBC];
  if (EPL == 0) {
    bst.load(a, tid, adapter_wg && staged);
  } else if (sizeof(T) == 2 && adapter_wg && wave == 0 && bid == nblocks - 1) {
    // B rows of the tail's lanes' experts (a chunk past r, or a row past n,
    // re-reads the first chunk of B and is dropped)
    const int rc = r / 8;
#pragma unroll
    for (int q = 0; q < (EPL ? EPL : 1); ++q) {
      const int e = lane + 64 * q;
#pragma unroll
      for (int c = 0; c < kBC; ++c) {
        const bool ok = e < n && c < rc;
        const uint4 v = ld16(static_cast<const uint8_t*>(a.Bm) + (ok ? (static_cast<size_t>(e) * r + 8 * c) * 2 : 0));
        rbf[q][c] = ok ? v : make_uint4(0, 0, 0, 0);
      }
    }
  }

  // slots of this lane's experts, for the workgroup that may select
  int slt[EPL ? EPL : 1];
#pragma unroll
  for (int q = 0; q < (EPL ? EPL : 1); ++q)
    slt[q] = EPL && !adapter_wg && wave == 0 && a.slot_tab ? a.slot_tab[min(lane + 64 * q, n - 1)] : 0;

  float xv[NCH][V];
  input_x<T, NCH, FULL>(a, lane, nch, xv);
  // x goes out from the last wave of the last workgroup: never a tail wave,
  // whose first wait would otherwise include these stores
  if (bid == nblocks - 1 && wave == kWaves - 1 && a.x_out) {
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const int c = lane + 64 * j;
      if (c < nch) {
        float* dst = a.x_out + c * V;
#pragma unroll
        for (int v = 0; v < V; ++v) dst[v] = xv[j][v];
        if (a.xh) {
#pragma unroll
          for (int v = 0; v < V; v += 2)
            split2(xv[j][v], xv[j][v + 1], reinterpret_cast<uint32_t*>(a.xh) + (c * V + v) / 2,
                   reinterpret_cast<uint32_t*>(a.xl) + (c * V + v) / 2);
        }
      }
    }
  }
  unsigned seq = a.seq;
  if (ALONE && EPL && a.tickets) {
    __shared__ unsigned s_seq;
    if (tid == 0) s_seq = ticket / static_cast<unsigned>(nblocks) + 1u;
    __syncthreads();
    seq = s_seq;
  }
  if (has_row) {
    const float acc = row_dot<T, NCH>(w, xv);
    if (lane == 0) {
      st_agent(a.zbuf + zcol, acc);
      if (EPL) st_tag((adapter_wg ? a.atag : a.ztag) + row, seq, acc);
    }
  }

  if (EPL) {
    constexpr int Q = EPL ? EPL : 1;
    // Handoff: wave 0 of its kind's last workgroup polls the tagged values (it
    // waits only for workgroups dispatched before it)
    if (wave != 0 || bid != (adapter_wg ? nblocks : gr) - 1) return;
    float zv[Q];
    // a poll that runs out leaves this launch's records unwritten: the host reports it
    if (!adapter_wg) {
      if (!poll_tags<Q>(a.ztag, n, lane, seq, kPollMax, zv)) return;
    } else {
      if constexpr (sizeof(T) == 4) return;  // fp32 adapters take the general tail
      if (!poll_tags<1>(a.atag, na, lane, seq, ALONE ? a.polls : kPollMax, zv)) {
        if constexpr (!ALONE) return;
        // rows that are late, or that an overlapping launch numbered: form them here, with the same operations
        input_x<T, NCH, FULL>(a, lane, nch, xv);
#pragma unroll 1
        for (int j = 0; j < na; ++j) {
          load_chunks<NCH, FULL>(reinterpret_cast<const T*>(a.A) + static_cast<size_t>(j) * D, lane, nch, w);
          const float z = row_dot<T, NCH>(w, xv);
          zv[0] = lane == j ? z : zv[0];
        }
      }
    }
    if (!adapter_wg) {
      int isel, slot;
      const float gk = select_wave<Q>(zv, slt, n, a.K, lane, &isel, &slot);
      if (a.route_tag) {  // first: the FFN workgroups of this launch wait for it
        const float word = __uint_as_float(route_word(slot, gk, lane));
        if ((lane & 31) < a.K)
#pragma unroll
          for (int c = 0; c < kRouteCopies; ++c) st_tag(a.route_tag + c * kRouteWords + lane, a.seq, word);
      }
      if (lane < a.K) {
        a.topk[lane] = isel;
        a.gates[lane] = gk;
        if (a.slot_tab) a.sel[lane] = slot;
        if (a.route_rec) {
          st_record(a.route_rec + lane, a.seq, static_cast<uint32_t>(isel));
          st_record(a.gate_rec + lane, a.seq, __float_as_uint(gk));
        }
      }
      return;
    }
    // adapter distribution pi_hat = softmax(B a)
    const float av = lane < na ? zv[0] : 0.f;
    float zh[Q];
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      float acc = 0.f;
#pragma unroll
      for (int c = 0; c < kBC; ++c) {
        float f[8];
        unpack<uint16_t>(rbf[q][c], f);
#pragma unroll
        for (int v = 0; v < 8; ++v) acc += f[v] * lane_value(av, 8 * c + v);
      }
      zh[q] = lane + 64 * q < n ? acc : -INFINITY;
      mx = fmaxf(mx, zh[q]);
    }
    mx = wave_max(mx);
    float pi[Q];
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      pi[q] = lane + 64 * q < n ? expf(zh[q] - mx) : 0.f;
      sum = q == 0 ? wave_sum(pi[q]) : sum + wave_sum(pi[q]);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = lane + 64 * q;
      if (e < n) {
        const float p = pi[q] / sum;
        a.s[e] = p;
        if (a.s_rec) st_record(a.s_rec + e, a.seq, __float_as_uint(p));
      }
    }
    return;
  }
  const int kind = adapter_wg ? 1 : 0;
  const unsigned total = adapter_wg ? nblocks - gr : gr;
  wait_own_stores();  // release this wave's value
  __syncthreads();
  if (tid == 0) {
    const unsigned prev = __hip_atomic_fetch_add(a.counter + kind, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (prev == total - 1);
  }
  __syncthreads();
  if (!s_last) return;

  if (!adapter_wg) {
    // Top-K and gates over the n logits (agent-scope loads: other workgroups wrote them)
    float z[kEQ];
#pragma unroll
    for (int q = 0; q < kEQ; ++q) z[q] = ld_agent(a.zbuf + min(tid + kThreads * q, n - 1));
#pragma unroll
    for (int q = 0; q < kEQ; ++q) {
      const int e = tid + kThreads * q;
      if (e < n) s_key[e] = topk_key(z[q], e);
    }
    __syncthreads();
    select_topk(a, s_key, 0, tid, s_rk, s_zsel, s_isel);
    if (tid == 0) __hip_atomic_store(a.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    route_records(a, 0, tid, s_zsel, s_isel);
    return;
  }

  // adapter distribution pi_hat = softmax(B a) over the r hidden units
  if (tid < na) s_a[tid] = ld_agent(a.zbuf + n + tid);
  bst.store(a, tid, s_B);
  __syncthreads();
  float pi[kEQ];
  adapter_token<T>(a, s_a, staged, s_B, tid, lane, wave, s_red, pi);
#pragma unroll
  for (int q = 0; q < kEQ; ++q) {
    const int e = tid + kThreads * q;
    if (e < n) {
      a.s[e] = pi[q];
      if (a.s_rec) st_record(a.s_rec + e, a.seq, __float_as_uint(pi[q]));
    }
  }
  if (tid == 0) __hip_atomic_store(a.counter + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T, int NCH, bool FULL, int EPL>
__global__ __launch_bounds__(kThreads) void router_adapter_kernel(RouterArgs a) {
  // one argument of each 64-byte line: the lines come together, not one by one
  // as the code first needs them (0.25 us of 5.9)
  static_assert(sizeof(RouterArgs) > 192 && sizeof(RouterArgs) <= 256, "four lines of arguments");
  asm volatile("" ::"s"(a.h), "s"(a.atag), "s"(a.sel), "s"(a.n));
  router_adapter_body<T, NCH, FULL, EPL, false>(a, blockIdx.x, gridDim.x);
}

// Adapter rows alone (bf16, one-wave tail).
template <int NCH, bool FULL, int EPL>
__global__ __launch_bounds__(kThreads) void adapter_kernel(RouterArgs a) {
  router_adapter_body<uint16_t, NCH, FULL, EPL, true>(a, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// Selection for B > 1 tokens (their rows: router_rows_kernel, below with the
// MFMA kernels): one workgroup per token -- Top-K, gates and
// the adapter distribution; the last workgroup to finish sums the
// distributions over the tokens, in token order, into s.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kThreads) void router_select_kernel(RouterArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = a.n, r = a.r, ldz = a.n + a.r;
  const int na = a.A ? r : 0;
  const int b = blockIdx.x;
  __shared__ int s_last;
  __shared__ float s_zsel[32];
  __shared__ int s_isel[32];
  __shared__ float s_red[kWaves];
  __shared__ int s_rk[kThreads];
  __shared__ float s_a[256];
  __shared__ uint64_t s_key[kMaxExpertsTopK];
  __shared__ float s_B[kBStage];

  const bool staged = na && n * r <= kBStage;
  BStage<T> bst;
  bst.load(a, tid, staged);
  float* zrow = a.zbuf + static_cast<size_t>(b) * ldz;  // written by the rows launch
  float z[kEQ];
#pragma unroll
  for (int q = 0; q < kEQ; ++q) z[q] = zrow[min(tid + kThreads * q, n - 1)];
  const float hid = tid < na ? zrow[n + tid] : 0.f;  // without an adapter the row may end at its n logits
#pragma unroll
  for (int q = 0; q < kEQ; ++q) {
    const int e = tid + kThreads * q;
    if (e < n) s_key[e] = topk_key(z[q], e);
  }
  if (tid < na) s_a[tid] = hid;
  bst.store(a, tid, s_B);
  __syncthreads();
  if (a.router_on) select_topk(a, s_key, b, tid, s_rk, s_zsel, s_isel);
  if (!na) {
    if (a.router_on) route_records(a, b, tid, s_zsel, s_isel);
    return;
  }
  if (na) {
    float pi[kEQ];
    adapter_token<T>(a, s_a, staged, s_B, tid, lane, wave, s_red, pi);
    // this token's distribution replaces its logits in zbuf (only this workgroup touches row b)
#pragma unroll
    for (int q = 0; q < kEQ; ++q) {
      const int e = tid + kThreads * q;
      if (e < n) st_agent(zrow + e, pi[q]);
    }
  }
  wait_own_stores();  // release this token's distribution (device stores only so far)
  __syncthreads();
  if (tid == 0) {
    const unsigned prev = __hip_atomic_fetch_add(a.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (prev == gridDim.x - 1);
  }
  // the host records go out after the release: nothing waits for them
  if (a.router_on) route_records(a, b, tid, s_zsel, s_isel);
  __syncthreads();
  if (!s_last) return;
  {
    // s = sum over the tokens, in token order, of their distributions; the
    // loads go out 64 tokens at a time
    constexpr int kTB = 64;
    for (int e = tid; e < n; e += kThreads) {
      float acc = 0.f;
      for (int b0 = 0; b0 < a.B; b0 += kTB) {
        float v[kTB];
#pragma unroll
        for (int q = 0; q < kTB; ++q) v[q] = ld_agent(a.zbuf + static_cast<size_t>(min(b0 + q, a.B - 1)) * ldz + e);
#pragma unroll
        for (int q = 0; q < kTB; ++q)
          if (b0 + q < a.B) acc += v[q];
      }
      a.s[e] = acc;
      if (a.s_rec) st_record(a.s_rec + e, a.seq, __float_as_uint(acc));
    }
  }
  if (tid == 0) __hip_atomic_store(a.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Selection for B > 1 tokens with one wave per token (n <= 64 EPL; with an
// adapter: bf16, r <= 64 and a multiple of 8): lane l holds experts l + 64 q.  Top-K
// by K rounds of a wave maximum over the 32-bit logit order (the lowest index
// taking a tie), the gates, and the adapter distribution from B's rows of the
// lane's experts in registers -- the products, maxima and sums of
// router_select_kernel in the same order, so the same bits -- then, as there,
// the token's distribution replaces its logits in zbuf, and the last token's
// wave sums the distributions over the tokens in token order.
template <int EPL>
__global__ __launch_bounds__(64) void router_select_wave_kernel(RouterArgs a) {
  using T = uint16_t;
  constexpr int kBC = 8;
  const int lane = threadIdx.x;
  const int n = a.n, r = a.r, ldz = a.n + a.r;
  const int na = a.A ? r : 0;
  const int b = blockIdx.x;
  float* zrow = a.zbuf + static_cast<size_t>(b) * ldz;  // written by the rows launch
  uint4 rbf[EPL][kBC];
  if (na) {
    const int rc = r / 8;
#pragma unroll
    for (int q = 0; q < EPL; ++q) {
      const int e = lane + 64 * q;
#pragma unroll
      for (int c = 0; c < kBC; ++c) {
        const bool ok = e < n && c < rc;
        const uint4 v = ld16(static_cast<const uint8_t*>(a.Bm) + (ok ? (static_cast<size_t>(e) * r + 8 * c) * 2 : 0));
        rbf[q][c] = ok ? v : make_uint4(0, 0, 0, 0);
      }
    }
  }
  uint32_t u[EPL];
  bool av[EPL];
#pragma unroll
  for (int q = 0; q < EPL; ++q) {
    const int e = lane + 64 * q;
    av[q] = e < n;
    u[q] = logit_order(zrow[min(e, n - 1)]);
  }
  const float hid = lane < na ? zrow[n + lane] : 0.f;
  float zsel = 0.f, gk = 0.f;
  int isel = 0;
  if (a.router_on) {
    for (int k = 0; k < a.K; ++k) {
      uint32_t c = 0;
#pragma unroll
      for (int q = 0; q < EPL; ++q) c = max(c, av[q] ? u[q] : 0u);
      const uint32_t m = wave_max_u32(c);
      int e = -1;
#pragma unroll
      for (int q = 0; q < EPL; ++q) {
        const uint64_t hit = __ballot(av[q] && u[q] == m);
        if (e < 0 && hit) e = 64 * q + __builtin_ctzll(hit);
      }
      if (lane == (e & 63)) {
#pragma unroll
        for (int q = 0; q < EPL; ++q)
          if (q == (e >> 6)) av[q] = false;
      }
      if (lane == k) {
        zsel = order_logit(m);
        isel = e;
      }
    }
    const bool on = lane < a.K;
    const float m0 = lane_value(zsel, 0);
    const float v = on ? expf(zsel - m0) : 0.f;
    const float sum = wave_sum(v);
    if (on) {
      gk = v / sum;
      a.topk[b * a.K + lane] = isel;
      a.gates[b * a.K + lane] = gk;
      if (a.slot_tab) a.sel[b * a.K + lane] = a.slot_tab[isel];
    }
  }
  auto records = [&]() {
    if (a.router_on && a.route_rec && lane < a.K) {
      st_record(a.route_rec + b * a.K + lane, a.seq, static_cast<uint32_t>(isel));
      st_record(a.gate_rec + b * a.K + lane, a.seq, __float_as_uint(gk));
    }
  };
  if (!na) {
    records();
    return;
  }
  // adapter distribution pi_hat = softmax(B a) of this token
  float zh[EPL];
  float mx = -INFINITY;
#pragma unroll
  for (int q = 0; q < EPL; ++q) {
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < kBC; ++c) {
      float f[8];
      unpack<T>(rbf[q][c], f);
#pragma unroll
      for (int v = 0; v < 8; ++v) acc += f[v] * lane_value(hid, 8 * c + v);
    }
    zh[q] = lane + 64 * q < n ? acc : -INFINITY;
    mx = fmaxf(mx, zh[q]);
  }
  mx = wave_max(mx);
  float pi[EPL];
  float sum = 0.f;
#pragma unroll
  for (int q = 0; q < EPL; ++q) {
    pi[q] = lane + 64 * q < n ? expf(zh[q] - mx) : 0.f;
    sum = q == 0 ? wave_sum(pi[q]) : sum + wave_sum(pi[q]);
  }
#pragma unroll
  for (int q = 0; q < EPL; ++q) {
    const int e = lane + 64 * q;
    if (e < n) st_agent(zrow + e, pi[q] / sum);
  }
  wait_own_stores();  // release this token's distribution
  unsigned prev = 0;
  if (lane == 0) prev = __hip_atomic_fetch_add(a.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  prev = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(prev)));
  records();  // the host records go out after the release: nothing waits for them
  if (prev != gridDim.x - 1) return;
  // s = sum over the tokens, in token order, of their distributions
  constexpr int kTB = 64;
#pragma unroll
  for (int q = 0; q < EPL; ++q) {
    const int e = lane + 64 * q;
    const int ec = min(e, n - 1);
    float acc = 0.f;
    for (int b0 = 0; b0 < a.B; b0 += kTB) {
      float v[kTB];
#pragma unroll
      for (int t = 0; t < kTB; ++t) v[t] = ld_agent(a.zbuf + static_cast<size_t>(min(b0 + t, a.B - 1)) * ldz + ec);
#pragma unroll
      for (int t = 0; t < kTB; ++t)
        if (b0 + t < a.B) acc += v[t];
    }
    if (e < n) {
      a.s[e] = acc;
      if (a.s_rec) st_record(a.s_rec + e, a.seq, __float_as_uint(acc));
    }
  }
  if (lane == 0) __hip_atomic_store(a.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// Routed-expert SwiGLU FFN, one pass over the expert blobs.  The work is the
// flat list of (expert, unit i) pairs; unit i of an expert is the contiguous
// [gate row i | up row i | down column i].  A wave computes
//   h_i = silu(gate_i . x) * (up_i . x) * g_k
// and accumulates h_i * down_i into its lane-owned slice of y; the workgroup
// then sums its waves and writes one partial y.  Expert addresses and gates
// sit in LDS, so each wave issues the loads of UPP units (3*UPP*NCH 16-byte
// loads per lane) before waiting on any of them.
// ---------------------------------------------------------------------------
constexpr int kFfnWaves = 4;
constexpr int kFfnThreads = 64 * kFfnWaves;

// Blob of work item d (wave-uniform): the slot that the router launch named
// for a routed expert, or the address the host gave.
__device__ __forceinline__ const void* work_blob(const FfnArgs& a, int d) {
  if (d < a.nsel) return a.slots + static_cast<uint64_t>(static_cast<uint32_t>(a.sel[d])) * a.stride;
  return a.blob[d];
}

template <int NCH>
constexpr int ffn_upp() {
  return NCH <= 3 ? 4 : (NCH == 4 ? 3 : (NCH == 5 ? 2 : 1));
}

template <typename T, int NCH, bool FULL>
__global__ __launch_bounds__(kFfnThreads) void ffn_units_kernel(FfnArgs a) {
  constexpr int V = Vec<T>::N;
  constexpr int UPP = ffn_upp<NCH>();
  extern __shared__ float s_red[];  // [kFfnWaves / 2][D] wave partials
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, nch = D / V, I = a.I;
  if ((a.skip_mask >> ((static_cast<int>(blockIdx.x) * a.upw) / I)) & 1u) return;  // another launch's item

  float acc[NCH][V];
#pragma unroll
  for (int j = 0; j < NCH; ++j)
#pragma unroll
    for (int v = 0; v < V; ++v) acc[j][v] = 0.f;
  // x goes out first: each unit's dot products then wait only for that
  // unit's loads, and the math of the first units overlaps the arrival of
  // the later ones
  float xv[NCH][V];
  load_row_f32<T, NCH, FULL>(a.x, lane, nch, xv);
  __builtin_amdgcn_sched_barrier(0);

  const int total = a.nW * I;
  const int u0 = blockIdx.x * a.upw;
  const int u1 = min(u0 + a.upw, total);
  const size_t unit_elems = static_cast<size_t>(3) * D;

  for (int ub = u0 + wave; ub < u1; ub += kFfnWaves * UPP) {
    uint4 rg[UPP][NCH], ru[UPP][NCH], rd[UPP][NCH];
    float gate[UPP];
#pragma unroll
    for (int p = 0; p < UPP; ++p) {
      const int uu = ub + p * kFfnWaves;
      gate[p] = 0.f;
      if (uu < u1) {  // wave-uniform
        const int d = uu / I;
        const int i = uu - d * I;
        const T* base = reinterpret_cast<const T*>(work_blob(a, d)) + static_cast<size_t>(i) * unit_elems;
        load_chunks<NCH, FULL, true>(base, lane, nch, rg[p]);
        load_chunks<NCH, FULL, true>(base + D, lane, nch, ru[p]);
        load_chunks<NCH, FULL, true>(base + 2 * D, lane, nch, rd[p]);
        const int gi = a.gate_idx[d];
        gate[p] = gi >= 0 ? a.gates[gi] : 1.f;
      } else {
#pragma unroll
        for (int j = 0; j < NCH; ++j) rg[p][j] = ru[p][j] = rd[p][j] = make_uint4(0, 0, 0, 0);
      }
    }
#pragma unroll
    for (int p = 0; p < UPP; ++p) {
      float gs = 0.f, us = 0.f;
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        float fg[V], fu[V];
        unpack<T>(rg[p][j], fg);
        unpack<T>(ru[p][j], fu);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          gs += fg[v] * xv[j][v];
          us += fu[v] * xv[j][v];
        }
      }
      const float g = wave_sum(gs);
      const float u = wave_sum(us);
      const float hval = g / (1.f + expf(-g)) * u * gate[p];
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        float fd[V];
        unpack<T>(rd[p][j], fd);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[j][v] += hval * fd[v];
      }
    }
  }

  // sum the waves of this workgroup in a fixed order: (w + w+H) for w < H,
  // then slots 0..H-1.  With 8 values per chunk (bf16) a chunk's two 16-byte
  // halves are swapped in every other group of four chunks (element 8c + 4h + e
  // at word 8c + 4 (h ^ ((c >> 2) & 1)) + e), so that the 16-byte stores of
  // eight consecutive lanes and the natural-order reads of the last pass touch
  // every bank once; fp32 (4 values per chunk) needs no swizzle.  The swizzle
  // is taken within each wave pair's D-float region.
  constexpr int H = kFfnWaves / 2;
  auto widx = [](int d) -> int {
    if (V != 8) return d;
    const int c = d >> 3, e = d & 7;
    return 8 * c + 4 * ((e >> 2) ^ ((c >> 2) & 1)) + (e & 3);
  };
  float4* s_red4 = reinterpret_cast<float4*>(s_red);
  if (wave >= H) {
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const int c = lane + 64 * j;
      if (c < nch) {
#pragma unroll
        for (int h = 0; h < V / 4; ++h)
          s_red4[((wave - H) * D + widx(c * V + 4 * h)) / 4] =
              make_float4(acc[j][4 * h], acc[j][4 * h + 1], acc[j][4 * h + 2], acc[j][4 * h + 3]);
      }
    }
  }
  __syncthreads();
  if (wave < H) {
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const int c = lane + 64 * j;
      if (c < nch) {
#pragma unroll
        for (int h = 0; h < V / 4; ++h) {
          float4* slot = &s_red4[(wave * D + widx(c * V + 4 * h)) / 4];
          const float4 o = *slot;
          *slot = make_float4(acc[j][4 * h] + o.x, acc[j][4 * h + 1] + o.y, acc[j][4 * h + 2] + o.z,
                              acc[j][4 * h + 3] + o.w);
        }
      }
    }
  }
  __syncthreads();
  float* out = a.partial + static_cast<size_t>(blockIdx.x) * D;
  for (int d = tid; d < D; d += kFfnThreads) {
    const int w = widx(d);
    float v = s_red[w];
#pragma unroll
    for (int wv = 1; wv < H; ++wv) v += s_red[wv * D + w];
    out[d] = v;
  }
}

// ---------------------------------------------------------------------------
// Routed-expert SwiGLU FFN, batch 1, in sweep rounds with per-wave output
// slices (the default batch-1 kernel over bf16/fp32 experts).
//
// Units (work item, unit i) are taken in R rounds: in round r, wave w of
// workgroup b takes unit r*G*W + b*W + w (G workgroups of W waves), so at any
// moment the whole grid reads one band of consecutive units -- a 75 MB read
// in this order streams about 1.7 us faster on MI355X than one where each
// workgroup reads its own contiguous range.  D is cut into W slices of
// cpw = ceil(nch / W) chunks; wave w owns slice w.  Every wave
//   1. issues all its loads before any math: the gate and up rows of its R
//      units, and its slice of the down columns of all R*W units of its
//      workgroup;
//   2. forms h_u = silu(gate_u . x) * (up_u . x) * g for its own units and
//      publishes them in LDS (one barrier);
//   3. accumulates its slice of sum_u h_u down_u over the workgroup's units in
//      unit order and stores it into the workgroup's partial row.
// A partial row is written slice by slice: no reduction across waves (an LDS
// fold at the end of every workgroup cost about 1.3 us of a 17 us launch).
// The combine then sums the G partial rows in fixed order: the result is
// bitwise reproducible for a given grid.
// ---------------------------------------------------------------------------
constexpr int kSlWaves = 4;

// The words of RouterArgs::route_tag formed by one wave from x and the router's
// rows: the router's own operations, so the same bits.
template <typename T, int NCH, bool FULL>
__device__ __forceinline__ uint32_t route_self(const RouterArgs& ra, const float (&xv)[NCH][Vec<T>::N], int lane) {
  const int n = ra.n, nch = ra.D / Vec<T>::N;
  float zv[2] = {0.f, 0.f};
  int slt[2], isel, slot;
#pragma unroll 1
  for (int row = 0; row < n; ++row) {
    uint4 w[NCH];
    load_chunks<NCH, FULL>(reinterpret_cast<const T*>(ra.Wr) + static_cast<size_t>(row) * ra.D, lane, nch, w);
    const float z = row_dot<T, NCH>(w, xv);
#pragma unroll
    for (int q = 0; q < 2; ++q) zv[q] = row == lane + 64 * q ? z : zv[q];
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) slt[q] = ra.slot_tab[min(lane + 64 * q, n - 1)];
  const float gk = select_wave<2>(zv, slt, n, ra.K, lane, &isel, &slot);
  return route_word(slot, gk, lane);
}

// Wave 0 of a workgroup polls for the routing, or else calls self() for the
// words; the other waves get them through LDS.
template <typename F>
__device__ __forceinline__ uint32_t route_words(const RouterArgs& ra, int bid, int lane, int wave, F&& self) {
  __shared__ uint32_t s_route[kRouteWords];
  if (wave == 0) {
    uint32_t w;
    if (!poll_route(ra.route_tag + (bid % kRouteCopies) * kRouteWords, ra.K, lane, ra.seq, ra.polls, &w)) w = self();
    s_route[lane] = w;
  }
  __syncthreads();
  return s_route[lane];
}

// Where the work items of an FFN lie.  Routed: in the words that poll_route
// returned (wave-uniform lane reads); else in the arguments.
template <bool ROUTED>
struct Items {
  uint32_t words = 0;
  __device__ __forceinline__ const void* blob(const FfnArgs& a, int d) const {
    if (ROUTED && d < a.nsel)
      return a.slots + static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(words, d))) * a.stride;
    return ROUTED ? a.blob[d] : work_blob(a, d);
  }
  __device__ __forceinline__ float gate(const FfnArgs& a, int d) const {
    if (ROUTED) return d < a.nsel ? __uint_as_float(__builtin_amdgcn_readlane(words, 32 + d)) : 1.f;
    const int gi = a.gate_idx[d];
    return gi >= 0 ? a.gates[gi] : 1.f;
  }
};

template <typename T, int NCH, bool FULL, int R, int DS, bool ROUTED>
__device__ __forceinline__ void ffn_slices_body(const FfnArgs& a, const RouterArgs* ra, int bid, int nblocks) {
  constexpr int V = Vec<T>::N;
  constexpr int W = kSlWaves;
  __shared__ float s_h[R * W];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, nch = D / V, I = a.I;
  const int total = a.nW * I;
  const int band = nblocks * W;
  const int first = bid * W;
  const size_t unit_elems = static_cast<size_t>(3) * D;
  const int cpw = (nch + W - 1) / W;
  const int c0 = wave * cpw;

  // x first: each unit's dot products then wait only for that unit's loads
  float xv[NCH][V];
  Items<ROUTED> items;
  if constexpr (ROUTED) {
    input_x<T, NCH, FULL>(*ra, lane, nch, xv);
    items.words = route_words(*ra, bid, lane, wave, [&]() { return route_self<T, NCH, FULL>(*ra, xv, lane); });
  } else {
    load_row_f32<T, NCH, FULL>(a.x, lane, nch, xv);
  }
  __builtin_amdgcn_sched_barrier(0);

  // 1. every load of the wave, round by round (a unit past the end re-reads
  // the last unit, a lane past its slice re-reads chunk 0; neither is used)
  uint4 rg[R][NCH], ru[R][NCH], rd[R][W][DS];
  float gate[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int ub = r * band + first;
    const int u = ub + wave;
    const int uc = u < total ? u : total - 1;  // wave-uniform
    const int d = uc / I;
    const T* base = reinterpret_cast<const T*>(items.blob(a, d)) + static_cast<size_t>(uc - d * I) * unit_elems;
    load_chunks<NCH, FULL, true>(base, lane, nch, rg[r]);
    load_chunks<NCH, FULL, true>(base + D, lane, nch, ru[r]);
    gate[r] = items.gate(a, d);
#pragma unroll
    for (int w2 = 0; w2 < W; ++w2) {
      const int v = ub + w2;
      const int vc = v < total ? v : total - 1;  // wave-uniform
      const int d2 = vc / I;
      const T* dbase = reinterpret_cast<const T*>(items.blob(a, d2)) + static_cast<size_t>(vc - d2 * I) * unit_elems + 2 * D;
#pragma unroll
      for (int s = 0; s < DS; ++s) {
        const int c = c0 + lane + 64 * s;
        rd[r][w2][s] = ld_chunk<true>(dbase, lane + 64 * s < cpw && c < nch ? c : 0);
      }
    }
  }

  // 2. h of the wave's own units
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float gs = 0.f, us = 0.f;
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      float fg[V], fu[V];
      unpack<T>(rg[r][j], fg);
      unpack<T>(ru[r][j], fu);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        gs += fg[v] * xv[j][v];
        us += fu[v] * xv[j][v];
      }
    }
    const float g = wave_sum(gs);
    const float u = wave_sum(us);
    if (lane == 0) s_h[r * W + wave] = g / (1.f + expf(-g)) * u * gate[r];
  }
  __syncthreads();

  // 3. the wave's slice of sum_u h_u down_u over the workgroup's units, in unit order
  float acc[DS][V];
#pragma unroll
  for (int s = 0; s < DS; ++s)
#pragma unroll
    for (int v = 0; v < V; ++v) acc[s][v] = 0.f;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int w2 = 0; w2 < W; ++w2) {
      if (r * band + first + w2 >= total) continue;  // workgroup-uniform
      const float h = s_h[r * W + w2];
#pragma unroll
      for (int s = 0; s < DS; ++s) {
        float fd[V];
        unpack<T>(rd[r][w2][s], fd);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[s][v] += h * fd[v];
      }
    }
  float* out = a.partial + static_cast<size_t>(bid) * D;
#pragma unroll
  for (int s = 0; s < DS; ++s) {
    const int c = c0 + lane + 64 * s;
    if (lane + 64 * s < cpw && c < nch) {
#pragma unroll
      for (int v = 0; v < V; ++v) out[c * V + v] = acc[s][v];
    }
  }
}

template <typename T, int NCH, bool FULL, int R, int DS>
__global__ __launch_bounds__(64 * kSlWaves) void ffn_slices_kernel(FfnArgs a) {
  ffn_slices_body<T, NCH, FULL, R, DS, false>(a, nullptr, blockIdx.x, gridDim.x);
}

// Router and FFN of one token in one launch (device-routed layers): the first
// `rb` workgroups are router_adapter_body's, the others ffn_slices_body's.
// The FFN's workgroups are already resident and hold x when the routing
// appears, and the router's stores to the host leave the critical path; as a
// launch of its own the FFN started only after those stores, a launch's
// latency and a load of x.  The wait is a hint, never a dependence: these grids
// exceed what is resident at once and each XCD dispatches on its own, so two
// launches on two streams could hold each other's routers off the device.  A
// workgroup whose first wave does not see the routing within ra.polls polls
// (about a microsecond each; the routing takes some 5 us) forms it from the
// router's rows itself, with the same bits, and no workgroup's end waits for
// another's start.  Qwen-shaped: router 6.5 + FFN 14.8 us ->
// 19.1 in one launch, the layer 24.2 -> 22.1; 4-bit 6.5 + 9.8 -> 13.8, the
// layer 18.0 -> 16.9; 1,024 units of 256 fp32 columns 5.1 + 3.8 -> 6.0.  The
// same for a batch (selection and FFN in one launch, every workgroup waiting
// for the pairs' tagged words) gained 0.3 to 1.4% and was not kept.
template <typename T, int NCH, bool FULL, int R, int DS>
__global__ __launch_bounds__(64 * kSlWaves) void layer_slices_kernel(RouterArgs ra, FfnArgs fa, int rb) {
  static_assert(kSlWaves == kWaves, "one workgroup size for both parts");
  const int b = blockIdx.x;
  if (b < rb)
    router_adapter_body<T, NCH, FULL, 2, false>(ra, b, rb);
  else
    ffn_slices_body<T, NCH, FULL, R, DS, true>(fa, &ra, b - rb, static_cast<int>(gridDim.x) - rb);
}

// ---------------------------------------------------------------------------
// Read-ceiling probe (measurement only, never on the hot path): the loads of
// ffn_slices_kernel -- same grid, rounds, unit order and D-slices, the same
// non-temporal 16-byte loads -- with no arithmetic beyond folding the loaded
// words into one checksum per workgroup.  Its time is what the FFN's own
// access pattern can stream from HBM on this part.
// ---------------------------------------------------------------------------
template <int NCH, int R, int DS>
__global__ __launch_bounds__(64 * kSlWaves) void read_probe_kernel(FfnArgs a, uint32_t* sink) {
  using T = uint16_t;
  constexpr int V = Vec<T>::N;
  constexpr int W = kSlWaves;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int D = a.D, nch = D / V, I = a.I;
  const int total = a.nW * I;
  const int band = static_cast<int>(gridDim.x) * W;
  const int first = static_cast<int>(blockIdx.x) * W;
  const size_t unit_elems = static_cast<size_t>(3) * D;
  const int cpw = (nch + W - 1) / W;
  const int c0 = wave * cpw;
  uint4 rg[R][NCH], ru[R][NCH], rd[R][W][DS];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int ub = r * band + first;
    const int u = ub + wave;
    const int uc = u < total ? u : total - 1;
    const int d = uc / I;
    const T* base = reinterpret_cast<const T*>(a.blob[d]) + static_cast<size_t>(uc - d * I) * unit_elems;
    load_chunks<NCH, false, true>(base, lane, nch, rg[r]);
    load_chunks<NCH, false, true>(base + D, lane, nch, ru[r]);
#pragma unroll
    for (int w2 = 0; w2 < W; ++w2) {
      const int v = ub + w2;
      const int vc = v < total ? v : total - 1;
      const int d2 = vc / I;
      const T* dbase = reinterpret_cast<const T*>(a.blob[d2]) + static_cast<size_t>(vc - d2 * I) * unit_elems + 2 * D;
#pragma unroll
      for (int s = 0; s < DS; ++s) {
        const int c = c0 + lane + 64 * s;
        rd[r][w2][s] = ld_chunk<true>(dbase, lane + 64 * s < cpw && c < nch ? c : 0);
      }
    }
  }
  uint32_t z = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int j = 0; j < NCH; ++j) z ^= rg[r][j].x ^ rg[r][j].w ^ ru[r][j].y ^ ru[r][j].z;
#pragma unroll
    for (int w2 = 0; w2 < W; ++w2)
#pragma unroll
      for (int s = 0; s < DS; ++s) z ^= rd[r][w2][s].x ^ rd[r][w2][s].w;
  }
  z = __builtin_amdgcn_readfirstlane(z) ^ __builtin_amdgcn_readlane(z, 63);
  if (threadIdx.x == 0) sink[blockIdx.x] = z;
}

// ---------------------------------------------------------------------------
// Routed-expert SwiGLU FFN over 4-bit experts (batch 1).  Unit i of an expert
// is one contiguous run: [gate codes | up codes | down codes] (D/2 bytes each,
// two codes per byte, low nibble first) then [gate | up | down scales] (D/32
// fp16 each); value = scale * (q - 8) per block of 32 elements along D.
// Lane l owns blocks l and l + 64 (NQ of them): one 16-byte code load and one
// 2-byte scale load per row and block.
//   gate/up: integer dot products.  x of a block is taken in fixed point,
//     X_k = rint(x_k 2^(18 - e)) with e the frexp exponent of the block's
//     largest |x_k| (so |X_k| <= 2^18, |x_k - X_k 2^(e-18)| <= 2^-18 of that
//     largest value), written in five balanced base-16 digits
//     X_k = sum_j 16^j d_jk, d_jk in [-8, 7].  A code word XOR 0x88888888
//     holds q - 8 as signed nibbles, so sum_k (q_k - 8) X_k =
//     sum_j 16^j dot8(q ^ 8, d_j) with v_dot8c_i32_i4 (8 products per
//     instruction), exact in int32 (|.| <= 2^26); the block adds
//     scale 2^(e-18) float(that sum).  The workgroup forms the digit words
//     once: thread t takes word t % 4 (8 elements) of block t / 4, the
//     block's largest |x| by two quad permutes, X_k + 0x88888 by one float
//     add (rounding to nearest even), and the digit words by a nibble
//     transpose of byte and half-word permutes; the words pass through LDS
//     behind the first pass's weight loads.
//   down: the accumulation adds (h scale) q per element (q converted by
//     v_cvt_f32_ubyte*) and subtracts 8 sum(h scale) per block at the end.
// Work list and workgroup partials as in ffn_units_kernel.  PASSES = 0: the
// units kernel's assignment (workgroup b on units [b*upw, (b+1)*upw), which
// the FFN split needs); PASSES = 1 or 2: sweep order as in ffn_slices_kernel
// -- global wave g takes units g + NW (pass UPP + p), NW = G W, so the grid
// streams one band of consecutive units at a time (8 Qwen-shaped experts:
// 10.0 us at 512 workgroups of one pass against 11.0 us for the best range
// assignment, 256 workgroups of two passes).  The integer gate/up products
// took the Qwen-shaped launch from 8.5 to 8.0 us in isolation (9.5 to 9.0 us
// behind a 512 MB read); fp32 products cost a convert and an FMA per code.
// ---------------------------------------------------------------------------
constexpr int kQ4TargetWgs = 256;

__device__ __forceinline__ float q4_scale(uint16_t bits) {
  return static_cast<float>(__builtin_bit_cast(_Float16, bits));
}

// Nibble mask the optimiser cannot see through: with the mask visible it
// turns the four byte converts below into per-nibble extracts (two ops each)
// instead of v_cvt_f32_ubyte0..3 (one op each).
__device__ __forceinline__ uint32_t low_nibbles(uint32_t w) {
  uint32_t r;
  asm("v_and_b32 %0, 0x0f0f0f0f, %1" : "=v"(r) : "v"(w));
  return r;
}

// The 32 codes of one block (16 bytes) as floats q_0..q_31, in element order.
__device__ __forceinline__ void q4_codes(const uint4& c, float (&q)[32]) {
  const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const uint32_t lo = low_nibbles(w[m]), hi = low_nibbles(w[m] >> 4);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      q[8 * m + 2 * b] = static_cast<float>((lo >> (8 * b)) & 0xFFu);
      q[8 * m + 2 * b + 1] = static_cast<float>((hi >> (8 * b)) & 0xFFu);
    }
  }
}

// The weight loads of one pass: units ub + p * ustride (p < UPP) of this wave.
// No branch in front of the loads: a unit past the range re-reads the range's
// last unit, a lane past the row's blocks reads block 0 (its x digits are
// zero and its outputs are not stored).
template <int NQ, bool FULLQ, int UPP, bool ROUTED>
__device__ __forceinline__ void q4_pass_loads(const FfnArgs& a, const Items<ROUTED>& items, int ub, int ustride, int u1, int lane,
                                              uint4 (&cg)[UPP][NQ], uint4 (&cu)[UPP][NQ], uint4 (&cd)[UPP][NQ],
                                              uint16_t (&sg)[UPP][NQ], uint16_t (&su)[UPP][NQ],
                                              uint16_t (&sd)[UPP][NQ], float (&gate)[UPP]) {
  const int D = a.D, I = a.I, nblk = D / 32;
  const size_t cb = static_cast<size_t>(D) / 2, sb = static_cast<size_t>(nblk) * 2;
  const size_t unit_bytes = 3 * cb + 3 * sb;
#pragma unroll
  for (int p = 0; p < UPP; ++p) {
    const int uu = ub + p * ustride;
    const int uc = uu < u1 ? uu : u1 - 1;  // wave-uniform
    const int d = uc / I;
    const int i = uc - d * I;
    const uint8_t* base = reinterpret_cast<const uint8_t*>(items.blob(a, d)) + static_cast<size_t>(i) * unit_bytes;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int blk = (FULLQ || lane + 64 * q < nblk) ? lane + 64 * q : 0;
      const u32x4 g4 = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base + 16 * blk));
      const u32x4 u4 = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base + cb + 16 * blk));
      const u32x4 d4 = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base + 2 * cb + 16 * blk));
      cg[p][q] = make_uint4(g4.x, g4.y, g4.z, g4.w);
      cu[p][q] = make_uint4(u4.x, u4.y, u4.z, u4.w);
      cd[p][q] = make_uint4(d4.x, d4.y, d4.z, d4.w);
      sg[p][q] = *SPP_GLOBAL(uint16_t, base + 3 * cb + 2 * blk);
      su[p][q] = *SPP_GLOBAL(uint16_t, base + 3 * cb + sb + 2 * blk);
      sd[p][q] = *SPP_GLOBAL(uint16_t, base + 3 * cb + 2 * sb + 2 * blk);
    }
    gate[p] = items.gate(a, d);
  }
}

// Digit words of 8 consecutive elements x_0..x_7 of a block whose largest
// |x| has frexp exponent e: nibble k of word j is d_jk (two's complement).
// Y_k = (X_k + 0x88888) ^ 0x88888 holds d_0k..d_4k in its five low nibbles
// (X_k + 0x88888 = sum_j (d_jk + 8) 16^j with every digit in [0, 15]); the
// float sum x_k 2^(18-e) + 1.5 * 2^23 rounds X_k to nearest even and leaves
// X_k + 2^22 in the mantissa.  The transpose: half-words of Y_k and Y_k+4,
// then bytes of those pairs, then nibbles.
__device__ __forceinline__ void q4_x_digits(const float (&xe)[8], int e, uint32_t (&w)[5]) {
  const float sc = ldexpf(1.f, 18 - e);
  uint32_t Y[8];
#pragma unroll
  for (int k = 0; k < 8; ++k)
    Y[k] = (__float_as_uint(fmaf(xe[k], sc, 12582912.f)) - (0x4B400000u - 0x88888u)) ^ 0x88888u;
  uint32_t P[4], Q[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    P[k] = __builtin_amdgcn_perm(Y[k + 4], Y[k], 0x05040100u);  // low halves: nibbles 0-3 of Y_k, Y_k+4
    Q[k] = __builtin_amdgcn_perm(Y[k + 4], Y[k], 0x07060302u);  // high halves: nibble 4 of Y_k, Y_k+4
  }
  uint32_t R[2], S[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    R[k] = __builtin_amdgcn_perm(P[k + 2], P[k], 0x06020400u);  // byte 0 of Y_k, Y_k+2, Y_k+4, Y_k+6
    S[k] = __builtin_amdgcn_perm(P[k + 2], P[k], 0x07030501u);  // byte 1 of the same
  }
  w[0] = (R[0] & 0x0F0F0F0Fu) | ((R[1] & 0x0F0F0F0Fu) << 4);
  w[1] = ((R[0] >> 4) & 0x0F0F0F0Fu) | (R[1] & 0xF0F0F0F0u);
  w[2] = (S[0] & 0x0F0F0F0Fu) | ((S[1] & 0x0F0F0F0Fu) << 4);
  w[3] = ((S[0] >> 4) & 0x0F0F0F0Fu) | (S[1] & 0xF0F0F0F0u);
  w[4] = Q[0] | (Q[1] << 4) | (Q[2] << 8) | (Q[3] << 12);
}

template <int NQ, bool FULLQ, int UPP, int PASSES, bool ROUTED>
__device__ __forceinline__ void ffn_q4_body(const FfnArgs& a, const RouterArgs* ra, int bid, int nblocks) {
  static_assert(kFfnThreads == 256, "the digit words take four threads per block, 64 blocks per pass");
  extern __shared__ float s_red[];  // [kFfnWaves][D] wave partials
  __shared__ uint4 s_dig[NQ * 64 * 5];  // [block][digit j] words 0..3
  __shared__ float s_eb[NQ * 64];       // [block] 2^(e - 18)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, I = a.I, nblk = D / 32;
  if (PASSES == 0 && ((a.skip_mask >> ((bid * a.upw) / I)) & 1u)) return;  // another launch's item

  // this thread's 8 elements of x per q: word tid % 4 of block tid / 4 + 64 q
  // (a block past the row reads block 0; its words are never used)
  float xe[NQ][8];
  if constexpr (ROUTED) {
    // the row's scale as the router forms it (16-byte chunk lane + 64 j in lane
    // order); the thread's own elements are chunk tid + 256 q
    constexpr int NCH = 4 * NQ;
    const int nch = D / 8;
    float xv[NCH][8], own[NQ][8];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = tid + 256 * q;
      const int cc = FULLQ || c < nch ? c : 0;
      if (ra->u) {
        unpack<float>(ld16(ra->u + 8 * cc), own[q]);
        unpack<float>(ld16(ra->u + 8 * cc + 4), own[q] + 4);
      } else {
        unpack<uint16_t>(ld16(reinterpret_cast<const uint16_t*>(ra->h) + 8 * cc), own[q]);
      }
    }
    if (ra->u) {
      load_row_f32<uint16_t, NCH, FULLQ>(ra->u, lane, nch, xv);
    } else {
      load_row_storage<uint16_t, NCH, FULLQ>(reinterpret_cast<const uint16_t*>(ra->h), lane, nch, xv);
    }
    const float inv = rms_scale<uint16_t, NCH>(xv, D, ra->eps);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int k = 0; k < 8; ++k) xe[q][k] = own[q][k] * inv;
  } else {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int bq = (tid >> 2) + 64 * q;
      const float* xs = a.x + 32 * (FULLQ || bq < nblk ? bq : 0) + 8 * (tid & 3);
      const float4 v0 = *SPP_GLOBAL(float4, xs), v1 = *SPP_GLOBAL(float4, xs + 4);
      xe[q][0] = v0.x; xe[q][1] = v0.y; xe[q][2] = v0.z; xe[q][3] = v0.w;
      xe[q][4] = v1.x; xe[q][5] = v1.y; xe[q][6] = v1.z; xe[q][7] = v1.w;
    }
  }

  const int total = a.nW * I;
  // range assignment: units [u0, u1) of this workgroup, wave stride kFfnWaves;
  // sweep order: the whole grid's units, stride NW
  const int NW = nblocks * kFfnWaves;
  const int u0 = PASSES ? 0 : bid * a.upw;
  const int u1 = PASSES ? total : min(u0 + a.upw, total);
  const int ustride = PASSES ? NW : kFfnWaves;
  const int ub0 = PASSES ? bid * kFfnWaves + wave : u0 + wave;
  const int npass = PASSES ? PASSES : (a.upw + kFfnWaves * UPP - 1) / (kFfnWaves * UPP);
  uint4 cg[UPP][NQ], cu[UPP][NQ], cd[UPP][NQ];
  uint16_t sg[UPP][NQ], su[UPP][NQ], sd[UPP][NQ];
  float gate[UPP];
  // the first pass's weight loads go out before the digit words are formed
  // (a routed workgroup forms them while it waits for the routing)
  const bool first = !(PASSES == 0 && ub0 >= u1);  // wave-uniform
  Items<ROUTED> items;
  if (!ROUTED && first) q4_pass_loads<NQ, FULLQ, UPP>(a, items, ub0, ustride, u1, lane, cg, cu, cd, sg, su, sd, gate);
  __builtin_amdgcn_sched_barrier(0);

  // digit words of x, one block per four threads, through LDS
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    float m = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) m = fmaxf(m, fabsf(xe[q][k]));
    m = fmaxf(m, dpp<0xB1>(m));  // quad_perm [1,0,3,2]: the block's four threads
    m = fmaxf(m, dpp<0x4E>(m));  // quad_perm [2,3,0,1]
    const int e = m > 0.f ? __builtin_amdgcn_frexp_expf(m) : 0;
    uint32_t w[5];
    q4_x_digits(xe[q], e, w);
    const int bq = (tid >> 2) + 64 * q;
    uint32_t* s_dw = reinterpret_cast<uint32_t*>(s_dig);
#pragma unroll
    for (int j = 0; j < 5; ++j) s_dw[(bq * 5 + j) * 4 + (tid & 3)] = w[j];
    if ((tid & 3) == 0) s_eb[bq] = ldexpf(1.f, e - 18);
  }
  if constexpr (ROUTED) {
    items.words = route_words(*ra, bid, lane, wave, [&]() {  // its barrier also publishes the digit words
      constexpr int NCH = 4 * NQ;
      float xv[NCH][8];
      input_x<uint16_t, NCH, FULLQ>(*ra, lane, D / 8, xv);
      return route_self<uint16_t, NCH, FULLQ>(*ra, xv, lane);
    });
    q4_pass_loads<NQ, FULLQ, UPP>(a, items, ub0, ustride, u1, lane, cg, cu, cd, sg, su, sd, gate);
    __builtin_amdgcn_sched_barrier(0);
  } else {
    __syncthreads();
  }
  uint32_t xd[NQ][5][4];
  float eb[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int blk = lane + 64 * q;
    const bool ok = FULLQ || blk < nblk;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const uint4 t = s_dig[blk * 5 + j];
      xd[q][j][0] = ok ? t.x : 0u;
      xd[q][j][1] = ok ? t.y : 0u;
      xd[q][j][2] = ok ? t.z : 0u;
      xd[q][j][3] = ok ? t.w : 0u;
    }
    eb[q] = ok ? s_eb[blk] : 0.f;
  }

  float acc[NQ][32], corr[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    corr[q] = 0.f;
#pragma unroll
    for (int j = 0; j < 32; ++j) acc[q][j] = 0.f;
  }
  for (int pr = 0; pr < npass; ++pr) {
    const int ub = ub0 + pr * UPP * ustride;
    if (PASSES == 0 && ub >= u1) break;  // wave-uniform
    if (pr > 0) q4_pass_loads<NQ, FULLQ, UPP>(a, items, ub, ustride, u1, lane, cg, cu, cd, sg, su, sd, gate);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < UPP; ++p) {
      if (ub + p * ustride >= u1) continue;  // wave-uniform: no work past the range (its loads are harmless)
      float gs = 0.f, us = 0.f;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const uint32_t wg[4] = {cg[p][q].x, cg[p][q].y, cg[p][q].z, cg[p][q].w};
        const uint32_t wu[4] = {cu[p][q].x, cu[p][q].y, cu[p][q].z, cu[p][q].w};
        int tg[5] = {0, 0, 0, 0, 0}, tu[5] = {0, 0, 0, 0, 0};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int qg = static_cast<int>(wg[m] ^ 0x88888888u), qu = static_cast<int>(wu[m] ^ 0x88888888u);
#pragma unroll
          for (int j = 0; j < 5; ++j) {
            tg[j] = __builtin_amdgcn_sdot8(qg, static_cast<int>(xd[q][j][m]), tg[j], false);
            tu[j] = __builtin_amdgcn_sdot8(qu, static_cast<int>(xd[q][j][m]), tu[j], false);
          }
        }
        const int Tg = (((tg[4] * 16 + tg[3]) * 16 + tg[2]) * 16 + tg[1]) * 16 + tg[0];
        const int Tu = (((tu[4] * 16 + tu[3]) * 16 + tu[2]) * 16 + tu[1]) * 16 + tu[0];
        gs += q4_scale(sg[p][q]) * eb[q] * static_cast<float>(Tg);
        us += q4_scale(su[p][q]) * eb[q] * static_cast<float>(Tu);
      }
      const float g = wave_sum(gs);
      const float u = wave_sum(us);
      const float hval = g / (1.f + expf(-g)) * u * gate[p];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const float hs = hval * q4_scale(sd[p][q]);
        float qd[32];
        q4_codes(cd[p][q], qd);
        corr[q] += hs;
#pragma unroll
        for (int j = 0; j < 32; ++j) acc[q][j] += hs * qd[j];
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int j = 0; j < 32; ++j) acc[q][j] -= 8.f * corr[q];

  // sum the waves of this workgroup in a fixed order, (w0 + w2) + (w1 + w3),
  // after one barrier.  LDS layout per wave: element 32 blk + 4k + e (k < 8,
  // e < 4) at word 32 blk + 4 (k ^ (blk & 7)) + e, so that the 16-byte stores
  // of eight consecutive lanes (blocks 128 bytes apart) and the natural-order
  // reads both touch every bank once (a plain layout puts all 64 lanes on one
  // bank: 3-8 us per launch; a second barrier and pass cost 0.3 us).
  static_assert(kFfnWaves == 4, "the fold order below is written for four waves");
  float4* s_red4 = reinterpret_cast<float4*>(s_red);
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int blk = lane + 64 * q;
    if (FULLQ || blk < nblk) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        s_red4[(wave * D + 32 * blk) / 4 + (k ^ (blk & 7))] =
            make_float4(acc[q][4 * k], acc[q][4 * k + 1], acc[q][4 * k + 2], acc[q][4 * k + 3]);
    }
  }
  __syncthreads();
  float* out = a.partial + static_cast<size_t>(bid) * D;
  for (int d = tid; d < D; d += kFfnThreads) {
    const int blk = d >> 5, j = d & 31;
    const int w = 32 * blk + 4 * ((j >> 2) ^ (blk & 7)) + (j & 3);
    out[d] = (s_red[w] + s_red[2 * D + w]) + (s_red[D + w] + s_red[3 * D + w]);
  }
}

template <int NQ, bool FULLQ, int UPP, int PASSES>
__global__ __launch_bounds__(kFfnThreads) void ffn_q4_kernel(FfnArgs a) {
  ffn_q4_body<NQ, FULLQ, UPP, PASSES, false>(a, nullptr, blockIdx.x, gridDim.x);
}

// Router and 4-bit FFN of one token in one launch, as layer_slices_kernel.
template <int NCH, bool FULL, int NQ, bool FULLQ, int PASSES>
__global__ __launch_bounds__(kFfnThreads) void layer_q4_kernel(RouterArgs ra, FfnArgs fa, int rb) {
  const int b = blockIdx.x;
  if (b < rb)
    router_adapter_body<uint16_t, NCH, FULL, 2, false>(ra, b, rb);
  else
    ffn_q4_body<NQ, FULLQ, 3, PASSES, true>(fa, &ra, b - rb, static_cast<int>(gridDim.x) - rb);
}

// Plain streaming read (measurement only): n16 16-byte chunks from base,
// contiguous, each wave taking kStreamIn consecutive 1 KiB pieces (64 lanes x
// 16 bytes) per step of a grid-stride loop, non-temporal; the words are folded
// and stored only on a magic value.  The ceiling of reading the FFN's bytes
// with no access pattern of its own.
constexpr int kStreamIn = 8;
constexpr int kStreamGrid = 2048;
__global__ __launch_bounds__(256) void stream_probe_kernel(const u32x4* __restrict__ base, size_t n16, uint32_t* sink) {
  const size_t lane = threadIdx.x & 63;
  const size_t wave = (static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x) >> 6;
  const size_t nwaves = static_cast<size_t>(gridDim.x) * 4;
  uint32_t z = 0;
  for (size_t b0 = wave * 64 * kStreamIn; b0 < n16; b0 += nwaves * 64 * kStreamIn) {
    u32x4 v[kStreamIn];
#pragma unroll
    for (int k = 0; k < kStreamIn; ++k) {
      const size_t i = b0 + 64 * k + lane;
      v[k] = __builtin_nontemporal_load(base + (i < n16 ? i : n16 - 1));  // past the end: re-read the last chunk
    }
#pragma unroll
    for (int k = 0; k < kStreamIn; ++k) z ^= v[k].x ^ v[k].y ^ v[k].z ^ v[k].w;
  }
  if (z == 0x9E3779B9u) sink[threadIdx.x] = z;
}

// Read-ceiling probe of ffn_q4_kernel in sweep order (measurement only): the
// same grid, passes, unit order and loads -- 16-byte non-temporal code loads
// and 2-byte scale loads per row and block -- folded into one checksum per
// workgroup, with no decode, arithmetic or LDS.
template <int NQ, bool FULLQ, int PASSES>
__global__ __launch_bounds__(kFfnThreads) void read_probe_q4_kernel(FfnArgs a, uint32_t* sink) {
  constexpr int UPP = 3;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int D = a.D, I = a.I, nblk = D / 32;
  const size_t cb = static_cast<size_t>(D) / 2, sb = static_cast<size_t>(nblk) * 2;
  const size_t unit_bytes = 3 * cb + 3 * sb;
  const int total = a.nW * I;
  const int NW = static_cast<int>(gridDim.x) * kFfnWaves;
  const int ub0 = static_cast<int>(blockIdx.x) * kFfnWaves + wave;
  uint32_t z = 0;
#pragma unroll
  for (int pr = 0; pr < PASSES; ++pr) {
    const int ub = ub0 + pr * UPP * NW;
    u32x4 cg[UPP][NQ], cu[UPP][NQ], cd[UPP][NQ];
    uint16_t sg[UPP][NQ], su[UPP][NQ], sd[UPP][NQ];
#pragma unroll
    for (int p = 0; p < UPP; ++p) {
      const int uu = ub + p * NW;
      const int uc = uu < total ? uu : total - 1;
      const int d = uc / I;
      const uint8_t* base = reinterpret_cast<const uint8_t*>(a.blob[d]) + static_cast<size_t>(uc - d * I) * unit_bytes;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int blk = (FULLQ || lane + 64 * q < nblk) ? lane + 64 * q : 0;
        cg[p][q] = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base + 16 * blk));
        cu[p][q] = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base + cb + 16 * blk));
        cd[p][q] = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base + 2 * cb + 16 * blk));
        sg[p][q] = *SPP_GLOBAL(uint16_t, base + 3 * cb + 2 * blk);
        su[p][q] = *SPP_GLOBAL(uint16_t, base + 3 * cb + sb + 2 * blk);
        sd[p][q] = *SPP_GLOBAL(uint16_t, base + 3 * cb + 2 * sb + 2 * blk);
      }
    }
#pragma unroll
    for (int p = 0; p < UPP; ++p)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        z ^= cg[p][q].x ^ cu[p][q].y ^ cd[p][q].z ^ cg[p][q].w ^ (static_cast<uint32_t>(sg[p][q] ^ su[p][q] ^ sd[p][q]) << 7);
  }
  z = __builtin_amdgcn_readfirstlane(z) ^ __builtin_amdgcn_readlane(z, 63);
  if (threadIdx.x == 0) sink[blockIdx.x] = z;
}

// y = sum of the workgroup partials (fixed order), h_out = round(residual + y).
// kCombGroups groups split the partial rows: group g adds rows g*kCombRows..
// of every pass in order, then the groups are added in order.  A thread holds 4
// columns of one group; a pass's loads (512 rows) all go out before the first
// add, 128 contiguous bytes per row and workgroup.  Latency bound: 3.9 us for
// 512 rows of 2048 columns (4.05 with a column per thread, 64 per workgroup).
constexpr int kCombGroups = 16;
constexpr int kCombRows = 32;
constexpr int kCombCols = 32;
constexpr int kCombLanes = kCombCols / 4;
constexpr int kCombThreads = kCombGroups * kCombLanes;

template <typename T>
__global__ __launch_bounds__(kCombThreads) void ffn_combine_kernel(CombineArgs a) {
  __shared__ float4 s_part[kCombGroups][kCombLanes];
  const int tid = threadIdx.x;
  const int cl = tid % kCombLanes, grp = tid / kCombLanes;
  const int col = min(static_cast<int>(blockIdx.x) * kCombCols + 4 * cl, a.D - 4);  // lanes past D re-read the last columns
  // the residual of thread t < kCombCols: its column
  const int oc = static_cast<int>(blockIdx.x) * kCombCols + tid;
  const bool out = tid < kCombCols && oc < a.D;
  float res = 0.f;
  if (out) res = a.res_u ? a.res_u[oc] : load_elem<T>(a.res_h, oc);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int w0 = grp * kCombRows; w0 < a.nparts; w0 += kCombGroups * kCombRows) {
    float4 v[kCombRows];
#pragma unroll
    for (int k = 0; k < kCombRows; ++k)
      v[k] = *SPP_GLOBAL(float4, a.partial + static_cast<size_t>(min(w0 + k, a.nparts - 1)) * a.D + col);
#pragma unroll
    for (int k = 0; k < kCombRows; ++k) {
      const bool on = w0 + k < a.nparts;
      s.x += on ? v[k].x : 0.f;
      s.y += on ? v[k].y : 0.f;
      s.z += on ? v[k].z : 0.f;
      s.w += on ? v[k].w : 0.f;
    }
  }
  s_part[grp][cl] = s;
  __syncthreads();
  if (out) {
    const float* p = reinterpret_cast<const float*>(s_part) + tid;
    float y = p[0];
#pragma unroll
    for (int g = 1; g < kCombGroups; ++g) y += p[g * kCombCols];
    store_elem<T>(a.out, oc, res + y);
  }
}

// ---------------------------------------------------------------------------
// Batched decode over the tiled expert layout (nb = D/256 column blocks,
// I/16 tiles of 16 units):
//   gate/up part, 16-byte pieces in MFMA operand order: piece
//     (((tile*nb + blk)*2 + w)*8 + j)*64 + l  holds  W_w[16 tile + l%16][256 blk + 32 j + 8 (l/16) + e],
//     e < 8, w = 0 gate / 1 up -- one wave load of step j is 1 KiB contiguous;
//   down part, after the 2*I*D gate/up elements: run (s*I + i) holds
//     W_down[256 s + c][i], c < 256 -- consecutive units of a slice are contiguous.
// One workgroup takes one group (up to 32 tokens that share an expert) and one
// range of upw units of that expert.  The groups are not listed anywhere: every
// workgroup counts the routing's experts in LDS, finds the (expert, 32-token
// chunk) of its group index and collects that chunk's (token, k) pairs in pair
// order, so no list crosses the host link and the host need not know the
// routing.  Shared experts come first, over every token.
//   phase A: G = X W_gate^T and U = X W_up^T on v_mfma_f32_16x16x32_bf16, tokens
//     as rows (one or two tiles of 16), units as the 16 columns; wave w owns the
//     unit tiles w, w + 4, ... of the range.  x comes as a bf16 pair x = hi + lo
//     straight from global memory in operand order (rows past the group's end
//     repeat its last token; a few rows sit in the cache), both halves are
//     multiplied, so the contraction keeps x to ~2^-17 relative.  No barrier:
//     weights and x of the next columns load while these are multiplied.
//   H = silu(G) * U goes to LDS as three bf16 terms whose sum is the fp32 value
//     exactly (8 + 8 + 8 bits, truncated).
//   phase B: Y = H W_down^T on the same instruction, units as the contraction.
//     A lane loads 16 bytes (8 columns) of each of 8 units; the B operand of
//     column c is one byte permute per pair of units, so a wave covers 128
//     columns x 32 units per step with 8 loads, 32 permutes and 8 MFMAs per
//     term and token tile.  The first step's loads go out before the barrier.  One partial output row per (token, range).
// Bound by HBM: at 64 tokens over 128 Qwen-shaped experts the launch takes
// 183 us (6.5 TB/s of weights; its loads alone 176), from 205 us with x staged
// through LDS behind barriers, the down product on the vector units and 4
// ranges; at 256 tokens 215 us from 335 (16 tokens on the vector units, and
// experts of more than 16 tokens read twice); at 4 tokens 47 us from 56.
constexpr int kGrpBlk = 256;  // columns per block of the tiled layout: 8 k-steps of 32

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// H in LDS: [3 terms][kGroupTokens][row]; rows padded to whole steps of 32 units
// and by 16 bytes (rows then start on different banks)
__host__ __device__ constexpr int grp_h_row(int upw) { return (upw + 31) / 32 * 32 + 8; }
// position of unit u in a row: within each step of 32 units, lane group g's
// contraction index kk is unit 4 kk + g, so that one load of phase B reads
// four consecutive runs
__device__ __forceinline__ int grp_h_pos(int u) { return (u & ~31) + 8 * (u & 3) + ((u & 31) >> 2); }
uint32_t grp_lds_bytes(int upw) { return 3u * kGroupTokens * grp_h_row(upw) * sizeof(uint16_t); }

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// Phase A of one wave over NT unit tiles and TT token tiles; tile0 + 4 q are
// the tiles (of the expert), xo[tt] the lane's offset into the x planes.
template <int W, int NT, int TT>
__device__ __forceinline__ void grp_phase_a(const GroupArgs& a, const uint16_t* blob, int tile0, int local0, int lane,
                                            const uint32_t (&xo)[2], uint16_t* s_h, int hrow) {
  constexpr int KS = NT == 1 ? 4 : 2;  // k-steps of 32 columns per stage
  const int D = a.D, nb = D / kGrpBlk;
  struct Stage {
    u32x4 g[NT][KS], u[NT][KS], xh[TT][KS], xl[TT][KS];
  } s0, s1;
  f32x4 accg[NT][TT], accu[NT][TT];
#pragma unroll
  for (int q = 0; q < NT; ++q)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) accg[q][tt] = accu[q][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const u32x4* base[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q)
    base[q] = reinterpret_cast<const u32x4*>(blob) + static_cast<size_t>(tile0 + W * q) * nb * 1024 + lane;
  auto load = [&](Stage& s, int i) {
    const int k = i * KS;                            // k-step of 32 columns
    const size_t po = static_cast<size_t>(k >> 3) * 1024 + (k & 7) * 64;
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int j = 0; j < KS; ++j) {
        s.g[q][j] = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base[q] + po + j * 64));
        s.u[q][j] = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, base[q] + po + 512 + j * 64));
      }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int j = 0; j < KS; ++j) {
        s.xh[tt][j] = *SPP_GLOBAL(u32x4, a.xh + xo[tt] + 32 * (k + j));
        s.xl[tt][j] = *SPP_GLOBAL(u32x4, a.xl + xo[tt] + 32 * (k + j));
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mul = [&](const Stage& s) {
#pragma unroll
    for (int j = 0; j < KS; ++j)
#pragma unroll
      for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          accg[q][tt] = mfma_bf16(s.xh[tt][j], s.g[q][j], accg[q][tt]);
          accu[q][tt] = mfma_bf16(s.xh[tt][j], s.u[q][j], accu[q][tt]);
          accg[q][tt] = mfma_bf16(s.xl[tt][j], s.g[q][j], accg[q][tt]);
          accu[q][tt] = mfma_bf16(s.xl[tt][j], s.u[q][j], accu[q][tt]);
        }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int n = D / (32 * KS);  // even: D is a multiple of 256
  load(s0, 0);
  for (int i = 0; i < n; i += 2) {
    load(s1, i + 1);
    mul(s0);
    if (i + 2 < n) load(s0, i + 2);
    mul(s1);
  }
  // this lane holds tokens 16 tt + 4 (lane / 16) + j of unit lane % 16 of each tile
#pragma unroll
  for (int q = 0; q < NT; ++q)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float g = accg[q][tt][j];
        const float h = g / (1.f + expf(-g)) * accu[q][tt][j];
        const uint32_t hb = __float_as_uint(h);
        // exact: each term takes the next 8 significant bits (a non-finite h stays in the first)
        const float r1 = (hb & 0x7f800000u) == 0x7f800000u ? 0.f : h - __uint_as_float(hb & 0xffff0000u);
        const uint32_t mb = __float_as_uint(r1);
        const uint32_t lb = __float_as_uint(r1 - __uint_as_float(mb & 0xffff0000u));
        uint16_t* o = s_h + (16 * tt + 4 * (lane >> 4) + j) * hrow + grp_h_pos((local0 + W * q) * 16 + (lane & 15));
        o[0] = static_cast<uint16_t>(hb >> 16);
        o[kGroupTokens * hrow] = static_cast<uint16_t>(mb >> 16);
        o[2 * kGroupTokens * hrow] = static_cast<uint16_t>(lb >> 16);
      }
}

// Phase B's loads of one step: 128 columns of slab `slab` x units u0 + 4 kk + g.
__device__ __forceinline__ void grp_load_down(const GroupArgs& a, const uint16_t* down, int i0, int nu, int slab, int u0,
                                              int lane, u32x4 (&r)[8]) {
  const uint16_t* p = down + (static_cast<size_t>(slab >> 1) * a.I + i0) * kGrpBlk + (slab & 1) * 128 + 8 * (lane & 15);
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)  // a unit past the range re-reads its last one (zeroed before use)
    r[kk] = __builtin_nontemporal_load(
        SPP_GLOBAL(u32x4, p + static_cast<size_t>(min(u0 + 4 * kk + (lane >> 4), nu - 1)) * kGrpBlk));
  __builtin_amdgcn_sched_barrier(0);
}

// NaN outputs of the three-term products, formed again as one product per unit
// in unit order: a term of h that is 0 times an infinite weight is a NaN where
// h times the weight is infinite.  Reached only by a wave whose outputs add up to
// a NaN (one addition per value); each lane reads back what it stored itself.
template <int W, int TT>
__device__ __forceinline__ void grp_nan_outputs(const GroupArgs& a, const uint16_t* down, int i0, int nu, int m, int split,
                                           int wave, int lane, const uint16_t* s_h, int hrow, const int* s_pair) {
  const int D = a.D;
#pragma unroll 1
  for (int slab = wave; slab < D / 128; slab += W) {
    const int d0 = 128 * slab + 8 * (lane & 15);
    const uint16_t* p = down + (static_cast<size_t>(slab >> 1) * a.I + i0) * kGrpBlk + (slab & 1) * 128 + 8 * (lane & 15);
#pragma unroll 1
    for (int q = 0; q < 4 * TT; ++q) {
      const int t = 16 * (q >> 2) + 4 * (lane >> 4) + (q & 3);
      if (t >= m) continue;
      float* dst = a.ypart + (static_cast<size_t>(s_pair[t]) * a.nsplit + split) * D + d0;
      bool bad = false;
#pragma unroll
      for (int c = 0; c < 8; ++c) bad = bad || isnan(dst[c]);
      if (!bad) continue;
      float y[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int u = 0; u < nu; ++u) {
        const uint16_t* hp = s_h + t * hrow + grp_h_pos(u);
        float h = 0.f;  // the lowest term first: every sum is exact
#pragma unroll
        for (int k = 2; k >= 0; --k) h += __uint_as_float(static_cast<uint32_t>(hp[k * kGroupTokens * hrow]) << 16);
        float w[8];
        unpack<uint16_t>(ld16(p + static_cast<size_t>(u) * kGrpBlk), w);
#pragma unroll
        for (int c = 0; c < 8; ++c) y[c] = fmaf(h, w[c], y[c]);
      }
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (isnan(dst[c])) dst[c] = y[c];
    }
  }
}

// r0 holds the loads of the wave's first step.
template <int W, int TT>
__device__ __forceinline__ void grp_phase_b(const GroupArgs& a, const uint16_t* down, int i0, int nu, int m, int split,
                                            int wave, int lane, const uint16_t* s_h, int hrow, const int* s_pair,
                                            u32x4 (&r0)[8]) {
  const int D = a.D;
  const int nsteps = (nu + 31) >> 5;
  const int nslab = D / 128;
  const int mine = (nslab - wave + W - 1) / W;  // slabs wave, wave + 4, ...
  const int total = mine * nsteps;
  u32x4 r1[8];
  f32x4 acc[TT][8];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[tt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  // steps in order: every step of a slab, then the next slab
  int lslab = wave, lst = 0;  // of the next load
  auto advance = [&]() {
    if (++lst == nsteps) {
      lst = 0;
      lslab += W;
    }
  };
  int slab = wave, st = 0;  // of the next multiply
  float sum = 0.f;          // of the values stored: a NaN if one of them is
  auto mul = [&](u32x4 (&r)[8]) {
    if (32 * st + 32 > nu)  // nu is a multiple of 16: the upper half of the step is past the range
#pragma unroll
      for (int kk = 4; kk < 8; ++kk) r[kk] = u32x4{0, 0, 0, 0};
    u32x4 h[TT][3];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        h[tt][p] = *reinterpret_cast<const u32x4*>(s_h + (p * kGroupTokens + 16 * tt + (lane & 15)) * hrow + 32 * st +
                                                   8 * (lane >> 4));
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      u32x4 b;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        b[q] = __builtin_amdgcn_perm(r[2 * q + 1][c >> 1], r[2 * q][c >> 1], (c & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        acc[tt][c] = mfma_bf16(h[tt][2], b, acc[tt][c]);
        acc[tt][c] = mfma_bf16(h[tt][1], b, acc[tt][c]);
        acc[tt][c] = mfma_bf16(h[tt][0], b, acc[tt][c]);
      }
    }
    if (++st == nsteps) {
      // this lane holds tokens 16 tt + 4 (lane / 16) + j of 8 consecutive columns
      const int d0 = 128 * slab + 8 * (lane & 15);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int t = 16 * tt + 4 * (lane >> 4) + j;
          if (t < m) {
            // ordinary stores: non-temporal ones took 188 us against 183 (64 tokens, 128 Qwen-shaped experts)
            float* dst = a.ypart + (static_cast<size_t>(s_pair[t]) * a.nsplit + split) * D + d0;
            reinterpret_cast<f32x4*>(dst)[0] = f32x4{acc[tt][0][j], acc[tt][1][j], acc[tt][2][j], acc[tt][3][j]};
            reinterpret_cast<f32x4*>(dst)[1] = f32x4{acc[tt][4][j], acc[tt][5][j], acc[tt][6][j], acc[tt][7][j]};
#pragma unroll
            for (int c = 0; c < 8; ++c) sum += acc[tt][c][j];
          }
        }
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[tt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
      st = 0;
      slab += W;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  advance();
  for (int it = 0; it < total; it += 2) {
    if (it + 1 < total) {
      grp_load_down(a, down, i0, nu, lslab, 32 * lst, lane, r1);
      advance();
    }
    mul(r0);
    if (it + 2 < total) {
      grp_load_down(a, down, i0, nu, lslab, 32 * lst, lane, r0);
      advance();
    }
    if (it + 1 < total) mul(r1);
  }
  if (__any(isnan(sum))) grp_nan_outputs<W, TT>(a, down, i0, nu, m, split, wave, lane, s_h, hrow, s_pair);
}

// The group of this workgroup: its blob, its token count m and, in LDS, its
// pairs.  Returns false if there is no such group.
template <int W>
__device__ __forceinline__ bool grp_find(const GroupArgs& a, int g, int tid, int* s_cnt, int* s_wave, int* s_pair,
                                         const uint8_t** blob, int* m_out) {
  const int lane = tid & 63, wave = tid >> 6;
  const int BK = a.B * a.K, n = a.n;
  const int cs = (a.B + kGroupTokens - 1) / kGroupTokens;  // chunks of a shared expert
  const int nsg = a.n_shared * cs;
  if (g < nsg) {
    const int j = g / cs, b0 = (g - j * cs) * kGroupTokens;
    const int m = min(kGroupTokens, a.B - b0);
    if (tid < m) s_pair[tid] = BK + (b0 + tid) * a.n_shared + j;
    *blob = a.shared + static_cast<uint64_t>(j) * a.stride;
    *m_out = m;
    __syncthreads();
    return true;
  }
  // pairs per expert
  for (int e = tid; e < n; e += (64 * W)) s_cnt[e] = 0;
  __syncthreads();
  for (int p = tid; p < BK; p += (64 * W)) {
    const int e = a.topk[p];
    if (static_cast<unsigned>(e) < static_cast<unsigned>(n)) atomicAdd(&s_cnt[e], 1);
  }
  __syncthreads();
  // the (expert, chunk) of group g - nsg, in expert order: every wave scans the
  // whole table, a contiguous run of experts per lane
  const int per = (n + 63) / 64;
  int mine = 0;
  for (int q = 0; q < per; ++q) {
    const int e = lane * per + q;
    if (e < n && a.slot_tab[e] >= 0) mine += (s_cnt[e] + kGroupTokens - 1) / kGroupTokens;
  }
  int incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  const int want = g - nsg;
  const uint64_t hit = __ballot(want < incl);
  if (!hit) return false;
  const int src = __builtin_ctzll(hit);
  int e_found = 0, chunk = 0, slot = 0;
  if (lane == src) {
    int rest = want - (incl - mine);
    for (int q = 0; q < per; ++q) {
      const int e = lane * per + q;
      if (e >= n || a.slot_tab[e] < 0) continue;
      const int c = (s_cnt[e] + kGroupTokens - 1) / kGroupTokens;
      if (rest < c) {
        e_found = e;
        chunk = rest;
        slot = a.slot_tab[e];
        break;
      }
      rest -= c;
    }
  }
  const int e = __builtin_amdgcn_readlane(e_found, src);
  const int r0 = __builtin_amdgcn_readlane(chunk, src) * kGroupTokens;
  slot = __builtin_amdgcn_readlane(slot, src);
  const int cnt = s_cnt[e];
  // its pairs r0 .. r0 + 31 in pair order: wave w looks through a quarter of the routing
  const int seg = (BK + (64 * W) - 1) / (64 * W) * 64;
  int before = 0;
  for (int p0 = wave * seg; p0 < min(BK, (wave + 1) * seg); p0 += 64)
    before += __builtin_popcountll(__ballot(p0 + lane < BK && a.topk[min(p0 + lane, BK - 1)] == e));
  if (lane == 0) s_wave[wave] = before;
  __syncthreads();
  int rank0 = -r0;
  for (int w = 0; w < wave; ++w) rank0 += s_wave[w];
  for (int p0 = wave * seg; p0 < min(BK, (wave + 1) * seg); p0 += 64) {
    const bool is = p0 + lane < BK && a.topk[min(p0 + lane, BK - 1)] == e;
    const uint64_t mask = __ballot(is);
    const int rank = rank0 + __builtin_popcountll(mask & ((uint64_t{1} << lane) - 1));
    if (is && rank >= 0 && rank < kGroupTokens) s_pair[rank] = p0 + lane;
    rank0 += __builtin_popcountll(mask);
  }
  __syncthreads();
  *blob = a.slots + static_cast<uint64_t>(static_cast<uint32_t>(slot)) * a.stride;
  *m_out = min(kGroupTokens, cnt - r0);
  return true;
}

template <int W, int NT>
__global__ __launch_bounds__(64 * W, 2) void ffn_grouped_kernel(GroupArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t s_h[];
  __shared__ int s_cnt[kMaxExpertsTopK];
  __shared__ int s_wave[W];
  __shared__ int s_pair[kGroupTokens];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = blockIdx.x / a.nsplit, split = blockIdx.x - g * a.nsplit;
  const uint8_t* blob8 = nullptr;
  int m = 0;
  if (!grp_find<W>(a, g, tid, s_cnt, s_wave, s_pair, &blob8, &m)) return;
  m = __builtin_amdgcn_readfirstlane(m);
  const uint16_t* blob = reinterpret_cast<const uint16_t*>(blob8);
  const int i0 = split * a.upw;
  const int nu = min(a.upw, a.I - i0);  // a multiple of 16
  const int ntiles = nu >> 4;
  const int hrow = grp_h_row(a.upw);

  uint32_t xo[2];
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    const int pair = s_pair[min(16 * tt + (lane & 15), m - 1)];
    const int tok = pair < a.B * a.K ? pair / a.K : (pair - a.B * a.K) / a.n_shared;
    xo[tt] = static_cast<uint32_t>(tok) * a.D + 8 * (lane >> 4);
  }
  if (nu & 16) {  // the second half of the last step of 32 units
    for (int k = tid; k < 3 * kGroupTokens * 16; k += (64 * W))
      s_h[(k >> 4) * hrow + grp_h_pos(nu + (k & 15))] = 0;
  }
  const int tile0 = (i0 >> 4) + wave;
  const int nt = (ntiles - wave + W - 1) / W;  // this wave's tiles (0: none)
  auto phase_a = [&](auto tt_c) {
    constexpr int TT = decltype(tt_c)::value;
    if (nt >= NT) {
      grp_phase_a<W, NT, TT>(a, blob, tile0, wave, lane, xo, s_h, hrow);
    } else if (NT > 1 && nt == NT - 1) {
      grp_phase_a<W, (NT > 1 ? NT - 1 : 1), TT>(a, blob, tile0, wave, lane, xo, s_h, hrow);
    } else {
      for (int q = 0; q < nt; ++q)
        grp_phase_a<W, 1, TT>(a, blob, tile0 + W * q, wave + W * q, lane, xo, s_h, hrow);
    }
  };
  const uint16_t* down = blob + static_cast<size_t>(2) * a.I * a.D;
  u32x4 r0[8];  // phase B's first loads cross the barrier in flight
  const int slab0 = min(wave, a.D / 128 - 1);
  if (m <= 16) {
    phase_a(std::integral_constant<int, 1>{});
    grp_load_down(a, down, i0, nu, slab0, 0, lane, r0);
    __syncthreads();
    grp_phase_b<W, 1>(a, down, i0, nu, m, split, wave, lane, s_h, hrow, s_pair, r0);
  } else {
    phase_a(std::integral_constant<int, 2>{});
    grp_load_down(a, down, i0, nu, slab0, 0, lane, r0);
    __syncthreads();
    grp_phase_b<W, 2>(a, down, i0, nu, m, split, wave, lane, s_h, hrow, s_pair, r0);
  }
}

// ---------------------------------------------------------------------------
// Batched decode over experts in the unit layout (fp32, and bf16 shapes that
// the tiled layout does not take).  One workgroup takes one group (grp_find)
// and R x 4 units of its expert; every weight of the range is loaded into
// registers once and serves every token of the group.  As in
// ffn_slices_kernel a wave holds the gate and up rows of its own R units and
// its D-slice of all the down columns:
//   1. per token, h of the wave's units into LDS (the next token's x loads
//      beside it, see batch_x_ahead); one barrier;
//   2. per token, the wave's slice of sum_u h_u down_u to the partial row.
// A launch per token reads every expert once per token and pays two launches
// each: 6 fp32 tokens over 32 experts (D 1024, I 704) took 6 x (8.0 + 4.1) us.
// A few tokens that share hardly an expert take it all the same, see
// token_launches.
// ---------------------------------------------------------------------------
// Whether a second row of x fits beside the weights.  Rows of 7 or 8 chunks (8
// in fp32) then need more than 256 registers, one workgroup per compute unit
// instead of two: 6 tokens over 32 experts of 705 units of 3,104 columns, 4 per
// token, 121.6 us the layer with it, 92.8 without; 64 tokens 636 and 482; 16
// tokens over 704 units of 2,048 fp32 columns 150.9 and 129.1.
template <typename T>
constexpr bool batch_x_ahead(int nch) {
  return nch <= (sizeof(T) == 2 ? 6 : 7);
}

template <typename T, int NCH, bool FULL, int R, int DS>
__global__ __launch_bounds__(64 * kSlWaves) void ffn_units_batch_kernel(GroupArgs a) {
  constexpr int V = Vec<T>::N;
  constexpr int W = kSlWaves;
  __shared__ int s_cnt[kMaxExpertsTopK];
  __shared__ int s_wave[W];
  __shared__ int s_pair[kGroupTokens];
  __shared__ float s_h[kGroupTokens][R * W];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, nch = D / V, I = a.I;
  const int g = blockIdx.x / a.nsplit, split = blockIdx.x - g * a.nsplit;
  const uint8_t* blob = nullptr;
  int m = 0;
  if (!grp_find<W>(a, g, tid, s_cnt, s_wave, s_pair, &blob, &m)) return;
  m = __builtin_amdgcn_readfirstlane(m);
  const int i0 = split * R * W;
  const int cpw = (nch + W - 1) / W, c0 = wave * cpw;
  auto xrow = [&](int t) {
    const int pair = __builtin_amdgcn_readfirstlane(s_pair[t]);
    const int tok = pair < a.B * a.K ? pair / a.K : (pair - a.B * a.K) / a.n_shared;
    return a.x + static_cast<size_t>(tok) * D;
  };
  float xv[NCH][V];
  load_row_f32<T, NCH, FULL>(xrow(0), lane, nch, xv);
  __builtin_amdgcn_sched_barrier(0);
  // a unit past the end re-reads the last one, a lane past its slice chunk 0; neither is used
  uint4 rg[R][NCH], ru[R][NCH], rd[R][W][DS];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const T* base = reinterpret_cast<const T*>(blob) + static_cast<size_t>(min(i0 + r * W + wave, I - 1)) * 3 * D;
    load_chunks<NCH, FULL, true>(base, lane, nch, rg[r]);
    load_chunks<NCH, FULL, true>(base + D, lane, nch, ru[r]);
#pragma unroll
    for (int w2 = 0; w2 < W; ++w2) {
      const T* dbase = reinterpret_cast<const T*>(blob) + (static_cast<size_t>(min(i0 + r * W + w2, I - 1)) * 3 + 2) * D;
#pragma unroll
      for (int s = 0; s < DS; ++s) {
        const int c = c0 + lane + 64 * s;
        rd[r][w2][s] = ld_chunk<true>(dbase, lane + 64 * s < cpw && c < nch ? c : 0);
      }
    }
  }
  constexpr bool kAhead = batch_x_ahead<T>(NCH);
  for (int t = 0; t < m; ++t) {
    float xn[NCH][V];
    if constexpr (kAhead)
      load_row_f32<T, NCH, FULL>(xrow(min(t + 1, m - 1)), lane, nch, xn);
    else if (t > 0)
      load_row_f32<T, NCH, FULL>(xrow(t), lane, nch, xv);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float gs = 0.f, us = 0.f;
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        float fg[V], fu[V];
        unpack<T>(rg[r][j], fg);
        unpack<T>(ru[r][j], fu);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          gs += fg[v] * xv[j][v];
          us += fu[v] * xv[j][v];
        }
      }
      const float gv = wave_sum(gs);
      const float uv = wave_sum(us);
      if (lane == 0) s_h[t][r * W + wave] = gv / (1.f + expf(-gv)) * uv;
    }
    if constexpr (kAhead)
#pragma unroll
      for (int j = 0; j < NCH; ++j)
#pragma unroll
        for (int v = 0; v < V; ++v) xv[j][v] = xn[j][v];
  }
  __syncthreads();
  for (int t = 0; t < m; ++t) {
    float acc[DS][V];
#pragma unroll
    for (int s = 0; s < DS; ++s)
#pragma unroll
      for (int v = 0; v < V; ++v) acc[s][v] = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int w2 = 0; w2 < W; ++w2) {
        if (i0 + r * W + w2 >= I) continue;  // workgroup-uniform
        const float h = s_h[t][r * W + w2];
#pragma unroll
        for (int s = 0; s < DS; ++s) {
          float fd[V];
          unpack<T>(rd[r][w2][s], fd);
#pragma unroll
          for (int v = 0; v < V; ++v) acc[s][v] += h * fd[v];
        }
      }
    float* out = a.ypart + (static_cast<size_t>(s_pair[t]) * a.nsplit + split) * D;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
      const int c = c0 + lane + 64 * s;
      if (lane + 64 * s < cpw && c < nch) {
#pragma unroll
        for (int v = 0; v < V; v += 4)
          *reinterpret_cast<float4*>(out + c * V + v) = make_float4(acc[s][v], acc[s][v + 1], acc[s][v + 2], acc[s][v + 3]);
      }
    }
  }
}

// Batched combine: h_out[b] = round(residual[b] + sum_k g_bk sum_r ypart[(b,k), r]
//                                   + sum_j sum_r ypart[(b, shared j), r]), fixed order.
// Batched combine: y_b = sum_k g_bk * (sum over unit ranges of pair (b,k)'s
// partial rows) + the same sums of the shared experts (weight 1), plus the
// residual.  One workgroup per (256 columns, token), 4 columns per lane.  The
// ranges of a pair are cut into `parts` runs; wave w sums runs w, w + waves,
// ..., kCombRanges loads in flight; wave 0 then folds runs and pairs in order
// from LDS.  parts is 1 up to kCombRanges ranges; beyond, as many as give
// every wave of a full workgroup a run (59 ranges of 4 pairs in one run each
// would wait for four rounds of loads).
constexpr int kCombWaves = 16;
constexpr int kCombRanges = 16;  // range loads of one pair in flight per pass, at most
// RG: loads per pass, the smallest of 1, 2, 4, 8 and kCombRanges that holds a
// run (loads past a run's end re-read its last range: 16 of them per pair
// where a pair has 2 ranges took 19.4 us at 256 tokens of 8 Qwen-shaped
// experts each, 2 of them 10.3 us, at 64 tokens 6.1 and 4.8).
template <typename T, int RG>
__global__ __launch_bounds__(64 * kCombWaves) void ffn_combine_batched_kernel(CombineBArgs a) {
  __shared__ float4 s_v[kMaxWork][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  const int b = blockIdx.y;
  const int npairs = a.K + a.n_shared;
  const int parts = a.parts, per = (a.nsplit + parts - 1) / parts;
  const int col = 4 * (blockIdx.x * 64 + lane);
  const int c = min(col, a.D - 4);  // lanes past D re-read the last columns, unused
  for (int q0 = wave; q0 < npairs * parts; q0 += nwaves) {
    const int p = q0 / parts, rb = (q0 - p * parts) * per, re = min(a.nsplit, rb + per);
    const int pair = p < a.K ? b * a.K + p : a.B * a.K + b * a.n_shared + (p - a.K);
    const float* base = a.ypart + static_cast<size_t>(pair) * a.nsplit * a.D + c;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r0 = rb; r0 < re; r0 += RG) {
      float4 w[RG];
#pragma unroll
      for (int q = 0; q < RG; ++q)
        w[q] = *SPP_GLOBAL(float4, base + static_cast<size_t>(min(r0 + q, re - 1)) * a.D);
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        if (r0 + q < re) {  // ranges in order
          v.x += w[q].x;
          v.y += w[q].y;
          v.z += w[q].z;
          v.w += w[q].w;
        }
      }
    }
    s_v[q0][lane] = v;
  }
  // the gates and the residual go out while the other waves finish
  float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
  if (wave == 0) {
    const size_t o = static_cast<size_t>(b) * a.D + c;
    if (a.res_u) {
      res = *SPP_GLOBAL(float4, a.res_u + o);
    } else {
      res.x = load_elem<T>(a.res_h, o);
      res.y = load_elem<T>(a.res_h, o + 1);
      res.z = load_elem<T>(a.res_h, o + 2);
      res.w = load_elem<T>(a.res_h, o + 3);
    }
  }
  __syncthreads();
  if (wave != 0 || col >= a.D) return;
  float y[4] = {0.f, 0.f, 0.f, 0.f};
  for (int p = 0; p < npairs; ++p) {
    float4 v = s_v[p * parts][lane];
    for (int q = 1; q < parts; ++q) {
      const float4 w = s_v[p * parts + q][lane];
      v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
    }
    const float g = p < a.K ? a.gates[b * a.K + p] : 1.f;
    y[0] = p < a.K ? fmaf(g, v.x, y[0]) : y[0] + v.x;
    y[1] = p < a.K ? fmaf(g, v.y, y[1]) : y[1] + v.y;
    y[2] = p < a.K ? fmaf(g, v.z, y[2]) : y[2] + v.z;
    y[3] = p < a.K ? fmaf(g, v.w, y[3]) : y[3] + v.w;
  }
  const size_t o = static_cast<size_t>(b) * a.D + col;
  store_elem<T>(a.out, o, res.x + y[0]);
  store_elem<T>(a.out, o + 1, res.y + y[1]);
  store_elem<T>(a.out, o + 2, res.z + y[2]);
  store_elem<T>(a.out, o + 3, res.w + y[3]);
}

// Stand-in projection prologue: u = h + P rms(h) (fp32 result).  One wave per row of P.
template <typename T, int NCH, bool FULL>
__global__ __launch_bounds__(kThreads) void proj_kernel(ProjArgs a) {
  constexpr int V = Vec<T>::N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int D = a.D, nch = D / V;
  const int row = blockIdx.x * kWaves + wave;
  if (row >= D) return;
  const T* prow = reinterpret_cast<const T*>(a.P) + static_cast<size_t>(row) * D;
  uint4 w[NCH];
  load_chunks<NCH, FULL>(prow, lane, nch, w);
  // the first token's row and residual go out with the weight row: the
  // unpacked weights are hoisted out of the token loop, which waits for them
  uint4 hr[NCH];
  load_chunks<NCH, FULL>(a.h, lane, nch, hr);
  float res = load_elem<T>(a.h, row);
  for (int b = 0; b < a.B; ++b) {
    const T* hb = reinterpret_cast<const T*>(a.h) + static_cast<size_t>(b) * D;
    if (b > 0) {
      load_chunks<NCH, FULL>(hb, lane, nch, hr);
      res = load_elem<T>(hb, row);
    }
    float xv[NCH][V];
#pragma unroll
    for (int j = 0; j < NCH; ++j) unpack<T>(hr[j], xv[j]);
    const float inv = rms_scale<T, NCH>(xv, D, a.eps);
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      float wf[V];
      unpack<T>(w[j], wf);
#pragma unroll
      for (int v = 0; v < V; ++v) acc += wf[v] * (xv[j][v] * inv);
    }
    acc = wave_sum(acc);
    if (lane == 0) a.u[static_cast<size_t>(b) * D + row] = res + acc;
  }
}

// Router and adapter-A rows for B > 1 tokens:
//   z[b][row] = inv_b * sum_k u[b][k] W[row][k],  inv_b = 1 / rms(u_b)
// (inv_b = 1 when u already is the router input x); the router rows, then the
// adapter rows, form the row axis, written to zbuf at their columns.  One
// workgroup per 16 tokens x 16 rows; its waves split D into runs of KSW steps
// of 32 columns, every load of a run in flight at once: a lane loads 8
// consecutive columns of its token row and of its weight row.  bf16 states and
// weights multiply on the bf16 MFMA; an fp32 operand on the fp32 MFMA, step q
// of 8 taking column 8 (lane/16) + q of every lane (bf16 weights widen
// exactly).  Products are exact either way where one operand is bf16.  The
// waves' partial tiles and sums of squares add in wave order through LDS.  x =
// inv_b u_b (and its bf16 pair) goes out from the registers that hold u, each
// row tile writing its share of the steps.
// Bound by latency (cold weights, one round of loads): 64 tokens of the Qwen
// shape 10.2 us with fp32 states in front (12.0 with 8-byte loads in two
// rounds and a second read of u for x), 4 tokens 6.4 us from 9.2.  Measured
// and not kept: selecting in the last workgroup of a token tile instead of a
// launch of one wave per token (4 tokens 10.1 us against 6.4 + 3.2, 64 tokens
// with an adapter 27 against 10.2 + 7.5: two tokens per wave in series), and
// 16 waves (9.6 us, but fp32 9.1 against 6.7).
constexpr int kRowWaves = 8;

// 8 consecutive elements of a row as raw bits
template <typename T>
struct Raw8;
template <>
struct Raw8<uint16_t> {
  u32x4 v;
  __device__ __forceinline__ void load(const uint16_t* p) { v = *SPP_GLOBAL(u32x4, p); }
  __device__ __forceinline__ void zero() { v = u32x4{0, 0, 0, 0}; }
  __device__ __forceinline__ void get(float* f) const { unpack<uint16_t>(make_uint4(v.x, v.y, v.z, v.w), f); }
};
template <>
struct Raw8<float> {
  u32x4 v[2];
  __device__ __forceinline__ void load(const float* p) {
    v[0] = *SPP_GLOBAL(u32x4, p);
    v[1] = *SPP_GLOBAL(u32x4, p + 4);
  }
  __device__ __forceinline__ void zero() { v[0] = v[1] = u32x4{0, 0, 0, 0}; }
  __device__ __forceinline__ void get(float* f) const {
#pragma unroll
    for (int q = 0; q < 2; ++q) unpack<float>(make_uint4(v[q].x, v[q].y, v[q].z, v[q].w), f + 4 * q);
  }
};

// TU: element type of u (float, or T when the layer input itself is read)
template <typename T, typename TU, int KSW>
__global__ __launch_bounds__(64 * kRowWaves) void router_rows_kernel(RouterArgs a) {
  // for the selection that follows, where no earlier launch vouches for them
  if (a.clear && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) a.counter[threadIdx.x] = 0u;
  __shared__ f32x4 s_acc[kRowWaves][64];
  __shared__ float s_ss[kRowWaves][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D, n = a.n, ldz = a.n + a.r;
  const int nr = a.router_on ? n : 0, na = a.A ? a.r : 0, rows = nr + na;
  const int b0 = blockIdx.y * 16, r0 = blockIdx.x * 16;
  const int i = lane & 15, g = lane >> 4;
  const int tok = min(b0 + i, a.B - 1);
  const int row = min(r0 + i, rows - 1);
  const T* wrow = row < nr ? reinterpret_cast<const T*>(a.Wr) + static_cast<size_t>(row) * D
                           : reinterpret_cast<const T*>(a.A) + static_cast<size_t>(row - nr) * D;
  const TU* urow = (a.u ? reinterpret_cast<const TU*>(a.u) : reinterpret_cast<const TU*>(a.h)) +
                   static_cast<size_t>(tok) * D;
  const int nks = (D + 31) / 32;  // D is a multiple of 16: a lane's 8 columns are all in or all out
  const int per = (nks + kRowWaves - 1) / kRowWaves;  // <= KSW
  const int c0 = wave * per, cnt = max(0, min(nks - c0, per));
  Raw8<TU> ur[KSW];
  Raw8<T> wr[KSW];
#pragma unroll
  for (int q = 0; q < KSW; ++q) {
    const int k = 32 * (c0 + q) + 8 * g;
    const bool ok = q < cnt && k < D;
    ur[q].load(urow + (ok ? k : 0));
    wr[q].load(wrow + (ok ? k : 0));
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  float ss = 0.f;
#pragma unroll
  for (int q = 0; q < KSW; ++q) {
    if (q < cnt) {  // wave-uniform
      if (32 * (c0 + q) + 8 * g >= D) {
        ur[q].zero();
        wr[q].zero();
      }
      float uf[8];
      ur[q].get(uf);
  #pragma unroll
      for (int e = 0; e < 8; ++e) ss += uf[e] * uf[e];
      if constexpr (sizeof(T) == 2 && sizeof(TU) == 2) {
        acc = mfma_bf16(ur[q].v, wr[q].v, acc);
      } else {
        float wf[8];
        wr[q].get(wf);
  #pragma unroll
        for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(uf[e], wf[e], acc, 0, 0, 0);
      }
    }
  }
  // lanes i, i+16, i+32, i+48 hold the column groups of token b0 + i
  ss += __shfl_xor(ss, 16);
  ss += __shfl_xor(ss, 32);
  s_acc[wave][lane] = acc;
  if (lane < 16) s_ss[wave][lane] = ss;
  __syncthreads();
  auto inv_of = [&](int t) {
    float sst = s_ss[0][t];
#pragma unroll
    for (int w = 1; w < kRowWaves; ++w) sst += s_ss[w][t];
    return a.x_given ? 1.f : 1.0f / sqrtf(sst / static_cast<float>(D) + a.eps);
  };
  if (wave == 0) {
    f32x4 z = s_acc[0][lane];
#pragma unroll
    for (int w = 1; w < kRowWaves; ++w) {
      const f32x4 v = s_acc[w][lane];
      z = f32x4{z[0] + v[0], z[1] + v[1], z[2] + v[2], z[3] + v[3]};
    }
    // this lane holds tokens b0 + 4*(lane/16) + j of row r0 + lane%16
    const int zr = r0 + i;
    if (zr < rows) {
      const int zcol = zr < nr ? zr : n + (zr - nr);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = 4 * g + j;
        if (b0 + t < a.B) a.zbuf[static_cast<size_t>(b0 + t) * ldz + zcol] = z[j] * inv_of(t);
      }
    }
  }
  if (a.x_out && b0 + i < a.B) {
    const float inv = inv_of(i);
    const size_t xb = static_cast<size_t>(b0 + i) * D;
#pragma unroll
    for (int q = 0; q < KSW; ++q) {
      const int k = 32 * (c0 + q) + 8 * g;
      if (q >= cnt || (c0 + q) % static_cast<int>(gridDim.x) != static_cast<int>(blockIdx.x) || k >= D) continue;
      float f[8];
      ur[q].get(f);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] *= inv;
      float4* xo = reinterpret_cast<float4*>(a.x_out + xb + k);
      xo[0] = make_float4(f[0], f[1], f[2], f[3]);
      xo[1] = make_float4(f[4], f[5], f[6], f[7]);
      if (a.xh) {
        uint4 hi, lo;
        split2(f[0], f[1], &hi.x, &lo.x);
        split2(f[2], f[3], &hi.y, &lo.y);
        split2(f[4], f[5], &hi.z, &lo.z);
        split2(f[6], f[7], &hi.w, &lo.w);
        *reinterpret_cast<uint4*>(a.xh + xb + k) = hi;
        *reinterpret_cast<uint4*>(a.xl + xb + k) = lo;
      }
    }
  }
}

// Stand-in projection for a batch (bf16, B > 1) on MFMA.  h and P are bf16, so
// their products are exact on the bf16 MFMA; the normalisation moves to the
// epilogue,
//   u[b][o] = h[b][o] + (sum_i P[o][i] h[b][i]) / sqrt(mean_i h[b][i]^2 + eps),
// with sum_i h[b][i]^2 accumulated from the same loads.  One workgroup per
// kProjRB x 16 output rows x 16 tokens; its 8 waves split D in 256-column
// chunks (wave w takes chunks w, w+8, ...), each loading the chunk's h pieces
// once for its kProjRB 16x16 accumulators, and its tokens' partial sums of
// squares; the partials are added in wave order through LDS.  The kernel is
// bound by the operand traffic from L2 (h is re-read by every row block, P by
// every token block): measured as loads alone at B = 64, D = 2048, 16 rows
// per workgroup of 4 waves (the earlier design) took 8.3 us by events and 2
// row blocks per workgroup of 8 waves 6.3 us; 4 token or row blocks per
// workgroup were slower again (fewer workgroups).  Token rows past B read the
// last token and are not stored.
constexpr int kProjWaves = 8;
constexpr int kProjRB = 2;  // 16-row blocks of P per workgroup (D a multiple of 256)
__global__ __launch_bounds__(64 * kProjWaves) void proj_mfma_kernel(ProjArgs a) {
  __shared__ f32x4 s_acc[kProjWaves][kProjRB][64];
  __shared__ float s_ss[kProjWaves][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int o0 = blockIdx.x * 16 * kProjRB, b0 = blockIdx.y * 16;
  const int D = a.D, nck = D / 256;
  const int krow = lane & 15, koff = 8 * (lane >> 4);
  const int tok = min(b0 + krow, a.B - 1);
  const uint16_t* hrow = reinterpret_cast<const uint16_t*>(a.h) + static_cast<size_t>(tok) * D + koff;
  const uint16_t* prow[kProjRB];
#pragma unroll
  for (int r = 0; r < kProjRB; ++r)
    prow[r] = reinterpret_cast<const uint16_t*>(a.P) + static_cast<size_t>(o0 + 16 * r + krow) * D + koff;
  f32x4 acc[kProjRB];
#pragma unroll
  for (int r = 0; r < kProjRB; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
  float ss = 0.f;
  for (int c = wave; c < nck; c += kProjWaves) {
    const int k0 = 256 * c;
    u32x4 ha[8], pb[kProjRB][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      ha[j] = *SPP_GLOBAL(u32x4, hrow + k0 + 32 * j);
#pragma unroll
      for (int r = 0; r < kProjRB; ++r) pb[r][j] = __builtin_nontemporal_load(SPP_GLOBAL(u32x4, prow[r] + k0 + 32 * j));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const bf16x8 hv = __builtin_bit_cast(bf16x8, ha[j]);
#pragma unroll
      for (int r = 0; r < kProjRB; ++r)
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hv, __builtin_bit_cast(bf16x8, pb[r][j]), acc[r], 0, 0, 0);
      const uint32_t w[4] = {ha[j].x, ha[j].y, ha[j].z, ha[j].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float lo = __uint_as_float(w[q] << 16), hi = __uint_as_float(w[q] & 0xffff0000u);
        ss += lo * lo + hi * hi;
      }
    }
  }
  // lanes l, l+16, l+32, l+48 hold the k-slices of token b0 + l%16
  ss += __shfl_xor(ss, 16);
  ss += __shfl_xor(ss, 32);
#pragma unroll
  for (int r = 0; r < kProjRB; ++r) s_acc[wave][r][lane] = acc[r];
  if (lane < 16) s_ss[wave][lane] = ss;
  __syncthreads();
  if (wave >= kProjRB) return;
  // wave r finishes row block r
  f32x4 y = s_acc[0][wave][lane];
#pragma unroll
  for (int w = 1; w < kProjWaves; ++w) {
    const f32x4 v = s_acc[w][wave][lane];
    y = f32x4{y[0] + v[0], y[1] + v[1], y[2] + v[2], y[3] + v[3]};
  }
  // this lane holds tokens 4*(lane/16)+j of output row o0 + 16*wave + lane%16
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int t = 4 * (lane >> 4) + j;
    float sst = s_ss[0][t];
#pragma unroll
    for (int w = 1; w < kProjWaves; ++w) sst += s_ss[w][t];
    const int b = b0 + t;
    if (b < a.B) {
      const int o = o0 + 16 * wave + krow;
      const float inv = 1.0f / sqrtf(sst / static_cast<float>(D) + a.eps);
      const size_t idx = static_cast<size_t>(b) * D + o;
      a.u[idx] = __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(a.h)[idx]) << 16) +
                 inv * y[j];
    }
  }
}

// Bounded busy wait used only by the copy-delay test hook: returns after
// `ticks` of the constant-rate wall clock or after `max_iter` sleeps, whichever
// comes first.
// Host-to-device copies by shader loads: each source is the device-visible
// address of pinned host memory, each destination device memory, n16 the
// count of 16-byte chunks of every copy.  Each lane keeps one 16-byte read
// across the host link in flight per step of a grid-stride loop (a grid of a
// few dozen workgroups saturates the link), and the copies of the list follow
// one another without a gap between launches.  Loads and stores are
// non-temporal: the data is read once here and next by a later kernel, from HBM.
__global__ __launch_bounds__(256) void h2d_copy_kernel(CopyList a) {
  const size_t stride = static_cast<size_t>(gridDim.x) * blockDim.x;
  const size_t i0 = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  for (int t = 0; t < a.n; ++t) {
    const u32x4* src = static_cast<const u32x4*>(a.src[t]);
    u32x4* dst = static_cast<u32x4*>(a.dst[t]);
    for (size_t i = i0; i < a.n16; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
  }
}

constexpr int kTableChunk = 512;
struct TableArg {
  int32_t v[kTableChunk];
};
__global__ __launch_bounds__(256) void set_table_kernel(TableArg t, int32_t* dst, int n) {
  for (int i = threadIdx.x; i < n; i += 256) dst[i] = t.v[i];
}

__global__ void spin_kernel(uint64_t ticks, uint32_t max_iter) {
  const uint64_t t0 = wall_clock64();
  for (uint32_t it = 0; it < max_iter; ++it) {
    if (wall_clock64() - t0 >= ticks) break;
    __builtin_amdgcn_s_sleep(8);
  }
}

template <typename T>
int nch_for(int D) {
  const int nch = D / Vec<T>::N;
  return (nch + 63) / 64;
}

#define SPP_DISPATCH_NCH(NCHV, ...)                          \
  switch (NCHV) {                                            \
    case 1: { constexpr int NCH = 1; __VA_ARGS__; } break;   \
    case 2: { constexpr int NCH = 2; __VA_ARGS__; } break;   \
    case 3: { constexpr int NCH = 3; __VA_ARGS__; } break;   \
    case 4: { constexpr int NCH = 4; __VA_ARGS__; } break;   \
    case 5: { constexpr int NCH = 5; __VA_ARGS__; } break;   \
    case 6: { constexpr int NCH = 6; __VA_ARGS__; } break;   \
    case 7: { constexpr int NCH = 7; __VA_ARGS__; } break;   \
    case 8: { constexpr int NCH = 8; __VA_ARGS__; } break;   \
    default: return hipErrorInvalidValue;                    \
  }

// FULL: D fills every lane's chunks (D / elements-per-chunk a multiple of 64)
template <typename T>
bool full_rows(int D) {
  return (D / Vec<T>::N) % 64 == 0;
}

template <typename T, typename TU>
void router_rows_t(const RouterArgs& a, int rows, hipStream_t st) {
  const dim3 grid((rows + 15) / 16, (a.B + 15) / 16), block(64 * kRowWaves);
  const int per = ((a.D + 31) / 32 + kRowWaves - 1) / kRowWaves;  // steps of a wave: up to 16 at D 4096
  if (per <= 4)
    hipLaunchKernelGGL((router_rows_kernel<T, TU, 4>), grid, block, 0, st, a);
  else if (per <= 8)
    hipLaunchKernelGGL((router_rows_kernel<T, TU, 8>), grid, block, 0, st, a);
  else if constexpr (sizeof(T) == 2)  // fp32 rows have at most 2048 columns
    hipLaunchKernelGGL((router_rows_kernel<T, TU, 16>), grid, block, 0, st, a);
}

// Batch 1: router rows and adapter rows in workgroups of their own.
int router_wgs(const RouterArgs& a) {
  return ((a.router_on ? a.n : 0) + kWaves - 1) / kWaves + ((a.A ? a.r : 0) + kWaves - 1) / kWaves;
}

// Single-wave tails: n <= 128, K <= 32 (checked at launch), an
// adapter in bf16 with r <= 64 and a multiple of 8.
bool one_wave_tails(const RouterArgs& a, bool bf16) {
  return a.n <= 128 && (!a.A || (bf16 && a.r <= 64 && a.r % 8 == 0));
}

template <typename T, bool FULL>
hipError_t router_tf(const RouterArgs& a, hipStream_t st) {
  const int rows = (a.router_on ? a.n : 0) + (a.A ? a.r : 0);
  if (rows <= 0) return hipErrorInvalidValue;
  // the staged adapter path reads B in 16-byte chunks
  if (a.A && (static_cast<size_t>(a.n) * a.r * sizeof(T)) % 16 != 0) return hipErrorInvalidValue;
  if (a.B == 1) {
    const int g1 = router_wgs(a);
    const bool fast = one_wave_tails(a, sizeof(T) == 2);
    if (fast && ((a.router_on && !a.ztag) || (a.A && !a.atag))) return hipErrorInvalidValue;
    if (fast && a.router_on && a.tickets) return hipErrorInvalidValue;  // drawn by adapter_kernel only
    if (fast && !a.router_on && a.n <= 64) {
      SPP_DISPATCH_NCH(nch_for<T>(a.D),
                       hipLaunchKernelGGL((adapter_kernel<NCH, FULL, 1>), dim3(g1), dim3(kThreads), 0, st, a));
    } else if (fast && !a.router_on) {
      SPP_DISPATCH_NCH(nch_for<T>(a.D),
                       hipLaunchKernelGGL((adapter_kernel<NCH, FULL, 2>), dim3(g1), dim3(kThreads), 0, st, a));
    } else if (fast && a.n <= 64) {
      SPP_DISPATCH_NCH(nch_for<T>(a.D), hipLaunchKernelGGL((router_adapter_kernel<T, NCH, FULL, 1>), dim3(g1),
                                                           dim3(kThreads), 0, st, a));
    } else if (fast) {
      SPP_DISPATCH_NCH(nch_for<T>(a.D), hipLaunchKernelGGL((router_adapter_kernel<T, NCH, FULL, 2>), dim3(g1),
                                                           dim3(kThreads), 0, st, a));
    } else {
      SPP_DISPATCH_NCH(nch_for<T>(a.D), hipLaunchKernelGGL((router_adapter_kernel<T, NCH, FULL, 0>), dim3(g1),
                                                           dim3(kThreads), 0, st, a));
    }
    return hipGetLastError();
  }
  if (a.D % 16 != 0) return hipErrorInvalidValue;
  if (a.u || sizeof(T) == 4)
    router_rows_t<T, float>(a, rows, st);
  else
    router_rows_t<T, T>(a, rows, st);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  // one wave per token under the conditions of the batch-1 one-wave tails; 3.3 us
  // against 3.9 for a workgroup per token (6 fp32 tokens over 32 experts)
  const bool wave1 = one_wave_tails(a, sizeof(T) == 2);
  if (wave1 && a.n <= 64)
    hipLaunchKernelGGL((router_select_wave_kernel<1>), dim3(a.B), dim3(64), 0, st, a);
  else if (wave1)
    hipLaunchKernelGGL((router_select_wave_kernel<2>), dim3(a.B), dim3(64), 0, st, a);
  else
    hipLaunchKernelGGL((router_select_kernel<T>), dim3(a.B), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

template <typename T>
hipError_t router_t(const RouterArgs& a, hipStream_t st) {
  return full_rows<T>(a.D) ? router_tf<T, true>(a, st) : router_tf<T, false>(a, st);
}

template <typename T, bool FULL>
hipError_t ffn_tf(const FfnArgs& a, int grid, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  const uint32_t lds = sizeof(float) * (kFfnWaves / 2) * a.D;
  if (start || stop) {
    SPP_DISPATCH_NCH(nch_for<T>(a.D), hipExtLaunchKernelGGL((ffn_units_kernel<T, NCH, FULL>), dim3(grid),
                                                            dim3(kFfnThreads), lds, st, start, stop, 0u, a));
  } else {
    SPP_DISPATCH_NCH(nch_for<T>(a.D), hipLaunchKernelGGL((ffn_units_kernel<T, NCH, FULL>), dim3(grid),
                                                         dim3(kFfnThreads), lds, st, a));
  }
  return hipGetLastError();
}

// DS: chunks of a wave's D-slice per lane in the sweep-round kernel.
template <int NCH>
constexpr int slices_ds() {
  return NCH <= 4 ? 1 : 2;
}

// Most sweep rounds: what stays in 256 registers beside x (2 NCH + 4 DS chunks
// of 4 registers each per round), so that two workgroups share a compute unit
// (231 registers at 6 ragged chunks, 241 at 8 of fp32, alone; 221 and 233 in
// the launch with the router).  Up to 4 chunks per lane no more than 3: which
// units share a partial row is part of a stack's rounding, and 4 rounds on 448
// workgroups, although faster over 7,168 units (17.3 against 18.4 us), turn
// near-ties of later layers' routers.
constexpr int kSlMaxRounds = 3;
template <typename T>
constexpr int slices_rounds(int nch) {
  return nch <= 4 ? 3 : nch <= 6 ? 2 : (sizeof(T) == 4 ? 2 : 1);
}

// Units per wave of ffn_units_batch_kernel: as many as stay in 256 registers
// beside two rows of x (one where batch_x_ahead says so).
template <typename T>
constexpr int batch_rounds(int nch) {
  return sizeof(T) == 2 ? (nch <= 3 ? 3 : nch == 4 ? 2 : 1) : (nch <= 4 ? 3 : 2);
}

template <typename T, bool FULL, int R>
hipError_t ffn_slices_tr(const FfnArgs& a, int grid, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  const int nchl = nch_for<T>(a.D);
  if (R > slices_rounds<T>(nchl)) return hipErrorInvalidValue;
#define SPP_SLICES(NCHX) ffn_slices_kernel<T, NCHX, FULL, (R <= slices_rounds<T>(NCHX) ? R : 1), slices_ds<NCHX>()>
  if (start || stop) {
    SPP_DISPATCH_NCH(nchl, hipExtLaunchKernelGGL((SPP_SLICES(NCH)), dim3(grid), dim3(64 * kSlWaves), 0, st, start,
                                                  stop, 0u, a));
  } else {
    SPP_DISPATCH_NCH(nchl, hipLaunchKernelGGL((SPP_SLICES(NCH)), dim3(grid), dim3(64 * kSlWaves), 0, st, a));
  }
#undef SPP_SLICES
  return hipGetLastError();
}

template <typename T, bool FULL>
hipError_t ffn_slices_tf(const FfnArgs& a, int grid, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  switch (a.rounds) {
    case 1: return ffn_slices_tr<T, FULL, 1>(a, grid, st, start, stop);
    case 2: return ffn_slices_tr<T, FULL, 2>(a, grid, st, start, stop);
    case 3: return ffn_slices_tr<T, FULL, 3>(a, grid, st, start, stop);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t ffn_t(const FfnArgs& a, int grid, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  if (a.rounds > 0) {
    // the grid must cover every unit in a.rounds bands
    if (static_cast<long>(grid) * kSlWaves * a.rounds < static_cast<long>(a.nW) * a.I) return hipErrorInvalidValue;
    return full_rows<T>(a.D) ? ffn_slices_tf<T, true>(a, grid, st, start, stop)
                             : ffn_slices_tf<T, false>(a, grid, st, start, stop);
  }
  return full_rows<T>(a.D) ? ffn_tf<T, true>(a, grid, st, start, stop) : ffn_tf<T, false>(a, grid, st, start, stop);
}

template <typename T, bool FULL>
hipError_t proj_tf(const ProjArgs& a, hipStream_t st) {
  const int grid = (a.D + kWaves - 1) / kWaves;
  SPP_DISPATCH_NCH(nch_for<T>(a.D),
                   hipLaunchKernelGGL((proj_kernel<T, NCH, FULL>), dim3(grid), dim3(kThreads), 0, st, a));
  return hipGetLastError();
}

template <typename T>
hipError_t proj_t(const ProjArgs& a, hipStream_t st) {
  return full_rows<T>(a.D) ? proj_tf<T, true>(a, st) : proj_tf<T, false>(a, st);
}

}  // namespace

bool adapter_by_tickets(int n, int r, int B, int dtype) {
  RouterArgs a{};
  a.A = &a;  // an adapter is there
  a.n = n;
  a.r = r;
  return B == 1 && one_wave_tails(a, dtype == 1);
}

hipError_t launch_router(const RouterArgs& a, int dtype, hipStream_t st) {
  if (a.n > kMaxExpertsTopK || a.r > 256 || a.K > 32 || a.K > a.n) return hipErrorInvalidValue;
  return dtype == 1 ? router_t<uint16_t>(a, st) : router_t<float>(a, st);
}

namespace {

template <typename T, bool FULL, int R>
hipError_t layer_slices_tr(const RouterArgs& ra, const FfnArgs& fa, int rb, int grid, hipStream_t st) {
  const int nchl = nch_for<T>(fa.D);
  if (R > slices_rounds<T>(nchl)) return hipErrorInvalidValue;
  SPP_DISPATCH_NCH(nchl, hipLaunchKernelGGL(
                             (layer_slices_kernel<T, NCH, FULL, (R <= slices_rounds<T>(NCH) ? R : 1), slices_ds<NCH>()>),
                             dim3(rb + grid), dim3(64 * kSlWaves), 0, st, ra, fa, rb));
  return hipGetLastError();
}

template <typename T, bool FULL>
hipError_t layer_slices_tf(const RouterArgs& ra, const FfnArgs& fa, int rb, int grid, hipStream_t st) {
  switch (fa.rounds) {
    case 1: return layer_slices_tr<T, FULL, 1>(ra, fa, rb, grid, st);
    case 2: return layer_slices_tr<T, FULL, 2>(ra, fa, rb, grid, st);
    case 3: return layer_slices_tr<T, FULL, 3>(ra, fa, rb, grid, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t layer_slices_t(const RouterArgs& ra, const FfnArgs& fa, int rb, int grid, hipStream_t st) {
  if (static_cast<long>(grid) * kSlWaves * fa.rounds < static_cast<long>(fa.nW) * fa.I) return hipErrorInvalidValue;
  return full_rows<T>(fa.D) ? layer_slices_tf<T, true>(ra, fa, rb, grid, st)
                            : layer_slices_tf<T, false>(ra, fa, rb, grid, st);
}

template <int NCH, bool FULL, int NQ, bool FULLQ>
hipError_t layer_q4_t(const RouterArgs& ra, const FfnArgs& fa, int rb, int grid, hipStream_t st) {
  const uint32_t lds = sizeof(float) * kFfnWaves * fa.D;
  if (fa.rounds == 1)
    hipLaunchKernelGGL((layer_q4_kernel<NCH, FULL, NQ, FULLQ, 1>), dim3(rb + grid), dim3(kFfnThreads), lds, st, ra, fa,
                       rb);
  else
    hipLaunchKernelGGL((layer_q4_kernel<NCH, FULL, NQ, FULLQ, 2>), dim3(rb + grid), dim3(kFfnThreads), lds, st, ra, fa,
                       rb);
  return hipGetLastError();
}

}  // namespace

bool layer_launch_ok(const RouterArgs& ra, const FfnArgs& fa, int dtype) {
  return ra.B == 1 && ra.router_on && !ra.x_given && ra.slot_tab && ra.ztag && ra.route_tag &&
         one_wave_tails(ra, dtype == 1) && fa.rounds > 0 && fa.nsel == ra.K;
}

hipError_t launch_layer(const RouterArgs& ra, const FfnArgs& fa, int grid, int dtype, hipStream_t st) {
  if (!layer_launch_ok(ra, fa, dtype) || ra.K > 32 || ra.K > ra.n || ra.D != fa.D || fa.D > 4096 || fa.nW <= 0 ||
      fa.nW > kMaxWork || grid <= 0 || fa.skip_mask != 0 || fa.rounds > (fa.codec ? 2 : kSlMaxRounds))
    return hipErrorInvalidValue;
  const int rb = router_wgs(ra);
  if (fa.codec == 1) {
    if (dtype != 1 || fa.D % 256 != 0 || fa.upp != 3 ||
        static_cast<long>(grid) * kFfnWaves * 3 * fa.rounds < static_cast<long>(fa.nW) * fa.I)
      return hipErrorInvalidValue;
    const int nblk = fa.D / 32;
    if (nblk == 64) return layer_q4_t<4, true, 1, true>(ra, fa, rb, grid, st);
    if (nblk < 64) return layer_q4_t<4, false, 1, false>(ra, fa, rb, grid, st);
    if (nblk == 128) return layer_q4_t<8, true, 2, true>(ra, fa, rb, grid, st);
    return layer_q4_t<8, false, 2, false>(ra, fa, rb, grid, st);
  }
  return dtype == 1 ? layer_slices_t<uint16_t>(ra, fa, rb, grid, st) : layer_slices_t<float>(ra, fa, rb, grid, st);
}

template <int NQ, bool FULLQ, int UPP, int PASSES>
hipError_t ffn_q4_tu(const FfnArgs& a, int grid, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  const uint32_t lds = sizeof(float) * kFfnWaves * a.D;  // 64 KiB at D 4096
  if (start || stop)
    hipExtLaunchKernelGGL((ffn_q4_kernel<NQ, FULLQ, UPP, PASSES>), dim3(grid), dim3(kFfnThreads), lds, st, start,
                          stop, 0u, a);
  else
    hipLaunchKernelGGL((ffn_q4_kernel<NQ, FULLQ, UPP, PASSES>), dim3(grid), dim3(kFfnThreads), lds, st, a);
  return hipGetLastError();
}

template <int NQ, bool FULLQ>
hipError_t ffn_q4_t(const FfnArgs& a, int grid, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  if (a.rounds > 0) {
    // sweep order: 3 units per wave and pass, the grid's waves cover every unit
    if (a.upp != 3 || a.rounds > 2 ||
        static_cast<long>(grid) * kFfnWaves * 3 * a.rounds < static_cast<long>(a.nW) * a.I)
      return hipErrorInvalidValue;
    return a.rounds == 1 ? ffn_q4_tu<NQ, FULLQ, 3, 1>(a, grid, st, start, stop)
                         : ffn_q4_tu<NQ, FULLQ, 3, 2>(a, grid, st, start, stop);
  }
  if (a.upp == 4) return ffn_q4_tu<NQ, FULLQ, 4, 0>(a, grid, st, start, stop);
  if (a.upp == 3) return ffn_q4_tu<NQ, FULLQ, 3, 0>(a, grid, st, start, stop);
  return hipErrorInvalidValue;
}

hipError_t launch_ffn(const FfnArgs& a, int grid, int dtype, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  if (a.nW <= 0 || a.nW > kMaxWork || grid <= 0 || a.D > 4096) return hipErrorInvalidValue;
  if (a.rounds > 0 && (a.skip_mask != 0 || a.rounds > (a.codec ? 2 : kSlMaxRounds))) return hipErrorInvalidValue;
  if (a.rounds == 0 && a.upw <= 0) return hipErrorInvalidValue;
  if (a.skip_mask != 0 && a.I % a.upw != 0) return hipErrorInvalidValue;  // a workgroup would span two items
  if (a.codec == 1) {
    // 4-bit experts: 32 elements per lane and block, 64 blocks per 2048-element chunk
    if (dtype != 1 || a.D % 256 != 0) return hipErrorInvalidValue;
    const int nblk = a.D / 32;
    if (nblk == 64) return ffn_q4_t<1, true>(a, grid, st, start, stop);
    if (nblk < 64) return ffn_q4_t<1, false>(a, grid, st, start, stop);
    if (nblk == 128) return ffn_q4_t<2, true>(a, grid, st, start, stop);
    return ffn_q4_t<2, false>(a, grid, st, start, stop);
  }
  return dtype == 1 ? ffn_t<uint16_t>(a, grid, st, start, stop) : ffn_t<float>(a, grid, st, start, stop);
}

hipError_t launch_combine(const CombineArgs& a, int dtype, hipStream_t st) {
  const int grid = (a.D + kCombCols - 1) / kCombCols;
  if (dtype == 1)
    hipLaunchKernelGGL((ffn_combine_kernel<uint16_t>), dim3(grid), dim3(kCombThreads), 0, st, a);
  else
    hipLaunchKernelGGL((ffn_combine_kernel<float>), dim3(grid), dim3(kCombThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_proj(const ProjArgs& a, int dtype, hipStream_t st) {
  if (dtype == 1 && a.B > 1 && a.D % 256 == 0) {
    hipLaunchKernelGGL(proj_mfma_kernel, dim3(a.D / (16 * kProjRB), (a.B + 15) / 16), dim3(64 * kProjWaves), 0, st, a);
    return hipGetLastError();
  }
  return dtype == 1 ? proj_t<uint16_t>(a, st) : proj_t<float>(a, st);
}

hipError_t launch_ffn_grouped(const GroupArgs& a, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  if (a.ngroups <= 0 || a.nsplit <= 0 || a.upw < 16 || a.upw % 16 != 0 || (a.waves != 4 && a.waves != 8) ||
      a.D % kGrpBlk != 0 || a.I % 16 != 0 || a.nsplit * a.upw < a.I || (a.nsplit - 1) * a.upw >= a.I || !a.topk ||
      !a.slot_tab || !a.xh || !a.xl || !a.ypart || a.n > kMaxExpertsTopK)
    return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(a.ngroups * a.nsplit));
  const uint32_t lds = grp_lds_bytes(a.upw);
  const int nt = (a.upw / 16 + a.waves - 1) / a.waves;  // tiles of a wave
#define SPP_GROUPED(W, NT)                                                                                  \
  if (start || stop)                                                                                        \
    hipExtLaunchKernelGGL((ffn_grouped_kernel<W, NT>), grid, dim3(64 * W), lds, st, start, stop, 0u, a);    \
  else                                                                                                      \
    hipLaunchKernelGGL((ffn_grouped_kernel<W, NT>), grid, dim3(64 * W), lds, st, a)
  if (a.waves == 4) {
    switch (nt) {
      case 1: SPP_GROUPED(4, 1); break;
      case 2: SPP_GROUPED(4, 2); break;
      case 3: SPP_GROUPED(4, 3); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (nt) {
      case 1: SPP_GROUPED(8, 1); break;
      case 2: SPP_GROUPED(8, 2); break;
      case 3: SPP_GROUPED(8, 3); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef SPP_GROUPED
  return hipGetLastError();
}

void batch_units_split(int I, int D, int dtype, int* nsplit, int* upw) {
  const int nchl = dtype == 1 ? nch_for<uint16_t>(D) : nch_for<float>(D);
  *upw = (dtype == 1 ? batch_rounds<uint16_t>(nchl) : batch_rounds<float>(nchl)) * kSlWaves;
  *nsplit = (I + *upw - 1) / *upw;
}

template <typename T, bool FULL>
hipError_t ffn_units_batch_tf(const GroupArgs& a, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  const dim3 grid(static_cast<unsigned>(a.ngroups * a.nsplit)), block(64 * kSlWaves);
  if (start || stop) {
    SPP_DISPATCH_NCH(nch_for<T>(a.D),
                     hipExtLaunchKernelGGL((ffn_units_batch_kernel<T, NCH, FULL, batch_rounds<T>(NCH), slices_ds<NCH>()>),
                                           grid, block, 0, st, start, stop, 0u, a));
  } else {
    SPP_DISPATCH_NCH(nch_for<T>(a.D),
                     hipLaunchKernelGGL((ffn_units_batch_kernel<T, NCH, FULL, batch_rounds<T>(NCH), slices_ds<NCH>()>),
                                        grid, block, 0, st, a));
  }
  return hipGetLastError();
}

hipError_t launch_ffn_units_batch(const GroupArgs& a, int dtype, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  int nsplit = 0, upw = 0;
  batch_units_split(a.I, a.D, dtype, &nsplit, &upw);
  if (a.ngroups <= 0 || a.nsplit != nsplit || a.upw != upw || !a.topk || !a.slot_tab || !a.x || !a.ypart ||
      a.n > kMaxExpertsTopK)
    return hipErrorInvalidValue;
  if (dtype == 1)
    return full_rows<uint16_t>(a.D) ? ffn_units_batch_tf<uint16_t, true>(a, st, start, stop)
                                    : ffn_units_batch_tf<uint16_t, false>(a, st, start, stop);
  return full_rows<float>(a.D) ? ffn_units_batch_tf<float, true>(a, st, start, stop)
                               : ffn_units_batch_tf<float, false>(a, st, start, stop);
}

hipError_t launch_combine_batched(const CombineBArgs& args, int dtype, hipStream_t st) {
  CombineBArgs a = args;
  const int npairs = a.K + a.n_shared;
  if (a.D % 4 != 0 || npairs < 1 || npairs > kMaxWork || a.nsplit < 1) return hipErrorInvalidValue;
  a.parts = std::max(1, std::min(kCombWaves / npairs, (a.nsplit + kCombRanges - 1) / kCombRanges));
  const dim3 grid((a.D / 4 + 63) / 64, a.B);
  const dim3 block(64 * min(npairs * a.parts, kCombWaves));
  const int per = (a.nsplit + a.parts - 1) / a.parts;
#define SPP_COMBINE(RG)                                                                       \
  if (dtype == 1)                                                                             \
    hipLaunchKernelGGL((ffn_combine_batched_kernel<uint16_t, RG>), grid, block, 0, st, a);    \
  else                                                                                        \
    hipLaunchKernelGGL((ffn_combine_batched_kernel<float, RG>), grid, block, 0, st, a)
  if (per <= 1) {
    SPP_COMBINE(1);
  } else if (per <= 2) {
    SPP_COMBINE(2);
  } else if (per <= 4) {
    SPP_COMBINE(4);
  } else if (per <= 8) {
    SPP_COMBINE(8);
  } else {
    SPP_COMBINE(kCombRanges);
  }
#undef SPP_COMBINE
  return hipGetLastError();
}

hipError_t launch_h2d_copies(const CopyList& list, int wgs, hipStream_t st) {
  if (list.n < 0 || list.n > kMaxCopyList || wgs < 1) return hipErrorInvalidValue;
  for (int t = 0; t < list.n; ++t)
    if (reinterpret_cast<uintptr_t>(list.src[t]) % 16 != 0 || reinterpret_cast<uintptr_t>(list.dst[t]) % 16 != 0)
      return hipErrorInvalidValue;
  if (list.n == 0 || list.n16 == 0) return hipSuccess;
  hipLaunchKernelGGL(h2d_copy_kernel, dim3(wgs), dim3(256), 0, st, list);
  return hipGetLastError();
}

hipError_t launch_set_table(int32_t* dst, const int32_t* src, int n, hipStream_t st) {
  if (!dst || !src || n < 1) return hipErrorInvalidValue;
  for (int i0 = 0; i0 < n; i0 += kTableChunk) {
    TableArg t{};
    const int m = std::min(n - i0, kTableChunk);
    std::copy(src + i0, src + i0 + m, t.v);
    hipLaunchKernelGGL(set_table_kernel, dim3(1), dim3(256), 0, st, t, dst + i0, m);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_spin(uint64_t ticks, uint32_t max_iter, hipStream_t st) {
  hipLaunchKernelGGL(spin_kernel, dim3(1), dim3(64), 0, st, ticks, max_iter);
  return hipGetLastError();
}

int ffn_grid_q4(int nunits, int I, int* upw, int* upp) {
  // units per wave and pass: 3, or 4 where a pass of 3 per wave cannot tile
  // an expert's I units but one of 4 can (I = 896: 13.4 -> 12.3 us for one
  // launch over 8 DeepSeek-shaped experts); then whole passes per wave, as
  // many as keep the grid near 256 workgroups: a wave's later passes load
  // while its earlier ones decode (8 Qwen-shaped experts: 17.4 us at 512
  // workgroups of one pass, 13.9 us at 256 of two), at least as many as keep
  // the grid within the partial buffer (ffn_max_grid rows), and preferably
  // a count whose units per workgroup divide I, so that every workgroup
  // works on one expert
  *upp = (I % (kFfnWaves * 3) != 0 && I % (kFfnWaves * 4) == 0) ? 4 : 3;
  const int pass = kFfnWaves * *upp;
  int passes = (nunits + pass * kQ4TargetWgs - 1) / (pass * kQ4TargetWgs);
  passes = std::max(std::max(passes, (nunits + pass * 4096 - 1) / (pass * 4096)), 1);
  for (int p = passes; p < passes + 3; ++p)
    if (I % (pass * p) == 0) {
      passes = p;
      break;
    }
  *upw = pass * passes;
  return (nunits + *upw - 1) / *upw;
}

int ffn_grid_q4_sweep(int nunits, int* rounds, int* upp) {
  // one pass of 3 units per wave where the grid stays within the partial
  // buffer (ffn_max_grid rows), else two; 0 where two passes do not fit
  const int per_wg = kFfnWaves * 3;
  for (int r = 1; r <= 2; ++r) {
    const long grid = (static_cast<long>(nunits) + per_wg * r - 1) / (per_wg * r);
    if (grid <= static_cast<long>(ffn_max_grid())) {
      *rounds = r;
      *upp = 3;
      return static_cast<int>(grid);
    }
  }
  return 0;
}

template <int NQ, bool FULLQ>
hipError_t read_probe_q4_t(const FfnArgs& a, int grid, uint32_t* sink, hipStream_t st, hipEvent_t start,
                           hipEvent_t stop) {
  if (a.rounds == 1)
    hipExtLaunchKernelGGL((read_probe_q4_kernel<NQ, FULLQ, 1>), dim3(grid), dim3(kFfnThreads), 0, st, start, stop, 0u,
                          a, sink);
  else
    hipExtLaunchKernelGGL((read_probe_q4_kernel<NQ, FULLQ, 2>), dim3(grid), dim3(kFfnThreads), 0, st, start, stop, 0u,
                          a, sink);
  return hipGetLastError();
}

hipError_t launch_read_probe(const FfnArgs& a, int grid, uint32_t* sink, hipStream_t st, hipEvent_t start,
                             hipEvent_t stop) {
  if (a.nW <= 0 || a.nW > kMaxWork || grid <= 0 || a.rounds < 1 || a.rounds > kSlMaxRounds || !sink) return hipErrorInvalidValue;
  if (a.codec == 1) {
    // the sweep-order 4-bit FFN's loads: 3 units per wave and pass, 1 or 2 passes
    if (a.rounds > 2 || a.upp != 3 || a.D % 256 != 0 || a.D > 4096 ||
        static_cast<long>(grid) * kFfnWaves * 3 * a.rounds < static_cast<long>(a.nW) * a.I)
      return hipErrorInvalidValue;
    const int nblk = a.D / 32;
    if (nblk == 64) return read_probe_q4_t<1, true>(a, grid, sink, st, start, stop);
    if (nblk < 64) return read_probe_q4_t<1, false>(a, grid, sink, st, start, stop);
    if (nblk == 128) return read_probe_q4_t<2, true>(a, grid, sink, st, start, stop);
    return read_probe_q4_t<2, false>(a, grid, sink, st, start, stop);
  }
  if (static_cast<long>(grid) * kSlWaves * a.rounds < static_cast<long>(a.nW) * a.I) return hipErrorInvalidValue;
  const int nchl = nch_for<uint16_t>(a.D);
  if (a.rounds > slices_rounds<uint16_t>(nchl)) return hipErrorInvalidValue;
#define SPP_PROBE(RR)                                                                                       \
  SPP_DISPATCH_NCH(nchl, hipExtLaunchKernelGGL((read_probe_kernel<NCH, (RR <= slices_rounds<uint16_t>(NCH) ? RR : 1), slices_ds<NCH>()>), \
                                                dim3(grid), dim3(64 * kSlWaves), 0, st, start, stop, 0u, a, sink))
  switch (a.rounds) {
    case 1: SPP_PROBE(1); break;
    case 2: SPP_PROBE(2); break;
    default: SPP_PROBE(3); break;
  }
#undef SPP_PROBE
  return hipGetLastError();
}

hipError_t launch_stream_probe(const void* base, size_t bytes, uint32_t* sink, hipStream_t st, hipEvent_t start,
                               hipEvent_t stop) {
  if (!base || !sink || bytes < 16 || bytes % 16 != 0 || reinterpret_cast<uintptr_t>(base) % 16 != 0)
    return hipErrorInvalidValue;
  hipExtLaunchKernelGGL(stream_probe_kernel, dim3(kStreamGrid), dim3(256), 0, st, start, stop, 0u,
                        static_cast<const u32x4*>(base), bytes / 16, sink);
  return hipGetLastError();
}

int ffn_grid_slices(int nunits, int D, int dtype, int target_wgs, int* rounds) {
  const int nchl = dtype == 1 ? nch_for<uint16_t>(D) : nch_for<float>(D);
  const int rmax = dtype == 1 ? slices_rounds<uint16_t>(nchl) : slices_rounds<float>(nchl);
  const long per = static_cast<long>(kSlWaves) * std::max(target_wgs, 1);
  // Up to 4 chunks per lane: the number of rounds that puts the grid nearest
  // target_wgs (see slices_rounds).  Longer rows: the fewest with at most
  // target_wgs workgroups, two per compute unit, which is what two rounds leave
  // resident.  One round against two, the layer in us: 3,600 units of 2,304
  // columns 23.7 and 20.0, of 2,816 25.9 and 21.5, of 1,900 fp32 columns 28.9
  // and 24.1; 2,400 units 18.9 and 18.0, 20.4 and 19.3, 22.4 and 21.5.
  int r = static_cast<int>((nunits + (nchl <= 4 ? per / 2 : per - 1)) / per);
  r = std::min(std::max(r, 1), rmax);
  int grid = (nunits + kSlWaves * r - 1) / (kSlWaves * r);
  if (grid > static_cast<int>(ffn_max_grid())) return 0;  // the partial rows would not fit
  *rounds = r;
  return grid;
}

int ffn_grid_for(int nunits, int target_wgs, int* upw) {
  int grid = (nunits + kFfnWaves - 1) / kFfnWaves;
  if (grid > target_wgs) grid = target_wgs;
  if (grid < 1) grid = 1;
  *upw = (nunits + grid - 1) / grid;
  return (nunits + *upw - 1) / *upw;
}

size_t ffn_max_grid() { return 4096; }

}  // namespace spp
