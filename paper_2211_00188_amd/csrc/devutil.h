// Wavefront-64 device helpers shared by the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace adacgd {

__device__ __forceinline__ uint32_t lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// set bits of m that belong to lanes below the caller
__device__ __forceinline__ uint32_t below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ uint32_t popc64(uint64_t m) { return (uint32_t)__popcll(m); }

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    uint32_t w = __shfl_xor(v, o, 64);
    v = w > v ? w : v;
  }
  return v;
}

// Reductions and scans over a wavefront by data-parallel moves: a stage is a move and an add in the vector
// pipe, where a shuffle is a round trip through the LDS unit (a sum of doubles: 0.05 instead of 0.3 us).
// Stages: shifts by 1, 2, 4, 8 inside each row of 16 lanes, then the row totals are carried on, so the last lane
// ends with the sum of all.  A lane without a source adds zero.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or0(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or0(double v) {
  return __hiloint2double((int)dpp_or0<CTRL, ROWS>((uint32_t)__double2hiint(v)), (int)dpp_or0<CTRL, ROWS>((uint32_t)__double2loint(v)));
}
constexpr int kDppShr = 0x110, kDppBcast15 = 0x142, kDppBcast31 = 0x143;
template <typename T>
__device__ __forceinline__ T row_scan(T v) {       // inclusive prefix sums inside every row of 16 lanes
  v += dpp_or0<kDppShr + 1, 0xf>(v);
  v += dpp_or0<kDppShr + 2, 0xf>(v);
  v += dpp_or0<kDppShr + 4, 0xf>(v);
  v += dpp_or0<kDppShr + 8, 0xf>(v);
  return v;
}
template <typename T>
__device__ __forceinline__ T wave_scan(T v) {      // inclusive prefix sums over the wavefront
  v = row_scan(v);
  v += dpp_or0<kDppBcast15, 0xa>(v);
  v += dpp_or0<kDppBcast31, 0xc>(v);
  return v;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
template <typename T>
__device__ __forceinline__ T wave_total(T v) { return lane_value(wave_scan(v), 63); }
__device__ __forceinline__ uint32_t wave_top(uint32_t v) {      // maximum
  v = max(v, dpp_or0<kDppShr + 1, 0xf>(v));
  v = max(v, dpp_or0<kDppShr + 2, 0xf>(v));
  v = max(v, dpp_or0<kDppShr + 4, 0xf>(v));
  v = max(v, dpp_or0<kDppShr + 8, 0xf>(v));
  v = max(v, dpp_or0<kDppBcast15, 0xa>(v));
  v = max(v, dpp_or0<kDppBcast31, 0xc>(v));
  return lane_value(v, 63);
}

// Lane by lane: a + (a of the partner lane) where the lane's bit O is clear, b + (b of the partner lane) where it is
// set; partners are O = 32 or 16 lanes apart.  One swap a word (of the upper half -- or odd rows -- of a with the lower
// half -- or even rows -- of b) and one addition.
template <int O>
__device__ __forceinline__ double halves_sum(double a, double b) {
  const uint32_t al = (uint32_t)__double2loint(a), ah = (uint32_t)__double2hiint(a), bl = (uint32_t)__double2loint(b), bh = (uint32_t)__double2hiint(b);
  if constexpr (O == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap(al, bl, false, false), hi = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap(al, bl, false, false), hi = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
  }
}

// Sums of eight values over the wavefront: lane l gets that of p[l / 8].  Every exchange halves the values that a lane
// carries: ten additions instead of the 48 of eight wave_total.
__device__ __forceinline__ double wave_total8(double (&p)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) p[i] = halves_sum<32>(p[i], p[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) p[i] = halves_sum<16>(p[i], p[i + 2]);
  const bool up = (lane_id() & 8u) != 0;
  double a0 = p[0], a1 = p[1];
  asm volatile("" : "+v"(a0), "+v"(a1));      // (else: a select of addresses, and from that one of every element)
  p[0] = (up ? a1 : a0) + dpp_or0<0x128, 0xf>(up ? a0 : a1);      // row_ror:8
  p[0] += dpp_or0<0x141, 0xf>(p[0]);       // row_half_mirror
  p[0] += dpp_or0<0x4e, 0xf>(p[0]);        // quad_perm 2 3 0 1
  p[0] += dpp_or0<0xb1, 0xf>(p[0]);        // quad_perm 1 0 3 2
  return p[0];
}

// Sum over a 256-thread block in a fixed order; result valid in every thread.
__device__ __forceinline__ double block_sum(double v, double* lds4) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
  __syncthreads();
  return (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
}

// Exclusive prefix sum over the 256 threads of a block (thread order); *total gets the sum.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds4, uint32_t* total) {
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t t = __shfl_up(inc, o, 64);
    if (lane >= (uint32_t)o) inc += t;
  }
  __syncthreads();
  if (lane == 63) lds4[w] = inc;
  __syncthreads();
  uint32_t base = 0;
  for (uint32_t i = 0; i < w; ++i) base += lds4[i];
  *total = lds4[0] + lds4[1] + lds4[2] + lds4[3];
  return base + inc - v;
}

// Data that one block writes and another block of the same launch reads goes through
// agent-scope atomic accesses only (relaxed atomic stores, loads and read-modify-writes):
// those are performed at the device's point of coherence, so no cache write-back or
// invalidate is needed to make them visible -- a release/acquire fence at agent scope
// would write back and invalidate the whole L2 of the XCD once per block.
template <typename T>
__device__ __forceinline__ T ld_coherent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_coherent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A group of blocks that meet: every block adds one to the group's word as it begins.  Nobody waits for the group until the word
// says that all `count` blocks have begun, or that the group is given up: where it is `late`, the word is marked unless it
// is complete by then, and a mark is final, as completeness is -- all blocks of the group learn the same.  A complete group
// is running, so that its blocks may wait for each other from then on.  Called by whole wavefronts; returns the word.
constexpr uint32_t kGivenUp = 1u << 31;
__device__ __forceinline__ uint32_t poll_begun(uint32_t* word, uint32_t count, bool late) {
  uint32_t v = ld_coherent(word);
  if (late && v < count) {
    if (lane_id() == 0) {
      uint32_t there = v;
      if (__hip_atomic_compare_exchange_strong(word, &there, v | kGivenUp, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) there |= kGivenUp;
      v = there;
    }
  }
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Every block of a node calls this once after its last coherent write.  Returns true in
// all threads of exactly one block per node: the one that arrived last.  That block may
// then read what the others wrote (with ld_coherent) and finish the node's work; the
// counters are back at zero when it returns.  No block ever waits for another.
// Ordering: each wave first waits until its own vector stores and atomics have completed
// (vmcnt reaches 0), the block barrier extends that to the whole block, and only then is
// the arrival counted.
// Arrivals are counted in two levels (kArriveFan first-level counters per node, then one
// second-level counter) because a few thousand read-modify-writes on one address -- or on
// one cache line -- take ~12 ns each, one after the other.  `counters` points at the node's
// kArriveFan + 1 counters, one per kCounterStride words (= one per 64-byte line); `block` is the
// caller's index among the nblocks blocks.
constexpr int kArriveFan = 32;
constexpr int kCounterStride = 16;

__device__ __forceinline__ bool arrive_last(uint32_t* counters, uint32_t nblocks, uint32_t block, int* lds_flag) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t sub = block % kArriveFan;
    const uint32_t nsub = (nblocks - sub + kArriveFan - 1) / kArriveFan;     // blocks sharing this counter
    const uint32_t nfan = nblocks < (uint32_t)kArriveFan ? nblocks : (uint32_t)kArriveFan;
    int last = 0;
    uint32_t prev = __hip_atomic_fetch_add(&counters[(1 + sub) * kCounterStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (prev == nsub - 1) {
      __hip_atomic_store(&counters[(1 + sub) * kCounterStride], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      prev = __hip_atomic_fetch_add(&counters[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (prev == nfan - 1) {
        __hip_atomic_store(&counters[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = 1;
      }
    }
    *lds_flag = last;
  }
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return *lds_flag != 0;
}

// The same for up to 64 blocks: one counter is enough.
__device__ __forceinline__ bool arrive_last_few(uint32_t* counter, uint32_t nblocks, int* lds_flag) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = prev == nblocks - 1;
    if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *lds_flag = last;
  }
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return *lds_flag != 0;
}

// LDS histogram increment by the lanes that call it (they may be a divergent subset).  The
// lanes that share the first active lane's bin are counted with one atomic: vectors with many
// equal magnitudes (zeros above all) would otherwise serialise up to 64 same-address atomics.
__device__ __forceinline__ void hist_add(uint32_t* hist, uint32_t bin) {
  const uint32_t first = __builtin_amdgcn_readfirstlane(bin);
  const uint64_t same = ballot(bin == first);
  if (bin != first) atomicAdd(&hist[bin], 1u);
  else if (below(same) == 0) atomicAdd(&hist[first], popc64(same));
}

// A range of memory behind a buffer descriptor: accesses take a byte offset, need only the 4-byte alignment
// that every row of floats has, and are checked dword by dword -- what lies at or beyond `bytes` reads as zero
// and is not written.  Ragged ends then cost no branch, and an optional array is one of zero bytes.
typedef uint32_t bword4 __attribute__((ext_vector_type(4)));
typedef uint32_t bword2 __attribute__((ext_vector_type(2)));
struct Buf {
  __amdgpu_buffer_rsrc_t r;
};
__device__ __forceinline__ Buf make_buf(const void* p, uint32_t bytes) {
  return Buf{__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000)};
}
constexpr int kStream = 2;       // cache hint of a vector that is read or written once: do not keep
template <int HINT = 0>
__device__ __forceinline__ void buf_load4(const Buf& b, uint32_t off, uint32_t base, float (&o)[4]) {
  const bword4 q = __builtin_amdgcn_raw_buffer_load_b128(b.r, off, base, HINT);
#pragma unroll
  for (int c = 0; c < 4; ++c) o[c] = __uint_as_float(q[c]);
}
// (No scalar register for the offset: with one the compiler lets the next instruction overwrite the data registers, which
// the architecture's manual allows but for which stores of more than 64 bits were seen to write the new contents, a few
// times in a thousand.  Without one it puts the wait states in between.)
template <int HINT = 0>
__device__ __forceinline__ void buf_store4(const Buf& b, uint32_t off, uint32_t base, const float (&o)[4]) {
  bword4 q;
#pragma unroll
  for (int c = 0; c < 4; ++c) q[c] = __float_as_uint(o[c]);
  __builtin_amdgcn_raw_buffer_store_b128(q, b.r, off + base, 0, HINT);
}

__device__ __forceinline__ uint32_t fbits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t magkey(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

// d/dx_j of the regulariser lambda sum_j x_j^2 / (1 + x_j^2)
__device__ __forceinline__ double reg_grad(double lambda, double xj) {
  const double q = 1.0 + xj * xj;
  return 2.0 * lambda * xj / (q * q);
}

}  // namespace adacgd
