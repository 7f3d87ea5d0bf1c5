// Gradients of the logistic objective from dense features, in one launch (server.hip has the two-kernel form for rows too
// long for it, and the sparse one).
#include "devutil.h"
#include "engine.h"

namespace adacgd {

// ---------------------------------------------------------------------------
// The same gradient with the features read once (dense features, d <= kGradCols * kNodeParts).
// A block keeps kGradRows rows at a time of its columns in registers: forms their products with x, turns the
// complete products into the weights s_l, and adds s_l a_l to its column sums before it lets go of them.
// CW wavefronts of 256 columns share a row, RG groups of them hold different rows.  Rows longer than a block's
// columns are spread over col_parts blocks that leave each other their partial products; those are polled
// themselves: a slot holds zero until its value (a zero is stored as -0) is there, and a launch clears the set that
// the previous one used.
// Waiting.  Blocks take their place by ticket and wait only for the col_parts <= kNodeParts blocks of their own row chunk.
// Those need not be running all at once (other launches may have filled the device): a block counts itself as it begins,
// and where the count is not complete after some time the chunk is given up, its blocks leave, and the last of them to
// come forms its sums alone.
// Bound by the read of the features where that is long; two blocks a compute unit (16 rows x 4 columns a lane are half
// the registers), so that one reads while the other meets.  Measured against the two kernels that read the features
// twice: 1000 workers x 32 rows x 65536 columns 1.82 ms a gradient (2.90), 20 x 2500 x 300 16 us (29), 10 x 203 x 5003
// 19 us (37), 4 x 64 x 100 4.0 us (7.9).  Blocks have no more groups of wavefronts than a shard has rows for: with eight,
// 2000 x 8 x 300 took 24 us (18 with two kernels), now 10 us.
// ---------------------------------------------------------------------------

// Where a lane's four columns lie.  TURNS: the P blocks of a row take turns of 256 columns, so that what a block reads is spread
// over the memory's channels as the whole row is: with 2048 columns side by side some blocks had their rows after 4 us and waited
// 15 us for others' (1000 x 32 rows x 65536 columns: 1.95 ms, in turns 1.87).  Otherwise side by side.
struct GradColumns {
  uint32_t first, len;       // the row from `first` on, as far as the block may go
  uint32_t off;              // byte offset of the lane's columns in it
};
template <bool TURNS>
__device__ __forceinline__ GradColumns grad_columns(const LogisticData& ld, uint32_t d, uint32_t P, uint32_t part, uint32_t wave, uint32_t lane) {
  if (TURNS) return {0, d, ((wave * P + part) * 64 + lane) * 16};
  const uint32_t first = part * (uint32_t)ld.part_cols;
  return {first, min((uint32_t)ld.part_cols, d - first), (wave * 64 + lane) * 16};
}

__device__ __forceinline__ double grad_weight(double yl, double z, double N) { return -yl / (1.0 + exp(yl * z)) / N; }

// Sums of the RG groups of wavefronts, in group order, in group 0; share: four values of every thread, thread by thread (null if
// RG = 1), of which nobody reads any more (a barrier lies behind the last call's reads: arrive_last_few).
template <int RG>
__device__ __forceinline__ void add_groups(double (&acc)[4], double* share, int rg) {
  if (RG == 1) return;
  const int lanes = (int)blockDim.x / RG, mine = (int)threadIdx.x - rg * lanes;
#pragma unroll
  for (int c = 0; c < 4; ++c) share[(rg * 4 + c) * lanes + mine] = acc[c];
  __syncthreads();
  if (rg == 0) {
#pragma unroll
    for (int g = 1; g < RG; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] += share[(g * 4 + c) * lanes + mine];
  }
}

// What a block does with its column sums (four a lane, the part's quad `at`, in group 0 of its RG groups of
// wavefronts): the gradient, or with several chunks a shard -- each leaves its sums, and the last to arrive adds them:
// kGradFold of them; of more chunks, the last of every kGradFold leaves their sum, and the last of those adds these (one
// block adding all of them took 140 us for 1 x 4000 rows x 2048 columns, 250 chunks).  Several groups share the work, the groups'
// sums added in their order, where that takes rounds of loads off; up to kGradFoldAll chunks are then added at once (20 x 2500
// rows x 300 columns, 20 chunks: 18.0 us instead of 20.4).  Not more at once, since they arrive at one counter and end up in
// one block (128 at once: 1 x 20000 rows x 100 columns 16.2 us; 16 and then ten, 13.2, shared 12.7), and fewer are not shared
// (50 x 700 x 100, six chunks: 12.2 us shared and 11.6 not).
template <int RG>
__device__ __forceinline__ void finish(const LogisticData& ld, float* __restrict__ grads, int64_t d, int node, int rc, int nchunks, int slot0,
                                       uint32_t P, uint32_t part, const GradColumns& gc, uint32_t at, int rg, const float (&xq)[4], double (&acc)[4],
                                       double* share, int* flag) {
  const uint32_t l0 = gc.off / 4;
  if (nchunks > 1) {
    // (a part's columns 0, 4, 8, ... lie side by side, so that a wavefront's accesses do)
    const uint32_t quads = ((uint32_t)ld.part_cols + 3) / 4;
    const size_t slot_len = (size_t)P * quads * 4;
    double* __restrict__ sums = ld.part + (size_t)part * quads * 4 + at;
    auto leave = [&](int slot) {
      if (rg == 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (l0 + c < gc.len) st_coherent(&sums[(size_t)slot * slot_len + c * quads], acc[c]);
      }
    };
    auto add = [&](int slot, int count, int stride) {
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = 0.0;
      const bool shared = RG > 1 && count > kGradFoldShare;
      const int step = shared ? RG : 1;
      for (int r0 = shared ? rg : rg == 0 ? 0 : count; r0 < count; r0 += 8 * step) {        // eight loads of a column in flight
        double v[8][4];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            v[u][c] = r0 + u * step < count && l0 + c < gc.len ? ld_coherent(&sums[(size_t)(slot + (r0 + u * step) * stride) * slot_len + c * quads]) : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[c] += v[u][c];
      }
      if (shared) add_groups<RG>(acc, share, rg);
    };
    leave(slot0 + rc);
    const int fold = RG > 1 && nchunks <= kGradFoldAll ? nchunks : kGradFold;
    const int sub = rc - rc % fold, members = min(fold, nchunks - sub);
    if (!arrive_last_few(&ld.col_done[(size_t)(slot0 + sub) * P + part], (uint32_t)members, flag)) return;
    add(slot0 + sub, members, 1);
    if (nchunks > fold) {
      leave(slot0 + sub);
      const int subs = (nchunks + fold - 1) / fold;
      if (!arrive_last_few(&ld.col_done[(size_t)(ld.part_slots + slot0) * P + part], (uint32_t)subs, flag)) return;
      add(slot0, subs, fold);
    }
  }
  if (rg != 0) return;
  float g[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) g[c] = (float)(acc[c] + reg_grad(ld.lambda, (double)xq[c]));
  buf_store4(make_buf(grads + (size_t)node * (size_t)d + gc.first, 4 * gc.len), gc.off, 0, g);
}

// A whole row chunk by one block of eight wavefronts: the weights of its rows, left where the products were (nobody polls
// them any more), then one part of the columns after the other.
template <bool TURNS>
__device__ __forceinline__ void grad_alone(const LogisticData& ld, const float* __restrict__ x, float* __restrict__ grads, int64_t d, int node, int rc,
                                        int nchunks, int slot0, uint32_t r_begin, int rows, double N, double* slots, int* flag) {
  const uint32_t P = (uint32_t)ld.col_parts, lane = threadIdx.x & 63;
  for (int row = (int)(threadIdx.x >> 6); row < rows; row += 8) {
    const float* __restrict__ a = ld.A + (size_t)(r_begin + (uint32_t)row) * (size_t)d;
    double z = 0.0;
    for (uint32_t l = lane; l < (uint32_t)d; l += 64) z = fma((double)a[l], (double)x[l], z);
    z = wave_total(z);
    if (lane == 0) st_coherent(&slots[(size_t)row * P], grad_weight((double)ld.labels[r_begin + (uint32_t)row], z, N));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (uint32_t p = 0; p < P; ++p) {
    const GradColumns gc = grad_columns<TURNS>(ld, (uint32_t)d, P, p, threadIdx.x >> 6, lane);
    float xq[4];
    buf_load4(make_buf(x + gc.first, 4 * gc.len), gc.off, 0, xq);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int row = 0; row < rows; ++row) {
      float a[4];
      buf_load4(make_buf(ld.A + (size_t)(r_begin + (uint32_t)row) * (size_t)d + gc.first, 4 * gc.len), gc.off, 0, a);
      const double s = ld_coherent(&slots[(size_t)row * P]);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = fma(s, (double)a[c], acc[c]);
    }
    finish<1>(ld, grads, d, node, rc, nchunks, slot0, P, p, gc, threadIdx.x, 0, xq, acc, nullptr, flag);
  }
}

// PARTED: rows are longer than a block's columns (CW = 8, RG = 1).  STREAM: the features are read past the memory-side cache
// (1000 x 32 rows x 65536 columns: 1.87 ms, so 1.82).
template <int CW, int RG, bool PARTED, bool TURNS = false, bool STREAM = false>
__global__ __launch_bounds__(64 * CW * RG, 4) void k_grad(LogisticData ld, const float* __restrict__ x, float* __restrict__ grads, int64_t d) {
  constexpr int R = kGradRows, NT = 64 * CW * RG;
  __shared__ double red[CW * RG][R], s_m[RG][R];
  __shared__ double s_acc[RG > 1 ? RG * CW * 256 : 1];
  __shared__ uint32_t s_blk;
  __shared__ int s_flag, s_quit;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), cw = w % CW, rg = w / CW;
  const uint32_t lane = tid & 63;
  const uint32_t P = PARTED ? (uint32_t)ld.col_parts : 1u;
  uint32_t blk = blockIdx.x;
  if (PARTED && ld.ticket) {
    if (tid == 0) s_blk = __hip_atomic_fetch_add(&ld.ticket[ld.parity * kCounterStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    blk = s_blk;
    if (blk == 0 && tid == 0) ld.ticket[(ld.parity ^ 1) * kCounterStride] = 0;
  }
  // (kept in scalar registers, also the results of divisions and loads, and without 64-bit comparisons: buffer
  // descriptors made from vector registers would be taken apart lane by lane)
  auto scalar = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  blk = scalar(blk);
  const uint32_t group = scalar(blk / P), part = blk - group * P;
  // shard, chunk of its rows, number of its chunks, where their partial sums begin
  int node, rc, nchunks, slot0;
  if (ld.row_chunks) {
    nchunks = ld.row_chunks;
    node = (int)scalar(group / (uint32_t)nchunks);
    rc = (int)group - node * nchunks;
    slot0 = node * nchunks;
  } else {
    const int4 t = ld.chunks[group];
    node = (int)scalar((uint32_t)t.x);
    rc = (int)scalar((uint32_t)t.y);
    nchunks = (int)scalar((uint32_t)t.z);
    slot0 = (int)scalar((uint32_t)t.w);
  }
  // (a row number fits 31 bits: the host's choice of this kernel)
  const uint32_t r_first = scalar((uint32_t)ld.offsets[node]);
  const int count = (int)(scalar((uint32_t)ld.offsets[node + 1]) - r_first);
  const int skip = rc * ld.chunk_rows, rows = max(0, min(count - skip, ld.chunk_rows));
  const uint32_t r_begin = r_first + (uint32_t)skip;
  const double N = (double)count;
  const GradColumns gc = grad_columns<TURNS>(ld, (uint32_t)d, P, part, (uint32_t)cw, lane);
  const size_t set = (size_t)ld.rows * P;
  double* __restrict__ slots = PARTED ? ld.meet + ld.parity * set + (size_t)r_begin * P : nullptr;
  if (PARTED) {       // the set the previous launch used, cleared for the next one
    double* __restrict__ old = ld.meet + (ld.parity ^ 1) * set + (size_t)r_begin * P;
    for (int i = tid; i < rows; i += NT) old[(size_t)i * P + part] = 0.0;
    if (tid == 0) {
      atomicAdd(&ld.begun[((size_t)ld.parity * ld.groups + group) * kCounterStride], 1u);
      if (part == 0) ld.begun[((size_t)(ld.parity ^ 1) * ld.groups + group) * kCounterStride] = 0;
    }
  }
  if (tid == 0) s_quit = 0;
  float xq[4];
  buf_load4(make_buf(x + gc.first, 4 * gc.len), gc.off, 0, xq);
  auto label = [&](int row) { return row < rows ? ld.labels[r_begin + (uint32_t)row] : 0.f; };      // (asked for before it is needed)
  auto weight = [&](double yl, double z) { return grad_weight(yl, z, N); };
  // The first round's labels come before its rows; later rounds ask when they need them.  Asked for when needed in the first as
  // well, 20 x 2500 rows x 300 columns took 18.7 us (18.0) and 2000 x 8 x 2048 29.6 (27.7); asked for early in all rounds, 400 x 500 x
  // 200, four rounds a block, 30.3 (29.2).
  const float yl_first = !PARTED && tid < R * RG ? label(tid % R * RG + tid / R) : 0.f;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int base = 0; base < rows; base += R * RG) {
    // rows base + r RG + rg of the chunk (rows beyond its end read as zero and get weight zero)
    float a[R][4];
    const float* __restrict__ ap = ld.A + (size_t)(r_begin + (uint32_t)(base + rg)) * (size_t)d + gc.first;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool live = base + r * RG + rg < rows;
      buf_load4<STREAM ? kStream : 0>(make_buf(live ? ap + (size_t)(r * RG) * (size_t)d : ld.A, live ? 4 * gc.len : 0u), gc.off, 0, a[r]);
    }
    // products with x, eight rows at a time (lane l gets the sum of row l / 8)
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += 8) {
      double p[8];
#pragma unroll
      for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(xq[c]));     // (not widened once and for all)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (r % 4 == 0) __builtin_amdgcn_sched_barrier(0);       // (values widened a few rows at a time: more would spill)
        p[r] = (double)a[r0 + r][0] * (double)xq[0];
#pragma unroll
        for (int c = 1; c < 4; ++c) p[r] = fma((double)a[r0 + r][c], (double)xq[c], p[r]);
      }
      const double all = wave_total8(p);
      if ((lane & 7u) == 0) red[w][r0 + (lane >> 3)] = all;
    }
    // (the values widened to fp64 are formed anew below: carrying them along would not fit the registers)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(a[r][c]));
    __syncthreads();
    if (PARTED) {
      if (tid < R && base + tid < rows) {
        double z = 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) z += red[j][tid];
        st_coherent(&slots[(size_t)(base + tid) * P + part], z == 0.0 ? -0.0 : z);
      }
      const int r = tid >> 5, j = tid & 31;
      const bool live = base + r < rows;
      const float yl = label(base + r);
      // (a wavefront leaves the loop as one)
      static_assert(kNodeParts <= 64, "two blocks a lane");
      double t[2] = {0.0, 0.0};                // of blocks j and j + 32
      auto none = [](double v) { return __double_as_longlong(v) == 0; };
      uint32_t begun = base == 0 && w == 0 ? 0u : P;
      for (uint32_t polls = 0;; ++polls) {
        bool open = false;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if (live && (uint32_t)(j + 32 * k) < P && none(t[k])) {
            t[k] = ld_coherent(&slots[(size_t)(base + r) * P + j + 32 * k]);
            open = open || none(t[k]);
          }
        }
        if (begun != P) begun = poll_begun(&ld.begun[((size_t)ld.parity * ld.groups + group) * kCounterStride], P, polls >= ld.polls);
        if (begun & kGivenUp) {
          if (lane == 0) __hip_atomic_store(&s_quit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          break;
        }
        if (begun == P && !ballot(open)) break;
        if (base == 0 && w != 0 && __hip_atomic_load(&s_quit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
      }
      double z = t[0] + t[1];
      z += dpp_or0<0x128, 0xf>(z);             // row_ror: the sum over 16 lanes, in all of them
      z += dpp_or0<0x124, 0xf>(z);
      z += dpp_or0<0x122, 0xf>(z);
      z += dpp_or0<0x121, 0xf>(z);
      z += __shfl_xor(z, 16, 64);
      if (j == 0) s_m[0][r] = live ? weight((double)yl, z) : 0.0;
    } else if (tid < R * RG) {
      const int g = tid / R, r = tid % R, row = base + r * RG + g;
      double z = 0.0;
#pragma unroll
      for (int j = 0; j < CW; ++j) z += red[g * CW + j][r];
      s_m[g][r] = row < rows ? weight((double)(base == 0 ? yl_first : label(row)), z) : 0.0;
    }
    __syncthreads();
    if (PARTED && base == 0 && __builtin_expect(s_quit, 0)) {
      if (arrive_last_few(&ld.alone[group], P, &s_flag)) grad_alone<TURNS>(ld, x, grads, d, node, rc, nchunks, slot0, r_begin, rows, N, slots, &s_flag);
      return;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r % 4 == 0) __builtin_amdgcn_sched_barrier(0);
      const double s = s_m[rg][r];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = fma(s, (double)a[r][c], acc[c]);
    }
  }
  add_groups<RG>(acc, s_acc, rg);
  if (rg == 0 || nchunks > 1) finish<RG>(ld, grads, d, node, rc, nchunks, slot0, P, part, gc, (uint32_t)(cw * 64) + lane, rg, xq, acc, s_acc, &s_flag);
}

hipError_t launch_grad(const LogisticData& ld, const float* x, float* grads, int64_t d, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  const dim3 grid((unsigned)((size_t)ld.groups * ld.col_parts));
  auto go = [&](auto kern, int waves) -> hipError_t {
    hipLaunchKernelGGL(kern, grid, dim3(64 * waves), 0, st, ld, x, grads, d);
    return hipGetLastError();
  };
  const int rg = ld.row_groups;
  switch (grad_col_waves(ld.part_cols)) {
    case 1: return rg == 1 ? go(k_grad<1, 1, false>, 1) : rg == 2 ? go(k_grad<1, 2, false>, 2) : rg == 4 ? go(k_grad<1, 4, false>, 4) : go(k_grad<1, 8, false>, 8);
    case 2: return rg == 1 ? go(k_grad<2, 1, false>, 2) : rg == 2 ? go(k_grad<2, 2, false>, 4) : go(k_grad<2, 4, false>, 8);
    case 4: return rg == 1 ? go(k_grad<4, 1, false>, 4) : go(k_grad<4, 2, false>, 8);
    default: return ld.col_parts == 1 ? go(k_grad<8, 1, false>, 8)
                                  : ld.stream ? go(k_grad<8, 1, true, true, true>, 8) : ld.turns ? go(k_grad<8, 1, true, true>, 8) : go(k_grad<8, 1, true>, 8);
  }
}

}  // namespace adacgd
