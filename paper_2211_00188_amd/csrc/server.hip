// Server side and objective of the AdaCGD iteration:
//   iterate update x <- x - gamma g                       (Algorithm 1)
//   aggregation    g~ <- g~ + (1/n) sum_i message_i       (Algorithm 1, incremental form)
//   local gradients of the logistic objective with the nonconvex regulariser (Section 6)
#include "devutil.h"
#include "engine.h"

namespace adacgd {

// ---------------------------------------------------------------------------
// small dense kernels
// ---------------------------------------------------------------------------
// (out may be x)
__global__ __launch_bounds__(kBlock) void k_xupdate(float* out, const float* x, const float* __restrict__ g, double gamma,
                                                     int64_t d) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < d) out[i] = (float)((double)x[i] - gamma * (double)g[i]);   // one rounding
}

// g~^0 = (1/n) sum_i g~_i^0, summed in ascending i in fp64; written to up to three vectors
__global__ __launch_bounds__(kBlock) void k_mean(const float* __restrict__ gi, float* o0, float* o1, float* o2, int n,
                                                  int64_t d) {
  const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (c >= d) return;
  double acc = 0.0;
  for (int i = 0; i < n; ++i) acc += (double)gi[(size_t)i * d + c];
  const float r = (float)(acc / (double)n);
  o0[c] = r;
  if (o1) o1[c] = r;
  if (o2) o2[c] = r;
}

__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t* p, uint32_t v, size_t count) {
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (size_t)gridDim.x * kBlock) p[i] = v;
}

__global__ __launch_bounds__(kBlock) void k_copy_f32(float* __restrict__ dst, const float* __restrict__ src,
                                                      size_t count) {
  for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (size_t)gridDim.x * kBlock)
    dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// aggregation: one block per group (2048 coordinates) of the server vector.  The group's
// share of every worker's sorted message is a contiguous range (known from the message
// offsets per group).  The ranges of up to 256 workers at a time are laid end to end and the
// threads stride over that flattened list, adding into an fp64 accumulator in LDS; then
// g~_new = fl(g~_old + acc / n).  Sums of fp32 values in fp64 are exact unless their exponents
// spread over more than ~29 bits, so the result does not depend on the order of the additions.
// ---------------------------------------------------------------------------
// DENSE_LATER (level sets with quantisers): the fp64 sums of the sparse messages go to ws.accbuf and
// k_aggregate_dense adds the dense messages and finishes.
// `xu`: with the identity master g is g~, so the kernel that finishes g~_new can also write the next
// iterate x_next = fl(x - gamma g~_new) (xu.out null = not asked for).
template <bool DENSE_LATER>
__global__ __launch_bounds__(kBlock) void k_aggregate(NodeSet ws, const float* __restrict__ gt_old,
                                                       float* __restrict__ gt_new, IterateUpdate xu) {
  __shared__ double acc[kWaveTile];
  __shared__ uint32_t s_lo[kBlock], s_pre[kBlock + 1];
  __shared__ uint32_t lds4[4];
  __shared__ int s_flag;
  const int g = blockIdx.x, tid = threadIdx.x;
  const int64_t d = ws.d;
  const int64_t base = (int64_t)g * kWaveTile;
  // this block's share of the workers (all of them unless several blocks share the group)
  const int AS = gridDim.y, per = (ws.nn + AS - 1) / AS;
  const int n_lo = (int)blockIdx.y * per, n_hi = min(ws.nn, n_lo + per);
  for (int c = tid; c < kWaveTile; c += kBlock) acc[c] = 0.0;
  __syncthreads();
  for (int n0 = n_lo; n0 < n_hi; n0 += kBlock) {
    const int i = n0 + tid;
    uint32_t lo = 0, cnt = 0;
    if (i < n_hi) {
      if (ws.sel_slot[i] >= 0) {
        lo = ws.grp_off[(size_t)i * (ws.groups + 1) + g];
        cnt = ws.grp_off[(size_t)i * (ws.groups + 1) + g + 1] - lo;
      }
    }
    uint32_t total;
    const uint32_t pre = block_excl_scan(cnt, lds4, &total);
    s_lo[tid] = lo;
    s_pre[tid] = pre;
    if (tid == 0) s_pre[kBlock] = total;
    __syncthreads();
    // (four entries a thread side by side: one after the other, the search and the loads of each would be waited for)
    for (uint32_t e0 = tid; e0 < total; e0 += 4 * kBlock) {
      int32_t idx[4];
      float val[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t e = min(e0 + u * kBlock, total - 1);
        // the worker whose range holds flattened entry e: last j with s_pre[j] <= e
        int lo_j = 0, hi_j = kBlock;
#pragma unroll
        for (int step = kBlock / 2; step > 0; step >>= 1) {
          const int mid = (lo_j + hi_j) >> 1;
          if (s_pre[mid] <= e) lo_j = mid; else hi_j = mid;
        }
        const size_t off = (size_t)(n0 + lo_j) * ws.Kcap + s_lo[lo_j] + (e - s_pre[lo_j]);
        idx[u] = ws.msg_idx[off];
        val[u] = ws.msg_val[off];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (e0 + u * kBlock < total) unsafeAtomicAdd(&acc[idx[u] - base], (double)val[u]);
    }
    __syncthreads();
  }
  if (AS > 1) {
    // partial sums of the blocks that share this group; the last one to arrive adds them in block order
    for (int c = tid; c < kWaveTile; c += kBlock)
      st_coherent(&ws.agg_part[((size_t)blockIdx.y * ws.groups + g) * kWaveTile + c], acc[c]);
    if (!arrive_last(&ws.agg_done[(size_t)g * (kArriveFan + 1) * kCounterStride], (uint32_t)AS, blockIdx.y, &s_flag)) return;
    // (sixteen loads in flight a thread: one after the other, each was waited for)
    constexpr int PER = kWaveTile / kBlock, U = 2;
    double t[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) t[k] = 0.0;
    for (int b0 = 0; b0 < AS; b0 += U) {
      double v[U][PER];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < PER; ++k)
          v[u][k] = b0 + u < AS ? ld_coherent(&ws.agg_part[((size_t)(b0 + u) * ws.groups + g) * kWaveTile + k * kBlock + tid]) : 0.0;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < PER; ++k) t[k] += v[u][k];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) acc[k * kBlock + tid] = t[k];       // thread tid wrote and reads the same entries: no barrier needed
  }
  if (DENSE_LATER) {
    for (int c = tid; c < kWaveTile; c += kBlock)
      if (base + c < d) ws.accbuf[base + c] = acc[c];
    return;
  }
  const double n = (double)ws.nn;
  for (int c = tid; c < kWaveTile; c += kBlock) {
    if (base + c < d) {
      const float gn = (float)((double)gt_old[base + c] + acc[c] / n);
      gt_new[base + c] = gn;
      if (xu.out) xu.out[base + c] = (float)((double)xu.x[base + c] - xu.gamma * (double)gn);
    }
  }
}

// Top-K messages of at most kOrderedMax workers: the same sums taken in ASCENDING WORKER INDEX, so that the
// result is the sequential fp64 sum whatever the data (the kernel above adds in arbitrary order, which gives
// the same bits only while the exponents met at one coordinate spread over less than 53 - 24 - log2 n bits).
// One block per group of 2048 coordinates, and inside it every wavefront owns a quarter of them: it walks
// the group's range of every worker's message, worker after worker, and adds the entries that fall into its
// quarter.  A wavefront's LDS operations execute in the order they are issued, and the coordinates of one
// message are distinct, so every coordinate receives its additions in worker order without any barrier; the
// four wavefronts read the same few kilobytes of messages (the later ones from the cache).
// Bound by dependent loads: where the ranges lie is read for all workers at once, a lane each, and the entries of the next two
// senders are on their way while those of two are added, 128 of each (the 64 there were before are less than a message of 5 %
// has in a group, and the rest was waited for worker by worker).  Measured against that: 16 workers of 11.2 million coordinates,
// the four largest sizes sent in turn, 95 -> 57 us, nothing sent 30 -> 20; 8 of 1000003 14.8 -> 7.7; 8 of 20000 9.0 -> 6.1.
// What lies beyond the 128 is waited for 64 by 64 as before: of 64 workers of 1000003 coordinates 5 % 61 -> 30 us, 10 % 116 -> 93,
// 30 % 350 -> 326, all 1061 -> 1073; the shortest messages, 0.01 %, 30 -> 13.7, nothing 15.9 -> 8.5.
constexpr int kOrderedMax = 64;
constexpr int kAggChunk = 2;          // workers whose first kAggAhead entries are on their way while those of the two before are added
constexpr int kAggAhead = 128;

__global__ __launch_bounds__(kBlock) void k_aggregate_ordered(NodeSet ws, const float* __restrict__ gt_old,
                                                               float* __restrict__ gt_new, IterateUpdate xu) {
  static_assert(kOrderedMax <= 64, "a lane per worker");
  __shared__ double acc[kWaveTile];
  constexpr int QUARTER = kWaveTile / 4, PER = QUARTER / 64, A = kAggAhead / 64;
  const int g = blockIdx.x, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int64_t d = ws.d;
  const int64_t base = (int64_t)g * kWaveTile;
  double* mine = acc + w * QUARTER;                       // only this wavefront touches these entries
  const int64_t first = base + w * QUARTER;
  // where every worker's share of the group lies, a lane per worker, all at once
  uint32_t my_lo = 0, my_cnt = 0;
  {
    const size_t at = (size_t)min(lane, ws.nn - 1) * (ws.groups + 1) + g;
    const int slot = ws.sel_slot[min(lane, ws.nn - 1)];
    const uint32_t l0 = ws.grp_off[at], l1 = ws.grp_off[at + 1];
    if (lane < ws.nn && slot >= 0) {
      my_cnt = l1 - l0;
      my_lo = my_cnt ? l0 : 0u;        // (an empty share may begin where the array ends)
    }
  }
  float old[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) old[k] = gt_old[min(first + k * 64 + lane, d - 1)];
#pragma unroll
  for (int k = 0; k < PER; ++k) mine[k * 64 + lane] = 0.0;
  uint64_t left = ballot(my_cnt != 0);                    // workers with entries here, still to be asked for
  // (loads without a branch: what lies beyond a worker's share is its last entry again, and not added)
  struct Chunk {
    int who[kAggChunk];                                   // in ascending order; -1: none
    int32_t idx[kAggChunk][A];
    float val[kAggChunk][A];
  };
  auto fetch = [&](Chunk& c) {
#pragma unroll
    for (int u = 0; u < kAggChunk; ++u) {
      c.who[u] = left ? __builtin_ctzll(left) : -1;
      left &= left - 1;                                   // (zero stays zero)
      const int i = max(c.who[u], 0);
      const uint32_t cnt = lane_value(my_cnt, i);
      const size_t from = (size_t)i * ws.Kcap + lane_value(my_lo, i);
#pragma unroll
      for (int k = 0; k < A; ++k) {
        const size_t off = from + min((uint32_t)(lane + 64 * k), cnt ? cnt - 1 : 0u);
        c.idx[u][k] = ws.msg_idx[off];
        c.val[u][k] = ws.msg_val[off];
      }
    }
  };
  auto add = [&](const Chunk& c) {
#pragma unroll
    for (int u = 0; u < kAggChunk; ++u) {
      const int i = max(c.who[u], 0);
      const uint32_t cnt = c.who[u] >= 0 ? lane_value(my_cnt, i) : 0u;
#pragma unroll
      for (int k = 0; k < A; ++k) {
        if (64u * k < cnt) {                              // (the same in every lane)
          const uint64_t r = (uint64_t)((int64_t)c.idx[u][k] - first);         // (huge for coordinates below this quarter)
          if ((uint32_t)(lane + 64 * k) < cnt && r < (uint64_t)QUARTER) mine[r] += (double)c.val[u][k];
        }
      }
      for (uint32_t e = lane + kAggAhead; e < cnt; e += 64) {
        const size_t off = (size_t)i * ws.Kcap + lane_value(my_lo, i) + e;
        const uint64_t r = (uint64_t)((int64_t)ws.msg_idx[off] - first);
        if (r < (uint64_t)QUARTER) mine[r] += (double)ws.msg_val[off];
      }
    }
  };
  if (left) {
    Chunk one, two;
    fetch(one);
    for (;;) {
      fetch(two);
      add(one);
      if (two.who[0] < 0) break;
      fetch(one);
      add(two);
      if (one.who[0] < 0) break;
    }
  }
  const double n = (double)ws.nn;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int c = k * 64 + lane;
    const int64_t l = first + c;
    if (l < d) {
      const float gn = (float)((double)old[k] + mine[c] / n);
      gt_new[l] = gn;
      if (xu.out) xu.out[l] = (float)((double)xu.x[l] - xu.gamma * (double)gn);
    }
  }
}

// The same sums where the workers' launch has also left every message as a whole vector (at most kServeWorkers workers of
// up to 16384 coordinates): a lane owns a coordinate and adds what the workers hold there, in ascending worker index;
// what a worker does not send adds +0, which changes no sum.  How much they send does not matter, and every coordinate is
// a chain of its own: where workers send most of their vectors, the kernel above walks n entry lists on a few blocks
// (a logistic step of 64 x 2000 341 us there, 44 here, of
// 30 x 4000 190 and 48; where they send little, of 10 x 4096 supplied gradients, 13.3 and 12).
__global__ __launch_bounds__(64) void k_aggregate_short(NodeSet ws, const float* __restrict__ gt_old, float* __restrict__ gt_new,
                                                        IterateUpdate xu) {
  static_assert(kServeWorkers <= 64, "a lane per worker");
  const int lane = threadIdx.x;
  const int64_t d = ws.d, l = (int64_t)blockIdx.x * 64 + lane;
  const bool live = l < d;
  const float old = live ? gt_old[l] : 0.f, x = live && xu.out ? xu.x[l] : 0.f;
  uint64_t senders = ballot(lane < ws.nn && ws.sel_slot[lane < ws.nn ? lane : 0] >= 0);
  double acc = 0.0;
  constexpr int U = 16;
  while (senders) {
    float t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      t[u] = 0.f;
      if (senders) {
        const int i = __builtin_ctzll(senders);
        senders &= senders - 1;
        if (live) t[u] = ws.dense[(size_t)i * (size_t)d + l];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc += (double)t[u];
  }
  if (!live) return;
  const float gn = (float)((double)old + acc / (double)ws.nn);
  gt_new[l] = gn;
  if (xu.out) xu.out[l] = (float)((double)x - xu.gamma * (double)gn);
}

// Dense (quantised, Rank-K) messages: a block owns 256 coordinates, each lane four of them; its eight wavefronts take
// one eighth of the workers each, in ascending order, and their partial sums are combined in wavefront order:
// g~_new = fl(g~_old + (sparse sums + dense sums) / n).  What the workers chose is read for 64 of them at a time, so
// that only the messages themselves are waited for, four workers' at a time (eight would halve the wavefronts in flight):
// with two coordinates a lane and the chain choice -> scale -> codes for every eight workers it took 53 us for 32 workers
// of 2^20 coordinates (now 20) and 135 us for 1000 of 65536 (now 45).
constexpr int kDenseCols = 256;
constexpr int kDenseWaves = 8;
__global__ __launch_bounds__(64 * kDenseWaves, 8) void k_aggregate_dense(NodeSet ws, const float* __restrict__ gt_old,
                                                                      float* __restrict__ gt_new, IterateUpdate xu) {
  __shared__ double part[kDenseWaves][kDenseCols];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int64_t d = ws.d;
  const int64_t c0 = (int64_t)blockIdx.x * kDenseCols + 4 * lane;
  const bool quad = d % 4 == 0;       // rows of codes are then 8-byte aligned at c0, and four coordinates exist or none
  const int q = (ws.nn + kDenseWaves - 1) / kDenseWaves;
  const int i0 = w * q, i1 = min(ws.nn, i0 + q);
  constexpr int U = 4;
  // (what the last part needs, asked for now)
  const int64_t col = (int64_t)blockIdx.x * kDenseCols + tid;
  const bool mine = tid < kDenseCols && col < d;
  const double sparse = mine ? ws.accbuf[col] : 0.0;
  const float gt = mine ? gt_old[col] : 0.f;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  // Rank-K messages are dense fp32 vectors (d is a multiple of 16 then): workers that chose one, in ascending order,
  // before this wavefront's quantised ones
  if (ws.lv.nr > 0) {
    for (int ib = i0; ib < i1; ib += 64) {
      uint64_t m = ballot(ib + lane < i1 && ws.sel_rk[ib + lane] >= 0);
      while (m) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (m) {
            const int i = ib + __builtin_ctzll(m);
            m &= m - 1;
            if (c0 < d) v[u] = *reinterpret_cast<const float4*>(ws.rdense + (size_t)i * d + c0);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          a[0] += (double)v[u].x;
          a[1] += (double)v[u].y;
          a[2] += (double)v[u].z;
          a[3] += (double)v[u].w;
        }
      }
    }
  }
  if (ws.lv.nq > 0) {
    for (int ib = i0; ib < i1; ib += 64) {
      const int i = ib + lane;
      const int qi = i < i1 ? ws.sel_q[i] : -1;
      const uint32_t Bl = qi >= 0 && ws.lv.nqb > 0 ? (uint32_t)ws.lv.qblock[qi] : 0u;      // block-wise level: its block length
      const uint32_t scl = i < i1 ? fbits(ws.qscale[i]) : 0u;
      uint64_t m = ballot(qi >= 0);
      while (m) {
        uint32_t k01[U], k23[U];
        float sc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          k01[u] = k23[u] = 0;
          sc[u] = 0.f;
          if (m) {
            const int j = __builtin_ctzll(m);
            m &= m - 1;
            const uint32_t B = lane_value(Bl, j);
            const int16_t* __restrict__ codes = ws.qcodes + (size_t)(ib + j) * d + c0;
            sc[u] = __uint_as_float(lane_value(scl, j));
            if (B) sc[u] = ws.qbscale[(size_t)(ib + j) * ws.nseg + (c0 < d ? (uint32_t)c0 / B : 0u)];
            if (quad) {
              if (c0 < d) {
                const uint2 two = *reinterpret_cast<const uint2*>(codes);
                k01[u] = two.x;
                k23[u] = two.y;
              }
            } else {
              uint32_t k[4];
#pragma unroll
              for (int c = 0; c < 4; ++c) k[c] = c0 + c < d ? (uint32_t)(uint16_t)codes[c] : 0u;
              k01[u] = k[0] | (k[1] << 16);
              k23[u] = k[2] | (k[3] << 16);
            }
          }
        }
        auto decode = [](int code, float s) {
          const float mag = (float)(code < 0 ? -code : code) * s;
          return (double)(code < 0 ? -mag : mag);
        };
#pragma unroll
        for (int u = 0; u < U; ++u) {
          a[0] += decode((int)(int16_t)(k01[u] & 0xFFFFu), sc[u]);
          a[1] += decode((int)(int16_t)(k01[u] >> 16), sc[u]);
          a[2] += decode((int)(int16_t)(k23[u] & 0xFFFFu), sc[u]);
          a[3] += decode((int)(int16_t)(k23[u] >> 16), sc[u]);
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) part[w][4 * lane + c] = a[c];
  __syncthreads();
  if (mine) {
    double tot = sparse;
#pragma unroll
    for (int j = 0; j < kDenseWaves; ++j) tot += part[j][tid];
    const float gn = (float)((double)gt + tot / (double)ws.nn);
    gt_new[col] = gn;
    if (xu.out) xu.out[col] = (float)((double)xu.x[col] - xu.gamma * (double)gn);
  }
}

// ---------------------------------------------------------------------------
// logistic gradient, Section 6, of features too long for the one-launch form (grad.hip):
//   grad f_i(x) = -(1/N_i) sum_l y_l a_l / (1 + exp(y_l a_l^T x)) + 2 lambda x_j / (1 + x_j^2)^2
// margins: LPR lanes per sample (64, or 16 for rows shorter than 1024 so that a wavefront works on four
//          rows at once) compute a_l^T x in fp64 and s_l = -y_l/(1+exp(y_l z_l))/N_i.
// cols   : a block owns 64 column groups (4 columns each on the 16-byte path) and a chunk of the shard's
//          rows; its four wavefronts take every fourth row, sum s_l a_l in fp64, and the four partial
//          sums are added in wavefront order.  Shards of more than 256 rows are shared by several
//          blocks; the one that finishes last adds their sums in chunk order.
// ---------------------------------------------------------------------------
template <int LPR, bool VEC>
__global__ __launch_bounds__(kBlock) void k_grad_margins(LogisticData ld, const float* __restrict__ x, int64_t d) {
  const int64_t l = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / LPR;
  const int sub = threadIdx.x % LPR;
  const bool live = l < ld.rows;
  const float* __restrict__ a = ld.A + (size_t)(live ? l : 0) * d;
  const int64_t dd = live ? d : 0;
  double acc0 = 0.0, acc1 = 0.0;
  if (VEC) {
#pragma unroll 4
    for (int64_t j = (int64_t)sub * 4; j < dd; j += LPR * 4) {
      const float4 av = *reinterpret_cast<const float4*>(a + j);
      const float4 xv = *reinterpret_cast<const float4*>(x + j);
      acc0 = fma((double)av.x, (double)xv.x, acc0);
      acc1 = fma((double)av.y, (double)xv.y, acc1);
      acc0 = fma((double)av.z, (double)xv.z, acc0);
      acc1 = fma((double)av.w, (double)xv.w, acc1);
    }
  } else {
#pragma unroll 4
    for (int64_t j = sub; j < dd; j += LPR) acc0 = fma((double)a[j], (double)x[j], acc0);
  }
  double z = acc0 + acc1;
#pragma unroll
  for (int o = LPR >> 1; o > 0; o >>= 1) z += __shfl_xor(z, o);
  if (live && sub == 0) {
    const int node = ld.row_node[l];
    const double N = (double)(ld.offsets[node + 1] - ld.offsets[node]);
    const double yl = (double)ld.labels[l];
    ld.margins[l] = -yl / (1.0 + exp(yl * z)) / N;
  }
}

template <bool VEC>
__global__ __launch_bounds__(kBlock) void k_grad_cols(LogisticData ld, const float* __restrict__ x,
                                                       float* __restrict__ grads, int64_t d, int rows_per_chunk) {
  constexpr int CPL = VEC ? 4 : 1;                 // columns per lane
  __shared__ double part[4][64 * CPL];
  __shared__ int s_flag;
  const int node = blockIdx.z, rc = blockIdx.y, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t j0 = ((int64_t)blockIdx.x * 64 + lane) * CPL;
  const bool live = j0 < d;
  const int64_t r_begin = ld.offsets[node] + (int64_t)rc * rows_per_chunk;
  const int64_t r_end = min(ld.offsets[node + 1], r_begin + rows_per_chunk);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (live) {
    const float* __restrict__ a = ld.A + (size_t)(r_begin + w) * d + j0;
#pragma unroll 4
    for (int64_t l = r_begin + w; l < r_end; l += 4, a += 4 * d) {
      const double s = ld.margins[l];
      if (VEC) {
        const float4 av = *reinterpret_cast<const float4*>(a);
        acc[0] = fma(s, (double)av.x, acc[0]);
        acc[1] = fma(s, (double)av.y, acc[1]);
        acc[2] = fma(s, (double)av.z, acc[2]);
        acc[3] = fma(s, (double)av.w, acc[3]);
      } else {
        acc[0] = fma(s, (double)a[0], acc[0]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < CPL; ++c) part[w][lane * CPL + c] = acc[c];
  __syncthreads();
  double t[4];
#pragma unroll
  for (int c = 0; c < CPL; ++c)
    t[c] = ((part[0][lane * CPL + c] + part[1][lane * CPL + c]) + part[2][lane * CPL + c]) + part[3][lane * CPL + c];
  if (ld.row_chunks > 1) {
    // several blocks share the shard's rows: each leaves its sums, the last to arrive adds them in chunk order
    if (w == 0 && live) {
#pragma unroll
      for (int c = 0; c < CPL; ++c) st_coherent(&ld.part[((size_t)node * ld.row_chunks + rc) * d + j0 + c], t[c]);
    }
    if (!arrive_last_few(&ld.col_done[(size_t)node * gridDim.x + blockIdx.x], (uint32_t)ld.row_chunks, &s_flag)) return;
#pragma unroll
    for (int c = 0; c < CPL; ++c) t[c] = 0.0;
    if (w == 0 && live) {
      for (int r0 = 0; r0 < ld.row_chunks; r0 += 8) {        // eight chunks' loads in flight, added in chunk order
        double v[8][4];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int c = 0; c < CPL; ++c)
            v[u][c] = r0 + u < ld.row_chunks ? ld_coherent(&ld.part[((size_t)node * ld.row_chunks + r0 + u) * d + j0 + c]) : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int c = 0; c < CPL; ++c) t[c] += v[u][c];
      }
    }
  }
  if (w != 0 || !live) return;
#pragma unroll
  for (int c = 0; c < CPL; ++c) grads[(size_t)node * d + j0 + c] = (float)(t[c] + reg_grad(ld.lambda, (double)x[j0 + c]));
}

// ---------------------------------------------------------------------------
// The same gradient for sparse features (rows in CSR form, and per worker by column).
// margins: LPR lanes per row (a power of two) sum the row's stored entries in fp64.
// cols   : 1, 16 or 64 lanes per (worker, column) sum s_l a_lj over the column's entries of that
//          worker's shard in a fixed order, then add the regulariser and round once.
// ---------------------------------------------------------------------------
template <int LPR>
__global__ __launch_bounds__(kBlock) void k_csr_margins(LogisticData ld, const float* __restrict__ x) {
  const int64_t l = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / LPR;
  const int sub = threadIdx.x % LPR;
  const bool live = l < ld.rows;
  const int64_t b = live ? ld.rp[l] : 0, e = live ? ld.rp[l + 1] : 0;
  double acc = 0.0;
  int64_t k = b + sub;
  for (; k + 3 * LPR < e; k += 4 * LPR) {          // four entries at a time: their gathers overlap
    int32_t c[4];
    float a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      c[u] = ld.ci[k + u * LPR];
      a[u] = ld.binary ? 1.f : ld.cv[k + u * LPR];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = fma((double)a[u], (double)x[c[u]], acc);
  }
  for (; k < e; k += LPR) {
    const double a = ld.binary ? 1.0 : (double)ld.cv[k];
    acc = fma(a, (double)x[ld.ci[k]], acc);
  }
#pragma unroll
  for (int o = LPR >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (live && sub == 0) {
    const int node = ld.row_node[l];
    const double N = (double)(ld.offsets[node + 1] - ld.offsets[node]);
    const double yl = (double)ld.labels[l];
    ld.margins[l] = -yl / (1.0 + exp(yl * acc)) / N;
  }
}

template <int LPC>   // lanes per column, a power of two: long columns are shared by 16 or 64 lanes
__global__ __launch_bounds__(kBlock) void k_csr_cols(LogisticData ld, const float* __restrict__ x,
                                                      float* __restrict__ grads, int64_t d) {
  const int node = blockIdx.y;
  const int64_t j = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / LPC;
  const int sub = threadIdx.x % LPC;
  const bool live = j < d;
  const uint32_t* __restrict__ cp = ld.cptr + (size_t)node * (size_t)(d + 1);
  const int64_t w0 = ld.wbase[node];
  const int64_t b = live ? w0 + cp[j] : 0, e = live ? w0 + cp[j + 1] : 0;
  double acc = 0.0;
  for (int64_t k = b + sub; k < e; k += LPC) {
    const double a = ld.binary ? 1.0 : (double)ld.tval[k];
    acc = fma(ld.margins[ld.trow[k]], a, acc);
  }
#pragma unroll
  for (int o = LPC >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (live && sub == 0) grads[(size_t)node * d + j] = (float)(acc + reg_grad(ld.lambda, (double)x[j]));
}

// Short columns (a few entries per worker-column): one thread owns four columns, 64 apart, and walks
// them side by side, so that four independent chains of gathers (row of the entry, then its margin)
// are in flight instead of one.  Same order of summation per column as k_csr_cols<1>.
template <bool BINARY>
__global__ __launch_bounds__(kBlock) void k_csr_cols4(LogisticData ld, const float* __restrict__ x,
                                                       float* __restrict__ grads, int64_t d) {
  const int node = blockIdx.y, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t j0 = ((int64_t)blockIdx.x * 4 + w) * 256 + lane;      // columns j0, j0+64, j0+128, j0+192
  const uint32_t* __restrict__ cp = ld.cptr + (size_t)node * (size_t)(d + 1);
  const int32_t* __restrict__ trow = ld.trow + ld.wbase[node];
  const float* __restrict__ tval = BINARY ? nullptr : ld.tval + ld.wbase[node];
  uint32_t b[4], e[4];
  double acc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int64_t j = j0 + 64 * c;
    const bool live = j < d;
    b[c] = live ? cp[j] : 0u;
    e[c] = live ? cp[j + 1] : 0u;
    acc[c] = 0.0;
  }
  uint32_t longest = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) longest = max(longest, e[c] - b[c]);
  // (62 us instead of 92 for 200 workers x 64000 entries x 65536 columns.  kDeep entries of every column at a time: entry
  // after entry, the longest of the wavefront's 256 columns -- five entries where the mean is one -- makes it wait for as
  // many pairs of dependent gathers)
  constexpr int kDeep = 4;
  for (uint32_t t = 0; t < longest; t += kDeep) {
    int32_t r[kDeep][4];
    float a[kDeep][4];
    double m[kDeep][4];
#pragma unroll
    for (int u = 0; u < kDeep; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const bool on = t + u < e[c] - b[c];
        r[u][c] = on ? trow[b[c] + t + u] : -1;
        a[u][c] = (on && !BINARY) ? tval[b[c] + t + u] : 1.f;
      }
#pragma unroll
    for (int u = 0; u < kDeep; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) m[u][c] = r[u][c] >= 0 ? ld.margins[r[u][c]] : 0.0;
#pragma unroll
    for (int u = 0; u < kDeep; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (r[u][c] >= 0) acc[c] = fma(m[u][c], (double)a[u][c], acc[c]);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int64_t j = j0 + 64 * c;
    if (j < d) grads[(size_t)node * d + j] = (float)(acc[c] + reg_grad(ld.lambda, (double)x[j]));
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned blocks_for(size_t count, unsigned cap = 65535u * 16u) {
  size_t b = (count + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  return (unsigned)(b > cap ? cap : b);
}

hipError_t launch_xupdate(float* out, const float* x, const float* g, double gamma, int64_t d, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  hipLaunchKernelGGL(k_xupdate, dim3((unsigned)((d + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, out, x, g, gamma, d);
  return hipGetLastError();
}

hipError_t launch_mean(const float* gi, float* o0, float* o1, float* o2, int n, int64_t d, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  hipLaunchKernelGGL(k_mean, dim3((unsigned)((d + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, gi, o0, o1, o2, n, d);
  return hipGetLastError();
}

hipError_t launch_aggregate(const NodeSet& ws, const float* gt_old, float* gt_new, const IterateUpdate& xu,
                            bool from_dense, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  if (from_dense) {
    hipLaunchKernelGGL(k_aggregate_short, dim3((unsigned)((ws.d + 63) / 64)), dim3(64), 0, st, ws, gt_old, gt_new, xu);
    return hipGetLastError();
  }
  if (ws.lv.nq == 0 && ws.lv.nr == 0) {
    if (ws.nn <= kOrderedMax)
      hipLaunchKernelGGL(k_aggregate_ordered, dim3(ws.groups), dim3(kBlock), 0, st, ws, gt_old, gt_new, xu);
    else
      hipLaunchKernelGGL((k_aggregate<false>), dim3(ws.groups, ws.AS), dim3(kBlock), 0, st, ws, gt_old, gt_new, xu);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_aggregate<true>), dim3(ws.groups, ws.AS), dim3(kBlock), 0, st, ws, gt_old, gt_new, IterateUpdate{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_aggregate_dense, dim3((unsigned)((ws.d + kDenseCols - 1) / kDenseCols)), dim3(64 * kDenseWaves), 0, st, ws,
                     gt_old, gt_new, xu);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, size_t count, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(count, 4096)), dim3(kBlock), 0, st, p, v, count);
  return hipGetLastError();
}

hipError_t launch_copy_f32(float* dst, const float* src, size_t count, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_f32, dim3(blocks_for(count, 8192)), dim3(kBlock), 0, st, dst, src, count);
  return hipGetLastError();
}

hipError_t launch_grad_margins(const LogisticData& ld, const float* x, int64_t d, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  if (ld.csr) {
    const int64_t per_row = ld.nnz / (ld.rows > 0 ? ld.rows : 1);
    const int lpr = per_row >= 128 ? 64 : per_row >= 16 ? 16 : 4;
    const unsigned grid = (unsigned)((ld.rows * lpr + kBlock - 1) / kBlock);
    if (lpr == 64) hipLaunchKernelGGL((k_csr_margins<64>), dim3(grid), dim3(kBlock), 0, st, ld, x);
    else if (lpr == 16) hipLaunchKernelGGL((k_csr_margins<16>), dim3(grid), dim3(kBlock), 0, st, ld, x);
    else hipLaunchKernelGGL((k_csr_margins<4>), dim3(grid), dim3(kBlock), 0, st, ld, x);
    return hipGetLastError();
  }
  const bool vec = (d % 4 == 0) && ((reinterpret_cast<uintptr_t>(ld.A) & 15u) == 0) &&
                   ((reinterpret_cast<uintptr_t>(x) & 15u) == 0);
  const int lpr = d >= 1024 ? 64 : 16;
  const dim3 grid((unsigned)((ld.rows * lpr + kBlock - 1) / kBlock));
  if (lpr == 64) {
    if (vec) hipLaunchKernelGGL((k_grad_margins<64, true>), grid, dim3(kBlock), 0, st, ld, x, d);
    else hipLaunchKernelGGL((k_grad_margins<64, false>), grid, dim3(kBlock), 0, st, ld, x, d);
  } else {
    if (vec) hipLaunchKernelGGL((k_grad_margins<16, true>), grid, dim3(kBlock), 0, st, ld, x, d);
    else hipLaunchKernelGGL((k_grad_margins<16, false>), grid, dim3(kBlock), 0, st, ld, x, d);
  }
  return hipGetLastError();
}

hipError_t launch_grad_cols(const LogisticData& ld, const float* x, float* grads, int n, int64_t d, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  if (ld.csr) {
    const int64_t per_col = ld.nnz / ((int64_t)n * d);
    const int lpc = per_col >= 256 ? 64 : per_col >= 16 ? 16 : 1;
    const dim3 grid((unsigned)((d * lpc + kBlock - 1) / kBlock), n);
    if (lpc == 64) hipLaunchKernelGGL((k_csr_cols<64>), grid, dim3(kBlock), 0, st, ld, x, grads, d);
    else if (lpc == 16) hipLaunchKernelGGL((k_csr_cols<16>), grid, dim3(kBlock), 0, st, ld, x, grads, d);
    else if (ld.binary) hipLaunchKernelGGL((k_csr_cols4<true>), dim3((unsigned)((d + 1023) / 1024), n), dim3(kBlock), 0, st, ld, x, grads, d);
    else hipLaunchKernelGGL((k_csr_cols4<false>), dim3((unsigned)((d + 1023) / 1024), n), dim3(kBlock), 0, st, ld, x, grads, d);
    return hipGetLastError();
  }
  const bool vec = (d % 4 == 0) && ((reinterpret_cast<uintptr_t>(ld.A) & 15u) == 0);
  const int rpc = (int)((ld.max_rows + ld.row_chunks - 1) / ld.row_chunks);
  const int64_t cols_per_block = 64 * (vec ? 4 : 1);
  const dim3 grid((unsigned)((d + cols_per_block - 1) / cols_per_block), ld.row_chunks, n);
  if (vec) hipLaunchKernelGGL((k_grad_cols<true>), grid, dim3(kBlock), 0, st, ld, x, grads, d, rpc);
  else hipLaunchKernelGGL((k_grad_cols<false>), grid, dim3(kBlock), 0, st, ld, x, grads, d, rpc);
  return hipGetLastError();
}

}  // namespace adacgd
