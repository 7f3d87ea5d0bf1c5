// The whole compression step of a node in one launch, for level sets without Rank-K levels: difference and
// norms, exact multi-level Top-K selection, realised error of every level, the cascade, the message and
// h <- h + C_j(x - h).
//
// A node's vector is cut into NB chunks of up to NT * VPT coordinates, one block each.  The chunk is read once and
// stays in registers (v and the estimator), so everything after the read is free of memory traffic.  With NB = 1
// nothing leaves the block: what bounds the launch are its dependent phases (a phase is a pass over the registers or a
// few LDS round trips, 0.3 - 1 us).  With NB > 1 the node's blocks meet a few times: each adds its histogram, or leaves its
// partial results, waits until all NB have done so, and reads the totals; every block then takes the same
// decisions from the same numbers.
//
// Meeting.  What the blocks leave for each other is polled itself, there is no counter: a histogram (of the second and
// third digit) is complete when its counts add up to the number of keys that go into it, which every block knows,
// and a partial result (never negative) is stored negated, so that it differs from the zero that was there before.
// A meeting is then one atomic or store on its way to memory and one load coming back.
// Waiting.  A block only waits for blocks of its own node.  Blocks take their (node, chunk) by an atomic ticket, so that the
// blocks of a node begin together whatever the order of dispatch (a launch of no more than kNodeParts blocks goes without).
// That they are running all at once cannot be relied on: other launches, of other contexts on other streams or of other
// processes, may have filled the device with blocks that wait themselves.  So a block counts itself in its node's word as
// it begins, and the first meeting also waits for that word: where it is not complete after some time the node is given
// up, its blocks leave, and the last of them to come does the node alone, from memory.  After the first meeting all blocks
// of the node are running, and what they wait for comes.
// What is polled exists twice: a launch uses one set and clears the other, which the previous launch of the node
// set has left behind (launches of a node set are ordered on a stream).
// Measured, per launch, against the general sequence of select.hip (sum of its kernels): Top-K sets, 8 nodes of 20000
// coordinates 20 us (55), 10 of 5003 14 us (95), one node of 2^20 (a master) 36 us (75), 8 of 1000003 45 us (100);
// 200 nodes of 65536 109 us (170); 1000 of 65536 with quantisers 439 us (595).
#include "devutil.h"
#include "engine.h"
#include "quant.h"

namespace adacgd {

// Reads one word of every 64 bytes of a kernel argument, all at once: fetched line by line where they are used,
// the argument structures would cost several round trips to memory on the way (about 1 us each).
template <typename T>
__device__ __forceinline__ void prefetch_args(const T& t) {
  const uint32_t* w = reinterpret_cast<const uint32_t*>(&t);
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 4; i += 16) asm volatile("" ::"s"(w[i]));
}

// Sum over the NW (a power of two up to 16) per-wavefront partial results in LDS, the same in every lane.
template <int NW, typename T>
__device__ __forceinline__ T waves_sum(const T* r, uint32_t lane) {
  return lane_value(row_scan(r[lane & (NW - 1)]), NW - 1);
}
// Likewise for counts; *before gets the sum over the wavefronts below w.
template <int NW>
__device__ __forceinline__ uint32_t waves_sum(const uint32_t* r, uint32_t lane, int w, uint32_t* before) {
  const uint32_t v = r[lane & (NW - 1)], inc = row_scan(v);
  *before = lane_value(inc - v, w);
  return lane_value(inc, NW - 1);
}

// Of PER bins that hold `sum` counts in all: finds, from the top, the one where the running count reaches `left`
// (nothing happens unless 1 <= left <= sum).  The bins are read again: keeping them would cost registers.
template <int PER>
__device__ __forceinline__ void find_bin(const uint32_t* bins, int base, uint32_t left, uint32_t sum, uint32_t* out) {
  if (left - 1u < sum) {
    uint32_t bin = 0, rank = 0, cnt = 0;
#pragma unroll 1
    for (int q0 = PER - 4; q0 >= 0; q0 -= 4) {
      const uint4 c4 = *reinterpret_cast<const uint4*>(bins + q0);
      const uint32_t c[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        const bool here = left - 1u < c[q];              // (after the bin is found, left is zero or has wrapped around)
        bin = here ? (uint32_t)(base + q0 + q) : bin;
        rank = here ? left : rank;
        cnt = here ? c[q] : cnt;
        left -= c[q];
      }
    }
    out[0] = bin;
    out[1] = rank;
    out[2] = cnt;
  }
}

// One wavefront walks an NB-bin histogram in LDS from its top bin down to the bin where the running count
// reaches `rank`: out = {bin, rank inside the bin, count of the bin} (untouched if the counts do not reach it).
template <int NB>
__device__ __forceinline__ void wave_walk(const uint32_t* hist, uint32_t rank, uint32_t* out) {
  constexpr int PER = NB / 64;
  const int base = NB - ((int)(threadIdx.x & 63) + 1) * PER;
  uint32_t sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) sum += hist[base + q];
  find_bin<PER>(hist + base, base, rank - (wave_scan(sum) - sum), sum, out);
}

// Exclusive scan, in place, of `n` <= 256 counts by one wavefront.
__device__ __forceinline__ void wave_scan_table(uint32_t* t, int n, uint32_t lane) {
  uint32_t v[4], sum = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) { v[q] = (int)lane * 4 + q < n ? t[lane * 4 + q] : 0u; sum += v[q]; }
  uint32_t cum = wave_scan(sum) - sum;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if ((int)lane * 4 + q < n) t[lane * 4 + q] = cum;
    cum += v[q];
  }
}

__device__ __forceinline__ uint32_t hist_slot(uint32_t bin) { return ((bin & 31u) << 7) | (bin >> 5); }
__device__ __forceinline__ uint32_t hist_bin(uint32_t slot) { return ((slot & 127u) << 5) | (slot >> 7); }

constexpr int kBatch = 4;            // Top-K sizes whose second and third digits are resolved side by side
constexpr int kErrBatch = 3;         // quantiser levels evaluated in one pass over the values

// Quad q of thread t is coordinates 4 (q NT + t) .. + 3 of the chunk, so that a wavefront's 16-byte accesses are
// contiguous and (q, wavefront, lane, component) is ascending coordinate.  Values beyond the chunk's end are +0 and
// never matter: they add nothing to a sum, zeros are not counted in a histogram, and they are not sent.
// CAP: candidates (values that can belong to the largest Top-K set below the identity) that fit the list in LDS;
// with more of them the passes over the candidates run over the registers instead.
// MULTI: several blocks per node.
template <int NT, int VPT, int CAP, bool QUANT, bool MULTI>
__global__ __launch_bounds__(NT, NT >= 512 ? 4 : 1) void k_node(NodeSet ns, PassArgs a) {
  constexpr int NQ4 = VPT / 4, NW = NT / 64;
  static_assert(!MULTI || CAP >= 2 * kMaxLevels * kNodeParts, "the counts of the node's blocks fit the list");
  extern __shared__ __align__(16) uint32_t dyn[];
  uint32_t* const hist = dyn;              // 4096 words: first digit; then kBatch histograms of 1024 or 512 bins
  uint32_t* const list = dyn + kBins0;     // CAP words: block scales of quantisers; keys of the candidates; counts of the node's blocks
  __shared__ double red[4][NW];            // per wavefront: S, D, energy below the candidates; quantiser errors
  __shared__ double redb[kBatch][NW];      // ... energy below the thresholds
  __shared__ uint32_t redu[3][NW], redc[2][kBatch][NW];
  __shared__ uint32_t s_K[kMaxLevels], s_T[kMaxLevels], s_r[kMaxLevels], s_eq[kMaxLevels];   // per Top-K size: threshold key, ties to take, keys equal to it
  __shared__ uint32_t s_cnt[2][kMaxLevels];          // ... this block's keys above and equal to the threshold
  __shared__ double s_fin[1 + 2 * kMaxLevels];       // energy below the candidates, below every threshold; quantiser errors
  __shared__ double s_first[4];
  __shared__ uint32_t s_walk[kMaxLevels][3];
  __shared__ uint32_t s_tab[NQ4 * NW + 1]; // message offset of every (quad, wavefront)
  __shared__ uint32_t s_teq[NQ4 * NW];
  __shared__ uint32_t segk[QUANT ? NT * VPT / kSeg : 1];      // largest key of every 64-coordinate segment
  __shared__ int s_kind[kMaxLevels], s_ref[kMaxLevels];
  __shared__ double s_tz[kMaxLevels + 1], s_te[kMaxLevels + 1];
  __shared__ uint32_t s_blk;
  __shared__ uint32_t s_fill[kBatch];
  __shared__ int s_flag, s_quit;

  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lane = tid & 63;
  prefetch_args(ns);
  prefetch_args(a);
  const int NB = MULTI ? ns.NB : 1;
  const LevelTable& lv = ns.lv;
  const int nq = lv.nq, pk = lv.pk;
  const uint32_t d = (uint32_t)ns.d;
  uint32_t blk = blockIdx.x;
  if (MULTI && ns.ticket) {
    if (tid == 0) s_blk = __hip_atomic_fetch_add(&ns.ticket[a.parity * kCounterStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    blk = __builtin_amdgcn_readfirstlane(s_blk);
  }
  const int node = (int)(blk / (uint32_t)NB), part = (int)(blk % (uint32_t)NB);
  const uint32_t c0 = (uint32_t)part * (uint32_t)ns.chunk;           // first coordinate of the chunk
  const uint32_t len = min((uint32_t)ns.chunk, d - c0);
  const size_t row = (size_t)node * d + c0;
  const bool diff = a.diff != 0;
  const Buf xb = make_buf(a.x + row, 4 * len), hb = make_buf(a.h + row, 4 * len);
  auto quad_at = [&](int q) { return (uint32_t)(q * NT + tid) * 4u; };     // its first coordinate in the chunk
  const uint32_t off0 = (uint32_t)tid * 16u;                                // byte offset of quad 0; quad q: + 16 q NT

  // where the node's blocks meet: histograms of the three digits, partial results [quantity][block]
  uint32_t *begun = nullptr, *gh1 = nullptr, *gh2 = nullptr, *gh3 = nullptr;
  double *part1 = nullptr, *part2 = nullptr;
  if (MULTI) {
    const size_t words = node_meet_words(pk, nq, NB);
    begun = ns.meet + ((size_t)a.parity * ns.nn + node) * words;
    part1 = reinterpret_cast<double*>(begun + kCounterStride);
    if (tid == 0) {
      atomicAdd(begun, 1u);
      s_quit = 0;
    }
    part2 = part1 + 4 * NB;
    gh1 = reinterpret_cast<uint32_t*>(part1 + node_part_quantities(pk, nq) * NB);
    gh2 = gh1 + kBins0;
    gh3 = gh2 + (size_t)pk * kBins1;
    // the set the previous launch used, cleared for the next one
    uint32_t* old = ns.meet + ((size_t)(a.parity ^ 1) * ns.nn + node) * words;
    for (uint32_t i = (uint32_t)part * NT + tid; i < (uint32_t)words; i += (uint32_t)NB * NT) old[i] = 0;
    if (ns.ticket && blk == 0 && tid == 0) ns.ticket[(a.parity ^ 1) * kCounterStride] = 0;
  }
  // A histogram of nw words that the node's blocks add their counts to: adds this block's (in LDS), waits until all
  // counts are there -- they add up to `total` -- and leaves them in LDS.
  auto meet_hist = [&](uint32_t* g, int nw, uint32_t total) {
    for (int b = tid; b < nw; b += NT) {
      const uint32_t c = hist[b];
      if (c) atomicAdd(&g[b], c);
    }
    for (;;) {
      uint32_t sum = 0;
      __syncthreads();
      for (int i = tid * 2; i < nw; i += NT * 2) {
        const uint64_t two = ld_coherent(reinterpret_cast<const uint64_t*>(g + i));
        *reinterpret_cast<uint64_t*>(&hist[i]) = two;
        sum += (uint32_t)two + (uint32_t)(two >> 32);
      }
      sum = wave_total(sum);
      if (lane == 0) redc[0][0][w] = sum;
      __syncthreads();
      if (waves_sum<NW>(redc[0][0], lane) == total) break;
    }
  };
  auto none = [](double t) { return t == 0.0 && !(__double2hiint(t) < 0); };
  // One partial result of every block of the node, lane by lane (zero beyond them), once it is there.
  auto meet_value = [&](const double* p) {
    double t = -0.0;
    if ((int)lane < NB) {
      do t = ld_coherent(p + lane); while (none(t));
    }
    return -t;
  };
  // The same at the first meeting (wavefronts leave the loop as one; wavefront 0 finds out whether the node is complete).
  auto meet_first = [&](const double* p) {
    double t = (int)lane < NB ? 0.0 : -0.0;
    uint32_t there = w == 0 ? 0u : (uint32_t)NB;
    for (uint32_t polls = 0;; ++polls) {
      if (none(t)) t = ld_coherent(p + lane);
      if (there != (uint32_t)NB) there = poll_begun(begun, (uint32_t)NB, polls >= ns.polls);
      if (there & kGivenUp) {
        if (lane == 0) __hip_atomic_store(&s_quit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        break;
      }
      if (there == (uint32_t)NB && !ballot(none(t))) break;
      if (w != 0 && __hip_atomic_load(&s_quit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
    }
    return -t;
  };

  // what is needed of the level set later on, here, so that no memory latency is left when it is
  if (tid < kMaxLevels) {
    s_K[tid] = lv.K[tid];
    s_kind[tid] = lv.kind[tid];
    s_ref[tid] = lv.ref[tid];
    s_tz[tid] = lv.tz[tid];
    s_te[tid] = lv.te[tid];
  }

  // ---- the cascade (every wavefront for itself, lane j the level j + 1); the node's results by one wavefront of `writer` ----
  auto choose = [&](double S, double Dn, bool skip, bool writer, int* slot_out, int* q_out) {
    double my_err = __longlong_as_double(0x7FF8000000000000ll);      // not evaluated on a skip
    bool hit = false;
    if (!skip && (int)lane < lv.m) {
      const int ref = s_ref[lane];
      if (s_kind[lane] != kTopK) {
        my_err = s_fin[1 + kMaxLevels + ref];
      } else if (ref >= pk) {                // the identity
        my_err = 0.0;
      } else {
        const double tv = (double)__uint_as_float(s_T[ref]);
        my_err = s_fin[0] + s_fin[1 + ref] + (double)(s_eq[ref] - s_r[ref]) * (tv * tv);    // (ties not taken)
      }
      hit = (int)lane + 1 < lv.m && my_err <= __dadd_rn(__dmul_rn(s_tz[lane + 1], Dn), __dmul_rn(s_te[lane + 1], S));
    }
    const uint64_t good = ballot(hit);
    const int jstar = skip ? 0 : good ? __ffsll((unsigned long long)good) : lv.m;
    int slot = -1, q_sel = -1;
    if (jstar > 0) {
      const int ref = __builtin_amdgcn_readfirstlane(s_ref[jstar - 1]);
      if (__builtin_amdgcn_readfirstlane(s_kind[jstar - 1]) == kTopK) slot = ref;
      else q_sel = ref;
    }
    if (w == 0 && writer) {
      if ((int)lane < lv.m) ns.err[node * lv.m + lane] = my_err;
      if (lane == 0) {
        ns.S[node] = S;
        ns.D[node] = Dn;
        ns.level[node] = jstar;
        atomicAdd(&ns.level_hist[jstar], 1ull);
        ns.sel_slot[node] = slot;
        ns.sel_q[node] = q_sel;
        ns.msg_count[node] = slot >= 0 ? s_K[slot] : 0u;
        if (nq > 0) ns.qscale[node] = 0.f;
      }
    }
    *slot_out = slot;
    *q_out = q_sel;
  };

  // ---- a whole node by one block, for one that was given up (NB > 1): the vector is read again for every digit and level ----
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  const uint32_t ctr1 = (uint32_t)node | a.node_flag;
  auto alone = [&] {
    constexpr uint32_t STEP = NT * 4;        // coordinates a pass of the block: four a thread, in order
    static_assert(!MULTI || STEP == kWaveTile, "message offsets are kept for every kWaveTile coordinates");
    const size_t start = (size_t)node * d;
    const Buf xn = make_buf(a.x + start, 4 * d), hn = make_buf(a.h + start, 4 * d), yn = make_buf(diff ? nullptr : a.y + start, diff ? 0u : 4 * d);
    auto load = [&](uint32_t l0, float (&vq)[4], float (&hq)[4]) {       // (zero beyond the end)
      float xq[4];
      buf_load4(xn, 4 * l0, 0, xq);
      buf_load4(hn, 4 * l0, 0, hq);
#pragma unroll
      for (int c = 0; c < 4; ++c) vq[c] = diff ? xq[c] : xq[c] - hq[c];
    };
    auto total = [&](double e) {
      e = wave_total(e);
      __syncthreads();
      if (lane == 0) red[0][w] = e;
      __syncthreads();
      return waves_sum<NW>(red[0], lane);
    };
    auto scan = [&](uint32_t n, uint32_t* sum) {       // exclusive, in thread order
      const uint32_t inc = wave_scan(n);
      __syncthreads();
      if (lane == 63) redu[0][w] = inc;
      __syncthreads();
      uint32_t before;
      *sum = waves_sum<NW>(redu[0], lane, w, &before);
      return before + inc - n;
    };
    auto block_scale = [&](const float (&vq)[4], int B) {       // largest magnitude of the quantiser block of these coordinates
      uint32_t m = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) m = max(m, magkey(vq[c]));
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) m = max(m, (uint32_t)__shfl_xor(m, o, 64));
      __syncthreads();
      if ((lane & 15) == 0) segk[tid / 16] = m;
      __syncthreads();
      const int per = B / kSeg, first = tid / 16 / per * per;
      m = 0;
      for (int j = 0; j < per; ++j) m = max(m, segk[first + j]);
      return __uint_as_float(m);
    };
    double S = 0.0, D = 0.0;
    uint32_t kmax = 0, nonzero = 0;
#pragma unroll 1
    for (uint32_t l0 = tid * 4; l0 < d; l0 += STEP) {
      float vq[4], hq[4], xq[4], yq[4];
      load(l0, vq, hq);
      buf_load4(xn, 4 * l0, 0, xq);
      buf_load4(yn, 4 * l0, 0, yq);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        S = fma((double)vq[c], (double)vq[c], S);
        const double dw = (double)(xq[c] - yq[c]);
        D = fma(dw, dw, D);
        kmax = max(kmax, magkey(vq[c]));
        nonzero += magkey(vq[c]) ? 1u : 0u;
      }
    }
    S = total(S);
    D = total(D);
    scan(nonzero, &nonzero);
    kmax = wave_top(kmax);
    if (lane == 0) redu[1][w] = kmax;
    __syncthreads();
    kmax = wave_top(redu[1][lane & (NW - 1)]);
    const double Dn = diff ? a.extD[node] : D;
    const bool skip = !a.assign && S <= trigger_bound(lv, 0, S, Dn);
    const float qa = __uint_as_float(kmax);
    if (!skip) {
      if (tid == 0) s_fin[0] = 0.0;
#pragma unroll 1
      for (int s = 0; s < pk; ++s) {
        const uint32_t K = lane_value(s_K[s], 0);
        uint32_t T = 0, r = K - nonzero, eq = d - nonzero;       // a size that the non-zero keys do not reach: threshold zero
        if (K <= nonzero) {
          r = K;
#pragma unroll 1
          for (int digit = 0; digit < 3; ++digit) {
            const int above = digit == 0 ? 31 : digit == 1 ? kShift0 : kShift1, at = digit == 0 ? kShift0 : digit == 1 ? kShift1 : 0;
            const int bins = digit == 0 ? kBins0 : digit == 1 ? kBins1 : kBins2;
            __syncthreads();
            for (int b = tid; b < kBins0; b += NT) hist[b] = 0;
            __syncthreads();
#pragma unroll 1
            for (uint32_t l0 = tid * 4; l0 < d; l0 += STEP) {
              float vq[4], hq[4];
              load(l0, vq, hq);
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                const uint32_t key = magkey(vq[c]);
                if (key && (key >> above) == T) atomicAdd(&hist[(key >> at) & (bins - 1)], 1u);
              }
            }
            __syncthreads();
            if (w == 0) wave_walk<kBins0>(hist, r, s_walk[0]);
            __syncthreads();
            T = T * bins + lane_value(s_walk[0][0], 0);
            r = lane_value(s_walk[0][1], 0);
            eq = lane_value(s_walk[0][2], 0);
          }
        }
        double e = 0.0;
#pragma unroll 1
        for (uint32_t l0 = tid * 4; l0 < d; l0 += STEP) {
          float vq[4], hq[4];
          load(l0, vq, hq);
#pragma unroll
          for (int c = 0; c < 4; ++c) e += magkey(vq[c]) < T ? (double)vq[c] * (double)vq[c] : 0.0;
        }
        e = total(e);
        if (tid == 0) { s_T[s] = T; s_r[s] = r; s_eq[s] = eq; s_fin[1 + s] = e; }
      }
      if (QUANT) {
#pragma unroll 1
        for (int q = 0; q < nq; ++q) {
          const int B = lv.qblock[q];
          double e = 0.0;
#pragma unroll 1
          for (uint32_t t0 = 0; t0 < d; t0 += STEP) {
            float vq[4], hq[4];
            load(t0 + tid * 4, vq, hq);
            const float aq = B ? block_scale(vq, B) : qa;
            const float cq = aq > 0.f ? (float)((double)aq / lv.qdenom[q]) : 0.f;
            uint32_t rnd[4];
            philox4x32_10((t0 >> 2) + tid, ctr1, a.step, 0u, k0, k1, rnd);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              float xi;
              const double er = (double)fabsf(vq[c]) - (double)quant_mag(aq > 0.f ? fabsf(vq[c]) / aq : 0.f, lv.qs[q], cq, dither_of(rnd[c]), &xi);
              e = fma(er, er, e);
            }
          }
          e = total(e);
          if (tid == 0) s_fin[1 + kMaxLevels + q] = e;
        }
      }
    }
    __syncthreads();
    int slot, q_sel;
    choose(S, Dn, skip, true, &slot, &q_sel);
    if (slot >= 0) {
      const bool ident = slot >= pk;
      const uint32_t T = ident ? 0u : lane_value(s_T[slot], 0), r = ident ? d : lane_value(s_r[slot], 0);
      uint32_t out = 0, ties = 0;          // entries, and keys equal to T, of the coordinates before these
      uint32_t* __restrict__ go = ns.grp_off + (size_t)node * (ns.groups + 1);
#pragma unroll 1
      for (uint32_t t0 = 0; t0 < d; t0 += STEP) {
        const uint32_t l0 = t0 + tid * 4;
        float vq[4], hq[4];
        load(l0, vq, hq);
        uint32_t n = 0, sum;
#pragma unroll
        for (int c = 0; c < 4; ++c) n += magkey(vq[c]) == T && l0 + c < d ? 1u : 0u;
        uint32_t rank = ties + scan(n, &sum), f = 0;
        ties += sum;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t key = magkey(vq[c]);
          if (l0 + c < d && (key > T || (key == T && rank < r))) f |= 1u << c;
          rank += key == T ? 1u : 0u;
        }
        if (tid == 0) go[t0 / STEP] = out;
        uint32_t pos = out + scan((uint32_t)__popc(f), &sum);
        out += sum;
        if (f) {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if ((f >> c) & 1u) {
              ns.msg_idx[(size_t)node * ns.Kcap + pos] = (int32_t)(l0 + c);
              ns.msg_val[(size_t)node * ns.Kcap + pos] = vq[c];
              ++pos;
              hq[c] = a.assign ? vq[c] : hq[c] + vq[c];
            }
          }
          buf_store4(hn, 4 * l0, 0, hq);
        }
      }
      if (tid == 0) go[ns.groups] = out;
    } else if (QUANT && q_sel >= 0) {
      const int B = lv.qblock[q_sel];
      const float qc = !B && qa > 0.f ? (float)((double)qa / lv.qdenom[q_sel]) : 0.f;
      if (tid == 0) ns.qscale[node] = qc;
#pragma unroll 1
      for (uint32_t t0 = 0; t0 < d; t0 += STEP) {
        const uint32_t l0 = t0 + tid * 4;
        float vq[4], hq[4];
        load(l0, vq, hq);
        const float aq = B ? block_scale(vq, B) : qa;
        const float cq = B ? (aq > 0.f ? (float)((double)aq / lv.qdenom[q_sel]) : 0.f) : qc;
        if (B && l0 < d && l0 % (uint32_t)B == 0) ns.qbscale[(size_t)node * ns.nseg + l0 / (uint32_t)B] = cq;
        uint32_t rnd[4];
        philox4x32_10(l0 >> 2, ctr1, a.step, 0u, k0, k1, rnd);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          int code = 0;
          hq[c] += aq > 0.f ? quant_one(vq[c], aq, lv.qs[q_sel], cq, dither_of(rnd[c]), &code) : 0.f;
          if (l0 + c < d) ns.qcodes[start + l0 + c] = (int16_t)code;
        }
        buf_store4(hn, 4 * l0, 0, hq);
      }
    }
    if (a.xu_out && node == 0) {
#pragma unroll 1
      for (uint32_t l0 = tid * 4; l0 < d; l0 += STEP) {        // (of what is read again, this thread's own stores)
        float hq[4], xq[4];
        buf_load4(hn, 4 * l0, 0, hq);
        buf_load4(make_buf(a.xu_x, 4 * d), 4 * l0, 0, xq);
#pragma unroll
        for (int c = 0; c < 4; ++c) xq[c] = (float)((double)xq[c] - a.xu_gamma * (double)hq[c]);
        buf_store4(make_buf(a.xu_out, 4 * d), 4 * l0, 0, xq);
      }
    }
  };

  // ---- read: v, ||v||^2, ||x - y||^2, largest key ----
  // (the estimator's first KH quads stay in registers, the rest is read again when it is updated)
  constexpr int KH = QUANT && VPT > 16 ? 3 : NQ4;
  float v[VPT], hv[4 * KH];
  auto h_quad = [&](int q, float (&o)[4]) {
    if (q < KH) {
#pragma unroll
      for (int c = 0; c < 4; ++c) o[c] = hv[q < KH ? q * 4 + c : 0];
    } else {
      buf_load4(hb, off0, q * NT * 16, o);
    }
  };
  auto keep_h = [&](int q, const float (&o)[4]) {
    if (q < KH) {
#pragma unroll
      for (int c = 0; c < 4; ++c) hv[q < KH ? q * 4 + c : 0] = o[c];
    }
  };
  // Magnitude keys are formed anew in every pass over v, with a mask the compiler cannot see through: it
  // would otherwise carry what it derived from v (keys, values widened to fp64) from pass to pass, several
  // registers per value, and spill.
  auto key_mask = [] {
    uint32_t m;
    asm volatile("s_mov_b32 %0, 0x7fffffff" : "=s"(m));
    return m;
  };
  double S = 0.0, D = 0.0;
  uint32_t kmax = 0;
  {
    const Buf yb = make_buf(diff ? nullptr : a.y + row, diff ? 0u : 4 * len);
    const Buf yc = make_buf(a.ycopy ? a.ycopy + row : nullptr, a.ycopy ? 4 * len : 0u);
    for (int b = tid * 4; b < kBins0; b += NT * 4) *reinterpret_cast<uint4*>(&hist[b]) = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < NQ4; ++q) {
      // (loads of a few quads in flight per thread; more would not fit the registers)
      if (q % (VPT > 16 ? (QUANT ? 2 : 3) : 4) == 0) { asm volatile("" ::: "memory"); __builtin_amdgcn_sched_barrier(0); }
      float xv[4], yv[4], hq[4];
      buf_load4<kStream>(xb, off0, q * NT * 16, xv);
      buf_load4(hb, off0, q * NT * 16, hq);
      buf_load4<kStream>(yb, off0, q * NT * 16, yv);
      buf_store4(yc, off0, q * NT * 16, xv);
      uint32_t km = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float vv = diff ? xv[c] : xv[c] - hq[c];
        v[q * 4 + c] = vv;
        const double dv = (double)vv;
        S = fma(dv, dv, S);
        const double dw = (double)(xv[c] - yv[c]);     // (not used in difference mode)
        D = fma(dw, dw, D);
        if (QUANT) km = max(km, magkey(vv));
      }
      keep_h(q, hq);
      if (QUANT) kmax = max(kmax, km);
    }
  }
  if (QUANT && lv.nqb > 0) {             // 16 lanes x 4 coordinates = one segment
    const uint32_t mask = key_mask();
#pragma unroll
    for (int q = 0; q < NQ4; ++q) {
      uint32_t km = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) km = max(km, fbits(v[q * 4 + c]) & mask);
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) km = max(km, (uint32_t)__shfl_xor(km, o, 64));
      segk[quad_at(q) / kSeg] = km;      // (the same from all 16 lanes)
    }
  }
  S = wave_total(S);
  D = wave_total(D);
  if (QUANT) kmax = wave_top(kmax);
  if (lane == 0) { red[0][w] = S; red[1][w] = D; if (QUANT) redu[0][w] = kmax; }
  if (tid < kMaxLevels) { s_walk[tid][0] = 0; s_walk[tid][1] = 0; s_walk[tid][2] = 0; s_cnt[0][tid] = s_cnt[1][tid] = 0; }
  __syncthreads();
  S = waves_sum<NW>(red[0], lane);
  D = waves_sum<NW>(red[1], lane);
  if (QUANT) kmax = wave_top(redu[0][lane & (NW - 1)]);
  auto first_digit = [&] {               // histogram of the first digit of every key but zero
    const uint32_t m1 = key_mask();
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const uint32_t key = fbits(v[i]) & m1;
      if (key) atomicAdd(&hist[key >> kShift0], 1u);
    }
    __syncthreads();
  };
  if (MULTI) {
    uint32_t zeros = 0;
    if (pk > 0) {
      first_digit();
      uint32_t sum = 0;
#pragma unroll
      for (int q = 0; q < kBins0 / NT; ++q) {
        const uint32_t c = hist[q * NT + tid];
        if (c) atomicAdd(&gh1[hist_slot((uint32_t)(q * NT + tid))], c);
        sum += c;
      }
      sum = wave_total(sum);
      if (lane == 0) redu[1][w] = sum;
      // (this histogram is large: it is read once, when the partial results say that everybody's counts are in)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      zeros = len - waves_sum<NW>(redu[1], lane);
    }
    if (tid == 0) {
      st_coherent(&part1[part], -S);
      st_coherent(&part1[NB + part], -D);
      if (QUANT) st_coherent(&part1[2 * NB + part], -(double)kmax);
      if (pk > 0) st_coherent(&part1[3 * NB + part], -(double)zeros);
    }
    if (w < 4 && (w < 2 || (w == 2 ? QUANT : pk > 0))) {
      const double t = meet_first(part1 + w * NB);
      const double s = w == 2 ? (double)wave_top((uint32_t)t) : wave_total(t);
      if (lane == 0) s_first[w] = s;
    }
    __syncthreads();
    if (__builtin_expect(s_quit, 0)) {
      if (arrive_last_few(&ns.alone[node], (uint32_t)NB, &s_flag)) alone();
      return;
    }
    if (pk > 0) {
      for (uint32_t i = tid * 2; i < (uint32_t)kBins0; i += NT * 2) {
        const uint64_t two = ld_coherent(reinterpret_cast<const uint64_t*>(gh1 + i));
        hist[hist_bin(i)] = (uint32_t)two;
        hist[hist_bin(i + 1)] = (uint32_t)(two >> 32);
      }
      __syncthreads();
    }
    S = lane_value(s_first[0], 0);
    D = lane_value(s_first[1], 0);
    if (QUANT) kmax = lane_value((uint32_t)s_first[2], 0);
  }
  const double Dn = diff ? a.extD[node] : D;
  // first condition of the cascade: nothing else is evaluated (the compressed start applies its level unconditionally)
  const bool skip = !a.assign && S <= trigger_bound(lv, 0, S, Dn);

  // ---- realised error of every quantiser level: those that share a scale together, kErrBatch at a time ----
  const float qa = __uint_as_float(kmax);
  // block-wise levels: per block of B coordinates its scale a (the maximum over its segments) and c of up to
  // kErrBatch levels
  constexpr int NSEG = NT * VPT / kSeg;
  static_assert((1 + kErrBatch) * NSEG <= CAP, "block tables fit the list");
  float* const blk_a = reinterpret_cast<float*>(list);
  float* const blk_c = blk_a + NSEG;
  auto block_scales = [&](int B, const double* qd, int cnt) {
    const int nblk = (int)((len + B - 1) / B), per = B / kSeg;
    for (int b = tid; b < nblk; b += NT) {
      uint32_t m = 0;
      for (int j = 0; j < per && (b * per + j) * kSeg < (int)len; ++j) m = max(m, segk[b * per + j]);
      const float am = __uint_as_float(m);
      blk_a[b] = am;
      for (int j = 0; j < cnt; ++j) blk_c[j * NSEG + b] = am > 0.f ? (float)((double)am / qd[j]) : 0.f;
    }
  };
  if (QUANT && !skip) {
    uint32_t todo = (1u << nq) - 1u;
    while (todo) {
      int qi[kErrBatch], cnt = 0;
      const int B = lv.qblock[__ffs(todo) - 1];
      for (int q = 0; q < nq && cnt < kErrBatch; ++q)
        if (((todo >> q) & 1u) && lv.qblock[q] == B) { qi[cnt++] = q; todo &= ~(1u << q); }
      for (int j = cnt; j < kErrBatch; ++j) qi[j] = qi[0];
      float qs[kErrBatch], qc[kErrBatch];
      double qd[kErrBatch], acc[kErrBatch];
#pragma unroll
      for (int j = 0; j < kErrBatch; ++j) {
        qs[j] = lv.qs[qi[j]];
        qd[j] = lv.qdenom[qi[j]];
        qc[j] = qa > 0.f ? (float)((double)qa / qd[j]) : 0.f;
        acc[j] = 0.0;
      }
      const int lb = B ? __ffs(B) - 1 : 0;
      const uint32_t m5 = key_mask();
      if (B) {
        __syncthreads();                     // (the previous group's table is no longer in use)
        block_scales(B, qd, kErrBatch);
        __syncthreads();
      }
#pragma unroll
      for (int q = 0; q < NQ4; ++q) {
        const uint32_t l0 = quad_at(q);
        __builtin_amdgcn_sched_barrier(0);       // (one Philox block at a time: interleaving them would spill)
        if ((uint32_t)(q * NT) * 4u < len) {     // (the same in every thread)
          uint32_t rnd[4];
          philox4x32_10((c0 + l0) >> 2, ctr1, a.step, 0u, k0, k1, rnd);
          float aq = qa, cq[kErrBatch];
#pragma unroll
          for (int j = 0; j < kErrBatch; ++j) cq[j] = qc[j];
          if (B) {
            const uint32_t b = l0 < len ? l0 >> lb : 0u;
            aq = blk_a[b];
#pragma unroll
            for (int j = 0; j < kErrBatch; ++j) cq[j] = blk_c[j * NSEG + b];
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float av = __uint_as_float(fbits(v[q * 4 + c]) & m5);
            const float u = dither_of(rnd[c]);
            const float t = aq > 0.f ? av / aq : 0.f;
#pragma unroll
            for (int j = 0; j < kErrBatch; ++j) {
              if (j < cnt) {
                float xi;
                const double e = (double)av - (double)quant_mag(t, qs[j], cq[j], u, &xi);
                acc[j] = fma(e, e, acc[j]);
              }
            }
          }
        }
      }
      __syncthreads();                       // (every wavefront has read what `red` held before)
#pragma unroll
      for (int j = 0; j < kErrBatch; ++j) {
        const double e = wave_total(acc[j]);
        if (lane == 0) red[j][w] = e;
      }
      __syncthreads();
      if (tid < cnt) {
        double e = 0.0;
#pragma unroll 4
        for (int i = 0; i < NW; ++i) e += red[tid][i];
        int q = qi[0];
#pragma unroll
        for (int j = 1; j < kErrBatch; ++j) q = j == tid ? qi[j] : q;
        s_fin[1 + kMaxLevels + q] = e;
      }
      __syncthreads();
    }
  }

  if (!skip && pk > 0) {
    if (!(MULTI)) first_digit();
    uint32_t nonzero;                  // keys counted, of the whole node
    {
      constexpr int PER = kBins0 / NT;
      const int base = kBins0 - (tid + 1) * PER;
      uint32_t sum = 0;
#pragma unroll
      for (int q = 0; q < PER; ++q) sum += hist[base + q];
      const uint32_t inc = wave_scan(sum);
      if (lane == 63) redu[1][w] = inc;
      __syncthreads();
      uint32_t cum;
      nonzero = waves_sum<NW>(redu[1], lane, w, &cum);
      cum += inc - sum;
      for (int s = 0; s < pk; ++s) find_bin<PER>(hist + base, base, lv.K[s] - cum, sum, s_walk[s]);
    }
    __syncthreads();
    // (a size that the non-zero keys do not reach keeps rank 0: its threshold is zero, all of them are above it)
    // ---- candidates: keys from the lowest threshold's bin up; energy of the rest ----
    const uint32_t lowkey = max(lane_value(s_walk[pk - 1][0], 0) << kShift0, 1u);
    double Eb = 0.0;
    uint32_t mine = 0;
    const uint32_t m2 = key_mask();
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const uint32_t key = fbits(v[i]) & m2;
      const bool cand = key >= lowkey;
      const double dv = (double)__uint_as_float(cand ? 0u : key);
      Eb = fma(dv, dv, Eb);
      mine += cand ? 1u : 0u;
    }
    Eb = wave_total(Eb);
    const uint32_t inc = wave_scan(mine);
    if (lane == 63) redu[2][w] = inc;
    if (lane == 0) red[2][w] = Eb;
    __syncthreads();
    uint32_t at;
    const uint32_t C = waves_sum<NW>(redu[2], lane, w, &at);
    at += inc - mine;
    Eb = waves_sum<NW>(red[2], lane);
    if (tid == 0) s_fin[0] = Eb;
    const bool listed = C <= (uint32_t)CAP;
    if (listed) {
      const uint32_t m3 = key_mask();
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const uint32_t key = fbits(v[i]) & m3;
        if (key >= lowkey) list[at++] = key;
      }
    }
    // calls f(key, candidate) -- in all active lanes, lane 0 among them for as long as any is
    auto each_candidate = [&](auto&& f) {
      if (listed) {
#pragma unroll 2
        for (uint32_t i = tid; i < C; i += NT) f(list[i], true);
      } else {
        const uint32_t m4 = key_mask();
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
          const uint32_t key = fbits(v[i]) & m4;
          f(key, key >= lowkey);
        }
      }
    };
    for (int s0 = 0; s0 < pk; s0 += kBatch) {
      const int nb = min(kBatch, pk - s0);
      uint32_t pre[kBatch], T[kBatch], inbin = 0, most = 0;      // first digit of the thresholds; keys in those bins
#pragma unroll
      for (int s = 0; s < kBatch; ++s) {
        pre[s] = (s < nb && lane_value(s_walk[s0 + s][1], 0) != 0) ? lane_value(s_walk[s0 + s][0], 0) : 0xFFFFFFFFu;
        const uint32_t c = s < nb ? lane_value(s_walk[s0 + s][2], 0) : 0u;
        inbin += c;
        most = max(most, c);
      }
      if (!MULTI && most <= 64) {
        // ---- few keys in every threshold's bin: one wavefront per size ranks them directly ----
        if (tid < kBatch) s_fill[tid] = 0;
        __syncthreads();
        each_candidate([&](uint32_t key, bool cand) {
#pragma unroll
          for (int s = 0; s < kBatch; ++s)
            if (cand && (key >> kShift0) == pre[s]) hist[s * 64 + atomicAdd(&s_fill[s], 1u)] = key;
        });
        __syncthreads();
        if (w < nb) {
          const uint32_t c = lane_value(s_walk[s0 + w][2], 0), r = lane_value(s_walk[s0 + w][1], 0);
          const uint32_t key = lane < c ? hist[w * 64 + lane] : 0u;
          uint32_t gt = 0, eq = 0;
          for (uint32_t j = 0; j < c; ++j) {
            const uint32_t kj = lane_value(key, (int)j);
            gt += kj > key ? 1u : 0u;
            eq += kj == key ? 1u : 0u;
          }
          if (lane < c && gt < r && r <= gt + eq) {        // (equal keys write the same)
            s_walk[s0 + w][0] = key;
            s_walk[s0 + w][1] = r - gt;
            s_walk[s0 + w][2] = eq;
          }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kBatch; ++s) T[s] = pre[s] != 0xFFFFFFFFu ? lane_value(s_walk[s0 + s][0], 0) : 0u;
      } else {
        // ---- second digit ----
        for (int b = tid * 4; b < kBins0; b += NT * 4) *reinterpret_cast<uint4*>(&hist[b]) = make_uint4(0, 0, 0, 0);
        __syncthreads();
        each_candidate([&](uint32_t key, bool cand) {
#pragma unroll
          for (int s = 0; s < kBatch; ++s)
            if (cand && (key >> kShift0) == pre[s]) atomicAdd(&hist[s * kBins1 + ((key >> kShift1) & (kBins1 - 1))], 1u);
        });
        __syncthreads();
        if (MULTI) meet_hist(gh2 + (size_t)s0 * kBins1, nb * kBins1, inbin);
        if (w < nb) wave_walk<kBins1>(hist + w * kBins1, s_walk[s0 + w][1], s_walk[s0 + w]);
        __syncthreads();
        // ---- third digit ----
        inbin = 0;
#pragma unroll
        for (int s = 0; s < kBatch; ++s) {
          if (pre[s] != 0xFFFFFFFFu) {
            pre[s] = (pre[s] << 10) | lane_value(s_walk[s0 + s][0], 0);
            inbin += lane_value(s_walk[s0 + s][2], 0);
          }
        }
        for (int b = tid * 4; b < kBatch * kBins2; b += NT * 4) *reinterpret_cast<uint4*>(&hist[b]) = make_uint4(0, 0, 0, 0);
        __syncthreads();
        each_candidate([&](uint32_t key, bool cand) {
#pragma unroll
          for (int s = 0; s < kBatch; ++s)
            if (cand && (key >> kShift1) == pre[s]) atomicAdd(&hist[s * kBins2 + (key & (kBins2 - 1))], 1u);
        });
        __syncthreads();
        if (MULTI) meet_hist(gh3 + (size_t)s0 * kBins2, nb * kBins2, inbin);
        if (w < nb) wave_walk<kBins2>(hist + w * kBins2, s_walk[s0 + w][1], s_walk[s0 + w]);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kBatch; ++s) T[s] = pre[s] != 0xFFFFFFFFu ? (pre[s] << 9) | lane_value(s_walk[s0 + s][0], 0) : 0u;
      }
      // ---- energy strictly below every threshold, among the candidates; keys above and equal to it ----
      uint32_t gt[kBatch], eq[kBatch];
      double strict[kBatch];
#pragma unroll
      for (int s = 0; s < kBatch; ++s) {
        strict[s] = 0.0;
        gt[s] = eq[s] = 0;
      }
      each_candidate([&](uint32_t key, bool cand) {
        const double dv = (double)__uint_as_float(cand ? key : 0u);
        const double e = dv * dv;
#pragma unroll
        for (int s = 0; s < kBatch; ++s) {
          strict[s] += key < T[s] ? e : 0.0;
          if (MULTI) {
            gt[s] += popc64(ballot(cand && key > T[s]));
            eq[s] += popc64(ballot(cand && key == T[s]));
          }
        }
      });
#pragma unroll
      for (int s = 0; s < kBatch; ++s) {
        if (s < nb) {
          const double e = wave_total(strict[s]);
          if (lane == 0) {
            redb[s][w] = e;
            if (MULTI) { redc[0][s][w] = gt[s]; redc[1][s][w] = eq[s]; }
          }
        }
      }
      __syncthreads();
      if (tid < nb) {
        const int s = s0 + tid;
        double e = 0.0;
        uint32_t g = 0, q = 0;
#pragma unroll 4
        for (int i = 0; i < NW; ++i) {
          e += redb[tid][i];
          if (MULTI) { g += redc[0][tid][i]; q += redc[1][tid][i]; }
        }
        const bool zero = s_walk[s][1] == 0;              // threshold zero: K - nonzero of the d - nonzero zeros are taken
        uint32_t Ts = 0;
#pragma unroll
        for (int b = 0; b < kBatch; ++b) Ts = b == tid ? T[b] : Ts;
        s_T[s] = Ts;
        s_r[s] = zero ? s_K[s] - nonzero : s_walk[s][1];
        s_eq[s] = zero ? d - nonzero : s_walk[s][2];
        s_fin[1 + s] = e;
        if (MULTI) { s_cnt[0][s] = g; s_cnt[1][s] = zero ? len - C : q; }
      }
      __syncthreads();
    }
  }

  // ---- totals over the node's blocks ----
  if (MULTI && !skip && (pk > 0 || nq > 0)) {
    const int ne = 1 + pk + nq;            // energies: below the candidates, below every threshold, quantiser errors
    __syncthreads();
    if (tid < ne + 2 * pk) {
      double t;
      if (tid < 1 + pk) t = pk > 0 ? s_fin[tid] : 0.0;
      else if (tid < ne) t = s_fin[1 + kMaxLevels + (tid - 1 - pk)];
      else t = (double)s_cnt[(tid - ne) / pk][(tid - ne) % pk];
      st_coherent(&part2[(size_t)tid * NB + part], -t);
    }
    for (int i = w; i < ne + 2 * pk; i += NW) {
      const double t = meet_value(part2 + (size_t)i * NB);
      if (i < ne) {
        const double s = wave_total(t);
        if (lane == 0) s_fin[i < 1 + pk ? i : 1 + kMaxLevels + (i - 1 - pk)] = s;
      } else {
        list[(i - ne) * 64 + lane] = (uint32_t)t;      // (the candidates are no longer needed)
      }
    }
    __syncthreads();
  }
  __syncthreads();

  int slot, q_sel;
  choose(S, Dn, skip, part == 0, &slot, &q_sel);
  const uint32_t K_sel = slot >= 0 ? __builtin_amdgcn_readfirstlane(s_K[slot]) : 0u;

  if (slot >= 0) {
    // ---- message of the chosen Top-K size in ascending coordinate, h <- h + C(v) ----
    const bool ident = slot >= pk;
    const uint32_t T = ident ? 0u : lane_value(s_T[slot], 0);
    uint32_t r = ident ? 0u : lane_value(s_r[slot], 0);         // ties this block takes, below
    const bool all = ident || lane_value(s_eq[slot], 0) == r;   // every key equal to T is taken
    uint32_t first = ident ? c0 : 0u;            // message offset of the chunk's first entry
    if (MULTI && !ident) {
      const uint32_t g = list[slot * 64 + lane], e = list[(pk + slot) * 64 + lane];     // (zero beyond the node's blocks)
      const uint32_t before = wave_scan(e) - e;
      const uint32_t take = before >= r ? 0u : min(e, r - before);
      const uint32_t out = wave_scan(g + take) - (g + take);
      first = lane_value(out, part);
      const uint32_t eqb = lane_value(before, part);
      r = r > eqb ? r - eqb : 0u;
    }
    uint64_t taken = 0;                          // bit 4 q + c: component c of quad q is in the message
    const uint32_t m6 = key_mask();
    if (!all) {                                  // ties in coordinate order: rank of each among the chunk's keys equal to T
#pragma unroll
      for (int q = 0; q < NQ4; ++q) {
        uint32_t n = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) n += popc64(ballot((fbits(v[q * 4 + c]) & m6) == T && quad_at(q) + c < len));
        if (lane == 0) s_teq[q * NW + w] = n;
      }
      __syncthreads();
      if (w == 0) wave_scan_table(s_teq, NQ4 * NW, lane);
      __syncthreads();
    }
    const uint32_t m7 = key_mask();
#pragma unroll
    for (int q = 0; q < NQ4; ++q) {
      const uint32_t l0 = quad_at(q);
      uint32_t f = 0;
      if (all) {
#pragma unroll
        for (int c = 0; c < 4; ++c) f |= ((fbits(v[q * 4 + c]) & m7) >= T && l0 + c < len) ? 1u << c : 0u;
      } else {
        bool eq[4];
        uint32_t rk = s_teq[q * NW + w];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          eq[c] = (fbits(v[q * 4 + c]) & m7) == T && l0 + c < len;
          rk += below(ballot(eq[c]));
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          f |= ((fbits(v[q * 4 + c]) & m7) > T || (eq[c] && rk < r)) ? 1u << c : 0u;
          rk += eq[c] ? 1u : 0u;
        }
      }
      taken |= (uint64_t)f << (4 * q);
      const uint32_t n = popc64(ballot(f & 1u)) + popc64(ballot(f & 2u)) + popc64(ballot(f & 4u)) + popc64(ballot(f & 8u));
      if (lane == 0) s_tab[q * NW + w] = n;
    }
    __syncthreads();
    if (w == 0) wave_scan_table(s_tab, NQ4 * NW, lane);
    __syncthreads();
    // message offsets of the chunk's groups of 2048 coordinates (the aggregation reads them)
    constexpr int kPerGroup = kWaveTile / 256;   // (quad, wavefront) entries per group
    uint32_t* __restrict__ go = ns.grp_off + (size_t)node * (ns.groups + 1) + c0 / kWaveTile;
    for (int g = tid; g * kWaveTile < (int)len; g += NT) go[g] = first + s_tab[g * kPerGroup];
    if (tid == 0 && part == NB - 1) ns.grp_off[(size_t)node * (ns.groups + 1) + ns.groups] = K_sel;
    int32_t* __restrict__ midx = ns.msg_idx + (size_t)node * ns.Kcap + first;
    float* __restrict__ mval = ns.msg_val + (size_t)node * ns.Kcap + first;
#pragma unroll
    for (int q = 0; q < NQ4; ++q) {
      const uint32_t l0 = quad_at(q);
      const uint32_t f = (uint32_t)(taken >> (4 * q)) & 15u;
      uint32_t pos = s_tab[q * NW + w] + below(ballot(f & 1u)) + below(ballot(f & 2u)) + below(ballot(f & 4u)) + below(ballot(f & 8u));
      float hq[4];
      h_quad(q, hq);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float vv = v[q * 4 + c], hn = a.assign ? vv : hq[c] + vv;
        hq[c] = ((f >> c) & 1u) ? hn : hq[c];
      }
      keep_h(q, hq);
      if (f) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if ((f >> c) & 1u) {
            midx[pos] = (int32_t)(c0 + l0 + c);
            mval[pos] = v[q * 4 + c];
            ++pos;
          }
        }
        buf_store4(hb, off0, q * NT * 16, hq);
      }
      if (!MULTI && a.to_dense) {
        float cv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) cv[c] = ((f >> c) & 1u) ? v[q * 4 + c] : 0.f;
        buf_store4(make_buf(ns.dense + row, 4 * len), off0, q * NT * 16, cv);
      }
    }
  } else if (QUANT && q_sel >= 0) {
    // ---- dense update and codes of the chosen quantiser level ----
    const int B = lv.qblock[q_sel];
    const int lb = B ? __ffs(B) - 1 : 0;
    const float qs = lv.qs[q_sel];
    const double qd = lv.qdenom[q_sel];
    const float qc = (!B && qa > 0.f) ? (float)((double)qa / qd) : 0.f;
    const Buf cb = make_buf(ns.qcodes + row, 2 * len);
    const bool even4 = (d | len) % 4 == 0;
    if (tid == 0 && part == 0) ns.qscale[node] = qc;
    if (B) {
      __syncthreads();
      block_scales(B, &qd, 1);
      __syncthreads();
      for (uint32_t b = tid; b < (len + B - 1) / B; b += NT) ns.qbscale[(size_t)node * ns.nseg + c0 / B + b] = blk_c[b];
    }
#pragma unroll
    for (int q = 0; q < NQ4; ++q) {
      const uint32_t l0 = quad_at(q);
      __builtin_amdgcn_sched_barrier(0);
      if (l0 < len) {
        uint32_t rnd[4];
        philox4x32_10((c0 + l0) >> 2, ctr1, a.step, 0u, k0, k1, rnd);
        const float aq = B ? blk_a[l0 >> lb] : qa;
        const float cq = B ? blk_c[l0 >> lb] : qc;
        float hq[4];
        int code4[4];
        h_quad(q, hq);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          code4[c] = 0;
          hq[c] += aq > 0.f ? quant_one(v[q * 4 + c], aq, qs, cq, dither_of(rnd[c]), &code4[c]) : 0.f;
        }
        keep_h(q, hq);
        buf_store4(hb, off0, q * NT * 16, hq);
        const uint32_t c01 = (uint32_t)(uint16_t)code4[0] | ((uint32_t)(uint16_t)code4[1] << 16);
        const uint32_t c23 = (uint32_t)(uint16_t)code4[2] | ((uint32_t)(uint16_t)code4[3] << 16);
        if (even4) {
          __builtin_amdgcn_raw_buffer_store_b64(bword2{c01, c23}, cb.r, off0 / 2, q * NT * 8, 0);
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            __builtin_amdgcn_raw_buffer_store_b16((short)code4[c], cb.r, off0 / 2 + 2 * c, q * NT * 8, 0);
        }
      }
    }
  }

  // ---- iterate update that opens the next step, from this node's new estimator (the master) ----
  if (a.xu_out && node == 0) {
    const Buf xub = make_buf(a.xu_x + c0, 4 * len), xuo = make_buf(a.xu_out + c0, 4 * len);
#pragma unroll
    for (int q = 0; q < NQ4; ++q) {
      float xq[4], hq[4];
      h_quad(q, hq);       // (of what is read again, this thread's own stores)
      buf_load4(xub, off0, q * NT * 16, xq);
#pragma unroll
      for (int c = 0; c < 4; ++c) xq[c] = (float)((double)xq[c] - a.xu_gamma * (double)hq[c]);
      buf_store4(xuo, off0, q * NT * 16, xq);
    }
  }
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
template <int NT, int VPT, int CAP, bool MULTI>
static hipError_t launch_node_as(const NodeSet& ns, const PassArgs& a, hipStream_t st) {
  const size_t lds = sizeof(uint32_t) * (kBins0 + CAP);
  auto go = [&](auto kern) -> hipError_t {
    hipLaunchKernelGGL(kern, dim3((unsigned)ns.nn * ns.NB), dim3(NT), lds, st, ns, a);
    return hipGetLastError();
  };
  return ns.lv.nq > 0 ? go(k_node<NT, VPT, CAP, true, MULTI>) : go(k_node<NT, VPT, CAP, false, MULTI>);
}

hipError_t launch_node(const NodeSet& ns, const PassArgs& a, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  if (ns.NB > 1) {
    if (ns.chunk <= 4096) return launch_node_as<512, 8, 4096, true>(ns, a, st);
    if (ns.chunk <= 8192) return launch_node_as<512, 16, 8192, true>(ns, a, st);
    return launch_node_as<512, 32, 12288, true>(ns, a, st);
  }
  if (ns.chunk <= 1024) return launch_node_as<256, 4, 1024, false>(ns, a, st);
  if (ns.chunk <= 4096) return launch_node_as<512, 8, 4096, false>(ns, a, st);
  if (ns.chunk <= 8192) return launch_node_as<512, 16, 8192, false>(ns, a, st);
  return launch_node_as<512, 32, 12288, false>(ns, a, st);
}

}  // namespace adacgd
