// The compression step of vectors of at most kShortDim coordinates (Top-K levels only): one block per node, one thread per
// coordinate.  For workers of which every message can be added up where it is made, the same launch also aggregates, and with
// a master compressor of Top-K levels it goes on to compress the server's vector: a whole step after the gradient is one launch.
//
// Such a step is bound by its dependent phases, so there are few of them: every coordinate finds its exact place in the order
// (larger magnitude first, then lower index) and all levels follow from it -- a coordinate is in the Top-K set if its place is
// below K, whatever K is.  Places come from one histogram of the keys' leading bits, as fine as 16 bins an octave below the
// largest key: keys are put side by side bin by bin and compared inside their bin only.  Between two barriers lie one or two
// round trips to LDS; four barriers a node.  (k_node selects with a threshold for every Top-K size, from three digits of the
// key, which takes less work a coordinate and more phases a size.)
// Measured, a whole step with supplied gradients, against k_node for the workers and their aggregation and k_node for the
// master: 4 workers x 100 coordinates, five sizes, 19.6 and 9.0 us; 20 x 300 28 and 12.5; 64 x 512 40 and 15.3; without
// aggregation or master here, 200 x 300 38 and 32.5, 2000 x 500 147 and 143.  Not beyond 512 coordinates, whatever the number of
// workers: 1024 threads a block took 15.8 instead of 13.3 us for 64 x 1024 with one size and no master, 171 instead of 148 for
// 2000 x 1000.  (Few workers with a master would have gained there, 1.1 to 1.4 times as fast.)
#include "devutil.h"
#include "engine.h"

namespace adacgd {

// What the kernel needs of a node set and of one application of the compressor to it.
struct ShortSide {
  int m, p;
  uint32_t K[kMaxLevels];
  int ref[kMaxLevels];
  double tz[kMaxLevels], te[kMaxLevels];
  const float* x;
  float* h;
  const float* y;
  float* ycopy;
  const double* extD;
  int diff, assign;
  double *S, *D, *err;
  int32_t *level, *sel_slot, *sel_q;
  uint32_t* msg_count;
  unsigned long long* level_hist;
  uint32_t* grp_off;
  int32_t* msg_idx;
  float* msg_val;
  uint32_t Kcap;
};

struct ShortArgs {
  uint32_t d;
  int nn;
  int serve;             // this launch also aggregates
  int master;            // ... and compresses the server's vector
  float* dense;          // serve: [nn][d] C(v) of every node (zero where it keeps its estimator)
  uint32_t* done;        // serve: arrival counter
  const float* agg_old;
  float* agg_new;
  const float* xu_x;     // the iterate update that follows (xu_out null: none)
  float* xu_out;
  double xu_gamma;
  ShortSide W, M;
};

constexpr int kShortBins = 512;      // 32 octaves below the largest key; what is smaller shares the lowest bin
constexpr uint32_t kShortBin = 96;   // with more keys than that in one bin (equal values above all) all of them are sorted: that takes
                                     // 512 coordinates 2.5 us, as the comparisons inside a bin of about 110 keys do

template <int NT>
struct ShortLds {
  static constexpr int NW = NT / 64;
  uint32_t top[NW], zeros[NW];
  __align__(16) uint32_t hist[kShortBins];
  uint64_t sorted[NT];                               // key and index, bin by bin, in no order inside a bin
  double sum[kMaxLevels + 2][NW];                    // per wavefront: energy that a size leaves behind; S, D
  uint32_t count[kMaxLevels][NW];                    // ... coordinates in the Top-K set
  uint32_t edge[2][kMaxLevels];                      // with infinities or NaN: last key in the set, first key left out
};
struct ShortTable {      // the level set, in LDS: indexed lane by lane
  uint32_t K[kMaxLevels];
  int ref[kMaxLevels];
  double tz[kMaxLevels + 1], te[kMaxLevels + 1];
};

// One node: this thread's coordinate of the new point, the estimator and the previous point.  `send` gets the message's
// coordinate before anything else is stored (what it stores may be waited for); then the node's report, message and estimator
// are written.  Returns the new estimator's coordinate.
template <int NT, typename Send>
__device__ __forceinline__ float short_node(const ShortSide& s, const ShortTable& tab, ShortLds<NT>& L, uint32_t d, int node, float xv, float hv,
                                            float yv, double extD, Send&& send) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lane = tid & 63;
  const bool live = (uint32_t)tid < d;
  const float v = s.diff ? xv : xv - hv;             // (+0 beyond the vector's end)
  const uint32_t key = magkey(v);
  for (int b = tid * 4; b < kShortBins; b += NT * 4) *reinterpret_cast<uint4*>(&L.hist[b]) = make_uint4(0, 0, 0, 0);
  uint32_t top = wave_top(key);
  const uint64_t zero = ballot(live && key == 0);
  if (lane == 0) {
    L.top[w] = top;
    L.zeros[w] = popc64(zero);
  }
  __syncthreads();
  // ---- places (zeros by their index alone: there may be many) ----
  uint32_t nonzero = d, place = below(zero);
  top = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const uint32_t z = L.zeros[i];
    top = max(top, L.top[i]);
    nonzero -= z;
    place += i < w ? z : 0u;
  }
  place += nonzero;
  const int low = max((int)(top >> kShift0) - (kShortBins - 1), 0), bin = max((int)(key >> kShift0) - low, 0);
  const uint32_t at = key ? atomicAdd(&L.hist[bin], 1u) : 0u;
  const double dv = (double)v, dw = (double)(xv - yv);
  const double e2 = dv * dv, f2 = dw * dw;
  __syncthreads();
  const uint4 a0 = *reinterpret_cast<const uint4*>(&L.hist[lane * 8]), a1 = *reinterpret_cast<const uint4*>(&L.hist[lane * 8 + 4]);
  const uint32_t sum = a0.x + a0.y + a0.z + a0.w + a1.x + a1.y + a1.z + a1.w;
  const uint32_t above = nonzero - wave_scan(sum);   // keys in the bins of the lanes above
  const uint32_t most = wave_top(max(max(max(a0.x, a0.y), max(a0.z, a0.w)), max(max(a1.x, a1.y), max(a1.z, a1.w))));
  uint64_t mine = (uint64_t)key << 32 | (uint32_t)(NT - 1 - tid);
  if (most <= kShortBin) {
    const uint4 b0 = *reinterpret_cast<const uint4*>(&L.hist[bin & ~7]), b1 = *reinterpret_cast<const uint4*>(&L.hist[(bin & ~7) + 4]);
    const uint32_t bc[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    uint32_t first = (uint32_t)__builtin_amdgcn_ds_bpermute((bin >> 3) << 2, (int)above), members = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      first += q > (bin & 7) ? bc[q] : 0u;
      members = q == (bin & 7) ? bc[q] : members;
    }
    if (key) {
      L.sorted[first + at] = mine;
      place = first;
    } else {
      members = 0;
    }
    __syncthreads();
    for (uint32_t j = 0; j < members; j += 8) {
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) place += j + u < members && L.sorted[first + min(j + u, members - 1)] > mine ? 1u : 0u;
    }
  } else {
    // bitonic, descending; an exchange over less than a wavefront's width stays in it
    for (int k = 2; k <= NT; k *= 2) {
      for (int j = k / 2; j > 0; j /= 2) {
        uint64_t other;
        if (j >= 64) {
          __syncthreads();
          L.sorted[tid] = mine;
          __syncthreads();
          other = L.sorted[tid ^ j];
        } else {
          other = __shfl_xor(mine, j, 64);
        }
        const bool larger = ((tid & j) == 0) == ((tid & k) == 0);
        mine = (other > mine) == larger ? other : mine;
      }
    }
    __syncthreads();
    reinterpret_cast<uint32_t*>(L.sorted)[NT - 1 - (uint32_t)mine] = (uint32_t)tid;
    __syncthreads();
    place = reinterpret_cast<const uint32_t*>(L.sorted)[tid];
  }
  if (!live) place = d;                              // (in no Top-K set)
  const bool wild = top >= 0x7F800000u;
  if (wild) {
    for (int q = 0; q < s.p; ++q) {
      if (place == tab.K[q] - 1) L.edge[0][q] = key;
      if (place == tab.K[q]) L.edge[1][q] = key;
    }
  }
  // ---- what every size leaves behind; S, D (eight sums at a time; a size's first, so that with nothing left out it is S bit for bit) ----
  for (int s0 = 0; s0 < s.p + 2; s0 += 8) {
    double e[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = s0 + u;
      const bool in = place < tab.K[min(q, kMaxLevels - 1)];
      const uint32_t c = popc64(ballot(in));
      if (lane == 0 && q < s.p) L.count[q][w] = c;
      e[u] = q < s.p ? (in ? 0.0 : e2) : q == s.p ? e2 : f2;
    }
    const double all = wave_total8(e);
    const int q = s0 + (int)(lane >> 3);
    if ((lane & 7u) == 0 && q < s.p + 2) L.sum[q][w] = all;
  }
  __syncthreads();
  // ---- the cascade (every wavefront for itself, lane j the level j + 1) ----
  const int ref = tab.ref[min((int)lane, s.m - 1)];
  double S = 0.0, D = 0.0, my_err = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    S += L.sum[s.p][i];
    D += L.sum[s.p + 1][i];
    my_err += L.sum[ref][i];
  }
  // (where a size ends with an infinity or NaN and leaves no equal key behind, its error is not a number, as by the formula of
  // the other kernels: energy below the threshold plus number of ties left times the threshold's square)
  if (wild && tab.K[ref] < d && L.edge[0][ref] >= 0x7F800000u && L.edge[1][ref] != L.edge[0][ref]) my_err = __longlong_as_double(0x7FF8000000000000ll);
  if (s.diff) D = extD;
  auto bound = [&](double tz, double te) { return __dadd_rn(__dmul_rn(tz, D), __dmul_rn(te, S)); };      // trigger_bound
  // first condition of the cascade: nothing else is evaluated (the compressed start applies its level unconditionally)
  const bool skip = !s.assign && S <= bound(tab.tz[0], tab.te[0]);
  const uint32_t pos1 = min(lane + 1u, (uint32_t)kMaxLevels);
  const bool hit = !skip && (int)lane + 1 < s.m && my_err <= bound(tab.tz[pos1], tab.te[pos1]);
  const uint64_t good = ballot(hit);
  const int jstar = skip ? 0 : good ? __ffsll((unsigned long long)good) : s.m;
  const int slot = jstar > 0 ? __builtin_amdgcn_readlane(ref, jstar - 1) : -1;
  const uint32_t K = slot >= 0 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)tab.K[slot]) : 0u;
  const bool sent = slot >= 0 && place < K;
  send(sent ? v : 0.f);
  if (w == 0) {
    if ((int)lane < s.m) s.err[node * s.m + (int)lane] = skip ? __longlong_as_double(0x7FF8000000000000ll) : my_err;
    if (lane == 0) {
      s.S[node] = S;
      s.D[node] = D;
      s.level[node] = jstar;
      atomicAdd(&s.level_hist[jstar], 1ull);
      s.sel_slot[node] = slot;
      s.sel_q[node] = -1;
      s.msg_count[node] = K;
      s.grp_off[2 * node] = 0;
      s.grp_off[2 * node + 1] = K;
    }
  }
  // ---- message in ascending coordinate, h <- h + C(v) ----
  if (slot >= 0) {
    uint32_t pos = below(ballot(sent));
#pragma unroll
    for (int i = 0; i < NW; ++i) pos += i < w ? L.count[slot][i] : 0u;
    if (sent) {
      s.msg_idx[(size_t)node * s.Kcap + pos] = tid;
      s.msg_val[(size_t)node * s.Kcap + pos] = v;
      hv = s.assign ? v : hv + v;
      s.h[(size_t)node * d + tid] = hv;
    }
  }
  return hv;
}

template <int NT>
__global__ __launch_bounds__(NT) void k_short(ShortArgs a) {
  __shared__ ShortLds<NT> L;
  __shared__ ShortTable tw, tm;
  __shared__ int s_flag;
  const int tid = threadIdx.x, node = blockIdx.x;
  const uint32_t d = a.d;
  const bool live = (uint32_t)tid < d;
  const size_t at = (size_t)node * d + (uint32_t)tid;
  // everything that is read, at once
  float xv = 0.f, hv = 0.f, yv = 0.f, go = 0.f, gv = 0.f, xo = 0.f;
  if (live) {
    xv = a.W.x[at];
    hv = a.W.h[at];
    if (!a.W.diff) yv = a.W.y[at];
    if (a.serve) {
      go = a.agg_old[tid];
      if (a.master) gv = a.M.h[tid];
    }
    if (a.xu_out) xo = a.xu_x[tid];
  }
  const double extD = a.W.diff ? a.W.extD[node] : 0.0;
  if (tid < kMaxLevels) {
    tw.K[tid] = a.W.K[tid];
    tw.ref[tid] = a.W.ref[tid];
    tw.tz[tid] = a.W.tz[tid];
    tw.te[tid] = a.W.te[tid];
    tm.K[tid] = a.M.K[tid];
    tm.ref[tid] = a.M.ref[tid];
    tm.tz[tid] = a.M.tz[tid];
    tm.te[tid] = a.M.te[tid];
  }
  if (a.W.ycopy && live) a.W.ycopy[at] = xv;
  bool last = false;
  float gn = short_node<NT>(a.W, tw, L, d, node, xv, hv, yv, extD, [&](float cv) {
    if (a.serve) {
      if (live) st_coherent(&a.dense[at], cv);
      last = arrive_last_few(a.done, (uint32_t)a.nn, &s_flag);
    }
  });
  if (a.serve) {
    // ---- server aggregation by the block that finishes last: every coordinate's sum in ascending worker index (what a
    // worker does not send adds +0, which changes no sum) ----
    if (!last) return;
    double acc = 0.0;
    const float* __restrict__ from = a.dense + min((uint32_t)tid, d - 1);
    auto add = [&](int i0, auto&& t) {        // (no branch: all in flight)
      constexpr int U = sizeof(t) / sizeof(t[0]);
#pragma unroll
      for (int u = 0; u < U; ++u) t[u] = ld_coherent(&from[(size_t)min(i0 + u, a.nn - 1) * d]);
#pragma unroll
      for (int u = 0; u < U; ++u) acc += i0 + u < a.nn ? (double)t[u] : 0.0;
    };
    float t8[8], t32[32];
    if (a.nn <= 8) add(0, t8);
    else
      for (int i0 = 0; i0 < a.nn; i0 += 32) add(i0, t32);
    gn = (float)((double)go + acc / (double)a.nn);
    if (live) a.agg_new[tid] = gn;
    else gn = 0.f;
    // ---- g <- C^AC_{g, g~_old}(g~_new) ----
    if (a.master) gn = short_node<NT>(a.M, tm, L, d, 0, gn, gv, go, 0.0, [](float) {});
  }
  if (a.xu_out && live && (a.serve || node == 0)) a.xu_out[tid] = (float)((double)xo - a.xu_gamma * (double)gn);
}

static ShortSide short_side(const NodeSet& ns, const PassArgs& a) {
  ShortSide s;
  s.m = ns.lv.m;
  s.p = ns.lv.p;
  for (int j = 0; j < kMaxLevels; ++j) {
    s.K[j] = ns.lv.K[j];
    s.ref[j] = ns.lv.ref[j];
    s.tz[j] = ns.lv.tz[j];
    s.te[j] = ns.lv.te[j];
  }
  s.x = a.x; s.h = a.h; s.y = a.y; s.ycopy = a.ycopy; s.extD = a.extD;
  s.diff = a.diff; s.assign = a.assign;
  s.S = ns.S; s.D = ns.D; s.err = ns.err;
  s.level = ns.level; s.sel_slot = ns.sel_slot; s.sel_q = ns.sel_q;
  s.msg_count = ns.msg_count; s.level_hist = ns.level_hist; s.grp_off = ns.grp_off;
  s.msg_idx = ns.msg_idx; s.msg_val = ns.msg_val; s.Kcap = ns.Kcap;
  return s;
}

hipError_t launch_short(const NodeSet& ns, const PassArgs& a, const NodeSet* ms, const PassArgs* m, hipStream_t st) {
  (void)hipGetLastError();   // drop a stale error left by earlier runtime calls of this thread
  ShortArgs s{};
  s.d = (uint32_t)ns.d;
  s.nn = ns.nn;
  s.serve = a.agg_new != nullptr;
  s.master = ms != nullptr;
  s.dense = ns.dense;
  s.done = ns.done;
  s.agg_old = a.agg_old;
  s.agg_new = a.agg_new;
  const PassArgs& last = ms ? *m : a;
  s.xu_x = last.xu_x;
  s.xu_out = last.xu_out;
  s.xu_gamma = last.xu_gamma;
  s.W = short_side(ns, a);
  if (ms) s.M = short_side(*ms, *m);
  auto go = [&](auto kern, int threads) -> hipError_t {
    hipLaunchKernelGGL(kern, dim3((unsigned)ns.nn), dim3(threads), 0, st, s);
    return hipGetLastError();
  };
  if (ns.d <= 128) return go(k_short<128>, 128);
  if (ns.d <= 256) return go(k_short<256>, 256);
  return go(k_short<512>, 512);
}

}  // namespace adacgd
