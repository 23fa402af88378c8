// Steps 4-5 of the planner: integer replica matching and token split.
//
// Phase 2 (Alg. 2, Sec. A.3): K rounds of column-priority matching.  In each
// inner iteration every unmatched cold rank proposes its best expert under
// the three-level score min(spill, spare) + alpha*B + 0.1*alpha*T_norm, each
// proposed expert keeps its best proposer, and winners take
// g = min(spill, spare) into their slot for this round.
// Phase 3 (Alg. 3, Sec. A.4): Lagrangian auction.  Each round every open slot
// bids for the source rank with the highest bonus minus price among ranks
// still holding tokens of its expert; each rank serves its best bidder with
// min(tokens held, tokens still planned) and raises its price.
//
// Exactness.  All state is integer; scores are fp64 evaluated in the order
// stated in taot.h and compiled without FP contraction; every argmax is
// masked and breaks ties to the lowest index.  Two shortcuts are exact:
//   - a phase stops at the first iteration/round with no proposal/bid, which
//     leaves the state unchanged and so equals running the remaining ones;
//   - a Phase-3 slot re-bids only when the rank it bid for served (its price
//     rose, its stock fell) or ran out of the slot's expert: every other
//     rank's score can only fall and its validity only end, so the previous
//     argmax (including its tie-break) stands.
//
// One workgroup per problem, grid-stride over problems; per-workgroup state
// lives in a slab of the workspace (L2-resident), per-rank auction
// arbitration in LDS.
#include <limits.h>

#include "common.h"

namespace taot {
namespace {

constexpr int kSchThreads = 256;
constexpr int kSchWaves = kSchThreads / kWave;
constexpr int kSchMaxGrid = 1024;

struct SchParams {
  const int32_t* n;
  const int64_t* spill;
  const int64_t* spare;
  const int64_t* excess;
  const double* alpha;
  const int32_t* home;
  const float* T;
  const double* Bpref;
  const double* Bauct;
  int32_t B, R, E, K;
  double price_step;
  int64_t t_max;
  int32_t* slot_expert;
  int64_t* slot_amount;
  int32_t* X;
  int64_t* unfilled;
  int32_t* rounds_used;
  uint32_t* status;
  char* slab;
  int64_t slab_bytes;
  const int32_t* fallback;  // [B] 1 = the LDS-resident kernel left this problem to us (nullable)
  uint32_t flags;           // TAOT_SCH_*
};

// Weights of the Phase-2 score terms: alpha for alpha * Bpref and 0.1 * alpha
// for the flow hint, or 0 for a term the flags drop (it then enters the sum
// as +0, in the same evaluation order).
__device__ __forceinline__ double topo_weight(uint32_t flags, double alpha) {
  return (flags & TAOT_SCH_NO_TOPO) ? 0.0 : alpha;
}
__device__ __forceinline__ double flow_weight(uint32_t flags, double alpha) {
  return (flags & TAOT_SCH_NO_FLOW) ? 0.0 : 0.1 * alpha;
}

struct Slab {
  // Phase 2
  int32_t* cr;        // [R] cold ranks, ascending
  int64_t* spare_p;   // [R]
  int32_t* matched;   // [R]
  int32_t* prop_e;    // [R] proposed candidate index or -1
  double* prop_s;     // [R]
  int32_t* assigned;  // [R*K] candidate index assigned to cold rank rc in round k
  int32_t* ce;        // [E] candidate experts (spill > 0), ascending
  int64_t* spill_p;   // [E]
  int32_t* win;       // [E] winning cold-rank index or -1
  // Phase 3
  int32_t* dmap;      // [E] expert -> distinct slot-expert index or -1
  int32_t* dexp;      // [D] distinct slot experts, ascending
  int32_t* bid;       // [S]
  double* bid_s;      // [S]
  int64_t* Ap;        // [S] tokens still planned
  int32_t* dsl;       // [S] distinct index of the slot's expert or -1
  int32_t* need;      // [S] 1 = recompute the bid
  int32_t* work;      // [S] compacted list of slots to recompute
  int32_t* nprime;    // [D*R] tokens of distinct expert d still held by rank r
  size_t bytes;
};

__host__ __device__ Slab carve_slab(char* base, int32_t R, int32_t E, int32_t K) {
  Carver c{base};
  const int64_t S = (int64_t)R * K;
  const int64_t D = S < E ? S : E;
  Slab s;
  s.cr = c.take<int32_t>(R);
  s.spare_p = c.take<int64_t>(R);
  s.matched = c.take<int32_t>(R);
  s.prop_e = c.take<int32_t>(R);
  s.prop_s = c.take<double>(R);
  s.assigned = c.take<int32_t>((size_t)R * (K > 0 ? K : 1));
  s.ce = c.take<int32_t>(E);
  s.spill_p = c.take<int64_t>(E);
  s.win = c.take<int32_t>(E);
  s.dmap = c.take<int32_t>(E);
  s.dexp = c.take<int32_t>((size_t)(D > 0 ? D : 1));
  s.bid = c.take<int32_t>((size_t)(S > 0 ? S : 1));
  s.bid_s = c.take<double>((size_t)(S > 0 ? S : 1));
  s.Ap = c.take<int64_t>((size_t)(S > 0 ? S : 1));
  s.dsl = c.take<int32_t>((size_t)(S > 0 ? S : 1));
  s.need = c.take<int32_t>((size_t)(S > 0 ? S : 1));
  s.work = c.take<int32_t>((size_t)(S > 0 ? S : 1));
  s.nprime = c.take<int32_t>((size_t)(D > 0 ? D : 1) * R);
  s.bytes = c.off;
  return s;
}

// Exclusive position of `flag` among the kSchThreads threads (ascending
// thread id) and the chunk total.  All threads must call it.
__device__ __forceinline__ int32_t compact_pos(bool flag, int32_t* wave_cnt, int32_t& total) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const uint64_t m = __ballot(flag);
  const int32_t lp = __popcll(m & ((1ull << lane) - 1ull));
  if (lane == 0) wave_cnt[wid] = __popcll(m);
  __syncthreads();
  int32_t off = 0, tot = 0;
  for (int w = 0; w < kSchWaves; ++w) {
    const int32_t c = wave_cnt[w];
    off += w < wid ? c : 0;
    tot += c;
  }
  __syncthreads();
  total = tot;
  return off + lp;
}

// Block-wide OR of a flag.  All threads must call it.
__device__ __forceinline__ bool block_any(bool flag, int32_t* wave_cnt) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const uint64_t m = __ballot(flag);
  if (lane == 0) wave_cnt[wid] = m != 0;
  __syncthreads();
  bool any = false;
  for (int w = 0; w < kSchWaves; ++w) any |= wave_cnt[w] != 0;
  __syncthreads();
  return any;
}

__device__ __forceinline__ uint64_t auction_key(double x) {
  return ordered_key(x == 0.0 ? 0.0 : x);  // -0 and +0 compare equal
}

__global__ void __launch_bounds__(kSchThreads) schedule_kernel(SchParams p) {
  extern __shared__ char lds_raw[];
  __shared__ int32_t wave_cnt[kSchWaves];
  __shared__ int32_t sh_flag;
  __shared__ double sh_rbs[kSchWaves];  // row-priority argmax, per wave
  __shared__ int32_t sh_rbi[kSchWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
  const int32_t R = p.R, E = p.E, K = p.K;
  const int64_t S = (int64_t)R * K;
  // per-rank auction state in LDS
  double* price = reinterpret_cast<double*>(lds_raw);
  uint64_t* rkey = reinterpret_cast<uint64_t*>(price + R);
  int32_t* rwin = reinterpret_cast<int32_t*>(rkey + R);
  int32_t* served = rwin + R;

  Slab sl = carve_slab(p.slab + (int64_t)blockIdx.x * p.slab_bytes, R, E, K);

  for (int64_t b = blockIdx.x; b < p.B; b += gridDim.x) {
    if (p.fallback && p.fallback[b] == 0) continue;  // uniform per block
    const int64_t* spill = p.spill + b * E;
    const int64_t* spare = p.spare + b * R;
    const int64_t* excess = p.excess + b * R;
    const float* Tb = p.T + b * (int64_t)R * R;
    int32_t* se = p.slot_expert + b * S;
    int64_t* sa = p.slot_amount + b * S;
    int32_t* Xb = p.X + b * (int64_t)R * S;
    const double alpha = topo_weight(p.flags, p.alpha[b]);
    const double a2 = flow_weight(p.flags, p.alpha[b]);  // weight of the OT hint

    // ---- validation and setup -----------------------------------------------
    if (tid == 0) sh_flag = 0;
    __syncthreads();
    for (int32_t e = tid; e < E; e += kSchThreads) {
      const int32_t h = p.home[e];
      if (h < 0 || h >= R) sh_flag = 1;
    }
    for (int64_t s = tid; s < S; s += kSchThreads) { se[s] = -1; sa[s] = 0; }
    for (int64_t q = tid; q < (int64_t)R * S; q += kSchThreads) Xb[q] = 0;
    __syncthreads();
    if (sh_flag) {
      if (tid == 0) {
        p.unfilled[b] = 0;
        if (p.rounds_used) { p.rounds_used[2 * b] = 0; p.rounds_used[2 * b + 1] = 0; }
        if (p.status) p.status[b] = TAOT_ST_BAD_INPUT;
      }
      __syncthreads();
      continue;
    }

    // candidate experts (spill > 0) and cold ranks (spare > 0), ascending
    int32_t ne = 0, nc = 0;
    for (int32_t base = 0; base < E; base += kSchThreads) {
      const int32_t e = base + tid;
      const bool f = e < E && spill[e] > 0;
      int32_t tot;
      const int32_t pos = compact_pos(f, wave_cnt, tot);
      if (f) { sl.ce[ne + pos] = e; sl.spill_p[ne + pos] = spill[e]; }
      ne += tot;
    }
    for (int32_t base = 0; base < R; base += kSchThreads) {
      const int32_t r = base + tid;
      const bool f = r < R && spare[r] > 0;
      int32_t tot;
      const int32_t pos = compact_pos(f, wave_cnt, tot);
      if (f) { sl.cr[nc + pos] = r; sl.spare_p[nc + pos] = spare[r]; }
      nc += tot;
    }
    for (int64_t q = tid; q < (int64_t)nc * K; q += kSchThreads) sl.assigned[q] = -1;
    __syncthreads();

    // ---- Phase 2: column-priority iterative matching --------------------------
    int32_t used2 = 0;
    if (p.flags & TAOT_SCH_ROW_PRIORITY) {
      // the experts-outer greedy (ablation): per slot round, the experts with
      // spill left in order of spill (largest first, lower index on ties), each
      // taking its best ranks one at a time until its spill is gone
      for (int32_t k = 0; k < K; ++k) {
        int32_t nord = 0;
        for (int32_t base = 0; base < ne; base += kSchThreads) {
          const int32_t ec = base + tid;
          const int64_t v = ec < ne ? sl.spill_p[ec] : 0;
          int32_t tot;
          compact_pos(v > 0, wave_cnt, tot);
          if (v > 0) {
            int32_t pos = 0;
            for (int32_t o = 0; o < ne; ++o) {
              const int64_t u = sl.spill_p[o];
              pos += u > v || (u == v && o < ec);
            }
            sl.win[pos] = ec;
          }
          nord += tot;
        }
        __syncthreads();
        for (int32_t i = 0; i < nord; ++i) {
          const int32_t ec = sl.win[i];
          const int32_t h = p.home[sl.ce[ec]];
          for (;;) {
            const int64_t spl = sl.spill_p[ec];
            if (spl <= 0) break;
            double bs = -INFINITY;
            int32_t best = INT_MAX;
            for (int32_t rc = tid; rc < nc; rc += kSchThreads) {
              const int64_t sp = sl.spare_p[rc];
              const int32_t r = sl.cr[rc];
              if (sp <= 0 || r == h || sl.assigned[(int64_t)rc * K + k] >= 0) continue;
              bool taken = false;
              for (int32_t kk = 0; kk < k; ++kk) taken |= sl.assigned[(int64_t)rc * K + kk] == ec;
              if (taken) continue;
              const double q = (double)(spl < sp ? spl : sp);
              const double t1 = alpha * p.Bpref[(int64_t)h * R + r];
              const double ex = (double)excess[h];
              const double tn = (double)Tb[(int64_t)h * R + r] / (ex > kEps0 ? ex : kEps0);
              const double t2 = a2 * tn;
              const double score = (q + t1) + t2;
              if (score > bs) { bs = score; best = rc; }  // rc ascends within a thread
            }
            // block argmax: max score, then lowest cold-rank index (= lowest rank)
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
              const double os = __shfl_xor(bs, o, kWave);
              const int32_t oi = __shfl_xor(best, o, kWave);
              if (os > bs || (os == bs && oi < best)) { bs = os; best = oi; }
            }
            if (lane == 0) { sh_rbs[wid] = bs; sh_rbi[wid] = best; }
            __syncthreads();
            if (tid == 0) {
              double b2 = sh_rbs[0];
              int32_t i2 = sh_rbi[0];
              for (int w2 = 1; w2 < kSchWaves; ++w2)
                if (sh_rbs[w2] > b2 || (sh_rbs[w2] == b2 && sh_rbi[w2] < i2)) { b2 = sh_rbs[w2]; i2 = sh_rbi[w2]; }
              if (i2 != INT_MAX) {
                const int64_t g = spl < sl.spare_p[i2] ? spl : sl.spare_p[i2];
                sl.spill_p[ec] -= g;
                sl.spare_p[i2] -= g;
                sl.assigned[(int64_t)i2 * K + k] = ec;
                const int64_t s = (int64_t)sl.cr[i2] * K + k;
                se[s] = sl.ce[ec];
                sa[s] += g;
              }
              sh_flag = i2 != INT_MAX;
            }
            __syncthreads();
            const bool placed = sh_flag != 0;
            __syncthreads();
            if (!placed) break;
            ++used2;
          }
        }
      }
    } else
    for (int32_t k = 0; k < K; ++k) {
      for (int32_t rc = tid; rc < nc; rc += kSchThreads) sl.matched[rc] = 0;
      __syncthreads();
      for (int32_t inner = 0; inner < nc; ++inner) {
        // Step 1: each unmatched cold rank proposes its best candidate expert
        bool proposed = false;
        for (int32_t rc = tid; rc < nc; rc += kSchThreads) {
          int32_t best = -1;
          double bs = -INFINITY;
          const int64_t sp = sl.spare_p[rc];
          if (!sl.matched[rc] && sp > 0) {
            const int32_t r = sl.cr[rc];
            for (int32_t ec = 0; ec < ne; ++ec) {
              const int64_t spl = sl.spill_p[ec];
              if (spl <= 0) continue;
              const int32_t e = sl.ce[ec];
              const int32_t h = p.home[e];
              if (h == r) continue;
              bool taken = false;
              for (int32_t kk = 0; kk < k; ++kk) taken |= sl.assigned[(int64_t)rc * K + kk] == ec;
              if (taken) continue;
              const double q = (double)(spl < sp ? spl : sp);
              const double t1 = alpha * p.Bpref[(int64_t)h * R + r];
              const double ex = (double)excess[h];
              const double tn = (double)Tb[(int64_t)h * R + r] / (ex > kEps0 ? ex : kEps0);
              const double t2 = a2 * tn;
              const double score = (q + t1) + t2;
              if (score > bs) { bs = score; best = ec; }
            }
          }
          sl.prop_e[rc] = best;
          sl.prop_s[rc] = bs;
          proposed |= best >= 0;
        }
        if (!block_any(proposed, wave_cnt)) break;  // nothing can change any more
        // Steps 2-3: each proposed expert keeps its best proposer (lowest rank on ties)
        for (int32_t ec = tid; ec < ne; ec += kSchThreads) {
          int32_t w = -1;
          double ws = -INFINITY;
          for (int32_t rc = 0; rc < nc; ++rc)
            if (sl.prop_e[rc] == ec && sl.prop_s[rc] > ws) { ws = sl.prop_s[rc]; w = rc; }
          sl.win[ec] = w;
        }
        __syncthreads();
        // Step 4: winners take g = min(spill, spare) into slot k of their rank
        for (int32_t ec = tid; ec < ne; ec += kSchThreads) {
          const int32_t w = sl.win[ec];
          if (w < 0) continue;
          const int64_t g = sl.spill_p[ec] < sl.spare_p[w] ? sl.spill_p[ec] : sl.spare_p[w];
          sl.spill_p[ec] -= g;
          sl.spare_p[w] -= g;
          sl.matched[w] = 1;
          sl.assigned[(int64_t)w * K + k] = ec;
          const int64_t s = (int64_t)sl.cr[w] * K + k;
          se[s] = sl.ce[ec];
          sa[s] += g;
        }
        __syncthreads();
        ++used2;
      }
    }

    // ---- Phase 3: Lagrangian auction --------------------------------------------
    for (int32_t e = tid; e < E; e += kSchThreads) sl.dmap[e] = 0;
    __syncthreads();
    for (int64_t s = tid; s < S; s += kSchThreads)
      if (se[s] >= 0) sl.dmap[se[s]] = 1;
    __syncthreads();
    int32_t D = 0;
    for (int32_t base = 0; base < E; base += kSchThreads) {
      const int32_t e = base + tid;
      const bool f = e < E && sl.dmap[e] == 1;
      int32_t tot;
      const int32_t pos = compact_pos(f, wave_cnt, tot);
      if (e < E) sl.dmap[e] = f ? D + pos : -1;
      if (f) sl.dexp[D + pos] = e;
      D += tot;
    }
    __syncthreads();
    const int32_t* nb = p.n + b * (int64_t)R * E;
    for (int64_t q = tid; q < (int64_t)D * R; q += kSchThreads) {
      const int32_t d = (int32_t)(q / R), r = (int32_t)(q % R);
      sl.nprime[q] = nb[(int64_t)r * E + sl.dexp[d]];
    }
    for (int64_t s = tid; s < S; s += kSchThreads) {
      const int32_t e = se[s];
      sl.Ap[s] = e >= 0 ? sa[s] : 0;
      sl.dsl[s] = e >= 0 ? sl.dmap[e] : -1;
      sl.need[s] = 1;
      sl.bid[s] = -1;
    }
    for (int32_t r = tid; r < R; r += kSchThreads) {
      price[r] = 0.0;
      rkey[r] = 0;
      rwin[r] = INT_MAX;
      served[r] = 0;
    }
    __syncthreads();

    const int64_t tmax = p.t_max > 0 ? p.t_max : S * (R + 1);
    int64_t rounds = 0;
    for (int64_t t = 1; t <= tmax; ++t) {
      // (a) slots whose bid must be recomputed
      int32_t nw = 0;
      for (int64_t base = 0; base < S; base += kSchThreads) {
        const int64_t s = base + tid;
        const bool f = s < S && sl.Ap[s] > 0 && sl.dsl[s] >= 0 && sl.need[s];
        int32_t tot;
        const int32_t pos = compact_pos(f, wave_cnt, tot);
        if (f) sl.work[nw + pos] = (int32_t)s;
        nw += tot;
      }
      // the list (in the slab, device memory) is read by other waves below:
      // without this barrier a wave can read an entry of the previous round's
      // list, and a slot that must bid again keeps its old bid for a round
      __syncthreads();
      // one wave per slot: argmax over ranks r with tokens of the slot's expert
      // of Bauct[r][host] - price[r], lowest r on ties
      for (int32_t w = wid; w < nw; w += kSchWaves) {
        const int32_t s = sl.work[w];
        const int32_t host = s / K;
        const int32_t* np_ = sl.nprime + (int64_t)sl.dsl[s] * R;
        double bs = -INFINITY;
        int32_t br = INT_MAX;
        for (int32_t r = lane; r < R; r += kWave) {
          if (np_[r] <= 0) continue;
          const double sc = p.Bauct[(int64_t)r * R + host] - price[r];
          if (sc > bs) { bs = sc; br = r; }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          const double os = __shfl_xor(bs, o, kWave);
          const int32_t orr = __shfl_xor(br, o, kWave);
          if (os > bs || (os == bs && orr < br)) { bs = os; br = orr; }
        }
        if (lane == 0) {
          sl.bid[s] = br == INT_MAX ? -1 : br;
          sl.bid_s[s] = bs;
          sl.need[s] = 0;
        }
      }
      __syncthreads();
      // (b) each rank keeps its best bidder: max score, then lowest slot
      bool any = false;
      for (int64_t s = tid; s < S; s += kSchThreads) {
        if (sl.Ap[s] > 0 && sl.bid[s] >= 0) {
          atomicMax(reinterpret_cast<unsigned long long*>(&rkey[sl.bid[s]]),
                    (unsigned long long)auction_key(sl.bid_s[s]));
          any = true;
        }
      }
      if (!block_any(any, wave_cnt)) break;  // no bid: the state is final
      for (int64_t s = tid; s < S; s += kSchThreads) {
        if (sl.Ap[s] > 0 && sl.bid[s] >= 0 && auction_key(sl.bid_s[s]) == rkey[sl.bid[s]])
          atomicMin(&rwin[sl.bid[s]], (int32_t)s);
      }
      __syncthreads();
      // (c) transfers; a rank that moved tokens raises its price
      for (int32_t r = tid; r < R; r += kSchThreads) {
        const int32_t s = rwin[r];
        int32_t did = 0;
        if (s != INT_MAX) {
          int32_t* np_ = sl.nprime + (int64_t)sl.dsl[s] * R + r;
          const int64_t have = *np_;
          const int64_t x = have < sl.Ap[s] ? have : sl.Ap[s];
          Xb[(int64_t)r * S + s] += (int32_t)x;
          *np_ -= (int32_t)x;
          sl.Ap[s] -= x;
          if (x > 0) price[r] = price[r] + p.price_step;
          did = 1;
        }
        served[r] = did;
        rkey[r] = 0;
        rwin[r] = INT_MAX;
      }
      __syncthreads();
      // (d) a slot re-bids if its rank served or ran out of the slot's expert
      for (int64_t s = tid; s < S; s += kSchThreads) {
        const int32_t r = sl.bid[s];
        if (sl.Ap[s] > 0 && r >= 0 && (served[r] || sl.nprime[(int64_t)sl.dsl[s] * R + r] <= 0))
          sl.need[s] = 1;
      }
      __syncthreads();
      rounds = t;
    }

    // ---- outputs -----------------------------------------------------------------
    __shared__ int64_t red[kSchWaves];
    int64_t left = 0;
    for (int64_t s = tid; s < S; s += kSchThreads) left += sl.Ap[s];
    left = wave_sum_i64(left);
    if (lane == 0) red[wid] = left;
    __syncthreads();
    if (tid == 0) {
      int64_t tot = 0;
      for (int w = 0; w < kSchWaves; ++w) tot += red[w];
      p.unfilled[b] = tot;
      if (p.rounds_used) { p.rounds_used[2 * b] = used2; p.rounds_used[2 * b + 1] = (int32_t)rounds; }
      if (p.status) p.status[b] = tot > 0 ? TAOT_ST_UNFILLED : 0u;
    }
    __syncthreads();
  }
}


// ===========================================================================
// LDS-resident path.  Same arithmetic and order as schedule_kernel, with one
// workgroup per problem and all of its state in LDS and registers.  Three size
// configurations: one wave for R <= 64 and R*K <= 256, 256 threads for R <= 256
// and R*K <= 1024 (several problems per compute unit in both), 1024 threads for
// R <= 1024 and R*K <= 4096.  One wave runs matching and auction in one kernel;
// the others run the matching (36 to 100 KiB of LDS at R > 256) and then the
// auction in a kernel of its own (103 to 156 KiB there: one problem per compute
// unit).  All need bonuses (Bauct columns) that take few distinct values, as
// topology costs do.
//
// Phase-3 bids by tiers.  The ranks of host column h split into tiers of equal
// bonus (descending).  With prices that start at 0 and rise by a fixed step on
// each service, a rank's price is a function of its service count, and when
// the step is large against the spacing of doubles at the magnitudes reached,
// bonus - price falls strictly with every service.  Within a tier the argmax
// of the score is then the lowest-index rank among those with the fewest
// services.  Every service raises one count by one and the counts of all
// ranks stay close together, so the kernel keeps them relative to a base
// (the fewest services of any rank): the rank set at the base count, and the
// bit-planes of min(count - base, kRelMax), the relative code.  A tier's
// fewest-services candidate is its lowest rank at the base count when there
// is one, else the lowest rank of the smallest relative code (a bit-sliced
// minimum over the four code planes, words jointly), and when every
// candidate's code is saturated, the bit-sliced minimum over the planes of
// the full counts.  The bid is the best tier result under (max score, lowest
// rank).  No rank's price is below the price P0 of the base count, so a tier
// whose bonus minus P0 is below the best score so far cannot win, nor can any
// later (lower) tier.  A price step of 0 keeps every count and price at 0
// (every rank stays at the base count), and the argmax is the lowest rank of
// the first non-empty tier.
//
// Phase-3 arbitration by bonus.  Every live bid on rank r was placed at r's
// current price (a slot re-bids when its rank serves), so among r's bidders
// the score order is the order of their bonuses when distinct bonuses stay
// distinct after subtracting any reachable price.  A rank's winner is then the
// maximum of the 32-bit key (bonus rank, -slot), taken with one atomicMax.
//
// A prepass checks these conditions on the device and sends problems to
// schedule_kernel when they fail, as it does problems whose candidate or
// slot-expert counts exceed the LDS layout.

constexpr int kTierMax = 4;  // distinct bonus values per host column
constexpr int kRelPlanes = 4;                       // bit-planes of the relative code
constexpr int kRelMax = (1 << kRelPlanes) - 1;      // saturated code: count - base >= kRelMax

struct LdsSmall {
  static constexpr int kT = 256;     // threads per problem
  static constexpr int kTW = 4;      // 64-rank words of a rank set (R <= 256)
  static constexpr int kSC = 32;     // distinct host tier structures in LDS
  static constexpr int kDC = 64;     // distinct slot experts per problem
  static constexpr int kPL = 11;     // count bit-planes: counts <= R*K <= 1024
  static constexpr int kMaxS = 1024; // R*K
  static constexpr int kNEC = 128;   // candidate experts (spill > 0) in LDS
  static constexpr int kWavesPerEU = 8;  // large batches: eight problems per compute unit (17 KB of LDS each at R = 256, K = 2)
  static constexpr int kG = 2;       // bid groups per lane that the auction keeps in registers
  static constexpr int kAW = 1;      // waves of the auction while its list is long
};
struct LdsTiny {
  static constexpr int kT = 64;      // one wave per problem: its barriers cost next to nothing
  static constexpr int kTW = 1;      // R <= 64
  static constexpr int kSC = 64;
  static constexpr int kDC = 64;
  static constexpr int kPL = 9;      // counts <= R*K <= 256
  static constexpr int kMaxS = 256;
  static constexpr int kNEC = 128;
  static constexpr int kWavesPerEU = 8;
  static constexpr int kG = 1;
  static constexpr int kAW = 1;
};
struct LdsLarge {
  static constexpr int kT = 1024;
  static constexpr int kTW = 16;     // R <= 1024
  static constexpr int kSC = 128;
  static constexpr int kDC = 128;
  static constexpr int kPL = 13;     // counts <= R*K <= 4096
  static constexpr int kMaxS = 4096;
  static constexpr int kNEC = 1024;
  static constexpr int kWavesPerEU = 1;  // the auction, one problem per compute unit, is the longer part by far
  static constexpr int kG = 3;
  static constexpr int kAW = 8;
};
// The count window's rebuild takes rank r on thread r (wave w builds word w).
static_assert(LdsSmall::kT == LdsSmall::kTW * kWave && LdsTiny::kT == LdsTiny::kTW * kWave &&
                  LdsLarge::kT == LdsLarge::kTW * kWave,
              "one thread per rank of the largest R of each configuration");
// list entries pack (slot, slot-expert index, host structure): 12 + 7 + 7 bits
constexpr int kItemSlotBits = 12, kItemExpertBits = 7;

// Exclusive position of `flag` among the NT threads (ascending thread id) and
// the chunk total.  All threads must call it.
template <int NT>
__device__ __forceinline__ int32_t compact_pos_n(bool flag, int32_t* wave_cnt, int32_t& total) {
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const uint64_t m = __ballot(flag);
  const int32_t lp = __popcll(m & ((1ull << lane) - 1ull));
  if (lane == 0) wave_cnt[wid] = __popcll(m);
  __syncthreads();
  int32_t off = 0, tot = 0;
  for (int w = 0; w < NW; ++w) {
    const int32_t c = wave_cnt[w];
    off += w < wid ? c : 0;
    tot += c;
  }
  __syncthreads();
  total = tot;
  return off + lp;
}

// Tier structure of column h of Bauct: its distinct bonuses in descending
// order and the rank set of each ([h][kTierMax][TW] words); ntier[h] = -1 if
// there are more than kTierMax.  NaN and -inf bonuses never win a bid and
// belong to no tier; -0 and +0 are one value.  The distinct values come out
// one per step as a block maximum over the values below the previous one
// (order-preserving 64-bit keys).
__device__ __forceinline__ double key_double(uint64_t k) {
  return __longlong_as_double((long long)((k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k));
}

template <int NT>
__device__ __forceinline__ uint64_t block_max_u64(uint64_t v, uint64_t* buf) {
  constexpr int NW = NT / kWave;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t y = __shfl_xor(v, o, kWave);
    v = y > v ? y : v;
  }
  if ((threadIdx.x & (kWave - 1)) == 0) buf[threadIdx.x / kWave] = v;
  __syncthreads();
  uint64_t m = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) m = buf[w] > m ? buf[w] : m;
  __syncthreads();
  return m;
}

template <int TW>
__global__ void __launch_bounds__(256)
auction_tiers_kernel(const double* __restrict__ Bauct, int32_t R, int32_t* __restrict__ ntier,
                     double* __restrict__ tv, uint64_t* __restrict__ tmask) {
  __shared__ double col[TW * kWave];
  __shared__ double vals[kTierMax];
  __shared__ uint64_t red[256 / kWave];
  __shared__ unsigned long long msk[kTierMax * TW];
  const int32_t h = blockIdx.x, tid = threadIdx.x;
  for (int32_t q = tid; q < kTierMax * TW; q += blockDim.x) msk[q] = 0ull;
  for (int32_t r = tid; r < R; r += blockDim.x) col[r] = Bauct[(int64_t)r * R + h];
  __syncthreads();
  // the tier bonuses, descending: key 0 is below every value's key
  uint64_t prev = ~0ull;
  int32_t n = 0;
  for (int t = 0; t <= kTierMax; ++t) {
    uint64_t m = 0;
    for (int32_t r = tid; r < R; r += blockDim.x) {
      const double v = col[r];
      if (v != v || v == -INFINITY) continue;
      const uint64_t k = auction_key(v);
      if (k < prev && k > m) m = k;
    }
    m = block_max_u64<256>(m, red);
    if (m == 0) break;  // no value below the previous one
    if (t == kTierMax) { n = -1; break; }
    if (tid == 0) vals[t] = key_double(m);
    prev = m;
    n = t + 1;
  }
  __syncthreads();
  for (int32_t r = tid; r < R && n > 0; r += blockDim.x) {
    const double v = col[r];
    for (int32_t i = 0; i < n; ++i)
      if (vals[i] == v) atomicOr(&msk[i * TW + (r >> 6)], 1ull << (r & 63));
  }
  __syncthreads();
  if (tid == 0) ntier[h] = n;
  if (tid < kTierMax) tv[(int64_t)h * kTierMax + tid] = tid < n ? vals[tid] : -INFINITY;
  for (int32_t q = tid; q < kTierMax * TW; q += blockDim.x)
    tmask[(int64_t)h * kTierMax * TW + q] = q / TW < n ? msk[q] : 0ull;
}

// Deduplicates the host tier structures into a table of at most SC entries
// (one block, one thread per host; equal structures are found through a hash
// of each and then compared in full; the table keeps first occurrences in
// host order) and ranks the table's distinct bonuses (ascending, one per step
// as a block minimum above the previous one): sidx[h] is host h's entry, cw
// the words that hold ranks of each tier, cvr the bonus rank of each tier,
// hdr[0] the table size and hdr[1] = 1 when the LDS-resident auction is exact
// for this Bauct and price step: every column has at most kTierMax values,
// none is +inf, the table fits, and both the step (if not 0) and every gap
// between distinct bonuses exceed twice the spacing of doubles at max|bonus|
// + S * step (prices stay below S * step: a rank serves each slot at most
// once).
template <class CF>
__global__ void __launch_bounds__(CF::kT)
auction_struct_kernel(const int32_t* __restrict__ ntier_g, const double* __restrict__ tv_g,
                      const uint64_t* __restrict__ tmask, int32_t R, int64_t S, double step,
                      int32_t* __restrict__ sidx, int32_t* __restrict__ cn, double* __restrict__ cv,
                      int32_t* __restrict__ cvr, uint32_t* __restrict__ cw, uint64_t* __restrict__ cm,
                      int32_t* __restrict__ hdr) {
  constexpr int NT = CF::kT;
  constexpr int kRow = kTierMax * CF::kTW;
  constexpr int kMaxR = CF::kTW * kWave;
  constexpr int kMaxDv = CF::kSC * kTierMax;
  static_assert(NT >= kMaxR, "one thread per host");
  __shared__ int32_t ntier[kMaxR], first[kMaxR], sid[kMaxR], tab[CF::kSC];
  __shared__ uint64_t hsh[kMaxR];
  __shared__ double tv[kMaxR * kTierMax];
  __shared__ double dv[kMaxDv];
  __shared__ uint64_t red[NT / kWave];
  __shared__ int32_t wave_cnt[NT / kWave];
  const int32_t h = threadIdx.x;
  for (int32_t q = h; q < R * kTierMax; q += NT) tv[q] = tv_g[q];
  if (h < R) {
    const int32_t nh = ntier_g[h];
    ntier[h] = nh;
    uint64_t x = 0x9E3779B97F4A7C15ull ^ (uint64_t)(uint32_t)nh;
    for (int32_t t = 0; t < kTierMax; ++t) {
      x = (x ^ (uint64_t)__double_as_longlong(tv_g[h * kTierMax + t])) * 0x100000001B3ull;
      x ^= x >> 29;
    }
    for (int32_t q = 0; q < kRow; ++q) {
      x = (x ^ tmask[(int64_t)h * kRow + q]) * 0x100000001B3ull;
      x ^= x >> 29;
    }
    hsh[h] = x;
  }
  __syncthreads();
  if (h < R) {
    const int32_t nh = ntier[h];
    int32_t f = h;
    for (int32_t g = 0; g < h && f == h; ++g) {
      if (hsh[g] != hsh[h] || ntier[g] != nh) continue;
      bool eq = true;
      for (int32_t t = 0; t < kTierMax && eq; ++t) eq = tv[g * kTierMax + t] == tv[h * kTierMax + t];
      for (int32_t q = 0; q < kRow && eq; ++q) eq = tmask[(int64_t)g * kRow + q] == tmask[(int64_t)h * kRow + q];
      if (eq) f = g;
    }
    first[h] = f;
  }
  __syncthreads();
  // table entries: the first occurrences in host order
  int32_t ns;
  {
    const bool f = h < R && first[h] == h;
    const int32_t pos = compact_pos_n<NT>(f, wave_cnt, ns);
    if (f) {
      sid[h] = pos;
      if (pos < CF::kSC) tab[pos] = h;
    }
  }
  __syncthreads();
  if (h < R && first[h] != h) sid[h] = sid[first[h]];
  // exactness conditions over all hosts: at most kTierMax values per column,
  // no +inf, and max |bonus|
  bool okh = true;
  uint64_t vmk = 0;  // bits of max |bonus| (non-negative doubles order as integers)
  if (h < R) {
    okh = ntier[h] >= 0;
    for (int32_t t = 0; t < ntier[h]; ++t) {
      const double v = tv[h * kTierMax + t];
      okh &= v != INFINITY;
      const uint64_t a = (uint64_t)__double_as_longlong(fabs(v));
      vmk = a > vmk ? a : vmk;
    }
  }
  const bool all_ok = block_max_u64<NT>(okh ? 0ull : 1ull, red) == 0ull;
  const double vm = __longlong_as_double((long long)block_max_u64<NT>(vmk, red));
  // distinct bonuses of the table, ascending: value q is tier q % kTierMax of
  // entry q / kTierMax, dealt out over the threads
  const int32_t nt_tab = ns < CF::kSC ? ns : CF::kSC;
  int32_t nd = 0;
  {
    uint64_t prev = 0;  // keys above this; the smallest first
    for (;;) {
      // minimum key above prev, as a maximum of complements
      uint64_t c = 0;
      for (int32_t q = h; q < nt_tab * kTierMax; q += NT) {
        const int32_t g = tab[q / kTierMax], t = q % kTierMax;
        if (t >= ntier[g]) continue;
        const uint64_t k = auction_key(tv[g * kTierMax + t]);
        if (k > prev && ~k > c) c = ~k;
      }
      const uint64_t m = block_max_u64<NT>(c, red);
      if (m == 0) break;
      const uint64_t kmin = ~m;
      if (h == 0 && nd < kMaxDv) dv[nd] = key_double(kmin);
      prev = kmin;
      ++nd;
    }
  }
  __syncthreads();
  if (h == 0) {
    bool ok = all_ok && ns <= CF::kSC;
    const double top = vm + (double)S * step * 1.01 + 1.0;
    const double spacing2 = 2.0 * (nextafter(top, INFINITY) - top);
    ok &= step == 0.0 || (step > 0.0 && step > spacing2);
    for (int32_t i = 0; i + 1 < nd; ++i) ok &= dv[i + 1] - dv[i] > spacing2;
    hdr[0] = nt_tab;
    hdr[1] = ok ? 1 : 0;
  }
  // bonus ranks of the table's tiers
  for (int32_t q = h; q < nt_tab * kTierMax; q += NT) {
    const int32_t g = tab[q / kTierMax], t = q % kTierMax;
    int32_t rank = 0;
    if (t < ntier[g]) {
      const double v = tv[g * kTierMax + t];
      while (dv[rank] != v) ++rank;
    }
    cvr[q] = rank;
  }
  for (int32_t q = h; q < R; q += NT) sidx[q] = sid[q];
  for (int32_t q = h; q < nt_tab; q += NT) cn[q] = ntier[tab[q]] > 0 ? ntier[tab[q]] : 0;
  for (int32_t q = h; q < nt_tab * kTierMax; q += NT) {
    const int32_t g = tab[q / kTierMax], t = q % kTierMax;
    cv[q] = tv[g * kTierMax + t];
    uint32_t words = 0;
    for (int32_t w = 0; w < CF::kTW; ++w) words |= (tmask[(int64_t)g * kRow + t * CF::kTW + w] != 0ull ? 1u : 0u) << w;
    cw[q] = words;
  }
  for (int32_t q = h; q < nt_tab * kRow; q += NT) cm[q] = tmask[(int64_t)tab[q / kRow] * kRow + q % kRow];
}

template <class CF>
struct LdsState {
  // both phases
  int16_t* slot_ec;   // [S] candidate index of the slot's expert or -1
  int32_t* amt;       // [S] slot amounts (Phase 2), tokens still planned (Phase 3)
  int32_t* ce;        // [NEC] candidate experts (spill > 0), ascending
  // Phase 2
  int32_t* hce; double* den; int32_t* cr; int32_t* spare_p; int32_t* matched; int32_t* prop_e;
  double* prop_s; int32_t* assigned; int32_t* spill_p; uint64_t* ekey; int32_t* ewin;
  int32_t* qbest;  // [R] q = min(spill, spare) of each cold rank's standing proposal
  // Phase 3 (aliases the Phase-2 region)
  double* price; uint32_t* rkey; int32_t* work; uint16_t* sstate;
  uint64_t* vmask; uint32_t* vwords; int32_t* dexp; int32_t* dmap; int32_t* cnt; uint64_t* planes;
  // relative counts: lvl [2][TW] the ranks at the base count and those one
  // service above it, rel [kRelPlanes] [TW] the code planes
  uint64_t* lvl; uint64_t* rel;
  int8_t* cn; double* cv; int32_t* cvr; uint32_t* cw; uint64_t* cm;
  size_t bytes;
};

template <class CF>
__host__ __device__ inline LdsState<CF> carve_lds(char* base, int32_t R, int32_t K, int32_t NEC) {
  LdsState<CF> w{};
  const size_t S1 = R * K > 0 ? (size_t)R * K : 1, R_ = (size_t)R, N_ = (size_t)NEC;
  constexpr size_t TW = CF::kTW, SC = CF::kSC, DC = CF::kDC;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* q = base + off;
    off = (off + bytes + 15) & ~(size_t)15;
    return q;
  };
  w.slot_ec = (int16_t*)take(2 * S1);
  w.amt = (int32_t*)take(4 * S1);
  w.ce = (int32_t*)take(4 * N_);
  const size_t split = off;
  w.hce = (int32_t*)take(4 * N_); w.den = (double*)take(8 * R_); w.cr = (int32_t*)take(4 * R_);
  w.spare_p = (int32_t*)take(4 * R_); w.matched = (int32_t*)take(4 * R_); w.prop_e = (int32_t*)take(4 * R_);
  w.prop_s = (double*)take(8 * R_); w.assigned = (int32_t*)take(4 * S1);
  w.spill_p = (int32_t*)take(4 * N_); w.ekey = (uint64_t*)take(8 * N_); w.ewin = (int32_t*)take(4 * N_);
  w.qbest = (int32_t*)take(4 * R_);
  const size_t end2 = off;
  off = split;
  w.work = (int32_t*)take(4 * S1);
  // the list entries' bid states, by list position, over the candidates' slot
  // expert indices (read last when the list's items are built)
  w.dmap = (int32_t*)take(2 * S1 > 4 * N_ ? 2 * S1 : 4 * N_);
  w.sstate = (uint16_t*)w.dmap;
  // the word lists guide the per-word search of sets wider than 4 words only
  w.vmask = (uint64_t*)take(8 * DC * TW); w.vwords = (uint32_t*)take(TW > 4 ? 4 * DC : 0);
  w.dexp = (int32_t*)take(4 * DC);
  if constexpr (CF::kT == kWave) {  // the auction follows in the same kernel
    w.price = (double*)take(8 * R_); w.rkey = (uint32_t*)take(4 * R_);
    w.cnt = (int32_t*)take(4 * R_); w.planes = (uint64_t*)take(8 * CF::kPL * TW);
    w.lvl = (uint64_t*)take(2 * 8 * TW);
    w.rel = (uint64_t*)take(8 * kRelPlanes * TW);
    w.cn = (int8_t*)take(SC);
    w.cv = (double*)take(8 * SC * kTierMax); w.cvr = (int32_t*)take(4 * SC * kTierMax);
    w.cw = (uint32_t*)take(4 * SC * kTierMax);
    w.cm = (uint64_t*)take(8 * SC * kTierMax * TW);
  }
  w.bytes = end2 > off ? end2 : off;
  return w;
}

// What the matching kernel leaves for the auction's: per problem a header
// (listed groups, or -1: not for the auction; Phase-2 iterations; slot
// experts), tokens planned, next slots of the bid groups, list items [S]; most
// tokens and valid words [DC], valid ranks [DC][TW] of the slot experts.
struct Handoff {
  int4* hdr;        // [B]
  int32_t* amt;     // [B][S]
  int32_t* work;    // [B][S]
  int16_t* gnext;   // [B][S]
  int32_t* nmax;    // [B][DC]
  uint32_t* vwords; // [B][DC]
  uint64_t* vmask;  // [B][DC][TW]
};

struct LdsParams {
  SchParams s;
  Handoff h;
  const int32_t* sidx;   // [R] host -> tier structure
  const int32_t* cn;     // [SC] tiers per structure
  const double* cv;      // [SC][kTierMax] tier bonuses, descending
  const int32_t* cvr;    // [SC][kTierMax] rank of each tier bonus among the table's
  const uint32_t* cw;    // [SC][kTierMax] words holding ranks of the tier
  const uint64_t* cm;    // [SC][kTierMax][TW] tier rank sets
  const int32_t* hdr;    // [0] structures, [1] LDS-resident auction exact
  int32_t* fallback;     // [B] 1 = left to schedule_kernel
  int32_t* nprime;       // [B][DC][R]
  int32_t NEC;           // candidate-expert capacity of the LDS layout
};

// Block-wide OR with one barrier; flags alternate between two halves of buf
// ([2][NT / 64]) so that a call never overwrites flags still being read.
template <int NT>
__device__ __forceinline__ bool block_or(bool flag, int32_t* buf, int& parity) {
  constexpr int NW = NT / kWave;
  const uint64_t m = __ballot(flag);
  if ((threadIdx.x & (kWave - 1)) == 0) buf[parity * NW + threadIdx.x / kWave] = m != 0;
  __syncthreads();
  bool any = false;
#pragma unroll
  for (int w = 0; w < NW; ++w) any |= buf[parity * NW + w] != 0;
  parity ^= 1;
  return any;
}

// Appends the flagged items of a wave to a list whose length lives in LDS
// (*count); the order of the list is unspecified.  All lanes must call it;
// a flagged lane gets its item's position.
__device__ __forceinline__ int32_t list_append(bool flag, int32_t item, int32_t* list, int32_t* count) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t m = __ballot(flag);
  int32_t base = 0;
  if (lane == 0 && m) base = atomicAdd(count, __popcll(m));
  base = __builtin_amdgcn_readlane(base, 0);
  const int32_t pos = base + __popcll(m & ((1ull << lane) - 1ull));
  if (flag) list[pos] = item;
  return pos;
}

template <int CTRL>
__device__ __forceinline__ int32_t dpp_i32(int32_t x) {
  // every lane has a source lane for the patterns used here
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
// Max over the 64 lanes without LDS round trips: DPP steps within each
// 16-lane row, then the permlane16 and permlane32 swaps across rows.  All
// lanes must call it.
__device__ __forceinline__ int32_t wave_max_i32(int32_t v) {
  v = max(v, dpp_i32<0xB1>(v));   // quad_perm [1,0,3,2]
  v = max(v, dpp_i32<0x4E>(v));   // quad_perm [2,3,0,1]
  v = max(v, dpp_i32<0x141>(v));  // row_half_mirror
  v = max(v, dpp_i32<0x140>(v));  // row_mirror
  const auto r16 = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  v = max((int32_t)r16[0], (int32_t)r16[1]);
  const auto r32 = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  return max((int32_t)r32[0], (int32_t)r32[1]);
}

// Where word w of row `row` of a table of rank sets stands in its row.
template <int TW>
__device__ __forceinline__ int set_word(int32_t row, int w) {
  return w ^ (row & (TW - 1));
}

// Where the rounds of an auction stand: the next round, the list's length, the
// base count, the ranks at it, the epoch's parity, the base count's price,
// whether the planes of the full counts are kept, whether no bid was left.
struct AuctionRun {
  int64_t t;
  int32_t nw, base, base_left;
  uint32_t epoch;
  double P0;
  bool planes_on, done;
};
// What the waves of one auction share, in LDS: two counts of live groups (by the
// round's parity), ranks left at the base count, planes_on, the list's length.
constexpr int kShLive = 0, kShLeft = 2, kShPlanes = 3, kShList = 4, kShWords = 5;
// Up to this many groups one wave goes on alone.
constexpr int32_t kAuctionAlone = 64;

// Barrier for LDS alone: loads and stores of device memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The rounds of the auction from `run` on: on one wave to the end, or on NW
// waves until one wave can go on alone.
//
// Every bid names a rank, which then serves its best bidder with a positive
// amount; so every group with an open slot and a valid rank bids again in
// every round.  A group drops out once its slots are full or it finds no valid
// rank (validity only ends).  A round is
//   X: each listed group bids and posts a key to the rank it bid for;
//   Y: a group whose key stands moves tokens; the others lose.
// A round without a bid ends the auction.
//
// What bounds it: the rounds follow from one another (about 1200 at R = 256,
// 10000 at R = 1024) and hold few transfers (4 to 6) for the list they walk,
// so a round costs its chain of latencies.  One wave runs it without a barrier,
// as the LDS operations of a wave stay in order; lists of up to 64 kG groups
// stay in registers, kG to a lane, longer ones are walked 64 at a time.
//
// Above R = 256 a list can hold a thousand groups, and a wave's round over it
// grows with it.  There kAW waves hold the list in registers, with a barrier
// behind X and one behind Y, until kAuctionAlone groups are left.  64 x R = 1024,
// K = 2, lists of about 410: 24.0 ms a call on one wave, 20.9 with eight waves
// down to 256 groups, 16.2 down to 64; 16 problems of R = 1024 with 950 groups
// each: 21.5 ms on one wave, 17.0 and 13.8.  Four waves with five groups a lane:
// 15.0; sixteen with two: 13.8.
//
// Incremental bids.  Within an epoch (while the base count stays) a group keeps
// its first tier ts that holds a valid rank, the fewest services lev (above the
// base count) among that tier's valid ranks, and the lowest 64-rank word w of
// the tier with a valid rank that has them.  Its bid is the lowest such rank of
// the word.  All three only move forward: validity only ends and counts only
// rise, so a rank can reach lev services only from fewer, which no valid rank of
// the tier has.  A rank that drains for the group's expert was served and left
// the level with that, so the word's valid ranks (win) need not be read again
// while the level lasts.  When the word runs out the search goes on from it, and
// when the level does, it looks for the tier's smallest relative code.  Prices
// are functions of the count, so whether a later tier can reach the bid's score
// is settled for as long as the level lasts; only a group for which none can
// keeps its state (has).  Empty tiers stay empty: ts holds across epochs.
//
// Transfers.  A slot that plans more than any rank holds of its expert (nmax)
// takes all that the rank has, so its round does not wait for the count to
// arrive from device memory: the lane keeps the load in flight and books it
// with its next transfer.
//
// List entries: slot, slot-expert index, host structure (0-25); negative: none.
// Entry states: w (0-3), ts (4-5), lev (6-9), has (10), epoch parity (11: a
// listed group's state is rewritten in every round that does not bid from it,
// and the base moves at most once per round).  Between the two steps of a round
// over a longer list the spare bits hold the bit of the bid's rank in word w:
// two bits in the entry (26-27), four in the state (12-15).
template <class CF, int NW>
__device__ __forceinline__ void auction_rounds(const LdsState<CF>& L, AuctionRun& run, int32_t* sh,
                                               const int16_t* gnext, int32_t* np, int32_t* Xb, int32_t R, int32_t S,
                                               double step, int64_t tmax) {
  constexpr int TW = CF::kTW;
  constexpr int G = NW == 1 && CF::kAW > 1 ? kAuctionAlone / kWave : CF::kG;  // groups of a lane
  constexpr int32_t kSlotMask = (1 << kItemSlotBits) - 1, kExpMask = (1 << kItemExpertBits) - 1;
  constexpr int32_t kItemBits = 26, kItemMask = (1 << kItemBits) - 1;
  constexpr int32_t kStructMask = (1 << (kItemBits - kItemSlotBits - kItemExpertBits)) - 1;
  // a matched slot uses up its rank's spare or its expert's spill: no more slots than ranks and slot experts
  static_assert(NW == 1 || NW * kWave * G >= CF::kTW * kWave + CF::kDC, "the waves hold every list");
  constexpr uint32_t kHas = 1u << 10, kStateMask = (1u << 12) - 1u;
  static_assert(TW <= 16 && kTierMax <= 4 && kRelMax <= 15 && CF::kSC <= kStructMask + 1, "entry and state fields");
  const int lane = threadIdx.x & (kWave - 1);
  const bool track = step > 0.0;  // counts order the prices; with step 0 all prices stay 0
  uint32_t* rk = L.rkey;
  const int32_t* nmax = L.dexp;
  const int wid = NW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : 0;
  double P0 = run.P0;             // price of the base count
  int32_t base = run.base, base_left = run.base_left, nw = run.nw;
  uint32_t epoch = run.epoch;     // parity
  bool planes_on = run.planes_on; // the planes of the full counts are kept from their first use on

  // word w of tier e = structure * kTierMax + tier, and of expert d's valid
  // ranks (rows of TW words, rotated so that the same word of different rows
  // does not sit in the same banks)
  auto tier_word = [&](int32_t e, int w) { return L.cm[e * TW + set_word<TW>(e / kTierMax, w)]; };
  auto valid_word = [&](int32_t d, int w) { return L.vmask[d * TW + set_word<TW>(d, w)]; };
  auto expert = [](int32_t it) { return (it >> kItemSlotBits) & kExpMask; };
  auto structure = [](int32_t it) { return (it >> (kItemSlotBits + kItemExpertBits)) & kStructMask; };
  // ranks of word w with exactly lev services above the base count
  auto level = [&](uint32_t lev, int w) {
    if (lev < 2u) return L.lvl[lev * TW + w];
    uint64_t m = ~0ull;
#pragma unroll
    for (int j = 0; j < kRelPlanes; ++j) m &= ((lev >> j) & 1u) ? L.rel[j * TW + w] : ~L.rel[j * TW + w];
    return m;
  };
  struct Bid {
    int32_t r, v;    // rank (-1: no valid rank is left), bonus rank
    uint32_t state;
    uint64_t win;    // valid ranks of the state's word
  };
  // The search from the entry's state on; stuck: every candidate's code is
  // saturated and the count planes are off.
  auto search = [&](int32_t it, uint32_t state, bool& stuck) {
    const int32_t d = expert(it), st = structure(it);
    const int32_t nt = L.cn[st];
    const uint32_t vw = TW > 4 ? L.vwords[d] : ~0u;
    const int32_t ts = (int32_t)(state >> 4) & 3;
    const bool same = (state & kHas) != 0u && (state >> 11) == epoch;
    double bs = -INFINITY;
    Bid b{-1, 0, state & (3u << 4), 0ull};
    int found = 0;  // tiers with a valid rank that were looked at
    for (int32_t ti = ts; ti < nt; ++ti) {
      const double v = L.cv[st * kTierMax + ti];
      if (found && v - P0 < bs) break;  // no score in this tier or the next reaches bs
      const int32_t e = st * kTierMax + ti;
      const uint32_t words = L.cw[e] & vw;
      const bool resume = same && ti == ts;
      const uint32_t lev = resume ? (state >> 6) & 15u : 0u;
      int32_t rr = -1;
      uint32_t code = lev;
      uint64_t win = 0ull;
      // the lowest valid rank at the base count or one service above it
      if (lev < 2u)
        for (uint32_t ws = resume ? words & (~0u << (state & 15u)) : words; ws; ws &= ws - 1u) {
          const int w = __builtin_ctz(ws);
          const uint64_t c = tier_word(e, w) & valid_word(d, w), h = c & L.lvl[lev * TW + w];
          if (h) {
            rr = w * kWave + __builtin_ctzll(h);
            win = c;
            break;
          }
        }
      if (rr < 0) {
        // the smallest relative code (words ascend: equal codes keep the lower rank)
        uint32_t best = kRelMax + 1;
        for (uint32_t ws = words; ws; ws &= ws - 1u) {
          const int w = __builtin_ctz(ws);
          const uint64_t all = tier_word(e, w) & valid_word(d, w);
          uint64_t c = all, p[kRelPlanes];
#pragma unroll
          for (int j = 0; j < kRelPlanes; ++j) p[j] = L.rel[j * TW + w];
          if (!c) continue;
          uint32_t cw = 0;
#pragma unroll
          for (int j = kRelPlanes - 1; j >= 0; --j) {
            const uint64_t m = c & ~p[j];
            if (m) c = m;
            else cw |= 1u << j;
          }
          if (cw < best) {
            best = cw;
            rr = w * kWave + __builtin_ctzll(c);
            win = all;
          }
        }
        if (rr < 0) continue;  // no valid rank in this tier
        code = best;
        if (code == (uint32_t)kRelMax && track) {
          stuck |= !planes_on;
          // all saturated: the smallest full count
          uint32_t cmin = 0xFFFFFFFFu;
          for (uint32_t ws = planes_on ? words : 0u; ws; ws &= ws - 1u) {
            const int w = __builtin_ctz(ws);
            uint64_t x = tier_word(e, w) & valid_word(d, w);
            if (!x) continue;
            uint32_t mn = 0;
            for (int32_t j = CF::kPL - 1; j >= 0; --j) {
              const uint64_t m = x & ~L.planes[j * TW + w];
              if (m) x = m;
              else mn |= 1u << j;
            }
            if (mn < cmin) {
              cmin = mn;
              rr = w * kWave + __builtin_ctzll(x);
            }
          }
        }
      }
      if (found == 0) {
        b.state = (uint32_t)(rr >> 6) | ((uint32_t)ti << 4) | (code << 6) | (epoch << 11) |
                  (track && code < (uint32_t)kRelMax ? kHas : 0u);
        b.win = win;
      }
      ++found;
      const double sc = v - (code == 0u ? P0 : L.price[rr]);
      if (sc > bs || (sc == bs && rr < b.r)) {
        bs = sc;
        b.r = rr;
        b.v = L.cvr[st * kTierMax + ti];
      }
    }
    if (found > 1) {  // the tiers compete: search again in the next round
      b.state = (b.state & (3u << 4)) | (uint32_t)(b.r >> 6);
    }
    return b;
  };
  // (wave-uniform) the search of the flagged lanes; the count planes come into
  // being when a lane first needs them
  auto search_all = [&](bool need, int32_t it, Bid& b) {
    bool stuck = false;
    Bid x = b;
    if (need) x = search(it, b.state, stuck);
    if (__ballot(stuck) != 0) {
      for (int w = 0; w < TW; ++w) {
        const int32_t r = w * kWave + lane;
        const int32_t c = r < R ? L.cnt[r] : 0;
        for (int j = 0; j < CF::kPL; ++j) {
          const uint64_t m = __ballot((c >> j) & 1);
          if (lane == 0) L.planes[j * TW + w] = m;
        }
      }
      planes_on = true;
      if constexpr (NW > 1)
        if (lane == 0) sh[kShPlanes] = 1;  // (another wave that makes them now writes the same)
      if (need) x = search(it, b.state, stuck);
    }
    b = x;
  };
  // The bookkeeping of a service of rank r, which had c0 services at price pr;
  // returns whether it leaves the base count.
  auto serve = [&](int32_t r, int32_t c0, double pr) {
    rk[r] = 0u;  // the rank's key is cleared for the next round
    L.price[r] = pr + step;
    if (!track) return false;
    const unsigned long long bit = 1ull << (r & 63);
    const int w = r >> 6;
    const int32_t c1 = c0 + 1, k0 = c0 - base;
    L.cnt[r] = c1;
    if (planes_on)
      for (uint32_t flip = (uint32_t)(c0 ^ c1); flip; flip &= flip - 1)
        atomicXor(reinterpret_cast<unsigned long long*>(&L.planes[__builtin_ctz(flip) * TW + w]), bit);
    // the relative code rises by one (below saturation)
    if (k0 < kRelMax)
      for (uint32_t flip = (uint32_t)(k0 ^ (k0 + 1)); flip; flip &= flip - 1)
        atomicXor(reinterpret_cast<unsigned long long*>(&L.rel[__builtin_ctz(flip) * TW + w]), bit);
    // the rank leaves the base count, enters (code 0 -> 1) or leaves (1 -> 2) the set one above it
    if (k0 == 0) atomicXor(reinterpret_cast<unsigned long long*>(&L.lvl[w]), bit);
    if (k0 <= 1) atomicXor(reinterpret_cast<unsigned long long*>(&L.lvl[TW + w]), bit);
    return k0 == 0;
  };
  // rank r holds no more tokens of slot expert d
  auto drained = [&](int32_t d, int32_t r) {
    const unsigned long long bit = 1ull << (r & 63);
    const int w = r >> 6;
    const uint64_t old = atomicAnd(reinterpret_cast<unsigned long long*>(&L.vmask[d * TW + set_word<TW>(d, w)]), ~bit);
    if constexpr (TW > 4)  // the word list only guides the search
      if ((old & ~bit) == 0ull) atomicAnd(&L.vwords[d], ~(1u << w));
  };
  // Every rank has left the base count: the base moves to the new fewest
  // services and the relative codes are rebuilt from the counts.
  auto rebase = [&]() {
    int32_t mn = INT_MAX;
    for (int32_t r = lane; r < R; r += kWave) mn = min(mn, L.cnt[r]);
    base = __builtin_amdgcn_readfirstlane(-wave_max_i32(-mn));
    base_left = 0;
    const bool writes = lane == 0 && wid == 0;
    for (int w = 0; w < TW; ++w) {
      const int32_t r = w * kWave + lane;
      const int32_t kr = r < R ? min(L.cnt[r] - base, kRelMax) : -1;
      const uint64_t m0 = __ballot(kr == 0), m1 = __ballot(kr == 1);
      if (writes) {
        L.lvl[w] = m0;
        L.lvl[TW + w] = m1;
      }
#pragma unroll
      for (int j = 0; j < kRelPlanes; ++j) {
        const uint64_t m = __ballot(kr > 0 && ((kr >> j) & 1));
        if (writes) L.rel[j * TW + w] = m;
      }
      // every rank at the new base has the same price
      if (m0 != 0ull) P0 = L.price[w * kWave + (int)__builtin_ctzll(m0)];
      base_left += (int32_t)__popcll(m0);
    }
    epoch ^= 1u;
  };

  int64_t t = run.t;
  if constexpr (CF::kAW == 1) {
  // ---- lists longer than a wave: entries and states in LDS -----------------------------
  int32_t active = nw;
  for (; t <= tmax && nw > G * kWave; ++t) {
    // X: bids
    int32_t nit = lane < nw ? L.work[lane] : -1;
    uint32_t nst = lane < nw ? L.sstate[lane] : 0u;
    int32_t bids = 0;
    for (int32_t q0 = 0; q0 < nw; q0 += kWave) {
      const int32_t q = q0 + lane, it = nit & (nit < 0 ? -1 : kItemMask);
      Bid b{-1, 0, nst & kStateMask, 0ull};
      if (q0 + kWave < nw) {  // the next entries, while these are looked at
        const bool in = q + kWave < nw;
        nit = in ? L.work[q + kWave] : -1;
        nst = in ? L.sstate[q + kWave] : 0u;
      }
      if (it >= 0 && (b.state & kHas) != 0u && (b.state >> 11) == epoch) {
        const int32_t d = expert(it);
        const int w = (int)(b.state & 15u), e = structure(it) * kTierMax + (int)((b.state >> 4) & 3u);
        const uint64_t h = tier_word(e, w) & valid_word(d, w) & level((b.state >> 6) & 15u, w);
        b.v = L.cvr[e];
        if (h) b.r = w * kWave + __builtin_ctzll(h);
      }
      const bool need = it >= 0 && b.r < 0;
      if (__ballot(need) != 0) search_all(need, it, b);
      if (it >= 0) {
        if (b.r >= 0) {
          atomicMax(&rk[b.r], ((uint32_t)b.v << 16) | (uint32_t)(0xFFFF - (it & kSlotMask)));
          L.sstate[q] = (uint16_t)(b.state | (uint32_t)((b.r & 63) >> 2) << 12);
          L.work[q] = it | (b.r & 3) << kItemBits;
        } else {
          L.work[q] = -1;  // no valid rank is left
        }
      }
      bids += (int32_t)__popcll(__ballot(b.r >= 0));
    }
    if (bids == 0) {  // no bid: the state is final
      run.t = t;
      run.done = true;
      return;
    }
    active = bids;
    // Y: the winners of all entries, gathered a lane each, then their transfers
    int32_t wq = -1, have_n = 0;
    auto transfers = [&]() {
      bool left_base = false;
      if (wq >= 0) {
        int32_t it = L.work[wq];
        const uint32_t state = L.sstate[wq];
        const int32_t r = (int32_t)(state & 15u) * kWave + (int32_t)(state >> 12) * 4 + ((it >> kItemBits) & 3);
        it &= kItemMask;
        const int32_t s = it & kSlotMask, d = expert(it);
        const int32_t have = np[(int64_t)d * R + r];
        const int32_t a = L.amt[s], c0 = L.cnt[r], gn = gnext[s];
        left_base = serve(r, c0, L.price[r]);
        const int32_t x = have < a ? have : a;
        Xb[(int64_t)r * S + s] = x;
        L.amt[s] = a - x;
        if (x == have) drained(d, r);
        else np[(int64_t)d * R + r] = have - x;
        if (x == a) L.work[wq] = gn >= 0 ? (it & ~kSlotMask) | gn : -1;
        wq = x == a && gn < 0 ? -2 : -1;  // -2: the group is done
      }
      base_left -= (int32_t)__popcll(__ballot(left_base));
      active -= (int32_t)__popcll(__ballot(wq == -2));
      wq = -1;
      have_n = 0;
    };
    for (int32_t q0 = 0; q0 < nw; q0 += kWave) {
      const int32_t q = q0 + lane;
      const int32_t it = q < nw ? L.work[q] : -1;
      const uint32_t state = q < nw ? L.sstate[q] : 0u;
      const int32_t r = (int32_t)(state & 15u) * kWave + (int32_t)(state >> 12) * 4 + ((it >> kItemBits) & 3);
      // the slot is part of the key, so its low half tells the winner (0: served already)
      const uint32_t k = it >= 0 ? rk[r] : 0u;
      const bool won = k != 0u && (k & 0xFFFFu) == (uint32_t)(0xFFFF - (it & kSlotMask));
      const uint64_t m = __ballot(won);
      const int32_t c = (int32_t)__popcll(m);
      if (c == 0) continue;
      if (have_n + c > kWave) transfers();
      // lane have_n + j takes the j-th winner of these entries
      const int32_t j = lane - have_n;
      if (j >= 0 && j < c) {
        uint64_t rest = m;
        for (int32_t u = 0; u < j; ++u) rest &= rest - 1ull;
        wq = q0 + (int32_t)__builtin_ctzll(rest);
      }
      have_n += c;
    }
    if (have_n > 0) transfers();
    if (track && base_left == 0) rebase();
    if (active <= nw - kWave) {
      // a group of lanes less will do: the list closes up in place (an entry
      // moves to its own place or a lower one)
      int32_t kept = 0;
      for (int32_t q0 = 0; q0 < nw; q0 += kWave) {
        const int32_t q = q0 + lane;
        const int32_t it = q < nw ? L.work[q] : -1;
        const uint32_t state = q < nw ? L.sstate[q] : 0u;
        const uint64_t m = __ballot(it >= 0);
        const int32_t to = kept + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (it >= 0) {
          L.work[to] = it;
          L.sstate[to] = (uint16_t)state;
        }
        kept += (int32_t)__popcll(m);
      }
      nw = kept;
    }
  }
  }
  // ---- up to G groups per lane, in registers ------------------------------------------------
  bool done = false;
  while (t <= tmax && !done && (NW == 1 || nw > kAuctionAlone)) {
    const int32_t sets = (nw + NW * kWave - 1) / (NW * kWave);  // in use; the list closes up when one less will do
    int32_t it[G], a[G], most[G];  // entry, tokens planned, the most a rank can hold
    int32_t pr[G], pv[G];          // a transfer in flight: its rank and what the rank held
    Bid b[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int32_t q = (g * NW + wid) * kWave + lane;
      it[g] = q < nw ? L.work[q] : -1;
      b[g] = Bid{-1, 0, 0u, 0ull};
      a[g] = most[g] = pv[g] = 0;
      pr[g] = -1;
      if (it[g] >= 0) {
        it[g] &= kItemMask;
        b[g].state = L.sstate[q] & kStateMask & ~kHas;  // (win is not known)
        a[g] = L.amt[it[g] & kSlotMask];
        most[g] = nmax[expert(it[g])];
      }
    }
    auto book = [&](int g) {  // the transfer in flight
      Xb[(int64_t)pr[g] * S + (it[g] & kSlotMask)] = pv[g];
      a[g] -= pv[g];
      pr[g] = -1;
    };
    for (; t <= tmax; ++t) {
      int32_t r[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        r[g] = -1;
        if (g >= sets) continue;
        const bool ok = it[g] >= 0 && (b[g].state & kHas) != 0u && (b[g].state >> 11) == epoch;
        const int w = (int)(b[g].state & 15u);
        const uint32_t lev = (b[g].state >> 6) & 15u;
        uint64_t m = L.lvl[(lev != 0u ? TW : 0) + w];
        if (__ballot(ok && lev >= 2u) != 0)
          if (lev >= 2u) m = level(lev, w);
        const uint64_t h = b[g].win & m;
        if (ok && h != 0ull) r[g] = w * kWave + __builtin_ctzll(h);
      }
      int32_t live = 0;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g >= sets) continue;
        const bool need = it[g] >= 0 && r[g] < 0;
        if (__ballot(need) != 0) {
          search_all(need, it[g], b[g]);
          if (need) {
            r[g] = b[g].r;
            if (r[g] < 0) {  // no valid rank is left
              if (pr[g] >= 0) book(g);
              L.amt[it[g] & kSlotMask] = a[g];
              it[g] = -1;
            }
          }
        }
        live += (int32_t)__popcll(__ballot(it[g] >= 0));
      }
      uint32_t key[G], k[G];
      int32_t c0[G];
      double price[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        key[g] = ((uint32_t)b[g].v << 16) | (uint32_t)(0xFFFF - (it[g] & kSlotMask));
        if (g < sets && it[g] >= 0) atomicMax(&rk[r[g]], key[g]);
      }
      if constexpr (NW > 1) {
        int32_t* const count = sh + kShLive + (int)(t & 1);
        if (lane == 0) atomicAdd(count, live);
        lds_barrier();
        live = __builtin_amdgcn_readfirstlane(*count);
        planes_on = __builtin_amdgcn_readfirstlane(sh[kShPlanes]) != 0;
        if (threadIdx.x == 0) {  // (read last before the barrier above)
          sh[kShLive + (int)((t + 1) & 1)] = 0;
          sh[kShList] = 0;
        }
      }
      if (live == 0) {  // no bid: the state is final
        done = true;
        break;
      }
      int32_t gone = 0;  // ranks that leave the base count
#pragma unroll
      for (int g = 0; g < G; ++g) {  // (the rank's count and price come with its key)
        if (g >= sets) continue;
        const int32_t rr = it[g] >= 0 ? r[g] : 0;
        k[g] = __hip_atomic_load(&rk[rr], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        c0[g] = L.cnt[rr];
        price[g] = L.price[rr];
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g >= sets) continue;
        const bool won = it[g] >= 0 && k[g] == key[g];
        if (__ballot(won) == 0) continue;
        bool left_base = false;
        if (won) {
          if (pr[g] >= 0) book(g);
          pv[g] = np[(int64_t)expert(it[g]) * R + r[g]];
          pr[g] = r[g];
          left_base = serve(r[g], c0[g], price[g]);
        }
        gone += (int32_t)__popcll(__ballot(left_base));
        const bool wait = won && a[g] <= most[g];  // the slot may fill
        if (won && !wait) drained(expert(it[g]), r[g]);
        if (__ballot(wait) != 0) {
          if (wait) {
            const int32_t d = expert(it[g]), s = it[g] & kSlotMask, have = pv[g];
            if (have <= a[g]) drained(d, r[g]);
            else np[(int64_t)d * R + r[g]] = have - a[g];
            if constexpr (NW > 1) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // another wave may read it
            pv[g] = have < a[g] ? have : a[g];
            book(g);
            if (a[g] == 0) {
              const int32_t gn = gnext[s];
              L.amt[s] = 0;
              it[g] = gn >= 0 ? (it[g] & ~kSlotMask) | gn : -1;
              if (gn >= 0) a[g] = L.amt[gn];
            }
          }
        }
      }
      if constexpr (NW > 1) {
        if (lane == 0 && gone) atomicSub(&sh[kShLeft], gone);
        lds_barrier();
        if (track && __builtin_amdgcn_readfirstlane(sh[kShLeft]) == 0) {
          lds_barrier();  // every wave has read the count
          rebase();
          if (threadIdx.x == 0) sh[kShLeft] = base_left;
          lds_barrier();
        }
      } else {
        base_left -= gone;
        if (track && base_left == 0) rebase();
      }
      if ((sets > 1 && live <= NW * kWave * (sets - 1)) || (NW > 1 && live <= kAuctionAlone)) {
        ++t;
        break;
      }
    }
    if (done) break;
    int32_t kept = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (it[g] >= 0) {
        if (pr[g] >= 0) book(g);
        L.amt[it[g] & kSlotMask] = a[g];
      }
      const uint64_t m = __ballot(it[g] >= 0);
      if constexpr (NW > 1) {
        int32_t at = 0;
        if (lane == 0 && m) at = atomicAdd(&sh[kShList], (int32_t)__popcll(m));
        kept = __builtin_amdgcn_readfirstlane(at);
      }
      const int32_t to = kept + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
      if (it[g] >= 0) {
        L.work[to] = it[g];
        L.sstate[to] = (uint16_t)b[g].state;
      }
      kept += (int32_t)__popcll(m);
    }
    nw = kept;
    if constexpr (NW > 1) {
      lds_barrier();
      nw = __builtin_amdgcn_readfirstlane(sh[kShList]);
      base_left = __builtin_amdgcn_readfirstlane(sh[kShLeft]);
    }
  }
  run = AuctionRun{t, nw, base, base_left, epoch, P0, planes_on, done};
}

// LDS of the auction alone.
template <class CF>
__host__ __device__ inline LdsState<CF> carve_auction(char* base, int32_t R, int32_t K) {
  LdsState<CF> w{};
  const size_t S1 = R * K > 0 ? (size_t)R * K : 1, R_ = (size_t)R;
  constexpr size_t TW = CF::kTW, SC = CF::kSC, DC = CF::kDC;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* q = base + off;
    off = (off + bytes + 15) & ~(size_t)15;
    return q;
  };
  w.slot_ec = (int16_t*)take(2 * S1);  // next slots of the bid groups
  w.amt = (int32_t*)take(4 * S1);
  w.work = (int32_t*)take(4 * S1); w.sstate = (uint16_t*)take(2 * S1);
  w.price = (double*)take(8 * R_); w.rkey = (uint32_t*)take(4 * R_); w.cnt = (int32_t*)take(4 * R_);
  w.vmask = (uint64_t*)take(8 * DC * TW); w.vwords = (uint32_t*)take(TW > 4 ? 4 * DC : 0);
  w.dexp = (int32_t*)take(4 * DC);
  w.planes = (uint64_t*)take(8 * CF::kPL * TW);
  w.lvl = (uint64_t*)take(2 * 8 * TW); w.rel = (uint64_t*)take(8 * kRelPlanes * TW);
  w.cn = (int8_t*)take(SC);
  w.cv = (double*)take(8 * SC * kTierMax); w.cvr = (int32_t*)take(4 * SC * kTierMax);
  w.cw = (uint32_t*)take(4 * SC * kTierMax);
  w.cm = (uint64_t*)take(8 * SC * kTierMax * TW);
  w.bytes = off;
  return w;
}

// The auction's start by NT threads: no services, and the tables of the bonus
// tiers.
template <class CF, int NT>
__device__ __forceinline__ void auction_start(const LdsState<CF>& L, const LdsParams& wp, int32_t R) {
  constexpr int TW = CF::kTW;
  const int tid = threadIdx.x;
  for (int32_t r = tid; r < R; r += NT) {
    L.price[r] = 0.0;
    L.rkey[r] = 0;
    L.cnt[r] = 0;
  }
  for (int32_t q = tid; q < CF::kPL * TW; q += NT) L.planes[q] = 0ull;
  // every rank starts with 0 services: at the base count 0, code 0
  for (int32_t q = tid; q < TW; q += NT) {
    const int32_t lo = q * kWave;
    L.lvl[q] = lo >= R ? 0ull : (R - lo >= kWave ? ~0ull : (1ull << (R - lo)) - 1ull);
    L.lvl[TW + q] = 0ull;
  }
  for (int32_t q = tid; q < kRelPlanes * TW; q += NT) L.rel[q] = 0ull;
  const int32_t ns = wp.hdr[0];
  for (int32_t q = tid; q < ns; q += NT) L.cn[q] = (int8_t)wp.cn[q];
  for (int32_t q = tid; q < ns * kTierMax; q += NT) {
    L.cv[q] = wp.cv[q];
    L.cvr[q] = wp.cvr[q];
    L.cw[q] = wp.cw[q];
  }
  for (int32_t q = tid; q < ns * kTierMax * TW; q += NT) {
    const int32_t e = q / TW;
    L.cm[e * TW + set_word<TW>(e / kTierMax, q % TW)] = wp.cm[q];
  }
}

// Rounds and results of problem b on one wave.
template <class CF>
__device__ __forceinline__ void auction_problem(const LdsState<CF>& L, const LdsParams& wp, int64_t b, int32_t nw,
                                                int32_t used2, int32_t* sh) {
  const SchParams& p = wp.s;
  const int32_t R = p.R, S = p.R * p.K;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t tmax = p.t_max > 0 ? p.t_max : (int64_t)S * (R + 1);
  int32_t* const np = wp.nprime + b * (int64_t)CF::kDC * R;
  int32_t* const Xb = p.X + b * (int64_t)R * S;
  AuctionRun run{1, nw, 0, R, 0u, 0.0, false, false};
  if constexpr (CF::kAW > 1) {
    if (nw > kAuctionAlone) auction_rounds<CF, CF::kAW>(L, run, sh, L.slot_ec, np, Xb, R, S, p.price_step, tmax);
    if (threadIdx.x >= kWave) return;
  }
  if (!run.done) auction_rounds<CF, 1>(L, run, nullptr, L.slot_ec, np, Xb, R, S, p.price_step, tmax);
  const int64_t rounds = run.t - 1;
  int64_t left = 0;  // (a slot without an expert plans 0 tokens)
  for (int32_t s = lane; s < S; s += kWave) left += L.amt[s];
  const int64_t tot = wave_sum_i64(left);
  if (lane == 0) {
    p.unfilled[b] = tot;
    if (p.rounds_used) { p.rounds_used[2 * b] = used2; p.rounds_used[2 * b + 1] = (int32_t)rounds; }
    if (p.status) p.status[b] = tot > 0 ? TAOT_ST_UNFILLED : 0u;
    wp.fallback[b] = 0;
  }
}

// The auction of one problem per workgroup of kAW waves, for the configurations
// whose matching kernel has several waves: it needs few waves but many
// registers, and other workgroups' matching can take the compute unit's rest.
template <class CF>
__global__ void __launch_bounds__(CF::kAW * kWave) auction_kernel(LdsParams wp) {
  constexpr int TW = CF::kTW, NT = CF::kAW * kWave;
  __shared__ int32_t sh[kShWords];
  extern __shared__ __attribute__((aligned(16))) char lds_dyn[];
  const int64_t b = blockIdx.x;
  const int4 h = wp.h.hdr[b];
  if (h.x < 0) return;
  const int tid = threadIdx.x;
  const int32_t R = wp.s.R, S = wp.s.R * wp.s.K;
  const LdsState<CF> L = carve_auction<CF>(lds_dyn, R, wp.s.K);
  auction_start<CF, NT>(L, wp, R);
  for (int32_t q = tid; q < S; q += NT) {
    L.amt[q] = wp.h.amt[b * S + q];
    L.slot_ec[q] = wp.h.gnext[b * S + q];
    L.sstate[q] = 0;  // no bid yet
  }
  for (int32_t q = tid; q < h.x; q += NT) L.work[q] = wp.h.work[b * S + q];
  for (int32_t q = tid; q < h.z; q += NT) {
    L.dexp[q] = wp.h.nmax[b * CF::kDC + q];
    if constexpr (TW > 4) L.vwords[q] = wp.h.vwords[b * CF::kDC + q];
  }
  for (int32_t q = tid; q < h.z * TW; q += NT) L.vmask[q] = wp.h.vmask[b * CF::kDC * TW + q];
  if (tid < kShWords) sh[tid] = tid == kShLeft ? R : 0;
  __syncthreads();
  auction_problem<CF>(L, wp, b, __builtin_amdgcn_readfirstlane(h.x), h.y, sh);
}

// Validation, matching and the auction's lists of one problem per workgroup of
// CF::kT threads; a one-wave workgroup runs the auction too.  WPE waves per SIMD
// bound the registers: a batch that fills the chip needs all its problems
// resident at once, a smaller one is better served without the register cap.
template <class CF, int WPE>
__global__ void __launch_bounds__(CF::kT, WPE) schedule_lds_kernel(LdsParams wp) {
  constexpr int NT = CF::kT, NW = NT / kWave, TW = CF::kTW;
  extern __shared__ __attribute__((aligned(16))) char lds_dyn[];
  __shared__ int32_t wave_cnt[NW];
  __shared__ int32_t flagbuf[2 * NW];
  __shared__ int32_t sh_nw;
  __shared__ unsigned long long sh_sum, sh_big;
  const SchParams& p = wp.s;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
  const int64_t b = blockIdx.x;
  const int32_t R = p.R, E = p.E, K = p.K;
  const int32_t S = R * K;
  int parity = 0;
  LdsState<CF> L = carve_lds<CF>(lds_dyn, R, K, wp.NEC);

  if (wp.hdr[1] == 0) {  // the LDS-resident auction would not be exact for this Bauct and step
    if (tid == 0) {
      wp.fallback[b] = 1;
      if constexpr (NW > 1) wp.h.hdr[b] = int4{-1, 0, 0, 0};
    }
    return;
  }
  const int64_t* spill = p.spill + b * E;
  const int64_t* spare = p.spare + b * R;
  const int64_t* excess = p.excess + b * R;
  const float* Tb = p.T + b * (int64_t)R * R;
  int32_t* se = p.slot_expert + b * S;
  int64_t* sa = p.slot_amount + b * S;
  int32_t* Xb = p.X + b * (int64_t)R * S;
  const double alpha = topo_weight(p.flags, p.alpha[b]);
  const double a2 = flow_weight(p.flags, p.alpha[b]);

  // ---- validation, candidates, cold ranks ------------------------------------------
  bool badh = false;
  for (int32_t e = tid; e < E; e += NT) {
    const int32_t h = p.home[e];
    badh |= h < 0 || h >= R;
  }
  if (tid == 0) { sh_sum = 0; sh_big = 0; sh_nw = 0; }
  if (block_or<NT>(badh, flagbuf, parity)) {
    for (int32_t s = tid; s < S; s += NT) { se[s] = -1; sa[s] = 0; }
    for (int64_t q = tid; q < (int64_t)R * S; q += NT) Xb[q] = 0;
    if (tid == 0) {
      p.unfilled[b] = 0;
      if (p.rounds_used) { p.rounds_used[2 * b] = 0; p.rounds_used[2 * b + 1] = 0; }
      if (p.status) p.status[b] = TAOT_ST_BAD_INPUT;
      wp.fallback[b] = 0;
      if constexpr (NW > 1) wp.h.hdr[b] = int4{-1, 0, 0, 0};
    }
    return;
  }
  int32_t ne = 0, nc = 0;
  int64_t mass = 0, big = 0;  // amounts must fit the 32-bit LDS state
  for (int32_t base = 0; base < E; base += NT) {
    const int32_t e = base + tid;
    const int64_t v = e < E ? spill[e] : 0;
    const bool f = v > 0;
    int32_t tot;
    const int32_t pos = ne + compact_pos_n<NT>(f, wave_cnt, tot);
    if (f && pos < wp.NEC) {
      L.ce[pos] = e;
      L.spill_p[pos] = (int32_t)(v < INT_MAX ? v : INT_MAX);
      L.hce[pos] = p.home[e];
    }
    ne += tot;
    mass += f ? v : 0;
  }
  for (int32_t base = 0; base < R; base += NT) {
    const int32_t r = base + tid;
    const int64_t v = r < R ? spare[r] : 0;
    const bool f = v > 0;
    int32_t tot;
    const int32_t pos = nc + compact_pos_n<NT>(f, wave_cnt, tot);
    if (f) { L.cr[pos] = r; L.spare_p[pos] = (int32_t)(v < INT_MAX ? v : INT_MAX); }
    nc += tot;
    big = v > big ? v : big;
    if (r < R) {
      const double ex = (double)excess[r];
      L.den[r] = ex > kEps0 ? ex : kEps0;
    }
  }
  mass = wave_sum_i64(mass);
  big = wave_max_i64(big);
  if (lane == 0) {
    atomicAdd(&sh_sum, (unsigned long long)mass);
    atomicMax(&sh_big, (unsigned long long)big);
  }
  __syncthreads();
  if (ne > wp.NEC || sh_sum > (unsigned long long)INT_MAX || sh_big > (unsigned long long)INT_MAX) {
    if (tid == 0) {
      wp.fallback[b] = 1;
      if constexpr (NW > 1) wp.h.hdr[b] = int4{-1, 0, 0, 0};
    }
    return;
  }
  for (int32_t q = tid; q < nc * K; q += NT) L.assigned[q] = -1;
  for (int32_t ec = tid; ec < ne; ec += NT) { L.ekey[ec] = 0; L.ewin[ec] = INT_MAX; }
  for (int32_t s = tid; s < S; s += NT) { L.slot_ec[s] = -1; L.amt[s] = 0; se[s] = -1; }
  __syncthreads();

  // ---- Phase 2: column-priority iterative matching ---------------------------------
  // Every thread has one cold rank (nc <= R <= NT).  What bounds a proposal is
  // the scan of all candidates (two loads and a division each, most ranks of a
  // wave at once whenever the expert that they all want runs out), so a scan
  // keeps the rank's best kBestOf candidates with their score terms.  No score
  // rises after it (spill and spare only fall, the other terms are fixed, a
  // taken expert stays taken), so every candidate off the list stays at or
  // below the score of the list's last entry, and behind it in index on a tie:
  // while the best listed candidate is above that, or level and no later in
  // index, it is the best of all, and a rank whose list holds all its
  // candidates never scans again.  The register-capped build has no room for
  // lists and enough problems in flight to hide a scan's loads (1952 x R = 256:
  // 3.14 ms a call, 3.3 to 3.9 with lists of 1 to 4; one-wave problems, 3000 x R =
  // 64: 465 us, 541 and 548 with lists of 2 and 4; 3000 x R = 32, K = 4: 230, 265
  // and 273); elsewhere the scans are the matching's time (58 x R = 64: 345 -> 317
  // us a call).
  constexpr int kBestOf = WPE > 1 ? 0 : 4, kList = kBestOf > 0 ? kBestOf : 1;
  int32_t used2 = 0;
  const int32_t rc = tid;
  double ls[kList], l1[kList], l2[kList];  // scan's scores (descending), terms
  int32_t le[kList];                       // candidates (-1: none)
  int32_t lastc = -1;                            // the scan's last entry
  double bound = INFINITY;                       // its score; -inf: all candidates are listed
#pragma unroll
  for (int m = 0; m < kList; ++m) { le[m] = -1; ls[m] = -INFINITY; l1[m] = l2[m] = 0.0; }
  for (int32_t k = 0; k < K; ++k) {
    if (rc < nc) {
      const int32_t pa = k > 0 ? L.assigned[rc * K + k - 1] : -1;  // taken from here on
#pragma unroll
      for (int m = 0; m < kBestOf; ++m) le[m] = le[m] == pa ? -1 : le[m];
      L.matched[rc] = 0;
      L.prop_e[rc] = -1;
    }
    __syncthreads();
    for (int32_t inner = 0; inner < nc; ++inner) {
      // Step 1: every unmatched cold rank proposes its best candidate expert
      bool proposed = false;
      if (rc < nc && !L.matched[rc]) {
        const int32_t sp = L.spare_p[rc], pe = L.prop_e[rc];
        // a losing proposal stands while its expert's q = min(spill, spare) is unchanged
        const int32_t sl0 = pe >= 0 ? L.spill_p[pe] : 0;
        proposed = pe >= 0 && (sl0 < sp ? sl0 : sp) == L.qbest[rc];
        if (!proposed) {
          int32_t best = -1, bq = 0;
          double bs = -INFINITY;
          auto offer = [&](int32_t ec, int32_t q, double score) {
            if (score > bs || (score == bs && ec < best)) { bs = score; best = ec; bq = q; }
          };
          if (sp > 0) {
#pragma unroll
            for (int m = 0; m < kBestOf; ++m) {
              const int32_t sl = le[m] >= 0 ? L.spill_p[le[m]] : 0;
              const int32_t q = sl < sp ? sl : sp;
              if (sl > 0) offer(le[m], q, ((double)q + l1[m]) + l2[m]);
            }
          }
          if (sp > 0 && (kBestOf == 0 || !(bs > bound || (bs == bound && best <= lastc)))) {
            best = -1;
            bs = -INFINITY;
#pragma unroll
            for (int m = 0; m < kBestOf; ++m) { le[m] = -1; ls[m] = -INFINITY; }
            const int32_t r = L.cr[rc];
            const int32_t* asg = L.assigned + rc * K;
            const int32_t a0 = k > 0 ? asg[0] : -1, a1 = k > 1 ? asg[1] : -1;
            const int32_t a2_ = k > 2 ? asg[2] : -1, a3 = k > 3 ? asg[3] : -1;
            for (int32_t ec0 = 0; ec0 < ne; ec0 += 4) {
              int32_t sl[4], hh[4];
              double bp[4];
              float tt[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const bool in = ec0 + u < ne;
                sl[u] = in ? L.spill_p[ec0 + u] : 0;
                hh[u] = in ? L.hce[ec0 + u] : r;
              }
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const bool ok = sl[u] > 0 && hh[u] != r;
                const int64_t o = (int64_t)hh[u] * R + r;
                bp[u] = ok ? p.Bpref[o] : 0.0;
                tt[u] = ok ? Tb[o] : 0.f;
              }
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const int32_t ec = ec0 + u;
                if (sl[u] <= 0 || hh[u] == r) continue;
                bool taken = ec == a0 || ec == a1 || ec == a2_ || ec == a3;
                for (int32_t kk = 4; kk < k; ++kk) taken |= asg[kk] == ec;
                if (taken) continue;
                const double q = (double)(sl[u] < sp ? sl[u] : sp);
                const double t1 = alpha * bp[u];
                const double tn = (double)tt[u] / L.den[hh[u]];
                const double t2 = a2 * tn;
                const double score = (q + t1) + t2;
                if constexpr (kBestOf == 0) {
                  if (score > bs) { bs = score; best = ec; bq = sl[u] < sp ? sl[u] : sp; }
                  continue;
                }
                if (!(score > ls[kList - 1])) continue;
                // in behind the entries that score as much (lower indices)
                ls[kList - 1] = score;
                le[kList - 1] = ec;
                l1[kList - 1] = t1;
                l2[kList - 1] = t2;
#pragma unroll
                for (int m = kList - 1; m > 0; --m) {
                  const bool up = ls[m] > ls[m - 1];
                  const double s0 = ls[m - 1], x0 = l1[m - 1], y0 = l2[m - 1];
                  const int32_t e0 = le[m - 1];
                  ls[m - 1] = up ? ls[m] : s0; ls[m] = up ? s0 : ls[m];
                  l1[m - 1] = up ? l1[m] : x0; l1[m] = up ? x0 : l1[m];
                  l2[m - 1] = up ? l2[m] : y0; l2[m] = up ? y0 : l2[m];
                  le[m - 1] = up ? le[m] : e0; le[m] = up ? e0 : le[m];
                }
              }
            }
            if constexpr (kBestOf > 0) {
              lastc = le[kList - 1];
              bound = ls[kList - 1];  // (-inf: the list did not fill)
              best = le[0];
              bs = ls[0];
              if (best >= 0) bq = L.spill_p[best] < sp ? L.spill_p[best] : sp;
            }
          }
          L.prop_e[rc] = best;
          L.prop_s[rc] = bs;
          L.qbest[rc] = bq;
          proposed = best >= 0;
        }
      }
      if (!block_or<NT>(proposed, flagbuf, parity)) break;  // nothing can change any more
      // Steps 2-3: each proposed expert keeps its best proposer: max score, then lowest rank
      const int32_t pe = rc < nc ? L.prop_e[rc] : -1;
      const uint64_t key = pe >= 0 ? ordered_key(L.prop_s[rc]) : 0;
      if (pe >= 0) atomicMax(reinterpret_cast<unsigned long long*>(&L.ekey[pe]), (unsigned long long)key);
      __syncthreads();
      if (pe >= 0 && key == L.ekey[pe]) atomicMin(&L.ewin[pe], rc);
      __syncthreads();
      // Step 4: winners take g = min(spill, spare) into slot k of their rank
      for (int32_t ec = tid; ec < ne; ec += NT) {
        const int32_t w = L.ewin[ec];
        if (w != INT_MAX) {
          const int32_t g = L.spill_p[ec] < L.spare_p[w] ? L.spill_p[ec] : L.spare_p[w];
          L.spill_p[ec] -= g;
          L.spare_p[w] -= g;
          L.matched[w] = 1;
          L.prop_e[w] = -1;  // matched ranks stop proposing
          L.assigned[w * K + k] = ec;
          const int32_t s = L.cr[w] * K + k;
          L.slot_ec[s] = (int16_t)ec;
          L.amt[s] += g;
          se[s] = L.ce[ec];
        }
        L.ekey[ec] = 0;
        L.ewin[ec] = INT_MAX;
      }
      __syncthreads();
      ++used2;
    }
  }
  for (int32_t s = tid; s < S; s += NT) sa[s] = L.amt[s];

  // ---- Phase 3: Lagrangian auction ---------------------------------------------------
  // distinct slot experts, in ascending candidate (= expert) order
  __syncthreads();
  for (int32_t ec = tid; ec < ne; ec += NT) L.dmap[ec] = 0;
  __syncthreads();
  for (int32_t s = tid; s < S; s += NT)
    if (L.slot_ec[s] >= 0) L.dmap[L.slot_ec[s]] = 1;
  __syncthreads();
  int32_t D = 0;
  for (int32_t base = 0; base < ne; base += NT) {
    const int32_t ec = base + tid;
    const bool f = ec < ne && L.dmap[ec] == 1;
    int32_t tot;
    const int32_t pos = D + compact_pos_n<NT>(f, wave_cnt, tot);
    if (ec < ne) L.dmap[ec] = f ? pos : -1;
    if (f && pos < CF::kDC) L.dexp[pos] = L.ce[ec];
    D += tot;
  }
  if (D > CF::kDC) {
    if (tid == 0) {
      wp.fallback[b] = 1;
      if constexpr (NW > 1) wp.h.hdr[b] = int4{-1, 0, 0, 0};
    }
    return;
  }
  __syncthreads();
  // tokens of each slot expert per rank (device memory), the valid-rank sets
  // and the words of each set that hold ranks
  int32_t* np = wp.nprime + b * (int64_t)CF::kDC * R;
  const int32_t* nb = p.n + b * (int64_t)R * E;
  if constexpr (TW > 4)
    for (int32_t d = tid; d < D; d += NT) L.vwords[d] = 0u;
  for (int32_t d = tid; d < D; d += NT) L.work[d] = 0;  // D <= S
  __syncthreads();
  // (wave w takes word w, rank r on its lane; the strided loads of eight
  // experts are issued before any is used)
  static_assert(TW == NW, "one rank word per wave");
  {
    const int32_t r = wid * kWave + lane;
    for (int32_t d0 = 0; d0 < D; d0 += 8) {
      int32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = d0 + u < D && r < R ? nb[(int64_t)r * E + L.dexp[d0 + u]] : 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int32_t d = d0 + u;
        if (d >= D) break;
        if (r < R) np[(int64_t)d * R + r] = v[u];
        const uint64_t m = __ballot(v[u] > 0);
        const int32_t most = wave_max_i32(v[u]);
        if (lane == 0) {
          atomicMax(&L.work[d], most);
          L.vmask[d * TW + set_word<TW>(d, wid)] = m;
          if constexpr (TW > 4)
            if (m) atomicOr(&L.vwords[d], 1u << wid);
        }
      }
    }
  }
  // from here on dexp holds the most tokens of each slot expert on any rank
  __syncthreads();
  for (int32_t d = tid; d < D; d += NT) L.dexp[d] = L.work[d];
  __syncthreads();
  // The list of the first round: the first slot of each bid group.
  // Bid groups.  Two open slots with the same host tier structure and the
  // same expert (the item's bits above the slot) make the same bid: the
  // search reads only those and the shared state.  Their keys then differ
  // in the slot alone, so the lower slot wins wherever both bid, and a
  // slot of a group can only be served once every lower open slot of the
  // group is full.  A group without a valid rank is without one for all
  // its slots (validity depends on the expert only).  So each group bids
  // with its lowest open slot only; when that slot fills, the next open
  // slot of the group takes its place (and its bid state, which depends on
  // the group alone).  The rounds, bids and transfers are the same as
  // with every open slot bidding.  The items are built once, by slot, in
  // the list array (-1: no tokens planned).
  auto slot_item = [&](int32_t s, bool& f) {
    const int32_t ec = s < S ? L.slot_ec[s] : -1;
    f = ec >= 0 && L.amt[s] > 0;
    return f ? s | (L.dmap[ec] << kItemSlotBits) | (wp.sidx[s / K] << (kItemSlotBits + kItemExpertBits)) : 0;
  };
  // the next open slot of each slot's bid group (-1: none), over the slot
  // experts, which nothing reads once the items are built
  int16_t* const gnext = L.slot_ec;
  for (int32_t s = tid; s < S; s += NT) {
    bool f;
    const int32_t item = slot_item(s, f);
    L.work[s] = f ? item : -1;
  }
  __syncthreads();
  for (int32_t s = tid; s < S; s += NT) {
    const int32_t it0 = L.work[s];
    int32_t nx = -1;
    if (it0 >= 0) {
      // the group key; a slot without tokens (-1) has key -1
      const int32_t k = it0 >> kItemSlotBits;
      int32_t q = s + 1;
      for (; q < S && (q & 3); ++q)
        if ((L.work[q] >> kItemSlotBits) == k) { nx = q; break; }
      if (nx < 0) {
        // four items per 16-byte load (the list array is 16-byte aligned)
        for (; q + 3 < S; q += 4) {
          const int4 w4 = *reinterpret_cast<const int4*>(L.work + q);
          const bool x0 = (w4.x >> kItemSlotBits) == k, x1 = (w4.y >> kItemSlotBits) == k,
                     x2 = (w4.z >> kItemSlotBits) == k, x3 = (w4.w >> kItemSlotBits) == k;
          if (x0 || x1 || x2 || x3) {
            nx = x0 ? q : x1 ? q + 1 : x2 ? q + 2 : q + 3;
            break;
          }
        }
        if (nx < 0)
          for (; q < S; ++q)
            if ((L.work[q] >> kItemSlotBits) == k) { nx = q; break; }
      }
    }
    gnext[s] = (int16_t)nx;
  }
  __syncthreads();
  // a slot with a lower open slot in its group waits: its item is marked
  // negative (one writer per slot)
  for (int32_t s = tid; s < S; s += NT)
    if (gnext[s] >= 0) L.work[gnext[s]] |= (int32_t)0x80000000u;
  __syncthreads();
  // the groups' first slots, compacted
  constexpr int kSlotsPerThread = CF::kMaxS / NT;
  int32_t mine[kSlotsPerThread];
#pragma unroll
  for (int i = 0; i < kSlotsPerThread; ++i) mine[i] = i * NT + tid < S ? L.work[i * NT + tid] : -1;
  __syncthreads();  // every item is read before the list overwrites the array
#pragma unroll
  for (int i = 0; i < kSlotsPerThread; ++i) list_append(mine[i] >= 0, mine[i], L.work, &sh_nw);
  // X starts at zero; every (rank, slot) pair is served at most once (after a
  // transfer either the rank holds no more tokens of the slot's expert or the
  // slot is full), so transfers below are plain stores
  {
    int4* x4 = reinterpret_cast<int4*>(Xb);
    const int64_t n4 = ((int64_t)R * S) / 4;
    if ((reinterpret_cast<uintptr_t>(Xb) & 15u) == 0) {
      for (int64_t q = tid; q < n4; q += NT) x4[q] = make_int4(0, 0, 0, 0);
      for (int64_t q = n4 * 4 + tid; q < (int64_t)R * S; q += NT) Xb[q] = 0;
    } else {
      for (int64_t q = tid; q < (int64_t)R * S; q += NT) Xb[q] = 0;
    }
  }
  __syncthreads();
  if constexpr (NW == 1) {
    for (int32_t s = tid; s < S; s += NT) L.sstate[s] = 0;  // no bid yet
    auction_start<CF, NT>(L, wp, R);
    __syncthreads();
    auction_problem<CF>(L, wp, b, sh_nw, used2, nullptr);
  } else {
    for (int32_t q = tid; q < S; q += NT) {
      wp.h.amt[b * S + q] = L.amt[q];
      wp.h.gnext[b * S + q] = gnext[q];
      if (q < sh_nw) wp.h.work[b * S + q] = L.work[q];
    }
    for (int32_t q = tid; q < D; q += NT) {
      wp.h.nmax[b * CF::kDC + q] = L.dexp[q];
      if constexpr (TW > 4) wp.h.vwords[b * CF::kDC + q] = L.vwords[q];
    }
    for (int32_t q = tid; q < D * TW; q += NT) wp.h.vmask[b * CF::kDC * TW + q] = L.vmask[q];
    if (tid == 0) wp.h.hdr[b] = int4{sh_nw, used2, D, 0};
  }
}
}  // namespace

static int32_t sched_grid(int32_t B) { return B < kSchMaxGrid ? B : kSchMaxGrid; }

namespace {

struct SchWs {
  char* slab;          // general path: one slab per resident workgroup
  int32_t* fallback;   // [B]
  int32_t* ntier;      // [R]
  double* tv;          // [R][kTierMax]
  uint64_t* tmask;     // [R][kTierMax][TW]
  int32_t* sidx;       // [R]
  int32_t* cn;         // [SC]
  double* cv;          // [SC][kTierMax]
  int32_t* cvr;        // [SC][kTierMax]
  uint32_t* cw;        // [SC][kTierMax]
  uint64_t* cm;        // [SC][kTierMax][TW]
  int32_t* hdr;        // [2]
  int32_t* nprime;     // [B][DC][R]
  Handoff h;
  int64_t slab_bytes;
  size_t bytes;
};

// The tables are sized for the largest configuration, which any of them may use.
SchWs carve_sched(void* ws, int32_t B, int32_t R, int32_t E, int32_t K) {
  Carver c{static_cast<char*>(ws)};
  SchWs w;
  const bool lds_path = R <= LdsLarge::kTW * kWave;
  const size_t TW = LdsLarge::kTW, SC = LdsLarge::kSC, DC = lds_path ? LdsLarge::kDC : 0;
  w.slab_bytes = round_up((int64_t)carve_slab(nullptr, R, E, K).bytes, 256);
  w.slab = c.take<char>((size_t)w.slab_bytes * (B > 0 ? sched_grid(B) : 0));
  w.fallback = c.take<int32_t>((size_t)B);
  w.ntier = c.take<int32_t>((size_t)R);
  w.tv = c.take<double>((size_t)R * kTierMax);
  w.tmask = c.take<uint64_t>((size_t)R * kTierMax * TW);
  w.sidx = c.take<int32_t>((size_t)R);
  w.cn = c.take<int32_t>(SC);
  w.cv = c.take<double>(SC * kTierMax);
  w.cvr = c.take<int32_t>(SC * kTierMax);
  w.cw = c.take<uint32_t>(SC * kTierMax);
  w.cm = c.take<uint64_t>(SC * kTierMax * TW);
  w.hdr = c.take<int32_t>(2);
  w.nprime = c.take<int32_t>((size_t)B * DC * R);
  const size_t HB = lds_path ? (size_t)B : 0, S = (size_t)R * K;
  w.h.hdr = c.take<int4>(HB);
  w.h.amt = c.take<int32_t>(HB * S);
  w.h.work = c.take<int32_t>(HB * S);
  w.h.gnext = c.take<int16_t>(HB * S);
  w.h.nmax = c.take<int32_t>(HB * DC);
  w.h.vwords = c.take<uint32_t>(HB * DC);
  w.h.vmask = c.take<uint64_t>(HB * DC * TW);
  w.bytes = c.off;
  return w;
}

template <class CF, int WPE>
taot_status launch_lds_kernel(const LdsParams& wp, int32_t B, size_t lds, hipStream_t stream) {
  if (!allow_lds((const void*)schedule_lds_kernel<CF, WPE>, lds)) return TAOT_ERR_LAUNCH;
  hipLaunchKernelGGL((schedule_lds_kernel<CF, WPE>), dim3((unsigned)B), dim3(CF::kT), lds, stream, wp);
  return hipGetLastError() == hipSuccess ? TAOT_OK : TAOT_ERR_LAUNCH;
}

// Largest dynamic LDS a workgroup may use on the current device.
size_t max_lds_per_block() {
  static size_t cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 65536;
  if (cached[dev] == 0) {
    int v = 0;
    cached[dev] = hipDeviceGetAttribute(&v, hipDeviceAttributeSharedMemPerBlockOptin, dev) == hipSuccess && v > 0
                      ? (size_t)v
                      : 65536;
  }
  return cached[dev];
}

// Prepasses and the LDS-resident kernel of configuration CF; false when its
// layout does not fit (the general kernel then takes every problem).
template <class CF>
taot_status launch_lds_path(const SchParams& p, const SchWs& w, int32_t B, int32_t R, int32_t E, int32_t K,
                            double price_step, hipStream_t stream, bool& launched) {
  launched = false;
  const int32_t NEC = E < CF::kNEC ? E : CF::kNEC;  // candidate experts (spill > 0) held in LDS
  const int64_t S = (int64_t)R * K;
  const size_t slds = carve_lds<CF>(nullptr, R, K, NEC).bytes, alds = carve_auction<CF>(nullptr, R, K).bytes;
  if (R > CF::kTW * kWave || S <= 0 || S > CF::kMaxS || slds > max_lds_per_block() || alds > max_lds_per_block())
    return TAOT_OK;
  hipLaunchKernelGGL(auction_tiers_kernel<CF::kTW>, dim3((unsigned)R), dim3(256), 0, stream, p.Bauct, R, w.ntier,
                     w.tv, w.tmask);
  if (hipGetLastError() != hipSuccess) return TAOT_ERR_LAUNCH;
  hipLaunchKernelGGL(auction_struct_kernel<CF>, dim3(1), dim3(CF::kT), 0, stream, w.ntier, w.tv, w.tmask, R, S,
                     price_step, w.sidx, w.cn, w.cv, w.cvr, w.cw, w.cm, w.hdr);
  if (hipGetLastError() != hipSuccess) return TAOT_ERR_LAUNCH;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    return TAOT_ERR_LAUNCH;
  const LdsParams wp{p, w.h, w.sidx, w.cn, w.cv, w.cvr, w.cw, w.cm, w.hdr, w.fallback, w.nprime, NEC};
  taot_status st;
  // a batch of more problems than fit six to a compute unit takes the
  // register-capped build, which can hold CF::kWavesPerEU per SIMD
  const bool cap = (int64_t)B > (int64_t)6 * cus;
  st = cap ? launch_lds_kernel<CF, CF::kWavesPerEU>(wp, B, slds, stream) : launch_lds_kernel<CF, 1>(wp, B, slds, stream);
  if (st != TAOT_OK) return st;
  if constexpr (CF::kT > kWave) {
    if (!allow_lds((const void*)auction_kernel<CF>, alds)) return TAOT_ERR_LAUNCH;
    hipLaunchKernelGGL(auction_kernel<CF>, dim3((unsigned)B), dim3(CF::kAW * kWave), alds, stream, wp);
    if (hipGetLastError() != hipSuccess) return TAOT_ERR_LAUNCH;
  }
  launched = true;
  return TAOT_OK;
}

}  // namespace

size_t schedule_ws(int32_t B, int32_t R, int32_t E, int32_t K) { return carve_sched(nullptr, B, R, E, K).bytes; }

taot_status launch_schedule(const int32_t* n, const int64_t* spill, const int64_t* spare,
                            const int64_t* excess, const double* alpha, const int32_t* home,
                            const float* T, const double* Bpref, const double* Bauct, int32_t B,
                            int32_t R, int32_t E, int32_t K, double price_step, int64_t t_max,
                            uint32_t flags, int32_t* slot_expert, int64_t* slot_amount, int32_t* X,
                            int64_t* unfilled, int32_t* rounds_used, uint32_t* status, void* ws,
                            hipStream_t stream) {
  if (B == 0) return TAOT_OK;
  SchWs w = carve_sched(ws, B, R, E, K);
  SchParams p{n, spill, spare, excess, alpha, home, T, Bpref, Bauct, B, R, E, K, price_step, t_max,
              slot_expert, slot_amount, X, unfilled, rounds_used, status, w.slab, w.slab_bytes, w.fallback,
              flags};
  bool launched = false;
  taot_status st = TAOT_OK;
  // the row-priority ablation lives in the general kernel only
  if (!(flags & TAOT_SCH_ROW_PRIORITY)) {
    st = launch_lds_path<LdsTiny>(p, w, B, R, E, K, price_step, stream, launched);
    if (st == TAOT_OK && !launched) st = launch_lds_path<LdsSmall>(p, w, B, R, E, K, price_step, stream, launched);
    if (st == TAOT_OK && !launched) st = launch_lds_path<LdsLarge>(p, w, B, R, E, K, price_step, stream, launched);
  }
  if (st != TAOT_OK) return st;
  if (!launched) p.fallback = nullptr;  // the general kernel takes every problem
  const size_t lds = (size_t)R * (sizeof(double) + sizeof(uint64_t) + 2 * sizeof(int32_t));
  if (!allow_lds((const void*)schedule_kernel, lds)) return TAOT_ERR_LAUNCH;
  hipLaunchKernelGGL(schedule_kernel, dim3((unsigned)sched_grid(B)), dim3(kSchThreads), lds, stream, p);
  return hipGetLastError() == hipSuccess ? TAOT_OK : TAOT_ERR_LAUNCH;
}

}  // namespace taot
