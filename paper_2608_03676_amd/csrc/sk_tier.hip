// Sinkhorn on topology tiers: the iterate of Sec. A.2 for a shared cost matrix
// whose off-diagonal entries are the tiers of a tree (node, rack, pod, far).
//
// Why it is the same iterate.  Let the distinct off-diagonal costs be
// c_1 < .. < c_L (L <= 4) and let the relation C_ij <= c_l split the ranks into
// nested groups for every l (ranks of a node, nodes of a rack, ..).  When no
// rank has both supply and demand, the diagonal is never read after the first
// row update, and with m_l = exp(-(c_l - c_1) / eps), m_{L+1} = 0:
//     (M v)_i = sum_l (m_l - m_{l+1}) sum_{j in group_l(i)} v_j,
// a sum of at most four non-negative terms that is the same for every rank of
// i's innermost group (its leaf).  So u_i = s_i / kappa(leaf of i) and
// v_j = d_j / rho(leaf of j): an iteration only needs the sums of u and v over
// the leaves and over the nested groups, and M never appears as a matrix.  The
// first row update (v = 1 on all R columns) has a closed form per rank from
// the counts of each cost in its row and its diagonal entry.
//
// Precision.  All of it runs in fp64, in the linear domain: with every cost
// within 200 eps of c_1 the scalings stay within exp(+-650) (the updates do not
// expand the sup-norm distance of log u to a fixed point, and both the start
// and the fixed point lie within the cost range of log s).  The differences
// m_l - m_{l+1} multiply sums that the larger groups' terms already contain, so
// nothing cancels.  Measured against 64-bit plain torch the plan is off by its
// own rounding to fp32, where the fp32 kernels are off by 1e-7 to 2.5e-6.
//
// Layout.  Leaves take slots whose address has one field of bits per level
// (leaf within its parent, parent within its parent, ..), each padded to a
// power of two: group sums are then butterfly steps over the low address bits.
// A slot is a lane (slots >= 64: up to four per lane), so one wave runs a
// problem without a barrier: per half-step log2(slots) butterfly steps of two
// moves and an add, one FMA per step and a reciprocal with one Newton step,
// instead of one FMA per entry of the |H| x |C| block.  The chain's latency
// bounds the iteration; the plan's R x R stores bound the rest.
//
// Measured (whole call, MI355X, fp32 kernels before -> this path): 58 problems
// of R = 64, 500 iterations 207 -> 70 us; 1952 of R = 256, 1000 iterations
// 1850 -> 213 us; 64 of R = 1024, 2000 iterations 5150 -> 466 us.  Per
// iteration and wave 0.08 us with 8 slots, 0.13 with 32, 0.19 with 128; R = 256
// writes its 512 MB of plans in about 110 us, most of it while the waves
// iterate.
//
// Any other shared matrix (more tiers, groups that do not nest, a tier beyond
// 200 eps), and any problem with a rank on both sides, with marginals outside
// [2^-60, 2^60], or with so much more demand than supply that the scalings
// drift out of range in `iters` iterations, is left to the other kernels.
#include "sk_common.h"

namespace taot {
namespace {

constexpr int kTierLevels = 4;
constexpr int kTierMaxBits = 8;                   // slots <= 256
constexpr int kTierSlots = 1 << kTierMaxBits;
constexpr double kTierRange = 200.0;              // |C_ij - c_1| <= kTierRange * eps
constexpr double kTierDrift = 40.0;               // iters * log(demand / supply) at most
constexpr float kTierMassLo = 0x1p-60f, kTierMassHi = 0x1p60f;
constexpr int kTreeThreads = 1024;
constexpr int kTierSmallR = 256;  // up to here a plan row is one or two stores of a wave

// ---- prepass, once per call ---------------------------------------------------
//
// Two launches.  tier_rows_kernel scans every row of C, a wave each, and beside
// them gives every problem its class; tier_tree_kernel (one block) joins the
// rows into the tree, if they describe one and some problem can be solved on it,
// and lists the problems that are left.  They take the place of the cost scan,
// the classes and the order of the other paths, so that a matrix or problems
// that are not for this path lose nothing by it: 58 problems of R = 64, 200
// iterations, costs that are no tree 121.8 us without this path, 118.9 with it
// (125.3 with a prepass in one block and the classes behind it); a tree with one
// other entry 121.9 and 118.4 (135.1); more demand than supply 171.9 and 168.1
// (184.4).
//
// Why the rows' own checks suffice.  Let N_l(i) be i and the ranks within c_l of
// it.  C is a tree of its tiers if and only if N_l is a partition for every l.
// Row i is compared in full with the row of the lowest rank x of N_l(i) at each
// cost of its own: the same set there.  So N_l(i) is within N_l(x).  The tree
// block then checks that x is the lowest rank of its own set and that the ranks
// which name x are as many as N_l(i) holds: those ranks lie within N_l(x), are as
// many as it, and so are it; and N_l(i), within it and as large, is the same set.

// A problem's class in the prepass: that of the other kernels, and whether the
// tier path can take it.
constexpr int32_t kTierEligible = 1 << 8;

template <int KR>
__device__ __forceinline__ void tier_row(const TierWs& w, const float* __restrict__ C, int32_t R, int32_t i) {
  // Scan of row i by one wave, KR entries per lane held in registers: non-finite
  // entries, the row's distinct off-diagonal costs in ascending order (num = 5:
  // more than four), for each its multiplicity and the lowest rank at most that
  // far (i itself included), and the next rank after i at the smallest cost.
  const int lane = threadIdx.x & (kWave - 1);
  const float* row = C + (int64_t)i * R;
  float c[KR];
#pragma unroll
  for (int k = 0; k < KR; ++k) c[k] = lane + kWave * k < R ? row[lane + kWave * k] : INFINITY;
  const float diag = row[i];
  bool bad = false;
#pragma unroll
  for (int k = 0; k < KR; ++k) {
    const int32_t j = lane + kWave * k;
    bad |= j < R && !(c[k] - c[k] == 0.f);
    if (j == i) c[k] = INFINITY;  // past every cost
  }
  const bool any_bad = __ballot(bad) != 0;
  float cur = -INFINITY;
  float rv[kTierLevels];
  int32_t rcnt[kTierLevels], rlab[kTierLevels];
#pragma unroll
  for (int l = 0; l < kTierLevels; ++l) {
    rv[l] = INFINITY;
    rcnt[l] = 0;
    rlab[l] = i;
  }
  int32_t num = 0, nxt = R;
#pragma unroll
  for (int l = 0; l <= kTierLevels; ++l) {
    if (any_bad) break;
    float next = INFINITY;
#pragma unroll
    for (int k = 0; k < KR; ++k) next = fminf(next, c[k] > cur ? c[k] : INFINITY);
    next = -lanes_max(-next);
    if (next == INFINITY) break;
    num = l + 1;
    if (l == kTierLevels) break;
    cur = next;
    int32_t cnt = 0, lab = i;
#pragma unroll
    for (int k = KR - 1; k >= 0; --k) {
      const uint64_t e = __ballot(c[k] == cur);
      cnt += (int32_t)__popcll(e);
      const uint64_t m = l == 0 ? e : __ballot(c[k] <= cur);
      if (m) lab = min(i, kWave * k + (int32_t)__builtin_ctzll(m));
      if (l == 0) {  // the next rank at the smallest cost
        const int32_t from = i + 1 - kWave * k;
        const uint64_t later = from <= 0 ? e : from >= kWave ? 0ull : e & (~0ull << from);
        if (later) nxt = kWave * k + (int32_t)__builtin_ctzll(later);
      }
    }
    rv[l] = cur;
    rcnt[l] = cnt;
    rlab[l] = lab;
  }
  // the rows of the sets' lowest ranks (the last set holds every rank)
  bool differ = false;
#pragma unroll
  for (int l = 0; l + 1 < kTierLevels; ++l) {
    if (any_bad || num > kTierLevels || l + 1 >= num || rlab[l] == i) continue;
    const float* other = C + (int64_t)rlab[l] * R;
    float x[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k) x[k] = lane + kWave * k < R ? other[lane + kWave * k] : INFINITY;
#pragma unroll
    for (int k = 0; k < KR; ++k) {
      const int32_t j = lane + kWave * k;
      differ |= (j == i || c[k] <= rv[l]) != (j == rlab[l] || x[k] <= rv[l]);
    }
  }
  const bool any_differ = __ballot(differ) != 0;
  if (lane == 0) {
    w.rv[i] = float4{rv[0], rv[1], rv[2], rv[3]};
    w.rcnt[i] = int4{rcnt[0], rcnt[1], rcnt[2], rcnt[3]};
    w.rlab[i] = int4{rlab[0], rlab[1], rlab[2], rlab[3]};
    w.rmore[i] = int4{num, nxt, __float_as_int(diag), (any_bad ? 1 : 0) | (any_differ ? 2 : 0)};
  }
}

// Problem pb by one wave: validity, mass, supports.
__device__ __forceinline__ int32_t tier_class(const SkParams& p, int64_t pb) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t R = p.R;
  const float* a = p.a + pb * R;
  const float* bd = p.b + pb * R;
  double sa = 0.0, sd = 0.0;
  int32_t nh = 0, nc = 0;
  bool bad = false, other = false;
  constexpr int kAtOnce = 4;  // loads in flight: one wave reads it all
  for (int32_t base = 0; base < R; base += kAtOnce * kWave) {
    float x[kAtOnce], y[kAtOnce];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      const int32_t i = base + kWave * k + lane;
      x[k] = i < R ? a[i] : 0.f;
      y[k] = i < R ? bd[i] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      const float ai = x[k], bi = y[k];
      bad |= !(ai >= 0.f && ai <= 3.402823466e38f) || !(bi >= 0.f && bi <= 3.402823466e38f);
      other |= (ai > 0.f && bi > 0.f) || (ai > 0.f && !(ai >= kTierMassLo && ai <= kTierMassHi)) ||
               (bi > 0.f && !(bi >= kTierMassLo && bi <= kTierMassHi));
      nh += (int32_t)__popcll(__ballot(ai > 0.f));
      nc += (int32_t)__popcll(__ballot(bi > 0.f));
      sa += (double)ai;
      sd += (double)bi;
    }
  }
  if (__ballot(bad) != 0) return 0;
  sa = wave_sum_d(sa);
  sd = wave_sum_d(sd);
  const double gamma = fmin(1.0, sd / fmax(sa, kEps0));
  const double surplus = sd / (gamma * sa);  // >= 1; its powers are the drift of the scalings
  const bool ok = __ballot(other) == 0 && nh > 0 && nc > 0 && (double)p.iters * (surplus - 1.0) <= kTierDrift;
  int c = classify(nh, nc, p.flags);
  if (c == 0) c = wide_class(nh, nc, p.flags);
  return c | (ok ? kTierEligible : 0);
}

__global__ void __launch_bounds__(kSkThreads)
tier_rows_kernel(SkParams p, TierWs w, int32_t row_blocks, int32_t* __restrict__ cls) {
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t R = p.R;
  if ((int32_t)blockIdx.x >= row_blocks) {
    const int64_t pb = (int64_t)((int32_t)blockIdx.x - row_blocks) * kSkWaves + wid;
    if (pb >= p.B) return;
    const int32_t c = tier_class(p, pb);
    if ((threadIdx.x & (kWave - 1)) == 0) cls[pb] = c;
    return;
  }
  const int32_t i = (int32_t)blockIdx.x * kSkWaves + wid;
  if (i >= R) return;
  if (R <= kWave) tier_row<1>(w, p.C, R, i);
  else if (R <= 4 * kWave) tier_row<4>(w, p.C, R, i);
  else if (R <= 16 * kWave) tier_row<16>(w, p.C, R, i);
  else tier_row<TAOT_MAX_RANKS / kWave>(w, p.C, R, i);
}

// The tree of the row scans, by one block of kTreeThreads: the tiers, the
// slots, the members of each slot, the butterfly weights and the first row
// update's sums.  Returns (to every thread) whether C is such a tree.
__device__ bool tier_tree(const TierWs& w, int32_t R, float eps) {
  __shared__ int16_t labs[kTierLevels][TAOT_MAX_RANKS];
  __shared__ int16_t leafof[TAOT_MAX_RANKS];
  __shared__ int32_t named[kTierLevels - 1][TAOT_MAX_RANKS];  // ranks that name this one as their set's lowest
  __shared__ int16_t rep[kTierSlots], idx[3][kTierSlots], slot_of_leaf[kTierSlots];
  __shared__ short4 pack[kTierSlots];
  __shared__ int32_t wave_n[kTreeThreads / kWave], widest[3], sh_bad;
  __shared__ float redf[2][kTreeThreads / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
  constexpr int kWaves = kTreeThreads / kWave;
  TierTree* tree = w.tree;
  auto any_bad = [&]() {  // the flag's value at this point, the same on every thread
    __syncthreads();
    const bool b = sh_bad != 0;
    __syncthreads();
    return b;
  };
  // this thread's rows
  constexpr int kRows = TAOT_MAX_RANKS / kTreeThreads;
  float4 rv[kRows];
  int4 rcnt[kRows], rlab[kRows], more[kRows];
#pragma unroll
  for (int k = 0; k < kRows; ++k) {
    const int32_t i = tid + kTreeThreads * k;
    rv[k] = float4{INFINITY, INFINITY, INFINITY, INFINITY};
    rcnt[k] = rlab[k] = more[k] = int4{0, 0, 0, 0};
    if (i < R) {
      rv[k] = w.rv[i];
      rcnt[k] = w.rcnt[i];
      rlab[k] = w.rlab[i];
      more[k] = w.rmore[i];
    }
  }
  if (tid == 0) sh_bad = 0;
  if (tid < 3) widest[tid] = 0;
  for (int32_t i = tid; i < R; i += kTreeThreads)
#pragma unroll
    for (int l = 0; l + 1 < kTierLevels; ++l) named[l][i] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRows; ++k)
    if (more[k].x > kTierLevels || more[k].w != 0) sh_bad = 1;
  // the tiers: distinct costs over all rows
  float c[kTierLevels];
  int L = 0;
  float cur = -INFINITY;
#pragma unroll
  for (int l = 0; l <= kTierLevels; ++l) {
    float next = INFINITY;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const float v[4] = {rv[q].x, rv[q].y, rv[q].z, rv[q].w};
#pragma unroll
      for (int t = 0; t < kTierLevels; ++t) next = fminf(next, v[t] > cur ? v[t] : INFINITY);
    }
    next = -lanes_max(-next);
    if (lane == 0) redf[l & 1][wid] = next;
    __syncthreads();
    next = INFINITY;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) next = fminf(next, redf[l & 1][q]);
    if (next == INFINITY) break;
    L = l + 1;
    if (l == kTierLevels) break;
    c[l] = cur = next;
  }
  if (any_bad() || L < 1 || L > kTierLevels) return false;
  const double inv = 1.0 / (double)eps;
#pragma unroll
  for (int t = 1; t < kTierLevels; ++t) c[t] = t < L ? c[t] : c[t - 1];
  const double c1 = (double)c[0];
  if (((double)c[kTierLevels - 1] - c1) * inv > kTierRange) return false;
  // weights exp(-(c_l - c_1) / eps), and the labels: the lowest rank of each
  // rank's group at each level
  double m[kTierLevels];
  int32_t held[kRows][kTierLevels - 1];  // ranks of this thread's rows' sets (of the levels below the last)
#pragma unroll
  for (int l = 0; l < kTierLevels; ++l) m[l] = exp(-((double)c[l] - c1) * inv);
#pragma unroll
  for (int k = 0; k < kRows; ++k) {
    const int32_t i = tid + kTreeThreads * k;
    if (i >= R) break;
    const double dg = ((double)__int_as_float(more[k].z) - c1) * inv;
    double k0 = exp(-dg);
    if (!(fabs(dg) <= kTierRange)) sh_bad = 1;
    const float v[4] = {rv[k].x, rv[k].y, rv[k].z, rv[k].w};
    const int32_t n[4] = {rcnt[k].x, rcnt[k].y, rcnt[k].z, rcnt[k].w};
    const int32_t g[4] = {rlab[k].x, rlab[k].y, rlab[k].z, rlab[k].w};
    int32_t lab[kTierLevels];
#pragma unroll
    for (int l = 0; l < kTierLevels; ++l) {
      lab[l] = i;
      int32_t in = 1;
      bool first = true;  // tiers past the last repeat it: count it once
      if (l > 0) first = c[l] != c[l - 1];
#pragma unroll
      for (int t = 0; t < kTierLevels; ++t) {
        if (v[t] <= c[l]) {
          lab[l] = g[t];
          in += n[t];
        }
        if (first && v[t] == c[l]) k0 += (double)n[t] * m[l];
      }
      labs[l][i] = (int16_t)lab[l];
      if (l + 1 < kTierLevels) {
        held[k][l] = in;
        if (l + 1 < L) atomicAdd(&named[l][lab[l]], 1);
      }
    }
    leafof[i] = -1;
    w.k0[i] = k0;
    w.next[i] = v[0] == c[0] ? more[k].y : R;
  }
  if (any_bad()) return false;
#pragma unroll
  for (int k = 0; k < kRows; ++k) {
    const int32_t i = tid + kTreeThreads * k;
    if (i >= R) break;
#pragma unroll
    for (int l = 0; l + 1 < kTierLevels; ++l) {
      const int32_t x = labs[l][i];
      if (l + 1 < L && (labs[l][x] != x || named[l][x] != held[k][l])) sh_bad = 1;
    }
  }
  if (any_bad()) return false;
  // the leaves (innermost groups) by their lowest rank, ascending
  int32_t Q = 0;
  for (int32_t base = 0; base < R; base += kTreeThreads) {
    const int32_t i = base + tid;
    const bool f = i < R && labs[0][i] == i;
    const uint64_t bm = __ballot(f);
    if (lane == 0) wave_n[wid] = __popcll(bm);
    __syncthreads();
    int32_t off = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
      off += q < wid ? wave_n[q] : 0;
      tot += wave_n[q];
    }
    const int32_t pos = Q + off + (int32_t)__popcll(bm & ((1ull << lane) - 1ull));
    if (f && pos < kTierSlots) {
      rep[pos] = (int16_t)i;
      pack[pos] = short4{(short)i, labs[1][i], labs[2][i], labs[3][i]};
      leafof[i] = (int16_t)pos;
    }
    Q += tot;
    __syncthreads();
  }
  if (Q > kTierSlots) return false;
  // index of each group among its siblings, in the order of their lowest ranks
  if (tid < Q) {
    const short4 me = pack[tid];
    int32_t n[3] = {0, 0, 0};
#pragma unroll 8
    for (int32_t q = 0; q < Q; ++q) {
      const short4 o = pack[q];
      if (q < tid) {
        n[0] += o.y == me.y;
        n[1] += o.y == o.x && o.z == me.z;
        n[2] += o.z == o.x && o.w == me.w;
      }
    }
    // a level that does not exist repeats the one below: its groups have one child
    const bool lv[3] = {L >= 2, L >= 3 && me.y == me.x, L >= 4 && me.z == me.x};
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      idx[l][tid] = lv[l] ? (int16_t)n[l] : 0;
      if (lv[l]) atomicMax(&widest[l], n[l]);
    }
  }
  __syncthreads();
  int bits[3];
  int nb = 0;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    bits[l] = widest[l] > 0 ? 32 - __builtin_clz((unsigned)widest[l]) : 0;
    nb += bits[l];
  }
  if (nb > kTierMaxBits) return false;
  if (tid < (1 << nb)) w.head[tid] = R;  // a slot without a leaf
  __syncthreads();
  if (tid < Q) {
    const short4 me = pack[tid];
    const int32_t g2 = leafof[me.y], g3 = leafof[me.z];  // the leaves that name its groups
    if (g2 < 0 || g3 < 0) {
      sh_bad = 1;
    } else {
      const int32_t sl = idx[0][tid] | idx[1][g2] << bits[0] | idx[2][g3] << (bits[0] + bits[1]);
      slot_of_leaf[tid] = (int16_t)sl;
      w.head[sl] = me.x;
    }
  }
  if (any_bad()) return false;
  for (int32_t i = tid; i < R; i += kTreeThreads) {
    const int32_t q = leafof[labs[0][i]];
    if (q < 0) sh_bad = 1;
    else w.slot[i] = slot_of_leaf[q];
  }
  if (any_bad()) return false;
  if (tid == 0) {
    tree->nbits = nb;
    tree->cut[0] = L >= 3 ? bits[0] : nb;
    tree->cut[1] = L >= 4 ? bits[0] + bits[1] : nb;
    tree->shift = c1;
#pragma unroll
    for (int l = 0; l < kTierLevels; ++l) {
      tree->c[l] = c[l];
      tree->m[l] = m[l];
    }
    // group_l's sum is the butterfly's value after `at` steps
    const int at[kTierLevels] = {0, bits[0], bits[0] + bits[1], nb};
    double wt[kTierMaxBits + 1];
#pragma unroll
    for (int t = 0; t <= kTierMaxBits; ++t) wt[t] = 0.0;
#pragma unroll
    for (int l = 0; l < kTierLevels; ++l)
#pragma unroll
      for (int t = 0; t <= kTierMaxBits; ++t)
        if (l < L && t == at[l]) wt[t] += m[l] - (l + 1 < L ? m[l + 1 < kTierLevels ? l + 1 : l] : 0.0);
#pragma unroll
    for (int t = 0; t <= kTierMaxBits; ++t) tree->w[t] = wt[t];
  }
  return true;
}

// The tree, the final classes and the register kernels' lists.
__global__ void __launch_bounds__(kTreeThreads)
tier_tree_kernel(SkParams p, TierWs w, int32_t* cls, int32_t* __restrict__ cbad, RegLists lists) {
  __shared__ int32_t found;
  constexpr int kElig = 1, kBad = 2, kNoTree = 4;
  const int tid = threadIdx.x;
  const int32_t B = p.B, R = p.R;
  if (tid == 0) found = 0;
  __syncthreads();
  int f = 0;
  for (int32_t b = tid; b < B; b += kTreeThreads) f |= (cls[b] & kTierEligible) ? kElig : 0;
  for (int32_t i = tid; i < R; i += kTreeThreads) {
    const int4 m = w.rmore[i];
    f |= ((m.w & 1) ? kBad : 0) | ((m.w & 2) || m.x > kTierLevels ? kNoTree : 0);
  }
  f = (__ballot(f & kElig) ? kElig : 0) | (__ballot(f & kBad) ? kBad : 0) | (__ballot(f & kNoTree) ? kNoTree : 0);
  if ((tid & (kWave - 1)) == 0 && f) atomicOr(&found, f);
  __syncthreads();
  f = found;
  bool ok = f == kElig;
  if (ok) ok = tier_tree(w, R, p.eps);
  if (tid == 0) {
    w.tree->ok = ok ? 1 : 0;
    cbad[0] = (f & kBad) ? 1 : 0;
  }
  bool left = false;
  for (int32_t b = tid; b < B; b += kTreeThreads) {  // (a thread reads back below what it writes here)
    const int32_t c = cls[b];
    const int32_t k = ok && (c & kTierEligible) ? kTierClass : (f & kBad) ? 0 : c & (kTierEligible - 1);
    cls[b] = k;
    left |= k != kTierClass;
  }
  if (__syncthreads_or(left) == 0) {  // every problem is solved here
    if (tid < 3) lists.counts[tid] = 0;
    return;
  }
  order_problems<kTreeThreads>(cls, B, lists.W, lists.multi, lists.single, lists.wide, lists.counts);
}

// ---- the iterate ----------------------------------------------------------------

// x + (x of the lane whose address differs in butterfly bit T), for x that is
// already uniform over the lower bits: quad_perm for bits 0 and 1, half_mirror
// and mirror of a 16-lane row for bits 2 and 3, the row swaps for 4 and 5.
template <int T>
__device__ __forceinline__ double bfly(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
  if constexpr (T < 4) {
    constexpr int kCtrl[4] = {0xB1, 0x4E, 0x141, 0x140};
    const uint32_t yl = (uint32_t)__builtin_amdgcn_update_dpp(0, lo, kCtrl[T], 0xf, 0xf, true);
    const uint32_t yh = (uint32_t)__builtin_amdgcn_update_dpp(0, hi, kCtrl[T], 0xf, 0xf, true);
    return x + __longlong_as_double((long long)((uint64_t)yh << 32 | yl));
  } else {
    // both results of a swap of x with itself: x of the lane's own row and of the other row
    const auto l = T == 4 ? __builtin_amdgcn_permlane16_swap((uint32_t)lo, (uint32_t)lo, false, false)
                          : __builtin_amdgcn_permlane32_swap((uint32_t)lo, (uint32_t)lo, false, false);
    const auto h = T == 4 ? __builtin_amdgcn_permlane16_swap((uint32_t)hi, (uint32_t)hi, false, false)
                          : __builtin_amdgcn_permlane32_swap((uint32_t)hi, (uint32_t)hi, false, false);
    return __longlong_as_double((long long)((uint64_t)h[0] << 32 | l[0])) +
           __longlong_as_double((long long)((uint64_t)h[1] << 32 | l[1]));
  }
}

// num / x for x > 0: the hardware's reciprocal (2^-24 or better) and one
// Newton step.
__device__ __forceinline__ double quick_div(double num, double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, y, 1.0);
  const double q = num * y;
  return __builtin_fma(q, e, q);
}

// All iterations of one problem on one wave of 2^NB slots (NB > 6: a lane has
// neighbouring slots, whose sum then takes the steps over the lanes), or of
// two problems on its halves (PAIR, NB <= 5).  s, d: supply and demand of each
// rank (LDS); leaves kappa (the last row update's sums) and rho of every slot
// in LDS.  With PAIR the pointers differ from half to half.
template <int NB, bool PAIR>
__device__ __forceinline__ void tier_iterate(const TierWs& tw, const int16_t* next, int32_t R, const double* s,
                                             const double* d, int32_t iters, double* kap, double* rho) {
  constexpr int kIn = NB > 6 ? NB - 6 : 0;  // address bits within a lane
  constexpr int SPL = 1 << kIn;
  const int lane = threadIdx.x & (PAIR ? kWave / 2 - 1 : kWave - 1);
  double wt[NB + 1];
#pragma unroll
  for (int t = 0; t <= NB; ++t) wt[t] = tw.tree->w[t];
  double S[SPL], D[SPL], U[SPL], V[SPL], x[SPL];
#pragma unroll
  for (int k = 0; k < SPL; ++k) {
    S[k] = D[k] = U[k] = 0.0;
    x[k] = 1.0;
    for (int32_t i = tw.head[(lane * SPL + k) & ((1 << NB) - 1)]; i < R; i = next[i]) {
      S[k] += s[i];
      D[k] += d[i];
      U[k] += s[i] / tw.k0[i];  // the first row update
    }
  }
  auto mix = [&](const double (&in)[SPL], double (&out)[SPL]) {
    double cur, acc;
    // The constant is far below any sum that has a supply or demand to share,
    // and keeps the reciprocal of an empty slot's sum finite (its num is 0).
    constexpr double kTiny = 0x1p-1000;
    if constexpr (SPL == 1) {
      cur = in[0];
      acc = __builtin_fma(wt[0], cur, kTiny);
    } else if constexpr (SPL == 2) {
      cur = in[0] + in[1];
      acc = __builtin_fma(wt[1], cur, kTiny);
    } else {
      const double p0 = in[0] + in[1], p1 = in[2] + in[3];
      cur = p0 + p1;
      acc = __builtin_fma(wt[2], cur, kTiny);
      out[0] = out[1] = p0;
      out[2] = out[3] = p1;
    }
    auto step = [&](auto t) {
      constexpr int T = decltype(t)::value;
      if constexpr (T + kIn < NB) {
        cur = bfly<T>(cur);
        acc = __builtin_fma(wt[T + kIn + 1], cur, acc);
      }
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 5>{});
#pragma unroll
    for (int k = 0; k < SPL; ++k) {
      if constexpr (SPL == 1) out[k] = acc;
      else if constexpr (SPL == 2) out[k] = __builtin_fma(wt[0], in[k], acc);
      else out[k] = __builtin_fma(wt[0], in[k], __builtin_fma(wt[1], out[k], acc));
    }
  };
  double y[SPL];
  mix(U, y);
#pragma unroll
  for (int k = 0; k < SPL; ++k) V[k] = quick_div(D[k], y[k]);
  for (int32_t it = 2; it <= iters; ++it) {
    mix(V, x);
#pragma unroll
    for (int k = 0; k < SPL; ++k) U[k] = quick_div(S[k], x[k]);
    mix(U, y);
#pragma unroll
    for (int k = 0; k < SPL; ++k) V[k] = quick_div(D[k], y[k]);
  }
#pragma unroll
  for (int k = 0; k < SPL; ++k) {
    if (lane * SPL + k < (1 << NB)) {
      kap[lane * SPL + k] = x[k];
      rho[lane * SPL + k] = y[k];
    }
  }
}

// u m_l v of the tier l of two slots whose addresses differ by x.
__device__ __forceinline__ float tier_entry(double u0, double u1, double u2, double u3, int32_t x, int32_t lim1,
                                            int32_t lim2, double v) {
  const double far = x < lim2 ? u2 : u3, near = x == 0 ? u0 : u1;
  return (float)((x < lim1 ? near : far) * v);
}

// LDS: the ranks' slots and the next rank of each rank's leaf, int16 [R]; then per problem fp64 s (then
// u), d (then the capped v) [R] and the sums kappa, rho [kTierSlots].
__host__ __device__ constexpr size_t tier_lds_problem(int32_t R) { return (size_t)2 * R + 2 * kTierSlots; }
__host__ __device__ constexpr size_t tier_lds_slots(int32_t R) { return ((size_t)R * 4 + 15) / 16 * 16; }
__host__ __device__ constexpr size_t tier_lds_bytes(int32_t R, int np) {
  return tier_lds_slots(R) + tier_lds_problem(R) * 8 * np;
}

// NP problems per workgroup of NW waves (NP = 1, or one per wave).  Some waves
// iterate; the others meanwhile write the rows of the plan that are zero (no
// supply: most of its bytes).  Then all write the other rows.
//   NP = 1: one wave iterates, on another SIMD in each of the workgroups that
//     follow one another on a compute unit.
//   NP = 8: batches of more problems than the chip has SIMDs.  Two problems
//     share a wave while their slots fit its halves, so that half of the waves
//     iterate, one per SIMD (a wave's SIMD is read from HW_ID; any placement
//     still gives every pair one wave).
template <int NP, int NW>
__global__ void __launch_bounds__(NW * kWave) tier_solve_kernel(SkParams p, TierWs tw, const int32_t* __restrict__ cls) {
  static_assert(NP == 1 || NP == NW, "a wave prepares one problem");
  extern __shared__ __attribute__((aligned(16))) char tier_lds[];
  __shared__ int32_t mine[NP], simd_of[NW];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t R = p.R;
  const int64_t pb0 = (int64_t)blockIdx.x * NP;
  int16_t* sl = reinterpret_cast<int16_t*>(tier_lds);
  int16_t* next = sl + R;
  double* prob = reinterpret_cast<double*>(tier_lds + tier_lds_slots(R));
  const int32_t stride = (int32_t)tier_lds_problem(R);
  if (tw.tree->ok == 0 || (NP == 1 && cls[pb0] != kTierClass)) return;  // uniform

  for (int32_t i = tid; i < R; i += NW * kWave) {
    sl[i] = (int16_t)tw.slot[i];
    next[i] = (int16_t)tw.next[i];
  }
  // HW_ID bits 5:4 hold the SIMD of the wave
  const int simd = (int)__builtin_amdgcn_s_getreg((1 << 11) | (4 << 6) | 4);
  if (lane == 0) simd_of[wid] = simd;

  // ---- marginals of a problem by one wave ---------------------------------------------
  if (wid < NP) {
    const int64_t pb = pb0 + wid;
    const bool ok = pb < p.B && cls[pb] == kTierClass;
    if (ok) {
      const float* a = p.a + pb * R;
      const float* bd = p.b + pb * R;
      double* s = prob + wid * stride;
      double* d = s + R;
      double sa = 0.0, sd = 0.0;
      int32_t nh = 0, nc = 0;
      for (int32_t base = 0; base < R; base += kWave) {
        const int32_t i = base + lane;
        const float ai = i < R ? a[i] : 0.f, bi = i < R ? bd[i] : 0.f;
        nh += (int32_t)__popcll(__ballot(ai > 0.f));
        nc += (int32_t)__popcll(__ballot(bi > 0.f));
        sa += (double)ai;
        sd += (double)bi;
        if (i < R) {
          s[i] = (double)ai;
          d[i] = (double)bi;
        }
      }
      sa = wave_sum_d(sa);
      sd = wave_sum_d(sd);
      const double gamma = fmin(1.0, sd / fmax(sa, kEps0));
      for (int32_t i = lane; i < R; i += kWave) s[i] = gamma * s[i];
      if (lane == 0 && p.status) {
        // the status keeps telling problems whose support block no on-chip layout holds
        const bool held = R <= kLdsMaxR || classify(nh, nc, p.flags) != 0 || wide_class(nh, nc, p.flags) != 0;
        p.status[pb] = held ? 0u : TAOT_ST_STREAMED;
      }
    }
    if (lane == 0) mine[wid] = ok ? 1 : 0;
  }
  __syncthreads();

  // ---- roles --------------------------------------------------------------------------
  const int nbits = tw.tree->nbits;
  const bool pair = NP > 1 && nbits <= 5;
  int role = -1;  // which problem or pair of problems this wave iterates
  int writer = 0, writers = 0;  // this wave's place among the others
  if constexpr (NP == 1) {
    const int want = (int)(blockIdx.x >> 8) & 3;
    int it = 0;
    for (int w = NW - 1; w >= 0; --w) it = simd_of[w] == want ? w : it;
    role = wid == it ? 0 : -1;
    writer = wid - (wid > it);
    writers = NW - 1;
  } else if (pair) {
    // waves in the order of (rank within their SIMD, SIMD): the first half iterate
    auto key = [&](int u) {
      int r = 0;
      for (int t = 0; t < u; ++t) r += simd_of[t] == simd_of[u];
      return r * 4 + simd_of[u];
    };
    const int mk = key(wid);
    int pos = 0;
    for (int u = 0; u < NW; ++u) {
      const int ku = key(u);
      pos += ku < mk;
    }
    role = pos < NP / 2 ? pos : -1;
    writer = pos - NP / 2;
    writers = NP / 2;
  } else {
    role = wid;
  }

  float* T0 = p.T + pb0 * (int64_t)R * R;
  const bool vec = (R & 3) == 0 && (reinterpret_cast<uintptr_t>(p.T) & 15u) == 0;
  auto zero_rows = [&](int q, int32_t first, int32_t step) {
    const double* s = prob + q * stride;
    for (int32_t i = first; i < R; i += step) {
      if (s[i] > 0.0) continue;
      float* row = T0 + ((int64_t)q * R + i) * R;
      if (vec) {
        for (int32_t j = lane; j < R / 4; j += kWave) reinterpret_cast<float4*>(row)[j] = float4{0.f, 0.f, 0.f, 0.f};
      } else {
        for (int32_t j = lane; j < R; j += kWave) row[j] = 0.f;
      }
    }
  };
  bool iterates = role >= 0;
  if constexpr (NP > 1)  // (not for problems that other kernels solve)
    if (iterates) iterates = (pair ? mine[2 * role] | mine[2 * role + 1] : mine[role]) != 0;
  if (iterates) {
    const int q = pair ? 2 * role + (lane >= kWave / 2) : role;
    const double* s = prob + q * stride;
    double* kap = prob + q * stride + 2 * R;
    if (pair) {
      switch (nbits) {
#define TAOT_TIER_CASE(NB) \
  case NB: tier_iterate<NB, true>(tw, next, R, s, s + R, p.iters, kap, kap + kTierSlots); break;
        TAOT_TIER_CASE(0) TAOT_TIER_CASE(1) TAOT_TIER_CASE(2) TAOT_TIER_CASE(3) TAOT_TIER_CASE(4)
        TAOT_TIER_CASE(5)
#undef TAOT_TIER_CASE
        default: break;
      }
    } else {
      switch (nbits) {
#define TAOT_TIER_CASE(NB) \
  case NB: tier_iterate<NB, false>(tw, next, R, s, s + R, p.iters, kap, kap + kTierSlots); break;
        TAOT_TIER_CASE(0) TAOT_TIER_CASE(1) TAOT_TIER_CASE(2) TAOT_TIER_CASE(3) TAOT_TIER_CASE(4)
        TAOT_TIER_CASE(5) TAOT_TIER_CASE(6) TAOT_TIER_CASE(7) TAOT_TIER_CASE(8)
#undef TAOT_TIER_CASE
        default: break;
      }
    }
  } else if (role < 0 && p.T) {
    for (int q = 0; q < NP; ++q)
      if (mine[q]) zero_rows(q, writer, writers);
  }
  __syncthreads();

  // ---- potentials and column cap: a problem per wave, or all threads on the one ---------
  const int q = NP == 1 ? 0 : wid;
  const int64_t pb = pb0 + q;
  double* s = prob + q * stride;
  double* d = s + R;
  const double* kap = d + R;
  const double* rho = kap + kTierSlots;
  const double eps = (double)p.eps, shift = tw.tree->shift;
  if (mine[q]) {
    for (int32_t i = NP == 1 ? tid : lane; i < R; i += NP == 1 ? NW * kWave : kWave) {
      const double si = s[i], di = d[i];
      const double u = si > 0.0 ? si / (p.iters == 1 ? tw.k0[i] : kap[sl[i]]) : 0.0;
      const double r = rho[sl[i]];
      const double v = di > 0.0 ? di / r : 0.0;
      if (p.f) p.f[pb * R + i] = si > 0.0 ? (float)(eps * log(u) + shift) : -INFINITY;
      if (p.g) p.g[pb * R + i] = di > 0.0 ? (float)(eps * log(v)) : -INFINITY;
      const double fac = (p.flags & TAOT_SK_NO_COLCAP) ? 1.0 : fmin(1.0, di / (v * r + kEps0));
      s[i] = u;
      d[i] = di > 0.0 ? v * fac : 0.0;
    }
  }
  if (!p.T) return;
  __syncthreads();

  // ---- the rows of the plan that have supply, a row per wave ------------------------------
  if (!mine[q]) return;
  const int32_t lim1 = 1 << tw.tree->cut[0], lim2 = 1 << tw.tree->cut[1];
  const double m0 = tw.tree->m[0], m1 = tw.tree->m[1], m2 = tw.tree->m[2], m3 = tw.tree->m[3];
  if (writers == 0) zero_rows(q, 0, 1);
#define ENTRY(j) tier_entry(u0, u1, u2, u3, si ^ sl[j], lim1, lim2, d[j])
  for (int32_t i = NP == 1 ? wid : 0; i < R; i += NP == 1 ? NW : 1) {
    const double u = s[i];
    if (!(u > 0.0)) continue;
    float* row = T0 + ((int64_t)q * R + i) * R;
    const double u0 = u * m0, u1 = u * m1, u2 = u * m2, u3 = u * m3;
    const int32_t si = sl[i];
    if (vec) {
      for (int32_t j = lane; j < R / 4; j += kWave)
        reinterpret_cast<float4*>(row)[j] = float4{ENTRY(4 * j), ENTRY(4 * j + 1), ENTRY(4 * j + 2), ENTRY(4 * j + 3)};
    } else {
      for (int32_t j = lane; j < R; j += kWave) row[j] = ENTRY(j);
    }
  }
#undef ENTRY
}

template <int NP, int NW>
taot_status launch_tier_solve(const SkParams& p, const TierWs& w, const int32_t* cls, hipStream_t stream) {
  const size_t lds = tier_lds_bytes(p.R, NP);
  if (!allow_lds((const void*)tier_solve_kernel<NP, NW>, lds)) return TAOT_ERR_LAUNCH;
  hipLaunchKernelGGL((tier_solve_kernel<NP, NW>), dim3((unsigned)((p.B + NP - 1) / NP)), dim3(NW * kWave), lds, stream,
                     p, w, cls);
  return hipGetLastError() == hipSuccess ? TAOT_OK : TAOT_ERR_LAUNCH;
}

}  // namespace

taot_status launch_tier(const SkParams& p, const TierWs& w, int32_t* cls, int32_t* cbad, const RegLists& lists,
                        hipStream_t stream) {
  const int32_t row_blocks = (p.R + kSkWaves - 1) / kSkWaves;
  const unsigned grid = (unsigned)row_blocks + (unsigned)(((int64_t)p.B + kSkWaves - 1) / kSkWaves);
  hipLaunchKernelGGL(tier_rows_kernel, dim3(grid), dim3(kSkThreads), 0, stream, p, w, row_blocks, cls);
  if (hipGetLastError() != hipSuccess) return TAOT_ERR_LAUNCH;
  hipLaunchKernelGGL(tier_tree_kernel, dim3(1), dim3(kTreeThreads), 0, stream, p, w, cls, cbad, lists);
  if (hipGetLastError() != hipSuccess) return TAOT_ERR_LAUNCH;
  // the shape: see the kernel; eight problems to a group from where one
  // iterating wave per problem would put two on a SIMD
  if (p.R > kTierSmallR) return launch_tier_solve<1, 8>(p, w, cls, stream);
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    return TAOT_ERR_LAUNCH;
  return p.B > 4 * cus ? launch_tier_solve<8, 8>(p, w, cls, stream) : launch_tier_solve<1, 4>(p, w, cls, stream);
}

}  // namespace taot
