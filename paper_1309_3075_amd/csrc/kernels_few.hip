// Generic kernels for few patterns (a trait column, any K <= 64).
//
// With one or a few patterns the tree is the only parallelism: most levels of a coalescent tree
// hold a handful of nodes, and a launch per level costs 4-6 us plus the gap before the next one
// whatever it computes.  These kernels differ from the per-level ones of kernels_generic.hip in
// three ways, with the same arithmetic term by term (so the same bits):
//   - consecutive narrow levels run as one launch of one block, which keeps the partials (or the
//     outside vectors) of its nodes in LDS, one block barrier or two per level, and loads the next
//     level's matrix rows while it finishes the current one;
//   - other levels are launches over (node, pattern) items with lanes for an item's states only (a
//     block per node left 248 of 256 threads idle for 7 states and one pattern);
//   - with a gradient, the post-order pass keeps every branch's child vector S_v = P_v L_v, which the
//     pre-order pass and dlogL/dP would otherwise form again from the matrices.
// 522 taxa, 7 states, one column, FP64: the post- and pre-order passes took 294 us in 64 launches and
// take 77 us in two; 2,000 taxa, 40 states, FP32: 253 us in 44 launches, now 190 us in 25, and dlogL/dP
// 66 -> 45 us.  What is left of a run is latency: about 0.7 us a level down, 1.2 us up.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "device_common.h"
#include "generic_common.h"
#include "instance.h"

namespace epochlik {

namespace {

// Trait data hold one column or a few.  The line is where these kernels were tried, not where the
// per-level kernels overtake: with branch gradients, 7 states, 200 taxa, FP64, those and these take 164
// and 118 us at 16 patterns, 193 and 164 at 64.
constexpr int kFewMaxPatterns = 16;
constexpr size_t kFewLds = 64 * 1024;          // LDS of a run of levels, at most, besides its matrix buffers
constexpr size_t kFewVectorBytes = 256 << 20;  // child vectors, at most
// Blocks of a post-order level launch, until they are full: a block of items from several nodes reads
// their matrices through one CU, and its wavefronts walk every kind of child among them.  40 states,
// 64 taxa, one column, FP64, four categories, post-order pass: 177 us in full blocks, 159 in these.
constexpr int kFewBlocks = 2048;
// A level runs in one block while it takes it at most this many passes, and while its matrices are no more
// than one CU reads in about the time of a launch (a lane per row, of more than a cache line from 32
// states in FP64 on, reads slower than a wavefront per matrix).  FP64, one category, without gradient,
// per-level kernels, runs by the number of items alone, and by both: 20 states (generic kernels), 64
// taxa, 16 columns 104, 162 and 99 us; 12 states, 1,500 taxa, 8 columns 137, 157 and 138; 40 states,
// 1,500 taxa, one column 219, 195 and 191.
constexpr int kFewWide = 2;
constexpr size_t few_run_bytes(int lanes) { return (lanes == 32 ? 128 : 256) * 1024; }

// Orders LDS accesses of one wavefront (write, then read by other lanes).
__device__ inline void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One matrix of an item, loaded a level ahead.  Up to 32 states a lane holds its own row or column;
// from 33 on (an item is a whole wavefront) the wavefront loads the matrix in consecutive 16-byte
// pieces and passes it through an LDS buffer with padded rows, because a row per lane touches 64
// cache lines with every load and drops each before it has used it up.
template <typename T, int KQ, int COLS>
struct ItemMatrix {
  static constexpr bool kStaged = KQ == 64;
  static constexpr int W = 16 / sizeof(T);
  static constexpr int LDR = COLS + W;                                       // LDS row stride, elements
  static constexpr int NV = kStaged ? COLS * COLS / (64 * W) : COLS / W;     // 16-byte pieces per lane
  static constexpr size_t kLds = kStaged ? (size_t)COLS * LDR * sizeof(T) : 0;  // bytes per item
  typedef T vec __attribute__((ext_vector_type(W), aligned(16)));
  vec v[NV];

  __device__ inline void load_rows(const T* __restrict__ M, int i) {
    if constexpr (kStaged) {
      const vec* src = reinterpret_cast<const vec*>(M) + i;
#pragma unroll
      for (int k = 0; k < NV; ++k) v[k] = src[64 * k];
    } else {
      const vec* src = reinterpret_cast<const vec*>(M + i * COLS);
#pragma unroll
      for (int k = 0; k < NV; ++k)
        v[k] = src[k];
    }
  }
  __device__ inline void load_columns(const T* __restrict__ M, int i) {
    if constexpr (kStaged) {
      load_rows(M, i);
    } else {
#pragma unroll
      for (int j = 0; j < COLS; ++j)
        v[j / W][j % W] = M[j * COLS + i];
    }
  }
  __device__ inline void stage(T* buf, int i) const {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int e = (64 * k + i) * W;
      *reinterpret_cast<vec*>(buf + (e / COLS) * LDR + e % COLS) = v[k];
    }
    wave_lds_order();
  }
  // sum_j M[i][j] x[j] and sum_j M[j][i] x[j], in order of j (the padding's terms are zero)
  __device__ inline T row_dot(const T* buf, const T* x, int i) const {
    T r = 0;
    if constexpr (kStaged) {
      const T* row = buf + (i < COLS ? i : 0) * LDR;
#pragma unroll
      for (int j = 0; j < COLS; ++j) r += row[j] * x[j];
    } else {
#pragma unroll
      for (int j = 0; j < COLS; ++j)
        r += v[j / W][j % W] * x[j];
    }
    return r;
  }
  __device__ inline T column_dot(const T* buf, const T* x, int i) const {
    T r = 0;
    if constexpr (kStaged) {
      const T* col = buf + (i < COLS ? i : 0);
#pragma unroll
      for (int j = 0; j < COLS; ++j) r += col[j * LDR] * x[j];
    } else {
#pragma unroll
      for (int j = 0; j < COLS; ++j)
        r += v[j / W][j % W] * x[j];
    }
    return r;
  }
};

// Maximum over the KQ lanes of an item: DPP moves up to 16 lanes, lane exchanges beyond.
template <int CTRL>
__device__ inline float lanes_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ inline double lanes_mov(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int KQ, typename T>
__device__ inline T item_max(T v) {
  T u = lanes_mov<0xB1>(v);  // quad_perm [1,0,3,2]
  v = u > v ? u : v;
  u = lanes_mov<0x4E>(v);  // quad_perm [2,3,0,1]
  v = u > v ? u : v;
  if constexpr (KQ >= 8) {
    u = lanes_mov<0x141>(v);  // row_half_mirror: the other four lanes of eight
    v = u > v ? u : v;
  }
  if constexpr (KQ >= 16) {
    u = lanes_mov<0x140>(v);  // row_mirror: the other eight of sixteen
    v = u > v ? u : v;
  }
#pragma unroll
  for (int o = 16; o < KQ; o <<= 1) {
    u = __shfl_xor(v, o, 64);
    v = u > v ? u : v;
  }
  return v;
}

template <typename T>
struct FewArgs {
  const int32_t* data;  // the run's or the level's items
  int n_ints, n_levels, n_nodes, n_tips, max_branches;
  const int32_t *left, *right;
  const T* Pm;
  const uint8_t* tips;
  const uint64_t* amb;
  T* part;
  T* pre;
  int32_t* scales;
  T* S;  // [n_nodes, or tips][C][P][Kp] child vectors
  bool keep;  // every branch's child vector is kept for the gradient (else the tips' of a run, for the run itself)
  const double* pi;
  int root, N, P, K, Kp, C;
  unsigned inv_P;  // ceil(2^32 / P), 0 for one pattern
};

// Item k of a run or level as (place in its list, pattern): k (P - 1) < 2^32, so the quotient is the
// high half of one product.
struct Place {
  int node, p;
};
template <typename T>
__device__ inline Place place_of(const FewArgs<T>& g, int k) {
  const int q = g.inv_P ? (int)__umulhi((unsigned)k, g.inv_P) : k;
  return Place{q, k - q * g.P};
}

// ---------------------------------------------------------------------------
// Post-order, one level: an item is (node, pattern), KQ lanes each.
template <typename T, int KQ>
__global__ __launch_bounds__(256) void few_post_level_kernel(const FewArgs<T> g, const int32_t* __restrict__ nodes,
                                                             int n, int per) {
  __shared__ T sA[256], sB[256];
  const int i = threadIdx.x % KQ, item = blockIdx.x * per + threadIdx.x / KQ;
  const bool ok = (int)threadIdx.x / KQ < per && item < n * g.P;
  const Place at = place_of(g, ok ? item : blockIdx.x * per);  // idle lanes repeat the block's first item
  const int u = nodes[at.node], p = at.p;
  const int a = g.left[u], b = g.right[u];
  const int N = g.N, P = g.P, K = g.K, Kp = g.Kp, C = g.C;
  const size_t KK = (size_t)Kp * Kp;
  const int own = threadIdx.x - i;  // first LDS entry of this item
  T x[kMaxCategories];
  for (int c = 0; c < C; ++c) {
    if (a >= N) sA[threadIdx.x] = i < Kp ? g.part[(((size_t)(a - N) * C + c) * P + p) * Kp + i] : T(0);
    if (b >= N) sB[threadIdx.x] = i < Kp ? g.part[(((size_t)(b - N) * C + c) * P + p) * Kp + i] : T(0);
    wave_lds_order();
    T va = 0, vb = 0;
    if (i < K) {
      va = child_vector(a, N, p, P, K, Kp, i, g.Pm + ((size_t)a * C + c) * KK + (size_t)i * Kp, g.tips, g.amb, sA + own);
      vb = child_vector(b, N, p, P, K, Kp, i, g.Pm + ((size_t)b * C + c) * KK + (size_t)i * Kp, g.tips, g.amb, sB + own);
    }
    if (g.keep && ok && i < Kp) {
      g.S[(((size_t)a * C + c) * P + p) * Kp + i] = va;
      g.S[(((size_t)b * C + c) * P + p) * Kp + i] = vb;
    }
    x[c] = va * vb;
    wave_lds_order();
  }
  T mx = 0;
  for (int c = 0; c < C; ++c) mx = x[c] > mx ? x[c] : mx;
  const int e = scale_exponent(item_max<KQ>(mx));
  if (!ok) return;
  if (i < Kp)
    for (int c = 0; c < C; ++c)
      g.part[(((size_t)(u - N) * C + c) * P + p) * Kp + i] = i < K ? scale_by_pow2(x[c], e) : T(0);
  if (i == 0)
    g.scales[(size_t)(u - N) * P + p] = e + (a >= N ? g.scales[(size_t)(a - N) * P + p] : 0) +
                                       (b >= N ? g.scales[(size_t)(b - N) * P + p] : 0);
}

// Threads of a run's block: as many items as the registers (up to 32 states) or the LDS buffers of
// their matrices (about 70 to 80 KB) allow.
constexpr int few_threads(bool fp64, int kp) {
  return kp <= 32 ? 1024 : 64 * (kp == 48 ? (fp64 ? 4 : 8) : (fp64 ? 2 : 4));
}

// Post-order of consecutive narrow levels by one block (one category).  data: node offsets
// [n_levels + 1], branch offsets [n_levels + 1], nodes {u, ra, rb, slot}, branches {v, slot}, tips
// {v}; ra / rb: the child's place among its level's branches, or ~v for a tip; a branch's slot: the
// LDS place of its child's partial, or -1 when an earlier launch formed it.  Per level, the branches'
// child vectors S_v (one matrix row per lane, its loads issued a level ahead), a barrier, the nodes'
// partials, a barrier.
template <typename T, int KQ, int COLS, int NT>
__global__ __launch_bounds__(NT) void few_post_run_kernel(const FewArgs<T> g) {
  constexpr int G = NT / KQ;
  extern __shared__ __align__(16) unsigned char few_lds[];
  constexpr int Kp = COLS;  // the padded states: KQ up to 32, else 48 or 64
  constexpr size_t KK = (size_t)Kp * Kp;
  const int N = g.N, P = g.P, K = g.K;
  T* const sL = reinterpret_cast<T*>(few_lds);                          // [n_nodes][P][KQ]
  T* const sS = sL + (size_t)g.n_nodes * P * KQ;                        // [max_branches][P][KQ]
  typedef ItemMatrix<T, KQ, COLS> Matrix;
  T* const sM = sS + (size_t)g.max_branches * P * KQ;                   // [G] matrices (33 states or more)
  int* const sE = reinterpret_cast<int*>(reinterpret_cast<char*>(sM) + G * Matrix::kLds);  // [n_nodes][P]
  int* const data = sE + g.n_nodes * P;
  for (int t = threadIdx.x; t < g.n_ints; t += NT) data[t] = g.data[t];
  __syncthreads();
  const int* const node_off = data;
  const int* const br_off = data + g.n_levels + 1;
  const int* const nodes = br_off + g.n_levels + 1;
  const int* const branches = nodes + 4 * g.n_nodes;
  const int* const tip = branches + 2 * br_off[g.n_levels];
  const int grp = threadIdx.x / KQ, i = threadIdx.x % KQ;
  const bool row_ok = i < Kp;
  for (int k = grp; k < g.n_tips * P; k += G) {  // the tip children's vectors
    const Place at = place_of(g, k);
    const int v = tip[at.node], p = at.p;
    if (row_ok)
      g.S[((size_t)v * P + p) * Kp + i] =
          i < K ? child_vector(v, N, p, P, K, Kp, i, g.Pm + (size_t)v * KK + (size_t)i * Kp, g.tips, g.amb, (const T*)nullptr)
                : T(0);
  }
  __syncthreads();
  // operands of this group's first branch and node of a level, loaded a level ahead
  Matrix mat;
  T* const buf = sM + grp * (Matrix::kLds / sizeof(T));
  T out_L = 0, tip_a = 0, tip_b = 0;
  int out_sa = 0, out_sb = 0;
  auto load_branch = [&](int l, int k) {
    const Place at = place_of(g, k);
    const int* br = branches + 2 * (br_off[l] + at.node);
    mat.load_rows(g.Pm + (size_t)br[0] * KK, i);
    out_L = br[1] < 0 && row_ok ? g.part[((size_t)(br[0] - N) * P + at.p) * Kp + i] : T(0);
  };
  auto child_exponent = [&](int l, int ref, int p) {  // of a child formed by an earlier launch
    if (ref < 0) return 0;
    const int* br = branches + 2 * (br_off[l] + ref);
    return br[1] < 0 ? g.scales[(size_t)(br[0] - N) * P + p] : 0;
  };
  auto load_node = [&](int l, int k) {
    const Place at = place_of(g, k);
    const int* nd = nodes + 4 * (node_off[l] + at.node);
    const int p = at.p;
    tip_a = nd[1] < 0 && row_ok ? g.S[((size_t)~nd[1] * P + p) * Kp + i] : T(0);
    tip_b = nd[2] < 0 && row_ok ? g.S[((size_t)~nd[2] * P + p) * Kp + i] : T(0);
    out_sa = child_exponent(l, nd[1], p);
    out_sb = child_exponent(l, nd[2], p);
  };
  if (grp < (br_off[1] - br_off[0]) * P) load_branch(0, grp);
  if (grp < (node_off[1] - node_off[0]) * P) load_node(0, grp);
  for (int l = 0; l < g.n_levels; ++l) {
    const int nb = (br_off[l + 1] - br_off[l]) * P, nn = (node_off[l + 1] - node_off[l]) * P;
    for (int k = grp; k < nb; k += G) {
      if (k != grp) load_branch(l, k);
      const Place at = place_of(g, k);
      const int* br = branches + 2 * (br_off[l] + at.node);
      T* const mine = sS + (size_t)k * KQ;
      const T* vec = mine;
      if (br[1] >= 0) {
        vec = sL + ((size_t)br[1] * P + at.p) * KQ;
      } else {
        mine[i] = out_L;
        wave_lds_order();
      }
      if (Matrix::kStaged) mat.stage(buf, i);
      T r = mat.row_dot(buf, vec, i);
      wave_lds_order();
      r = i < K ? r : T(0);
      mine[i] = r;
      if (g.keep && row_ok) g.S[((size_t)br[0] * P + at.p) * Kp + i] = r;
    }
    const T ta = tip_a, tb = tip_b;
    const int ea = out_sa, eb = out_sb;
    if (l + 1 < g.n_levels) {
      if (grp < (br_off[l + 2] - br_off[l + 1]) * P) load_branch(l + 1, grp);
    }
    lds_barrier();
    for (int k = grp; k < nn; k += G) {
      const Place at = place_of(g, k);
      const int* nd = nodes + 4 * (node_off[l] + at.node);
      const int p = at.p;
      T xa = ta, xb = tb;
      int sa = ea, sb = eb;
      if (k != grp) {
        load_node(l, k);
        xa = tip_a;
        xb = tip_b;
        sa = out_sa;
        sb = out_sb;
      }
      if (nd[1] >= 0) {
        xa = sS[((size_t)nd[1] * P + p) * KQ + i];
        const int slot = branches[2 * (br_off[l] + nd[1]) + 1];
        if (slot >= 0) sa = sE[slot * P + p];
      }
      if (nd[2] >= 0) {
        xb = sS[((size_t)nd[2] * P + p) * KQ + i];
        const int slot = branches[2 * (br_off[l] + nd[2]) + 1];
        if (slot >= 0) sb = sE[slot * P + p];
      }
      const T x = i < K ? xa * xb : T(0);
      const int e = scale_exponent(item_max<KQ>(x));
      const T y = i < K ? scale_by_pow2(x, e) : T(0);
      sL[((size_t)nd[3] * P + p) * KQ + i] = y;
      if (row_ok) g.part[((size_t)(nd[0] - N) * P + p) * Kp + i] = y;
      if (i == 0) {
        sE[nd[3] * P + p] = e + sa + sb;
        g.scales[(size_t)(nd[0] - N) * P + p] = e + sa + sb;
      }
    }
    if (l + 1 < g.n_levels && grp < (node_off[l + 2] - node_off[l + 1]) * P) load_node(l + 1, grp);
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// Pre-order, one level: an item is (internal child, pattern).  children: {child, parent, sibling,
// LDS place of q_parent, LDS place of q_child}, the places used by the runs only.
template <typename T, int KQ>
__global__ __launch_bounds__(256) void few_pre_level_kernel(const FewArgs<T> g, const int32_t* __restrict__ children,
                                                            int n) {
  __shared__ T sT[256];
  const int i = threadIdx.x % KQ, item = blockIdx.x * (256 / KQ) + threadIdx.x / KQ;
  const bool ok = item < n * g.P;
  const Place at = place_of(g, ok ? item : 0);
  const int32_t* it = children + 5 * at.node;
  const int c_node = it[0], u = it[1], sib = it[2], p = at.p;
  const int N = g.N, P = g.P, K = g.K, Kp = g.Kp, C = g.C;
  const size_t KK = (size_t)Kp * Kp;
  const int own = threadIdx.x - i;
  T q[kMaxCategories];
  for (int c = 0; c < C; ++c) {
    T t = 0;
    if (i < K) {
      const T qu = u == g.root ? T(g.pi[i]) : g.pre[(((size_t)(u - N) * C + c) * P + p) * Kp + i];
      t = qu * g.S[(((size_t)sib * C + c) * P + p) * Kp + i];
    }
    sT[threadIdx.x] = t;
    wave_lds_order();
    q[c] = i < K ? dot_strided(g.Pm + ((size_t)c_node * C + c) * KK + i, (size_t)Kp, sT + own, K) : T(0);
    wave_lds_order();
  }
  T m = 0;
  for (int c = 0; c < C; ++c) m = q[c] > m ? q[c] : m;
  const int e = scale_exponent(item_max<KQ>(m));
  if (ok && i < Kp)
    for (int c = 0; c < C; ++c)
      g.pre[(((size_t)(c_node - N) * C + c) * P + p) * Kp + i] = i < K ? scale_by_pow2(q[c], e) : T(0);
}

// Pre-order of consecutive narrow levels, highest first, by one block (one category).  data: item
// offsets [n_levels + 1], items as above.  A lane holds column i of the child's matrix, loaded a level
// ahead; t = q_parent o S_sibling passes through LDS within the item's wavefront, so a level has one
// barrier.
template <typename T, int KQ, int COLS, int NT>
__global__ __launch_bounds__(NT) void few_pre_run_kernel(const FewArgs<T> g) {
  constexpr int G = NT / KQ;
  extern __shared__ __align__(16) unsigned char few_lds[];
  constexpr int Kp = COLS;
  constexpr size_t KK = (size_t)Kp * Kp;
  const int N = g.N, P = g.P, K = g.K;
  T* const sQ = reinterpret_cast<T*>(few_lds);       // [n_nodes][P][KQ]
  T* const sT = sQ + (size_t)g.n_nodes * P * KQ;     // [G][KQ]
  typedef ItemMatrix<T, KQ, COLS> Matrix;
  T* const sM = sT + NT;                             // [G] matrices (33 states or more)
  int* const data = reinterpret_cast<int*>(reinterpret_cast<char*>(sM) + G * Matrix::kLds);
  for (int t = threadIdx.x; t < g.n_ints; t += NT) data[t] = g.data[t];
  __syncthreads();
  const int* const off = data;
  const int* const items = data + g.n_levels + 1;
  const int grp = threadIdx.x / KQ, i = threadIdx.x % KQ;
  Matrix mat;
  T* const buf = sM + grp * (Matrix::kLds / sizeof(T));
  T sib = 0, out_q = 0;
  auto load = [&](int l, int k) {
    const Place at = place_of(g, k);
    const int* it = items + 5 * (off[l] + at.node);
    mat.load_columns(g.Pm + (size_t)it[0] * KK, i);
    const int p = at.p;
    sib = i < K ? g.S[((size_t)it[2] * P + p) * Kp + i] : T(0);
    out_q = 0;
    if (it[3] < 0 && i < K) out_q = it[1] == g.root ? T(g.pi[i]) : g.pre[((size_t)(it[1] - N) * P + p) * Kp + i];
  };
  if (grp < (off[1] - off[0]) * P) load(0, grp);
  for (int l = 0; l < g.n_levels; ++l) {
    const int n = (off[l + 1] - off[l]) * P;
    for (int k = grp; k < n; k += G) {
      if (k != grp) load(l, k);
      const Place at = place_of(g, k);
      const int* it = items + 5 * (off[l] + at.node);
      const int p = at.p;
      const T qu = it[3] >= 0 ? sQ[((size_t)it[3] * P + p) * KQ + i] : out_q;
      T* const t = sT + grp * KQ;
      t[i] = i < K ? qu * sib : T(0);
      if (Matrix::kStaged)
        mat.stage(buf, i);
      else
        wave_lds_order();
      T r = mat.column_dot(buf, t, i);
      wave_lds_order();
      r = i < K ? r : T(0);
      const int e = scale_exponent(item_max<KQ>(r));
      const T y = i < K ? scale_by_pow2(r, e) : T(0);
      if (it[4] >= 0) sQ[((size_t)it[4] * P + p) * KQ + i] = y;
      if (i < Kp) g.pre[((size_t)(it[0] - N) * P + p) * Kp + i] = y;
    }
    if (l + 1 < g.n_levels && grp < (off[l + 2] - off[l + 1]) * P) load(l + 1, grp);
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// dlogL/dP of one branch per block (grad_G_generic_kernel's sums, with the child vectors read
// instead of formed) and dlogL/dl = <G, dP/dl>.  G itself is stored only where dlogL/dQ or the time
// gradient will read it.
template <typename T, int KQ, int GPT>
__global__ __launch_bounds__(256) void few_grad_kernel(const FewArgs<T> g, const int32_t* __restrict__ parent,
                                                       const double* __restrict__ cat,
                                                       const double* __restrict__ weights, const T* __restrict__ dP,
                                                       double* __restrict__ G, double* __restrict__ dbranch) {
  constexpr int TP = 256 / KQ;
  __shared__ T sAc[kMaxCategories][256];
  __shared__ T sBc[kMaxCategories][256];
  __shared__ double sRed[256];
  const int N = g.N, P = g.P, K = g.K, Kp = g.Kp, C = g.C;
  const size_t KK = (size_t)Kp * Kp;
  const int nG = C * Kp * Kp;
  const int v = blockIdx.x;
  if (v == g.root) {  // uniform
    if (G)
      for (int e = threadIdx.x; e < nG; e += 256) G[(size_t)v * nG + e] = 0.0;
    if (threadIdx.x == 0) dbranch[v] = 0.0;
    return;
  }
  const int u = parent[v], w = g.left[u] == v ? g.right[u] : g.left[u];
  const int pl = threadIdx.x / KQ, i = threadIdx.x % KQ;
  double gr[GPT];  // FP64 over the tiles of TP patterns, as the partial-sum slots of the general form are added up
#pragma unroll
  for (int k = 0; k < GPT; ++k) gr[k] = 0;
  for (int p0 = 0; p0 < P; p0 += TP) {
    const int p = p0 + pl;
    const bool pok = p < P;
    T acc = 0;
    T tv[kMaxCategories];
    for (int c = 0; c < C; ++c) {
      T lv = 0, tvi = 0;
      if (pok && i < K) {
        const T q = u == g.root ? T(g.pi[i]) : g.pre[(((size_t)(u - N) * C + c) * P + p) * Kp + i];
        const T sv = g.S[(((size_t)v * C + c) * P + p) * Kp + i], sw = g.S[(((size_t)w * C + c) * P + p) * Kp + i];
        tvi = q * sw;
        acc += T(cat[kMaxCategories + c]) * tvi * sv;
        if (v >= N)
          lv = g.part[(((size_t)(v - N) * C + c) * P + p) * Kp + i];
        else
          lv = ((tip_set(g.tips[(size_t)v * P + p], K, g.amb) >> i) & 1) ? T(1) : T(0);
      }
      tv[c] = tvi;
      sBc[c][threadIdx.x] = lv;
    }
    const T Lt = group_sum<KQ>(acc);
    const T coef = (pok && Lt > T(0)) ? T(weights[p]) / Lt : T(0);
    for (int c = 0; c < C; ++c) sAc[c][threadIdx.x] = coef * T(cat[kMaxCategories + c]) * tv[c];
    __syncthreads();
    const int np = min(TP, P - p0);
#pragma unroll
    for (int k = 0; k < GPT; ++k) {
      const int e = threadIdx.x + k * 256;
      if (e < nG) {
        const int c = e / (int)KK, r = e % (int)KK;
        const int ii = r / Kp, jj = r % Kp;
        if (ii < K && jj < K) {
          T s = 0;
          for (int q = 0; q < np; ++q) s += sAc[c][q * KQ + ii] * sBc[c][q * KQ + jj];
          gr[k] += (double)s;
        }
      }
    }
    __syncthreads();
  }
  double d = 0.0;
#pragma unroll
  for (int k = 0; k < GPT; ++k) {
    const int e = threadIdx.x + k * 256;
    if (e < nG) {
      if (G) G[(size_t)v * nG + e] = gr[k];
      d += gr[k] * (double)dP[(size_t)v * nG + e];
    }
  }
  d = block_sum<256>(d, sRed);
  if (threadIdx.x == 0) dbranch[v] = d;
}

bool few_gradient(const EpochConfig& c) { return (c.flags & (EPOCH_GRAD_BRANCH | EPOCH_GRAD_Q | EPOCH_GRAD_TIME)) != 0; }

int few_lanes(const EpochInstance* in) {
  int q = 4;
  while (q < in->Kp) q <<= 1;
  return q;
}

template <typename T>
FewArgs<T> few_args(EpochInstance* in) {
  FewArgs<T> g{};
  g.left = in->d_left;
  g.right = in->d_right;
  g.Pm = static_cast<const T*>(in->Pm.ptr);
  g.tips = static_cast<const uint8_t*>(in->tips.ptr);
  g.amb = static_cast<const uint64_t*>(in->amb.ptr);
  g.part = static_cast<T*>(in->partials.ptr);
  g.pre = static_cast<T*>(in->pre.ptr);
  g.scales = static_cast<int32_t*>(in->scales.ptr);
  g.S = static_cast<T*>(in->few_S.ptr);
  g.keep = few_gradient(in->cfg);
  g.pi = static_cast<const double*>(in->pi.ptr);
  g.root = in->plan.root;
  g.N = in->N;
  g.P = in->P;
  g.K = in->K;
  g.Kp = in->Kp;
  g.C = in->C;
  g.inv_P = in->P == 1 ? 0u : (unsigned)(((1ull << 32) + in->P - 1) / in->P);
  return g;
}

int few_level_items(int items, int kq) { return std::min(256 / kq, std::max(1, (items + kFewBlocks - 1) / kFewBlocks)); }

// LDS of a run (kernel layouts above).
size_t few_matrix_lds(const EpochInstance* in) {  // every item's matrix buffer
  if (in->Kp <= 32) return 0;
  const size_t items = few_threads(in->fp64, in->Kp) / 64;
  return items * in->Kp * (in->Kp * in->real_size + 16);
}
size_t post_run_lds(const EpochInstance* in, const FewStep& s) {
  const size_t row = (size_t)in->P * few_lanes(in) * in->real_size;
  return (s.n_nodes + s.max_branches) * row + few_matrix_lds(in) + ((size_t)s.n_nodes * in->P + s.n_ints) * sizeof(int);
}
size_t pre_run_lds(const EpochInstance* in, const FewStep& s) {
  const size_t kq = few_lanes(in), threads = few_threads(in->fp64, in->Kp);
  return ((size_t)s.n_nodes * in->P * kq + threads) * in->real_size + few_matrix_lds(in) + s.n_ints * sizeof(int);
}

template <typename T, int KQ>
int few_post_launch(EpochInstance* in, const FewPlan& plan, const int32_t* d_data) {
  FewArgs<T> g = few_args<T>(in);
  for (const FewStep& s : plan.post) {
    if (!s.run) {
      const int items = s.n_nodes * in->P, per = few_level_items(items, KQ);
      hipLaunchKernelGGL((few_post_level_kernel<T, KQ>), dim3((items + per - 1) / per), dim3((per * KQ + 63) / 64 * 64),
                         0, in->stream, g, d_data + s.at, s.n_nodes, per);
      continue;
    }
    g.data = d_data + s.at;
    g.n_ints = s.n_ints;
    g.n_levels = s.n_levels;
    g.n_nodes = s.n_nodes;
    g.n_tips = s.n_tips;
    g.max_branches = s.max_branches;
    const size_t lds = post_run_lds(in, s);
    auto launch = [&](auto cols) {
      constexpr int COLS = decltype(cols)::value, NT = few_threads(sizeof(T) == 8, COLS);
      hipLaunchKernelGGL((few_post_run_kernel<T, KQ, COLS, NT>), dim3(1), dim3(NT), lds, in->stream, g);
    };
    if (KQ == 64 && in->Kp == 48)
      launch(std::integral_constant<int, KQ == 64 ? 48 : KQ>{});
    else
      launch(std::integral_constant<int, KQ>{});
  }
  return hip_check(hipGetLastError(), "few-pattern post-order launch");
}

template <typename T, int KQ>
int few_pre_launch(EpochInstance* in, const FewPlan& plan, const int32_t* d_data) {
  FewArgs<T> g = few_args<T>(in);
  for (const FewStep& s : plan.pre) {
    if (!s.run) {
      constexpr int per = 256 / KQ;
      hipLaunchKernelGGL((few_pre_level_kernel<T, KQ>), dim3((s.n_nodes * in->P + per - 1) / per), dim3(256), 0,
                         in->stream, g, d_data + s.at, s.n_nodes);
      continue;
    }
    g.data = d_data + s.at;
    g.n_ints = s.n_ints;
    g.n_levels = s.n_levels;
    g.n_nodes = s.n_nodes;
    const size_t lds = pre_run_lds(in, s);
    auto launch = [&](auto cols) {
      constexpr int COLS = decltype(cols)::value, NT = few_threads(sizeof(T) == 8, COLS);
      hipLaunchKernelGGL((few_pre_run_kernel<T, KQ, COLS, NT>), dim3(1), dim3(NT), lds, in->stream, g);
    };
    if (KQ == 64 && in->Kp == 48)
      launch(std::integral_constant<int, KQ == 64 ? 48 : KQ>{});
    else
      launch(std::integral_constant<int, KQ>{});
  }
  return hip_check(hipGetLastError(), "few-pattern pre-order launch");
}

template <typename T, int KQ, int GPT>
int few_grad_launch(EpochInstance* in) {
  const FewArgs<T> g = few_args<T>(in);
  const bool keep = (in->cfg.flags & (EPOCH_GRAD_Q | EPOCH_GRAD_TIME)) != 0;
  hipLaunchKernelGGL((few_grad_kernel<T, KQ, GPT>), dim3(in->n_nodes), dim3(256), 0, in->stream, g, in->d_parent,
                     static_cast<const double*>(in->cat.ptr), static_cast<const double*>(in->weights.ptr),
                     static_cast<const T*>(in->dPm.ptr), keep ? static_cast<double*>(in->G.ptr) : nullptr,
                     static_cast<double*>(in->dbranch.ptr));
  return hip_check(hipGetLastError(), "few-pattern gradient launch");
}

}  // namespace

// The launches of a pass over the listed nodes (level l's are nodes[level_off[l] ..
// level_off[l + 1])), with their item lists; with_pre: the pre-order pass too (the whole tree).
void few_plan(const EpochInstance* in, const int32_t* nodes, const int32_t* level_off, bool with_pre, FewPlan& out) {
  out = FewPlan{};
  const auto& pl = in->plan;
  const int N = in->N, P = in->P;
  const int kq = few_lanes(in), threads = few_threads(in->fp64, in->Kp), groups = threads / kq;
  const size_t row = (size_t)P * kq * in->real_size;
  auto width = [&](int l) { return level_off[l + 1] - level_off[l]; };
  const size_t pair = 2 * (size_t)in->Kp * in->Kp * in->real_size;  // an item's matrices
  auto narrow = [&](int l) {
    const int items = width(l) * P;
    return in->C == 1 && items <= kFewWide * groups && items * pair <= few_run_bytes(kq);
  };
  std::vector<int32_t> slot(in->n_nodes, -1);
  // post-order, lowest level first
  for (int l = 1; l <= pl.n_levels;) {
    if (width(l) == 0) {
      ++l;
      continue;
    }
    FewStep s;
    s.at = out.data.size();
    if (!narrow(l)) {
      s.n_nodes = width(l);
      out.data.insert(out.data.end(), nodes + level_off[l], nodes + level_off[l + 1]);
      out.post.push_back(s);
      ++l;
      continue;
    }
    s.run = true;
    std::vector<int32_t> noff(1, 0), boff(1, 0), nd, br, tp;
    while (l <= pl.n_levels && narrow(l)) {
      // would this level still fit?  (its branches: at most two per node)
      const size_t n_after = s.n_nodes + width(l);
      const size_t ints = 2 * (noff.size() + 2) + 4 * n_after + br.size() + 4 * (size_t)width(l) + tp.size() + 2 * (size_t)width(l);
      const size_t lds = (n_after + std::max(s.max_branches, 2 * width(l))) * row + (n_after * P + ints) * sizeof(int);
      if (lds > kFewLds && s.n_nodes > 0) break;
      int nb = 0;
      for (int k = level_off[l]; k < level_off[l + 1]; ++k) {
        const int u = nodes[k];
        int32_t ref[2];
        for (int side = 0; side < 2; ++side) {
          const int v = side ? pl.right[u] : pl.left[u];
          if (v < N) {
            ref[side] = ~v;
            tp.push_back(v);
          } else {
            ref[side] = nb++;
            br.push_back(v);
            br.push_back(slot[v]);
          }
        }
        nd.insert(nd.end(), {u, ref[0], ref[1], s.n_nodes});
        slot[u] = s.n_nodes++;
      }
      s.max_branches = std::max(s.max_branches, nb);
      noff.push_back(s.n_nodes);
      boff.push_back((int32_t)br.size() / 2);
      ++s.n_levels;
      ++l;
    }
    s.n_tips = (int)tp.size();
    for (const auto* part : {&noff, &boff, &nd, &br, &tp}) out.data.insert(out.data.end(), part->begin(), part->end());
    s.n_ints = (int)(out.data.size() - s.at);
    for (size_t k = 0; k < nd.size(); k += 4) slot[nd[k]] = -1;  // a later launch reads these from memory
    out.post.push_back(s);
  }
  if (!with_pre) return;
  // pre-order, highest level first: the internal children of each level's nodes
  auto child_items = [&](int l, std::vector<int32_t>& items) {
    for (int k = level_off[l]; k < level_off[l + 1]; ++k) {
      const int u = nodes[k], a = pl.left[u], b = pl.right[u];
      if (a >= N) items.insert(items.end(), {a, u, b, -1, -1});
      if (b >= N) items.insert(items.end(), {b, u, a, -1, -1});
    }
  };
  for (int l = pl.n_levels; l >= 1;) {
    std::vector<int32_t> items;
    child_items(l, items);
    if (items.empty()) {
      --l;
      continue;
    }
    FewStep s;
    s.at = out.data.size();
    if (!narrow(l)) {
      s.n_nodes = (int)items.size() / 5;
      out.data.insert(out.data.end(), items.begin(), items.end());
      out.pre.push_back(s);
      --l;
      continue;
    }
    s.run = true;
    std::vector<int32_t> off(1, 0), all, used;
    int next = 0;
    while (l >= 1 && narrow(l)) {
      items.clear();
      child_items(l, items);
      const size_t n_after = next + items.size() / 5;
      const size_t lds = n_after * row + threads * in->real_size + (off.size() + 1 + all.size() + items.size()) * sizeof(int);
      if (lds > kFewLds && s.n_levels > 0) break;
      for (size_t k = 0; k < items.size(); k += 5) {
        items[k + 3] = slot[items[k + 1]];
        items[k + 4] = slot[items[k]] = next++;
        used.push_back(items[k]);
      }
      all.insert(all.end(), items.begin(), items.end());
      off.push_back((int32_t)all.size() / 5);
      ++s.n_levels;
      --l;
    }
    s.n_nodes = next;
    out.data.insert(out.data.end(), off.begin(), off.end());
    out.data.insert(out.data.end(), all.begin(), all.end());
    s.n_ints = (int)(out.data.size() - s.at);
    for (int v : used) slot[v] = -1;
    out.pre.push_back(s);
  }
}

// Few patterns on the generic path, all evaluated at once: bytes of the child vectors, 0 where the
// per-level kernels run.  Without a gradient only the tips' are kept, and several categories, which no
// run serves, leave nothing to gain: 16 states, 1,000 taxa, one column, FP64, four categories 247 us
// by the per-level kernels and 322 by these.
size_t few_vector_bytes(const EpochConfig& c, int Kp) {
  const size_t row = (size_t)c.n_categories * c.n_patterns * Kp * (c.precision == EPOCH_FP64 ? 8 : 4);
  const size_t n_nodes = 2 * (size_t)c.n_tips - 1;
  if (!few_gradient(c) && c.n_categories > 1) return 0;
  if (c.hbm_budget_bytes != 0 || c.n_patterns > kFewMaxPatterns || n_nodes * row > kFewVectorBytes) return 0;
  return (few_gradient(c) ? n_nodes : c.n_tips) * row;
}

int few_prepare(EpochInstance* in) {
  in->few = in->few_S.ptr != nullptr;
  if (!in->few) return EPOCH_OK;
  few_plan(in, in->plan.level_nodes.data(), in->plan.level_offset.data(), true, in->few_plan);
  const int rc = ensure(in->few_dev, std::max<size_t>(1, in->few_plan.data.size()) * sizeof(int32_t));
  if (rc || in->few_plan.data.empty()) return rc;
  return stage_upload(in, in->few_dev.ptr, in->few_plan.data.data(), in->few_plan.data.size() * sizeof(int32_t));
}

#define EPOCH_FEW(T, FN, ...)                            \
  switch (few_lanes(in)) {                               \
    case 4: return FN<T, 4 __VA_ARGS__;                  \
    case 8: return FN<T, 8 __VA_ARGS__;                  \
    case 16: return FN<T, 16 __VA_ARGS__;                \
    case 32: return FN<T, 32 __VA_ARGS__;                \
    default: return FN<T, 64 __VA_ARGS__;                \
  }

int launch_few_post(EpochInstance* in, const FewPlan& plan, const int32_t* d_data) {
  if (in->fp64) EPOCH_FEW(double, few_post_launch, >(in, plan, d_data))
  EPOCH_FEW(float, few_post_launch, >(in, plan, d_data))
}

int launch_few_pre(EpochInstance* in) {
  const int32_t* d_data = static_cast<const int32_t*>(in->few_dev.ptr);
  if (in->fp64) EPOCH_FEW(double, few_pre_launch, >(in, in->few_plan, d_data))
  EPOCH_FEW(float, few_pre_launch, >(in, in->few_plan, d_data))
}

namespace {
template <typename T>
int few_grad_dispatch(EpochInstance* in) {
  const int gpt = (in->C * in->Kp * in->Kp + 255) / 256;
  if (gpt > 64) return set_error(EPOCH_ERR_ARG, "generic gradient supports C*Kp*Kp <= 16384");
  switch (few_lanes(in)) {  // lanes per pattern fix Kp, so only these pairs occur
    case 4: return few_grad_launch<T, 4, 1>(in);
    case 8: return few_grad_launch<T, 8, 4>(in);
    case 16: return few_grad_launch<T, 16, 16>(in);
    case 32: return few_grad_launch<T, 32, 32>(in);
    default: return gpt <= 16 ? few_grad_launch<T, 64, 16>(in) : few_grad_launch<T, 64, 64>(in);
  }
}
}  // namespace

int launch_few_grad(EpochInstance* in) {
  return in->fp64 ? few_grad_dispatch<double>(in) : few_grad_dispatch<float>(in);
}

}  // namespace epochlik
