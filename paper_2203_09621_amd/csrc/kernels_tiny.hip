// One workgroup runs the whole recursion of a small problem (split forms).
//
// A problem of N <= 96 with up to three responses (N <= 128 with one) keeps
// the 16-bit splits of S and of every S1_j in the LDS of one CU and their FP32
// masters in registers, so a layer needs no launch, no global memory and no
// other workgroup.  What bounds it is the chain of a layer: the MFMAs of a
// fragment depend on each other (24 at N = 64, about 2000 cycles), then the
// update and the next splits (about as long), with three barriers.  The two
// decisions run on one wave beside the products: Tr X needs X alone, so
// Algorithm 2's follows the first product while the second one runs, and
// Algorithm 3's runs during the next layer's first product, whose results are
// dropped if it stopped the recursion.
//
// Every X_ii, X and X1_j is formed with the operand chunks, k order and MFMA
// sequence of the general path's kernels, N_X is summed in their order, and
// the update, splits and decisions are theirs, so P0 and P1_j are bitwise the
// same.  (The FP64 sums of the stopping norms run in another order.)
#include <string.h>

#include "layer_common.h"
#include "split_mfma.h"

namespace dmpt {

namespace {

// LayerState of a problem in the deciding wave: the fields the decisions use,
// with the last four entries of the histories (they look back two layers).
struct TinyState {
  static constexpr int kHist = 3;
  double nocc, n_s, fro0;
  int32_t k, max_layers, n, done, error, converged;
  int32_t d0, d0_layer, x_computed, upd_s0, d0_now, sigma_cur, order2_slot;
  int32_t d1[kMaxKB], d1_layer[kMaxKB], s1_exp_split[kMaxKB], s1_exp_next[kMaxKB];
  double s1_max[kMaxKB];
  int32_t sigma[kHist + 1];
  double iderr[kHist + 1];
  double fro1[kMaxKB][kHist + 1];
  int32_t s1_exp_hist[kMaxKB][kHist + 1];
};

// What the other waves read of it: after Algorithm 3's decision of a layer, and
// after the next layer's Algorithm 2.
struct TinyAfter1 {
  int32_t done;
  int32_t d1[kMaxKB], exp_split[kMaxKB], exp_next[kMaxKB];
  int32_t par[kMaxKB];       // buffer of P1_j: layer d1_layer - 1, or the last layer
};
struct TinyAfter0 {
  int32_t done, sigma, upd0, d0;
};

// Transpose of four packed values per lane within each quad of lanes: lane i
// receives p[i] of lane j as p[j].
__device__ __forceinline__ uint32_t quad_swap(uint32_t v, int d) {
  // quad_perm by xor d
  return (uint32_t)(d == 1 ? __builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true)
                    : d == 2 ? __builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true)
                             : __builtin_amdgcn_update_dpp(0, (int)v, 0x1b, 0xf, 0xf, true));
}
// A workgroup-uniform value read from LDS, in a scalar register.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ void quad_transpose(uint32_t (&p)[4], int lane) {
  auto by_lane = [&]() {     // p[d] <- p[(lane & 3) ^ d]
    const bool b0 = lane & 1, b1 = lane & 2;
    const uint32_t a0 = b0 ? p[1] : p[0], a1 = b0 ? p[0] : p[1];
    const uint32_t a2 = b0 ? p[3] : p[2], a3 = b0 ? p[2] : p[3];
    p[0] = b1 ? a2 : a0;
    p[1] = b1 ? a3 : a1;
    p[2] = b1 ? a0 : a2;
    p[3] = b1 ? a1 : a3;
  };
  by_lane();
#pragma unroll
  for (int d = 1; d < 4; ++d) p[d] = quad_swap(p[d], d);
  by_lane();
}

constexpr int tiny_pitch(int nf) { return 32 * nf + 8; }   // 16-bit elements of an LDS row: an
                                                           // odd count of 16-byte chunks, so that
                                                           // rows fall on different banks

// Waves of a workgroup: two per SIMD cover each other's LDS latency and halve
// the update's work per wave (one 32-row block has at most four fragments).
constexpr int tiny_waves(int nf) { return nf == 1 ? 4 : 8; }
constexpr int kGershWaves = 4;   // waves that walk the rows of H0, as k_b_gersh does

}  // namespace

// NF: 32-row blocks of the problem (N <= 32 NF), K: responses.
template <typename T16, int NF, int K>
__global__ void __launch_bounds__(tiny_waves(NF) * kWave)
    __attribute__((amdgpu_waves_per_eu(NF == 1 ? 3 : 2))) k_tiny(const TinyArgs a) {
  using S = Split16<T16>;
  using V = typename S::V;
  constexpr int NR = 32 * NF, PITCH = tiny_pitch(NF);
  constexpr int MAT = NR * PITCH;              // one 16-bit matrix
  constexpr int NFR = NF * (NF + 1) / 2;       // 32 x 32 fragments of an upper triangle
  constexpr int NI = (1 + K) * NFR;            // fragments of all outputs, responses first
  constexpr int W = tiny_waves(NF), NT = W * kWave;
  constexpr int M = (NI + W - 1) / W;          // fragments per wave
  extern __shared__ uint16_t ops[];            // [matrix][hi, lo][row][PITCH], matrix 0: S
  __shared__ TinyState st;                     // written by lane 0 of the deciding wave
  __shared__ TinyAfter1 c1;
  __shared__ TinyAfter0 c0;
  __shared__ double tr[4], red_f[M * W], row_lo[kGershWaves], row_hi[kGershWaves],
      row_tr[kGershWaves][NF], red_h[W];
  __shared__ float red_m[M * W];                  // per item: norm partial, max |S1_j|

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const TinyProblem pr = a.probs ? a.probs[blockIdx.x] : a.one;
  const int n = pr.n;
  LayerState* g = pr.state;
  const double* H0 = a.h0tab ? a.h0tab[pr.h0] : nullptr;
  auto h1 = [&](int j) { return a.h1tab ? a.h1tab[pr.h1 + j] : a.h1[j]; };

  // ---- normalisation: the bounds of H0 (batch; in the order of k_b_gersh and
  // k_b_setup) or those dmpt_set_hamiltonian left in the state
  double eps1, epsN, n_s0;
  if (H0) {
    if (wave < kGershWaves) {
      double lo = INFINITY, hi = -INFINITY;
#pragma unroll 1
      for (int b = 0; b < NF; ++b) {
        double t = 0.0;
        for (int i = 32 * b + wave; i < min(32 * b + 32, n); i += kGershWaves) {
          const double* row = H0 + (int64_t)i * n;
          double r = 0.0;
          for (int j = lane; j < n; j += kWave) r += (j == i) ? 0.0 : fabs(row[j]);
          r = wave_sum(r);
          const double d = row[i];
          lo = fmin(lo, d - r);
          hi = fmax(hi, d + r);
          t += d;
        }
        if (lane == 0) row_tr[wave][b] = t;
      }
      if (lane == 0) {
        row_lo[wave] = lo;
        row_hi[wave] = hi;
      }
    }
    lds_barrier();
    double p[4] = {0.0, 0.0, 0.0, 0.0};
    eps1 = row_lo[0];
    epsN = row_hi[0];
#pragma unroll
    for (int w = 1; w < kGershWaves; ++w) {
      eps1 = fmin(eps1, row_lo[w]);
      epsN = fmax(epsN, row_hi[w]);
    }
#pragma unroll
    for (int b = 0; b < NF; ++b)
#pragma unroll
      for (int w = 0; w < kGershWaves; ++w) p[b] += row_tr[w][b];
    n_s0 = ((double)n * epsN - ((p[0] + p[2]) + (p[1] + p[3]))) / (epsN - eps1);
  } else {
    eps1 = g->eps1;
    epsN = g->epsN;
    n_s0 = g->n_s0;
  }
  const double w = epsN - eps1;

  // max |H1_j| and the split scale of S1_0
  const bool decider = wave == W - 1 && lane == 0;
  int error = w > 0.0 && isfinite(w) ? 0 : DMPT_ENONFINITE;
#pragma unroll 1
  for (int j = 0; j < K; ++j) {
    const double* H = h1(j);
    double m = 0.0;
#pragma unroll 2
    for (int q = tid; q < n * n; q += NT) {
      const double v = fabs(H[q]);
      m = (v > m || v != v) ? v : m;
    }
    m = wave_max(m);
    lds_barrier();                             // the previous response's maxima are read
    if (lane == 0) red_h[wave] = m;
    lds_barrier();
    m = red_h[0];
    for (int v = 1; v < W; ++v) m = fmax(m, red_h[v]);
    m /= w;
    if (!isfinite(m)) error = DMPT_ENONFINITE;
    if (decider) {
      const int e = split_exponent(m);
      st.s1_exp_split[j] = st.s1_exp_next[j] = e;
      st.s1_max[j] = m;
      st.d1[j] = st.d1_layer[j] = 0;
      for (int i = 0; i < 4; ++i) {
        st.fro1[j][i] = 0.0;
        st.s1_exp_hist[j][i] = 0;
      }
      g->s1_exp_hist[j][0] = e;
      c1.exp_split[j] = c1.exp_next[j] = e;
      c1.d1[j] = 0;
      c1.par[j] = 0;
    }
  }
  if (decider) {
    st.nocc = pr.nocc;
    st.n_s = n_s0;
    st.fro0 = 0.0;
    st.k = K;
    st.max_layers = a.max_layers;
    st.n = st.converged = 0;
    st.error = error;
    // (a single problem runs its first layer before the error stops it, as layer by layer)
    c1.done = st.done = H0 && error != 0;
    st.d0 = st.d0_layer = st.x_computed = st.upd_s0 = st.d0_now = st.sigma_cur = 0;
    st.order2_slot = -1;
    for (int i = 0; i < 4; ++i) {
      st.sigma[i] = 0;
      st.iderr[i] = 0.0;
      tr[i] = 0.0;
    }
  }
  lds_barrier();

  // S0 = (eps_N I - H0)/(eps_N - eps_1), S1_0 = -H1/(eps_N - eps_1) in FP32
  auto value = [&](int mat, const double* H, int r, int c) -> float {
    if (r >= n || c >= n) return 0.0f;
    if (!H) return pr.s_init[(int64_t)r * pr.ld + c];
    const double h = H[(int64_t)r * n + c];
    return (float)((mat > 0 ? -h : (r == c ? epsN : 0.0) - h) / w);
  };
  auto at = [&](int mat, int lo, int r, int c) { return (2 * mat + lo) * MAT + r * PITCH + c; };
  // FP32 matrices through the LDS of their splits (row pitch PITCH), so that
  // global memory is read and written row by row
  auto stage = [&](int mat) { return (float*)(ops + (size_t)2 * mat * MAT); };
#pragma unroll 1
  for (int mat = 0; mat <= K; ++mat) {
    const double* H = mat == 0 ? H0 : h1(mat - 1);
    float* T = stage(mat);
#pragma unroll 1
    for (int q = tid; q < NR * NR; q += NT)
      T[q / NR * PITCH + q % NR] = value(mat, H, q / NR, q % NR);
  }
  lds_barrier();

  // this wave's fragments: slot s is item s * W + wave (output, block
  // row, block column); element r of lane l sits in row 8 (r / 4) + 4 (l / 32)
  // + r % 4 and column l % 32
  int out[M], fi[M], fj[M];
  f32x16 master[M], next[M], acc[M];
#pragma unroll
  for (int s = 0; s < M; ++s) {
    const int i = s * W + wave;
    out[s] = i < NI ? (i < K * NFR ? 1 + i / NFR : 0) : -1;
    int f = i % NFR, r = 0;
#pragma unroll
    for (int b = 0; b < NF - 1; ++b)
      if (r == b && f >= NF - b) {
        f -= NF - b;
        r = b + 1;
      }
    fi[s] = r;
    fj[s] = r + f;
    const float* T = stage(out[s] > 0 ? out[s] : 0) +
                     (32 * fi[s] + 4 * (lane >> 5)) * PITCH + 32 * fj[s] + (lane & 31);
#pragma unroll
    for (int q = 0; q < 16; ++q) master[s][q] = T[(8 * (q >> 2) + (q & 3)) * PITCH];
  }
  lds_barrier();
#pragma unroll 1
  for (int mat = 0; mat <= K; ++mat) {
    const double* H = mat == 0 ? H0 : h1(mat - 1);
    const int e = mat == 0 ? 0 : c1.exp_split[mat - 1];
#pragma unroll 1
    for (int q = tid; q < NR * NR; q += NT) {
      const int r = q / NR, c = q % NR;
      split_one<T16>(value(mat, H, r, c), e, S::kShift, ops + at(mat, 0, r, c),
                     ops + at(mat, 1, r, c));
    }
  }
  lds_barrier();

  auto frag = [&](int mat, int lo, int blk, int ks) -> V {
    return *(const V*)(ops + at(mat, lo, 32 * blk + (lane & 31), 16 * ks + 8 * (lane >> 5)));
  };

  // products p of the slots in `on`: X = S S, X1_j = S S1_j + S1_j S
  auto products = [&](int p, const int (&on)[M]) {
#pragma unroll
    for (int ks = 0; ks < 2 * NF; ++ks)
#pragma unroll
      for (int s = 0; s < M; ++s)
        if (on[s] && (p == 0 || out[s] > 0)) {
          const int ma = p == 0 ? 0 : out[s], mb = p == 0 ? out[s] : 0;
          const V ah = frag(ma, 0, fi[s], ks), al = frag(ma, 1, fi[s], ks);
          const V bh = frag(mb, 0, fj[s], ks), bl = frag(mb, 1, fj[s], ks);
          acc[s] = S::mma(S::up(ah), bh, acc[s]);
          acc[s] = S::mma(ah, bl, acc[s]);
          acc[s] = S::mma(al, bh, acc[s]);
        }
  };
  // Algorithm 3 for the layer whose norms lie in red_f and red_m
  auto decide1 = [&]() {
    // lane o combines output o's items (responses first, then X); partials of
    // outputs at rest are stale and unused
    double f = 0.0, m = 0.0;
    if (lane <= K) {
      const int i0 = lane == 0 ? K * NFR : (lane - 1) * NFR;
#pragma unroll
      for (int i = 0; i < NFR; ++i) {
        f += red_f[i0 + i];
        m = fmax(m, (double)red_m[i0 + i]);
      }
    }
    auto from = [&](double v, int l) {
      const uint64_t u = __builtin_bit_cast(uint64_t, v);
      return __builtin_bit_cast(
          double, (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l) << 32);
    };
    double f1[K], m1[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      f1[j] = from(f, 1 + j);
      m1[j] = from(m, 1 + j);
    }
    const double f0sq = from(f, 0);
    if (lane == 0) {
      decide1_apply<K>(&st, f0sq, f1, m1, 1, S::kShift);
      c1.done = st.done;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        c1.d1[j] = st.d1[j];
        c1.exp_split[j] = st.s1_exp_split[j];
        c1.exp_next[j] = st.s1_exp_next[j];
        c1.par[j] = (st.d1[j] && st.d1_layer[j] > 0 ? st.d1_layer[j] - 1 : st.n) & 1;
        g->fro1[j][st.n] = st.fro1[j][st.n & TinyState::kHist];
        g->s1_exp_hist[j][st.n] = st.s1_exp_hist[j][st.n & TinyState::kHist];
      }
    }
  };

  // (flags as integers in scalar registers: every wave branches on them as one)
  int xopen = 1, later = 0;                    // D0 open; a layer's norms wait for decide1
  int on[M];
#pragma unroll
  for (int s = 0; s < M; ++s) on[s] = out[s] >= 0;
  int upd0 = 0;
  int stop = uniform(c1.done);
  while (!stop) {
    if (later && wave == W - 1) decide1();
#pragma unroll
    for (int s = 0; s < M; ++s) {
      if (out[s] == 0) on[s] = xopen;
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[s][q] = 0.0f;
    }
    products(0, on);
    // the diagonal of X into Tr X, per block as the trace kernel sums it
#pragma unroll
    for (int s = 0; s < M; ++s)
      if (on[s] && out[s] == 0 && fi[s] == fj[s]) {
        int c = lane & 31;
        asm volatile("" : "+v"(c));           // (no mask per element kept across layers)
        double v = 0.0;
        if ((lane >> 5) == ((c >> 2) & 1) && 32 * fi[s] + c < n) {
          const int ri = 4 * (c >> 3) + (c & 3);
          float x = 0.0f;
#pragma unroll
          for (int q = 0; q < 16; ++q)
            if (q == ri) x = acc[s][q];
          v = (double)(x * ldexpf(1.0f, -S::kShift));
        }
        v = wave_sum(v);
        if (lane == 0) tr[fi[s]] = v;
      }
    lds_barrier();                             // Tr X and the last layer's Algorithm 3 are known
    // the last layer's update: S_n while S is updated, S1_j,n unless its D1
    // test fired there (the result is then S1_j,n-1)
    if (later) {
#pragma unroll
      for (int s = 0; s < M; ++s) {
        if (out[s] < 0) continue;
        if (out[s] > 0) on[s] &= uniform(c1.d1[out[s] - 1]) ^ 1;
        if (out[s] == 0 ? upd0 : on[s]) master[s] = next[s];
      }
      stop = uniform(c1.done);
      if (stop) break;
    }
    if (decider) {
      // (the block sum's order over at most four partials)
      decide0_apply(&st, xopen ? (tr[0] + tr[2]) + (tr[1] + tr[3]) : 0.0);
      c0.done = st.done;
      c0.sigma = st.sigma_cur;
      c0.upd0 = st.upd_s0;
      c0.d0 = st.d0;
      g->sigma[st.n] = st.sigma_cur;
      if (xopen) g->iderr[st.n] = st.iderr[st.n & TinyState::kHist];
    }
    products(1, on);
    lds_barrier();                             // operands read, Algorithm 2 known
    stop = uniform(c0.done);                   // N_X not finite
    if (stop) break;

    // ---- update: the new splits, ||S - X||^2 or ||S1_j - X1_j||^2, max |S1_j|
    const int sig = uniform(c0.sigma);
    upd0 = uniform(c0.upd0);
    xopen = uniform(c0.d0) ^ 1;
#pragma unroll
    for (int s = 0; s < M; ++s) {
      if (!on[s]) continue;
      const int isx = out[s] == 0, diag = fi[s] == fj[s];
      const int diff = (isx ? upd0 : xopen) ^ 1;
      const int upd = isx ? upd0 : 1;
      const int e = isx ? 0 : uniform(c1.exp_next[out[s] - 1]);
      const int es = isx ? 0 : uniform(c1.exp_split[out[s] - 1]);
      const float scale = ldexpf(1.0f, -(S::kShift + es));
      double f = 0.0;
      float mxs = 0.0f;
      // (opaque: every element's address, weight and mask would otherwise be
      // hoisted out of the layer loop into registers of its own)
      int c = lane & 31, rb = 4 * (lane >> 5);
      asm volatile("" : "+v"(c), "+v"(rb));
      // mirror: row c of the block (fj, fi); direct: row r0 + c % 4 of the block
      // (fi, fj), four columns from c - c % 4 on
      const int mbase = at(out[s], 0, 32 * fj[s] + c, 32 * fi[s] + rb);
      const int dbase = at(out[s], 0, 32 * fi[s] + rb + (c & 3), 32 * fj[s] + (c & ~3));
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int r0 = 8 * q4 + rb;                       // rows r0 .. r0 + 3 of the fragment
        uint32_t own[4], tp[4];                           // hi << 16 | lo
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float x = acc[s][4 * q4 + q] * scale, so = master[s][4 * q4 + q];
          const float sn = sig > 0 ? x : 2.0f * so - x;
          next[s][4 * q4 + q] = sn;
          if (diff) {
            const double wt = !diag ? 2.0 : (r0 + q < c ? 2.0 : (r0 + q == c ? 1.0 : 0.0));
            const double d = (double)so - (double)x;
            f += wt * d * d;
          }
          if (!diag || r0 + q <= c) mxs = fmaxf(mxs, fabsf(sn));
          uint16_t h, l;
          split_one<T16>(sn, e, S::kShift, &h, &l);
          own[q] = tp[q] = ((uint32_t)h << 16) | l;
        }
        if (!upd) continue;
        typedef uint32_t U2 __attribute__((ext_vector_type(2)));
        auto store = [&](uint16_t* at0, const uint32_t (&v)[4]) {
          *(U2*)at0 = U2{__builtin_amdgcn_perm(v[1], v[0], 0x07060302u),
                         __builtin_amdgcn_perm(v[3], v[2], 0x07060302u)};
          *(U2*)(at0 + MAT) = U2{__builtin_amdgcn_perm(v[1], v[0], 0x05040100u),
                                 __builtin_amdgcn_perm(v[3], v[2], 0x05040100u)};
        };
        quad_transpose(tp, lane);
        uint16_t* mh = ops + mbase + 8 * q4;
        uint16_t* dh = ops + dbase + 8 * q4 * PITCH;
        if (!diag) {
          store(mh, own);
          store(dh, tp);
        } else {
          // upper half: the 4 x 4 blocks on the diagonal from both halves of
          // the quad's transpose, those above it and their mirrors
          if (c >= r0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) own[q] = r0 + q <= c ? own[q] : tp[q];
            store(mh, own);
          }
          if ((c & ~3) > r0) store(dh, tp);
        }
      }
      if (diff) f = wave_sum(f);
      mxs = wave_max(mxs);
      if (lane == 0) {
        red_f[s * W + wave] = f;
        red_m[s * W + wave] = mxs;
      }
    }
    later = 1;
    lds_barrier();                             // splits written, partials complete
  }

  // ---- results: FP64 outputs (single problem), or the FP32 masters that the
  // batch's output kernel copies out.  The upper triangles of the masters,
  // mirrored, through the LDS.
  lds_barrier();
#pragma unroll
  for (int s = 0; s < M; ++s) {
    if (out[s] < 0) continue;
    float* T = stage(out[s]);
    const int c = 32 * fj[s] + (lane & 31);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int r = 32 * fi[s] + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
      if (r <= c) {
        T[r * PITCH + c] = master[s][q];
        T[c * PITCH + r] = master[s][q];
      }
    }
  }
  lds_barrier();
#pragma unroll 1
  for (int mat = 0; mat <= K; ++mat) {
    const float* T = stage(mat);
    double* dst = mat == 0 ? a.p0 : a.p1[mat > 0 ? mat - 1 : 0];
    float* dm = pr.s_master;
    if (mat > 0 && a.probs) dm = a.probs[blockIdx.x].s1buf[mat - 1][c1.par[mat - 1]];
#pragma unroll 1
    for (int q = tid; q < NR * NR; q += NT) {
      const int r = q / NR, c = q % NR;
      if (r >= n || c >= n) continue;
      if (a.probs)
        dm[(int64_t)r * pr.ld + c] = T[r * PITCH + c];
      else if (dst)
        dst[(int64_t)r * n + c] = (double)T[r * PITCH + c];
    }
  }
  if (decider) {
    g->n_real = n;
    g->k = K;
    g->max_layers = a.max_layers;
    g->nocc = pr.nocc;
    g->n = st.n;
    g->done = 1;
    g->error = st.error;
    g->converged = st.converged;
    g->d0 = st.d0;
    g->d0_layer = st.d0_layer;
    g->order2_slot = -1;
    g->n_s = st.n_s;
    g->n_s0 = n_s0;
    g->fro0 = st.fro0;
    g->eps1 = eps1;
    g->epsN = epsN;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      g->d1[j] = st.d1[j];
      g->d1_layer[j] = st.d1_layer[j];
    }
  }
}

namespace {

template <typename T16, int NF, int K>
hipError_t launch_cfg(const TinyArgs& a, int count, hipStream_t s) {
  constexpr size_t lds = (size_t)(1 + K) * 2 * (32 * NF) * tiny_pitch(NF) * sizeof(uint16_t);
  static_assert(lds + 2048 <= 160 * 1024 - 256, "LDS of one CU");
  const void* k = (const void*)k_tiny<T16, NF, K>;
  hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_tiny<T16, NF, K>), dim3(count), dim3(tiny_waves(NF) * kWave), lds, s, a);
  return hipGetLastError();
}

template <typename T16>
hipError_t launch_type(int nf, int k, const TinyArgs& a, int count, hipStream_t s) {
  switch (4 * nf + k) {
    case 4 + 1: return launch_cfg<T16, 1, 1>(a, count, s);
    case 4 + 2: return launch_cfg<T16, 1, 2>(a, count, s);
    case 4 + 3: return launch_cfg<T16, 1, 3>(a, count, s);
    case 8 + 1: return launch_cfg<T16, 2, 1>(a, count, s);
    case 8 + 2: return launch_cfg<T16, 2, 2>(a, count, s);
    case 8 + 3: return launch_cfg<T16, 2, 3>(a, count, s);
    case 12 + 1: return launch_cfg<T16, 3, 1>(a, count, s);
    case 12 + 2: return launch_cfg<T16, 3, 2>(a, count, s);
    case 12 + 3: return launch_cfg<T16, 3, 3>(a, count, s);
    case 16 + 1: return launch_cfg<T16, 4, 1>(a, count, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

int tiny_blocks(int64_t n, int k) {
  const int nf = (int)((n + 31) / 32);
  return k <= kMaxKB && (nf <= 3 || (nf == 4 && k == 1)) ? nf : 0;
}

hipError_t launch_tiny(dmpt_precision prec, int nf, int k, const TinyArgs& a, int count,
                       hipStream_t s) {
  if (count <= 0) return hipSuccess;
  if (prec == DMPT_SPLIT_FP16) return launch_type<_Float16>(nf, k, a, count, s);
  if (prec == DMPT_SPLIT_BF16) return launch_type<__bf16>(nf, k, a, count, s);
  return hipErrorInvalidValue;
}

}  // namespace dmpt
