// Pair-matrix rounds: once few enough clusters are active, every cluster
// pair's value is kept in a dense FP64 matrix and the remaining rounds of
// Alg. 1 run on it.
//
//   build    exact values of all active pairs from the points: every point
//            pair once (complete: the largest squared distance; average: the
//            sum of the distances, always added in the same order)
//   pass     one sweep per round: the merged clusters' rows and columns are
//            combined by the Lance-Williams rules of Table 2 (complete: the
//            maximum, average: the sum), the matrix is compacted into the
//            other buffer, and every row's nearest neighbour is found on the
//            way. A sum along a chain of merges takes a rounding per merge, so
//            every entry of average linkage carries what its rounding left
//            over, in a byte (Low)
//   book     one block: reciprocal pairs, rows of the dendrogram, the next
//            round's cluster records
//
// No round waits for the host: the launches of several rounds are queued at
// once and kernels of rounds that are not needed any more exit at once.
//
// Both halves of the matrix are kept, bit for bit equal: a row is then read
// in one contiguous sweep, and a value does not depend on which side asks.
#include <float.h>
#include <math.h>

#include <algorithm>

#include "pc_common.hpp"

namespace pc {

namespace {

constexpr int kWin = 64;          // points per window of the build (rows and columns)
constexpr int kBookThreads = 1024;
constexpr int kBookItems = 4;

// row stride of a matrix of n clusters: an odd number of 256-byte segments,
// so that the same column of successive rows falls on different channels
__host__ __device__ __forceinline__ long long mx_ld(int n) { return (((long long)n + 31) / 32 | 1) * 32; }

// Average: every squared distance starts from kTiny, which keeps the
// reciprocal root finite at distance zero. Float distances are zero or at least
// 2^-149, so kTiny changes no other value, and a sum below kZero is one of
// roots of kTiny: zero.
constexpr double kTiny = 1e-300, kZero = 1e-120;

// Square root of a positive double for the sums of average linkage:
// hardware reciprocal root, then Goldschmidt's coupled iteration and one
// residual correction (Markstein). No scaling: x is at least kTiny and below
// 2^270 (2^258 a coordinate, 2048 of them), its reciprocal root between 2^-135 and
// 2^499, and no product or residual of the steps leaves the normal range.
__device__ __forceinline__ double root_sum(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  const double e = __builtin_fma(-g, g, x);
  return __builtin_fma(e, h, g);
}

// What the rounding of a sum left over, in units of 2^-8 of its last place: a
// sum and its byte hold 61 bits. Heights of 7151 points d = 64 over 4096 to 65536
// point pairs, against long double, in units of 2^-53 (rms, largest): 2.2 and 4.6
// without it, 0.7 and 1.6 with it (the search rounds, which add the points
// themselves, 1.0 and 1.7).
typedef signed char Low;
struct Sum {
  double v, r;  // rounded, and the rest
};
// the unit at v >= 0 (2^-60 below v's power of two), and its inverse; from their
// exponent bits, the same unit for all v below 2^-960 (sums of distances are zero
// or at least 2^-149)
__device__ __forceinline__ int low_exp(double v) { return max(__double2hiint(v) >> 20, 64); }
__device__ __forceinline__ double low_value(double v, Low l) {
  return (double)(int)l * __hiloint2double((low_exp(v) - 60) << 20, 0);
}
__device__ __forceinline__ Low low_byte(const Sum &s) {
  // (the addition rounds to a whole number, which the low word then holds)
  const double q = s.r * __hiloint2double((2106 - low_exp(s.v)) << 20, 0) + 0x1.8p52;
  return (Low)max(min(__double2loint(q), 127), -127);
}
// a + b: its rounding, and what that left over, exactly (Knuth's two-sum)
__device__ __forceinline__ Sum two_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return Sum{s, (a - (s - t)) + (b - t)};
}
// s + rest, rounded again (the rest is far below s)
__device__ __forceinline__ Sum settled(double s, double rest) {
  const double v = s + rest;
  return Sum{v, rest - (v - s)};
}
// Both are the same bits with the operands (pairs) exchanged.
__device__ __forceinline__ Sum add2(double a, Low la, double b, Low lb) {
  const Sum s = two_sum(a, b);
  return settled(s.v, s.r + (low_value(a, la) + low_value(b, lb)));
}
__device__ __forceinline__ Sum add4(double a, Low la, double b, Low lb, double c, Low lc, double d, Low ld) {
  const Sum s = two_sum(a, b), t = two_sum(c, d), u = two_sum(s.v, t.v);
  return settled(u.v, u.r + ((s.r + (low_value(a, la) + low_value(b, lb))) +
                             (t.r + (low_value(c, lc) + low_value(d, ld)))));
}

// a cluster whose points do not lie in one window: several tiles meet in its entries
__device__ __forceinline__ bool straddles(int beg, int size) { return beg / kWin != (beg + size - 1) / kWin; }

// Complete: tiles of different wavefronts meet in the entries of a cluster that
// reaches into another window; those start at zero and keep the maximum.
// Average: a sum depends on the order of its terms, so the clusters are cut into
// pieces at the multiples of X.unit positions, and the tiles of one pair of
// pieces belong to one wavefront (block, d > 16), which takes them in a fixed
// order: the first stores, the others add (a wavefront's operations on an
// address stay in order). The pieces' sums are then added up per cluster.
template <int LINK>
__device__ __forceinline__ void put(double *p, double v, bool meet) {
  if (!meet) *p = v;
  else if (LINK == kComplete) atomicMax((unsigned long long *)p, pos_bits(v));
  else unsafeAtomicAdd(p, v);
}

// ------------------------------------------------------------------ enter --
// Cluster records of the active list (from slots, or of single points).
__global__ void k_mx_enter(State S, Mx X, int merges, int direct) {
  const int n = S.n;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    S.cnt->mx_merges = merges;
    const long long m = direct ? n : S.cnt->n_act;
    S.cnt->mx_terms += m;
    // every pair's exact value is computed from all its point pairs
    S.cnt->cluster_evals += m * (m - 1) / 2;
    S.cnt->refined += m * (m - 1) / 2;
    S.cnt->mx_exact += m * (m - 1) / 2;
    S.cnt->point_pairs += (long long)n * (n - 1) / 2;
    S.cnt->visits[1] += m * (m - 1);
  }
  if (direct) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
      X.c[0].id[i] = make_int4(i, 1, i, 0);
      X.c[0].eff[i] = 0.0;
      X.c[0].rsize[i] = 1.0;
      X.beg[i] = i;
      X.own[i] = i;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) S.cnt->n_act = n;
    return;
  }
  const int nact = S.cnt->n_act;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nact; i += gridDim.x * blockDim.x) {
    const int s = S.act[i];
    X.c[0].id[i] = make_int4(S.cid[s], S.csize[s], S.node[s], 0);
    X.c[0].eff[i] = S.eff[s];
    X.c[0].rsize[i] = 1.0 / (double)S.csize[s];
    X.beg[i] = S.cbeg[s];
    S.mdst[s] = i;  // slot -> place in the active list
  }
}
// cluster of every point position (points lie in active-list order). Average:
// its piece, numbered by the cluster's place plus the unit: along the positions
// one or the other grows from piece to piece, so the numbers are distinct (a
// cluster that ends with a unit leaves one unused).
__global__ void k_mx_own(State S, Mx X) {
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < S.n; p += gridDim.x * blockDim.x)
    X.own[p] = S.mdst[S.powner[p]] + (X.unit ? p / X.unit : 0);
}

// complete: entries in which several tiles meet start at zero
__global__ __launch_bounds__(kBlock) void k_mx_zero(Mx X, int m) {
  const long long ld = mx_ld(m);
  for (int i = blockIdx.x; i < m; i += gridDim.x) {
    const bool all = straddles(X.beg[i], X.c[0].id[i].y);
    for (int j = i + 1 + threadIdx.x; j < m; j += kBlock)
      if (all || straddles(X.beg[j], X.c[0].id[j].y)) X.k[0][i * ld + j] = 0.0;
  }
}

// ------------------------------------------------------------------ build --
// Values of all cluster (average: piece) pairs, upper half, d <= 16. A block
// stages 64 row points in LDS as FP64; each wavefront takes two windows of 64
// column points at a time, two column points per lane, and walks the rows. At the
// last row of a cluster the lanes' sums (maxima) go to LDS; after kHold of them
// the wavefront adds up the columns of every column cluster, a (row cluster,
// column cluster) pair per lane, and stores one value per pair.
// A block takes `rw` row windows in turn, a wavefront `cp` pairs of column
// windows: one window and one pair, or (average, clusters) a unit of either.
// Bound by the FP64 vector units: d subtractions and fused multiply-adds, the
// root (7 and the hardware's reciprocal root) and the sum per point pair. All
// loads are amortised over 64 rows. 500K points d = 2 average: 68 ms, 1.8e12
// pairs/s (the tiles of the search rounds 6.4e11); 250,007 points d = 10 average:
// 38 ms, 8.3e11 pairs/s.
constexpr int kHold = 8;
template <int LINK, int MAXD>
__global__ __launch_bounds__(kBlock) void k_mx_build_lo(const float *px, Mx X, double *K, long long ld, int n, int d,
                                                        int rw, int cp, int group) {
  __shared__ __attribute__((aligned(16))) double rows[kWin][MAXD];
  __shared__ int rown[kWin];
  __shared__ double held[kBlock / kWave][kHold][2 * kWin];
  __shared__ int heldr[kBlock / kWave][kHold];
  __shared__ int sown[kBlock / kWave][2 * kWin];             // column clusters: owner,
  __shared__ unsigned char sbeg[kBlock / kWave][2 * kWin];   // first column,
  __shared__ unsigned char send[kBlock / kWave][2 * kWin];   // last column, top bit
                                                             // set if tiles meet there
  const int nwin = (n + kWin - 1) / kWin, npair = (nwin + 1) / 2;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  // units of column pairs, from the row windows' own on
  const int ubeg = blockIdx.x * rw / (2 * cp) + blockIdx.y * group;
  const int uend = min((npair + cp - 1) / cp, ubeg + group);
  if (ubeg >= uend) return;  // uniform per block
  const double q0 = LINK == kAverage ? kTiny : 0.0;
  for (int I = blockIdx.x * rw; I < min(nwin, ((int)blockIdx.x + 1) * rw); ++I) {
    const int r0 = I * kWin, nrow = min(kWin, n - r0);
    __syncthreads();
    for (int t = threadIdx.x; t < kWin * MAXD; t += kBlock) {
      const int i = t / MAXD, k = t % MAXD;
      rows[i][k] = i < nrow && k < d ? (double)px[(size_t)(r0 + i) * d + k] : 0.0;
    }
    if (threadIdx.x < kWin) rown[threadIdx.x] = threadIdx.x < nrow ? X.own[r0 + threadIdx.x] : -1;
    __syncthreads();
    // rows that end a cluster within this window
    const int ro = rown[lane];
    const int rnext = lane + 1 < nrow ? rown[lane + 1] : -1;
    const unsigned long long ends = __ballot(lane < nrow && ro != rnext);
    const bool row_in = r0 > 0 && X.own[r0 - 1] == rown[0];  // first row's cluster began earlier
    // last row's cluster goes on (complete; a later tile adds to what average stores)
    const bool row_out = LINK == kComplete && r0 + nrow < n && X.own[r0 + nrow] == rown[nrow - 1];
    const int rfirst = rown[0], rlast = rown[nrow - 1];
    for (int u = ubeg + w; u < uend; u += kBlock / kWave)
      for (int P = max(u * cp, I / 2); P < min(npair, (u + 1) * cp); ++P) {
        double cv[2][MAXD];
        int oc[2];
        int nseg = 0, ncol = 0;
        // the columns: both windows, or the second one if the first lies before the rows
        const int p0 = max(2 * P, I) * kWin, p1 = min(n, (2 * P + 2) * kWin) - 1;
        const bool col_in = p0 > 0 && X.own[p0 - 1] == X.own[p0];
        const bool col_out = LINK == kComplete && p1 + 1 < n && X.own[p1 + 1] == X.own[p1];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int pos = (2 * P + c) * kWin + lane;
          const bool in = pos >= p0 && pos <= p1;
          oc[c] = in ? X.own[pos] : -1;
#pragma unroll
          for (int k = 0; k < MAXD; ++k) cv[c][k] = in && k < d ? (double)px[(size_t)pos * d + k] : 0.0;
          const bool head = in && (pos == p0 || X.own[pos - 1] != oc[c]);
          const bool tail = in && (pos == p1 || X.own[pos + 1] != oc[c]);
          const unsigned long long heads = __ballot(head);
          const int k = nseg + __popcll(heads & lanemask_lt()) - (head ? 0 : 1);
          if (head) {
            sown[w][k] = oc[c];
            sbeg[w][k] = (unsigned char)(c * kWin + lane);
          }
          if (tail) send[w][k] = (unsigned char)((c * kWin + lane) | ((k == 0 && col_in) || (pos == p1 && col_out) ? 0x80 : 0));
          nseg += __popcll(heads);
          ncol += __popcll(__ballot(in));
        }
        const bool points = nseg == ncol;  // every column cluster here is one point
        double acc[2] = {0.0, 0.0};
        int hold = 0;
        for (int r = 0; r < nrow; ++r) {
          double q[2] = {q0, q0};
#pragma unroll
          for (int k = 0; k < MAXD; ++k) {
            const double a = rows[r][k];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              const double u2 = a - cv[c][k];
              if (LINK == kComplete) q[c] += u2 * u2;  // as the oracle sums: bit-identical maxima
              else q[c] = __builtin_fma(u2, u2, q[c]);
            }
          }
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            if (LINK == kComplete) acc[c] = q[c] > acc[c] ? q[c] : acc[c];
            else acc[c] += root_sum(q[c]);
          }
          if (!((ends >> r) & 1ull)) continue;  // uniform
          if (points) {
            const int ri = __builtin_amdgcn_readfirstlane(rown[r]);
            const bool rs = (row_in && ri == rfirst) || (row_out && ri == rlast);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
              const int pos = (2 * P + c) * kWin + lane;
              if (ri < oc[c])
                put<LINK>(K + (size_t)ri * ld + oc[c], LINK == kAverage && acc[c] < kZero ? 0.0 : acc[c],
                          rs || (pos == p0 && col_in) || (pos == p1 && col_out));
            }
          } else {
            held[w][hold][lane] = acc[0];
            held[w][hold][kWin + lane] = acc[1];
            if (lane == 0) heldr[w][hold] = rown[r];
            if (++hold == kHold || (ends >> r) == 1ull) {
              // (a wavefront's LDS operations complete in order)
              for (int t = lane; t < hold * nseg; t += kWave) {
                const int h = t / nseg, k = t - h * nseg;
                const int e = send[w][k] & 0x7f;
                auto both = [](double x, double y) { return LINK == kComplete ? (y > x ? y : x) : x + y; };
                const double *v = held[w][h];
                int c = sbeg[w][k];
                double x = v[c++];
                for (; c + 3 <= e; c += 4) x = both(x, both(both(v[c], v[c + 1]), both(v[c + 2], v[c + 3])));
                for (; c <= e; ++c) x = both(x, v[c]);
                const int ri = heldr[w][h], ci = sown[w][k];
                if (ri < ci)
                  put<LINK>(K + (size_t)ri * ld + ci, LINK == kAverage && x < kZero ? 0.0 : x,
                            (row_in && ri == rfirst) || (row_out && ri == rlast) || (send[w][k] & 0x80));
              }
              hold = 0;
            }
          }
          acc[0] = acc[1] = 0.0;
        }
      }
  }
}

// The same for d > 16: 64 x 64 tiles, each thread a 4 x 4 block, coordinates
// staged 16 at a time; the tile's values go through LDS, where the rows and
// columns of each cluster are combined. Bound by the FP64 units (3 operations
// per pair and coordinate, complete; 2, average) and, next, by the LDS reads.
// The next stage is in flight while one is used, one barrier a stage, and the
// values take the stages' LDS (four blocks a CU). 50K points d = 128 complete
// (1.25e9 pairs): 24.6 ms with one stage and two barriers, 20.7 so; at the units'
// nominal rate 12.3. Stages of doubles, which save the conversions, 20.7 too.
constexpr int kKc = 16;
constexpr int kStageIt = kWin * kKc / kBlock;
template <int LINK>
__global__ __launch_bounds__(kBlock) void k_mx_build_hi(const float *px, Mx X, double *K, long long ld, int n, int d,
                                                        int rw, int group) {
  // two stages of coordinates; the values of the tile take their place
  struct Stage {
    float a[kKc][kWin + 4], b[kKc][kWin + 4];
  };
  static_assert(2 * sizeof(Stage) <= sizeof(double) * kWin * (kWin + 1), "both stages lie under the tile");
  __shared__ __attribute__((aligned(16))) double tile[kWin][kWin + 1];
  Stage *st = (Stage *)&tile[0][0];
  __shared__ int rown[kWin + 2], cown[kWin + 2];  // with the neighbours outside the window
  const int nwin = (n + kWin - 1) / kWin;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  // a block takes `rw` row windows in turn: one, or (average, clusters) a unit,
  // as many as divide `group`
  const int jbeg = blockIdx.x * rw + blockIdx.y * group, jend = min(nwin, jbeg + group);
  for (int I = blockIdx.x * rw; I < min(nwin, ((int)blockIdx.x + 1) * rw); ++I)
  for (int J = max(jbeg, I); J < jend; ++J) {
    const int r0 = I * kWin, nrow = min(kWin, n - r0);
    const int c0 = J * kWin, ncol = min(kWin, n - c0);
    __syncthreads();
    for (int t = threadIdx.x; t < kWin + 2; t += kBlock) {
      const int pr = r0 + t - 1, pc = c0 + t - 1;
      rown[t] = pr >= 0 && pr < n ? X.own[pr] : -1;
      cown[t] = pc >= 0 && pc < n ? X.own[pc] : -1;
    }
    double q[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) q[a][b] = LINK == kAverage ? kTiny : 0.0;
    // the next coordinates are loaded while these are used
    float pa[kStageIt], pb[kStageIt];
    auto load = [&](int k0) {
#pragma unroll
      for (int it = 0; it < kStageIt; ++it) {
        const int t = threadIdx.x + it * kBlock, i = t / kKc, k = k0 + t % kKc;
        pa[it] = k < d && i < nrow ? px[(size_t)(r0 + i) * d + k] : 0.0f;
        pb[it] = k < d && i < ncol ? px[(size_t)(c0 + i) * d + k] : 0.0f;
      }
    };
    load(0);
    for (int k0 = 0, cur = 0; k0 < d; k0 += kKc, cur ^= 1) {
      Stage &g = st[cur];
#pragma unroll
      for (int it = 0; it < kStageIt; ++it) {
        const int t = threadIdx.x + it * kBlock;
        g.a[t % kKc][t / kKc] = pa[it];
        g.b[t % kKc][t / kKc] = pb[it];
      }
      // one barrier: the stage written next was last read before it
      __syncthreads();
      if (k0 + kKc < d) load(k0 + kKc);
#pragma unroll 4
      for (int k = 0; k < kKc; ++k) {
        const float4 av = *(const float4 *)&g.a[k][ty * 4];
        const float4 bv = *(const float4 *)&g.b[k][tx * 4];
        const double ar[4] = {(double)av.x, (double)av.y, (double)av.z, (double)av.w};
        const double br[4] = {(double)bv.x, (double)bv.y, (double)bv.z, (double)bv.w};
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const double u = ar[a] - br[b];
            if (LINK == kComplete) q[a][b] += u * u;
            else q[a][b] = __builtin_fma(u, u, q[a][b]);
          }
      }
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) tile[ty * 4 + a][tx * 4 + b] = LINK == kComplete ? q[a][b] : root_sum(q[a][b]);
    __syncthreads();
    // columns of a cluster, row by row: the value lands in the cluster's last column
    for (int t = threadIdx.x; t < kWin * kWin; t += kBlock) {
      const int r = t / kWin, c = t % kWin;
      if (r >= nrow || c >= ncol) continue;
      const int o = cown[c + 1];
      if (c + 1 < ncol && cown[c + 2] == o) continue;  // not its last column here
      if (c > 0 && cown[c] == o) {
        double v = tile[r][c];
        for (int cc = c - 1; cc >= 0 && cown[cc + 1] == o; --cc) {
          const double u = tile[r][cc];
          v = LINK == kComplete ? (u > v ? u : v) : v + u;
        }
        tile[r][c] = v;
      }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kWin * kWin; t += kBlock) {
      const int r = t / kWin, c = t % kWin;
      if (r >= nrow || c >= ncol) continue;
      const int o = cown[c + 1], ri = rown[r + 1];
      if (c + 1 < ncol && cown[c + 2] == o) continue;
      if (r + 1 < nrow && rown[r + 2] == ri) continue;  // not its last row here
      if (ri >= o) continue;
      double v = tile[r][c];
      int rr = r - 1;
      for (; rr >= 0 && rown[rr + 1] == ri; --rr) {
        const double u = tile[rr][c];
        v = LINK == kComplete ? (u > v ? u : v) : v + u;
      }
      // another window's tile meets this one: the cluster lies across an edge
      // (average: an earlier tile's, of this block)
      bool sh = rown[0] == ri || cown[0] == o;
      if (LINK == kComplete) sh = sh || (r == nrow - 1 && rown[r + 2] == ri) || (c == ncol - 1 && cown[c + 2] == o);
      put<LINK>(K + (size_t)ri * ld + o, LINK == kAverage && v < kZero ? 0.0 : v, sh);
    }
  }
}

// Average, clusters: the sums of a cluster's pieces, rows first. A block takes 64
// clusters and 256 columns; the sums replace the first piece's row. Pieces are
// few (a unit holds two clusters or more on average), so both sweeps are short
// of the build.
__device__ __forceinline__ int2 mx_pieces(const Mx &X, int i) {  // first piece, number
  const int b = X.beg[i], e = b + X.c[0].id[i].y - 1;
  return make_int2(i + b / X.unit, e / X.unit - b / X.unit + 1);
}
__global__ __launch_bounds__(kBlock) void k_mx_fold_rows(Mx X, int m) {
  __shared__ int2 pc[kWin];
  const long long ld = mx_ld(X.pieces);
  const int i0 = blockIdx.x * kWin, nc = min(kWin, m - i0);
  if (threadIdx.x < nc) pc[threadIdx.x] = mx_pieces(X, i0 + threadIdx.x);
  __syncthreads();
  const int b = blockIdx.y * kBlock + threadIdx.x;
  if (b >= X.pieces) return;
  for (int r = 0; r < nc; ++r) {
    const int f = pc[r].x, k = pc[r].y;
    if (k == 1 || b < f + k) continue;
    double *p = X.kp + (size_t)f * ld + b;
    Sum s{*p, 0.0};
    for (int j = 1; j < k; ++j) {
      const Sum u = two_sum(s.v, p[j * ld]);
      s.v = u.v;
      s.r += u.r;
    }
    *p = s.v + s.r;
  }
}
// then columns, into both halves of the matrix: 64 x 64 tiles through LDS;
// infinity on the diagonal
__global__ __launch_bounds__(kBlock) void k_mx_fold(Mx X, int m) {
  __shared__ double t[kWin][kWin + 1];
  __shared__ Low tl[kWin][kWin + 4];
  __shared__ int2 pr[kWin], pc[kWin];
  const int I = blockIdx.x, J = blockIdx.y;
  if (J < I) return;
  const long long lp = mx_ld(X.pieces), ld = mx_ld(m);
  double *K = X.k[0];
  const int r0 = I * kWin, c0 = J * kWin;
  if (threadIdx.x < kWin) {
    if (r0 + (int)threadIdx.x < m) pr[threadIdx.x] = mx_pieces(X, r0 + threadIdx.x);
    if (c0 + (int)threadIdx.x < m) pc[threadIdx.x] = mx_pieces(X, c0 + threadIdx.x);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < kWin * kWin; j += kBlock) {
    const int r = j / kWin, c = j % kWin;
    if (r0 + r >= m || c0 + c >= m || c0 + c <= r0 + r) continue;
    const double *p = X.kp + (size_t)pr[r].x * lp + pc[c].x;
    Sum s{p[0], 0.0};
    for (int q = 1; q < pc[c].y; ++q) {
      const Sum u = two_sum(s.v, p[q]);
      s.v = u.v;
      s.r += u.r;
    }
    s = settled(s.v, s.r);
    const Low l = low_byte(s);
    t[r][c] = s.v;
    tl[r][c] = l;
    K[(size_t)(r0 + r) * ld + c0 + c] = s.v;
    X.kl[0][(size_t)(r0 + r) * ld + c0 + c] = l;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < kWin * kWin; j += kBlock) {
    const int r = j / kWin, c = j % kWin;  // of the transposed tile
    if (c0 + r < m && r0 + c < m && c0 + r >= r0 + c) {
      K[(size_t)(c0 + r) * ld + r0 + c] = c0 + r > r0 + c ? t[c][r] : INFINITY;
      X.kl[0][(size_t)(c0 + r) * ld + r0 + c] = c0 + r > r0 + c ? tl[c][r] : (Low)0;
    }
  }
}

// average, single points: nothing is left over yet (`words` of 16 bytes)
__global__ __launch_bounds__(kBlock) void k_mx_zero_low(uint4 *l, long long words) {
  const long long step = (long long)gridDim.x * kBlock;
  for (long long i = blockIdx.x * (long long)kBlock + threadIdx.x; i < words; i += step) l[i] = make_uint4(0, 0, 0, 0);
}

// lower half = upper half transposed, 64 x 64 tiles through LDS; infinity on
// the diagonal
__global__ __launch_bounds__(kBlock) void k_mx_mirror(Mx X, int m) {
  __shared__ double t[kWin][kWin + 1];
  const int I = blockIdx.x, J = blockIdx.y;
  if (J < I) return;
  const long long ld = mx_ld(m);
  double *K = X.k[0];
  const int r0 = I * kWin, c0 = J * kWin;
  for (int j = threadIdx.x; j < kWin * kWin; j += kBlock) {
    const int r = j / kWin, c = j % kWin;
    if (r0 + r < m && c0 + c < m) t[r][c] = K[(size_t)(r0 + r) * ld + c0 + c];
  }
  __syncthreads();
  for (int j = threadIdx.x; j < kWin * kWin; j += kBlock) {
    const int r = j / kWin, c = j % kWin;  // of the transposed tile
    if (c0 + r < m && r0 + c < m && c0 + r >= r0 + c)
      K[(size_t)(c0 + r) * ld + r0 + c] = c0 + r > r0 + c ? t[c][r] : INFINITY;
  }
}

// ------------------------------------------------------------------- pass --
struct Near {
  double v;
  int cid, q;
};
__device__ __forceinline__ void nearer(Near &b, double v, int cid, int q) {
  if (v < b.v || (v == b.v && cid < b.cid)) {
    b.v = v;
    b.cid = cid;
    b.q = q;
  }
}

// FIRST: nearest neighbours of the matrix as built. Else one round: row p of
// the new matrix from the rows and columns of its sources, and its nearest
// neighbour (key, then cluster ID) unless that is known: an unmerged cluster
// whose neighbour did not merge keeps it (merging brings no cluster nearer,
// Sec. 2.1). TPR threads per row, four columns of a thread in flight; a column
// index past the end repeats the last one, so no lane is masked. Average
// linkage compares sums times 1/size first (the row's own size is common to
// all) and divides only for a value that may win: the product and the quotient
// differ by less than 2^-50.
// Bound by memory: about (n_old^2 + n_new^2) * 8 bytes a round (9, average).
// 24 rounds from 7151 clusters on, average linkage: 53 us a round without the low
// bytes, 66 with them.
// A merged cluster's row (TWO sources) takes up to four values per column, so two
// columns at a time.
template <int LINK, bool FIRST, bool NEAR, bool TWO>
__device__ __forceinline__ void pass_row(const double *__restrict__ A, const Low *__restrict__ Al,
                                         const double *__restrict__ B, const Low *__restrict__ Bl,
                                         double *__restrict__ out, Low *__restrict__ outl, const int2 *__restrict__ src,
                                         const double *__restrict__ rsize, const int4 *__restrict__ id, int p,
                                         double sz, int nn, int t, int tpr, Near &b) {
  constexpr int U = TWO && LINK == kAverage ? 2 : 4;
  constexpr bool LOW = LINK == kAverage && !FIRST;
  double lim = INFINITY;  // b.v, for average in units of the sums over size
  for (int q0 = t; q0 < nn; q0 += U * tpr) {
    double v[U], rs[U];
    Low l[U];
    int2 c[U];
    int q[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      q[j] = min(q0 + j * tpr, nn - 1);
      if (!FIRST) c[j] = src[q[j]];
      if (NEAR && LINK == kAverage) rs[j] = rsize[q[j]];
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      v[j] = A[FIRST ? q[j] : c[j].x];
      if (LOW) l[j] = Al[c[j].x];
    }
    if (!FIRST) {
      if constexpr (TWO) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const double x = B[c[j].x];
          if (LINK == kComplete) {
            v[j] = x > v[j] ? x : v[j];
            if (c[j].y >= 0) {
              const double y = A[c[j].y], z = B[c[j].y];
              const double m2 = z > y ? z : y;
              v[j] = v[j] > m2 ? v[j] : m2;
            }
          } else {
            const Low lx = Bl[c[j].x];
            Sum s;
            if (c[j].y < 0) {
              s = add2(v[j], l[j], x, lx);
            } else {
              const double y = A[c[j].y], z = B[c[j].y];
              const Low ly = Al[c[j].y], lz = Bl[c[j].y];
              // the same grouping on both sides of the diagonal
              s = p < q[j] ? add4(v[j], l[j], x, lx, y, ly, z, lz) : add4(v[j], l[j], y, ly, x, lx, z, lz);
            }
            v[j] = s.v;
            l[j] = low_byte(s);
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < U; ++j)
          if (c[j].y >= 0) {
            const double y = A[c[j].y];
            if (LINK == kComplete) {
              v[j] = y > v[j] ? y : v[j];
            } else {
              const Sum s = add2(v[j], l[j], y, Al[c[j].y]);
              v[j] = s.v;
              l[j] = low_byte(s);
            }
          }
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        out[q[j]] = v[j];
        if (LOW) outl[q[j]] = l[j];
      }
    }
    if (NEAR) {
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const double key = LINK == kAverage ? v[j] * rs[j] : v[j];
        if (key <= lim && q[j] != p) {
          const int4 o = id[q[j]];
          nearer(b, LINK == kAverage ? v[j] / (sz * (double)o.y) : v[j], o.x, q[j]);
          lim = LINK == kAverage ? b.v * sz * (1.0 + 0x1p-49) : b.v;
        }
      }
    }
  }
}

template <int LINK, bool FIRST, int TPR>
__global__ __launch_bounds__(kBlock) void k_mx_pass(Mx X, const Counters *cnt) {
  const int nn = cnt->n_act;
  if (cnt->mx_err || (!FIRST && (nn <= 1 || !cnt->mx_ran))) return;
  const int src = FIRST ? 0 : (cnt->mx_rounds & 1) ^ 1;
  const bool fresh = FIRST || cnt->mx_merged == 0;  // every cluster looks again, see k_mx_book
  const int dst = FIRST ? src : src ^ 1;
  const long long lo = mx_ld(FIRST ? nn : cnt->mx_old), ln = mx_ld(nn);
  const MxClusters &C = X.c[dst];
  const int t = threadIdx.x % TPR;
  constexpr int RPB = kBlock / TPR;
  __shared__ Near red[kBlock / kWave];
  for (int p0 = blockIdx.x * RPB; p0 < nn; p0 += gridDim.x * RPB) {
    // (uniform in a wavefront)
    const int p = TPR == kBlock ? p0 : __builtin_amdgcn_readfirstlane(p0 + threadIdx.x / TPR);
    if (TPR < kBlock && p >= nn) break;
    int ra = p, rb = -1, old = -1;
    if (!FIRST) {
      const int2 c = X.src[p];
      ra = c.x;
      rb = c.y;
      if (rb < 0 && !fresh) old = X.place[X.nni[src][ra]];
    }
    const size_t oa = (size_t)ra * lo, ob = (size_t)(rb < 0 ? ra : rb) * lo, oo = (size_t)p * ln;
    const double *A = X.k[src] + oa, *B = X.k[src] + ob;
    double *out = X.k[dst] + oo;
    const Low *Al = LINK == kAverage ? X.kl[src] + oa : nullptr, *Bl = LINK == kAverage ? X.kl[src] + ob : nullptr;
    Low *outl = LINK == kAverage ? X.kl[dst] + oo : nullptr;
    Near b{INFINITY, 0x7fffffff, -1};
    if (old >= 0) {
      pass_row<LINK, FIRST, false, false>(A, Al, B, Bl, out, outl, X.src, C.rsize, C.id, p, 0.0, nn, t, TPR, b);
      if (t == 0) {
        X.nnv[dst][p] = X.nnv[src][ra];
        X.nni[dst][p] = old;
      }
      continue;
    }
    const double sz = (double)C.id[p].y;
    if (!FIRST && rb >= 0)  // uniform in the row
      pass_row<LINK, FIRST, true, !FIRST>(A, Al, B, Bl, out, outl, X.src, C.rsize, C.id, p, sz, nn, t, TPR, b);
    else
      pass_row<LINK, FIRST, true, false>(A, Al, B, Bl, out, outl, X.src, C.rsize, C.id, p, sz, nn, t, TPR, b);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      const double ov = __shfl_xor(b.v, o, kWave);
      const int oc = __shfl_xor(b.cid, o, kWave), oq = __shfl_xor(b.q, o, kWave);
      nearer(b, ov, oc, oq);
    }
    if (TPR > kWave) {
      const int w = threadIdx.x / kWave;
      if ((threadIdx.x & (kWave - 1)) == 0) red[w] = b;
      __syncthreads();
      if (threadIdx.x == 0)
        for (int j = 1; j < kBlock / kWave; ++j) nearer(b, red[j].v, red[j].cid, red[j].q);
      __syncthreads();
    }
    if (t == 0) {
      X.nnv[dst][p] = b.v;
      X.nni[dst][p] = b.q;
    }
  }
}

// ------------------------------------------------------------------- book --
constexpr int kScanMaxDim = 8;  // a searching cluster per lane up to this d

// Var of the union (the merge rule of Sec. 2.1 with its size factor), as k_merge
__device__ __forceinline__ void merge_var(const State &S, int4 M, double cab) {
  const double ns = (double)(M.z + M.w);
  const double v = S.cvar[M.x] + S.cvar[M.y] + ((double)M.z * (double)M.w / ns) * cab;
  S.cvar[M.x] = v;
  S.cmv[M.x] = v / ns;
}

// centroid of a merged cluster (kept slot, dropped slot, their sizes), as k_merge
template <int LINK>
__device__ __forceinline__ void merge_centroid(const State &S, int4 M) {
  const int d = S.d;
  double *sa = S.wsum + (size_t)M.x * d, *ca = S.wcen + (size_t)M.x * d;
  const double *sb = S.wsum + (size_t)M.y * d, *cb = S.wcen + (size_t)M.y * d;
  const double ns = (double)(M.z + M.w);
  if (LINK == kAvgSq) {
    double cab = 0.0;
    for (int k = 0; k < d; ++k) {
      const double t = ca[k] - cb[k];
      cab += t * t;
    }
    merge_var(S, M, cab);
  }
  for (int k = 0; k < d; ++k) {
    const double sum = sa[k] + sb[k];
    sa[k] = sum;
    ca[k] = sum / ns;
  }
}

// Exclusive scan of one value per thread over the block; `total` for all.
__device__ __forceinline__ unsigned long long book_scan(unsigned long long v, unsigned long long *ws,
                                                        unsigned long long &total) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  constexpr int kW = kBookThreads / kWave;
  unsigned long long x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  if (lane == kWave - 1) ws[w] = x;
  __syncthreads();
  unsigned long long before = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kW; ++k) {
    const unsigned long long y = ws[k];
    before += k < w ? y : 0ull;
    tot += y;
  }
  __syncthreads();
  total = tot;
  return x - v + before;
}

// One block, one round: the reciprocal pairs of the nearest neighbours found
// by the last pass merge (Alg. 1), every cluster gets its place in the next
// round's records, and the merges their dendrogram rows. Exact ties between a
// kept neighbour and a new cluster can leave a round without a reciprocal pair;
// then every cluster looks again, and the pair of the smallest value whose
// lower ID is lowest is reciprocal.
// Rounds of at most `stop` clusters are left to the tail kernels.
// Nothing is merged on non-finite input (a direct call's check is read by the
// host only after these kernels ran), and no row past the n - 1 there are is
// written, whatever the values.
template <int LINK>
__global__ __launch_bounds__(kBookThreads) void k_mx_book(State S, Mx X, int stop) {
  constexpr bool CEN = centroid_link(LINK);
  Counters *cnt = S.cnt;
  const int n = cnt->n_act;
  if (n <= 1 || n <= stop || cnt->mx_err || cnt->nonfinite) {  // uniform
    if (threadIdx.x == 0) cnt->mx_ran = 0;
    return;
  }
  __shared__ unsigned long long ws[kBookThreads / kWave];
  const int rounds = cnt->mx_rounds, src = rounds & 1;
  const MxClusters &O = X.c[src], &N = X.c[src ^ 1];
  int *nni = X.nni[src];
  double *nnv = X.nnv[src];
  const int base = cnt->mx_merges, before = cnt->mx_merged;
  int kept = 0, merged = 0, bad = 0;
  constexpr int kTileN = kBookThreads * kBookItems;
  if (CEN && X.parts > 1) {
    // the best of the column parts of the last scan
    const int nt = cnt->mx_nterm;
    for (int i = threadIdx.x; i < nt; i += kBookThreads) {
      Near b{INFINITY, 0x7fffffff, -1};
      for (int k = 0; k < X.parts; ++k) {
        const int2 c = X.pc[(size_t)k * X.cap + i];
        nearer(b, X.pv[(size_t)k * X.cap + i], c.x, c.y);
      }
      const int p = X.term[i];
      nnv[p] = b.v;
      nni[p] = b.q;
    }
    __syncthreads();
  }
  for (int b0 = 0; b0 < n; b0 += kTileN) {
    int mate[kBookItems], part[kBookItems];
    int4 id[kBookItems], idm[kBookItems];
    double eff[kBookItems], effm[kBookItems];
    unsigned long long cntv = 0;
    // two dependent loads in all: the neighbour, then everything of both
#pragma unroll
    for (int j = 0; j < kBookItems; ++j) {
      const int i = min(b0 + (int)threadIdx.x * kBookItems + j, n - 1);
      mate[j] = nni[i];
      id[j] = O.id[i];
      eff[j] = O.eff[i];
    }
#pragma unroll
    for (int j = 0; j < kBookItems; ++j) {
      const int u = max(mate[j], 0);
      part[j] = nni[u];
      idm[j] = O.id[u];
      effm[j] = O.eff[u];
    }
#pragma unroll
    for (int j = 0; j < kBookItems; ++j) {
      const int i = b0 + threadIdx.x * kBookItems + j;
      if (i >= n) {
        mate[j] = -2;  // no cluster here
        continue;
      }
      if (mate[j] < 0 || mate[j] == i) bad = 1;  // no neighbour: cannot occur on finite input
      if (part[j] != i || mate[j] == i) mate[j] = -1;
      else if (idm[j].x < id[j].x) mate[j] = -2;  // merges into the other one
      if (mate[j] != -1) X.place[i] = -1;
      if (mate[j] != -2) cntv += mate[j] >= 0 ? (1ull << 32) + 1ull : 1ull;
    }
    unsigned long long tot;
    const unsigned long long ex = book_scan(cntv, ws, tot);
    int p = kept + (int)(ex & 0xffffffffu), ml = merged + (int)(ex >> 32);
#pragma unroll
    for (int j = 0; j < kBookItems; ++j) {
      const int i = b0 + threadIdx.x * kBookItems + j;
      const int b = mate[j];
      if (b == -2) continue;
      X.src[p] = make_int2(i, b);
      int sz = id[j].y, node = id[j].z;
      double e = eff[j];
      if (b >= 0) {
        if (base + ml > S.n - 2) bad = 1;  // (never on sound records)
        const int mr = min(base + ml, S.n - 2);
        const double h = key_to_height(LINK, nnv[i]);
        S.row_na[mr] = node;
        S.row_nb[mr] = idm[j].z;
        S.row_h[mr] = h;
        S.row_lo[mr] = id[j].x;
        if (CEN) X.mpair[ml] = make_int4(id[j].w, idm[j].w, id[j].y, idm[j].y);
        sz += idm[j].y;
        S.row_size[mr] = sz;
        e = fmax(fmax(e, effm[j]), h);
        S.row_eff[mr] = e;
        node = S.n + mr;
        ++ml;
      } else {
        X.place[i] = p;
      }
      N.id[p] = make_int4(id[j].x, sz, node, id[j].w);
      N.eff[p] = e;
      if (LINK == kAverage) N.rsize[p] = 1.0 / (double)sz;
      ++p;
    }
    kept += (int)(tot & 0xffffffffu);
    merged += (int)(tot >> 32);
  }
  bad = __syncthreads_or(bad);
  int nterm = n;
  if (CEN) {
    // merged clusters' centroids, then the clusters that search again: merged,
    // or their neighbour did (see k_mx_pass)
    if (S.d <= kScanMaxDim && !bad)
      for (int m = threadIdx.x; m < merged; m += kBookThreads) merge_centroid<LINK>(S, X.mpair[m]);
    nterm = 0;
    for (int b0 = 0; b0 < kept && !bad; b0 += kTileN) {
      int old[kBookItems];
      double v[kBookItems];
      unsigned long long c = 0;
#pragma unroll
      for (int j = 0; j < kBookItems; ++j) {
        const int p = b0 + threadIdx.x * kBookItems + j;
        old[j] = -2;
        if (p >= kept) continue;
        const int2 s = X.src[p];
        old[j] = s.y < 0 && merged > 0 ? X.place[nni[s.x]] : -1;
        v[j] = nnv[s.x];
        c += old[j] < 0 ? 1ull : 0ull;
      }
      unsigned long long tot;
      int t = nterm + (int)book_scan(c, ws, tot);
#pragma unroll
      for (int j = 0; j < kBookItems; ++j) {
        const int p = b0 + threadIdx.x * kBookItems + j;
        if (old[j] == -1) {
          X.term[t++] = p;
        } else if (old[j] >= 0) {
          X.nnv[src ^ 1][p] = v[j];
          X.nni[src ^ 1][p] = old[j];
        }
      }
      nterm += (int)tot;
    }
  }
  if (threadIdx.x == 0) {
    if (bad) cnt->mx_err = 1;
    else if (merged == 0 && rounds > 0 && before == 0) cnt->mx_err = 2;
    cnt->mx_old = n;
    cnt->mx_merged = merged;
    cnt->n_act = kept;
    cnt->mx_merges = base + merged;
    cnt->mx_rounds = rounds + 1;
    cnt->mx_ran = 1;
    if (CEN) {
      cnt->mx_nterm = nterm;
      cnt->cluster_evals += (long long)nterm * (kept - 1);
      cnt->refined += (long long)nterm * (kept - 1);
      cnt->mx_exact += (long long)nterm * (kept - 1);
      cnt->visits[1] += (long long)nterm * (kept - 1);
    }
    cnt->mx_terms += CEN ? nterm : kept;
  }
}

// -------------------------------------------------------------------- scan --
// Ward and avg-2: values follow from the centroids in O(d), so nothing is kept
// but the records: a round compares every searching cluster with all others.
// Up to kScanMaxDim coordinates: a searching cluster per lane, its centroid in
// registers; the columns of a part are dealt out to the block's 16 wavefronts,
// which stage 64 at a time in LDS and walk them (broadcast reads). The keys are
// those of the other searches, evaluated in the same order. Ward's division is
// taken only where the cross-multiplied test leaves the column a chance.
// Bound by the FP64 units (about 3 d + 8 slots per pair) and, below some
// thousand clusters, by the launch and the two dependent sweeps of a round.
constexpr int kScanThreads = 1024;
template <int LINK, int MAXD>
__global__ __launch_bounds__(kScanThreads) void k_sc_scan(State S, Mx X) {
  const Counters *cnt = S.cnt;
  const int nn = cnt->n_act, nt = cnt->mx_nterm, dst = cnt->mx_rounds & 1;
  if (nn <= 1 || cnt->mx_err || !cnt->mx_ran) return;
  constexpr int kW = kScanThreads / kWave;
  __shared__ double cen[kW][kWave][MAXD];
  __shared__ double vcol[kW][kWave];
  __shared__ int4 idc[kW][kWave];
  __shared__ Near red[kW][kWave];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const int d = S.d, parts = gridDim.y;
  const int chunks = (nn + kWave - 1) / kWave;
  for (int t0 = blockIdx.x * kWave; t0 < nt; t0 += gridDim.x * kWave) {
    const int ti = min(t0 + lane, nt - 1);
    const int p = X.term[ti];
    const int4 me = X.c[dst].id[p];
    double ct[MAXD];
#pragma unroll
    for (int k = 0; k < MAXD; ++k) ct[k] = k < d ? S.wcen[(size_t)me.w * d + k] : 0.0;
    const double sz = (double)me.y, vt = LINK == kAvgSq ? S.cmv[me.w] : 0.0;
    Near b{INFINITY, 0x7fffffff, -1};
    double lim = INFINITY;
    for (int c = blockIdx.y * kW + w; c < chunks; c += parts * kW) {
      const int q0 = c * kWave, cols = min(kWave, nn - q0);
      {
        const int4 o = X.c[dst].id[min(q0 + lane, nn - 1)];
        idc[w][lane] = o;
#pragma unroll
        for (int k = 0; k < MAXD; ++k) cen[w][lane][k] = k < d ? S.wcen[(size_t)o.w * d + k] : 0.0;
        vcol[w][lane] = LINK == kAvgSq ? S.cmv[o.w] : (double)o.y;
      }
      // (a wavefront's LDS operations complete in order)
      for (int j = 0; j < cols; ++j) {
        double q = 0.0;
#pragma unroll
        for (int k = 0; k < MAXD; ++k) {
          const double u = ct[k] - cen[w][j][k];
          q += u * u;  // (coordinates past d add zero)
        }
        const double x = vcol[w][j];
        bool near;
        double key = 0.0;
        if (LINK == kWard) {
          near = q * (2.0 * sz * x) <= lim * (sz + x);
        } else {
          key = q + (vt + x);
          near = key <= lim;
        }
        if (near && q0 + j != p) {
          if (LINK == kWard) key = ((2.0 * sz * x) / (sz + x)) * q;
          nearer(b, key, idc[w][j].x, q0 + j);
          lim = LINK == kWard ? b.v * (1.0 + 0x1p-48) : b.v;
        }
      }
    }
    red[w][lane] = b;
    __syncthreads();
    if (w == 0) {
      for (int k = 1; k < kW; ++k) nearer(b, red[k][lane].v, red[k][lane].cid, red[k][lane].q);
      if (t0 + lane < nt) {
        if (parts == 1) {
          X.nnv[dst][p] = b.v;
          X.nni[dst][p] = b.q;
        } else {
          X.pv[(size_t)blockIdx.y * X.cap + t0 + lane] = b.v;
          X.pc[(size_t)blockIdx.y * X.cap + t0 + lane] = make_int2(b.cid, b.q);
        }
      }
    }
    __syncthreads();
  }
}

// More coordinates: 64 x 64 tiles of centroids, each thread a 4 x 4 block, 16
// coordinates staged at a time.
template <int LINK>
__global__ __launch_bounds__(kBlock) void k_sc_scan_hi(State S, Mx X) {
  const Counters *cnt = S.cnt;
  const int nn = cnt->n_act, nt = cnt->mx_nterm, dst = cnt->mx_rounds & 1;
  if (nn <= 1 || cnt->mx_err || !cnt->mx_ran) return;
  __shared__ __attribute__((aligned(16))) double As[kKc][kWin + 2];
  __shared__ __attribute__((aligned(16))) double Bs[kKc][kWin + 2];
  __shared__ int4 idr[kWin], idc[kWin];
  __shared__ int place[kWin];
  __shared__ double vr[kWin], vc[kWin];
  const int d = S.d, parts = gridDim.y;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int chunks = (nn + kWin - 1) / kWin;
  for (int t0 = blockIdx.x * kWin; t0 < nt; t0 += gridDim.x * kWin) {
    __syncthreads();
    if (threadIdx.x < kWin) {
      const int p = X.term[min(t0 + (int)threadIdx.x, nt - 1)];
      const int4 o = X.c[dst].id[p];
      place[threadIdx.x] = p;
      idr[threadIdx.x] = o;
      vr[threadIdx.x] = LINK == kAvgSq ? S.cmv[o.w] : (double)o.y;
    }
    Near b[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) b[a] = Near{INFINITY, 0x7fffffff, -1};
    for (int c = blockIdx.y; c < chunks; c += parts) {
      const int q0 = c * kWin;
      __syncthreads();
      if (threadIdx.x < kWin) {
        const int4 o = X.c[dst].id[min(q0 + (int)threadIdx.x, nn - 1)];
        idc[threadIdx.x] = o;
        vc[threadIdx.x] = LINK == kAvgSq ? S.cmv[o.w] : (double)o.y;
      }
      double q[4][4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int e = 0; e < 4; ++e) q[a][e] = 0.0;
      for (int k0 = 0; k0 < d; k0 += kKc) {
        __syncthreads();
        for (int t = threadIdx.x; t < kWin * kKc; t += kBlock) {
          const int i = t / kKc, k = t % kKc;
          const bool in = k0 + k < d;
          As[k][i] = in ? S.wcen[(size_t)idr[i].w * d + k0 + k] : 0.0;
          Bs[k][i] = in ? S.wcen[(size_t)idc[i].w * d + k0 + k] : 0.0;
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < kKc; ++k) {
          const double2 a0 = *(const double2 *)&As[k][ty * 4], a1 = *(const double2 *)&As[k][ty * 4 + 2];
          const double2 b0 = *(const double2 *)&Bs[k][tx * 4], b1 = *(const double2 *)&Bs[k][tx * 4 + 2];
          const double ar[4] = {a0.x, a0.y, a1.x, a1.y}, br[4] = {b0.x, b0.y, b1.x, b1.y};
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double u = ar[a] - br[e];
              q[a][e] += u * u;
            }
        }
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int r = ty * 4 + a;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int cc = tx * 4 + e, col = q0 + cc;
          if (col >= nn || col == place[r]) continue;
          const double x = vc[cc], sz = vr[r];
          const double key = LINK == kWard ? ((2.0 * sz * x) / (sz + x)) * q[a][e] : q[a][e] + (sz + x);
          nearer(b[a], key, idc[cc].x, col);
        }
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        const double ov = __shfl_xor(b[a].v, o, kWave);
        const int oc = __shfl_xor(b[a].cid, o, kWave), oq = __shfl_xor(b[a].q, o, kWave);
        nearer(b[a], ov, oc, oq);
      }
      const int r = ty * 4 + a;
      if (tx == 0 && t0 + r < nt) {
        if (parts == 1) {
          X.nnv[dst][place[r]] = b[a].v;
          X.nni[dst][place[r]] = b[a].q;
        } else {
          X.pv[(size_t)blockIdx.y * X.cap + t0 + r] = b[a].v;
          X.pc[(size_t)blockIdx.y * X.cap + t0 + r] = make_int2(b[a].cid, b[a].q);
        }
      }
    }
  }
}

// centroids of the round's merged clusters, d > kScanMaxDim: a wavefront each
template <int LINK>
__global__ __launch_bounds__(kBlock) void k_sc_merge(State S, Mx X) {
  const Counters *cnt = S.cnt;
  if (cnt->mx_err || cnt->n_act <= 1 || !cnt->mx_ran) return;
  extern __shared__ double sq[];  // d per wavefront (avg-2)
  const int d = S.d, nm = cnt->mx_merged;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  for (int m = blockIdx.x * (kBlock / kWave) + w; m < nm; m += gridDim.x * (kBlock / kWave)) {
    const int4 M = X.mpair[m];
    double *sa = S.wsum + (size_t)M.x * d, *ca = S.wcen + (size_t)M.x * d;
    const double *sb = S.wsum + (size_t)M.y * d, *cb = S.wcen + (size_t)M.y * d;
    const double ns = (double)(M.z + M.w);
    for (int k = lane; k < d; k += kWave) {
      if (LINK == kAvgSq) {
        const double t = ca[k] - cb[k];
        sq[w * d + k] = t * t;
      }
      const double sum = sa[k] + sb[k];
      sa[k] = sum;
      ca[k] = sum / ns;
    }
    if (LINK == kAvgSq && lane == 0) {
      double cab = 0.0;
      for (int k = 0; k < d; ++k) cab += sq[w * d + k];  // in order, as k_merge
      merge_var(S, M, cab);
    }
  }
}

// -------------------------------------------------------------------- tail --
// The last rounds in one block, everything in LDS: a round of a few hundred
// clusters is otherwise bound by two launches and some ten dependent loads
// from memory (25 us); here it is bound by its barriers (about 3 us). Clusters
// keep their places; `act` lists the ones alive.
constexpr int kTailThreads = 1024;
constexpr int kMatTail = 176;    // lower triangle of 176 clusters: 123 KB, and 15 KB of low bytes
constexpr int kCenTail = 512;    // scan rounds: one cluster per thread at most,
constexpr int kCenTailNd = 4096; // and two FP64 values per coordinate: 64 KB

struct TailShared {
  unsigned long long ws[kTailThreads / kWave];
  int nact, merged, nterm, err;
};

// rank of this thread among those with `f`, and their number
__device__ __forceinline__ int tail_rank(bool f, unsigned long long *ws, int &total) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const unsigned long long m = __ballot(f);
  if (lane == 0) ws[w] = (unsigned long long)__popcll(m);
  __syncthreads();
  int before = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kTailThreads / kWave; ++k) {
    const int c = (int)ws[k];
    before += k < w ? c : 0;
    tot += c;
  }
  __syncthreads();
  total = tot;
  return before + __popcll(m & lanemask_lt());
}

// Records of the tail's clusters in LDS.
struct TailRec {
  double *eff, *nnv;
  int *cid, *size, *node, *nni, *st, *act, *term;  // st: merge number, -1 unmerged, -2 dropped
  int *ma, *mb;                                    // merged pairs
};
__device__ __forceinline__ char *tail_carve(TailRec &R, char *p, int n) {
  auto take = [&](size_t bytes) {
    char *q = p;
    p += (bytes + 15) & ~(size_t)15;
    return q;
  };
  R.eff = (double *)take(n * 8);
  R.nnv = (double *)take(n * 8);
  R.cid = (int *)take(n * 4);
  R.size = (int *)take(n * 4);
  R.node = (int *)take(n * 4);
  R.nni = (int *)take(n * 4);
  R.st = (int *)take(n * 4);
  R.act = (int *)take(n * 4);
  R.term = (int *)take(n * 4);
  R.ma = (int *)take(n * 4);
  R.mb = (int *)take(n * 4);
  return p;
}
inline size_t tail_rec_bytes(int n) { return (size_t)n * 52 + 11 * 16; }

// One round's reciprocal pairs: rows, merged records (value, size, node, eff)
// and the new active list; the clusters that search again. Every thread holds
// at most one cluster. Returns the number of merges.
template <int LINK>
__device__ __forceinline__ int tail_book(State &S, TailRec &R, TailShared &T, int &nact, int &base, int &nterm) {
  const int t = threadIdx.x;
  const int a = t < nact ? R.act[t] : -1;
  int b = -1;
  bool drop = false;
  if (a >= 0) {
    const int j = R.nni[a];
    if (j >= 0 && j != a && R.nni[j] == a) {
      if (R.cid[j] < R.cid[a]) drop = true;
      else b = j;
    }
    if (j < 0 || j == a) T.err = 1;
  }
  int merged, kept;
  const int m = tail_rank(b >= 0, T.ws, merged);
  const int k = tail_rank(a >= 0 && !drop, T.ws, kept);
  if (a >= 0) {
    R.st[a] = drop ? -2 : (b >= 0 ? m : -1);
    if (!drop) R.act[k] = a;  // (every thread has read its own entry)
    if (b >= 0 && base + m >= S.n - 1) T.err = 1;  // (never on sound records)
    if (b >= 0 && base + m < S.n - 1) {
      const int mr = base + m;
      const double h = key_to_height(LINK, R.nnv[a]);
      const int sz = R.size[a] + R.size[b];
      const double e = fmax(fmax(R.eff[a], R.eff[b]), h);
      S.row_na[mr] = R.node[a];
      S.row_nb[mr] = R.node[b];
      S.row_h[mr] = h;
      S.row_lo[mr] = R.cid[a];
      S.row_size[mr] = sz;
      S.row_eff[mr] = e;
      R.ma[m] = a;
      R.mb[m] = b;
    }
  }
  __syncthreads();
  const bool again = a >= 0 && !drop && (merged == 0 || b >= 0 || R.st[max(R.nni[a], 0)] != -1);
  const int q = tail_rank(again, T.ws, nterm);
  if (again) R.term[q] = a;
  nact = kept;
  base += merged;
  return merged;
}

// size, node and eff of the merged clusters, once their old values are read
template <int LINK>
__device__ __forceinline__ void tail_merge_rec(const State &S, TailRec &R, int m, int base) {
  const int a = R.ma[m], b = R.mb[m];
  R.eff[a] = fmax(fmax(R.eff[a], R.eff[b]), key_to_height(LINK, R.nnv[a]));
  R.size[a] += R.size[b];
  R.node[a] = S.n + base + m;
}

// Lanes per searching cluster: a power of two that gives every thread work.
__device__ __forceinline__ int tail_group(int nterm) {
  int g = 1;
  while (g < kWave && nterm * g * 2 <= kTailThreads) g *= 2;
  return g;
}
__device__ __forceinline__ void tail_near(TailRec &R, int p, Near b, int g, bool in) {
  for (int o = g / 2; o > 0; o >>= 1) {
    const double ov = __shfl_xor(b.v, o, kWave);
    const int oc = __shfl_xor(b.cid, o, kWave), oq = __shfl_xor(b.q, o, kWave);
    nearer(b, ov, oc, oq);
  }
  if (in && (threadIdx.x & (g - 1)) == 0) {
    R.nnv[p] = b.v;
    R.nni[p] = b.q;
  }
}

__device__ __forceinline__ void tail_begin(const Mx &X, TailRec &R, int src, int n) {
  const int t = threadIdx.x;
  if (t < n) {
    const int4 o = X.c[src].id[t];
    R.cid[t] = o.x;
    R.size[t] = o.y;
    R.node[t] = o.z;
    R.eff[t] = X.c[src].eff[t];
    R.nnv[t] = X.nnv[src][t];
    R.nni[t] = X.nni[src][t];
    R.act[t] = t;
  }
}
__device__ __forceinline__ void tail_end(Counters *cnt, int err, int nact, int base, int rounds, long long terms,
                                         long long evals) {
  cnt->mx_err = err;
  cnt->n_act = nact;
  cnt->mx_merges = base;
  cnt->mx_rounds += rounds;
  cnt->mx_terms += terms;
  if (evals) {
    cnt->cluster_evals += evals;
    cnt->refined += evals;
    cnt->mx_exact += evals;
    cnt->visits[1] += evals;
  }
}

// complete, average: the matrix's lower triangle in LDS
template <int LINK>
__global__ __launch_bounds__(kTailThreads) void k_mx_tail(State S, Mx X, int stop) {
  Counters *cnt = S.cnt;
  int nact = cnt->n_act;
  if (nact <= 1 || nact > stop || cnt->mx_err || cnt->nonfinite) return;
  extern __shared__ __attribute__((aligned(16))) char sm[];
  __shared__ TailShared T;
  const int n = nact, src = cnt->mx_rounds & 1;
  const long long ld = mx_ld(n);
  TailRec R;
  double *K = (double *)tail_carve(R, sm, stop);
  Low *L = (Low *)(K + stop * (stop - 1) / 2);
  auto at = [](int i, int j) { return i > j ? i * (i - 1) / 2 + j : j * (j - 1) / 2 + i; };
  tail_begin(X, R, src, n);
  if (threadIdx.x == 0) T.err = 0;
  for (int e = threadIdx.x; e < n * n; e += kTailThreads) {
    const int i = e / n, j = e - i * n;
    if (j >= i) continue;
    K[at(i, j)] = X.k[src][i * ld + j];
    if (LINK == kAverage) L[at(i, j)] = X.kl[src][i * ld + j];
  }
  int base = cnt->mx_merges, rounds = 0, before = cnt->mx_merged;
  long long terms = 0;
  __syncthreads();
  // a round of m merges leaves n - m clusters: at most (kMatTail / 2)^2 new values
  constexpr int kHeld = (kMatTail / 2 * (kMatTail / 2) + kTailThreads - 1) / kTailThreads;
  while (nact > 1) {
    int nterm;
    const int was = base;
    const int merged = tail_book<LINK>(S, R, T, nact, base, nterm);
    if (T.err || (merged == 0 && before == 0 && rounds > 0)) break;  // uniform
    before = merged;
    // new rows from the old values, held in registers until all are read
    double v[kHeld];
    Low l[kHeld];
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
      const int e = u * kTailThreads + threadIdx.x;
      v[u] = -1.0;
      if (e >= merged * nact) continue;
      const int m = e / nact, c = R.act[e - m * nact];
      const int a = R.ma[m], b = R.mb[m];
      if (c == a) continue;
      const int cm = R.st[c];
      const int ac = at(a, c), bc = at(b, c);
      const double x = K[ac], y = K[bc];
      int cb = 0, az = 0, bz = 0;
      double z = 0.0, w = 0.0;
      if (cm >= 0) {
        cb = R.mb[cm];
        az = at(a, cb);
        bz = at(b, cb);
        z = K[az];
        w = K[bz];
      }
      if (LINK == kComplete) {
        v[u] = y > x ? y : x;
        if (cm >= 0) {
          const double q = w > z ? w : z;
          v[u] = q > v[u] ? q : v[u];
        }
      } else {
        Sum s;
        if (cm < 0) s = add2(x, L[ac], y, L[bc]);
        else  // the same on both sides
          s = a < c ? add4(x, L[ac], y, L[bc], z, L[az], w, L[bz]) : add4(x, L[ac], z, L[az], y, L[bc], w, L[bz]);
        v[u] = s.v;
        l[u] = low_byte(s);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
      const int e = u * kTailThreads + threadIdx.x;
      if (e >= merged * nact || v[u] < 0.0) continue;
      const int m = e / nact;
      const int to = at(R.ma[m], R.act[e - m * nact]);
      K[to] = v[u];
      if (LINK == kAverage) L[to] = l[u];
    }
    for (int m = threadIdx.x; m < merged; m += kTailThreads) tail_merge_rec<LINK>(S, R, m, was);
    __syncthreads();
    const int g = tail_group(nterm);
    for (int e0 = 0; e0 < nterm * g; e0 += kTailThreads) {
      const int e = e0 + threadIdx.x;
      const bool in = e < nterm * g;
      const int p = R.term[in ? e / g : 0];
      Near b{INFINITY, 0x7fffffff, -1};
      if (in) {
        const double sz = (double)R.size[p];
        for (int i = e & (g - 1); i < nact; i += g) {
          const int c = R.act[i];
          if (c == p) continue;
          double key = K[at(p, c)];
          if (LINK == kAverage) key = key / (sz * (double)R.size[c]);
          nearer(b, key, R.cid[c], c);
        }
      }
      tail_near(R, p, b, g, in);
    }
    ++rounds;
    terms += nact > 1 ? nact : 0;
    __syncthreads();
  }
  if (threadIdx.x == 0) tail_end(cnt, T.err ? 1 : (nact > 1 ? 2 : 0), nact, base, rounds, terms, 0);
}

// Ward, avg-2: centroids and coordinate sums in LDS
template <int LINK>
__global__ __launch_bounds__(kTailThreads) void k_sc_tail(State S, Mx X, int stop) {
  Counters *cnt = S.cnt;
  int nact = cnt->n_act;
  if (nact <= 1 || nact > stop || cnt->mx_err || cnt->nonfinite) return;
  extern __shared__ __attribute__((aligned(16))) char sm[];
  __shared__ TailShared T;
  const int n = nact, src = cnt->mx_rounds & 1, d = S.d;
  TailRec R;
  double *cen = (double *)tail_carve(R, sm, stop);
  double *sum = cen + (size_t)stop * d, *var = sum + (size_t)stop * d, *mv = var + stop;
  if (X.parts > 1) {
    // the best of the column parts of the last scan
    const int nt = cnt->mx_nterm;
    for (int i = threadIdx.x; i < nt; i += kTailThreads) {
      Near b{INFINITY, 0x7fffffff, -1};
      for (int k = 0; k < X.parts; ++k) {
        const int2 c = X.pc[(size_t)k * X.cap + i];
        nearer(b, X.pv[(size_t)k * X.cap + i], c.x, c.y);
      }
      const int p = X.term[i];
      X.nnv[src][p] = b.v;
      X.nni[src][p] = b.q;
    }
    __syncthreads();
  }
  tail_begin(X, R, src, n);
  if (threadIdx.x == 0) T.err = 0;
  for (int e = threadIdx.x; e < n * d; e += kTailThreads) {
    const int i = e / d, k = e - i * d;
    const size_t o = (size_t)X.c[src].id[i].w * d + k;
    cen[e] = S.wcen[o];
    sum[e] = S.wsum[o];
  }
  if (LINK == kAvgSq && threadIdx.x < n) {
    const int s = X.c[src].id[threadIdx.x].w;
    var[threadIdx.x] = S.cvar[s];
    mv[threadIdx.x] = S.cmv[s];
  }
  int base = cnt->mx_merges, rounds = 0, before = cnt->mx_merged;
  long long terms = 0, evals = 0;
  __syncthreads();
  while (nact > 1) {
    int nterm;
    const int was = base;
    const int merged = tail_book<LINK>(S, R, T, nact, base, nterm);
    if (T.err || (merged == 0 && before == 0 && rounds > 0)) break;  // uniform
    before = merged;
    if (LINK == kAvgSq && (int)threadIdx.x < merged) {
      const int a = R.ma[threadIdx.x], b = R.mb[threadIdx.x];
      double cab = 0.0;
      for (int k = 0; k < d; ++k) {
        const double u = cen[a * d + k] - cen[b * d + k];
        cab += u * u;
      }
      const double sa = (double)R.size[a], sb = (double)R.size[b], ns = (double)(R.size[a] + R.size[b]);
      var[a] = var[a] + var[b] + (sa * sb / ns) * cab;
      mv[a] = var[a] / ns;
    }
    if (LINK == kAvgSq) __syncthreads();
    for (int e = threadIdx.x; e < merged * d; e += kTailThreads) {
      const int m = e / d, k = e - m * d, a = R.ma[m], b = R.mb[m];
      const double s = sum[a * d + k] + sum[b * d + k];
      sum[a * d + k] = s;
      cen[a * d + k] = s / (double)(R.size[a] + R.size[b]);
    }
    __syncthreads();
    if ((int)threadIdx.x < merged) tail_merge_rec<LINK>(S, R, threadIdx.x, was);
    __syncthreads();
    const int g = tail_group(nterm);
    for (int e0 = 0; e0 < nterm * g; e0 += kTailThreads) {
      const int e = e0 + threadIdx.x;
      const bool in = e < nterm * g;
      const int p = R.term[in ? e / g : 0];
      Near b{INFINITY, 0x7fffffff, -1};
      if (in) {
        const double sz = (double)R.size[p];
        const double vp = LINK == kAvgSq ? mv[p] : 0.0;
        const double *cp = cen + p * d;
        for (int i = e & (g - 1); i < nact; i += g) {
          const int c = R.act[i];
          if (c == p) continue;
          const double *cc = cen + c * d;
          double q = 0.0;
          for (int k = 0; k < d; ++k) {
            const double u = cp[k] - cc[k];
            q += u * u;
          }
          const double x = LINK == kAvgSq ? mv[c] : (double)R.size[c];
          const double key = LINK == kWard ? ((2.0 * sz * x) / (sz + x)) * q : q + (vp + x);
          nearer(b, key, R.cid[c], c);
        }
      }
      tail_near(R, p, b, g, in);
    }
    ++rounds;
    terms += nterm;
    evals += (long long)nterm * (nact - 1);
    __syncthreads();
  }
  if (threadIdx.x == 0) tail_end(cnt, T.err ? 1 : (nact > 1 ? 2 : 0), nact, base, rounds, terms, evals);
}

constexpr int kMaxGridY = 65535;

inline int nblk(long long n, int cap = 4096) {
  const long long b = (n + kBlock - 1) / kBlock;
  return (int)(b < 1 ? 1 : (b < cap ? b : cap));
}

template <int LINK, bool FIRST>
void launch_pass(State &S, Mx &X, int bound, hipStream_t s) {
  // a wavefront per row while that fills the chip, else a block: wider rows
  // then have four times the loads in flight
  if (bound <= 2048) k_mx_pass<LINK, FIRST, kWave><<<(bound + 3) / 4, kBlock, 0, s>>>(X, S.cnt);
  else k_mx_pass<LINK, FIRST, kBlock><<<bound, kBlock, 0, s>>>(X, S.cnt);
}

template <int LINK>
void launch_build(State &S, Mx &X, const float *px, int m, hipStream_t s) {
  const int n = S.n, d = S.d;
  const int nwin = (n + kWin - 1) / kWin;
  const bool pieces = X.unit > 0;
  double *K = pieces ? X.kp : X.k[0];
  const long long ld = mx_ld(pieces ? X.pieces : m);
  const int rw = pieces ? X.unit / kWin : 1;  // row windows per block
  if (LINK == kComplete && m < n) k_mx_zero<<<std::min(m, 1 << 16), kBlock, 0, s>>>(X, m);
  const int gx = (nwin + rw - 1) / rw;
  if (d <= 16) {
    const int cp = pieces ? rw / 2 : 1;  // pairs of column windows per wavefront
    const int units = ((nwin + 1) / 2 + cp - 1) / cp;
    // units per block: enough blocks for small inputs, few stagings for large ones
    int group = units <= 256 ? 4 : std::max(4, 32 / cp);
    while ((units + group - 1) / group > kMaxGridY) group *= 2;
    const dim3 g(gx, (units + group - 1) / group);
    if (d <= 2) k_mx_build_lo<LINK, 2><<<g, kBlock, 0, s>>>(px, X, K, ld, n, d, rw, cp, group);
    else if (d <= 3) k_mx_build_lo<LINK, 3><<<g, kBlock, 0, s>>>(px, X, K, ld, n, d, rw, cp, group);
    else if (d <= 5) k_mx_build_lo<LINK, 5><<<g, kBlock, 0, s>>>(px, X, K, ld, n, d, rw, cp, group);
    else if (d <= 10) k_mx_build_lo<LINK, 10><<<g, kBlock, 0, s>>>(px, X, K, ld, n, d, rw, cp, group);
    else k_mx_build_lo<LINK, 16><<<g, kBlock, 0, s>>>(px, X, K, ld, n, d, rw, cp, group);
  } else {
    int group = std::max(nwin <= 64 ? 1 : 8, rw);
    while ((nwin + group - 1) / group > kMaxGridY) group *= 2;
    k_mx_build_hi<LINK><<<dim3(gx, (nwin + group - 1) / group), kBlock, 0, s>>>(px, X, K, ld, n, d, rw, group);
  }
  const int t = (m + kWin - 1) / kWin;
  if (pieces) {
    k_mx_fold_rows<<<dim3(t, (X.pieces + kBlock - 1) / kBlock), kBlock, 0, s>>>(X, m);
    k_mx_fold<<<dim3(t, t), kBlock, 0, s>>>(X, m);
  } else {
    k_mx_mirror<<<dim3(t, t), kBlock, 0, s>>>(X, m);
    const long long words = m * mx_ld(m) / 16;  // (rows are multiples of 32 bytes)
    if (LINK == kAverage) k_mx_zero_low<<<nblk(words), kBlock, 0, s>>>((uint4 *)X.kl[0], words);
  }
}

// Column parts of a scan: enough blocks to fill the chip while a wavefront
// still has a chunk of 64 columns of its own.
constexpr int kScanParts = 8;

template <int LINK>
void launch_scan(State &S, Mx &X, int bound, bool first, hipStream_t s) {
  const int tiles = (bound + kWave - 1) / kWave;
  tmark(S, 1, false, s);
  if (S.d <= kScanMaxDim) {
    const int chunks = (bound + kWave - 1) / kWave, per = kScanThreads / kWave;
    X.parts = std::max(1, std::min(kScanParts, std::min(chunks / per, 512 / tiles)));
    const dim3 g(tiles, X.parts);
    if (S.d <= 2) k_sc_scan<LINK, 2><<<g, kScanThreads, 0, s>>>(S, X);
    else if (S.d <= 3) k_sc_scan<LINK, 3><<<g, kScanThreads, 0, s>>>(S, X);
    else if (S.d <= 5) k_sc_scan<LINK, 5><<<g, kScanThreads, 0, s>>>(S, X);
    else k_sc_scan<LINK, 8><<<g, kScanThreads, 0, s>>>(S, X);
  } else {
    if (!first) k_sc_merge<LINK><<<std::min(1024, bound / 8 + 1), kBlock,
                                   LINK == kAvgSq ? S.d * sizeof(double) * (kBlock / kWave) : 0, s>>>(S, X);
    X.parts = std::max(1, std::min(kScanParts, std::min(tiles, 2048 / tiles)));
    k_sc_scan_hi<LINK><<<dim3(tiles, X.parts), kBlock, 0, s>>>(S, X);
  }
  tmark(S, 1, true, s);
}

// Records of the active list; direct: of single points, with their centroids.
__global__ void k_sc_enter(State S, Mx X, int merges, int direct) {
  const int n = direct ? S.n : S.cnt->n_act, d = S.d;
  const long long tid = blockIdx.x * (long long)blockDim.x + threadIdx.x, step = (long long)gridDim.x * blockDim.x;
  for (long long i = tid; i < n; i += step) {
    const int s = direct ? (int)i : S.act[i];
    X.c[0].id[i] = direct ? make_int4(s, 1, s, s) : make_int4(S.cid[s], S.csize[s], S.node[s], s);
    X.c[0].eff[i] = direct ? 0.0 : S.eff[s];
    X.term[i] = (int)i;
    if (direct && S.linkage == kAvgSq) {
      S.cvar[s] = 0.0;
      S.cmv[s] = 0.0;
    }
  }
  if (direct)
    for (long long j = tid; j < (long long)n * d; j += step) S.wsum[j] = S.wcen[j] = (double)S.xin[j];
  if (tid == 0) {
    Counters *c = S.cnt;
    c->n_act = n;
    c->mx_merges = merges;
    c->mx_nterm = n;
    c->mx_ran = 1;
    c->mx_terms += n;
    const long long pairs = (long long)n * (n - 1);
    c->cluster_evals += pairs;
    c->refined += pairs;
    c->mx_exact += pairs;
    c->visits[1] += pairs;
  }
}

inline size_t mat_tail_bytes(int stop, bool low) {
  return tail_rec_bytes(stop) + (size_t)stop * (stop - 1) / 2 * (sizeof(double) + (low ? sizeof(Low) : 0));
}
inline size_t cen_tail_bytes(int stop, int d) { return tail_rec_bytes(stop) + (size_t)stop * (2 * d + 2) * sizeof(double); }

}  // namespace

int mx_tail_max(int linkage, int d) {
  if (!centroid_link(linkage)) return kMatTail;
  return std::max(1, std::min(kCenTail, kCenTailNd / d));
}

size_t mx_layout(Mx &X, char *base, int m, int n, int linkage) {
  size_t off = 0;
  // average, clusters: two windows a unit, or as many more as keep the pieces
  // below 1.4 times the clusters (they are few then, and the units still many)
  X.unit = X.pieces = 0;
  if (linkage == kAverage && m < n) {
    long long unit = 2 * kWin;
    while ((n - 1) / unit > m * 2LL / 5 + kWin) unit *= 2;
    X.unit = (int)unit;
    X.pieces = m + (int)((n - 1) / unit);
  }
  auto take = [&](size_t bytes) {
    off = (off + 255) & ~(size_t)255;
    char *p = base ? base + off : nullptr;
    off += bytes;
    return p;
  };
  X.cap = m;
  const size_t ents = (size_t)m * (size_t)mx_ld(m), low = linkage == kAverage ? ents * sizeof(Low) : 0;
  const size_t mat = (ents * sizeof(double) + 255) & ~(size_t)255;
  const size_t pmat = (size_t)X.pieces * (size_t)mx_ld(X.pieces) * sizeof(double);
  for (int i = 0; i < 2; ++i) {
    char *p = take(i == 0 ? mat + low : std::max(mat + low, pmat));
    X.k[i] = (double *)p;
    X.kl[i] = low && base ? (Low *)(p + mat) : nullptr;
  }
  X.kp = X.k[1];  // (dead once the first round writes there)
  for (int i = 0; i < 2; ++i) {
    X.c[i].id = (int4 *)take((size_t)m * sizeof(int4));
    X.c[i].eff = (double *)take((size_t)m * sizeof(double));
    X.c[i].rsize = (double *)take((size_t)m * sizeof(double));
    X.nnv[i] = (double *)take((size_t)m * sizeof(double));
    X.nni[i] = (int *)take((size_t)m * sizeof(int));
  }
  X.src = (int2 *)take((size_t)m * sizeof(int2));
  X.place = (int *)take((size_t)m * sizeof(int));
  X.beg = (int *)take((size_t)m * sizeof(int));
  X.own = (int *)take((size_t)n * sizeof(int));
  return off + 256;
}

void launch_mx_enter(State &S, Mx &X, int m, int merges, bool direct, hipStream_t s) {
  k_mx_enter<<<nblk(m), kBlock, 0, s>>>(S, X, merges, direct ? 1 : 0);
  if (!direct) k_mx_own<<<nblk(S.n), kBlock, 0, s>>>(S, X);
  const float *px = direct ? S.xin : S.px;
  tmark(S, 2, false, s);
  if (S.linkage == kComplete) launch_build<kComplete>(S, X, px, m, s);
  else launch_build<kAverage>(S, X, px, m, s);
  tmark(S, 2, true, s);
  tmark(S, 1, false, s);
  if (S.linkage == kComplete) launch_pass<kComplete, true>(S, X, m, s);
  else launch_pass<kAverage, true>(S, X, m, s);
  tmark(S, 1, true, s);
}

// ------------------------------------------------------------ scan rounds --
size_t sc_layout(Mx &X, char *base, int m) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    off = (off + 255) & ~(size_t)255;
    char *p = base ? base + off : nullptr;
    off += bytes;
    return p;
  };
  X.cap = m;
  for (int i = 0; i < 2; ++i) {
    X.c[i].id = (int4 *)take((size_t)m * sizeof(int4));
    X.c[i].eff = (double *)take((size_t)m * sizeof(double));
    X.nnv[i] = (double *)take((size_t)m * sizeof(double));
    X.nni[i] = (int *)take((size_t)m * sizeof(int));
  }
  X.src = (int2 *)take((size_t)m * sizeof(int2));
  X.place = (int *)take((size_t)m * sizeof(int));
  X.term = (int *)take((size_t)m * sizeof(int));
  X.mpair = (int4 *)take((size_t)(m / 2 + 1) * sizeof(int4));
  X.pv = (double *)take((size_t)kScanParts * m * sizeof(double));
  X.pc = (int2 *)take((size_t)kScanParts * m * sizeof(int2));
  return off + 256;
}

void launch_sc_enter(State &S, Mx &X, int m, int merges, bool direct, hipStream_t s) {
  k_sc_enter<<<nblk(direct ? (long long)m * S.d : m), kBlock, 0, s>>>(S, X, merges, direct ? 1 : 0);
  if (S.linkage == kWard) launch_scan<kWard>(S, X, m, true, s);
  else launch_scan<kAvgSq>(S, X, m, true, s);
}

void launch_mx_round(State &S, Mx &X, int bound, hipStream_t s) {
  const int stop = mx_tail_max(S.linkage, S.d);
  switch (S.linkage) {
  case kComplete: k_mx_book<kComplete><<<1, kBookThreads, 0, s>>>(S, X, stop); break;
  case kAverage: k_mx_book<kAverage><<<1, kBookThreads, 0, s>>>(S, X, stop); break;
  case kWard: k_mx_book<kWard><<<1, kBookThreads, 0, s>>>(S, X, stop); break;
  default: k_mx_book<kAvgSq><<<1, kBookThreads, 0, s>>>(S, X, stop); break;
  }
  if (S.phases) (void)hipEventRecord(S.rev[3], s);
  switch (S.linkage) {
  case kComplete:
    tmark(S, 1, false, s);
    launch_pass<kComplete, false>(S, X, bound, s);
    tmark(S, 1, true, s);
    break;
  case kAverage:
    tmark(S, 1, false, s);
    launch_pass<kAverage, false>(S, X, bound, s);
    tmark(S, 1, true, s);
    break;
  case kWard: launch_scan<kWard>(S, X, bound, false, s); break;
  default: launch_scan<kAvgSq>(S, X, bound, false, s); break;
  }
}

void launch_mx_tail(State &S, Mx &X, hipStream_t s) {
  const int stop = mx_tail_max(S.linkage, S.d);
  tmark(S, 1, false, s);
  switch (S.linkage) {
  case kComplete: k_mx_tail<kComplete><<<1, kTailThreads, mat_tail_bytes(stop, false), s>>>(S, X, stop); break;
  case kAverage: k_mx_tail<kAverage><<<1, kTailThreads, mat_tail_bytes(stop, true), s>>>(S, X, stop); break;
  case kWard: k_sc_tail<kWard><<<1, kTailThreads, cen_tail_bytes(stop, S.d), s>>>(S, X, stop); break;
  default: k_sc_tail<kAvgSq><<<1, kTailThreads, cen_tail_bytes(stop, S.d), s>>>(S, X, stop); break;
  }
  tmark(S, 1, true, s);
}

}  // namespace pc
