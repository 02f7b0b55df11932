// f evaluation at lattice vertices (the edge sign tests of Sec. V-A and the
// subdivision vertices of Sec. V-B need f at every vertex they touch).
//
// Canonical FP64 kernels: the terms of a vertex may be formed in any order
// and place, but are added in index order, so the result is the canonical one
// of ip.h and bit-identical on every device.
//
// FP32 certified kernel: the decision function of a degree-p polynomial
// kernel is a polynomial of degree p in d variables; it is evaluated in FP32
// in its monomial basis (C(d+p, p) coefficients, precomputed on the host in
// FP64 with rigorous error bounds) together with a rigorous bound B32 on
// |f32 - F|, F the exact value at the canonical FP64 coordinates.  With B64 a
// bound on |f64 - F| for the canonical FP64 value, a vertex with
// |f32| > B32 + B64 has sign(f32) = sign(F) = sign(f64); every other vertex
// is re-evaluated by the canonical FP64 kernel, so the sign bits, and the
// traced set, equal the FP64 ones.
#include <algorithm>
#include <mutex>

#include "ip_internal.h"

// Device scratch of ip_feval_noalloc, one copy per device at its own
// address: a 256-byte header holding two counters (the fallback-list length
// and the FP64-monomial settlements), then the fallback list, one 4-byte
// vertex index per vertex of the largest call.  Host code never passes this
// name to a kernel: it passes the address hipGetSymbolAddress returned for
// the current device (noalloc_scratch of the context).
static __device__ __align__(256) unsigned char scratch[256 + 4 * (size_t)IP_NOALLOC_MAX_VERTICES];

namespace {

// The canonical FP64 sum comes in two kernels with the same MODEs:
// MODE 0: vertex-table entries listed by slot (key at keys[slot * 4], result
//         to out[slot * 4]);
// MODE 1: raw int32 vertices, result to out[i];
// MODE 2: raw int32 vertices at the indices in list, result to out[index].
// n_dev (may be NULL): the item count is *n_dev, written by an earlier
// kernel on the stream, at most n (the grid is sized for n).
//
// Both read the support vectors through vector loads: one record per
// wave-uniform scalar load ties a wave to the scalar cache's miss rate
// (about 115 ns per 64-byte record at S = 2000, whatever the unrolling,
// against the 17 ns of its arithmetic).

__device__ __forceinline__ void put_stamp(unsigned long long *stamp) {
  if (stamp && blockIdx.x == 0 && threadIdx.x == 0) *stamp = wall_clock64();
}

// Vertex i of the call: its destination and coordinates.
template <int D, int MODE>
__device__ __forceinline__ uint64_t load_vertex(const LatDev &L, const uint32_t *__restrict__ list, uint64_t i,
                                                const uint64_t *__restrict__ keys,
                                                const int32_t *__restrict__ vraw, double *x) {
  const uint64_t src = MODE == 1 ? i : (uint64_t)list[i];
  int32_t v[D];
  if (MODE == 0) {
    vunpack<D>(L, keys[src * 4], v);
  } else {
#pragma unroll
    for (int j = 0; j < D; ++j) v[j] = vraw[src * D + j];
  }
  lat_coords<D>(L, v, x);
  return src;
}

// Few vertices: a block of eight waves takes 7 V of them.  Seven waves hold
// V vertices each in registers and form their terms one support vector per
// lane (the vectors as columns, read coalesced one tile of 64 ahead); the
// eighth adds the terms of the tile before in index order, one vertex per
// lane, from LDS.  A dependent fma takes 4.4 cycles; what bounds the chain of
// S of them is its operands' way through LDS, 8 cycles per double and wave
// whatever lanes use it, so terms lie in a row per vertex and are read in
// pairs like the weights (alone in a block: 16 cycles a term, 21 with the
// terms of a support vector side by side).  d = 6, S = 2000: 21 us for up
// to 1792 vertices, where one vertex per lane took 314.
template <int D, int P, int MODE, int V>
__global__ __launch_bounds__(512) void feval64_split_kernel(FDev F, LatDev L, const uint32_t *__restrict__ list,
                                                            uint64_t n, const unsigned long long *n_dev,
                                                            const uint64_t *__restrict__ keys,
                                                            const int32_t *__restrict__ vraw,
                                                            double *__restrict__ out, unsigned long long *stamp) {
  put_stamp(stamp);
  constexpr int T = IP_COL_PAD, NW = 7, G = NW * V, TS = T + 2;
  constexpr uint64_t S4 = MODE == 0 ? 4 : 1;
  __shared__ __align__(16) double term[2][G * TS];  // a row per vertex
  __shared__ __align__(16) double alpha[2][T];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (n_dev) n = (uint64_t)*n_dev < n ? (uint64_t)*n_dev : n;
  const int64_t ld = F.ld;
  const int nt = (int)(ld / T);
  for (uint64_t blk = (uint64_t)blockIdx.x * G; blk < n; blk += (uint64_t)gridDim.x * G) {
    // step t of either branch: the terms of tile t are formed while those of
    // tile t - 1 are added; both meet at one barrier per step
    if (wv < NW) {
      const uint64_t v0 = blk + (uint64_t)wv * V;
      double x[V][D];
#pragma unroll
      for (int r = 0; r < V; ++r) load_vertex<D, MODE>(L, list, v0 + r < n ? v0 + r : n - 1, keys, vraw, x[r]);
      // the next tile's records are asked for once this one's are used up, and
      // waited for after the barrier
      double sv[D], al;
      auto fetch = [&](int64_t s) {
#pragma unroll
        for (int j = 0; j < D; ++j) sv[j] = F.col[j * ld + s];
        al = F.col[D * ld + s];
      };
      fetch(lane);
      for (int t = 0; t <= nt; ++t) {
        if (t < nt && v0 < n) {
          if (wv == 0) alpha[t & 1][lane] = al;
          double *tw = &term[t & 1][wv * V * TS + lane];
#pragma unroll
          for (int r = 0; r < V; ++r) tw[r * TS] = sv_term<D, P>(F, sv, x[r]);
          __builtin_amdgcn_sched_barrier(0);
          fetch((t + 1 < nt ? (int64_t)(t + 1) * T : 0) + lane);
        }
        __syncthreads();
      }
    } else {
      double acc = 0.0;
      const int c = lane < G ? lane : 0;
      for (int t = 0; t <= nt; ++t) {
        if (t > 0) {
          const double *tr = term[(t - 1) & 1] + c * TS;
          const double *al = alpha[(t - 1) & 1];
          const int64_t m = F.S - (int64_t)(t - 1) * T;
          if (m >= T) {
            // 16 terms and weights in flight while 16 are added
            constexpr int H = 16;
            double a0[H], b0[H], a1[H], b1[H];
#pragma unroll
            for (int s = 0; s < H; ++s) {
              a0[s] = al[s];
              b0[s] = tr[s];
            }
#pragma unroll
            for (int h = 0; h < T; h += 2 * H) {
#pragma unroll
              for (int s = 0; s < H; ++s) {
                a1[s] = al[h + H + s];
                b1[s] = tr[h + H + s];
              }
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int s = 0; s < H; ++s) acc = fma(a0[s], b0[s], acc);
              if (h + 2 * H < T) {
#pragma unroll
                for (int s = 0; s < H; ++s) {
                  a0[s] = al[h + 2 * H + s];
                  b0[s] = tr[h + 2 * H + s];
                }
              }
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int s = 0; s < H; ++s) acc = fma(a1[s], b1[s], acc);
            }
          } else {
            for (int s = 0; s < (int)m; ++s) acc = fma(al[s], tr[s], acc);
          }
        }
        __syncthreads();
      }
      const uint64_t i = blk + lane;
      if (lane < G && i < n) out[(MODE == 1 ? i : (uint64_t)list[i]) * S4] = acc + F.bias;
    }
  }
}

// Many vertices: R of them per lane, the records shared through LDS
// (tile_sum).  The loop over vertex groups is uniform across the block, so
// every thread reaches the barrier of each tile.
template <int D, int P, int R, int U, int MODE>
__global__ __launch_bounds__(256, (P < 0 || R < 4) ? 4 : 2) void feval64_tile_kernel(
    FDev F, LatDev L, const uint32_t *__restrict__ list, uint64_t n, const unsigned long long *n_dev,
    const uint64_t *__restrict__ keys, const int32_t *__restrict__ vraw, double *__restrict__ out,
    unsigned long long *stamp) {
  put_stamp(stamp);
  constexpr uint64_t S4 = MODE == 0 ? 4 : 1;
  __shared__ __align__(16) double tile[2][kRecTile * 8];
  if (n_dev) n = (uint64_t)*n_dev < n ? (uint64_t)*n_dev : n;
  for (uint64_t blk = (uint64_t)blockIdx.x * 256 * R; blk < n; blk += (uint64_t)gridDim.x * 256 * R) {
    double x[R][D], acc[R];
    uint64_t dst[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint64_t q = blk + r * 256 + threadIdx.x;
      dst[r] = load_vertex<D, MODE>(L, list, q < n ? q : n - 1, keys, vraw, x[r]);
    }
    tile_sum<D, P, R, U>(F, tile, x, acc);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (blk + r * 256 + threadIdx.x < n) out[dst[r] * S4] = acc[r] + F.bias;
  }
}

// Which kernel, by the vertex count n and the support vectors S (times in us,
// d = 6, p = 3, S = 2000 unless given).  Up to 16384 vertices one lane each
// fills less than one wave per CU, and the split form is the faster (4096: 23
// against 90; 16384: 60 against 92), with as few vertices per forming wave as
// still give each CU a block (1000: 21 with one, 24 with four).  It has a cost
// of its own per block, so few support vectors need few vertices (split and
// one lane each, S = 8: 61: 17 and 15; S = 50: 7000: 19 and 17, 16384: 28 and
// 17; S = 200: 7000: 20 and 24, 16384: 28 and 24; S = 1000: 50 and 58).  Above,
// the least number of vertices per lane that still fills the SIMDs once: 65 536
// lanes are one wave on each (65536: 1 per lane 101, 2 per lane 148; 200003: 1,
// 2 and 4 per lane 264, 209, 232; 600000, S = 1000: 309, 244 and 286; 700000:
// 337, 286, 293; 1048576: 1006, 772, 730).  A degree without an instantiation
// of its own (p = 5: the power is a loop) gains from sharing only where waves
// abound, and never with four (S = 1000, 200000: 180, 246; 700000: 413, 493, 525;
// 3000000: 1569, 1494, 1931).  The Gaussian term is 34 operations long and
// needs no sharing (d = 5, S = 300, 1048576 vertices: 351 with one per lane, 438
// with two), nor do very few support vectors (S = 8, 200000: 17 and 17).
constexpr uint64_t kSplitMax = 16384;
inline bool eval_split(uint64_t n, int64_t S) {
  return n <= kSplitMax && S >= (n <= 3584 ? 32 : n <= 7168 ? 96 : 256);
}

// Threads that fill the chip (1024 on each CU).
constexpr uint64_t kFill = 262144;

// One call of the canonical sum: see the MODEs above and launch_feval64.
struct Eval64 {
  hipStream_t st;
  const uint32_t *list;
  uint64_t n;
  const unsigned long long *n_dev;
  const uint64_t *keys;
  const int32_t *vraw;
  double *out;
  uint64_t hint;  // items the launch is shaped for
  unsigned long long *stamp;
  uint64_t spread;  // the grid covers this many, up to what fills the chip (0: hint)
};

template <int D, int P, int MODE>
void launch64(const Eval64 &e, const FDev &F, const LatDev &L) {
  const uint64_t n = e.hint;
  auto grid = [&](uint64_t per, uint64_t fill) {
    const uint64_t more = std::min<uint64_t>((e.spread + per - 1) / per, fill);
    return dim3((unsigned)std::max(more, std::min<uint64_t>((n + per - 1) / per, 65536)));
  };
#define IP_L64(KERNEL, PER, BLOCK)                                                                              \
  hipLaunchKernelGGL(KERNEL, grid(PER, kFill / (BLOCK)), dim3(BLOCK), 0, e.st, F, L, e.list, e.n, e.n_dev, e.keys, \
                     e.vraw, e.out, e.stamp)
  if (eval_split(n, F.S)) {
    if (n <= 1792)
      IP_L64((feval64_split_kernel<D, P, MODE, 1>), 7, 512);
    else if (n <= 3584)
      IP_L64((feval64_split_kernel<D, P, MODE, 2>), 14, 512);
    else
      IP_L64((feval64_split_kernel<D, P, MODE, 4>), 28, 512);
  } else if constexpr (P < 0) {
    IP_L64((feval64_tile_kernel<D, P, 1, 2, MODE>), 256, 256);
  } else if (n <= 98304 || (P == 0 && n <= 786432) || (F.S < 32 && n <= 524288)) {
    IP_L64((feval64_tile_kernel<D, P, 1, 4, MODE>), 256, 256);
  } else if (P == 0 || n <= 655360) {
    IP_L64((feval64_tile_kernel<D, P, 2, 4, MODE>), 512, 256);
  } else if constexpr (P > 0) {
    IP_L64((feval64_tile_kernel<D, P, 4, 4, MODE>), 1024, 256);
  }
#undef IP_L64
}

template <int D, int MODE>
void launch64_p(const Eval64 &e, const FDev &F, const LatDev &L) {
  if (F.kernel == IP_KERNEL_RBF) {
    launch64<D, -1, MODE>(e, F, L);
    return;
  }
  switch (F.p) {
    case 1: launch64<D, 1, MODE>(e, F, L); break;
    case 2: launch64<D, 2, MODE>(e, F, L); break;
    case 3: launch64<D, 3, MODE>(e, F, L); break;
    case 4: launch64<D, 4, MODE>(e, F, L); break;
    default: launch64<D, 0, MODE>(e, F, L); break;
  }
}

template <int MODE>
int dispatch64(ip_ctx *ctx, const FDev &F, const LatDev &L, const uint32_t *list, uint64_t n,
               const uint64_t *keys, const int32_t *vraw, double *out,
               const unsigned long long *n_dev = nullptr, uint64_t hint = 0, unsigned long long *stamp = nullptr,
               uint64_t spread = 0) {
  if (n == 0) return IP_OK;
  const Eval64 e{ctx->stream, list, n, n_dev, keys, vraw, out, hint ? std::min(hint, n) : n, stamp, spread};
  switch (L.d) {
    case 2: launch64_p<2, MODE>(e, F, L); break;
    case 3: launch64_p<3, MODE>(e, F, L); break;
    case 4: launch64_p<4, MODE>(e, F, L); break;
    case 5: launch64_p<5, MODE>(e, F, L); break;
    case 6: launch64_p<6, MODE>(e, F, L); break;
    case 7: launch64_p<7, MODE>(e, F, L); break;
    default: return ip_fail(ctx, IP_EINVAL, "dimension out of range");
  }
  IP_TRY_HIP(ctx, hipGetLastError());
  return IP_OK;
}

// ---------------------------------------------------------------------------
// FP32 monomial-basis evaluation with certification
// ---------------------------------------------------------------------------
// Tiered certification.  Tier 1: f in FP32 in the monomial basis; settled
// when |f32| > B32 + B64.  Tier 2 (only for the rest): f in FP64 in the
// monomial basis; settled when |f64m| > B64m + B64.  Tier 3: the canonical
// FP64 sum over the support vectors, for what is left.
// MODE 0: vertex-table slots (f to vt[slot].f, bound to vb[slot]);
// MODE 1: raw vertices (f to out[i], bound to bout[i]).
// Tier-3 vertices get vb = -1 (resp. bout = 0) and are appended to fb (slot,
// resp. index) for the canonical FP64 kernel.
template <int D, int P, int MODE>
__global__ __launch_bounds__(256) void feval32_kernel(PolyDev Q, LatDev L, const uint32_t *__restrict__ list,
                                                      uint64_t n, const unsigned long long *n_dev, VEnt *vt,
                                                      float *vb, const int32_t *__restrict__ vraw, double *out,
                                                      double *bout, uint32_t *fb, unsigned long long *fb_ctr,
                                                      unsigned long long *c64_ctr, unsigned long long *stamp) {
  if constexpr (MODE == 0) {
    put_stamp(stamp);
    if (n_dev) n = (uint64_t)*n_dev < n ? (uint64_t)*n_dev : n;
  }
  constexpr int kStage = 128;
  __shared__ uint32_t st[4][kStage];
  const int wib = threadIdx.x >> 6;
  int sn = 0;
  auto put = [&](unsigned long long pos, uint32_t s) { fb[pos] = s; };
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t start = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t rounds = (n + stride - 1) / stride;
  unsigned long long n64 = 0;
  for (uint64_t it = 0; it < rounds; ++it) {
    const uint64_t i = start + it * stride;
    bool unsure = false;
    uint32_t id = 0;
    if (i < n) {
      int32_t v[D];
      if (MODE == 0) {
        id = list[i];
        vunpack<D>(L, vt[id].key, v);
      } else {
        id = (uint32_t)i;
#pragma unroll
        for (int j = 0; j < D; ++j) v[j] = vraw[i * D + j];
      }
      double x64[D];
      lat_coords<D>(L, v, x64);
      double fv, bnd;
      const int tier = cert_eval<D, P>(Q, x64, &fv, &bnd);
      unsure = tier == 3;
      if (tier == 2) ++n64;
      if (MODE == 0) {
        if (!unsure) vt[id].f = fv;
        vb[id] = unsure ? -1.0f : (float)(bnd * (1.0 + 1e-6));
      } else {
        out[i] = fv;
        if (bout) bout[i] = unsure ? 0.0 : bnd + Q.B64;
      }
    }
    stage_put<kStage>(st[wib], sn, unsure, id, put, fb_ctr);
  }
  stage_flush(st[wib], sn, put, fb_ctr);
  if (n64) atomicAdd(c64_ctr, n64);
}

// FP32 certified RBF evaluation (same MODEs and outputs as feval32_kernel).
// With u = 2^-24, at the canonical FP64 coordinates x (rounded to FP32):
// per support vector d2 = the FP32 fma chain of (x_j - s_j)^2, e = the own
// FP32 exponential of -(gamma d2), term = alpha e; the terms are summed in
// blocks of 32 and the block sums added, A = sum |term| and W = sum |term| d2
// beside them.  The bound on |f32 - F| (F the exact value at x):
//   43 u A'  (exponential 40 u, alpha and product 2 u, sum of A 1 u)
// + gamma u ((d + 4) W' + 9 (|x|^2 + max |s|^2) A')  (the rounding of d2
//   and of gamma d2 moves the exponent: |dt| <= gamma u ((d + 3) d2 +
//   8.1 (|x|^2 + |s|^2)) per term, and |d exp| <= exp |dt| (1 + |dt|))
// + (32 + S / 32 + 3) u A'  (two-level summation)
// + u (|bias| + |f32|) + 2e-38 S max|alpha|  (final add; exponential underflow)
// with A' = A (1 + (S + 60) u), W' likewise (the FP32 sums of positive terms
// and the relative errors of their terms), all times 1.01 for the products
// of the first-order terms.  Tier 1 settles the sign when |f32| exceeds the
// bound plus B64; the rest go to the canonical FP64 kernel.
constexpr int kRbf32Tile = 512;

template <int D, int MODE>
__global__ __launch_bounds__(256) void rbf32_kernel(RbfDev Q, LatDev L,
                                                    const uint32_t *__restrict__ list, uint64_t n, VEnt *vt,
                                                    float *vb, const int32_t *__restrict__ vraw, double *out,
                                                    double *bout, uint32_t *fb, unsigned long long *fb_ctr) {
  __shared__ float tile[kRbf32Tile * 8];
  constexpr int kStage = 128;
  __shared__ uint32_t st[4][kStage];
  const int wib = threadIdx.x >> 6;
  int sn = 0;
  auto put = [&](unsigned long long pos, uint32_t s) { fb[pos] = s; };
  const double u = 5.9604644775390625e-08;
  for (uint64_t blk = (uint64_t)blockIdx.x * blockDim.x; blk < n; blk += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t i = blk + threadIdx.x;
    const bool valid = i < n;
    const uint64_t ii = valid ? i : n - 1;
    uint32_t id = 0;
    int32_t v[D];
    if (MODE == 0) {
      id = list[ii];
      vunpack<D>(L, vt[id].key, v);
    } else {
      id = (uint32_t)ii;
#pragma unroll
      for (int j = 0; j < D; ++j) v[j] = vraw[ii * D + j];
    }
    double x64[D];
    lat_coords<D>(L, v, x64);
    float x[D];
    float X2 = 0.0f;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      x[j] = (float)x64[j];
      X2 = fmaf(x[j], x[j], X2);
    }
    float acc = 0.0f, blk_acc = 0.0f, A = 0.0f, W = 0.0f;
    int in_blk = 0;
    for (int64_t t0 = 0; t0 < Q.S; t0 += kRbf32Tile) {
      const int nt = (int)(Q.S - t0 < kRbf32Tile ? Q.S - t0 : kRbf32Tile);
      __syncthreads();
      for (int q = threadIdx.x; q < nt * 8; q += blockDim.x) tile[q] = Q.rec[t0 * 8 + q];
      __syncthreads();
      for (int s = 0; s < nt; ++s) {
        const float *sv = tile + s * 8;
        float d2 = 0.0f;
#pragma unroll
        for (int j = 0; j < D; ++j) {
          const float df = x[j] - sv[j];
          d2 = fmaf(df, df, d2);
        }
        const float term = sv[D] * exp32_own(-(Q.gamma * d2));
        blk_acc += term;
        A += fabsf(term);
        W = fmaf(fabsf(term), d2, W);
        if (++in_blk == 32) {
          acc += blk_acc;
          blk_acc = 0.0f;
          in_blk = 0;
        }
      }
    }
    acc += blk_acc;
    const float f32 = acc + Q.bias;
    const double S = (double)Q.S;
    const double grow = 1.0 + (S + 60.0) * u;
    const double Ap = (double)A * grow, Wp = (double)W * grow;
    const double X2p = (double)X2 * (1.0 + (D + 2) * u) + 1e-30;
    const double bnd = 1.01 * (43.0 * u * Ap + (double)Q.gamma * u * ((D + 4) * Wp + 9.0 * (X2p + (double)Q.nrm_max) * Ap) +
                               (35.0 + S / 32.0) * u * Ap + u * (fabs((double)Q.bias) + fabs((double)f32))) +
                       2e-38 * S * Q.amax;
    const double B64 = Q.B64;
    const bool unsure = !(fabs((double)f32) > bnd + B64);
    if (valid) {
      if (MODE == 0) {
        if (!unsure) vt[id].f = (double)f32;
        vb[id] = unsure ? -1.0f : (float)(bnd * (1.0 + 1e-6));
      } else {
        out[i] = (double)f32;
        if (bout) bout[i] = unsure ? 0.0 : bnd + B64;
      }
    }
    stage_put<kStage>(st[wib], sn, valid && unsure, id, put, fb_ctr);
  }
  stage_flush(st[wib], sn, put, fb_ctr);
}

__global__ void set_vb_kernel(const uint32_t *list, uint64_t n, float *vb, float v) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    vb[list[i]] = v;
}

template <int D, int MODE>
void launch32_p(hipStream_t st, const PolyDev &Q, const LatDev &L, const uint32_t *list, uint64_t n,
                const unsigned long long *n_dev, uint64_t hint, VEnt *vt, float *vb, const int32_t *vraw, double *out,
                double *bout, uint32_t *fb, unsigned long long *fb_ctr, unsigned long long *c64,
                unsigned long long *stamp) {
  uint64_t blocks = (hint + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) return;
#define IP_L32(PP)                                                                                               \
  hipLaunchKernelGGL((feval32_kernel<D, PP, MODE>), dim3((unsigned)blocks), dim3(256), 0, st, Q, L, list, n, n_dev,    \
                     vt, vb, vraw, out, bout, fb, fb_ctr, c64, stamp)
  switch (Q.p) {
    case 1: IP_L32(1); break;
    case 2: IP_L32(2); break;
    case 3: IP_L32(3); break;
    case 4: IP_L32(4); break;
    default: break;
  }
#undef IP_L32
}

template <int MODE>
int dispatch32(ip_ctx *ctx, const PolyDev &Q, const LatDev &L, const uint32_t *list, uint64_t n, VEnt *vt, float *vb,
               const int32_t *vraw, double *out, double *bout, uint32_t *fb, unsigned long long *fb_ctr,
               unsigned long long *c64, const unsigned long long *n_dev, uint64_t hint, unsigned long long *stamp) {
  if (!c64) c64 = &ctx->ctr_dev->n_cert64;
  if (n == 0) return IP_OK;
  hint = hint ? std::min(hint, n) : n;
  hipStream_t st = ctx->stream;
  switch (L.d) {
    case 2: launch32_p<2, MODE>(st, Q, L, list, n, n_dev, hint, vt, vb, vraw, out, bout, fb, fb_ctr, c64, stamp); break;
    case 3: launch32_p<3, MODE>(st, Q, L, list, n, n_dev, hint, vt, vb, vraw, out, bout, fb, fb_ctr, c64, stamp); break;
    case 4: launch32_p<4, MODE>(st, Q, L, list, n, n_dev, hint, vt, vb, vraw, out, bout, fb, fb_ctr, c64, stamp); break;
    case 5: launch32_p<5, MODE>(st, Q, L, list, n, n_dev, hint, vt, vb, vraw, out, bout, fb, fb_ctr, c64, stamp); break;
    case 6: launch32_p<6, MODE>(st, Q, L, list, n, n_dev, hint, vt, vb, vraw, out, bout, fb, fb_ctr, c64, stamp); break;
    case 7: launch32_p<7, MODE>(st, Q, L, list, n, n_dev, hint, vt, vb, vraw, out, bout, fb, fb_ctr, c64, stamp); break;
    default: return ip_fail(ctx, IP_EINVAL, "dimension out of range");
  }
  IP_TRY_HIP(ctx, hipGetLastError());
  return IP_OK;
}

__global__ void zero_u64_kernel(unsigned long long *p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

__global__ void fill_f64_kernel(double *p, uint64_t n, double v) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {nullptr};

template <int MODE>
int dispatch32_rbf(ip_ctx *ctx, const RbfDev &Q, const LatDev &L, const uint32_t *list, uint64_t n, VEnt *vt,
                   float *vb, const int32_t *vraw, double *out, double *bout, uint32_t *fb,
                   unsigned long long *fb_ctr) {
  if (n == 0) return IP_OK;
  const uint64_t blocks = std::min<uint64_t>((n + 255) / 256, 16384);
  hipStream_t st = ctx->stream;
#define IP_R32(DD)                                                                                              \
  hipLaunchKernelGGL((rbf32_kernel<DD, MODE>), dim3((unsigned)blocks), dim3(256), 0, st, Q, L, list, n, vt, vb, \
                     vraw, out, bout, fb, fb_ctr)
  switch (L.d) {
    case 2: IP_R32(2); break;
    case 3: IP_R32(3); break;
    case 4: IP_R32(4); break;
    case 5: IP_R32(5); break;
    case 6: IP_R32(6); break;
    case 7: IP_R32(7); break;
    default: return ip_fail(ctx, IP_EINVAL, "dimension out of range");
  }
#undef IP_R32
  IP_TRY_HIP(ctx, hipGetLastError());
  return IP_OK;
}

// The certified FP32 tier of problem p (polynomial or RBF form).
template <int MODE>
int dispatch32_p(ip_ctx *ctx, const ip_problem *p, const LatDev &L, const uint32_t *list, uint64_t n, VEnt *vt,
                 float *vb, const int32_t *vraw, double *out, double *bout, uint32_t *fb,
                 unsigned long long *fb_ctr, unsigned long long *c64 = nullptr,
                 const unsigned long long *n_dev = nullptr, uint64_t hint = 0, unsigned long long *stamp = nullptr) {
  if (p->f.kernel == IP_KERNEL_RBF)
    return dispatch32_rbf<MODE>(ctx, p->rbf, L, list, n, vt, vb, vraw, out, bout, fb, fb_ctr);
  return dispatch32<MODE>(ctx, p->poly, L, list, n, vt, vb, vraw, out, bout, fb, fb_ctr, c64, n_dev, hint, stamp);
}

// One support vector's factors for f and its gradient at x (the order of
// ip.h's ip_seed_search): f = fma(alpha, e, f), g_j = fma(w, s_j, g_j)
// (RBF: fma(w, x_j - s_j, g_j)); pg is p gamma (RBF: -2 gamma).
template <int D, bool RBF>
__device__ __forceinline__ void grad_factors(const FDev &F, const double *sv, const double *x, double pg, double *e,
                                             double *w) {
  if (RBF) {
    *e = sv_term<D, -1>(F, sv, x);
    *w = (sv[D] * *e) * pg;
    return;
  }
  double dot = 0.0;
#pragma unroll
  for (int j = 0; j < D; ++j) dot = fma(sv[j], x[j], dot);
  const double t = fma(F.gamma, dot, F.coef0);
  double tp1 = 1.0;
  if (F.p > 1) {
    tp1 = t;
    for (int r = 2; r < F.p; ++r) tp1 = tp1 * t;
  }
  *e = tp1 * t;
  *w = (sv[D] * tp1) * pg;
}

// Seed search (Sec. V-A: minimise |f| from given configurations), one lane
// per start: `iters` minimum-norm Newton steps, each clamped into the box;
// a zero gradient ends a lane's steps.  Then f at the final point.  The
// records pass through LDS in tiles, as in feval64_tile_kernel (the loops
// are uniform across the block; a lane whose steps have ended keeps its x).
template <int D, bool RBF>
__global__ __launch_bounds__(256) void seed_kernel(FDev F, LatDev L, const double *__restrict__ q0, uint64_t n,
                                                   int iters, double *__restrict__ q, double *__restrict__ fq) {
  constexpr int T = 64, U = RBF ? 2 : 4;
  __shared__ __align__(16) double tile[2][T * 8];
  const double pg = RBF ? -2.0 * F.gamma : (double)F.p * F.gamma;
  const int64_t nd = F.S * 8, nt = (F.S + T - 1) / T;
  for (uint64_t blk = (uint64_t)blockIdx.x * 256; blk < n; blk += (uint64_t)gridDim.x * 256) {
    const uint64_t i = blk + threadIdx.x < n ? blk + threadIdx.x : n - 1;
    double x[D], g[D], f = 0.0;
    bool done = false;
#pragma unroll
    for (int j = 0; j < D; ++j) x[j] = q0[i * D + j];
    for (int it = 0; it <= iters; ++it) {
      f = 0.0;
#pragma unroll
      for (int j = 0; j < D; ++j) g[j] = 0.0;
      double2 nx;
      auto fetch = [&](int64_t t) {
        const int64_t o = t * T * 8 + threadIdx.x * 2;
        nx = o < nd ? *(const double2 *)(F.rec + o) : make_double2(0.0, 0.0);
      };
      auto add = [&](const double *sv, double e, double w) {
        f = fma(sv[D], e, f);
#pragma unroll
        for (int j = 0; j < D; ++j) g[j] = fma(w, RBF ? x[j] - sv[j] : sv[j], g[j]);
      };
      fetch(0);
      __syncthreads();
      for (int64_t t = 0; t < nt; ++t) {
        *(double2 *)&tile[t & 1][threadIdx.x * 2] = nx;
        __syncthreads();
        if (t + 1 < nt) fetch(t + 1);
        const double *tl = tile[t & 1];
        const int m = (int)(F.S - t * T < T ? F.S - t * T : T);
        int s = 0;
        for (; s + U <= m; s += U) {
          double sv[U][8], e[U], w[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int j = 0; j < (D + 2) / 2; ++j) {
              const double2 z = *(const double2 *)&tl[(s + u) * 8 + 2 * j];
              sv[u][2 * j] = z.x;
              sv[u][2 * j + 1] = z.y;
            }
            grad_factors<D, RBF>(F, sv[u], x, pg, &e[u], &w[u]);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) add(sv[u], e[u], w[u]);
        }
        for (; s < m; ++s) {
          double e, w;
          grad_factors<D, RBF>(F, tl + s * 8, x, pg, &e, &w);
          add(tl + s * 8, e, w);
        }
      }
      f = f + F.bias;
      double n2 = 0.0;
#pragma unroll
      for (int j = 0; j < D; ++j) n2 = fma(g[j], g[j], n2);
      done = done || !(n2 > 0.0);
      if (it == iters || done) continue;
      const double c = f / n2;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const double v = fma(-c, g[j], x[j]);
        x[j] = v < L.lo[j] ? L.lo[j] : (v > L.hi[j] ? L.hi[j] : v);
      }
    }
    if (blk + threadIdx.x < n) {
#pragma unroll
      for (int j = 0; j < D; ++j) q[i * D + j] = x[j];
      fq[i] = f;
    }
  }
}

// The part of FDev that f_grad needs.
struct FRec {
  const double *rec;
  int64_t S;
  int32_t p, kernel;
  double gamma, coef0, bias;
};

// Canonical f and gradient at x (the order of ip.h's ip_seed_search): per
// support vector in index order, read as a wave-uniform record.
template <int D>
__device__ __forceinline__ double f_grad(const FRec &F, const double *x, double *g) {
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < D; ++j) g[j] = 0.0;
  if (F.kernel == IP_KERNEL_RBF) {
    const double m2g = -2.0 * F.gamma;
    for (int64_t i = 0; i < F.S; ++i) {
      const double *rec = F.rec + i * 8;
      double df[D], d2 = 0.0;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        df[j] = x[j] - rec[j];
        d2 = fma(df[j], df[j], d2);
      }
      const double e = exp_own(-(F.gamma * d2));
      acc = fma(rec[D], e, acc);
      const double w = (rec[D] * e) * m2g;
#pragma unroll
      for (int j = 0; j < D; ++j) g[j] = fma(w, df[j], g[j]);
    }
    return acc + F.bias;
  }
  const double pg = (double)F.p * F.gamma;
  for (int64_t i = 0; i < F.S; ++i) {
    const double *rec = F.rec + i * 8;
    double dot = 0.0;
#pragma unroll
    for (int j = 0; j < D; ++j) dot = fma(rec[j], x[j], dot);
    const double t = fma(F.gamma, dot, F.coef0);
    double tp1 = 1.0;
    if (F.p > 1) {
      tp1 = t;
      for (int r = 2; r < F.p; ++r) tp1 = tp1 * t;
    }
    acc = fma(rec[D], tp1 * t, acc);
    const double w = (rec[D] * tp1) * pg;
#pragma unroll
    for (int j = 0; j < D; ++j) g[j] = fma(w, rec[j], g[j]);
  }
  return acc + F.bias;
}

// Most starts whose records go through LDS; above, one lane per start reads
// them by scalar loads.  These hit while the records (64 bytes each) fit the
// scalar cache (16 KiB); else each is a miss, which three waves on a SIMD hide
// (65 536 starts are one).  Scalar and LDS in us, 10 steps: d = 6, S = 100:
// 65 536 starts 131 and 128, 131 072: 157 and 166, 196 608: 194 and 223; d = 6,
// S = 300: 131 072: 449 and 465, 180 000: 540 and 593; d = 4, S = 300: 131 072:
// 451 and 384, 196 608: 506 and 469; d = 5, S = 500: 131 072: 907 and 689, 180 000:
// 960 and 919, 196 608: 831 and 884, 262 144: 1042 and 1087; Gaussian, d = 4, S =
// 100: 65 536: 201 and 188, 131 072: 279 and 294, 196 608: 376 and 395; d = 6, S =
// 300: 150 000: 1273 and 1169, 262 144: 1569 and 1672.  Of very few records
// the way through their tile costs what it saves (S = 24, d = 6: 65 536: 45 and
// 47; S = 8: 13 000: 23 and 24).
int64_t seed_lds_max(int64_t S, bool rbf) {
  if (S < 32) return 0;
  if (S <= 256) return 65536;
  return S <= 384 && !rbf ? 131072 : 184320;
}

template <int D>
__global__ __launch_bounds__(256) void seed_scalar_kernel(FRec F, LatDev L, const double *__restrict__ q0, uint64_t n,
                                                          int iters, double *__restrict__ q,
                                                          double *__restrict__ fq) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    double x[D], g[D];
#pragma unroll
    for (int j = 0; j < D; ++j) x[j] = q0[i * D + j];
    for (int it = 0; it < iters; ++it) {
      const double fv = f_grad<D>(F, x, g);
      double n2 = 0.0;
#pragma unroll
      for (int j = 0; j < D; ++j) n2 = fma(g[j], g[j], n2);
      if (!(n2 > 0.0)) break;
      const double c = fv / n2;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const double v = fma(-c, g[j], x[j]);
        x[j] = v < L.lo[j] ? L.lo[j] : (v > L.hi[j] ? L.hi[j] : v);
      }
    }
    const double fv = f_grad<D>(F, x, g);
#pragma unroll
    for (int j = 0; j < D; ++j) q[i * D + j] = x[j];
    fq[i] = fv;
  }
}

// The same search with the sums of a step formed side by side, for few starts:
// a block takes 16 starts.  Waves 2 to 7 form, per support vector and start,
// the two factors that the sums share (t^p or the exponential, and the
// gradient weight), one tile of 48 vectors ahead; waves 0 and 1 add them, one
// lane per (sum, start), f and the d gradient components side by side, each
// in index order.  Serial per step: S dependent fma instead of S times the
// whole term; both operands of each come through LDS, which bounds it, as rows
// read in pairs (d = 6, S = 2000, 20 steps, 3001 starts: 7.06 ms with one lane
// per start, 0.76 with single reads, 0.67 now).
constexpr int kSeedG = 16, kSeedT = 48;
// One lane per start takes the same time up to 65 536 starts (a wave per
// SIMD); the split form takes a step more with every 4096 (a block per CU)
// and has a cost per step of its own, so it needs the more vectors the more
// starts there are.  Split and one lane each in us, 10 steps, d = 3: S = 8:
// 4096 starts 27 and 23; S = 24: 34 and 38, 8192: 55 and 38; S = 50: 8192: 50
// and 61, 12 288: 68 and 61; S = 100: 12 288: 92 and 105; Gaussian S = 24: 4096: 38
// and 53, 8192: 62 and 53; S = 50: 12 288: 83 and 90.  d = 5, S = 500: 12 000: 292
// and 527, 16 000: 367 and 527.
constexpr int64_t kSeedSplitMax = 12288;

bool seed_split(int64_t n, int64_t S, bool rbf) {
  if (n > kSeedSplitMax) return false;
  const int step = (int)((n + 4095) / 4096) - 1;  // 0, 1, 2
  return S >= ((rbf ? 16 : 24) << step);
}

template <int D, bool RBF>
__global__ __launch_bounds__(512) void seed_split_kernel(FDev F, LatDev L, const double *__restrict__ q0, uint64_t n,
                                                         int iters, double *__restrict__ q, double *__restrict__ fq) {
  constexpr int G = kSeedG, T = kSeedT, NR = T / 24;  // 24 vectors per round of the six forming waves
  constexpr int TS = T + 2;                           // a row per start or component, read in pairs
  __shared__ __align__(16) double val[2][2][G * TS];  // [buffer][sum factor, gradient weight]
  __shared__ __align__(16) double recs[2][(D + 1) * TS];
  __shared__ double xs[G * 8], res[8 * G];
  __shared__ int done[G];
  const int tid = threadIdx.x, g = tid & (G - 1);
  const bool adds = tid < 128;
  const int c = tid >> 4;                    // adding waves: the sum, 0 for f, 1 + j for component j
  const int sr = (tid - 128) >> 4;           // forming waves: vector within a round
  const int nt = (int)((F.S + T - 1) / T);
  const double pg = RBF ? -2.0 * F.gamma : (double)F.p * F.gamma;
  for (uint64_t blk = (uint64_t)blockIdx.x * G; blk < n; blk += (uint64_t)gridDim.x * G) {
    const uint64_t i = blk + g < n ? blk + g : n - 1;
    if (tid < G) {
#pragma unroll
      for (int j = 0; j < D; ++j) xs[g * 8 + j] = q0[i * D + j];
      done[g] = 0;
    }
    __syncthreads();
    for (int it = 0;; ++it) {
      double acc = 0.0;
      if (adds) {
        const int cc = c <= D ? c : 0;       // lanes past the last sum repeat f
        const double xc = cc ? xs[g * 8 + cc - 1] : 0.0;
        const int col = cc ? cc - 1 : D;
        for (int t = 0; t <= nt; ++t) {
          if (t > 0) {
            const double *v = &val[(t - 1) & 1][cc ? 1 : 0][g * TS];
            const double *r = &recs[(t - 1) & 1][col * TS];
            const int m = (int)(F.S - (int64_t)(t - 1) * T < T ? F.S - (int64_t)(t - 1) * T : T);
            int s = 0;
            if (m == T) {
              // H factors in flight while H are added
              constexpr int H = 12;
              double a0[H], b0[H], a1[H], b1[H];
              auto get = [&](double *a, double *b, int s0) {
#pragma unroll
                for (int u = 0; u < H; ++u) {
                  a[u] = v[s0 + u];
                  b[u] = r[s0 + u];
                }
              };
              auto add = [&](const double *a, const double *b) {
#pragma unroll
                for (int u = 0; u < H; ++u) acc = fma(a[u], RBF && cc ? xc - b[u] : b[u], acc);
              };
              get(a0, b0, 0);
#pragma unroll
              for (; s < T; s += 2 * H) {
                get(a1, b1, s + H);
                __builtin_amdgcn_sched_barrier(0);
                add(a0, b0);
                if (s + 2 * H < T) get(a0, b0, s + 2 * H);
                __builtin_amdgcn_sched_barrier(0);
                add(a1, b1);
              }
            }
            for (; s < m; ++s) acc = fma(v[s], RBF && cc ? xc - r[s] : r[s], acc);
          }
          __syncthreads();
        }
        if (c <= D) res[c * G + g] = c == 0 ? acc + F.bias : acc;
      } else {
        double x[D];
#pragma unroll
        for (int j = 0; j < D; ++j) x[j] = xs[g * 8 + j];
        double sv[NR][D + 1];
        // asked for once the tile before is used up, waited for after the barrier
        auto fetch = [&](int t) {
#pragma unroll
          for (int k = 0; k < NR; ++k) {
            const int64_t s = (int64_t)t * T + k * 24 + sr;
            const double *rec = F.rec + (s < F.S ? s : F.S - 1) * 8;
#pragma unroll
            for (int j = 0; j <= D; ++j) sv[k][j] = rec[j];
          }
        };
        fetch(0);
        for (int t = 0; t <= nt; ++t) {
          if (t < nt) {
#pragma unroll
            for (int k = 0; k < NR; ++k) {
              const int s = k * 24 + sr;
              double e, w;
              grad_factors<D, RBF>(F, sv[k], x, pg, &e, &w);
              val[t & 1][0][g * TS + s] = e;
              val[t & 1][1][g * TS + s] = w;
              if (g == 0) {
#pragma unroll
                for (int j = 0; j <= D; ++j) recs[t & 1][j * TS + s] = sv[k][j];
              }
            }
            __builtin_amdgcn_sched_barrier(0);
            fetch(t + 1 < nt ? t + 1 : 0);
          }
          __syncthreads();
        }
      }
      __syncthreads();
      if (it == iters) break;
      if (tid < G && !done[g]) {
        double gr[D], n2 = 0.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
          gr[j] = res[(1 + j) * G + g];
          n2 = fma(gr[j], gr[j], n2);
        }
        if (!(n2 > 0.0)) {
          done[g] = 1;
        } else {
          const double cf = res[g] / n2;
#pragma unroll
          for (int j = 0; j < D; ++j) {
            const double v = fma(-cf, gr[j], xs[g * 8 + j]);
            xs[g * 8 + j] = v < L.lo[j] ? L.lo[j] : (v > L.hi[j] ? L.hi[j] : v);
          }
        }
      }
      __syncthreads();
    }
    if (tid < G && blk + g < n) {
#pragma unroll
      for (int j = 0; j < D; ++j) q[i * D + j] = xs[g * 8 + j];
      fq[i] = res[g];
    }
    __syncthreads();
  }
}

}  // namespace

int ip_seed_search_impl(ip_ctx *ctx, const ip_problem *p, const double *q0, int64_t n, int32_t iters, double *q,
                        double *fq) {
  const bool rbf = p->f.kernel == IP_KERNEL_RBF;
  const bool split = seed_split(n, p->f.S, rbf), lds = n <= seed_lds_max(p->f.S, rbf);
  const unsigned blocks = (unsigned)std::min<int64_t>(split ? (n + kSeedG - 1) / kSeedG : (n + 255) / 256, 16384);
  const FRec fr{p->f.rec, p->f.S, p->f.p, p->f.kernel, p->f.gamma, p->f.coef0, p->f.bias};
#define IP_SDF(KERNEL, THREADS, F) \
  hipLaunchKernelGGL(KERNEL, dim3(blocks), dim3(THREADS), 0, ctx->stream, F, p->fine, q0, (uint64_t)n, (int)iters, q, fq)
#define IP_SDK(KERNEL, THREADS) IP_SDF(KERNEL, THREADS, p->f)
#define IP_SD(DD)                                \
  if (split && rbf)                              \
    IP_SDK((seed_split_kernel<DD, true>), 512);  \
  else if (split)                                \
    IP_SDK((seed_split_kernel<DD, false>), 512); \
  else if (!lds)                                 \
    IP_SDF((seed_scalar_kernel<DD>), 256, fr);   \
  else if (rbf)                                  \
    IP_SDK((seed_kernel<DD, true>), 256);        \
  else                                           \
    IP_SDK((seed_kernel<DD, false>), 256)
  switch (p->d) {
    case 2: IP_SD(2); break;
    case 3: IP_SD(3); break;
    case 4: IP_SD(4); break;
    case 5: IP_SD(5); break;
    case 6: IP_SD(6); break;
    case 7: IP_SD(7); break;
    default: return ip_fail(ctx, IP_EINVAL, "dimension out of range");
  }
#undef IP_SD
#undef IP_SDK
#undef IP_SDF
  IP_TRY_HIP(ctx, hipGetLastError());
  return IP_OK;
}

bool ip_has_fp32_form(const ip_problem *p) {
  return p->f.kernel == IP_KERNEL_RBF ? p->rbf.ok != 0 : p->poly.ok != 0;
}

int ip_noalloc_setup(ip_ctx *ctx) {
  if (ctx->device < 0 || ctx->device >= 64) return ip_fail(ctx, IP_EINVAL, "device index out of range");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[ctx->device]) {
    // the device is current (ip_create set it): its own copy of the array
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) return ip_hip(ctx, e == hipSuccess ? hipErrorInvalidSymbol : e, "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[ctx->device] = ptr;
  }
  ctx->noalloc_scratch = g_scratch_ptr[ctx->device];
  return IP_OK;
}

// Same kernels and launch shapes as ip_feval_impl, with the fallback list and
// its counters in the device scratch and the FP64 pass sized on the device
// (it reads the list length the FP32 pass left), so nothing is allocated and
// nothing waits for the host.
int ip_feval_noalloc_impl(ip_ctx *ctx, const ip_problem *p, const int32_t *v_dev, int64_t n, int32_t prec,
                          double *f_dev, double *bound_dev) {
  if (!ctx->noalloc_scratch) return ip_fail(ctx, IP_EDEVICE, "device scratch not set up");
  hipStream_t st = ctx->stream;
  if (prec == IP_FP64 || !ip_has_fp32_form(p)) {
    if (bound_dev) {
      const uint64_t blocks = std::min<uint64_t>(((uint64_t)n + 255) / 256, 4096);
      hipLaunchKernelGGL(fill_f64_kernel, dim3((unsigned)blocks), dim3(256), 0, st, bound_dev, (uint64_t)n, 0.0);
      IP_TRY_HIP(ctx, hipGetLastError());
    }
    return dispatch64<1>(ctx, p->f, p->fine, nullptr, (uint64_t)n, nullptr, v_dev, f_dev);
  }
  unsigned long long *hdr = (unsigned long long *)ctx->noalloc_scratch;
  uint32_t *fbl = (uint32_t *)((unsigned char *)ctx->noalloc_scratch + 256);
  hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, st, hdr, 2);
  IP_TRY_HIP(ctx, hipGetLastError());
  IP_TRY(dispatch32_p<1>(ctx, p, p->fine, nullptr, (uint64_t)n, nullptr, nullptr, v_dev, f_dev, bound_dev, fbl,
                         hdr, hdr + 1));
  // None or all of the vertices may be left over, and the launch cannot know.
  // Up to 65 536 the form for an eighth of them: a few take 21 us at S = 2000
  // instead of the 90 of a lane each, all of 60 000 take 207.  Above, a lane
  // each or more (all of 140 000: 252).  The grid is for all of them, up to
  // what fills the chip: with the grid for an eighth, all of 140 000 took
  // 748.
  const uint64_t eighth = ((uint64_t)n + 7) / 8;
  const uint64_t hint = (uint64_t)n <= 65536 ? eighth : std::max<uint64_t>(eighth, 65536);
  return dispatch64<2>(ctx, p->f, p->fine, fbl, (uint64_t)n, nullptr, v_dev, f_dev, hdr, hint, nullptr, (uint64_t)n);
}

int launch_feval64(ip_ctx *ctx, const ip_problem *p, const LatDev &L, const uint32_t *list, uint64_t n, VEnt *vt,
                   const unsigned long long *n_dev, uint64_t hint, unsigned long long *stamp) {
  return dispatch64<0>(ctx, p->f, L, list, n, (const uint64_t *)vt, nullptr, (double *)vt + 1, n_dev, hint, stamp);
}

int launch_feval64_raw(ip_ctx *ctx, const ip_problem *p, const LatDev &L, const int32_t *v, uint64_t n,
                       double *out) {
  return dispatch64<1>(ctx, p->f, L, nullptr, n, nullptr, v, out);
}

// (a vertex table holds a polynomial f in this mode: RBF traces run in FP64)
int launch_feval32(ip_ctx *ctx, const ip_problem *p, const LatDev &L, const uint32_t *list, uint64_t n, VEnt *vt,
                   float *vb, uint32_t *fb, unsigned long long *fb_ctr, const unsigned long long *n_dev, uint64_t hint,
                   unsigned long long *stamp) {
  return dispatch32<0>(ctx, p->poly, L, list, n, vt, vb, nullptr, nullptr, nullptr, fb, fb_ctr, nullptr, n_dev, hint,
                       stamp);
}

int launch_set_vb(ip_ctx *ctx, const uint32_t *list, uint64_t n, float *vb, float v) {
  if (n == 0) return IP_OK;
  uint64_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(set_vb_kernel, dim3((unsigned)blocks), dim3(256), 0, ctx->stream, list, n, vb, v);
  IP_TRY_HIP(ctx, hipGetLastError());
  return IP_OK;
}

int ip_feval_impl(ip_ctx *ctx, const ip_problem *p, const int32_t *v_dev, int64_t n, int32_t prec,
                  double *f_dev, double *bound_dev) {
  if (prec == IP_FP64 || !ip_has_fp32_form(p)) {
    if (bound_dev) IP_TRY_HIP(ctx, hipMemsetAsync(bound_dev, 0, sizeof(double) * (size_t)n, ctx->stream));
    return dispatch64<1>(ctx, p->f, p->fine, nullptr, (uint64_t)n, nullptr, v_dev, f_dev);
  }
  // FP32 pass, then canonical FP64 for the unsettled indices
  if (n >= (1ll << 32)) return ip_fail(ctx, IP_EINVAL, "ip_feval: at most 2^32 - 1 vertices per call");
  double *bnd = bound_dev;
  void *tmp_b = nullptr, *fbl = nullptr;
  if (!bnd) {
    IP_TRY(ip_dalloc(ctx, &tmp_b, sizeof(double) * (size_t)n));
    bnd = (double *)tmp_b;
  }
  if (ip_dalloc(ctx, &fbl, sizeof(uint32_t) * (size_t)n) != IP_OK) {
    ip_dfree(ctx, tmp_b);
    return IP_ENOMEM;
  }
  IP_TRY_HIP(ctx, hipMemsetAsync(ctx->ctr_dev, 0, sizeof(Counters), ctx->stream));
  int rc = dispatch32_p<1>(ctx, p, p->fine, nullptr, (uint64_t)n, nullptr, nullptr, v_dev, f_dev, bnd,
                           (uint32_t *)fbl, &ctx->ctr_dev->n_fb);
  unsigned long long nfb = 0;
  if (rc == IP_OK) {
    hipError_t e = hipMemcpyAsync(ctx->ctr_host, ctx->ctr_dev, sizeof(Counters), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) rc = ip_hip(ctx, e, "ip_feval counters");
    nfb = ctx->ctr_host->n_fb;
  }
  if (rc == IP_OK) rc = dispatch64<2>(ctx, p->f, p->fine, (const uint32_t *)fbl, nfb, nullptr, v_dev, f_dev);
  (void)hipStreamSynchronize(ctx->stream);
  ip_dfree(ctx, tmp_b);
  ip_dfree(ctx, fbl);
  ctx->last_fallback = (int64_t)nfb;
  return rc;
}
