// HIP kernels of the GSGP hot path for gfx950 (MI355X, CDNA4, wave64).
//
// Method: "GSGP-CUDA - a CUDA framework for Geometric Semantic Genetic
// Programming" (Trujillo et al., arXiv 2106.04034), Algorithm 1 and the
// Section 2.2 paragraphs on initialization, the interpreter, fitness, GSM and
// survival.  The paper's own CUDA design (one thread per individual for the
// interpreter and the fitness, cuBLAS I?AMIN / I?AMAX for survival) is prior
// art; the mapping here is:
//   k_genome     one thread per gene, counter-based Philox draws;
//   k_compile, k_interpret*  (interp.hip) the genome compiler and the
//                stack-machine interpreter;
//   k_vary       the hot loop: every offspring row of one 2 KiB case chunk is
//                formed from its parent and pool rows with 16-byte loads and
//                non-temporal 16-byte stores, and the chunk's squared
//                residual sum is reduced across the wave in registers;
//                blocks on one XCD share a chunk so distinct parent and pool
//                rows are fetched from HBM about once per chunk;
//   k_mutate_block, k_mutate_slices, k_block_*  up to 15 generations of the
//                loop without selection at a time;
//   k_fitness    16 individuals a block, 16 threads an individual own chunk
//                ranges; FP64 sums, and the group's extremes;
//   k_survive    best and worst with lowest-index ties, elite row copy,
//                per-generation summary and the next generation's tournaments;
//   k_lineage*, k_replay_*  an individual's ancestry, walked and replayed;
//   k_fetch_*    what the getters return, in one piece.
// All kernels are compiled without floating-point contraction so that the
// per-element arithmetic matches the method's definitions operation by
// operation.
#include "device.hpp"

namespace gsgp {
namespace {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC 2011): ten rounds of two
// 32x32 -> 64-bit products with a Weyl key schedule.
struct Words4 {
  uint32_t w0, w1, w2, w3;
};

__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint32_t lo0 = 0xD2511F53u * c0;
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0);
    const uint32_t lo1 = 0xCD9E8D57u * c2;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2);
    const uint32_t x0 = hi1 ^ c1 ^ k0;
    const uint32_t x2 = hi0 ^ c3 ^ k1;
    c0 = x0;
    c1 = lo1;
    c2 = x2;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Words4{c0, c1, c2, c3};
}

// Integer in [0, n) by multiply-shift of one 32-bit word.
__device__ __forceinline__ int32_t draw_below(uint32_t w, uint32_t n) {
  return (int32_t)(((uint64_t)w * (uint64_t)n) >> 32);
}

// Uniform in [0, 1) on the 2^-53 grid from two words (27 + 26 bits).
__device__ __forceinline__ double draw_u53(uint32_t a, uint32_t b) {
  const double hi = (double)(a >> 5);
  const double lo = (double)(b >> 6);
  return (hi * 67108864.0 + lo) * (1.0 / 9007199254740992.0);
}

// ---------------------------------------------------------------------------
// Data preparation: FP64 row-major cases -> feature-major padded X, target in
// the storage type with zero pads, non-finite detection.  One thread per
// column of every run's X tiles (whole tiles: columns from ld on have no
// target).  A padding column of X repeats the last case before it, which lies
// in the same tile: the interpreter evaluates it with the others and stores
// zeros for it, and an all-zero case would meet a zero divisor in nearly every
// program, each of which the threaded evaluator then has to give up (64 runs of
// 200 to 2,531 cases, 512 programs each: 930 -> 611 us).
template <typename T>
__global__ __launch_bounds__(256) void k_prep(const RunDev* __restrict__ runs, Params p,
                                              int64_t total, const double* const* __restrict__ src) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const int run = find_run(p.n_runs, g, [&](int r) { return runs[r].col0; });
  const RunDev& R = runs[run];
  const int64_t col = g - R.col0;
  const bool train = col < R.tr_pad || R.n_test == 0;
  const int64_t at = train ? col : col - R.tr_pad, n = train ? R.n_train : R.n_test;
  const bool real = at < n;
  const int64_t row = real ? at : n - 1;
  const double* Xs = src[4 * run + (train ? 0 : 2)];
  const double* ys = src[4 * run + (train ? 1 : 3)];
  bool bad = false, big = false;
  for (int f = 0; f < R.l; ++f) {
    const double v = Xs[row * R.l + f];
    bad |= !isfinite(v);
    big |= fabs(v) > 0x1p128;
    R.X[x_index(col, f, R.l)] = v;
  }
  const double yv = real ? ys[row] : 0.0;
  bad |= !isfinite(yv) || fabs(yv) > kFltMax;
  if (col < R.ld) ((T*)R.y)[col] = (T)yv;
  if (bad) atomicOr(&R.state[kStNonFinite], 1);
  if (big) atomicOr(&R.state[kStXBig], 1);
}

// ---------------------------------------------------------------------------
// CreatePopulation (Algorithm 1; Section 2.2 "Initialization"): gene q of
// tree t draws Philox counter (q, t, 0, tag), key (seed, run), tag 1 for the
// population and 2 for the random-tree pool.  Word 0 picks the gene type
// against the cumulative thresholds, word 1 the function or feature, words 2
// and 3 the constant.
__global__ __launch_bounds__(256) void k_genome(const RunDev* __restrict__ runs, Params p,
                                                int64_t total) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const int64_t per_run = (int64_t)(p.m + p.r) * p.k;
  const int run = (int)(g / per_run);
  const int64_t local = g - (int64_t)run * per_run;
  const int row = (int)(local / p.k);
  const int q = (int)(local - (int64_t)row * p.k);
  const RunDev& R = runs[run];
  const uint32_t tag = row < p.m ? 1u : 2u;
  const uint32_t t = row < p.m ? (uint32_t)row : (uint32_t)(row - p.m);
  const Words4 w = philox4x32_10((uint32_t)q, t, 0u, tag, p.seed, R.run_id);
  int32_t code;
  double val = 0.0;
  if ((uint64_t)w.w0 < p.t_func) {
    code = -1 - (int32_t)(w.w1 >> 30);
  } else if ((uint64_t)w.w0 < p.t_feat) {
    code = draw_below(w.w1, (uint32_t)R.l);
  } else {
    const double u = draw_u53(w.w2, w.w3);
    const double span = p.erc_hi - p.erc_lo;
    const double scaled = span * u;
    code = -5;
    val = p.erc_lo + scaled;
  }
  R.code[local] = code;
  R.cval[local] = val;
}

// ---------------------------------------------------------------------------
// Wave reductions.  A butterfly over lane distances 32, 16, 8, 4, 2, 1: each
// step adds the same two operands in both partner lanes, so every lane has the
// same bits.  It stays in the vector registers: halves and rows of 16 trade
// places (permlane swaps), then a row rotates by DPP (after the step of
// distance 8 the values repeat every 8 lanes, so a rotation by 4 reaches the
// partner at distance 4, and so on).  Through LDS (__shfl_xor) a step took a
// round trip and the LDS pipe of the CU: 128 individuals on 700 FP64 cases 4.2
// -> 3.8 us a generation, local search (three sums) 27.9 -> 27.0 us for 512 on
// 25,000 cases, blocks of 15 generations 160 -> 132 us for 2,048 on 10,240.
struct LanePair {
  uint32_t own, other;
};
template <int O>
__device__ __forceinline__ LanePair lane_pair(uint32_t v) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  if constexpr (O == 32) {
    const u2 r = __builtin_bit_cast(u2, __builtin_amdgcn_permlane32_swap(v, v, false, false));
    return LanePair{r[0], r[1]};
  } else if constexpr (O == 16) {
    const u2 r = __builtin_bit_cast(u2, __builtin_amdgcn_permlane16_swap(v, v, false, false));
    return LanePair{r[0], r[1]};
  } else {
    static_assert(O == 8 || O == 4 || O == 2 || O == 1, "a distance of the butterfly");
    return LanePair{v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x120 + 16 - O, 0xf, 0xf, false)};  // row_ror
  }
}

template <int O>
__device__ __forceinline__ void lane_pair(float v, float& own, float& other) {
  const LanePair q = lane_pair<O>(__builtin_bit_cast(uint32_t, v));
  own = __builtin_bit_cast(float, q.own);
  other = __builtin_bit_cast(float, q.other);
}
template <int O>
__device__ __forceinline__ void lane_pair(double v, double& own, double& other) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const LanePair lo = lane_pair<O>((uint32_t)u), hi = lane_pair<O>((uint32_t)(u >> 32));
  own = __builtin_bit_cast(double, (uint64_t)hi.own << 32 | lo.own);
  other = __builtin_bit_cast(double, (uint64_t)hi.other << 32 | lo.other);
}

// step(O) for the distances of the butterfly in turn
template <typename Step>
__device__ __forceinline__ void butterfly(Step step) {
  step(std::integral_constant<int, 32>{});
  step(std::integral_constant<int, 16>{});
  step(std::integral_constant<int, 8>{});
  step(std::integral_constant<int, 4>{});
  step(std::integral_constant<int, 2>{});
  step(std::integral_constant<int, 1>{});
}

template <typename A>
__device__ __forceinline__ A wave_sum(A v) {
  butterfly([&](auto o) {
    A own, other;
    lane_pair<decltype(o)::value>(v, own, other);
    v = own + other;
  });
  return v;
}

// Compensated combination of Kahan pairs (value = s - c) with Knuth's
// two-sum: exact error of s1 + s2 is folded into the compensation term.
__device__ __forceinline__ void wave_sum_kahan(float& s, float& c) {
  butterfly([&](auto o) {
    float s1, s2, c1, c2;
    lane_pair<decltype(o)::value>(s, s1, s2);
    lane_pair<decltype(o)::value>(c, c1, c2);
    const float sum = s1 + s2;
    const float bp = sum - s1;
    const float err = (s1 - (sum - bp)) + (s2 - bp);
    c = (c1 + c2) - err;
    s = sum;
  });
}

// Sum over one chunk of (o - t)^2 in the canonical order: each lane adds its
// elements in address order (LaneSse, fed one 16-byte vector at a time as
// the offspring values are formed), then the wave butterfly (sse_finish).
// FP32 forms fall back to FP64 when a square overflows.  The fallback takes
// the offspring values from registers (each offspring vector occupies the
// registers its three operands free) and reads the target chunk again from
// memory (`tgt`, an L2 hit): converting the target vectors to FP64 ahead of
// the rare branch would hold 32 more registers for the whole kernel.
template <typename T, int PREC>
struct LaneSse {
  typedef typename std::conditional<PREC == GSGP_FP64, double, float>::type A;
  A s = 0, c = 0;
  template <typename VT>
  __device__ __forceinline__ void add(const VT& o, const VT& t) {
    constexpr int N = VecOf<T>::N;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const A e = (A)o[k] - (A)t[k];
      if constexpr (PREC == GSGP_FP32_KAHAN) {
        const A y = e * e - c;
        const A u = s + y;
        c = (u - s) - y;
        s = u;
      } else {
        s += e * e;
      }
    }
  }
};

template <typename T, int PREC, int NJ, typename VT>
__device__ __forceinline__ double sse_finish(LaneSse<T, PREC> acc, const bool (&ok)[NJ], const VT (&o)[NJ],
                                             const T* tgt, int lane) {
  constexpr int N = VecOf<T>::N;
  if constexpr (PREC == GSGP_FP64) {
    return wave_sum(acc.s);
  } else {
    double total;
    if constexpr (PREC == GSGP_FP32) {
      total = (double)wave_sum(acc.s);
    } else {
      wave_sum_kahan(acc.s, acc.c);
      total = (double)acc.s - (double)acc.c;
    }
    if (!isfinite(total)) {
      double s = 0.0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (!ok[j]) continue;
        const int e = j * kWave * N + lane * N;
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const double d = (double)o[j][c] - (double)tgt[e + c];
          s += d * d;
        }
      }
      total = wave_sum(s);
    }
    return total;
  }
}

template <typename T, int PREC, int NJ, typename VT>
__device__ __forceinline__ double chunk_sse(const VT (&o)[NJ], const VT (&t)[NJ], const bool (&ok)[NJ],
                                            const T* tgt, int lane) {
  LaneSse<T, PREC> acc;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (ok[j]) acc.add(o[j], t[j]);
  return sse_finish<T, PREC, NJ>(acc, ok, o, tgt, lane);
}

// One offspring's operands for one chunk.  Mutation reads S[p1], sR[r1],
// sR[r2]; crossover reads S[p1], S[p2], sR[r1].  The pointer choice is
// wave-uniform, so both kinds issue the same three 16-byte loads per slot.
// FULL chunks need no lane masks (only a segment's last chunk can be short).
template <typename T, int PREC, bool FULL, int NJ>
__device__ __forceinline__ void vary_offspring(const gsgp_record* rc, const T* Sc, const T* gc, T* dst,
                                               int lane, int64_t len,
                                               const typename VecOf<T>::type (&t)[NJ], const T* tgt,
                                               double* part_out) {
  typedef typename VecOf<T>::type VT;
  constexpr int N = VecOf<T>::N;
  constexpr int64_t kChunk = chunk_cases(sizeof(T));
  // row stride inside a chunk block is the chunk length (compile-time for full chunks)
  const int64_t stride = FULL ? kChunk : len;
  const int op = uni(cload(&rc->op));
  const int p1 = uni(cload(&rc->p1));
  const int r1 = uni(cload(&rc->r1));
  const int second = uni(op == 1 ? cload(&rc->p2) : cload(&rc->r2));
  const T ms = (T)cload(&rc->ms);
  const T* A = Sc + (int64_t)p1 * stride;
  const T* B = (op == 1 ? Sc : gc) + (int64_t)(op == 1 ? second : r1) * stride;
  const T* C = gc + (int64_t)(op == 1 ? r1 : second) * stride;
  bool ok[NJ];
  VT x[NJ], y[NJ], z[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * kWave * N + lane * N;
    ok[j] = FULL || e < len;
    if (ok[j]) {
      x[j] = gload<VT>(A + e);
      y[j] = gload<VT>(B + e);
      z[j] = gload<VT>(C + e);
    } else {
      x[j] = VT(0);
      y[j] = VT(0);
      z[j] = VT(0);
    }
  }
  // Form, clamp, store and accumulate one 16-byte vector at a time, so the
  // operands of a vector die as soon as its offspring value is stored.
  LaneSse<T, PREC> acc;
  VT o[NJ];
  auto emit = [&](int j, VT v) {
    if constexpr (PREC != GSGP_FP64) {
      // a convex combination of two values near +-FLT_MAX can round past it;
      // operands are finite, so a median-of-three clamps exactly
#pragma unroll
      for (int c = 0; c < N; ++c) v[c] = __builtin_amdgcn_fmed3f(v[c], (T)-kFltMax, (T)kFltMax);
    }
    o[j] = v;
    if (ok[j]) {
      gstore_nt<VT>(v, dst + j * kWave * N + lane * N);
      acc.add(v, t[j]);
    }
  };
  if (op == 1) {
    // GSC: O = S[p1] * sR[r1] + S[p2] * (1 - sR[r1])
#pragma unroll
    for (int j = 0; j < NJ; ++j) emit(j, x[j] * z[j] + y[j] * ((T)1 - z[j]));
  } else {
    // GSM: O = S[p1] + ms * (sR[r1] - sR[r2])
#pragma unroll
    for (int j = 0; j < NJ; ++j) emit(j, x[j] + ms * (y[j] - z[j]));
  }
  const double sse = sse_finish<T, PREC, NJ>(acc, ok, o, tgt, lane);
  if (lane == 0) *part_out = sse;
}

// Local search form of vary_offspring.  Stored rows are the operators'
// outputs; individual p's semantics are alpha_p + beta_p * S[p] with its
// scaling from the generation's table `lsg` ([m][2]), applied here as the
// parents are read (so scaling costs no extra pass over the rows).  The
// offspring row is stored unscaled, and the chunk's sums of o, o^2 and o * t
// (FP64, lane then butterfly, over the real cases only) go to part_out[0],
// part_out[m], part_out[2 m]; the fitness kernel fits the offspring's own
// scaling from them.  Real cases of the chunk are its first `real` columns.
template <typename T, bool FULL, int NJ>
__device__ __forceinline__ void vary_offspring_ls(const gsgp_record* rc, const double* lsg, const T* Sc, const T* gc,
                                                  T* dst, int lane, int64_t len, int64_t real,
                                                  const typename VecOf<T>::type (&t)[NJ], double* part_out,
                                                  int64_t m) {
  typedef typename VecOf<T>::type VT;
  constexpr int N = VecOf<T>::N;
  constexpr int64_t kChunk = chunk_cases(sizeof(T));
  const int64_t stride = FULL ? kChunk : len;
  const int op = uni(cload(&rc->op));
  const int p1 = uni(cload(&rc->p1));
  const int r1 = uni(cload(&rc->r1));
  const int second = uni(op == 1 ? cload(&rc->p2) : cload(&rc->r2));
  const T ms = (T)cload(&rc->ms);
  const T* A = Sc + (int64_t)p1 * stride;
  const T* B = (op == 1 ? Sc : gc) + (int64_t)(op == 1 ? second : r1) * stride;
  const T* C = gc + (int64_t)(op == 1 ? r1 : second) * stride;
  // scaling of the parents (the second one only for crossover); in the FP32
  // forms the coefficients are rounded to FP32 and kept finite
  auto coef = [](double v) {
    if constexpr (std::is_same<T, float>::value) return (T)fmin(fmax(v, -kFltMax), kFltMax);
    else return (T)v;
  };
  const T a1 = coef(cload(&lsg[2 * (int64_t)p1])), b1 = coef(cload(&lsg[2 * (int64_t)p1 + 1]));
  const T a2 = op == 1 ? coef(cload(&lsg[2 * (int64_t)second])) : (T)0;
  const T b2 = op == 1 ? coef(cload(&lsg[2 * (int64_t)second + 1])) : (T)1;
  const bool padded = real < len;
  bool ok[NJ];
  VT x[NJ], y[NJ], z[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * kWave * N + lane * N;
    ok[j] = FULL || e < len;
    if (ok[j]) {
      x[j] = gload<VT>(A + e);
      y[j] = gload<VT>(B + e);
      z[j] = gload<VT>(C + e);
    } else {
      x[j] = VT(0);
      y[j] = VT(0);
      z[j] = VT(0);
    }
  }
  auto clamp = [](VT v) {
    if constexpr (std::is_same<T, float>::value) {
#pragma unroll
      for (int c = 0; c < N; ++c) v[c] = __builtin_amdgcn_fmed3f(v[c], (T)-kFltMax, (T)kFltMax);
    }
    return v;
  };
  double so = 0.0, soo = 0.0, sot = 0.0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * kWave * N + lane * N;
    const VT xe = clamp(a1 + b1 * x[j]);
    VT o;
    if (op == 1) {
      // GSC on the parents' semantics: O = T1 * sR[r1] + T2 * (1 - sR[r1])
      const VT ye = clamp(a2 + b2 * y[j]);
      o = clamp(xe * z[j] + ye * ((T)1 - z[j]));
    } else {
      // GSM: O = T + ms * (sR[r1] - sR[r2])
      o = clamp(xe + ms * (y[j] - z[j]));
    }
    if (padded) {
#pragma unroll
      for (int c = 0; c < N; ++c) o[c] = (e + c < real) ? o[c] : (T)0;  // pads stay exact zeros
    }
    if (ok[j]) {
      gstore_nt<VT>(o, dst + e);
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const double ov = (double)o[c];
        so += ov;
        soo += ov * ov;
        sot += ov * (double)t[j][c];
      }
    }
  }
  so = wave_sum(so);
  soo = wave_sum(soo);
  sot = wave_sum(sot);
  if (lane == 0) {
    part_out[0] = so;
    part_out[m] = soo;
    part_out[2 * m] = sot;
  }
}

// Partial sums of an existing row (generation-0 fitness).
template <typename T, int PREC, bool FULL, int NJ>
__device__ __forceinline__ void row_partial(const T* row, int lane, int64_t len,
                                            const typename VecOf<T>::type (&t)[NJ], const T* tgt,
                                            double* part_out) {
  typedef typename VecOf<T>::type VT;
  constexpr int N = VecOf<T>::N;
  bool ok[NJ];
  VT o[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * kWave * N + lane * N;
    ok[j] = FULL || e < len;
    o[j] = ok[j] ? gload<VT>(row + e) : VT(0);
  }
  const double sse = chunk_sse<T, PREC, NJ, VT>(o, t, ok, tgt, lane);
  if (lane == 0) *part_out = sse;
}

template <typename T, int PREC, bool ROWS, bool FULL, bool LS>
__device__ __forceinline__ void vary_task(const RunDev& R, const Params& p, const VaryLaunch& lc, int chunk,
                                          int grp, int lane, int wave) {
  typedef typename VecOf<T>::type VT;
  constexpr int N = VecOf<T>::N;
  constexpr int kChunk = chunk_cases(sizeof(T));
  constexpr int NJ = kChunk / (kWave * N);
  // each instance derives the chunk geometry itself from the chunk index
  const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, chunk, kChunk);
  const int64_t cs = g.cs;
  const int64_t len = FULL ? (int64_t)kChunk : g.len;
  const int gen = ROWS ? 0 : uni(cload(&R.state[kStGen]));
  const int cur = gen & 1;
  // chunk blocks of the tiled buffers (see chunk_geom): rows * cs elements in
  const T* Sc = (const T*)R.S[cur] + (int64_t)p.m * cs;
  T* Oc = (T*)R.S[cur ^ 1] + (int64_t)p.m * cs;
  const T* gc = (const T*)R.sigR + (int64_t)p.r * cs;
  const T* yv = (const T*)R.y + cs;
  const int64_t stride = FULL ? (int64_t)chunk_cases(sizeof(T)) : len;
  VT t[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * kWave * N + lane * N;
    t[j] = (FULL || e < len) ? gload<VT>(yv + e) : VT(0);
  }
  int i_end = (grp + 1) * lc.opb;
  i_end = i_end < p.m ? i_end : p.m;
  double* part = R.part + (int64_t)chunk * p.m;
  if constexpr (ROWS) {
    for (int i = grp * lc.opb + wave; i < i_end; i += lc.waves)
      row_partial<T, PREC, FULL, NJ>(Sc + (int64_t)i * stride, lane, len, t, yv, part + i);
  } else if constexpr (LS) {
    const gsgp_record* recs = R.rec + (int64_t)gen * p.m;
    const double* lsg = R.ls + (int64_t)gen * p.m * 2;
    // real cases of this chunk: the segment's real cases past its first column
    const bool train = chunk < R.nch_tr;
    const int64_t first = train ? cs : cs - R.tr_pad;
    int64_t real = (train ? R.n_train : R.n_test) - first;
    real = real < 0 ? 0 : (real > len ? len : real);
    double* part3 = R.part + (int64_t)chunk * 3 * p.m;
    for (int i = grp * lc.opb + wave; i < i_end; i += lc.waves)
      vary_offspring_ls<T, FULL, NJ>(recs + i, lsg, Sc, gc, Oc + (int64_t)i * stride, lane, len, real, t,
                                     part3 + i, p.m);
  } else {
    const gsgp_record* recs = R.rec + (int64_t)gen * p.m;
    for (int i = grp * lc.opb + wave; i < i_end; i += lc.waves)
      vary_offspring<T, PREC, FULL, NJ>(recs + i, Sc, gc, Oc + (int64_t)i * stride, lane, len, t, yv, part + i);
  }
}

// ---------------------------------------------------------------------------
// GSM / GSC + fitness partials (Algorithm 1 loop: GSM, ComputeFitness).
// Task = (run, 2 KiB chunk of cases, group of `opb` offspring).  Each wave
// takes offspring grp*opb + wave, + waves, ...; per offspring it reads its
// variation record, forms the chunk of the offspring row
//   mutation:  O = S[p1] + ms * (sR[r1] - sR[r2])
//   crossover: O = S[p1] * sR[r1] + S[p2] * (1 - sR[r1])
// (sR holds the squashed pool semantics), stores it with non-temporal
// 16-byte stores and writes the chunk's sum of squared residuals.  With
// ROWS the kernel only forms the partial sums of the current population
// (generation-0 fitness).
template <typename T, int PREC, bool ROWS, bool LOOP, bool LS>
__global__ __launch_bounds__(512) void k_vary(const RunDev* __restrict__ runs, Params p, VaryLaunch lc) {
  constexpr int kChunk = chunk_cases(sizeof(T));
  const int lane = threadIdx.x & 63;
  const int wave = uni(threadIdx.x >> 6);
  // Hardware dispatch sends block b to XCD b % 8.  remap 1: each XCD takes a
  // contiguous range of tasks.  remap 2: XCD x takes the x-th group of
  // `ogroups` tasks (one chunk) of every run of 8 chunks, so the XCDs sweep
  // the rows side by side through an 8-chunk window, every other generation
  // from the last chunk back: what the generation before wrote and read last
  // is still in the memory-side cache (1,024 individuals on 125,000 FP32 cases
  // 221 -> 216 us, 512 on 125,000 FP64 216 -> 211 us).
  // LOOP: a persistent grid, blocks sweep the tasks; otherwise the grid
  // covers every task in one sweep and the loop body runs once (no values
  // hoisted across iterations, fewer registers).
  const int64_t xcd = blockIdx.x & 7, per = lc.grid >> 3;
  const bool back = lc.remap == 2 && !ROWS && (uni(cload(&runs[0].state[kStGen])) & 1);
  const int64_t slot = back ? per - 1 - (blockIdx.x >> 3) : blockIdx.x >> 3;
  for (int64_t it = 0; LOOP || it == 0; ++it) {
    int64_t task;
    if (lc.remap == 2) {
      const int64_t q = slot + it * per;
      task = (q / lc.ogroups) * 8 * lc.ogroups + xcd * lc.ogroups + q % lc.ogroups;
      if ((q / lc.ogroups) * 8 * lc.ogroups >= lc.total_tasks) break;
      if (task >= lc.total_tasks) continue;
    } else {
      task = (lc.remap ? xcd * per + slot : (int64_t)blockIdx.x) + it * lc.grid;
      if (task >= lc.total_tasks) break;
    }
    const int run = find_run(p.n_runs, task, [&](int r) { return runs[r].vary_task0; });
    const RunDev& R = runs[run];
    const int64_t local = task - R.vary_task0;
    const int chunk = (int)(local / lc.ogroups);
    const int grp = (int)(local - (int64_t)chunk * lc.ogroups);
    const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, chunk, kChunk);
    if (g.len == kChunk)
      vary_task<T, PREC, ROWS, true, LS>(R, p, lc, chunk, grp, lane, wave);
    else
      vary_task<T, PREC, ROWS, false, LS>(R, p, lc, chunk, grp, lane, wave);
  }
}

// (the generation-0 partial sums never scale: every individual starts with
// alpha = 0, beta = 1)

// A value and the individual it belongs to; the lowest index wins ties, as
// the first extremum that I?AMIN / I?AMAX return.
struct ValIdx {
  double v;
  int i;
};

__device__ __forceinline__ ValIdx pick_min(ValIdx a, ValIdx b) {
  return (b.v < a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}
__device__ __forceinline__ ValIdx pick_max(ValIdx a, ValIdx b) {
  return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}

// A value and index from the lane that DPP control CTRL names.
template <int CTRL>
__device__ __forceinline__ ValIdx dpp_move(ValIdx x) {
  const uint64_t v = __builtin_bit_cast(uint64_t, x.v);
  const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, false);
  return ValIdx{__builtin_bit_cast(double, (uint64_t)hi << 32 | lo), __builtin_amdgcn_mov_dpp(x.i, CTRL, 0xf, 0xf, false)};
}

__device__ __forceinline__ ValIdx read_lane(ValIdx x, int lane) {
  const uint64_t v = __builtin_bit_cast(uint64_t, x.v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ValIdx{__builtin_bit_cast(double, (uint64_t)hi << 32 | lo), __builtin_amdgcn_readlane(x.i, lane)};
}

// Extrema over groups of W lanes, 16 or 64: within a row of 16 by DPP (its
// pairs, its quads' halves, the halves of its halves, its halves), and the
// four rows through scalar registers; a round through LDS (__shfl_xor) waits
// about 100 cycles for its six reads.
template <int W>
__device__ __forceinline__ void lane_extrema(ValIdx& lo, ValIdx& hi) {
  static_assert(W == 16 || W == kWave, "a DPP row or a wave");
  auto round = [&](ValIdx l, ValIdx h) {
    lo = pick_min(lo, l);
    hi = pick_max(hi, h);
  };
  round(dpp_move<0xb1>(lo), dpp_move<0xb1>(hi));    // quad_perm 1, 0, 3, 2
  round(dpp_move<0x4e>(lo), dpp_move<0x4e>(hi));    // quad_perm 2, 3, 0, 1
  round(dpp_move<0x141>(lo), dpp_move<0x141>(hi));  // row_half_mirror
  round(dpp_move<0x140>(lo), dpp_move<0x140>(hi));  // row_mirror
  if constexpr (W == kWave) {
    const ValIdx l = lo, h = hi;
#pragma unroll
    for (int row = 0; row < 4; ++row) round(read_lane(l, 16 * row), read_lane(h, 16 * row));
  }
}

// ComputeFitness (Section 2.2 "Fitness computation"): a block takes
// kFitGroup individuals of one run; its threads split each segment's chunks
// into kFitRanges contiguous ranges per individual, sum them in chunk order,
// and the ranges are added in range order in FP64.  Then the root mean, and
// the group's best and worst train fitness for the survival kernel.
// What bounds it is the latency of the chunk sums (8 B per individual and
// chunk, read once): kFitUnroll of them are in flight per thread.  16
// individuals a block (128-byte segments) put four times as many CUs to work
// as 64: 1,024 individuals on 2,442 chunks 30.4 -> 13.6 us, on 245 chunks
// 6.9 -> 5.5 us; on 13 chunks, where the launch is all of it, 4.6 -> 4.8 us.
constexpr int kFitRanges = 16;
constexpr int kFitUnroll = 16;

__device__ __forceinline__ double sum_range(const double* __restrict__ part, int64_t stride, int c0, int c1) {
  double s = 0.0;
  int c = c0;
  for (; c + kFitUnroll <= c1; c += kFitUnroll) {
    double v[kFitUnroll];
#pragma unroll
    for (int u = 0; u < kFitUnroll; ++u) v[u] = part[(int64_t)(c + u) * stride];
#pragma unroll
    for (int u = 0; u < kFitUnroll; ++u) s += v[u];
  }
  if (c < c1) {
    double v[kFitUnroll];
#pragma unroll
    for (int u = 0; u < kFitUnroll; ++u) v[u] = c + u < c1 ? part[(int64_t)(c + u) * stride] : 0.0;
#pragma unroll
    for (int u = 0; u < kFitUnroll; ++u)
      if (c + u < c1) s += v[u];
  }
  return s;
}

// Writes the extremes of a group's fitness (threads 0 .. kFitGroup - 1 hold
// the individuals' values).
__device__ __forceinline__ void store_extremes(const RunDev& R, int group, bool live, double f, int i) {
  ValIdx lo{live ? f : INFINITY, live ? i : 0x7fffffff}, hi{live ? f : -INFINITY, live ? i : 0x7fffffff};
  lane_extrema<kFitGroup>(lo, hi);
  if (threadIdx.x == 0) R.extremes[group] = Extremes{lo.v, hi.v, lo.i, hi.i};
}

__global__ __launch_bounds__(kFitRanges * kFitGroup) void k_fitness(const RunDev* __restrict__ runs, Params p,
                                                                     int32_t blocks_per_run, int init) {
  __shared__ double sh_tr[kFitRanges][kFitGroup];
  __shared__ double sh_te[kFitRanges][kFitGroup];
  const int l = threadIdx.x % kFitGroup;
  const int w = threadIdx.x / kFitGroup;
  const int run = blockIdx.x / blocks_per_run;
  const int group = blockIdx.x - run * blocks_per_run;
  const int i = group * kFitGroup + l;
  const RunDev& R = runs[run];
  const bool live = i < p.m;
  const double* part = R.part + (live ? i : 0);
  const int nt = R.nch_tr, ne = R.nch - R.nch_tr;
  const int a0 = (int)((int64_t)nt * w / kFitRanges), a1 = (int)((int64_t)nt * (w + 1) / kFitRanges);
  const int b0 = nt + (int)((int64_t)ne * w / kFitRanges), b1 = nt + (int)((int64_t)ne * (w + 1) / kFitRanges);
  sh_tr[w][l] = sum_range(part, p.m, a0, a1);
  sh_te[w][l] = sum_range(part, p.m, b0, b1);
  __syncthreads();
  if (threadIdx.x < kFitGroup) {
    double s = sh_tr[0][l], st = sh_te[0][l];
#pragma unroll
    for (int q = 1; q < kFitRanges; ++q) {
      s += sh_tr[q][l];
      st += sh_te[q][l];
    }
    const int dst = init ? 0 : ((R.state[kStGen] + 1) & 1);
    const double f = sqrt(s / (double)R.n_train);
    if (live) {
      R.F[dst][i] = f;
      R.Ft[dst][i] = R.n_test > 0 ? sqrt(st / (double)R.n_test) : 0.0;
    }
    store_extremes(R, group, live, f, i);
  }
}

// Local search fitness: each offspring's least-squares scaling and the RMSE
// of its scaled semantics, in closed form from its chunk sums (o, o^2, o * t
// over the real cases; laid out [chunk][3][m]) and the run's target sums.
// With n cases, D = So2 - So^2 / n (n times the variance of o) and
// Sxy = Sot - So * St / n:
//   beta = Sxy / D,  alpha = (St - beta * So) / n,
//   SSE_train = (Stt - St^2 / n) - beta * Sxy   (residual orthogonal to 1, o),
//   SSE_test = sum (alpha + beta o - t)^2 expanded over the test sums.
// A numerically constant offspring (D <= 1e-10 * So2) keeps alpha = 0,
// beta = 1 and SSE = So2 - 2 Sot + Stt.  Chunk sums combine as in k_fitness.
// The scaling goes to the table row of the offspring generation.
__global__ __launch_bounds__(kFitRanges * kFitGroup) void k_fitness_ls(const RunDev* __restrict__ runs, Params p,
                                                                        int32_t blocks_per_run) {
  __shared__ double sh[6][kFitRanges][kFitGroup];
  const int l = threadIdx.x % kFitGroup;
  const int w = threadIdx.x / kFitGroup;
  const int run = blockIdx.x / blocks_per_run;
  const int group = blockIdx.x - run * blocks_per_run;
  const int i = group * kFitGroup + l;
  const RunDev& R = runs[run];
  const bool live = i < p.m;
  const int64_t m = p.m;
  const double* part = R.part + (live ? i : 0);
  const int nt = R.nch_tr, ne = R.nch - R.nch_tr;
  const int a0 = (int)((int64_t)nt * w / kFitRanges), a1 = (int)((int64_t)nt * (w + 1) / kFitRanges);
  const int b0 = nt + (int)((int64_t)ne * w / kFitRanges), b1 = nt + (int)((int64_t)ne * (w + 1) / kFitRanges);
  for (int q = 0; q < 3; ++q) {
    sh[q][w][l] = sum_range(part + q * m, 3 * m, a0, a1);
    sh[3 + q][w][l] = sum_range(part + q * m, 3 * m, b0, b1);
  }
  __syncthreads();
  if (threadIdx.x < kFitGroup) {
    double v[6];
    for (int q = 0; q < 6; ++q) {
      v[q] = sh[q][0][l];
      for (int r = 1; r < kFitRanges; ++r) v[q] += sh[q][r][l];
    }
    const double n = (double)R.n_train, So = v[0], Soo = v[1], Sot = v[2];
    const double St = R.tsum[0], Stt = R.tsum[1];
    const double D = Soo - So * So / n;
    double alpha = 0.0, beta = 1.0, sse;
    if (D > 1e-10 * Soo) {
      const double Sxy = Sot - So * St / n;
      beta = Sxy / D;
      alpha = (St - beta * So) / n;
      sse = (Stt - St * St / n) - beta * Sxy;
    } else {
      sse = Soo - 2.0 * Sot + Stt;
    }
    sse = sse > 0.0 ? sse : 0.0;
    double sse_te = 0.0;
    if (R.n_test > 0) {
      const double ne_ = (double)R.n_test, Se = v[3], See = v[4], Set = v[5];
      const double Ste = R.tsum[2], Stte = R.tsum[3];
      // sum (alpha + beta o - t)^2 = beta^2 See + sum (alpha - t)^2 + 2 beta sum o (alpha - t)
      sse_te = beta * beta * See + (ne_ * alpha * alpha - 2.0 * alpha * Ste + Stte) +
               2.0 * beta * (alpha * Se - Set);
      sse_te = sse_te > 0.0 ? sse_te : 0.0;
    }
    const int g1 = R.state[kStGen] + 1;
    const int dst = g1 & 1;
    const double f = sqrt(sse / n);
    if (live) {
      R.F[dst][i] = f;
      R.Ft[dst][i] = R.n_test > 0 ? sqrt(sse_te / (double)R.n_test) : 0.0;
      R.ls[((int64_t)g1 * m + i) * 2] = alpha;
      R.ls[((int64_t)g1 * m + i) * 2 + 1] = beta;
    }
    store_extremes(R, group, live, f, i);
  }
}

// Local search: sums of the stored target over a run's real train and test
// cases (one block per run; thread-strided FP64 sums, then a fixed-order LDS
// tree, so the bits never vary).  Also writes generation 0's scaling table
// row (alpha = 0, beta = 1).
template <typename T>
__global__ __launch_bounds__(256) void k_target_sums(const RunDev* __restrict__ runs, Params p) {
  __shared__ double sh[4][256];
  const RunDev& R = runs[blockIdx.x];
  const T* y = (const T*)R.y;
  double a = 0.0, b = 0.0, c = 0.0, d = 0.0;
  for (int64_t k = threadIdx.x; k < R.n_train; k += blockDim.x) {
    const double v = (double)y[k];
    a += v;
    b += v * v;
  }
  for (int64_t k = threadIdx.x; k < R.n_test; k += blockDim.x) {
    const double v = (double)y[R.tr_pad + k];
    c += v;
    d += v * v;
  }
  sh[0][threadIdx.x] = a;
  sh[1][threadIdx.x] = b;
  sh[2][threadIdx.x] = c;
  sh[3][threadIdx.x] = d;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int q = 0; q < 4; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) R.tsum[threadIdx.x] = sh[threadIdx.x][0];
  for (int i = threadIdx.x; i < p.m; i += blockDim.x) {
    R.ls[2 * (int64_t)i] = 0.0;
    R.ls[2 * (int64_t)i + 1] = 1.0;
  }
}

// ---------------------------------------------------------------------------
// Survival, summary and the next generation's variation draws.
// The best of m individuals, by all threads of a block.
template <typename View>
__device__ ValIdx block_min(int m, View F, ValIdx* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  ValIdx x{INFINITY, 0x7fffffff};
  for (int i = threadIdx.x; i < m; i += blockDim.x) x = pick_min(x, ValIdx{F(i), i});
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = pick_min(x, ValIdx{__shfl_xor(x.v, o, kWave), __shfl_xor(x.i, o, kWave)});
  if (lane == 0) sh[wave] = x;
  __syncthreads();
  ValIdx r = sh[0];
  for (int w = 1; w < nw; ++w) r = pick_min(r, sh[w]);
  __syncthreads();
  if (r.i < 0 || r.i >= m) r.i = 0;  // fitness is always finite; keep indices in range regardless
  return r;
}

// Sequential access to the Philox words W[0], W[1], ... of one offspring:
// word w is lane w % 4 of Philox(counter (i, w / 4, gen, 3)).
struct WordStream {
  uint32_t i, gen, k0, k1;
  int block;
  Words4 cur;
  __device__ uint32_t at(int w) {
    const int b = w >> 2;
    if (b != block) {
      cur = philox4x32_10(i, (uint32_t)b, gen, 3u, k0, k1);
      block = b;
    }
    const int s = w & 3;
    return s == 0 ? cur.w0 : (s == 1 ? cur.w1 : (s == 2 ? cur.w2 : cur.w3));
  }
};

// Tournament: s uniform candidates, the first with strictly smaller fitness
// wins (ties go to the earlier draw).  Bound by the latency of the fitness
// reads, so eight candidates are read at a time (the last ones again where s is
// no multiple of eight: a candidate does not beat itself).  A generation with
// tournaments of 64, one read after the other -> eight at a time: 256 individuals
// on 25,000 cases 60.9 -> 50.5 us (52.4 with the fitness staged in LDS), 4,096 on
// 1,250 66.7 -> 50.3 us (496).
template <typename View>
__device__ __forceinline__ int32_t tournament(WordStream& ws, int first, int s, int m, View F) {
  constexpr int B = 8;
  int32_t best = 0;
  double fb = INFINITY;
  for (int j0 = 0; j0 < s; j0 += B) {
    int32_t c[B];
    double f[B];
#pragma unroll
    for (int q = 0; q < B; ++q) {
      c[q] = draw_below(ws.at(first + (j0 + q < s ? j0 + q : s - 1)), (uint32_t)m);
      f[q] = F(c[q]);
    }
#pragma unroll
    for (int q = 0; q < B; ++q) {
      if ((j0 == 0 && q == 0) || f[q] < fb) {
        best = c[q];
        fb = f[q];
      }
    }
  }
  return best;
}

template <typename View>
__device__ gsgp_record draw_record(const Params& p, uint32_t run_id, int gen_draw, int i, View F) {
  WordStream ws{(uint32_t)i, (uint32_t)gen_draw, p.seed, run_id, -1, Words4{0, 0, 0, 0}};
  const uint32_t w0 = ws.at(0), w1 = ws.at(1), w2 = ws.at(2), w3 = ws.at(3), w4 = ws.at(4);
  gsgp_record rc;
  rc.reserved = 0;
  if (p.tsize > 0 && (uint64_t)w0 < p.t_xo) {
    rc.op = 1;
    rc.p1 = tournament(ws, 5, p.tsize, p.m, F);
    rc.p2 = tournament(ws, 5 + p.tsize, p.tsize, p.m, F);
    rc.r1 = draw_below(w1, (uint32_t)p.r);
    rc.r2 = -1;
    rc.ms = 0.0;
  } else {
    rc.op = 0;
    rc.p1 = p.tsize > 0 ? tournament(ws, 5, p.tsize, p.m, F) : i;
    rc.p2 = -1;
    rc.r1 = draw_below(w1, (uint32_t)p.r);
    rc.r2 = draw_below(w2, (uint32_t)p.r);
    rc.ms = p.ms_random ? p.ms * draw_u53(w3, w4) : p.ms;
  }
  return rc;
}

// draw_record in two halves for tournaments of up to kAheadTournament: the
// candidates and their fitness are read before it is known which individual
// the elite replaces (`dst`, fitness f_dst, or -1), all of them at once.  Sizes
// up to four, the usual ones; beyond, the candidates' registers would double and
// the draws follow the decision (survival of 256 individuals with four
// candidates 7.0 us, with five 8.2, with eight 8.5).
constexpr int kAheadTournament = 4;
struct DrawAhead {
  Words4 w;
  uint32_t w4;
  int32_t c[2 * kAheadTournament];
  double f[2 * kAheadTournament];
};

__device__ __forceinline__ DrawAhead draw_ahead(const Params& p, uint32_t run_id, int gen_draw, int i,
                                                const GSGP_GLOBAL double* F) {
  DrawAhead d;
  d.w = philox4x32_10((uint32_t)i, 0, (uint32_t)gen_draw, 3u, p.seed, run_id);
  const Words4 a = philox4x32_10((uint32_t)i, 1, (uint32_t)gen_draw, 3u, p.seed, run_id);
  const Words4 b = philox4x32_10((uint32_t)i, 2, (uint32_t)gen_draw, 3u, p.seed, run_id);
  const Words4 c = philox4x32_10((uint32_t)i, 3, (uint32_t)gen_draw, 3u, p.seed, run_id);
  d.w4 = a.w0;
  const uint32_t word[2 * kAheadTournament] = {a.w1, a.w2, a.w3, b.w0, b.w1, b.w2, b.w3, c.w0};
#pragma unroll
  for (int q = 0; q < 2 * kAheadTournament; ++q) {
    d.c[q] = q < 2 * p.tsize ? draw_below(word[q], (uint32_t)p.m) : 0;
    d.f[q] = F[d.c[q]];
  }
  return d;
}

__device__ __forceinline__ gsgp_record draw_finish(const Params& p, const DrawAhead& d, int dst, double f_dst) {
  int32_t best[2] = {0, 0};
  double fb[2] = {INFINITY, INFINITY};
#pragma unroll
  for (int q = 0; q < 2 * kAheadTournament; ++q) {
    if (q >= 2 * p.tsize) continue;
    const double f = d.c[q] == dst ? f_dst : d.f[q];
    const bool second = q >= p.tsize;
    // the first candidate of each tournament, then strictly smaller ones
    if (q == 0 || q == p.tsize || f < fb[second]) {
      if (second) {
        best[1] = d.c[q];
        fb[1] = f;
      } else {
        best[0] = d.c[q];
        fb[0] = f;
      }
    }
  }
  const bool xo = (uint64_t)d.w.w0 < p.t_xo;
  gsgp_record rc;
  rc.reserved = 0;
  rc.op = xo ? 1 : 0;
  rc.p1 = best[0];
  rc.p2 = xo ? best[1] : -1;
  rc.r1 = draw_below(d.w.w1, (uint32_t)p.r);
  rc.r2 = xo ? -1 : draw_below(d.w.w2, (uint32_t)p.r);
  rc.ms = xo ? 0.0 : p.ms_random ? p.ms * draw_u53(d.w.w3, d.w4) : p.ms;
  return rc;
}

// Best and worst of a run's fitness from its groups' extremes: every wave
// reduces them for itself, so no barrier is needed; `first` is the lane's
// first group's, where it has one.
__device__ __forceinline__ void run_extrema(const RunDev& R, int m, const Extremes& first, ValIdx& lo, ValIdx& hi) {
  const int groups = (m + kFitGroup - 1) / kFitGroup;
  const int lane = threadIdx.x & 63;
  lo = lane < groups ? ValIdx{first.min, first.min_i} : ValIdx{INFINITY, 0x7fffffff};
  hi = lane < groups ? ValIdx{first.max, first.max_i} : ValIdx{-INFINITY, 0x7fffffff};
  for (int g = lane + kWave; g < groups; g += kWave) {
    const Extremes e = R.extremes[g];
    lo = pick_min(lo, ValIdx{e.min, e.min_i});
    hi = pick_max(hi, ValIdx{e.max, e.max_i});
  }
  lane_extrema<kWave>(lo, hi);
  // fitness is always finite; keep indices in range regardless
  if (lo.i < 0 || lo.i >= m) lo.i = 0;
  if (hi.i < 0 || hi.i >= m) hi.i = 0;
}

// Survival with elitism (Section 2.2 "Survival"; Algorithm 1): offspring
// replace parents; when the best parent is strictly better than the best
// offspring it overwrites the worst offspring (lowest index on ties, as the
// first extremum that I?AMIN / I?AMAX return).  Then the summary and the next
// generation's draws.  The best parent is in its generation's summary, the
// best and worst offspring come from the fitness kernel's groups, so a block
// reads m / 16 entries where it read and reduced 2 m values; surv_blks blocks
// per run take the decision redundantly and share the elite row copy (16 KiB
// a block) and the draws (64 a block: with the copy going on, one wave takes
// them; a row of a few cases gave two blocks, whose one wave each drew 512).
// The last block to arrive publishes the elite fitness and advances the
// generation counter.  Bound by latency: extremes, the last best and the
// tournaments' candidates are read before any of them is waited for, and the
// decision's reduction goes by DPP.  1,024 individuals on 5,000 cases 4.8 us,
// on 100,000 5.9 us; 7.7 and 8.4 us when the draws began after the decision,
// 14.2 and 11.0 us when every block reduced the whole fitness.
template <typename T>
__global__ __launch_bounds__(256) void k_survive(const RunDev* __restrict__ runs, Params p,
                                                 int32_t total, int mode) {
  __shared__ ValIdx sh[8];
  const int run = find_run(p.n_runs, (int64_t)blockIdx.x, [&](int r) { return (int64_t)runs[r].surv_blk0; });
  const RunDev& R = runs[run];
  const int bl = blockIdx.x - R.surv_blk0;
  const int nb = R.surv_blks;
  const int m = p.m;
  const int gen = (mode == kSurvInit) ? 0 : uni(cload(&R.state[kStGen]));
  const int replay_elite = uni(cload(&R.state[kStReplayElite]));
  const int replay_select = uni(cload(&R.state[kStReplaySelect]));
  const int cur = gen & 1, nxt = cur ^ 1;
  const GSGP_GLOBAL double* FP = (const GSGP_GLOBAL double*)R.F[cur];
  const GSGP_GLOBAL double* FtP = (const GSGP_GLOBAL double*)R.Ft[cur];
  GSGP_GLOBAL double* FO = (GSGP_GLOBAL double*)R.F[nxt];
  GSGP_GLOBAL double* FtO = (GSGP_GLOBAL double*)R.Ft[nxt];
  const bool gen_mode = mode == kSurvGen;
  int copied = 0, src = -1, dst = -1;
  ValIdx bo{0.0, 0}, wo{0.0, 0};
  // What the decision and the draws read, before either waits for it.
  const int lane = threadIdx.x & 63;
  const GSGP_GLOBAL Extremes* ex =
      (const GSGP_GLOBAL Extremes*)R.extremes + (lane < (m + kFitGroup - 1) / kFitGroup ? lane : 0);
  const Extremes first{ex->min, ex->max, ex->min_i, ex->max_i};
  const GSGP_GLOBAL gsgp_gen_stats* stats = (const GSGP_GLOBAL gsgp_gen_stats*)R.stats;
  const double prev_best = gen_mode ? stats[gen].best_train_rmse : 0.0;
  const int prev_index = gen_mode ? stats[gen].best_index : 0;
  const int gen_draw = gen_mode ? gen + 2 : gen + 1;
  const bool draws = !replay_select && gen_draw <= p.gmax;
  const bool ahead = draws && p.tsize > 0 && p.tsize <= kAheadTournament;
  const int per_draw = (m + nb - 1) / nb;
  const int i0 = per_draw * bl;
  const int i1 = (i0 + per_draw) < m ? (i0 + per_draw) : m;
  const GSGP_GLOBAL double* F = gen_mode ? FO : FP;
  DrawAhead mine;
  if (ahead && i0 + (int)threadIdx.x < i1) mine = draw_ahead(p, R.run_id, gen_draw, i0 + (int)threadIdx.x, F);
  const double f_prev = gen_mode && (uint32_t)prev_index < (uint32_t)m ? FP[prev_index] : 0.0;
  if (mode != kSurvSelectOnly) run_extrema(R, m, first, bo, wo);  // of the offspring, or of generation 0
  if (gen_mode) {
    if (replay_elite) {
      const gsgp_gen_stats e = R.elite_in[gen];
      copied = e.elite_copied;
      src = e.elite_src;
      dst = e.elite_dst;
    } else if (prev_best < bo.v) {
      copied = 1;
      src = prev_index;
      dst = wo.i;
    }
    if (copied) {
      typedef typename VecOf<T>::type VT;
      constexpr int N = VecOf<T>::N;
      constexpr int64_t CH = chunk_cases(sizeof(T));
      const int64_t nvec = R.ld / N;
      const int64_t per = (nvec + nb - 1) / nb;
      const int64_t v0 = per * bl;
      const int64_t v1 = (v0 + per) < nvec ? (v0 + per) : nvec;
      const T* from = (const T*)R.S[cur];
      T* to = (T*)R.S[nxt];
      // four vectors in flight per thread; all N cases of a vector lie in one chunk.
      // With more than one wave, wave 0 takes the draws below while the
      // other waves copy, so the copy's memory latency overlaps the draws.
      constexpr int U = 4;
      const bool split = blockDim.x > kWave;
      const int ct = split ? (int)threadIdx.x - kWave : (int)threadIdx.x;
      const int cn = split ? (int)blockDim.x - kWave : (int)blockDim.x;
      const int64_t step = (int64_t)cn * U;
      if (ct >= 0) {
        for (int64_t v = v0 + ct; v < v1; v += step) {
          VT buf[U];
          int64_t at[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int64_t w = v + (int64_t)u * cn;
            if (w < v1) {
              const int64_t col = w * N;
              buf[u] = *(const VT*)(from + tiled_index(R.tr_pad, R.te_pad, R.nch_tr, CH, m, src, col));
              at[u] = tiled_index(R.tr_pad, R.te_pad, R.nch_tr, CH, m, dst, col);
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (v + (int64_t)u * cn < v1) *(VT*)(to + at[u]) = buf[u];
        }
      }
    }
  }
  const double f_src = copied ? (replay_elite ? FP[src] : f_prev) : 0.0;
  // when the other waves copied the elite row, wave 0 alone takes the draws
  const bool draw_split = copied && blockDim.x > kWave;
  // fitness of the individuals the next draw selects from
  auto view_new = [&](int i) { return (copied && i == dst) ? f_src : FO[i]; };
  auto view_cur = [&](int i) { return FP[i]; };
  if (bl == 0 && mode != kSurvSelectOnly) {
    ValIdx b = bo;
    if (gen_mode) {
      if (replay_elite) {
        b = block_min(m, view_new, sh);
      } else if (copied) {
        // an elite copy is strictly better than every offspring
        b = ValIdx{f_src, dst};
      }
    }
    if (threadIdx.x == 0) {
      gsgp_gen_stats st;
      st.best_train_rmse = b.v;
      st.best_test_rmse = gen_mode ? ((copied && b.i == dst) ? FtP[src] : FtO[b.i]) : FtP[b.i];
      st.best_index = b.i;
      st.elite_copied = copied;
      st.elite_src = src;
      st.elite_dst = dst;
      R.stats[gen_mode ? gen + 1 : 0] = st;
    }
  }
  if (draws) {
    gsgp_record* out = R.rec + (int64_t)(gen_draw - 1) * m;
    const int dn = draw_split ? kWave : (int)blockDim.x;  // threads taking draws
    for (int i = i0 + (int)threadIdx.x; (int)threadIdx.x < dn && i < i1; i += dn) {
      if (ahead) {
        if (i != i0 + (int)threadIdx.x) mine = draw_ahead(p, R.run_id, gen_draw, i, F);
        out[i] = draw_finish(p, mine, copied ? dst : -1, f_src);
      } else {
        out[i] = gen_mode ? draw_record(p, R.run_id, gen_draw, i, view_new)
                          : draw_record(p, R.run_id, gen_draw, i, view_cur);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && atomicAdd(&R.state[kStDone], 1) == nb - 1) {
    R.state[kStDone] = 0;
    if (gen_mode) {
      if (copied) {
        FO[dst] = FP[src];
        FtO[dst] = FtP[src];
        if (p.ls) {  // the copy keeps its source's scaling
          const int64_t m64 = m;
          R.ls[((int64_t)(gen + 1) * m64 + dst) * 2] = R.ls[((int64_t)gen * m64 + src) * 2];
          R.ls[((int64_t)(gen + 1) * m64 + dst) * 2 + 1] = R.ls[((int64_t)gen * m64 + src) * 2 + 1];
        }
      }
      R.state[kStGen] = gen + 1;
    }
  }
}

// ---------------------------------------------------------------------------
// Blocks of generations of the loop without selection (the paper's own loop:
// every individual is mutated once a generation, Section 2.1 stage 5).
//
// Without tournaments the draws do not depend on the fitness, and an
// individual's line crosses another one only where the elite copy overwrites
// it.  So a wave takes one individual's chunk through all generations of a
// block in registers (k_mutate_block), each generation's squared error sums
// are combined for all of them (k_block_fitness), and the elite decisions are
// then made step by step (k_block_elite): a copy gives individual dst another
// line, which k_block_row follows through the rest of the block for that one
// row, correcting its sums and its final values.  Values and sums are formed
// by the operations, and in the order, of one generation at a time.
//
// What a generation reads and writes falls from a parent, two pool rows and an
// offspring row to the two pool rows, which mostly come from the caches, plus
// one in 7 or 15 of the other two.  Per generation, one at a time -> 7 -> 15 a
// block: 10,240 individuals on 102,400 FP32 cases 2,233 -> 1,104 -> 1,006 us (a
// chunk's pool column is 20 MB, so most of its reads leave the XCD's L2: 565 us
// slice by slice, see k_mutate_slices); 4,000 on 30,000 185 -> 104 -> 93 us
// (whole chunks); 2,048 on 10,240 (22 us now, with sums in registers)
// 58 -> 25.8 -> 25.4 us; 600 on 2,000 23 -> 11.9 -> 13.8 us; 128 on 500 (FP64)
// 23 -> 11.0 -> 12.6 us.

__device__ __forceinline__ double lane_value(double v, int lane) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One block step's fitness arrays: the table for steps inside the block, the
// run's own arrays for its last one (and its start, step 0).
__device__ __forceinline__ double* step_F(const RunDev& R, int m, int base, int gens, int step, bool test) {
  if (step == 0 || step == gens) {
    const int at = (base + step) & 1;
    return test ? R.Ft[at] : R.F[at];
  }
  return R.block_F + ((int64_t)(test ? kBlockGens - 1 : 0) + (step - 1)) * m;
}

// The draws of steps 2 .. gens + 1 (step 1's were made with the generation
// before it): what k_survive draws, one thread a record.
__global__ __launch_bounds__(256) void k_block_draws(const RunDev* __restrict__ runs, Params p, int32_t gens,
                                                     int64_t total) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= total) return;
  const int64_t per_run = (int64_t)gens * p.m;
  const int run = (int)(q / per_run);
  const int64_t local = q - run * per_run;
  const RunDev& R = runs[run];
  const int g = R.state[kStGen] + 2 + (int)(local / p.m);
  const int i = (int)(local % p.m);
  if (local == 0) {
    R.block->base = R.state[kStGen];
    R.block->n = 0;
    R.block->dst = -1;
  }
  if (g <= p.gmax)
    R.rec[(int64_t)(g - 1) * p.m + i] = draw_record(p, R.run_id, g, i, [](int) { return 0.0; });
}

// One individual's chunk through the generations of a block.
template <typename T, int PREC, bool FULL>
__device__ __forceinline__ void mutate_block_one(const RunDev& R, const Params& p, int gens, int chunk, int i,
                                                 int lane) {
  typedef typename VecOf<T>::type VT;
  constexpr int N = VecOf<T>::N;
  constexpr int kChunk = chunk_cases(sizeof(T));
  constexpr int NJ = kChunk / (kWave * N);
  const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, chunk, kChunk);
  const int64_t len = FULL ? (int64_t)kChunk : g.len;
  const int gen = uni(cload(&R.state[kStGen]));
  const int cur = gen & 1;
  const T* Sc = (const T*)R.S[cur] + (int64_t)p.m * g.cs;
  T* Oc = (T*)R.S[cur ^ 1] + (int64_t)p.m * g.cs;  // gens is odd
  const T* gc = (const T*)R.sigR + (int64_t)p.r * g.cs;
  const T* yv = (const T*)R.y + g.cs;
  VT t[NJ];
  bool ok[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * kWave * N + lane * N;
    ok[j] = FULL || e < len;
    t[j] = ok[j] ? gload<VT>(yv + e) : VT(0);
  }
  VT x[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) x[j] = ok[j] ? gload<VT>(Sc + (int64_t)i * len + j * kWave * N + lane * N) : VT(0);
  // a step's pool rows are read while the step before is worked on
  auto read = [&](int s, T& ms, VT (&a)[NJ], VT (&b)[NJ]) {
    const gsgp_record* rc = R.rec + (int64_t)(gen + s) * p.m + i;
    const T* A = gc + (int64_t)uni(cload(&rc->r1)) * len;
    const T* B = gc + (int64_t)uni(cload(&rc->r2)) * len;
    ms = (T)cload(&rc->ms);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int e = j * kWave * N + lane * N;
      a[j] = ok[j] ? gload<VT>(A + e) : VT(0);
      b[j] = ok[j] ? gload<VT>(B + e) : VT(0);
    }
  };
  auto step = [&](int s, T ms, const VT (&a)[NJ], const VT (&b)[NJ]) {
    LaneSse<T, PREC> acc;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      VT v = x[j] + ms * (a[j] - b[j]);
      if constexpr (PREC != GSGP_FP64) {
#pragma unroll
        for (int c = 0; c < N; ++c) v[c] = __builtin_amdgcn_fmed3f(v[c], (T)-kFltMax, (T)kFltMax);
      }
      x[j] = v;
      if (ok[j]) acc.add(v, t[j]);
    }
    const double sse = sse_finish<T, PREC, NJ>(acc, ok, x, yv, lane);
    if (lane == 0) R.part[((int64_t)s * R.nch + chunk) * p.m + i] = sse;
  };
  T ms0, ms1;
  VT a0[NJ], b0[NJ], a1[NJ], b1[NJ];
  read(0, ms0, a0, b0);
  for (int s = 0;;) {
    if (s + 1 < gens) read(s + 1, ms1, a1, b1);
    step(s, ms0, a0, b0);
    if (++s >= gens) break;
    if (s + 1 < gens) read(s + 1, ms0, a0, b0);
    step(s, ms1, a1, b1);
    if (++s >= gens) break;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (ok[j]) gstore_nt<VT>(x[j], Oc + (int64_t)i * len + j * kWave * N + lane * N);
}

template <typename T, int PREC, bool FULL>
__device__ __forceinline__ void mutate_block_task(const RunDev& R, const Params& p, const VaryLaunch& lc, int gens,
                                                  int chunk, int grp, int lane, int wave) {
  int i_end = (grp + 1) * lc.opb;
  i_end = i_end < p.m ? i_end : p.m;
  for (int i = grp * lc.opb + wave; i < i_end; i += lc.waves) mutate_block_one<T, PREC, FULL>(R, p, gens, chunk, i, lane);
}

// k_mutate_block for pools whose chunk column is larger than an XCD's L2, FP32
// (where: slices_pay): a wave takes a slice of eight lanes' cases (two pieces of
// 128 bytes a row) of eight individuals through the generations, then the next
// slice, so that the blocks of an XCD, which start together and do the same
// work, read an eighth of the pool column at a time.  A lane's cases and their order are those of
// k_mutate_block's lane 8 slice + lane % 8, so the slices are taken in
// bit-reversed order and their sums added like the butterfly's first three
// distances: 0 + 4, 2 + 6, ....  The draws of a block's individuals are in LDS,
// which all slices read.  An individual with a sum that is not finite is done
// again by mutate_block_one, which falls back to FP64.
//
// What bounds it is the L2 (73 % hits against 23 %) and the start of a slice,
// whose rows come from HBM.  Blocks of 16 waves in step are the best: 15
// generations of 10,240 on 25,600 cases 1,777 us, of 8 waves 2,020, of 4 2,700;
// reading a step's rows one step ahead costs a quarter of the waves: 2,199.
constexpr int kSlices = 8;
constexpr int kSliceWaves = 16;                     // waves a block
constexpr int kSliceGroup = kSliceWaves * kSlices;  // individuals a block

struct SliceDraw {
  uint32_t r1, r2;  // byte offsets of the pool rows in a chunk's column
  float ms;
};

__global__ __launch_bounds__(kSliceWaves * kWave) void k_mutate_slices(const RunDev* __restrict__ runs, Params p,
                                                                       VaryLaunch lc, int64_t total_tasks,
                                                                       int32_t groups, int32_t gens) {
  typedef float T;
  typedef f4 VT;
  constexpr int N = 4, NJ = 2, kLanes = kWave / kSlices;
  constexpr int kChunk = chunk_cases(sizeof(T));
  static_assert(kChunk == NJ * kWave * N, "a lane has two vectors of a chunk");
  __shared__ SliceDraw draws[kBlockGens][kSliceGroup];
  const int lane = threadIdx.x & 63;
  const int wave = uni(threadIdx.x >> 6);
  const int64_t task = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (task >= total_tasks) return;
  const int64_t at = task / groups;  // chunk over all runs
  const int run = find_run(p.n_runs, at, [&](int r) { return runs[r].vary_task0 / lc.ogroups; });
  const RunDev& R = runs[run];
  const int chunk = (int)(at - R.vary_task0 / lc.ogroups);
  const int i0 = (int)(task - at * groups) * kSliceGroup;
  const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, chunk, kChunk);
  if (g.len != kChunk) {
    for (int q = wave; q < kSliceGroup && i0 + q < p.m; q += kSliceWaves)
      mutate_block_one<T, GSGP_FP32, false>(R, p, gens, chunk, i0 + q, lane);
    return;
  }
  const int gen = uni(cload(&R.state[kStGen]));
  const int cur = gen & 1;
  for (int q = threadIdx.x; q < gens * kSliceGroup; q += kSliceWaves * kWave) {
    const int s = q / kSliceGroup, k = q % kSliceGroup;
    const int i = i0 + k < p.m ? i0 + k : p.m - 1;
    const gsgp_record* rc = R.rec + (int64_t)(gen + s) * p.m + i;
    draws[s][k] = SliceDraw{(uint32_t)rc->r1 * kChunkBytes, (uint32_t)rc->r2 * kChunkBytes, (T)rc->ms};
  }
  __syncthreads();
  const int own = wave * kSlices + lane / kLanes;  // the lane's individual in the block
  const int i = i0 + own;
  const bool live = i < p.m;
  const int64_t row = (int64_t)(live ? i : p.m - 1) * kChunk;
  const T* Sc = (const T*)R.S[cur] + (int64_t)p.m * g.cs + row;
  T* Oc = (T*)R.S[cur ^ 1] + (int64_t)p.m * g.cs + row;  // gens is odd
  const GSGP_GLOBAL char* gc = (const GSGP_GLOBAL char*)((const T*)R.sigR + (int64_t)p.r * g.cs);
  const T* yv = (const T*)R.y + g.cs;
  T sum[kBlockGens], pair[kBlockGens], quad[kBlockGens], half[kBlockGens];
#pragma unroll 1
  for (int v = 0; v < kSlices; ++v) {
    const int slice = (v & 1) << 2 | (v & 2) | v >> 2;
    const int e0 = (slice * kLanes + lane % kLanes) * N;
    VT x[NJ], t[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      x[j] = gload_nt<VT>(Sc + e0 + j * kWave * N);
      t[j] = gload<VT>(yv + e0 + j * kWave * N);
    }
    struct Rows {
      VT a[NJ], b[NJ];
      T ms;
    };
    auto read = [&](int s) {
      const SliceDraw d = draws[s][own];
      Rows q;
      q.ms = d.ms;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint32_t e = (uint32_t)(e0 + j * kWave * N) * sizeof(T);
        q.a[j] = *(const GSGP_GLOBAL VT*)(gc + (d.r1 + e));
        q.b[j] = *(const GSGP_GLOBAL VT*)(gc + (d.r2 + e));
      }
      return q;
    };
    // The steps past `gens` are branches, not a loop of its own for each
    // number: in one region of code the compiler moves the reads of several
    // steps together, and spills.
#pragma unroll
    for (int s = 0; s < kBlockGens; ++s) {
      if (s >= gens) continue;
      const Rows now = read(s);
      LaneSse<T, GSGP_FP32> acc;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        VT u = x[j] + now.ms * (now.a[j] - now.b[j]);
#pragma unroll
        for (int c = 0; c < N; ++c) u[c] = __builtin_amdgcn_fmed3f(u[c], -kFltMax, (T)kFltMax);
        x[j] = u;
        acc.add(u, t[j]);
      }
      sum[s] = acc.s;
    }
    if (live) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) gstore_nt<VT>(x[j], Oc + e0 + j * kWave * N);
    }
    // the butterfly's distances 32, 16, 8
#pragma unroll
    for (int s = 0; s < kBlockGens; ++s) {
      if (!(v & 1)) {
        pair[s] = sum[s];
      } else {
        sum[s] = pair[s] + sum[s];
        if (!(v & 2)) {
          quad[s] = sum[s];
        } else {
          sum[s] = quad[s] + sum[s];
          if (!(v & 4))
            half[s] = sum[s];
          else
            sum[s] = half[s] + sum[s];
        }
      }
    }
    __syncthreads();  // the waves of a block stay at one slice
  }
  bool finite = true;
#pragma unroll
  for (int s = 0; s < kBlockGens; ++s) {
    if (s >= gens) continue;
    T w = sum[s];
    w += __shfl_xor(w, 4, kWave);
    w += __shfl_xor(w, 2, kWave);
    w += __shfl_xor(w, 1, kWave);
    finite = finite && isfinite(w);
    if (live && lane % kLanes == 0) R.part[((int64_t)s * R.nch + chunk) * p.m + i] = (double)w;
  }
  uint64_t again = __builtin_amdgcn_ballot_w64(live && !finite && lane % kLanes == 0);
  while (again) {
    const int q = __builtin_ctzll(again);
    again &= again - 1;
    mutate_block_one<T, GSGP_FP32, true>(R, p, gens, chunk, i0 + wave * kSlices + q / kLanes, lane);
  }
}

// Task = (run, chunk, group of offspring) as in k_vary, same block order.
template <typename T, int PREC>
__global__ __launch_bounds__(512) void k_mutate_block(const RunDev* __restrict__ runs, Params p, VaryLaunch lc,
                                                      int32_t gens) {
  constexpr int kChunk = chunk_cases(sizeof(T));
  const int lane = threadIdx.x & 63;
  const int wave = uni(threadIdx.x >> 6);
  const int64_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, per = lc.grid >> 3;
  const int64_t task = lc.remap ? xcd * per + slot : (int64_t)blockIdx.x;
  if (task >= lc.total_tasks) return;
  const int run = find_run(p.n_runs, task, [&](int r) { return runs[r].vary_task0; });
  const RunDev& R = runs[run];
  const int64_t local = task - R.vary_task0;
  const int chunk = (int)(local / lc.ogroups);
  const int grp = (int)(local - (int64_t)chunk * lc.ogroups);
  const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, chunk, kChunk);
  if (g.len == kChunk)
    mutate_block_task<T, PREC, true>(R, p, lc, gens, chunk, grp, lane, wave);
  else
    mutate_block_task<T, PREC, false>(R, p, lc, gens, chunk, grp, lane, wave);
}

// k_fitness for every step of a block (grid.y), without the extremes.
__global__ __launch_bounds__(kFitRanges * kFitGroup) void k_block_fitness(const RunDev* __restrict__ runs, Params p,
                                                                           int32_t blocks_per_run, int32_t gens) {
  __shared__ double sh_tr[kFitRanges][kFitGroup];
  __shared__ double sh_te[kFitRanges][kFitGroup];
  const int l = threadIdx.x % kFitGroup;
  const int w = threadIdx.x / kFitGroup;
  const int run = blockIdx.x / blocks_per_run;
  const int i = (blockIdx.x - run * blocks_per_run) * kFitGroup + l;
  const int step = blockIdx.y + 1;
  const RunDev& R = runs[run];
  const bool live = i < p.m;
  const double* part = R.part + (int64_t)(step - 1) * R.nch * p.m + (live ? i : 0);
  const int nt = R.nch_tr, ne = R.nch - R.nch_tr;
  const int a0 = (int)((int64_t)nt * w / kFitRanges), a1 = (int)((int64_t)nt * (w + 1) / kFitRanges);
  const int b0 = nt + (int)((int64_t)ne * w / kFitRanges), b1 = nt + (int)((int64_t)ne * (w + 1) / kFitRanges);
  sh_tr[w][l] = sum_range(part, p.m, a0, a1);
  sh_te[w][l] = sum_range(part, p.m, b0, b1);
  __syncthreads();
  if (threadIdx.x < kFitGroup && live) {
    double s = sh_tr[0][l], st = sh_te[0][l];
#pragma unroll
    for (int q = 1; q < kFitRanges; ++q) {
      s += sh_tr[q][l];
      st += sh_te[q][l];
    }
    const int base = R.state[kStGen];
    step_F(R, p.m, base, gens, step, false)[i] = sqrt(s / (double)R.n_train);
    step_F(R, p.m, base, gens, step, true)[i] = R.n_test > 0 ? sqrt(st / (double)R.n_test) : 0.0;
  }
}

// Survival of one step (k_survive's decision and summary), one block per run.
// Fitness of the individuals that have left their line is formed again from
// their corrected sums first, in k_fitness's order: a wave an individual,
// lanes 0 .. 15 the ranges of the train chunks, 16 .. 31 of the test chunks.
__global__ __launch_bounds__(1024) void k_block_elite(const RunDev* __restrict__ runs, Params p, int32_t gens,
                                                      int32_t step) {
  __shared__ ValIdx sh_lo[16], sh_hi[16];
  const RunDev& R = runs[blockIdx.x];
  BlockState& B = *R.block;
  const int m = p.m, base = B.base, n = B.n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* F = step_F(R, m, base, gens, step, false);
  double* Ft = step_F(R, m, base, gens, step, true);
  for (int j = wave; j < n; j += (int)(blockDim.x >> 6)) {
    const int i = B.who[j];
    const double* part = R.part + (int64_t)(step - 1) * R.nch * m + i;
    const int w = lane & 15;
    const bool test = lane >= 16;
    const int c0 = test ? R.nch_tr : 0, nc = test ? R.nch - R.nch_tr : R.nch_tr;
    double s = 0.0;
    if (lane < 32)
      s = sum_range(part, m, c0 + (int)((int64_t)nc * w / kFitRanges), c0 + (int)((int64_t)nc * (w + 1) / kFitRanges));
    double tr = lane_value(s, 0), te = lane_value(s, 16);
#pragma unroll
    for (int q = 1; q < kFitRanges; ++q) {
      tr += lane_value(s, q);
      te += lane_value(s, 16 + q);
    }
    if (lane == 0) {
      F[i] = sqrt(tr / (double)R.n_train);
      Ft[i] = R.n_test > 0 ? sqrt(te / (double)R.n_test) : 0.0;
    }
  }
  __syncthreads();
  ValIdx lo{INFINITY, 0x7fffffff}, hi{-INFINITY, 0x7fffffff};
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    const ValIdx y{F[i], i};
    lo = pick_min(lo, y);
    hi = pick_max(hi, y);
  }
  lane_extrema<kWave>(lo, hi);
  if (lane == 0) {
    sh_lo[wave] = lo;
    sh_hi[wave] = hi;
  }
  __syncthreads();
  if (wave != 0) return;
  const int q = lane & 15;
  if (q < (int)(blockDim.x >> 6)) {
    lo = sh_lo[q];
    hi = sh_hi[q];
  }
  lane_extrema<16>(lo, hi);  // idle lanes hold wave 0's own
  // fitness is always finite; keep indices in range regardless
  if (lo.i < 0 || lo.i >= m) lo.i = 0;
  if (hi.i < 0 || hi.i >= m) hi.i = 0;
  const gsgp_gen_stats before = R.stats[base + step - 1];
  const int src = uni(before.best_index), dst = uni(hi.i);
  const bool copied = before.best_train_rmse < lo.v;
  gsgp_gen_stats st{lo.v, 0.0, lo.i, copied, copied ? src : -1, copied ? dst : -1};
  int at = -1;
  if (copied) {
    st.best_train_rmse = step_F(R, m, base, gens, step - 1, false)[src];
    st.best_test_rmse = step_F(R, m, base, gens, step - 1, true)[src];
    st.best_index = dst;
    // dst's line from here on: src's up to the step before, the copy, its own
    const int who = lane < n ? B.who[lane] : -1;
    const uint64_t is_src = __builtin_amdgcn_ballot_w64(who == src), is_dst = __builtin_amdgcn_ballot_w64(who == dst);
    const int from = is_src ? __builtin_ctzll(is_src) : -1;
    at = is_dst ? __builtin_ctzll(is_dst) : n;
    const int root = from >= 0 ? B.root[from] : src;
    if (lane >= 1 && lane <= kBlockGens)
      B.by[at][lane] = lane < step ? (from >= 0 ? B.by[from][lane] : src) : lane == step ? -1 : dst;
    if (lane == 0) {
      F[dst] = st.best_train_rmse;
      Ft[dst] = st.best_test_rmse;
      B.root[at] = root;
      B.who[at] = dst;
      if (at == n) B.n = n + 1;
    }
  } else {
    st.best_test_rmse = Ft[lo.i];
  }
  if (lane == 0) {
    B.dst = at;
    R.stats[base + step] = st;
    if (step == gens) R.state[kStGen] = base + gens;
  }
}

// The rest of the block for the row that the step's copy overwrote: one wave
// a chunk forms its values along its line, the squared error sums of the
// steps after the copy, and its values at the end of the block.  Bound by
// latency: lane s reads the draws of the line's step s, so that they are one
// round trip for all steps, and a step's pool rows are read while the step
// before is worked on.  After blocks of 15 of 2,048 individuals on 10,240 cases
// 9.0 -> 6.3 us, of 10,240 on 102,400 10.9 -> 7.5 us.
template <typename T, int PREC, bool FULL>
__device__ __forceinline__ void block_row_chunk(const RunDev& R, const Params& p, int gens, int step, int chunk, int at,
                                                int lane) {
  typedef typename VecOf<T>::type VT;
  constexpr int N = VecOf<T>::N;
  constexpr int kChunk = chunk_cases(sizeof(T));
  constexpr int NJ = kChunk / (kWave * N);
  const BlockState& B = *R.block;
  const int base = uni(B.base), dst = uni(B.who[at]), root = uni(B.root[at]);
  const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, chunk, kChunk);
  const int64_t len = FULL ? (int64_t)kChunk : g.len;
  const T* Sc = (const T*)R.S[base & 1] + (int64_t)p.m * g.cs + (int64_t)root * len;
  T* Oc = (T*)R.S[(base & 1) ^ 1] + (int64_t)p.m * g.cs + (int64_t)dst * len;
  const T* gc = (const T*)R.sigR + (int64_t)p.r * g.cs;
  const T* yv = (const T*)R.y + g.cs;
  VT x[NJ], t[NJ];
  bool ok[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = j * kWave * N + lane * N;
    ok[j] = FULL || e < len;
    x[j] = ok[j] ? gload<VT>(Sc + e) : VT(0);
    t[j] = ok[j] ? gload<VT>(yv + e) : VT(0);
  }
  const int own = lane >= 1 && lane <= gens ? lane : 1;
  const int by = ((const GSGP_GLOBAL int32_t*)B.by[at])[own];
  const GSGP_GLOBAL gsgp_record* rc =
      (const GSGP_GLOBAL gsgp_record*)R.rec + (int64_t)(base + own - 1) * p.m + (by < 0 ? 0 : by);
  const int r1 = rc->r1, r2 = rc->r2;
  const double ms = rc->ms;
  // the steps of the line (a copy's step applies nothing)
  uint64_t left = __builtin_amdgcn_ballot_w64(lane >= 1 && lane <= gens && by >= 0);
  struct Rows {
    VT a[NJ], c[NJ];
    int s;
  };
  auto read = [&](Rows& q) {
    q.s = __builtin_ctzll(left);
    left &= left - 1;
    const T* A = gc + (int64_t)__builtin_amdgcn_readlane(r1, q.s) * len;
    const T* C = gc + (int64_t)__builtin_amdgcn_readlane(r2, q.s) * len;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int e = j * kWave * N + lane * N;
      q.a[j] = ok[j] ? gload<VT>(A + e) : VT(0);
      q.c[j] = ok[j] ? gload<VT>(C + e) : VT(0);
    }
  };
  auto apply = [&](const Rows& q) {
    const T w = (T)lane_value(ms, q.s);
    LaneSse<T, PREC> acc;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      VT v = x[j] + w * (q.a[j] - q.c[j]);
      if constexpr (PREC != GSGP_FP64) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = __builtin_amdgcn_fmed3f(v[k], (T)-kFltMax, (T)kFltMax);
      }
      x[j] = v;
      if (ok[j]) acc.add(v, t[j]);
    }
    if (q.s > step) {
      const double sse = sse_finish<T, PREC, NJ>(acc, ok, x, yv, lane);
      if (lane == 0) R.part[((int64_t)(q.s - 1) * R.nch + chunk) * p.m + dst] = sse;
    }
  };
  Rows q0, q1;
  if (left) {
    read(q0);
    for (;;) {
      const bool more = left != 0;
      if (more) read(q1);
      apply(q0);
      if (!more) break;
      const bool still = left != 0;
      if (still) read(q0);
      apply(q1);
      if (!still) break;
    }
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j)
    if (ok[j]) gstore_nt<VT>(x[j], Oc + j * kWave * N + lane * N);
}

constexpr int kRowWaves = 4;

template <typename T, int PREC>
__global__ __launch_bounds__(kRowWaves * kWave) void k_block_row(const RunDev* __restrict__ runs, Params p, int32_t gens,
                                                                  int32_t step) {
  const int run = find_run(p.n_runs, (int64_t)blockIdx.x, [&](int r) { return (int64_t)runs[r].row_blk0; });
  const RunDev& R = runs[run];
  const int at = uni(R.block->dst);
  const int chunk = (blockIdx.x - R.row_blk0) * kRowWaves + uni(threadIdx.x >> 6);
  if (at < 0 || chunk >= R.nch) return;
  const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, chunk, chunk_cases(sizeof(T)));
  if (g.len == chunk_cases(sizeof(T)))
    block_row_chunk<T, PREC, true>(R, p, gens, step, chunk, at, threadIdx.x & 63);
  else
    block_row_chunk<T, PREC, false>(R, p, gens, step, chunk, at, threadIdx.x & 63);
}

// ---------------------------------------------------------------------------
// Lineage reconstruction helpers (all FP64).
__global__ __launch_bounds__(256) void k_transpose(const double* __restrict__ X, int64_t n, int32_t l,
                                                   double* __restrict__ Xfm, int64_t ld) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ld) return;
  for (int f = 0; f < l; ++f) Xfm[(int64_t)f * ld + c] = c < n ? X[c * l + f] : 0.0;
}

// A recorded step on one case: the parents' values a (and b, crossover) and
// the squashed pool values r1 (and r2, mutation), then the offspring's
// recorded scaling of the local search (never for copies, and skipped when it
// is the identity so that unscaled runs keep their bits).
__device__ __forceinline__ double replay_mutant(const ReplayNode& nd, double a, double r1, double r2) {
  return a + nd.ms * (r1 - r2);
}
__device__ __forceinline__ double replay_mix(double a, double b, double r1) { return a * r1 + b * (1.0 - r1); }
__device__ __forceinline__ bool replay_scaled(const ReplayNode& nd) {
  return nd.op != 2 && (nd.alpha != 0.0 || nd.beta != 1.0);
}

// One generation of a lineage, rows in global memory (for lineages whose
// rows of one generation exceed LDS, see k_replay_lineage).
__global__ __launch_bounds__(256) void k_replay_nodes(const ReplayNode* __restrict__ nodes,
                                                      const double* __restrict__ prev,
                                                      const double* __restrict__ pool,
                                                      double* __restrict__ next, int64_t ld, int64_t n) {
  const ReplayNode nd = nodes[blockIdx.y];
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  double o = prev[(int64_t)nd.a * ld + c];
  if (nd.op != 2) {
    const double r1 = pool[(int64_t)nd.r1 * ld + c];
    o = nd.op == 1 ? replay_mix(o, prev[(int64_t)nd.b * ld + c], r1)
                   : replay_mutant(nd, o, r1, pool[(int64_t)nd.r2 * ld + c]);
  }
  if (replay_scaled(nd)) o = nd.alpha + nd.beta * o;
  next[(int64_t)nd.out * ld + c] = o;
}

// The walk back through the ancestry record from one individual, on one block.
// Thread t has individuals t, t + threads, ...: it reads their records up to
// two generations ahead, and those whose individual matters claim a slot for
// every parent and pool tree met for the first time.  Slots are given in the
// order of the claims: nothing depends on it.  What bounds it is the chain of
// LDS round trips of a generation (slot, claims, count, two barriers).  The
// records of all individuals are read for that, but a list of those that
// matter, whose records are then read, put the latency of that read on the
// chain; so did building the nodes here, which k_lineage_nodes does from the
// slots ([gen + 1][m], then the pool's; none are written without).  A walk over
// 200 generations of 1,024 takes 186 us, over 100 of 128 59 us; with the list
// 382 us, with the list and nodes built on the host 1,800 and 75 us.
template <int K>
__global__ __launch_bounds__(1024) void k_lineage(const gsgp_record* __restrict__ records,
                                                  const gsgp_gen_stats* __restrict__ stats, Params p, int32_t gen,
                                                  int32_t individual, int32_t* __restrict__ begin,
                                                  int32_t* __restrict__ tree0, int32_t* __restrict__ pool,
                                                  int32_t* __restrict__ slots, LineageSummary* __restrict__ out) {
  constexpr int kAhead = K > 4 ? 1 : 2;  // generations in registers
  extern __shared__ int32_t lin[];  // slots of two generations' individuals, then of the pool trees; -1 without
  __shared__ int32_t met[2];
  int32_t* now = lin;
  int32_t* before = lin + p.m;
  int32_t* pslot = lin + 2 * p.m;
  const int t = threadIdx.x, T = blockDim.x;
  for (int i = t; i < 2 * p.m + p.r; i += T) lin[i] = i == individual ? 0 : -1;
  if (t == 0) {
    met[0] = met[1] = 0;
    begin[0] = 0;
  }
  struct Step {
    int copied, src, dst;
    gsgp_record d[K];
  };
  int zero = 0;
  asm("" : "+v"(zero));  // a vector load: a scalar one would be waited for with every LDS access
  auto read = [&](int g) {
    g = g < 1 ? 1 : g;
    const gsgp_gen_stats& s = stats[g + zero];
    Step x;
    x.copied = s.elite_copied;
    x.src = s.elite_src;
    x.dst = s.elite_dst;
    const gsgp_record* rec = records + (int64_t)(g - 1) * p.m;
#pragma unroll
    for (int k = 0; k < K; ++k) x.d[k] = rec[t + k * T < p.m ? t + k * T : 0];
    return x;
  };
  int n = 1, np = 0, total = 0, most = 1;
  auto walk = [&](int g, Step& x) {
    // Up to three claims of an individual: a parent, a pool tree, and one of
    // either.  They are in flight together, and a wave counts the ones that
    // succeeded with one addition (parents in the low half, pool trees in the
    // high half).
    __syncthreads();  // the slots of `now` are complete
    int j[K], first[K], tree[K], second[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = t + k * T;
      j[k] = i < p.m ? now[i] : -1;
      if (slots && i < p.m) slots[(int64_t)g * p.m + i] = j[k];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = t + k * T;
      first[k] = tree[k] = second[k] = 0;
      if (j[k] < 0) continue;
      gsgp_record& d = x.d[k];
      now[i] = -1;
      if (x.copied && i == x.dst) {
        d.op = 2;
        d.p1 = x.src;
      }
      first[k] = atomicCAS(&before[d.p1], -1, -2);
      if (d.op == 2) continue;
      tree[k] = atomicCAS(&pslot[d.r1], -1, -2);
      second[k] = atomicCAS(d.op == 1 ? &before[d.p2] : &pslot[d.r2], -1, -2);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const gsgp_record& d = x.d[k];
      const uint64_t c1 = __ballot(first[k] == -1), c2 = __ballot(second[k] == -1 && d.op == 1);
      const uint64_t q1 = __ballot(tree[k] == -1), q2 = __ballot(second[k] == -1 && d.op == 0);
      const int parents = __popcll(c1) + __popcll(c2), trees = __popcll(q1) + __popcll(q2);
      if (parents + trees == 0) continue;
      int at = 0;
      if (t % kWave == 0) at = atomicAdd(&met[g & 1], parents | trees << 16);
      at = uni(at);
      const uint64_t below = ((uint64_t)1 << (t % kWave)) - 1;
      const int at_parent = at & 0xffff, at_tree = np + (int)((unsigned)at >> 16);
      auto give = [&](bool mine, int q, int to) {
        if (mine) before[q] = to;
      };
      auto give_tree = [&](bool mine, int q, int to) {
        if (mine) {
          pslot[q] = to;
          pool[to] = q;
        }
      };
      give(first[k] == -1, d.p1, at_parent + __popcll(c1 & below));
      give(second[k] == -1 && d.op == 1, d.p2, at_parent + __popcll(c1) + __popcll(c2 & below));
      give_tree(tree[k] == -1, d.r1, at_tree + __popcll(q1 & below));
      give_tree(second[k] == -1 && d.op == 0, d.r2, at_tree + __popcll(q1) + __popcll(q2 & below));
    }
    if (t == 0) met[(g & 1) ^ 1] = 0;
    __builtin_amdgcn_sched_barrier(0);
    x = read(g - kAhead);  // into the same registers: a copy would wait for it
    __builtin_amdgcn_sched_barrier(0);
    total += n;
    if (t == 0) begin[gen - g + 1] = total;
    __syncthreads();
    const int counted = met[g & 1];
    n = counted & 0xffff;
    np += (int)((unsigned)counted >> 16);
    most = most > n ? most : n;
    int32_t* q = now;
    now = before;
    before = q;
  };
  // Generations in pairs and loads in the order of their use, so that each
  // wait is for its own loads only.
  int g = gen;
  if (kAhead == 1 || (g & 1)) {
    Step x = read(g);
    for (; g >= 1 && (kAhead == 1 || (g & 1)); --g) walk(g, x);
  }
  if constexpr (kAhead > 1) {
    Step a = read(g);
    __builtin_amdgcn_sched_barrier(0);
    Step b = read(g - 1);
    __builtin_amdgcn_sched_barrier(0);
    for (; g >= 1; g -= 2) {
      walk(g, a);
      walk(g - 1, b);
    }
  }
  __syncthreads();
  for (int i = t; i < p.m; i += T) {
    if (slots) slots[i] = now[i];
    if (now[i] >= 0) tree0[now[i]] = i;
  }
  if (slots)
    for (int i = t; i < p.r; i += T) slots[(int64_t)(gen + 1) * p.m + i] = pslot[i];
  if (t == 0) *out = LineageSummary{most, n, np, total};
}

// The nodes of a walk, one block a generation: the crossovers first and the
// others last, for the waves of k_replay_lineage to have one kind.
__global__ __launch_bounds__(1024) void k_lineage_nodes(const gsgp_record* __restrict__ records,
                                                        const gsgp_gen_stats* __restrict__ stats,
                                                        const double* __restrict__ ls, int32_t m, int32_t gen,
                                                        const int32_t* __restrict__ begin,
                                                        const int32_t* __restrict__ slots,
                                                        ReplayNode* __restrict__ nodes) {
  __shared__ int32_t front, back;
  const int g = gen - (int)blockIdx.x;
  const int32_t* own = slots + (int64_t)g * m;
  const int32_t* before = own - m;
  const int32_t* pslot = slots + (int64_t)(gen + 1) * m;
  const gsgp_record* rec = records + (int64_t)(g - 1) * m;
  const gsgp_gen_stats s = stats[g];
  if (threadIdx.x == 0) {
    front = begin[gen - g];
    back = begin[gen - g + 1];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    const int j = own[i];
    if (j < 0) continue;
    ReplayNode nd{2, 0, 0, 0, 0, j, 0.0, 0.0, 1.0};
    if (s.elite_copied && i == s.elite_dst) {
      nd.a = before[s.elite_src];
    } else {
      const gsgp_record d = rec[i];
      nd.op = d.op;
      nd.a = before[d.p1];
      nd.r1 = pslot[d.r1];
      if (d.op == 1) {
        nd.b = before[d.p2];
      } else {
        nd.r2 = pslot[d.r2];
        nd.ms = d.ms;
      }
      if (ls) {
        nd.alpha = ls[2 * ((int64_t)g * m + i)];
        nd.beta = ls[2 * ((int64_t)g * m + i) + 1];
      }
    }
    nodes[nd.op == 1 ? atomicAdd(&front, 1) : atomicSub(&back, 1) - 1] = nd;
  }
}

// A whole lineage in one launch.  Cases are independent, so a block takes C
// of them through every generation with the live rows of two generations
// (and, when they fit too, the pool rows) in LDS: [slot][C].  A thread works
// on all C cases of nodes lane, lane + lanes, ....  What bounds it is the chain
// of generations (a barrier and two LDS round trips each) and the bandwidth of
// LDS, so nothing else may be on it: nodes depend on no value and are read
// two generations ahead, and no wait is for more than it has to be. 10,000 cases of 200
// generations with at most 251 live rows: 438 us; 492 with nodes one
// generation ahead, 530 with both operators evaluated and chosen from, 1,435
// with 8 cases a block, one a thread.
template <int C, bool POOL>
__global__ __launch_bounds__(1024) void k_replay_lineage(const ReplayNode* __restrict__ nodes,
                                                         const int32_t* __restrict__ begin, int32_t gen, int32_t n0,
                                                         int32_t np, int32_t slots, int32_t out_slot,
                                                         const double* __restrict__ first,
                                                         const double* __restrict__ pool, int64_t ld, int64_t n,
                                                         double* __restrict__ out) {
  // A row is H pieces of P cases, each in a plane of its own: 16-byte accesses
  // to 16-byte rows reach all banks, to 32-byte rows half of them (2 % slower).
  constexpr int P = C > 1 ? 2 : 1, H = C / P;
  struct alignas(8 * P) Piece {
    double v[P];
  };
  struct Part {
    Piece h[H];
  };
  extern __shared__ __attribute__((aligned(16))) double rows[];  // two generations of slots x C, then the pool's np x C
  const int64_t c0 = (int64_t)blockIdx.x * C;  // ld is a multiple of 64, so c0 + C <= ld
  const int lane = threadIdx.x, lanes = blockDim.x;
  auto get = [](const double* p, int64_t row, int64_t row_step, int64_t plane) {
    Part x;
#pragma unroll
    for (int h = 0; h < H; ++h) x.h[h] = *(const Piece*)(p + row * row_step + h * plane);
    return x;
  };
  auto put = [](double* p, int row, int plane, const Part& x) {
#pragma unroll
    for (int h = 0; h < H; ++h) *(Piece*)(p + row * P + h * plane) = x.h[h];
  };
  const int plane = slots * P, pool_plane = np * P;
  double* cur = rows;
  double* nxt = rows + (int64_t)slots * C;
  double* pl = rows + 2 * (int64_t)slots * C;
  for (int j = lane; j < n0; j += lanes) put(cur, j, plane, get(first + c0, j, ld, P));
  if constexpr (POOL)
    for (int j = lane; j < np; j += lanes) put(pl, j, pool_plane, get(pool + c0, j, ld, P));
  auto pool_at = [&](int r) { return POOL ? get(pl, r, P, pool_plane) : get(pool + c0, r, ld, P); };
  // nodes of generation g: begin[gen - g] .. begin[gen - g + 1] - 1
  const int last = begin[gen] - 1;
  auto node = [&](int q) { return nodes[q < last ? q : last]; };
  // A lane of each wave holds the start of one of 64 generations and moves on
  // by 48: a scalar load would be waited for with every LDS read.
  const int wl = threadIdx.x % kWave;
  constexpr int kMove = kWave - 16;
  auto starts = [&](int g) { return begin[g + wl < gen ? gen - g - wl : 0]; };
  int base = 0, held = starts(0), held_next = starts(kMove);
  auto start = [&](int g) { return __builtin_amdgcn_readlane(held, g - base); };
  struct Ahead {
    int from, end;
    ReplayNode x;
  };
  auto read = [&](int g) {
    const int from = start(g);
    return Ahead{from, start(g - 1), node(from + lane)};
  };
  auto step = [&](const ReplayNode& x) {
    const Part a = get(cur, x.a, P, plane), r1 = x.op == 2 ? a : pool_at(x.r1);
    Part o = a;
    if (x.op == 1) {
      const Part b = get(cur, x.b, P, plane);
#pragma unroll
      for (int v = 0; v < C; ++v)
        o.h[v / P].v[v % P] = replay_mix(a.h[v / P].v[v % P], b.h[v / P].v[v % P], r1.h[v / P].v[v % P]);
    } else if (x.op == 0) {
      const Part r2 = pool_at(x.r2);
#pragma unroll
      for (int v = 0; v < C; ++v)
        o.h[v / P].v[v % P] = replay_mutant(x, a.h[v / P].v[v % P], r1.h[v / P].v[v % P], r2.h[v / P].v[v % P]);
    }
    if (replay_scaled(x)) {
#pragma unroll
      for (int v = 0; v < C; ++v) o.h[v / P].v[v % P] = x.alpha + x.beta * o.h[v / P].v[v % P];
    }
    put(nxt, x.out, plane, o);
  };
  auto generation = [&](int g, Ahead& q) {
    __syncthreads();
    const int from = q.from + lane;
    if (from < q.end) step(q.x);
    if (q.end - q.from > lanes) {
      ReplayNode then = node(from + lanes);
      for (int i = from + lanes; i < q.end; i += lanes) {
        const ReplayNode x = then;
        then = node(i + lanes);
        step(x);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    q = read(g + 2);  // into the same registers: a copy would wait for it
    __builtin_amdgcn_sched_barrier(0);
    double* t = cur;
    cur = nxt;
    nxt = t;
  };
  int g = 1;
  if (gen & 1) {
    Ahead q = read(1);
    generation(g++, q);
  }
  Ahead odd = read(g);
  __builtin_amdgcn_sched_barrier(0);
  Ahead even = read(g + 1);
  __builtin_amdgcn_sched_barrier(0);
  for (; g < gen; g += 2) {
    if (g + 3 - base >= kWave) {
      base += kMove;
      held = held_next;
      held_next = starts(base + kMove);
    }
    generation(g, odd);
    generation(g + 1, even);
  }
  __syncthreads();
  if (lane < C && c0 + lane < n) out[c0 + lane] = cur[out_slot * P + lane / P * plane + lane % P];
}

// ---------------------------------------------------------------------------
// Read-back.  A row of a chunk-tiled buffer lies in one 2 KiB piece per chunk,
// so copying it from the host took a copy call per chunk (about 12 us each).
// These kernels put what a getter returns into one contiguous array in its
// final form; what remains is the transfer to the host.  One row of 125,000
// cases: 3.07 -> 0.10 ms; of 1,250,000: 30.5 -> 0.74 ms; summaries of 64 runs
// 0.64 -> 0.05 ms.

// Elements [e0, e0 + count) of the rows x cases array (row-major, n_cases a
// row) of semantics row0.., case0.. (train cases first, then test cases), as
// FP64; with `ls` (the generation's scaling table, [m][2]) as
// alpha + beta * stored value.  One thread an element: consecutive threads
// read consecutive stored values.
template <typename T>
__global__ __launch_bounds__(256) void k_fetch_semantics(const T* __restrict__ buf, int64_t rows, int64_t tr_pad,
                                                         int64_t te_pad, int32_t nch_tr, int64_t n_train,
                                                         int64_t row0, int64_t case0, int64_t n_cases, int64_t e0,
                                                         int64_t count, const double* __restrict__ ls,
                                                         double* __restrict__ out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= count) return;
  const int64_t e = e0 + q;
  const int64_t i = row0 + e / n_cases;
  const int64_t c = case0 + e % n_cases;
  const int64_t col = c < n_train ? c : tr_pad + (c - n_train);
  double v = (double)buf[tiled_index(tr_pad, te_pad, nch_tr, chunk_cases(sizeof(T)), rows, i, col)];
  if (ls) {
    const double a = ls[2 * i], b = ls[2 * i + 1];
    if (a != 0.0 || b != 1.0) v = a + b * v;
  }
  out[q] = v;
}

// Entries [e0, e0 + count) of the runs x n array of summaries gen0 .. of
// every run from run0 on, as 16-byte halves.
__global__ __launch_bounds__(256) void k_fetch_stats(const RunDev* __restrict__ runs, int32_t run0, int32_t gen0,
                                                     int32_t n, int64_t e0, int64_t count, d2* __restrict__ out) {
  static_assert(sizeof(gsgp_gen_stats) == 2 * sizeof(d2), "a summary is two 16-byte halves");
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= 2 * count) return;
  const int64_t e = e0 + (q >> 1);
  const gsgp_gen_stats* st = runs[run0 + e / n].stats + gen0 + e % n;
  out[q] = ((const d2*)st)[q & 1];
}

// Two arrays of n values one after the other.
__global__ __launch_bounds__(256) void k_fetch_pair(const double* __restrict__ a, const double* __restrict__ b,
                                                    int32_t n, double* __restrict__ out) {
  const int32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  out[q] = a[q];
  out[n + q] = b[q];
}

// Writes one state word of every run (generation counter, replay flags...).
__global__ void k_set_state(const RunDev* __restrict__ runs, int32_t n_runs, int32_t word, int32_t value) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n_runs) runs[r].state[word] = value;
}

// The state words that a restart begins from, in one launch (one launch a
// word cost an initialisation ten).
__global__ void k_reset_state(const RunDev* __restrict__ runs, int32_t n_runs, int32_t* __restrict__ given_up) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < kWideLaunches * 8) given_up[r * kGivenUpStride] = 0;
  if (r >= n_runs) return;
  int32_t* st = runs[r].state;
  st[kStGen] = 0;
  st[kStDone] = 0;
  st[kStReplaySelect] = 0;
  st[kStReplayElite] = 0;
  st[kStMaxDepth] = 0;
  for (int b = 0; b < kLists; ++b) st[kStList0 + b] = 0;
}

}  // namespace

hipError_t launch_fetch_semantics(int32_t precision, const RunDev& R, const void* buf, int64_t rows, int64_t row0,
                                  int64_t case0, int64_t n_cases, int64_t e0, int64_t count, const double* ls,
                                  double* out, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const dim3 grid(blocks_for(count, 256)), block(256);
  if (precision == GSGP_FP64)
    hipLaunchKernelGGL(k_fetch_semantics<double>, grid, block, 0, s, (const double*)buf, rows, R.tr_pad, R.te_pad,
                       R.nch_tr, R.n_train, row0, case0, n_cases, e0, count, ls, out);
  else
    hipLaunchKernelGGL(k_fetch_semantics<float>, grid, block, 0, s, (const float*)buf, rows, R.tr_pad, R.te_pad,
                       R.nch_tr, R.n_train, row0, case0, n_cases, e0, count, ls, out);
  return hipGetLastError();
}

hipError_t launch_fetch_stats(const RunDev* d_runs, int32_t run0, int32_t gen0, int32_t n, int64_t e0, int64_t count,
                              gsgp_gen_stats* out, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fetch_stats, dim3(blocks_for(2 * count, 256)), dim3(256), 0, s, d_runs, run0, gen0, n, e0,
                     count, (d2*)out);
  return hipGetLastError();
}

hipError_t launch_fetch_pair(const double* a, const double* b, int32_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_fetch_pair, dim3(blocks_for(n, 256)), dim3(256), 0, s, a, b, n, out);
  return hipGetLastError();
}

hipError_t launch_set_state(const RunDev* d_runs, int32_t n_runs, int32_t word, int32_t value,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_set_state, dim3(blocks_for(n_runs, 256)), dim3(256), 0, s, d_runs, n_runs, word,
                     value);
  return hipGetLastError();
}

hipError_t launch_reset_state(const RunDev* d_runs, int32_t n_runs, int32_t* given_up, hipStream_t s) {
  hipLaunchKernelGGL(k_reset_state, dim3(blocks_for(n_runs, 256)), dim3(256), 0, s, d_runs, n_runs, given_up);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Launchers.
hipError_t launch_prep(const RunDev* d_runs, const Params& p, int64_t total_cols,
                       const double* const* Xsrc, const double* const* /*unused*/, hipStream_t s) {
  if (total_cols <= 0) return hipSuccess;
  if (p.precision == GSGP_FP64)
    hipLaunchKernelGGL(k_prep<double>, dim3(blocks_for(total_cols, 256)), dim3(256), 0, s, d_runs, p,
                       total_cols, Xsrc);
  else
    hipLaunchKernelGGL(k_prep<float>, dim3(blocks_for(total_cols, 256)), dim3(256), 0, s, d_runs, p,
                       total_cols, Xsrc);
  return hipGetLastError();
}

hipError_t launch_genome(const RunDev* d_runs, const Params& p, hipStream_t s) {
  const int64_t total = (int64_t)p.n_runs * (p.m + p.r) * p.k;
  hipLaunchKernelGGL(k_genome, dim3(blocks_for(total, 256)), dim3(256), 0, s, d_runs, p, total);
  return hipGetLastError();
}

template <typename T, int PREC>
void launch_vary_as(const RunDev* d_runs, const Params& p, const VaryLaunch& lc, bool rows_only, bool one_shot,
                    dim3 grid, dim3 block, hipStream_t s) {
  if (rows_only) {
    if (one_shot)
      hipLaunchKernelGGL((k_vary<T, PREC, true, false, false>), grid, block, 0, s, d_runs, p, lc);
    else
      hipLaunchKernelGGL((k_vary<T, PREC, true, true, false>), grid, block, 0, s, d_runs, p, lc);
  } else if (p.ls) {
    // local search sums are FP64 in every form, so one instance per storage type
    if constexpr (PREC != GSGP_FP32_KAHAN) {
      if (one_shot)
        hipLaunchKernelGGL((k_vary<T, PREC, false, false, true>), grid, block, 0, s, d_runs, p, lc);
      else
        hipLaunchKernelGGL((k_vary<T, PREC, false, true, true>), grid, block, 0, s, d_runs, p, lc);
    } else {
      launch_vary_as<T, GSGP_FP32>(d_runs, p, lc, rows_only, one_shot, grid, block, s);
    }
  } else {
    if (one_shot)
      hipLaunchKernelGGL((k_vary<T, PREC, false, false, false>), grid, block, 0, s, d_runs, p, lc);
    else
      hipLaunchKernelGGL((k_vary<T, PREC, false, true, false>), grid, block, 0, s, d_runs, p, lc);
  }
}

hipError_t launch_vary(const RunDev* d_runs, const Params& p, const VaryLaunch& lc, bool rows_only,
                       hipStream_t s) {
  if (lc.total_tasks <= 0) return hipSuccess;
  const dim3 grid((unsigned)lc.grid), block(lc.waves * kWave);
  // every task in the first sweep of the grid: the loop-free instance
  const int64_t sweep = lc.remap == 2 ? (lc.total_tasks + 8 * (int64_t)lc.ogroups - 1) / (8 * (int64_t)lc.ogroups) *
                                            (8 * (int64_t)lc.ogroups)
                                      : lc.total_tasks;
  const bool one_shot = lc.grid >= sweep;
  switch (p.precision) {
    case GSGP_FP64:
      launch_vary_as<double, GSGP_FP64>(d_runs, p, lc, rows_only, one_shot, grid, block, s);
      break;
    case GSGP_FP32:
      launch_vary_as<float, GSGP_FP32>(d_runs, p, lc, rows_only, one_shot, grid, block, s);
      break;
    default:
      launch_vary_as<float, GSGP_FP32_KAHAN>(d_runs, p, lc, rows_only, one_shot, grid, block, s);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_fitness(const RunDev* d_runs, const Params& p, bool init, hipStream_t s) {
  const int32_t per_run = (p.m + kFitGroup - 1) / kFitGroup;
  const dim3 grid((unsigned)(per_run * p.n_runs)), block(kFitRanges * kFitGroup);
  if (p.ls && !init)
    hipLaunchKernelGGL(k_fitness_ls, grid, block, 0, s, d_runs, p, per_run);
  else
    hipLaunchKernelGGL(k_fitness, grid, block, 0, s, d_runs, p, per_run, init ? 1 : 0);
  return hipGetLastError();
}

// Where k_mutate_slices is faster than k_mutate_block: pool columns beyond an
// XCD's L2 (those just beyond it only in many rounds of blocks), read by a
// population large enough to come back to a slice, and blocks (one a CU) that
// fill their last round of the CUs to three fifths at least.  A generation, us,
// k_mutate_block / slices, at the lines:
//   pool: 10,240 individuals on 25,600 cases, pools of 1,024 rows 20 / 22, of 2,048 43 / 43;
//     10,000 on 40,000, pools of 2,200 189 / 165, of 4,000 271 / 171, of 20,000 444 / 296;
//     5,000 on 5,000, pools of 2,560 26.9 / 31.2, of 4,000 31.7 / 31.6, of 7,000 37.0 / 32.1;
//     pools of 2,200 in 790, 1,264, 1,576 and 1,738 blocks 38.5 / 41.4, 52.6 / 53.5, 66.8 / 71.2,
//     65.9 / 59.6;
//   population: 1,000 on 100,000 cases, pool of 4,000, 87.7 / 81.9; 500, pool of 10,000, 66.8 / 80.4;
//     128 on 6,250, pool of 40,000, 13.4 / 24.5;
//   blocks: 160 (2,000 on 5,000 cases, pool of 4,000) 20.8 / 22.5; 208 24.0 / 23.5; 264
//     (1,400 on 12,000) 26.2 / 30.8; 384 (2,000) 30.6 / 27.5.
// There is no form for FP64 and compensated sums, which would hold twice the
// registers a step.
constexpr size_t kSlicePoolBytes = (size_t)4 << 20;
constexpr size_t kSlicePoolFar = (size_t)11 << 19;
constexpr int64_t kSliceBlocksNear = 1600;  // pools between the two
constexpr int32_t kSliceMaxPool = 1 << 20;  // byte offsets of pool rows are 32 bits
constexpr int32_t kSlicePop = 1000;
constexpr int64_t kSliceBlocks = 200;
constexpr int64_t kCUs = 256;

inline bool slices_pay(const Params& p, int64_t blocks) {
  const size_t pool = (size_t)p.r * kChunkBytes;
  const int64_t rounds = (blocks + kCUs - 1) / kCUs;
  return pool > kSlicePoolBytes && p.r <= kSliceMaxPool && p.m >= kSlicePop &&
         blocks >= (pool > kSlicePoolFar ? kSliceBlocks : kSliceBlocksNear) && 5 * blocks >= 3 * rounds * kCUs;
}

template <typename T, int PREC>
hipError_t launch_block_as(const RunDev* d_runs, const Params& p, const VaryLaunch& lc, int32_t gens,
                           int32_t row_blocks, hipStream_t s) {
  const int64_t draws = (int64_t)p.n_runs * gens * p.m;
  hipLaunchKernelGGL(k_block_draws, dim3(blocks_for(draws, 256)), dim3(256), 0, s, d_runs, p, gens, draws);
  const int32_t groups = (p.m + kSliceGroup - 1) / kSliceGroup;
  const int64_t tasks = lc.total_tasks / lc.ogroups * groups;
  if (PREC == GSGP_FP32 && slices_pay(p, tasks)) {
    const dim3 grid((unsigned)((tasks + 7) / 8 * 8)), block(kSliceWaves * kWave);
    hipLaunchKernelGGL(k_mutate_slices, grid, block, 0, s, d_runs, p, lc, tasks, groups, gens);
  } else {
    hipLaunchKernelGGL((k_mutate_block<T, PREC>), dim3((unsigned)lc.grid), dim3(lc.waves * kWave), 0, s, d_runs, p, lc,
                       gens);
  }
  const int32_t per_run = (p.m + kFitGroup - 1) / kFitGroup;
  hipLaunchKernelGGL(k_block_fitness, dim3((unsigned)(per_run * p.n_runs), (unsigned)gens), dim3(kFitRanges * kFitGroup),
                     0, s, d_runs, p, per_run, gens);
  hipError_t e = hipGetLastError();
  for (int32_t step = 1; step <= gens && e == hipSuccess; ++step) {
    hipLaunchKernelGGL(k_block_elite, dim3((unsigned)p.n_runs), dim3(p.m <= 2048 ? 512 : 1024), 0, s, d_runs, p, gens, step);
    hipLaunchKernelGGL((k_block_row<T, PREC>), dim3((unsigned)row_blocks), dim3(kRowWaves * kWave), 0, s, d_runs, p, gens, step);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_block(const RunDev* d_runs, const Params& p, const VaryLaunch& lc, int32_t gens,
                        int32_t row_blocks, hipStream_t s) {
  if (gens < 1 || gens > kBlockGens || gens % 2 == 0) return hipErrorInvalidValue;
  switch (p.precision) {
    case GSGP_FP64: return launch_block_as<double, GSGP_FP64>(d_runs, p, lc, gens, row_blocks, s);
    case GSGP_FP32: return launch_block_as<float, GSGP_FP32>(d_runs, p, lc, gens, row_blocks, s);
    default: return launch_block_as<float, GSGP_FP32_KAHAN>(d_runs, p, lc, gens, row_blocks, s);
  }
}

hipError_t launch_target_sums(const RunDev* d_runs, const Params& p, hipStream_t s) {
  if (p.precision == GSGP_FP64)
    hipLaunchKernelGGL(k_target_sums<double>, dim3((unsigned)p.n_runs), dim3(256), 0, s, d_runs, p);
  else
    hipLaunchKernelGGL(k_target_sums<float>, dim3((unsigned)p.n_runs), dim3(256), 0, s, d_runs, p);
  return hipGetLastError();
}

hipError_t launch_survive(const RunDev* d_runs, const Params& p, int32_t total_blocks, int mode,
                          hipStream_t s) {
  const dim3 grid(total_blocks), block(256);
  if (p.precision == GSGP_FP64)
    hipLaunchKernelGGL(k_survive<double>, grid, block, 0, s, d_runs, p, total_blocks, mode);
  else
    hipLaunchKernelGGL(k_survive<float>, grid, block, 0, s, d_runs, p, total_blocks, mode);
  return hipGetLastError();
}

hipError_t launch_transpose(const double* X, int64_t n, int32_t l, double* Xfm, int64_t ld,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_transpose, dim3(blocks_for(ld, 256)), dim3(256), 0, s, X, n, l, Xfm, ld);
  return hipGetLastError();
}

hipError_t launch_lineage(const RunDev& R, const Params& p, int32_t gen, int32_t individual, int32_t* begin,
                          int32_t* tree0, int32_t* pool, int32_t* slots, LineageSummary* out, hipStream_t s) {
  const int64_t lds = lineage_lds(p.m, p.r);
  if (lds > kReplayLdsBytes || gen < 1) return hipErrorInvalidValue;
  const dim3 block((unsigned)(p.m < 1024 ? (p.m + kWave - 1) / kWave * kWave : 1024));
  const int k = (p.m + 1023) / 1024;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1), block, (size_t)lds, s, R.rec, R.stats, p, gen, individual, begin, tree0, pool,
                       slots, out);
    return hipGetLastError();
  };
  if (k <= 1) return go(k_lineage<1>);
  if (k <= 2) return go(k_lineage<2>);
  if (k <= 4) return go(k_lineage<4>);
  return k <= kLineagePop / 1024 ? go(k_lineage<kLineagePop / 1024>) : hipErrorInvalidValue;
}

hipError_t launch_lineage_nodes(const RunDev& R, const Params& p, int32_t gen, const int32_t* begin,
                                const int32_t* slots, ReplayNode* nodes, hipStream_t s) {
  const dim3 block((unsigned)(p.m < 1024 ? (p.m + kWave - 1) / kWave * kWave : 1024));
  hipLaunchKernelGGL(k_lineage_nodes, dim3((unsigned)gen), block, 0, s, R.rec, R.stats, p.ls ? R.ls : nullptr, p.m,
                     gen, begin, slots, nodes);
  return hipGetLastError();
}

// Cases per block of k_replay_lineage whose two generations of rows fit in
// LDS, 0 when not even one case's do.  More cases a block read each node less
// often and with more loads in flight.  When nodes were read one generation
// ahead: 532 us for 4, 628 for 2 and 1,147 for 1 (10,000 cases, 200
// generations with at most 251 live rows); 913 for 8, whose rows leave a CU
// one block.  Where every block is resident anyway, fewer have the shorter
// chain: 42, 36 and 35 us for 16 cases.
int replay_cases(int64_t slots, int64_t n) {
  for (int c = n > 512 ? 4 : 2; c >= 1; c >>= 1)
    if (2 * slots * c * (int64_t)sizeof(double) <= kReplayLdsBytes) return c;
  return 0;
}

template <int C>
void launch_replay_lineage_as(bool pool_lds, dim3 grid, dim3 block, size_t shmem, hipStream_t s,
                              const ReplayNode* nodes, const int32_t* begin, int32_t gen, int32_t n0, int32_t np,
                              int32_t slots, int32_t out_slot, const double* first, const double* pool, int64_t ld,
                              int64_t n, double* out) {
  if (pool_lds)
    hipLaunchKernelGGL((k_replay_lineage<C, true>), grid, block, shmem, s, nodes, begin, gen, n0, np, slots, out_slot,
                       first, pool, ld, n, out);
  else
    hipLaunchKernelGGL((k_replay_lineage<C, false>), grid, block, shmem, s, nodes, begin, gen, n0, np, slots, out_slot,
                       first, pool, ld, n, out);
}

hipError_t launch_replay_lineage(const ReplayNode* nodes, const int32_t* begin, int32_t gen, int32_t n0, int32_t np,
                                 int32_t slots, int32_t out_slot, const double* first,
                                 const double* pool, int64_t ld, int64_t n, double* out, hipStream_t s) {
  const int c = replay_cases(slots, n);
  if (c == 0 || gen < 1) return hipErrorInvalidValue;
  size_t shmem = 2 * (size_t)slots * c * sizeof(double);
  const size_t pool_bytes = (size_t)(np > 0 ? np : 1) * c * sizeof(double);  // slot 0 is read where there is none
  const bool pool_lds = shmem + pool_bytes <= (size_t)kReplayLdsBytes;
  if (pool_lds) shmem += pool_bytes;
  // one sweep of the threads per generation where a block may be that large
  const int64_t want = slots;
  const int threads = (int)(want > 1024 ? 1024 : (want + kWave - 1) / kWave * kWave);
  const dim3 block(threads);
  const int64_t most = kMaxThreads / threads * c;  // cases a launch
  hipError_t e = hipSuccess;
  for (int64_t c0 = 0; c0 < n && e == hipSuccess; c0 += most) {
    const int64_t nc = n - c0 < most ? n - c0 : most;
    const dim3 grid((unsigned)((nc + c - 1) / c));
    auto go = [&](auto launch) {
      launch(pool_lds, grid, block, shmem, s, nodes, begin, gen, n0, np, slots, out_slot, first + c0, pool + c0, ld, nc,
             out + c0);
    };
    switch (c) {
      case 4: go(launch_replay_lineage_as<4>); break;
      case 2: go(launch_replay_lineage_as<2>); break;
      default: go(launch_replay_lineage_as<1>); break;
    }
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_replay_nodes(const ReplayNode* nodes, int32_t nnodes, const double* prev,
                               const double* pool, double* next, int64_t ld, int64_t n,
                               hipStream_t s) {
  if (nnodes <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_replay_nodes, dim3(blocks_for(n, 256), (unsigned)nnodes), dim3(256), 0, s, nodes,
                     prev, pool, next, ld, n);
  return hipGetLastError();
}

}  // namespace gsgp
