// The genome compiler and the stack-machine interpreter of libgsgp.so
// (ComputeSemantics of Algorithm 1; Section 2.2 "Interpreter" of the
// GSGP-CUDA paper, arXiv 2106.04034), for gfx950:
//   k_compile         one wave per genome: drops the functions the
//                     interpreter would skip, the pushes after the last
//                     function and the values its result does not use, fuses
//                     each push with a function that directly consumes it,
//                     and gives every op its stack depth and its handler;
//                     k_order files the programs into lists by stack need,
//                     longest first;
//   k_interpret_wide  one wavefront per (program, 256 cases), four cases per
//                     lane, threaded code: the compiled program is
//                     wave-uniform (no divergence), the top three stack values
//                     live in registers and the rest in a lane-strided LDS
//                     column sized for the list;
//   k_interpret       the programs with deeper stacks, LDS columns up to 63
//                     values; k_interpret_spill beyond;
//   k_interpret_list  given programs on new cases (lineage reconstruction).
// This translation unit is built with
// -structurizecfg-skip-uniform-regions: the interpreter dispatches every op
// on wave-uniform bits, and those branches stay plain scalar branches.  The
// other kernels are built without it (it made the variation kernel about
// 0.5 % slower).
#include "device.hpp"

namespace gsgp {
namespace {

// End of a compiled program for eval_program_wide: a push-class word with
// bit 1 set (a push uses only bit 0).
constexpr int32_t kOpEnd = 2;

// Division (the protected division of Section 2.2: a / b where |b| >= 1e-6).
// The FP64 division the compiler emits is a reciprocal estimate refined by
// two Newton-Raphson steps, a quotient, and one correction by its residual,
// all with FMA, inside an operand range scaling and a special-case fix-up.
// When |b| lies in [1e-6, 2^128], |a| >= 2^-700 and the quotient is at most
// FLT_MAX in magnitude (where nothing is clamped), |a| is at most 2^256: no
// operand, reciprocal or quotient comes near either end of the exponent range
// and no two exponents are far apart, so the scaling and the fix-up leave every
// value as it is and the core steps alone (div_recip, div_short) give the same
// bits.  The reciprocal depends on b alone: a constant divisor's is refined once
// for all of a wave's cases, each time the op runs.
constexpr double kDivShortMinDivisor = 1e-6;
constexpr double kDivShortMaxDivisor = 0x1p128;
constexpr double kDivShortMinDividend = 0x1p-700;
constexpr double kDivShortMaxQuotient = kFltMax;

__device__ __forceinline__ double div_recip(double b) {
  double y = __builtin_amdgcn_rcp(b);
  double e = fma(-b, y, 1.0);
  y = fma(y, e, y);
  e = fma(-b, y, 1.0);
  return fma(y, e, y);
}

__device__ __forceinline__ double div_short(double a, double b, double y) {
  const double q = a * y;
  const double r = fma(-b, q, a);
  return fma(r, y, q);
}

// Layout of eval_program_threaded's code: a handler per op kind, and all of
// them once for each of the eight places an op can have in the scalar
// registers.  Byte sizes, in the order of the enum (the assembler checks that
// each handler fits).
enum Handler : int {
  kHFeature = 0,       // + function + 4 x (which of the two feature buffers)
  kHConst = 8,         // add, multiply, divide
  kHPushFeature = 11,  // + stack use (depth before the push 0, 1, 2, deeper) + 4 x buffer
  kHPushConst = 19,    // + stack use
  kHStack = 23,        // + 3 function + stack use: depth before 2, 3, deeper
  kHEnd = 35,
  kHandlers = 36
};
constexpr int kHandlerBytes[kHandlers] = {128, 128, 128, 384, 128, 128, 128, 384,  // feature + - * /
                                          96,  96,  224,                           // constant + * /
                                          96,  96,  128, 160, 96,  96,  128, 160,  // push feature
                                          64,  96,  96,  128,                      // push constant
                                          96,  128, 160, 96,  128, 160,            // stack + -
                                          96,  128, 160, 352, 352, 416,            // stack * /
                                          32};                                     // end
constexpr int handler_offset(int h) {
  int at = 0;
  for (int i = 0; i < h; ++i) at += kHandlerBytes[i];
  return at;
}
constexpr int kHandlerSpan = handler_offset(kHandlers);
struct HandlerTable {
  int32_t at[kHandlers];
};
constexpr HandlerTable make_handlers() {
  HandlerTable t{};
  for (int i = 0; i < kHandlers; ++i) t.at[i] = handler_offset(i);
  return t;
}
__constant__ HandlerTable c_handlers = make_handlers();

// Code offset of the op `w` at entry `at` of its program; buffer: of an op
// that uses a feature, which of the two it finds the feature in.
__device__ __forceinline__ int32_t handler_code(int32_t w, int at, int buffer) {
  const int cls = (w >> 2) & 3, fn = w & 3, d = (w >> 4) & kOpDepthMax;
  int h;
  if (w == kOpEnd)
    h = kHEnd;
  else if (cls == kClsFeature)
    h = kHFeature + fn + 4 * buffer;
  else if (cls == kClsConst)
    h = kHConst + (fn == kFnAdd ? 0 : fn == kFnMul ? 1 : 2);
  else if (cls == kClsPush)
    h = (fn == kPushConst ? kHPushConst : kHPushFeature + 4 * buffer) + (d < 3 ? d : 3);
  else
    h = kHStack + 3 * fn + (d < 4 ? d - 2 : 2);
  return (at & 7) * kHandlerSpan + c_handlers.at[h];
}

// Compile a genome: drop the functions the stack machine would skip (fewer
// than two operands), everything after the last function that runs and the
// values below its result, which nothing reads; fuse each push with the
// function that directly consumes it; and store each op's stack depth so the
// interpreter needs no depth counter.
//
// One wave per genome, 64 genes at a time.  The depth is the only thing that
// depends on the genes before: a push maps depth d to d + 1 and, once a value
// is on the stack, a function maps it to max(d - 1, 1) (skipped at d = 1).
// Both have the form max(d + a, b), which composition keeps, so a scan over
// the lanes gives every gene its depth, and what a gene compiles to depends
// on its neighbours alone:
//   - a function runs when the depth before it is at least 2;
//   - the op before a function that runs is the gene before it (a skipped
//     function leaves depth 1 and a push must follow);
//   - the result of the last function is the top of depth D; the last gene
//     at or before which the depth is D - 1 ends what lies below it.
// One thread per genome walked its genes one by one: 0.7 us a gene whatever
// the population, 90 us for 127 genes and 687 us for 1,023 (4,096 genomes).
// Dropping dead values and not counting fused pushes as stack need shortens
// the interpretation itself: 2,048 programs of 127 genes on 125,000 cases,
// compilation included, 2.19 -> 1.96 ms; 4,096 of 1,023 genes on 10,240 cases
// 3.06 -> 2.24 ms.
constexpr int kCompileWaves = 4;

// Depth after every gene of one chunk: (a, b) of the map max(d + a, b).
struct DepthMap {
  int a, b;
};
constexpr int kNoFloor = -(1 << 20);  // below every depth plus any a

__device__ __forceinline__ DepthMap scan_depth(DepthMap f, int lane) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int a = __shfl_up(f.a, o, kWave), b = __shfl_up(f.b, o, kWave);
    if (lane >= o) {  // f after (a, b)
      f.b = max(b + f.a, f.b);
      f.a += a;
    }
  }
  return f;
}

__device__ __forceinline__ bool is_function(int32_t c) { return c < 0 && c != -5; }

__global__ __launch_bounds__(kCompileWaves * kWave) void k_compile(const RunDev* __restrict__ runs, Params p,
                                                                    int32_t groups) {
  extern __shared__ uint16_t s_depth[];  // depth after every gene, [kCompileWaves][k]
  const int lane = threadIdx.x & 63;
  const int wave = uni(threadIdx.x >> 6);
  const int rows = p.m + p.r;
  const int run = blockIdx.x / groups;
  const int prog = (blockIdx.x - run * groups) * kCompileWaves + wave;
  if (prog >= rows) return;
  const RunDev& R = runs[run];
  const int32_t* code = R.code + (int64_t)prog * p.k;
  const double* cval = R.cval + (int64_t)prog * p.k;
  CompiledOp* ops = R.ops + (int64_t)prog * op_stride(p.k);
  uint16_t* after = s_depth + (int64_t)wave * p.k;

  // depths, the last function that runs, and the deepest stack before it
  int d0 = 0, last = -1, deepest = 0, peak = 0;
  for (int q0 = 0; q0 < p.k; q0 += kWave) {
    const int q = q0 + lane;
    const int32_t c = q < p.k ? code[q] : -1;
    const bool push = q < p.k && !is_function(c);
    // functions before the first push leave the empty stack as it is
    const uint64_t pushes = __builtin_amdgcn_ballot_w64(push);
    const int first = d0 > 0 ? 0 : (pushes ? __builtin_ctzll(pushes) : kWave);
    DepthMap f = push ? DepthMap{1, kNoFloor} : DepthMap{-1, 1};
    if (q >= p.k || lane < first) f = DepthMap{0, kNoFloor};
    f = scan_depth(f, lane);
    const int da = max(d0 + f.a, f.b);
    int db = __shfl_up(da, 1, kWave);
    if (lane == 0) db = d0;
    if (q < p.k) after[q] = (uint16_t)da;
    const uint64_t runs_fn = __builtin_amdgcn_ballot_w64(q < p.k && !push && db >= 2);
    int top = da;  // running maximum over the lanes
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) top = max(top, __shfl_up(top, o, kWave));
    if (runs_fn) {
      const int at = 63 - __builtin_clzll(runs_fn);
      last = q0 + at;
      deepest = max(peak, __shfl(top, at, kWave));
    }
    peak = max(peak, __shfl(top, kWave - 1, kWave));
    d0 = __shfl(da, kWave - 1, kWave);
  }
  last = uni(last);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // `after` is read across lanes from here on

  int n = 0, need = 0;
  if (last >= 0) {
    // what lies below the result ends at the last gene with that depth
    const int base = uni((int)after[last]) - 1;
    int start = 0;
    if (base > 0) {
      for (int q0 = last & ~63;; q0 -= kWave) {
        const int q = q0 + lane;
        const uint64_t at = __builtin_amdgcn_ballot_w64(q < last && (int)after[q] == base);
        if (at) {
          start = q0 + 64 - __builtin_clzll(at);
          break;
        }
        if (q0 == 0) break;
      }
    }
    int live = 0, uses = 0;   // uses: features used so far
    int before = 0;           // entry of the last op that uses a feature (the header before the first)
    for (int q0 = start & ~63; q0 <= last; q0 += kWave) {
      const int q = q0 + lane;
      const bool in = q >= start && q <= last;
      const int32_t c = in ? code[q] : -1;
      const int db = in && q > start ? (int)after[q - 1] : base;
      const bool push = in && !is_function(c);
      const int32_t next = in && q < last ? code[q + 1] : 0;  // 0: a push
      const bool fuse = push && is_function(next) && (int)after[q] >= 2;
      const bool stack = in && !push && db >= 2 && is_function(code[q - 1]);
      const bool feature = push && c != -5;
      const uint64_t below = ((uint64_t)1 << lane) - 1;
      const uint64_t all = __builtin_amdgcn_ballot_w64(push || stack);
      const uint64_t with = __builtin_amdgcn_ballot_w64(feature);
      const int at = 1 + n + __builtin_popcountll(all & below);
      // the entry of the feature use before this lane's
      const uint64_t earlier = with & below;
      const int from = __shfl(at, earlier ? 63 - __builtin_clzll(earlier) : 0, kWave);
      if (push || stack) {
        const int depth = db - base;  // of what is kept; at most k - 1 <= kOpDepthMax
        int32_t w = depth << 4;
        if (stack) {
          w |= (kClsStack << 2) | (-1 - c);
        } else if (fuse) {
          // push b, then op(a, b) with a the value below it: one op on the
          // top of the stack; a - c is compiled as a + (-c)
          const int fn = !feature && -1 - next == kFnSub ? kFnAdd : -1 - next;
          w |= ((feature ? kClsFeature : kClsConst) << 2) | fn;
        } else {
          w |= (kClsPush << 2) | (feature ? kPushFeature : kPushConst);
          live = max(live, depth + 1);
        }
        if (feature) {
          w |= c << 16;
          // this row's byte offset in a tile of X, for the op that reads ahead
          const int64_t row = (int64_t)c * kXTile * (int64_t)sizeof(double);
          ops[earlier ? from : before].value = __longlong_as_double((long long)row);
        } else if (push) {
          ops[at].value = fuse && -1 - next == kFnSub ? -cval[q] : cval[q];
        }
        ops[at].word = w;
        ops[at].code = handler_code(w, at, (uses + __builtin_popcountll(earlier)) & 1);
      }
      if (with) before = __shfl(at, 63 - __builtin_clzll(with), kWave);
      uses += __builtin_popcountll(with);
      n += __builtin_popcountll(all);
    }
    if (lane == 0) ops[before].value = 0.0;  // nothing to read ahead
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) live = max(live, __shfl_xor(live, o, kWave));
    // the top two values live in registers; a fused push takes no room
    need = live > 2 ? live - 2 : 0;
  }
  if (lane == 0) {
    R.nops[prog] = n;
    // the header (its row is written above) and the end word: a program with a
    // valid function has a push fused into one, so n <= k - 1 and both stay in
    // the program's entries
    ops[0].code = 0;
    ops[0].word = kOpEnd;
    if (n == 0) ops[0].value = 0.0;
    ops[n + 1] = CompiledOp{handler_code(kOpEnd, n + 1, 0), kOpEnd, 0.0};
    R.need[prog] = need;
    // the deepest stack of the genome as it is written, up to its last
    // function: a bound on every need, and what a checkpoint is checked with.
    // One atomic a genome costs too much on one address: most find the word
    // at their value already.
    if (deepest > __hip_atomic_load(&R.state[kStMaxDepth], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&R.state[kStMaxDepth], deepest);
  }
}

// Files each run's programs into the stack-need lists (one list after the
// other in R.lists), each list in order
// of decreasing length (a counting sort on kOrderBins length bins, one block
// per run): the long programs of a case block start first and the launch
// ends on short ones (3.5 % faster at the Section 3.1 shape).  The order
// within a bin is arbitrary; semantics do not depend on it.
constexpr int kOrderBins = 256;
__global__ __launch_bounds__(1024) void k_order(const RunDev* __restrict__ runs, Params p, int shift) {
  __shared__ int32_t at[kLists * kOrderBins];
  __shared__ int32_t total[kLists];
  const RunDev& R = runs[blockIdx.x];
  const int rows = p.m + p.r;
  auto key = [&](int prog, int& list) {
    list = list_of(R.need[prog]);
    return list * kOrderBins + ((p.k - R.nops[prog]) >> shift);
  };
  for (int i = threadIdx.x; i < kLists * kOrderBins; i += blockDim.x) at[i] = 0;
  __syncthreads();
  for (int prog = threadIdx.x; prog < rows; prog += blockDim.x) {
    int list;
    atomicAdd(&at[key(prog, list)], 1);
  }
  __syncthreads();
  if (threadIdx.x < kLists) {  // bin counts to first positions in the list
    int32_t* h = at + threadIdx.x * kOrderBins;
    int32_t sum = 0;
    for (int j = 0; j < kOrderBins; ++j) {
      const int32_t c = h[j];
      h[j] = sum;
      sum += c;
    }
    total[threadIdx.x] = sum;
    R.state[kStList0 + threadIdx.x] = sum;
  }
  __syncthreads();
  for (int prog = threadIdx.x; prog < rows; prog += blockDim.x) {
    int list, slot = 0;
    const int bin = key(prog, list);
    for (int b = 0; b < list; ++b) slot += total[b];
    slot += atomicAdd(&at[bin], 1);
    R.lists[slot] = prog;
  }
}

// Evaluate one compiled program on V cases per lane (Section 2.2
// "Interpreter").  The op stream is wave-uniform and read with scalar loads,
// eight ops (two 64-byte lines) a batch.  Stack element i of depth d (0 =
// bottom) lives in registers for the top two (tos = d-1, nos = d-2) and in LDS
// below them, at stk[(i * V + v) * 64 + lane]; a function of the top two values
// reads its new second operand from LDS only after it has produced its result,
// so the LDS latency falls outside the op's dependency chain.  A fused op (a
// push the next function consumes) applies the function to tos and the
// terminal and touches neither nos nor LDS.  The value of the program is the
// output of its last function (the Out register), 0.0 if none runs.
// This form serves the list interpreter (programs on a caller's cases): X is
// feature-major in global memory, row stride ld, and a feature op's index
// sits in its op word.
typedef GSGP_LDS double* LdsStack;        // stack column in LDS
typedef GSGP_GLOBAL double* GlobalStack;  // stack column in the workspace (spill pass)

template <int V, typename Stack>
__device__ __forceinline__ void eval_program(const CompiledOp* ops, int n, const double* X,
                                             int64_t ld, const int64_t (&col)[V], const bool (&ok)[V],
                                             Stack stk, int lane, double (&out)[V]) {
  constexpr int kBatch = kOpPad;
  const GSGP_CONST CompiledOp* cops = (const GSGP_CONST CompiledOp*)ops;
  double tos[V], nos[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    tos[v] = 0.0;
    nos[v] = 0.0;
  }
  // lanes past the last column read the last column instead (no exec-mask
  // branches around the loads); their values are never stored
  int64_t at[V];
#pragma unroll
  for (int v = 0; v < V; ++v) at[v] = ok[v] ? col[v] : ld - 1;
  auto feature = [&](int w, double (&x)[V]) {
    const GSGP_GLOBAL double* xg = (const GSGP_GLOBAL double*)X + (int64_t)((uint32_t)w >> 16) * ld;
#pragma unroll
    for (int v = 0; v < V; ++v) x[v] = xg[at[v]];
  };
  for (int j0 = 0; j0 < n; j0 += kBatch) {
    int wv[kBatch];
    double cv[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      // one contiguous batch (two 64-byte lines); the last batch of a program
      // may read up to kBatch - 1 ops past it, which the buffer's padding
      // after the last program keeps in bounds, and never uses them
      wv[u] = cops[j0 + u].word;
      cv[u] = cops[j0 + u].value;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (j0 + u >= n) break;
      const int w = wv[u];
      const int cls = (w >> 2) & 3;
      const int fn = w & 3;
      const int d = (w >> 4) & kOpDepthMax;  // stack depth before the op
      if (cls == kClsPush) {
        if (d >= 2) {
#pragma unroll
          for (int v = 0; v < V; ++v) stk[((d - 2) * V + v) * kWave + lane] = nos[v];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) nos[v] = tos[v];
        if (fn == kPushFeature) {
          feature(w, tos);
        } else {
#pragma unroll
          for (int v = 0; v < V; ++v) tos[v] = cv[u];
        }
      } else {
        // op(a, b): b is the top of the stack (or the fused terminal), a the
        // value below it (or the top of the stack).  The two forms are
        // separate call sites of `apply`, so neither first copies its
        // operands into a common pair of registers.
        // Every operand is finite (finite features and constants, results
        // clamped here, protected division), so min/max clamp exactly as a
        // compare-and-select would.  The clamp sits in each branch, on the
        // arithmetic result itself, where the compiler knows the value needs
        // no NaN canonicalisation before min/max.
        auto clamp = [](double x) { return fmin(fmax(x, -kFltMax), kFltMax); };
        auto apply = [&](const double (&a)[V], const double (&b)[V]) {
          if (fn == kFnAdd) {
#pragma unroll
            for (int v = 0; v < V; ++v) tos[v] = clamp(a[v] + b[v]);
          } else if (fn == kFnSub) {
#pragma unroll
            for (int v = 0; v < V; ++v) tos[v] = clamp(a[v] - b[v]);
          } else if (fn == kFnMul) {
#pragma unroll
            for (int v = 0; v < V; ++v) tos[v] = clamp(a[v] * b[v]);
          } else {
#pragma unroll
            for (int v = 0; v < V; ++v) {
              // protected division without a per-lane branch: the quotient
              // of a safe denominator is kept only where |b| >= 1e-6, and
              // there it is a / b
              const bool tiny = fabs(b[v]) < 1e-6;
              const double q = a[v] / (tiny ? 1.0 : b[v]);
              tos[v] = clamp(tiny ? 1.0 : q);
            }
          }
        };
        if (cls == kClsStack) {
          double t0[V];
#pragma unroll
          for (int v = 0; v < V; ++v) t0[v] = tos[v];
          apply(nos, t0);
        } else {
          double x[V], t0[V];
#pragma unroll
          for (int v = 0; v < V; ++v) t0[v] = tos[v];
          if (cls == kClsFeature) {
            feature(w, x);
          } else {
#pragma unroll
            for (int v = 0; v < V; ++v) x[v] = cv[u];
          }
          apply(t0, x);
        }
        if (cls == kClsStack && d >= 3) {
#pragma unroll
          for (int v = 0; v < V; ++v) nos[v] = stk[((d - 3) * V + v) * kWave + lane];
        }
      }
    }
  }
#pragma unroll
  for (int v = 0; v < V; ++v) out[v] = tos[v];
}

// eval_program over the handle's X for V cases per lane, with every limit
// tested where it applies: the programs with deep stacks, and those that
// eval_program_threaded leaves.
//   - Dispatch tests single bits of the op word: bit 3 a function applied
//     to the top of the stack and a terminal (fused op), else bit 2 a
//     function of the top two values, else a push; bit 1 multiplication or
//     division, bit 0 subtraction or division (or, for a push, a constant).
//   - Features are read through a buffer resource over the block's tile: the
//     scalar offset is the row's offset and each lane's fixed 32-bit byte
//     offset (its pair of cases) is the vector offset, so a feature load takes
//     no vector address arithmetic.
//   - Both function forms share one `apply` (tos = f(tos, b)): a function of
//     the top two values first moves them into place.
//   - The program ends at its end word (kOpEnd), tested only on the push
//     path, instead of a count compared before every op.
//   - REG = 1 keeps a third stack value (n2, element d - 3) in registers as
//     well, so that a program needs one LDS value per lane fewer (the LDS
//     column is what bounds the resident waves of the deeper lists).
// The FP64 operations and their order are those of eval_program, so results
// are the same bits.
template <int V, int REG, int BATCH = kOpPad, typename Stack>
__device__ __forceinline__ void eval_program_wide(const CompiledOp* ops, const double* X, bool short_feature_div,
                                                  const uint32_t (&off)[V], Stack stk, int lane, double (&out)[V]) {
  static_assert(REG == 0 || REG == 1, "two or three stack values in registers");
  constexpr int kBatch = BATCH;
  const GSGP_CONST CompiledOp* cops = (const GSGP_CONST CompiledOp*)ops;
  double tos[V], nos[V], n2[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    tos[v] = 0.0;
    nos[v] = 0.0;
    n2[v] = 0.0;
  }
  // raw buffer over X: no stride, num_records at the largest offset, and the
  // third descriptor word of a plain dword buffer on gfx9-family parts
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)X, (short)0, 0x7fffffff, 0x00020000);
  // cases v and v + 1 (v even) of a lane are adjacent: one 16-byte load.
  // The vector memory unit, busy nearly all the time here, costs about the
  // same per instruction for 8 or 16 bytes a lane, so pairs halve its time
  // (10 % faster at the Section 3.1 shape with 127 genes, 14 % with 2,047).
  auto feature = [&](int w, double (&x)[V]) {
    const int row = (int)((uint32_t)w >> 16) * (kXTile * (int)sizeof(double));  // the row's byte offset in the tile
#pragma unroll
    for (int v = 0; v < V; v += 2) {
      typedef double double2v __attribute__((ext_vector_type(2)));
      const double2v t = __builtin_bit_cast(double2v, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)off[v], row, 0));
      x[v] = t.x;
      x[v + 1] = t.y;
    }
  };
  auto clamp = [](double x) { return fmin(fmax(x, -kFltMax), kFltMax); };
  // The clamp changes nothing where |x| <= FLT_MAX: one compare per case,
  // and the min/max only when some case of the wave needs them (NaN, which
  // finite operands never produce, takes them too).
  auto settle = [&]() {
    uint64_t out_of_range = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) out_of_range |= __builtin_amdgcn_ballot_w64(!(fabs(tos[v]) <= kFltMax));
    if (out_of_range) {
#pragma unroll
      for (int v = 0; v < V; ++v) tos[v] = clamp(tos[v]);
    }
  };
  auto divide_full = [&](const double (&b)[V]) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const bool tiny = fabs(b[v]) < 1e-6;  // protected division, as in eval_program
      const double q = tos[v] / (tiny ? 1.0 : b[v]);
      tos[v] = clamp(tiny ? 1.0 : q);
    }
  };
  // The short division (div_short): taken when every case of the wave has
  // |b| >= 1e-6 (with y its reciprocal refinement), |tos| >= 2^-700 and a
  // quotient of at most FLT_MAX, where it gives the bits of the full one.
  auto divide = [&](const double (&b)[V], const double (&y)[V], uint64_t bad) {
    double q[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      q[v] = div_short(tos[v], b[v], y[v]);
      bad |= __builtin_amdgcn_ballot_w64(!(fabs(tos[v]) >= kDivShortMinDividend)) |
             __builtin_amdgcn_ballot_w64(!(fabs(q[v]) <= kDivShortMaxQuotient));
    }
    if (bad) {
      divide_full(b);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) tos[v] = q[v];
    }
  };
  // a divisor from the registers: every case refines its own reciprocal
  auto divide_by = [&](const double (&b)[V]) {
    double y[V];
    uint64_t bad = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      y[v] = div_recip(b[v]);
      bad |= __builtin_amdgcn_ballot_w64(!(fabs(b[v]) >= kDivShortMinDivisor));
    }
    divide(b, y, bad);
  };
  auto arith = [&](int w, const double (&b)[V]) {
    if (w & 2) {
#pragma unroll
      for (int v = 0; v < V; ++v) tos[v] = tos[v] * b[v];
    } else if (w & 1) {
#pragma unroll
      for (int v = 0; v < V; ++v) tos[v] = tos[v] - b[v];
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) tos[v] = tos[v] + b[v];
    }
    settle();
  };
  for (int j0 = 0;; j0 += kBatch) {
    int wv[kBatch];
    double cv[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      // a batch of eight is two 64-byte lines; reads past a program's end
      // word stay inside the buffer's padding and are never used
      wv[u] = cops[j0 + u].word;
      cv[u] = cops[j0 + u].value;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int w = wv[u];
      if (w & 8) {  // fused: tos = f(tos, terminal)
        double b[V];
        if (w & 4) {
#pragma unroll
          for (int v = 0; v < V; ++v) b[v] = cv[u];
          if ((w & 3) != kFnDiv) {
            arith(w, b);
          } else if (fabs(cv[u]) >= kDivShortMinDivisor && fabs(cv[u]) <= kDivShortMaxDivisor) {
            // the constant's reciprocal, once for all cases
            const double y1 = div_recip(cv[u]);
            double y[V];
#pragma unroll
            for (int v = 0; v < V; ++v) y[v] = y1;
            divide(b, y, 0);
          } else {
            divide_full(b);
          }
        } else {
          feature(w, b);
          if ((w & 3) != kFnDiv)
            arith(w, b);
          else if (short_feature_div)
            divide_by(b);
          else
            divide_full(b);
        }
      } else if (w & 4) {  // tos = f(nos, tos), then the new nos from LDS
        double b[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
          b[v] = tos[v];
          tos[v] = nos[v];
        }
        // b is the output of a function, so |b| <= FLT_MAX
        if ((w & 3) != kFnDiv)
          arith(w, b);
        else
          divide_by(b);
        const int d = (w >> 4) & kOpDepthMax;
        if constexpr (REG == 0) {
          if (d >= 3) {
#pragma unroll
            for (int v = 0; v < V; ++v) nos[v] = stk[((d - 3) * V + v) * kWave + lane];
          }
        } else {
#pragma unroll
          for (int v = 0; v < V; ++v) nos[v] = n2[v];
          if (d >= 4) {
#pragma unroll
            for (int v = 0; v < V; ++v) n2[v] = stk[((d - 4) * V + v) * kWave + lane];
          }
        }
      } else {  // push: the lowest register value to LDS, the rest down one, the terminal to tos
        if (w & 2) goto done;  // kOpEnd
        const int d = (w >> 4) & kOpDepthMax;
        if constexpr (REG == 0) {
          if (d >= 2) {
#pragma unroll
            for (int v = 0; v < V; ++v) stk[((d - 2) * V + v) * kWave + lane] = nos[v];
          }
        } else {
          if (d >= 3) {
#pragma unroll
            for (int v = 0; v < V; ++v) stk[((d - 3) * V + v) * kWave + lane] = n2[v];
          }
#pragma unroll
          for (int v = 0; v < V; ++v) n2[v] = nos[v];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) nos[v] = tos[v];
        if (w & 1) {
#pragma unroll
          for (int v = 0; v < V; ++v) tos[v] = cv[u];
        } else {
          feature(w, tos);
        }
      }
    }
  }
done:
#pragma unroll
  for (int v = 0; v < V; ++v) out[v] = tos[v];
}

// The interpreter of the stack-need lists: one wave, a program, four cases per
// lane.  Written as threaded code in assembly, because what bounded the
// compiled form (eval_program_wide) was not the arithmetic but everything
// around it: per op about 20 scalar instructions and 7 branches (a taken branch
// waits for its instructions), copies where the paths of an op meet again, a
// wait for the next ops' scalar loads every eighth op, and the tests below; the
// vector unit was 70 % busy with twice the instructions the values need.
//   - An op's `code` is the offset of its handler; a handler ends by adding the
//     next op's to the table's address and jumping there (one branch an op).
//   - Ops are read four at a time (a 64-byte line) into two sets of scalar
//     registers: one set is read while the other's ops run.  An op therefore
//     has one of eight places, with a copy of the handlers for each.
//   - An op that uses a feature finds it in one of two buffers and starts the
//     load of the next such op's feature into the other one, so a row's
//     latency is spent on the ops in between.
//   - Three stack values live in registers, at fixed ones; the compile step
//     knows the depth, so a handler moves only the values that exist and
//     touches the LDS column only when it must.
//   - Nothing is tested inside the program.  The clamp, the protected division
//     and the short division's limits are decided by values that almost never
//     come near them (1 % of random programs of 127 genes on 20 features meet
//     one on some case of a tile, 2-4 % of 1,023 to 2,047 genes).  Three running
//     extremes are kept per lane and tested at the end; when they say that some
//     step may have been outside its limits, the caller runs the program again
//     with eval_program_wide:
//       mx   largest |function result|: below FLT_MAX nothing would be clamped,
//            and a quotient below it is inside the short division's limit;
//       mnb  smallest |divisor|: at least 1e-6, so no division is protected (a
//            constant divisor counts in mx too, as no other bound holds for it);
//       mna  smallest |dividend|: at least 2^-700.
//     They are taken of the values' high words read as FP32, two values an
//     instruction: for finite values below 2^1017 the order is that of the
//     values, and the first result past FLT_MAX is at most 2^256 (operands
//     inside the limits), or infinite or NaN where a constant is larger.
//     What follows it may be anything, so the extremes must never recover:
//     v_maximum3 / v_minimum3 (IEEE 754-2019) keep a NaN, and the tests are
//     written so that NaN fails.  Callers use this only where no feature
//     exceeds 2^128.
// The operations and their order are those of eval_program_wide (a - c is
// compiled as a + (-c)), so results are the same bits.  Every load is waited
// for inside the block.  What bounds it now is the vector unit (86 % busy; 324
// of about 500 instructions a program of 127 genes are its ops).  Whole
// interpretation, compiled form -> this -> with the launches and the padding of
// now: 2,048 programs of 127 genes on 125,000 cases 1.94 -> 1.61 -> 1.33 ms,
// 1,250,000 cases 17.3 -> 14.6 -> 14.5 ms, 20,480 on 102,400 cases x 1,024 features
// 14.6 -> 12.4 -> 12.3 ms, 64 runs 2.89 -> 2.51 -> 2.0 ms, 256 programs on 700
// cases 80 -> 54 -> 29 us (one launch for all lists).  Handlers that load each feature
// where they use it were within 3 % either way (20 features 2 % slower, 1,024
// features 3 % faster).
//
// Registers: s[36:67] the entries of places 0 .. 7 (code, word, value), s[68:71]
// the buffer over the X tile, s[72:73] the table, s[74:75] the jump target,
// s[76:77] the program, s78 scratch, s79 the LDS column less three slots;
// v[8:15] top of the stack, v[16:23] the value below it, v[24:31] the third,
// v[32:39] and v[64:71] the feature buffers, v[40:55] scratch, v56-v58 mx, mnb,
// mna, v59 16 bytes times the lane: its first pair of cases in an X row (the
// second is 1,024 bytes on) and in an LDS slot; v62 scratch.
constexpr uint32_t kMaxHigh = 0x47EFFFFFu;       // high word of FLT_MAX as FP64
constexpr uint32_t kDivisorHigh = 0x3EB0C6F7u;   // of 1e-6: at or below, not sure to be at least 1e-6
constexpr uint32_t kDividendHigh = 0x14300000u;  // of 2^-700
constexpr int kThreadedV = 4;
constexpr int kThreadedReg = 1;  // stack values in registers beyond the top two
constexpr int kSlotBytes = kThreadedV * kWave * (int)sizeof(double);
static_assert(kSlotBytes == 2048, "the handlers shift depths by 11 bits");

// clang-format off
#define GSGP_THREADED_MACROS \
  /* at the first op of each set, the other set's next ops */ \
  ".macro GSGP_PRE p\n" \
  ".if \\p == 0\n s_load_dwordx16 s[52:67], s[76:77], 64\n .endif\n" \
  ".if \\p == 4\n s_add_u32 s76, s76, 128\n s_addc_u32 s77, s77, 0\n s_load_dwordx16 s[36:51], s[76:77], 0\n .endif\n" \
  ".endm\n" \
  /* on to the next op; the last op of a set waits for the other set */ \
  ".macro GSGP_GO p\n" \
  ".if (\\p & 3) == 3\n s_waitcnt lgkmcnt(0)\n .endif\n" \
  "s_add_u32 s74, s72, s[36+((\\p+1)&7)*4]\n s_addc_u32 s75, s73, 0\n s_setpc_b64 s[74:75]\n" \
  ".endm\n" \
  ".macro GSGP_FEATURE r, p\n" \
  "buffer_load_dwordx4 v[\\r:\\r+3], v59, s[68:71], s[38+\\p*4] offen\n" \
  "buffer_load_dwordx4 v[\\r+4:\\r+7], v59, s[68:71], s[38+\\p*4] offen offset:1024\n" \
  ".endm\n" \
  ".macro GSGP_MAX\n v_maximum3_f32 v56, v56, |v9|, |v11|\n v_maximum3_f32 v56, v56, |v13|, |v15|\n .endm\n" \
  ".macro GSGP_MIN m, r\n v_minimum3_f32 v\\m, v\\m, |v[\\r+1]|, |v[\\r+3]|\n v_minimum3_f32 v\\m, v\\m, |v[\\r+5]|, |v[\\r+7]|\n .endm\n" \
  ".macro GSGP_MOV to, from\n" \
  "v_mov_b64_e32 v[\\to:\\to+1], v[\\from:\\from+1]\n v_mov_b64_e32 v[\\to+2:\\to+3], v[\\from+2:\\from+3]\n" \
  "v_mov_b64_e32 v[\\to+4:\\to+5], v[\\from+4:\\from+5]\n v_mov_b64_e32 v[\\to+6:\\to+7], v[\\from+6:\\from+7]\n" \
  ".endm\n" \
  /* top = a op b on four cases; op: an instruction of two operands */ \
  ".macro GSGP_OP op, a, b, neg\n" \
  "\\op v[8:9], v[\\a:\\a+1], \\neg\\()v[\\b:\\b+1]\n \\op v[10:11], v[\\a+2:\\a+3], \\neg\\()v[\\b+2:\\b+3]\n" \
  "\\op v[12:13], v[\\a+4:\\a+5], \\neg\\()v[\\b+4:\\b+5]\n \\op v[14:15], v[\\a+6:\\a+7], \\neg\\()v[\\b+6:\\b+7]\n" \
  ".endm\n" \
  ".macro GSGP_FMA d, a, b, c, na\n" \
  "v_fma_f64 v[\\d:\\d+1], \\na\\()v[\\a:\\a+1], v[\\b:\\b+1], v[\\c:\\c+1]\n v_fma_f64 v[\\d+2:\\d+3], \\na\\()v[\\a+2:\\a+3], v[\\b+2:\\b+3], v[\\c+2:\\c+3]\n" \
  "v_fma_f64 v[\\d+4:\\d+5], \\na\\()v[\\a+4:\\a+5], v[\\b+4:\\b+5], v[\\c+4:\\c+5]\n v_fma_f64 v[\\d+6:\\d+7], \\na\\()v[\\a+6:\\a+7], v[\\b+6:\\b+7], v[\\c+6:\\c+7]\n" \
  ".endm\n" \
  ".macro GSGP_ERR d, b, y\n" /* d = 1 - b y */ \
  "v_fma_f64 v[\\d:\\d+1], -v[\\b:\\b+1], v[\\y:\\y+1], 1.0\n v_fma_f64 v[\\d+2:\\d+3], -v[\\b+2:\\b+3], v[\\y+2:\\y+3], 1.0\n" \
  "v_fma_f64 v[\\d+4:\\d+5], -v[\\b+4:\\b+5], v[\\y+4:\\y+5], 1.0\n v_fma_f64 v[\\d+6:\\d+7], -v[\\b+6:\\b+7], v[\\y+6:\\y+7], 1.0\n" \
  ".endm\n" \
  /* top = a / b (div_recip and div_short), with r free for the residual */ \
  ".macro GSGP_DIV a, b, r\n" \
  "v_rcp_f64_e32 v[40:41], v[\\b:\\b+1]\n v_rcp_f64_e32 v[42:43], v[\\b+2:\\b+3]\n" \
  "v_rcp_f64_e32 v[44:45], v[\\b+4:\\b+5]\n v_rcp_f64_e32 v[46:47], v[\\b+6:\\b+7]\n" \
  "GSGP_MIN 57, \\b\n GSGP_MIN 58, \\a\n" \
  "GSGP_ERR 48, \\b, 40\n GSGP_FMA 40, 40, 48, 40\n GSGP_ERR 48, \\b, 40\n GSGP_FMA 40, 40, 48, 40\n" \
  "v_mul_f64 v[48:49], v[\\a:\\a+1], v[40:41]\n v_mul_f64 v[50:51], v[\\a+2:\\a+3], v[42:43]\n" \
  "v_mul_f64 v[52:53], v[\\a+4:\\a+5], v[44:45]\n v_mul_f64 v[54:55], v[\\a+6:\\a+7], v[46:47]\n" \
  "GSGP_FMA \\r, \\b, 48, \\a, -\n GSGP_FMA 8, \\r, 40, 48\n" \
  "GSGP_MAX\n" \
  ".endm\n" \
  /* the third value to its LDS slot, from an op at depth d >= 3 */ \
  ".macro GSGP_SPILL p\n" \
  "s_bfe_u32 s78, s[37+\\p*4], 0xc0004\n s_lshl_b32 s78, s78, 11\n s_add_u32 s78, s78, s79\n v_add_u32_e32 v62, s78, v59\n" \
  "ds_write_b128 v62, v[24:27]\n ds_write_b128 v62, v[28:31] offset:1024\n" \
  ".endm\n" \
  /* after a function of the top two at a depth above 3: the rest move up */ \
  ".macro GSGP_FILL p\n GSGP_MOV 16, 24\n" \
  "s_bfe_u32 s78, s[37+\\p*4], 0xc0004\n s_lshl_b32 s78, s78, 11\n s_add_u32 s78, s78, s79\n" \
  "s_add_u32 s78, s78, 0xfffff800\n v_add_u32_e32 v62, s78, v59\n" \
  "ds_read_b128 v[24:27], v62\n ds_read_b128 v[28:31], v62 offset:1024\n s_waitcnt lgkmcnt(0)\n" \
  ".endm\n" \
  ".macro GSGP_AT at\n .org GSGP_TABLE%= + \\at\n .endm\n"

#define GSGP_THREADED_PLACE \
  ".macro GSGP_PLACE p, at\n" \
  /* feature in v32: + - * / */ \
  "GSGP_AT \\at+0\n GSGP_PRE \\p\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_OP v_add_f64, 8, 32\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+128\n GSGP_PRE \\p\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_OP v_add_f64, 8, 32, -\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+256\n GSGP_PRE \\p\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_OP v_mul_f64, 8, 32\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+384\n GSGP_PRE \\p\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_DIV 8, 32, 8\n GSGP_GO \\p\n" \
  /* feature in v64: + - * / */ \
  "GSGP_AT \\at+768\n GSGP_PRE \\p\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_OP v_add_f64, 8, 64\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+896\n GSGP_PRE \\p\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_OP v_add_f64, 8, 64, -\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+1024\n GSGP_PRE \\p\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_OP v_mul_f64, 8, 64\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+1152\n GSGP_PRE \\p\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_DIV 8, 64, 8\n GSGP_GO \\p\n" \
  /* constant: + * / */ \
  "GSGP_AT \\at+1536\n GSGP_PRE \\p\n GSGP_OPC v_add_f64, \\p\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+1632\n GSGP_PRE \\p\n GSGP_OPC v_mul_f64, \\p\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+1728\n GSGP_PRE \\p\n GSGP_DIVC \\p\n GSGP_GO \\p\n" \
  /* push of the feature in v32 at depth 0, 1, 2, deeper */ \
  "GSGP_AT \\at+1952\n GSGP_PRE \\p\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 32\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+2048\n GSGP_PRE \\p\n GSGP_MOV 16, 8\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 32\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+2144\n GSGP_PRE \\p\n GSGP_MOV 24, 16\n GSGP_MOV 16, 8\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 32\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+2272\n GSGP_PRE \\p\n GSGP_SPILL \\p\n GSGP_MOV 24, 16\n GSGP_MOV 16, 8\n GSGP_FEATURE 64, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 32\n GSGP_GO \\p\n" \
  /* push of the feature in v64 at depth 0, 1, 2, deeper */ \
  "GSGP_AT \\at+2432\n GSGP_PRE \\p\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 64\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+2528\n GSGP_PRE \\p\n GSGP_MOV 16, 8\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 64\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+2624\n GSGP_PRE \\p\n GSGP_MOV 24, 16\n GSGP_MOV 16, 8\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 64\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+2752\n GSGP_PRE \\p\n GSGP_SPILL \\p\n GSGP_MOV 24, 16\n GSGP_MOV 16, 8\n GSGP_FEATURE 32, \\p\n s_waitcnt vmcnt(2)\n GSGP_MOV 8, 64\n GSGP_GO \\p\n" \
  /* push of a constant */ \
  "GSGP_AT \\at+2912\n GSGP_PRE \\p\n GSGP_CONST \\p\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+2976\n GSGP_PRE \\p\n GSGP_MOV 16, 8\n GSGP_CONST \\p\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+3072\n GSGP_PRE \\p\n GSGP_MOV 24, 16\n GSGP_MOV 16, 8\n GSGP_CONST \\p\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+3168\n GSGP_PRE \\p\n GSGP_SPILL \\p\n GSGP_MOV 24, 16\n GSGP_MOV 16, 8\n GSGP_CONST \\p\n GSGP_GO \\p\n" \
  /* function of the top two values at depth 2, 3, deeper: + - * / */ \
  "GSGP_AT \\at+3296\n GSGP_PRE \\p\n GSGP_OP v_add_f64, 16, 8\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+3392\n GSGP_PRE \\p\n GSGP_OP v_add_f64, 16, 8\n GSGP_MAX\n GSGP_MOV 16, 24\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+3520\n GSGP_PRE \\p\n GSGP_OP v_add_f64, 16, 8\n GSGP_MAX\n GSGP_FILL \\p\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+3680\n GSGP_PRE \\p\n GSGP_OP v_add_f64, 16, 8, -\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+3776\n GSGP_PRE \\p\n GSGP_OP v_add_f64, 16, 8, -\n GSGP_MAX\n GSGP_MOV 16, 24\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+3904\n GSGP_PRE \\p\n GSGP_OP v_add_f64, 16, 8, -\n GSGP_MAX\n GSGP_FILL \\p\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+4064\n GSGP_PRE \\p\n GSGP_OP v_mul_f64, 16, 8\n GSGP_MAX\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+4160\n GSGP_PRE \\p\n GSGP_OP v_mul_f64, 16, 8\n GSGP_MAX\n GSGP_MOV 16, 24\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+4288\n GSGP_PRE \\p\n GSGP_OP v_mul_f64, 16, 8\n GSGP_MAX\n GSGP_FILL \\p\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+4448\n GSGP_PRE \\p\n GSGP_DIV 16, 8, 16\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+4800\n GSGP_PRE \\p\n GSGP_DIV 16, 8, 16\n GSGP_MOV 16, 24\n GSGP_GO \\p\n" \
  "GSGP_AT \\at+5152\n GSGP_PRE \\p\n GSGP_DIV 16, 8, 16\n GSGP_FILL \\p\n GSGP_GO \\p\n" \
  /* end: what is in flight is waited for and not used */ \
  "GSGP_AT \\at+5568\n s_waitcnt vmcnt(0) lgkmcnt(0)\n s_branch GSGP_DONE%=\n" \
  ".endm\n" \
  ".macro GSGP_OPC op, p\n" \
  "\\op v[8:9], v[8:9], s[38+\\p*4:39+\\p*4]\n \\op v[10:11], v[10:11], s[38+\\p*4:39+\\p*4]\n" \
  "\\op v[12:13], v[12:13], s[38+\\p*4:39+\\p*4]\n \\op v[14:15], v[14:15], s[38+\\p*4:39+\\p*4]\n" \
  ".endm\n" \
  ".macro GSGP_CONST p\n" \
  "v_mov_b64_e32 v[8:9], s[38+\\p*4:39+\\p*4]\n v_mov_b64_e32 v[10:11], s[38+\\p*4:39+\\p*4]\n" \
  "v_mov_b64_e32 v[12:13], s[38+\\p*4:39+\\p*4]\n v_mov_b64_e32 v[14:15], s[38+\\p*4:39+\\p*4]\n" \
  ".endm\n" \
  /* top / constant: the reciprocal once for all cases */ \
  ".macro GSGP_DIVC p\n" \
  "v_rcp_f64_e32 v[40:41], s[38+\\p*4:39+\\p*4]\n" \
  "v_minimum3_f32 v57, v57, |s[39+\\p*4]|, |s[39+\\p*4]|\n v_maximum3_f32 v56, v56, |s[39+\\p*4]|, |s[39+\\p*4]|\n GSGP_MIN 58, 8\n" \
  "v_fma_f64 v[42:43], -s[38+\\p*4:39+\\p*4], v[40:41], 1.0\n v_fma_f64 v[40:41], v[40:41], v[42:43], v[40:41]\n" \
  "v_fma_f64 v[42:43], -s[38+\\p*4:39+\\p*4], v[40:41], 1.0\n v_fma_f64 v[40:41], v[40:41], v[42:43], v[40:41]\n" \
  "v_mul_f64 v[48:49], v[8:9], v[40:41]\n v_mul_f64 v[50:51], v[10:11], v[40:41]\n" \
  "v_mul_f64 v[52:53], v[12:13], v[40:41]\n v_mul_f64 v[54:55], v[14:15], v[40:41]\n" \
  "v_fma_f64 v[8:9], -s[38+\\p*4:39+\\p*4], v[48:49], v[8:9]\n v_fma_f64 v[10:11], -s[38+\\p*4:39+\\p*4], v[50:51], v[10:11]\n" \
  "v_fma_f64 v[12:13], -s[38+\\p*4:39+\\p*4], v[52:53], v[12:13]\n v_fma_f64 v[14:15], -s[38+\\p*4:39+\\p*4], v[54:55], v[14:15]\n" \
  "v_fma_f64 v[8:9], v[8:9], v[40:41], v[48:49]\n v_fma_f64 v[10:11], v[10:11], v[40:41], v[50:51]\n" \
  "v_fma_f64 v[12:13], v[12:13], v[40:41], v[52:53]\n v_fma_f64 v[14:15], v[14:15], v[40:41], v[54:55]\n" \
  "GSGP_MAX\n" \
  ".endm\n"

#define GSGP_THREADED_PURGE \
  ".purgem GSGP_PRE\n .purgem GSGP_GO\n .purgem GSGP_FEATURE\n .purgem GSGP_MAX\n .purgem GSGP_MIN\n .purgem GSGP_MOV\n" \
  ".purgem GSGP_OP\n .purgem GSGP_FMA\n .purgem GSGP_ERR\n .purgem GSGP_DIV\n .purgem GSGP_SPILL\n .purgem GSGP_FILL\n" \
  ".purgem GSGP_AT\n .purgem GSGP_PLACE\n .purgem GSGP_OPC\n .purgem GSGP_CONST\n .purgem GSGP_DIVC\n"
// clang-format on

static_assert(kHandlerSpan == 5600 && handler_offset(kHConst) == 1536 && handler_offset(kHPushFeature) == 1952 &&
                  handler_offset(kHPushConst) == 2912 && handler_offset(kHStack) == 3296 &&
                  handler_offset(kHEnd) == 5568,
              "GSGP_PLACE places the handlers where the compile step sends them");

// Evaluates one program on a wave's four cases per lane; false when some step
// may have been outside the limits (out is then not the program's value).
__device__ __forceinline__ bool eval_program_threaded(const CompiledOp* ops, const double* X, uint32_t lane16,
                                                      LdsStack stk, double (&out)[kThreadedV]) {
  typedef int int4v __attribute__((ext_vector_type(4)));
  const uint64_t x = (uint64_t)(uintptr_t)X;
  // raw buffer over the tile, as in eval_program_wide
  int4v rsrc = {(int)(uint32_t)x, (int)((uint32_t)(x >> 32) & 0xffffu), 0x7fffffff, 0x00020000};
  const GSGP_CONST CompiledOp* at = (const GSGP_CONST CompiledOp*)ops;
  const uint32_t column = (uint32_t)(uintptr_t)stk - 3u * kSlotBytes;
  float mx, mnb, mna;
  asm volatile(
      GSGP_THREADED_MACROS GSGP_THREADED_PLACE
      "s_load_dwordx16 s[36:51], s[76:77], 0\n"
      "s_getpc_b64 s[72:73]\n"
      "GSGP_PC%=:\n"
      "s_add_u32 s72, s72, GSGP_TABLE%=-GSGP_PC%=\n"
      "s_addc_u32 s73, s73, 0\n"
      "v_mov_b64_e32 v[8:9], 0\n v_mov_b64_e32 v[10:11], 0\n v_mov_b64_e32 v[12:13], 0\n v_mov_b64_e32 v[14:15], 0\n"
      "v_mov_b32_e32 v56, 0\n v_mov_b32_e32 v57, 0x7f000000\n v_mov_b32_e32 v58, 0x7f000000\n"
      "s_waitcnt lgkmcnt(0)\n"
      /* the header: the first feature's load, the second set of entries */
      "GSGP_FEATURE 32, 0\n"
      "GSGP_PRE 0\n"
      "GSGP_GO 0\n"
      ".p2align 6\n"
      "GSGP_TABLE%=:\n"
      "GSGP_PLACE 0, 0\n GSGP_PLACE 1, 5600\n GSGP_PLACE 2, 11200\n GSGP_PLACE 3, 16800\n"
      "GSGP_PLACE 4, 22400\n GSGP_PLACE 5, 28000\n GSGP_PLACE 6, 33600\n GSGP_PLACE 7, 39200\n"
      "GSGP_DONE%=:\n" GSGP_THREADED_PURGE
      : "=&{v[8:9]}"(out[0]), "=&{v[10:11]}"(out[1]), "=&{v[12:13]}"(out[2]), "=&{v[14:15]}"(out[3]),
        "=&{v56}"(mx), "=&{v57}"(mnb), "=&{v58}"(mna), "+&{s[76:77]}"(at)
      : "{s[68:71]}"(rsrc), "{v59}"(lane16), "{s79}"(column)
      : "memory", "scc", "s36", "s37", "s38", "s39", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48",
        "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63",
        "s64", "s65", "s66", "s67", "s72", "s73", "s74", "s75", "s78", "v16", "v17", "v18", "v19", "v20", "v21",
        "v22", "v23", "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", "v36",
        "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", "v48", "v49", "v50", "v51",
        "v52", "v53", "v54", "v55", "v62", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71");
  const bool fine = mx < __uint_as_float(kMaxHigh) && mnb > __uint_as_float(kDivisorHigh) &&
                    mna >= __uint_as_float(kDividendHigh);
  return __builtin_amdgcn_ballot_w64(!fine) == 0;
}

constexpr int kInterpV = 2;              // cases per lane
constexpr int kInterpTile = kWave * kInterpV;  // cases per block
static_assert(kInterpTile == kInterpCases, "the runtime plans kInterpCases-case blocks");
// Position of a stack-need list's first program in R.lists.
__device__ __forceinline__ int list_start(const RunDev& R, int list) {
  int at = 0;
  for (int b = 0; b < list; ++b) at += uni(cload(&R.state[kStList0 + b]));
  return at;
}

// Hardware dispatch sends block b of a grid of n to XCD b % 8.  Interpreter
// blocks are numbered case block by case block; xcd_block gives each XCD a
// contiguous range of them, so the CUs of one XCD work on the same X tile
// and each tile is read into one XCD's L2, not into all eight.
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t n) {
  const int64_t x = b & 7, i = b >> 3, q = n >> 3, rem = n & 7;
  return x * q + (x < rem ? x : rem) + i;
}

// The cases of a lane in a block of 64 x V cases starting at case `first`
// (a multiple of 64 x V inside one X tile): lane l owns cases 2l and 2l + 1
// (and, for V = 4, 128 + 2l and 129 + 2l), so that each pair is one 16-byte
// load; off[v] is the case's byte offset in its row of the X tile.
template <int V>
__device__ __forceinline__ void lane_cases(int64_t first, int lane, int64_t ld, int64_t (&col)[V], bool (&ok)[V],
                                           uint32_t (&off)[V]) {
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int c = (v >> 1) * (2 * kWave) + 2 * lane + (v & 1);
    col[v] = first + c;
    ok[v] = col[v] < ld;
    off[v] = (uint32_t)((first % kXTile + c) * sizeof(double));
  }
}

// Writes one program's values for one case block: population rows as they
// are, pool rows squashed by the logistic function (the random functions R_u
// of GSM, Section 2); padding columns as exact zeros.
template <typename T, int V>
__device__ __forceinline__ void store_program(const RunDev& R, const Params& p, int prog, const int64_t (&col)[V],
                                              const bool (&ok)[V], const double (&out)[V]) {
  const bool pool = prog >= p.m;
  T* dst = pool ? (T*)R.sigR : (T*)R.S[0];
  const int64_t nrows = pool ? p.r : p.m;
  const int64_t row = pool ? prog - p.m : prog;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    if (!ok[v]) continue;
    const int64_t c = col[v];
    const bool real = c < R.n_train || (c >= R.tr_pad && c < R.tr_pad + R.n_test);
    double val = out[v];
    if (pool) val = 1.0 / (1.0 + exp(-val));
    dst[tiled_index(R.tr_pad, R.te_pad, R.nch_tr, chunk_cases(sizeof(T)), nrows, row, c)] = real ? (T)val : (T)0;
  }
}

// Where 128 neighbouring columns from `first` on (a lane's pair v, v + 1 of a
// block) lie in the chunk-tiled buffers: row 0 of the population and of the
// pool there, and the distance of rows.  Computed once for all programs of a
// wave: the general form costs about 25 vector instructions a value.
template <typename T>
struct StoreSpan {
  T *pop, *pool;
  uint32_t len;
  bool whole;  // the span lies in one chunk and holds real cases only
};

template <typename T>
__device__ __forceinline__ StoreSpan<T> store_span(const RunDev& R, const Params& p, int64_t first) {
  constexpr int64_t kChunk = chunk_cases(sizeof(T));
  const bool train = first < R.tr_pad;
  const int64_t c = train ? first / kChunk : R.nch_tr + (first - R.tr_pad) / kChunk;
  const ChunkGeom g = chunk_geom(R.tr_pad, R.te_pad, R.nch_tr, (int32_t)c, kChunk);
  const int64_t end = first + 2 * kWave;
  return StoreSpan<T>{(T*)R.S[0] + p.m * g.cs + (first - g.cs), (T*)R.sigR + p.r * g.cs + (first - g.cs), (uint32_t)g.len,
                      end <= g.cs + g.len && end <= (train ? R.n_train : R.tr_pad + R.n_test)};
}

// The logistic function 1 / (1 + e^-v) of a wave's values, by the short
// division where every divisor is within its limits (1 + e^-v is at least 1).
template <int V>
__device__ __forceinline__ void squash(double (&x)[V]) {
  uint64_t far = 0;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    x[v] = 1.0 + exp(-x[v]);
    far |= __builtin_amdgcn_ballot_w64(!(x[v] <= kDivShortMaxDivisor));
  }
  if (far) {
#pragma unroll
    for (int v = 0; v < V; ++v) x[v] = 1.0 / x[v];
  } else {
#pragma unroll
    for (int v = 0; v < V; ++v) x[v] = div_short(1.0, x[v], div_recip(x[v]));
  }
}

// store_program for half a block of the wide kernel: a lane's pair a, b of
// columns first + 2 lane and the next.
template <typename T>
__device__ __forceinline__ void store_pair(const RunDev& R, const Params& p, bool pool, uint32_t row, int64_t first,
                                           const StoreSpan<T>& sp, int lane, double a, double b) {
  if (sp.whole) {
    typedef T pair __attribute__((ext_vector_type(2)));
    T* to = (pool ? sp.pool : sp.pop) + (uint64_t)row * sp.len;
    *(GSGP_GLOBAL pair*)(to + 2 * lane) = pair{(T)a, (T)b};
    return;
  }
  // the last spans of a segment; `lane` hidden so that nothing of this is
  // prepared ahead of the programs
  asm("" : "+v"(lane));
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int64_t c = first + 2 * lane + e;
    if (c >= R.ld) continue;
    const bool real = c < R.n_train || (c >= R.tr_pad && c < R.tr_pad + R.n_test);
    T* dst = pool ? (T*)R.sigR : (T*)R.S[0];
    dst[tiled_index(R.tr_pad, R.te_pad, R.nch_tr, chunk_cases(sizeof(T)), pool ? p.r : p.m, row, c)] =
        real ? (T)(e ? b : a) : (T)0;
  }
}

// ComputeSemantics(P) and ComputeSemantics(R) (Algorithm 1) of the last list's
// programs that fit an LDS column of `slots` values: a block takes 128 cases of
// one run, each of its waves a program.  Pool rows are squashed by the logistic
// function (the random functions R_u of GSM, Section 2) before storage.
// Padding columns are written as exact zeros.
template <typename T>
__global__ __launch_bounds__(256) void k_interpret(const RunDev* __restrict__ runs, Params p, int32_t pgroups,
                                                   int slots) {
  extern __shared__ double lds[];
  const int lane = threadIdx.x & 63;
  const int wave = uni(threadIdx.x >> 6);
  const int W = blockDim.x >> 6;
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t cbg = blk / pgroups;  // case block over all runs
  const int pg = (int)(blk - cbg * pgroups);
  const int run = find_run(p.n_runs, cbg, [&](int r) { return runs[r].cblk0; });
  const RunDev& R = runs[run];
  const int64_t cb = cbg - R.cblk0;
  const int idx = pg * W + wave;
  if (idx >= uni(cload(&R.state[kStList0 + kLists - 1]))) return;
  double* stk = lds + wave * slots * kInterpV * kWave;
  const int64_t first = cb * kInterpTile;
  int64_t col[kInterpV];
  bool ok[kInterpV];
  uint32_t off[kInterpV];
  lane_cases<kInterpV>(first, lane, R.ld, col, ok, off);
  const int prog = uni(cload(&R.lists[list_start(R, kLists - 1) + idx]));
  // this pass takes the programs that need at most `slots`
  if (uni(cload(&R.need[prog])) > slots) return;
  double out[kInterpV];
  eval_program_wide<kInterpV, 0>(R.ops + (int64_t)prog * op_stride(p.k) + 1, R.X + (first / kXTile) * R.l * kXTile,
                              uni(R.x_big) == 0, off, (LdsStack)stk, lane, out);
  store_program<T, kInterpV>(R, p, prog, col, ok, out);
}

// ComputeSemantics of the other lists: a block of one wave takes one tile of X
// (256 cases of one run, four a lane) and per_wave programs, one after the
// other, of the lists list0 .. list1, with an LDS column for the deepest of
// them.  One wave per block: a block's LDS and slot are released as soon as its
// programs are done, where four waves of unequal programs held them until the
// longest ended.  Programs whose values left the limits of the threaded code
// are run again at the end.  Lanes past the last case read the tile's padding
// and are never stored.
//
// A program that the threaded code gives up has cost more than the checked
// evaluator alone (1.25 times the threaded one's time), so on data where that is
// the rule (columns with zeros, features so large that products are clamped)
// the rest of a launch does without it: once kGivenUpLeast programs were given
// up and they are more than one in kGivenUpShare of those started,
// kStopThreaded is set.  Each XCD counts for itself (blocks b % 8), in a cache
// line of its own and at a scope that its L2 serves; every wave reads the count
// with a scalar load, whose small cache the ops turn over quickly.  A stale
// count costs time and changes no result.  (One count for all, read past the
// L2s, doubled a launch of 500,000 waves; read through the vector cache it went
// unseen.)  kGivenUpLeast is several tiles' worth, as zeros may sit in a few
// tiles only.  Initialisation of 2,048 programs of 127 genes on 125,000 cases of 20
// features, us: all features 0 or 1 3,718 -> 2,481, three of them 2,928 -> 2,156;
// without the threaded code 2,759 and 2,452.  Of features in [-1, 1] 1,795 -> 1,754.
// The checked evaluator keeps two stack values in registers where the column
// holds the rest, else three: 6 % faster than three always (fewer copies).  The
// second form reads two ops at a time, a quarter of the code: with both unrolled
// eight times the kernel came to 112 KB, close to what a branch can span (128 KB;
// 90 KB now), and beyond it without the optimisations of the normal build.
constexpr int32_t kGivenUpLeast = 1024;
constexpr int32_t kGivenUpShare = 4;
constexpr int32_t kStopThreaded = 1 << 30;
static_assert(kXTile == 4 * kWave && kXTile % kInterpTile == 0, "interpreter case blocks lie inside one X tile");
static_assert(65535LL * kXTile * sizeof(double) < (1LL << 31), "a tile of the most features the runtime accepts "
                                                                  "takes 32-bit buffer offsets");

template <typename T>
__global__ __launch_bounds__(kWave, 7) void k_interpret_wide(const RunDev* __restrict__ runs, Params p, int32_t pgroups,
                                                             int32_t per_wave, int list0, int list1, int slots,
                                                             int32_t* __restrict__ given_up) {
  constexpr int V = kThreadedV, REG = kThreadedReg;
  constexpr int kTile = kWave * V;
  static_assert(kTile == kXTile, "a block's cases are one tile of X");
  extern __shared__ double lds[];
  const int lane = threadIdx.x & 63;
  given_up += (blockIdx.x & 7) * kGivenUpStride;
  const int32_t seen = cload(given_up);
  const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t cbg = (uint32_t)blk / (uint32_t)pgroups;  // case block over all runs
  const int pg = (int)(blk - cbg * pgroups);
  const int run = find_run(p.n_runs, cbg, [&](int r) { return runs[r].cblk0w; });
  const RunDev& R = runs[run];
  const int start = list_start(R, list0);
  int count = 0;
  for (int b = list0; b <= list1; ++b) count += uni(cload(&R.state[kStList0 + b]));
  if (pg * per_wave >= count) return;
  const int64_t cb = cbg - R.cblk0w;
  const int64_t first = cb * kTile;  // the block's first case
  const uint32_t off0 = (uint32_t)lane * 2 * sizeof(double);
  const StoreSpan<T> near = store_span<T>(R, p, first), far = store_span<T>(R, p, first + 2 * kWave);
  auto store = [&](int prog, double (&out)[V]) {
    const bool pool = prog >= p.m;
    const uint32_t row = (uint32_t)(pool ? prog - p.m : prog);
    if (pool) squash<V>(out);
    store_pair<T>(R, p, pool, row, first, near, lane, out[0], out[1]);
    store_pair<T>(R, p, pool, row, first + 2 * kWave, far, lane, out[2], out[3]);
  };
  const double* X = R.X + cb * R.l * kXTile;
  const int32_t* progs = R.lists + start + pg * per_wave;
  const int n = count - pg * per_wave < per_wave ? count - pg * per_wave : per_wave;
  uint32_t again = (uint32_t)((1ull << n) - 1);  // programs left to eval_program_wide
  const int32_t before = uni(seen);
  if (uni(R.x_big) == 0 && before < kStopThreaded) {
    for (int j = 0; j < n; ++j) {
      const int prog = uni(cload(&progs[j]));
      double out[V];
      if (!eval_program_threaded(R.ops + (int64_t)prog * op_stride(p.k), X, off0, (LdsStack)lds, out)) continue;
      store(prog, out);
      again &= ~(1u << j);
    }
    if (again && lane == 0) {
      const int32_t far =
          __hip_atomic_fetch_add(given_up, __builtin_popcount(again), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (far >= kGivenUpLeast && far < kStopThreaded &&
          (int64_t)far * kGivenUpShare > (int64_t)(blockIdx.x >> 3) * per_wave)
        __hip_atomic_fetch_or(given_up, kStopThreaded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  while (again) {
    const int j = __builtin_ctz(again);
    again &= again - 1;
    const int prog = uni(cload(&progs[j]));
    const CompiledOp* ops = R.ops + (int64_t)prog * op_stride(p.k) + 1;
    const uint32_t off[V] = {off0, 0, off0 + 2 * kWave * (uint32_t)sizeof(double), 0};
    double out[V];
    if (uni(cload(&R.need[prog])) <= slots)
      eval_program_wide<V, 0>(ops, X, uni(R.x_big) == 0, off, (LdsStack)lds, lane, out);
    else
      eval_program_wide<V, REG, 2>(ops, X, uni(R.x_big) == 0, off, (LdsStack)lds, lane, out);
    store(prog, out);
  }
}

// Last pass: the programs of the last list whose stack exceeds the largest
// LDS column (need > kMaxLdsSlots).  kSpillWaves waves, one per block, each own
// a column of `slots` x kInterpV x 64 doubles in `spill` (lane-strided as in
// LDS, so every stack access is one coalesced 512-byte row) and sweep the
// (program, case block) tasks of every run in turn.
template <typename T>
__global__ __launch_bounds__(64) void k_interpret_spill(const RunDev* __restrict__ runs, Params p, double* spill,
                                                        int slots) {
  const int lane = threadIdx.x & 63;
  const int w = blockIdx.x;
  double* stk = spill + (int64_t)w * slots * kInterpV * kWave;
  for (int run = 0; run < p.n_runs; ++run) {
    const RunDev& R = runs[run];
    const int cnt = uni(cload(&R.state[kStList0 + kLists - 1]));
    const int32_t* list = R.lists + list_start(R, kLists - 1);
    const int64_t cblocks = (R.ld + kInterpTile - 1) / kInterpTile;
    const int64_t tasks = (int64_t)cnt * cblocks;
    for (int64_t t = w; t < tasks; t += gridDim.x) {
      const int j = (int)(t / cblocks);
      const int64_t cb = t - (int64_t)j * cblocks;
      const int prog = uni(cload(&list[j]));
      const int need = uni(cload(&R.need[prog]));
      if (need <= kMaxLdsSlots || need > slots) continue;  // LDS passes took it; never beyond the column
      const int64_t first = cb * kInterpTile;
      int64_t col[kInterpV];
      bool ok[kInterpV];
      uint32_t off[kInterpV];
      lane_cases<kInterpV>(first, lane, R.ld, col, ok, off);
      double out[kInterpV];
      eval_program_wide<kInterpV, 0>(R.ops + (int64_t)prog * op_stride(p.k) + 1, R.X + (first / kXTile) * R.l * kXTile,
                                  uni(R.x_big) == 0, off, (GlobalStack)stk, lane, out);
      store_program<T, kInterpV>(R, p, prog, col, ok, out);
    }
  }
}

// ---------------------------------------------------------------------------
// One (program, 128-case block) task of the list interpreter: the n0
// generation-0 trees (as they are, to out0[j][ld]) and then the np pool trees
// (squashed by the logistic, to outp[j][ld]) of a lineage on cases of the
// feature-major Xfm.
struct ListArgs {
  const CompiledOp* ops;
  const int32_t* nops;
  int32_t k, m;
  const int32_t *tree0, *pool;
  int32_t n0, np;
  const double* Xfm;
  int64_t ld, n;
  double *out0, *outp;
};

template <typename Stack>
__device__ __forceinline__ void list_task(const ListArgs& a, int64_t task, Stack stk, int lane) {
  const int nprog = a.n0 + a.np;
  const int64_t cb = task / nprog;
  const int j = (int)(task - cb * nprog);
  const bool sq = j >= a.n0;
  const int pr = uni(sq ? a.m + a.pool[j - a.n0] : a.tree0[j]);
  int64_t col[kInterpV];
  bool ok[kInterpV];
#pragma unroll
  for (int v = 0; v < kInterpV; ++v) {
    col[v] = cb * (kWave * kInterpV) + v * kWave + lane;
    ok[v] = col[v] < a.ld;
  }
  double val[kInterpV];
  eval_program<kInterpV>(a.ops + (int64_t)pr * op_stride(a.k) + 1, uni(a.nops[pr]), a.Xfm, a.ld, col, ok, stk, lane, val);
  double* out = sq ? a.outp + (int64_t)(j - a.n0) * a.ld : a.out0 + (int64_t)j * a.ld;
#pragma unroll
  for (int v = 0; v < kInterpV; ++v) {
    if (!ok[v]) continue;
    double x = val[v];
    if (sq) x = 1.0 / (1.0 + exp(-x));
    out[col[v]] = col[v] < a.n ? x : 0.0;
  }
}

__global__ __launch_bounds__(256) void k_interpret_list(ListArgs a, int slots, int64_t task0, int64_t total) {
  extern __shared__ double lds[];
  const int lane = threadIdx.x & 63;
  const int wave = uni(threadIdx.x >> 6);
  const int64_t task = task0 + (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
  if (task >= total) return;
  double* stk = lds + wave * slots * kInterpV * kWave;
  list_task(a, task, (LdsStack)stk, lane);
}

// The same with stacks deeper than an LDS column: kSpillWaves one-wave
// blocks, each with a column of `slots` x kInterpV x 64 doubles in `spill`,
// sweep the tasks.
__global__ __launch_bounds__(64) void k_interpret_list_spill(ListArgs a, double* spill, int slots, int64_t total) {
  const int lane = threadIdx.x & 63;
  double* stk = spill + (int64_t)blockIdx.x * slots * kInterpV * kWave;
  for (int64_t task = blockIdx.x; task < total; task += gridDim.x) list_task(a, task, (GlobalStack)stk, lane);
}

// Waves per interpreter block so that the LDS stacks of one block stay
// within 64 KiB: each wave needs slots * kInterpV * 64 doubles.
inline int interp_waves(int slots) {
  const int per_wave = slots * kInterpV * kWave * (int)sizeof(double);
  int w = 65536 / per_wave;
  return w < 1 ? 1 : (w > 4 ? 4 : w);
}

}  // namespace

hipError_t launch_compile(const RunDev* d_runs, const Params& p, hipStream_t s) {
  const int32_t groups = (p.m + p.r + kCompileWaves - 1) / kCompileWaves;  // blocks per run
  const int32_t most = (int32_t)(kMaxThreads / ((int64_t)groups * kCompileWaves * kWave));  // runs a launch: at least 4
  for (int32_t run = 0; run < p.n_runs; run += most) {
    const int32_t n = p.n_runs - run < most ? p.n_runs - run : most;
    hipLaunchKernelGGL(k_compile, dim3((unsigned)n * groups), dim3(kCompileWaves * kWave),
                       sizeof(uint16_t) * kCompileWaves * p.k, s, d_runs + run, p, groups);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // length bins: (k - length) >> shift < kOrderBins for lengths 0 .. k
  int shift = 0;
  while ((p.k >> shift) >= kOrderBins) ++shift;
  hipLaunchKernelGGL(k_order, dim3(p.n_runs), dim3(1024), 0, s, d_runs, p, shift);
  return hipGetLastError();
}

hipError_t launch_interpret(const RunDev* d_runs, const Params& p, int64_t case_blocks, int slots, int32_t progs,
                            hipStream_t s) {
  if (slots < 1) slots = 1;
  if (slots > kMaxLdsSlots) return hipErrorInvalidValue;  // deeper stacks take the spill pass
  if (progs <= 0) return hipSuccess;
  // one LDS stack column block per wave, at most 64 KiB per block
  const int waves = interp_waves(slots);
  const size_t shmem = (size_t)waves * slots * kInterpV * kWave * sizeof(double);
  const int32_t pgroups = (progs + waves - 1) / waves;
  // any workspace that fits on the device keeps this far below the limit
  if (case_blocks * pgroups > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(case_blocks * pgroups)), block(waves * kWave);
  if (p.precision == GSGP_FP64)
    hipLaunchKernelGGL((k_interpret<double>), grid, block, shmem, s, d_runs, p, pgroups, slots);
  else
    hipLaunchKernelGGL((k_interpret<float>), grid, block, shmem, s, d_runs, p, pgroups, slots);
  return hipGetLastError();
}

hipError_t launch_interpret_wide(const RunDev* d_runs, const Params& p, int64_t case_blocks, int first, int last,
                                 int64_t progs, int32_t per_wave, int32_t* given_up, hipStream_t s) {
  if (first < 0 || last < first || last >= kLists - 1 || per_wave < 1 || per_wave > 32) return hipErrorInvalidValue;
  if (progs <= 0) return hipSuccess;
  const int64_t pgroups = (progs + per_wave - 1) / per_wave;
  if (case_blocks * pgroups > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(case_blocks * pgroups));
  const int slots = kListSlots[last] > 1 + kThreadedReg ? kListSlots[last] - kThreadedReg : 1;
  const size_t shmem = (size_t)slots * kSlotBytes;
  if (p.precision == GSGP_FP64)
    hipLaunchKernelGGL((k_interpret_wide<double>), grid, dim3(kWave), shmem, s, d_runs, p, (int32_t)pgroups, per_wave,
                       first, last, slots, given_up);
  else
    hipLaunchKernelGGL((k_interpret_wide<float>), grid, dim3(kWave), shmem, s, d_runs, p, (int32_t)pgroups, per_wave,
                       first, last, slots, given_up);
  return hipGetLastError();
}

hipError_t launch_interpret_spill(const RunDev* d_runs, const Params& p, double* spill, int slots,
                                  hipStream_t s) {
  if (slots <= kMaxLdsSlots) return hipSuccess;
  if (!spill) return hipErrorInvalidValue;
  if (p.precision == GSGP_FP64)
    hipLaunchKernelGGL((k_interpret_spill<double>), dim3(kSpillWaves), dim3(kWave), 0, s, d_runs, p, spill, slots);
  else
    hipLaunchKernelGGL((k_interpret_spill<float>), dim3(kSpillWaves), dim3(kWave), 0, s, d_runs, p, spill, slots);
  return hipGetLastError();
}

hipError_t launch_interpret_list(const CompiledOp* ops, const int32_t* nops, int32_t k, int32_t m,
                                 const int32_t* tree0, int32_t n0, const int32_t* pool, int32_t np, const double* Xfm,
                                 int64_t ld, int64_t n, double* out0, double* outp, int slots, double* spill,
                                 hipStream_t s) {
  if (n0 + np <= 0) return hipSuccess;
  if (slots < 1) slots = 1;
  const ListArgs a{ops, nops, k, m, tree0, pool, n0, np, Xfm, ld, n, out0, outp};
  const int64_t cblocks = (ld + kWave * kInterpV - 1) / (kWave * kInterpV);
  const int64_t total = cblocks * (n0 + np);
  if (slots > kMaxLdsSlots) {
    if (!spill) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_interpret_list_spill, dim3(kSpillWaves), dim3(kWave), 0, s, a, spill, slots, total);
    return hipGetLastError();
  }
  const int waves = interp_waves(slots);
  const size_t shmem = (size_t)waves * slots * kInterpV * kWave * sizeof(double);
  const int64_t most = kMaxThreads / (waves * kWave) * waves;  // tasks a launch
  hipError_t e = hipSuccess;
  for (int64_t task0 = 0; task0 < total && e == hipSuccess; task0 += most) {
    const int64_t tasks = total - task0 < most ? total - task0 : most;
    hipLaunchKernelGGL(k_interpret_list, dim3(blocks_for(tasks, waves)), dim3(waves * kWave), shmem, s, a, slots, task0,
                       task0 + tasks);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace gsgp
