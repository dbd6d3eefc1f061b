// Generation-side kernels of Section 3.3 (gfx950):
//   reflection-token penalty, Eq. 3 (reward band) and Eq. 4 (subtract beta);
//   the same penalty fused with drawing the next token from softmax(z~ / T);
//   answer perplexity, Eq. 5, and the stop rule, Eq. 6.
#include "reco_device.hpp"
#include "reco_kernels.hpp"

#include <math.h>

namespace reco {

namespace {

constexpr int kPenThreads = 256;
constexpr int kMaxIds = 4096;

__global__ __launch_bounds__(kPenThreads) void logit_penalty_kernel(float *logits, int vocab, int64_t ld,
                                                                    const int32_t *ids, int n_ids,
                                                                    const float *reward, float tau_lo,
                                                                    float tau_hi, float b_lo, float b_mid,
                                                                    float b_hi, int32_t *dev_err) {
  __shared__ int32_t s_ids[kMaxIds];
  const int row = blockIdx.x;
  for (int i = threadIdx.x; i < n_ids; i += kPenThreads) s_ids[i] = ids[i];
  __syncthreads();
  const float v = reward[row];
  // Eq. 3 exactly as written: v <= tau_lo, tau_lo < v < tau_hi, v >= tau_hi.
  const float beta = (v <= tau_lo) ? b_lo : ((v >= tau_hi) ? b_hi : b_mid);
  float *z = logits + static_cast<int64_t>(row) * ld;
  for (int i = threadIdx.x; i < n_ids; i += kPenThreads) {
    const int u = s_ids[i];
    if (u < 0 || u >= vocab) {
      report(dev_err, 4 /*RECO_DEV_BAD_TOKEN_ID*/);
      continue;
    }
    bool first = true;  // R is a set: only the first occurrence of an id subtracts
    for (int j = 0; j < i; ++j) first = first && (s_ids[j] != u);
    if (first) z[u] = z[u] - beta;
  }
}

// ---- fused penalty + sampling ------------------------------------------------
//
// One pass over each logit row: Eq. 3 picks beta from the row's reward, Eq. 4
// subtracts it from the reflection ids (written back in place, as the plain
// penalty does), and the next token is the argmax of z~ (T = 0) or, for
// T > 0, the Gumbel-max draw argmax(z~ / T + G), which is an exact sample of
// softmax(z~ / T).  G = -log(-log U) with U from Philox4x32-10.  Workgroups
// take chunks of a row (one Philox block of four logits per thread and round)
// and leave (best value, index) partials; a one-wave-per-row kernel merges
// them.  Ties and equal partials go to the lowest index; NaN values never win.
//
// Bound by VALU issue: per logit the Philox rounds, two logarithms and a
// division.  Only one logit of a chunk can win, so calls of many chunks bound
// every value from two bare v_log_f32 first and compute y as defined only
// where it can reach the chunk's maximum (256 rows x 152,064:
// 83.9 us with every value computed, 43.9 us).

constexpr int kSmpThreads = 256;
constexpr int kSmpRound = kSmpThreads * 4;   // logits a workgroup takes at once: one Philox block of 4 per thread
constexpr int kSmpRounds = 4;                // rounds of a workgroup in calls of many chunks
constexpr int64_t kSmpWideMin = 2048;        // chunks of one round from which a call has many

// Philox4x32 with 10 rounds (Salmon, Moraes, Dror and Shaw, SC 2011): each
// round multiplies counter words 0 and 2 by the two round constants, crosses
// the 64-bit products' halves with words 1 and 3 and the key, and the key
// advances by the Weyl increments between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // 64-bit products: one v_mad_u64_u32 instead of a v_mul_lo and a v_mul_hi
    const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c[0];
    const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c[2];
    const uint32_t lo0 = static_cast<uint32_t>(p0), hi0 = static_cast<uint32_t>(p0 >> 32);
    const uint32_t lo1 = static_cast<uint32_t>(p1), hi1 = static_cast<uint32_t>(p1 >> 32);
    c[0] = hi1 ^ c[1] ^ k0;
    c[1] = lo1;
    c[2] = hi0 ^ c[3] ^ k1;
    c[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// Midpoint of one of 2^23 equal cells of (0, 1): exact in fp32, never 0 or 1.
__device__ __forceinline__ float unit_open(uint32_t x) {
  return static_cast<float>(x >> 9) * 0x1.0p-23f + 0x1.0p-24f;
}

__device__ __forceinline__ void arg_better(float &v, int &i, float v2, int i2) {
  if (v2 > v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}

__device__ __forceinline__ void wave_argmax(float &v, int &i) {
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) {
    const float v2 = __shfl_xor(v, m, kWave);
    const int i2 = __shfl_xor(i, m, kWave);
    arg_better(v, i, v2, i2);
  }
}

struct SamplePart {
  float v;
  int32_t i;
};

// The value a logit enters the draw with (T > 0).
__device__ __forceinline__ float gumbel_value(float x, float temperature, uint32_t bits) {
  const float g = -logf(-logf(unit_open(bits)));
  return x / temperature + g;
}

// ROUNDS > 1 takes only T in [kFilterMinT, kFilterMaxT], where x * (1 / T)
// is x / T to 2 ulp or overflows with it.
constexpr float kFilterMinT = 1e-30f;
constexpr float kFilterMaxT = 1e30f;

// The largest y of a chunk whose largest estimate is `a` has an estimate no
// smaller than this.  Estimate and y differ by a constant (log ln 2) and by
// less than 2e-5 + 4e-7 |x / T|: the two forms of G differ by at most 1.6e-6
// over all 2^23 uniforms (measured), the rest is the rounding of x / T and of
// the sum; |G| < 17, so |x / T| < |a| + 18 where the estimate is near a.
// NaN for an infinite a: every comparison with it lets the exact value decide.
__device__ __forceinline__ float filter_floor(float a) { return a - (2e-4f + 4e-6f * fabsf(a)); }

template <int ROUNDS, bool VEC>
__global__ __launch_bounds__(kSmpThreads) void penalty_sample_partial_kernel(
    float *logits, int vocab, int64_t ld, const int32_t *ids, int n_ids, const float *reward, float tau_lo,
    float tau_hi, float b_lo, float b_mid, float b_hi, float temperature, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t off_lo, uint32_t off_hi, int chunks, SamplePart *part, int32_t *dev_err) {
  constexpr int kChunk = ROUNDS * kSmpRound;
  constexpr int kBitWords = kChunk / 32;
  constexpr int kWaves = kSmpThreads / kWave;
  __shared__ uint32_t s_bits[kBitWords];
  __shared__ SamplePart s_red[kWaves];
  __shared__ float s_top[kWaves];
  const int chunk = blockIdx.x;
  const int row = blockIdx.y;
  const int c0 = chunk * kChunk;
  const int r0 = threadIdx.x * 4;                    // round-relative, multiple of 4
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  float *z = logits + static_cast<int64_t>(row) * ld;
  // Issue every global load before the first barrier so their latencies overlap.
  float x[ROUNDS][4];
#pragma unroll
  for (int t = 0; t < ROUNDS; ++t) {
    const int j0 = c0 + t * kSmpRound + r0;
    if (VEC && j0 + 3 < vocab) {
      const float4 u = *reinterpret_cast<const float4 *>(z + j0);
      x[t][0] = u.x;
      x[t][1] = u.y;
      x[t][2] = u.z;
      x[t][3] = u.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[t][e] = (j0 + e < vocab) ? z[j0 + e] : -INFINITY;
    }
  }
  const float v = reward[row];
  const int my_id = (static_cast<int>(threadIdx.x) < n_ids) ? ids[threadIdx.x] : -1;
  if (threadIdx.x < kBitWords) s_bits[threadIdx.x] = 0u;
  __syncthreads();
  // Mark the reflection ids that fall in this chunk; a set, so duplicates merge.
  for (int i = threadIdx.x; i < n_ids; i += kSmpThreads) {
    const int u = (i == static_cast<int>(threadIdx.x)) ? my_id : ids[i];
    if (u < 0 || u >= vocab) {
      if (chunk == 0) report(dev_err, 4 /*RECO_DEV_BAD_TOKEN_ID*/);
      continue;
    }
    const int r = u - c0;
    if (r >= 0 && r < kChunk) atomicOr(&s_bits[r >> 5], 1u << (r & 31));
  }
  __syncthreads();
  const float beta = (v <= tau_lo) ? b_lo : ((v >= tau_hi) ? b_hi : b_mid);   // Eq. 3 as written
#pragma unroll
  for (int t = 0; t < ROUNDS; ++t) {
    const int r = t * kSmpRound + r0;
    const uint32_t bits = (s_bits[r >> 5] >> (r & 31)) & 0xFu;   // ids are inside the row
    if (bits) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((bits >> e) & 1u) {                      // Eq. 4, one fp32 subtraction
          x[t][e] = x[t][e] - beta;
          z[c0 + r + e] = x[t][e];
        }
    }
  }

  float best = -INFINITY;
  int best_i = 0x7fffffff;
  const auto draw = [&](int j0, uint32_t (&c)[4]) {
    c[0] = static_cast<uint32_t>(j0 >> 2);
    c[1] = static_cast<uint32_t>(row);
    c[2] = off_lo;
    c[3] = off_hi;
    philox4x32_10(c, seed_lo, seed_hi);
  };
  if (temperature == 0.f) {
#pragma unroll
    for (int t = 0; t < ROUNDS; ++t) {
      const int j0 = c0 + t * kSmpRound + r0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (j0 + e < vocab) arg_better(best, best_i, x[t][e], j0 + e);
    }
  } else if constexpr (ROUNDS == 1) {
    const int j0 = c0 + r0;
    if (j0 < vocab) {
      uint32_t c[4];
      draw(j0, c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float y = gumbel_value(x[0][e], temperature, c[e]);
        if (j0 + e < vocab) arg_better(best, best_i, y, j0 + e);
      }
    }
  } else {
    // Estimates of y - log ln 2, the largest of each thread and round kept.
    const float inv_t = 1.f / temperature;
    float top[ROUNDS];
    float a = -INFINITY;
#pragma unroll
    for (int t = 0; t < ROUNDS; ++t) {
      const int j0 = c0 + t * kSmpRound + r0;
      uint32_t c[4];
      draw(j0, c);
      top[t] = -INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) {                  // logits past the row are -inf
        const float l = __builtin_amdgcn_logf(-__builtin_amdgcn_logf(unit_open(c[e])));
        top[t] = fmaxf(top[t], fmaf(l, -kLn2, x[t][e] * inv_t));
      }
      a = fmaxf(a, top[t]);
    }
    a = wave_max(a);
    if (lane == 0) s_top[wave] = a;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) a = fmaxf(a, s_top[w]);
    const float floor_a = filter_floor(a);
    // Only infinite logits (and NaN, which never wins) in the chunk: y is x.
    const bool masked = a == -INFINITY;
#pragma unroll
    for (int t = 0; t < ROUNDS; ++t) {
      const int j0 = c0 + t * kSmpRound + r0;
      if (top[t] < floor_a) continue;
      bool infinite = masked;
#pragma unroll
      for (int e = 0; e < 4; ++e) infinite = infinite && !(fabsf(x[t][e]) < INFINITY);
      if (infinite) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j0 + e < vocab) arg_better(best, best_i, x[t][e], j0 + e);
      } else {
        uint32_t c[4];
        draw(j0, c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float y = gumbel_value(x[t][e], temperature, c[e]);
          if (j0 + e < vocab) arg_better(best, best_i, y, j0 + e);
        }
      }
    }
  }
  wave_argmax(best, best_i);
  if (lane == 0) s_red[wave] = SamplePart{best, best_i};
  __syncthreads();
  if (threadIdx.x == 0) {
    SamplePart r = s_red[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) arg_better(r.v, r.i, s_red[w].v, s_red[w].i);
    part[static_cast<size_t>(row) * chunks + chunk] = r;
  }
}

// One wave per row: merge the chunk partials into the row's token.
__global__ __launch_bounds__(kSmpThreads) void penalty_sample_final_kernel(const SamplePart *part, int rows,
                                                                           int chunks, int32_t *tokens,
                                                                           int32_t *dev_err) {
  const int row = blockIdx.x * (kSmpThreads / kWave) + threadIdx.x / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  if (row >= rows) return;
  float best = -INFINITY;
  int best_i = 0x7fffffff;
  for (int c = lane; c < chunks; c += kWave) {
    const SamplePart q = part[static_cast<size_t>(row) * chunks + c];
    arg_better(best, best_i, q.v, q.i);
  }
  wave_argmax(best, best_i);
  if (lane == 0) {
    if (best_i == 0x7fffffff) {             // every value of the row was NaN
      report(dev_err, 6 /*RECO_DEV_BAD_LOGIT*/);
      best_i = -1;
    }
    tokens[row] = best_i;
  }
}

constexpr int kPplThreads = 256;
constexpr int kPplFinalThreads = 1024;
// Logits per workgroup: small chunks spread a call evenly over the chip.  The
// large ones need a quarter of the partials, for callers with a workspace of
// that size.
constexpr int kPplChunk = 4096;
constexpr int kPplLargeChunk = 16384;

// Per (row, chunk): the chunk's max and sum of exp(z - max), natural log domain.
// Each thread holds its logits of the chunk in registers (all requested in
// one round trip, as 16-byte non-temporal loads where the rows allow), so
// the max and the sum need a single read of the chunk.
template <int CHUNK, bool VEC>
__global__ __launch_bounds__(kPplThreads) void ppl_partial_kernel(const float *logits, int vocab, int chunks,
                                                                  float *part) {
  constexpr int kPer = CHUNK / kPplThreads;
  __shared__ float red[kPplThreads / kWave];
  const int chunk = blockIdx.x;
  const size_t row = blockIdx.y;
  const int c0 = chunk * CHUNK;
  const int c1 = min(vocab, c0 + CHUNK);
  const float *z = logits + row * static_cast<size_t>(vocab);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;

  float x[kPer];
  if constexpr (VEC) {
#pragma unroll
    for (int i = 0; i < kPer / 4; ++i) {
      const int j = c0 + (i * kPplThreads + static_cast<int>(threadIdx.x)) * 4;   // c1 - j is a multiple of 4
      const uint4 u = j < c1 ? nt_load_u4(z + j) : make_uint4(0xff800000u, 0xff800000u, 0xff800000u, 0xff800000u);
      x[4 * i + 0] = __uint_as_float(u.x);
      x[4 * i + 1] = __uint_as_float(u.y);
      x[4 * i + 2] = __uint_as_float(u.z);
      x[4 * i + 3] = __uint_as_float(u.w);
    }
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int j = c0 + i * kPplThreads + static_cast<int>(threadIdx.x);
      x[i] = j < c1 ? z[j] : -INFINITY;
    }
  }
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < kPer; ++i) m = fmaxf(m, x[i]);
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  float M = red[0];
#pragma unroll
  for (int w = 1; w < kPplThreads / kWave; ++w) M = fmaxf(M, red[w]);
  __syncthreads();
  float s = 0.f;
  if (M != -INFINITY) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) s += expf(x[i] - M);     // x = -inf (past the row) adds 0
  }
  s = wave_sum(s);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float S = 0.f;
#pragma unroll
    for (int w = 0; w < kPplThreads / kWave; ++w) S += red[w];
    part[(row * chunks + chunk) * 2 + 0] = M;
    part[(row * chunks + chunk) * 2 + 1] = S;
  }
}

// Per sequence: LSE of every answer position (fp64 merge of the chunk
// partials), the mean negative log-likelihood, PPL and the stop flag.  Bound
// by its chain of dependent reads: `per_row` lanes (a power of two up to 64)
// take a row and share its chunks, so that every row is read at once, its
// partials and its token's logit together, wherever the rows fit a workgroup
// (whole call, with the chunk size above: 32 rows x 152,064 12.5 us with a
// thread a row and 16,384 a chunk, 9.9 us; 256 rows 32.7 us, 29.3 us).
constexpr int kPplHold = 4;                           // chunks a lane keeps in registers

__global__ __launch_bounds__(kPplFinalThreads) void ppl_final_kernel(const float *logits, const int32_t *tokens,
                                                                     int n, int vocab, int chunks, int per_row,
                                                                     const float *part, float tau_p, float *ppl,
                                                                     int32_t *stop, int32_t *dev_err) {
  constexpr int kHold = kPplHold;
  __shared__ double red[kPplFinalThreads / kWave];
  const int b = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int waves = static_cast<int>(blockDim.x) / kWave;
  const int c0 = static_cast<int>(threadIdx.x) & (per_row - 1);
  double nll = 0.0;
  bool bad = false;
  // Every lane of a wave takes as many turns (the groups exchange values).
  for (int t0 = 0; t0 < n; t0 += static_cast<int>(blockDim.x) / per_row) {
    const int t = t0 + static_cast<int>(threadIdx.x) / per_row;
    const bool row_ok = t < n;
    const size_t row = static_cast<size_t>(b) * n + (row_ok ? t : 0);
    const float *pr = part + row * chunks * 2;
    const int x = tokens[row];
    float m[kHold], s[kHold];
#pragma unroll
    for (int i = 0; i < kHold; ++i) {
      const int c = c0 + i * per_row;
      m[i] = c < chunks ? pr[2 * c] : -INFINITY;
      s[i] = c < chunks ? pr[2 * c + 1] : 0.f;
    }
    const bool in = x >= 0 && x < vocab;
    const float z = in ? logits[row * vocab + x] : 0.f;
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < kHold; ++i) M = fmaxf(M, m[i]);
    for (int c = c0 + kHold * per_row; c < chunks; c += per_row) M = fmaxf(M, pr[2 * c]);
    for (int d = 1; d < per_row; d <<= 1) M = fmaxf(M, shfl_xor(M, d));
    double S = 0.0;
    const auto add = [&](float mc, float sc) {
      if (mc != -INFINITY) S += static_cast<double>(sc) * exp(static_cast<double>(mc) - M);
    };
#pragma unroll
    for (int i = 0; i < kHold; ++i) add(m[i], s[i]);
    for (int c = c0 + kHold * per_row; c < chunks; c += per_row) add(pr[2 * c], pr[2 * c + 1]);
    for (int d = 1; d < per_row; d <<= 1) S += __shfl_xor(S, d, kWave);
    if (row_ok && c0 == 0) {
      bad = bad || !in;
      if (in) nll += static_cast<double>(M) + log(S) - static_cast<double>(z);
    }
  }
  for (int d = per_row; d < kWave; d <<= 1) nll += __shfl_xor(nll, d, kWave);   // first lanes of the rows hold sums
  bad = __any(bad);
  if (lane == 0) red[wave] = bad ? NAN : nll;
  __syncthreads();
  if (threadIdx.x == 0) {
    double total = 0.0;
    for (int w = 0; w < waves; ++w) total += red[w];
    if (isnan(total)) report(dev_err, 4 /*RECO_DEV_BAD_TOKEN_ID*/);
    const double pp = exp(total / n);
    ppl[b] = static_cast<float>(pp);
    if (stop) stop[b] = (pp <= static_cast<double>(tau_p)) ? 1 : 0;
  }
}

}  // namespace

hipError_t launch_logit_penalty(float *logits, int rows, int vocab, int64_t ld, const int32_t *ids, int n_ids,
                                const float *reward, float tau_lo, float tau_hi, float b_lo, float b_mid,
                                float b_hi, int32_t *dev_err, hipStream_t s) {
  hipLaunchKernelGGL(logit_penalty_kernel, dim3(rows), dim3(kPenThreads), 0, s, logits, vocab, ld, ids, n_ids,
                     reward, tau_lo, tau_hi, b_lo, b_mid, b_hi, dev_err);
  return hipGetLastError();
}

namespace {
int sample_chunks(int vocab, int rounds) {
  const int64_t chunk = static_cast<int64_t>(rounds) * kSmpRound;
  return static_cast<int>((static_cast<int64_t>(vocab) + chunk - 1) / chunk);
}
}  // namespace

// Sized for the smallest chunk; larger ones need less.
size_t penalty_sample_workspace_bytes(int rows, int vocab) {
  return static_cast<size_t>(rows) * sample_chunks(vocab, 1) * sizeof(SamplePart);
}

hipError_t launch_penalty_sample(float *logits, int rows, int vocab, int64_t ld, const int32_t *ids, int n_ids,
                                 const float *reward, float tau_lo, float tau_hi, float b_lo, float b_mid,
                                 float b_hi, float temperature, uint64_t seed, uint64_t offset, int32_t *tokens,
                                 void *ws, int32_t *dev_err, hipStream_t s) {
  // Many chunks: workgroups of four rounds fill the chip and need a third of
  // the instructions (16 rows x 152,064: 10.6 us in single rounds, 9.4 us in
  // four; 256 rows: 72.4 us and 43.9 us, 43.4 us in eight; greedy 45.5 us and
  // 31.0 us).  Fewer leave it idle (32 rows x 32,000: 7.4 us and 7.8 us; one
  // row x 128,256: 6.3 us and 7.5 us).
  const bool wide = static_cast<int64_t>(rows) * sample_chunks(vocab, 1) >= kSmpWideMin &&
                    (temperature == 0.f || (temperature >= kFilterMinT && temperature <= kFilterMaxT));
  const bool vec = ld % 4 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0;
  const int chunks = sample_chunks(vocab, wide ? kSmpRounds : 1);
  SamplePart *part = reinterpret_cast<SamplePart *>(ws);
  const auto kernel = wide ? (vec ? penalty_sample_partial_kernel<kSmpRounds, true>
                                  : penalty_sample_partial_kernel<kSmpRounds, false>)
                           : (vec ? penalty_sample_partial_kernel<1, true> : penalty_sample_partial_kernel<1, false>);
  hipLaunchKernelGGL(kernel, dim3(chunks, rows), dim3(kSmpThreads), 0, s, logits, vocab, ld, ids, n_ids, reward,
                     tau_lo, tau_hi, b_lo, b_mid, b_hi, temperature, static_cast<uint32_t>(seed),
                     static_cast<uint32_t>(seed >> 32), static_cast<uint32_t>(offset),
                     static_cast<uint32_t>(offset >> 32), chunks, part, dev_err);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int per_wg = kSmpThreads / kWave;
  hipLaunchKernelGGL(penalty_sample_final_kernel, dim3((rows + per_wg - 1) / per_wg), dim3(kSmpThreads), 0, s, part,
                     rows, chunks, tokens, dev_err);
  return hipGetLastError();
}

namespace {
int64_t ppl_chunks(int vocab, int chunk) { return (static_cast<int64_t>(vocab) + chunk - 1) / chunk; }

size_t ppl_bytes(int batch, int n, int vocab, int chunk) {
  return static_cast<size_t>(batch) * n * ppl_chunks(vocab, chunk) * 2 * sizeof(float);
}
}  // namespace

size_t ppl_workspace_bytes(int batch, int n, int vocab) { return ppl_bytes(batch, n, vocab, kPplChunk); }

size_t ppl_min_workspace_bytes(int batch, int n, int vocab) { return ppl_bytes(batch, n, vocab, kPplLargeChunk); }

hipError_t launch_answer_ppl(const float *logits, const int32_t *tokens, int batch, int n, int vocab, float tau_p,
                             float *ppl, int32_t *stop, void *ws, size_t ws_bytes, int32_t *dev_err,
                             hipStream_t s) {
  // Small chunks are the faster ones everywhere (start of the call to its end,
  // 16,384 and 4,096 a chunk: 1 x 4 rows x 128,256 8.7 and 6.5 us; 1 x 32 x
  // 152,064 13.6 and 11.8 us; 8 x 32 x 152,064 33.2 and 32.8 us).
  const bool small = ws_bytes >= ppl_workspace_bytes(batch, n, vocab);
  const int chunks = static_cast<int>(ppl_chunks(vocab, small ? kPplChunk : kPplLargeChunk));
  float *part = reinterpret_cast<float *>(ws);
  const bool vec = vocab % 4 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0;
  const auto kernel = small ? (vec ? ppl_partial_kernel<kPplChunk, true> : ppl_partial_kernel<kPplChunk, false>)
                            : (vec ? ppl_partial_kernel<kPplLargeChunk, true>
                                   : ppl_partial_kernel<kPplLargeChunk, false>);
  hipLaunchKernelGGL(kernel, dim3(chunks, batch * n), dim3(kPplThreads), 0, s, logits, vocab, chunks, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // As few lanes a row as hold its chunks in registers, fewer where the rows
  // need the lanes, and no more waves than that takes.
  int per_row = 1;
  while (per_row < kWave && per_row * kPplHold < chunks) per_row *= 2;
  while (per_row > 1 && static_cast<int64_t>(n) * per_row > kPplFinalThreads) per_row /= 2;
  const int64_t lanes = (static_cast<int64_t>(n) * per_row + kWave - 1) / kWave * kWave;
  const int threads = lanes < kPplFinalThreads ? static_cast<int>(lanes) : kPplFinalThreads;
  hipLaunchKernelGGL(ppl_final_kernel, dim3(batch), dim3(threads), 0, s, logits, tokens, n, vocab, chunks, per_row,
                     part, tau_p, ppl, stop, dev_err);
  return hipGetLastError();
}

}  // namespace reco
