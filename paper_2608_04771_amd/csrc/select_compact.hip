// Reward-budgeted selection and in-place compaction of the KV cache (gfx950).
//
// select: one 1024-thread workgroup per unit.  The budget m follows from the
//   unit's length and the sequence's retention in fp64; the k = m - w_eff
//   best prefix scores are found with an exact MSB-first radix select on the
//   fp32 bit patterns (non-negative floats order like their bits): three
//   histogram passes of 11, 11 and 10 bits over LDS bins give the k-th value
//   theta and how many of the entries equal to theta are still needed.  Each
//   wave owns a contiguous stretch of the prefix, 64 positions at a time, so
//   one scan over the waves' counts and ballots within a wave then give every
//   kept position (entries above theta, plus the first `need` entries equal to
//   theta) its place in ascending order, and the window positions come after
//   them.  A workgroup is bound by its chain of passes: up to kHeld scores a
//   thread stay in registers instead of being read four times, each bin is
//   counted in four copies (scores crowd into few bins of the first pass), and a
//   bin is found by all threads (112 units of 16,384: the whole call, 229 us of
//   it compaction, 264 -> 247 us).  With more units than CUs two workgroups share
//   a CU, if their waves' scalar registers fit a SIMD: of more than 80 (and the
//   trap handler's 16) not eight do (512 units of 1,000 rows: with 94 40.3 us, with
//   80 36.6 us; 2,048 of 200 85.6 us, 66.3 us; 512 of 30,000 936 us, 881 us; what
//   is spilled to keep to 80 takes 0.3 us of the smaller calls).
// compact: one 256-thread workgroup per (unit, K or V, 128-byte column slice)
//   moves row idx[p] to row p for p = 0..m-1 in ascending chunks of 256
//   rows.  Because idx is strictly increasing, idx[p] >= p: a chunk's sources
//   lie at or after its own destinations, and rows a later chunk reads lie at
//   or after that chunk's destinations, beyond everything stored so far.  So
//   loading a whole chunk, waiting at a barrier, then storing it never
//   overwrites a row that is still to be read; no second buffer is needed.
#include "reco_device.hpp"
#include "reco_kernels.hpp"

#include <math.h>

namespace reco {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kHeld = 16;                    // scores a thread keeps in registers
constexpr int kCopies = 4;                   // copies of each histogram bin
constexpr int kMaxBins = 2048;
constexpr int kSelSgprs = 80;                // two workgroups on a CU
constexpr int kCompThreads = 256;
constexpr int kSliceBytes = 128;             // row slice per compaction workgroup
constexpr int kLanesPerRow = kSliceBytes / 16;
constexpr int kRowsPerPass = kCompThreads / kLanesPerRow;  // 32
constexpr int kRowsPerThread = 8;
constexpr int kChunkRows = kRowsPerPass * kRowsPerThread;  // 256

// Inclusive wave scan of an int.
__device__ __forceinline__ int wave_incl_scan(int v, int lane) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int o = __shfl_up(v, d, kWave);
    if (lane >= d) v += o;
  }
  return v;
}

__device__ __forceinline__ uint32_t score_bits(float s, bool *bad) {
  uint32_t u = __float_as_uint(s);
  if (u == 0x80000000u) u = 0;                    // -0 ranks as +0
  if ((u >> 31) || u > 0x7f800000u) *bad = true;  // negative or NaN
  return u;
}

__global__ __launch_bounds__(kSelThreads) __attribute__((amdgpu_num_sgpr(kSelSgprs))) void select_kernel(SelectParams p) {
  __shared__ __attribute__((aligned(16))) int hist[kMaxBins * kCopies];
  __shared__ int wsum[kSelWaves];
  __shared__ int2 wcount[kSelWaves];
  __shared__ int s_bin, s_krem, s_bad;

  const int unit = blockIdx.x;
  const int per_layer = p.batch * p.hkv;
  const int lc = unit / per_layer;
  const int b = (unit % per_layer) / p.hkv;
  const int h = unit % p.hkv;
  const size_t cunit = (static_cast<size_t>(p.layer0 + lc) * p.batch + b) * p.hkv + h;
  const int tid = threadIdx.x;

  const int L = p.len[cunit];
  const double r = p.retention[static_cast<int64_t>(lc) * p.ret_stride + b];
  if (L < 0 || L > p.cap) {
    if (tid == 0) {
      report(p.dev_err, 5 /*RECO_DEV_BAD_LENGTH*/);
      p.kept[unit] = -1;
    }
    return;
  }
  if (!(r > 0.0 && r <= 1.0)) {
    if (tid == 0) {
      report(p.dev_err, 2 /*RECO_DEV_BAD_RETENTION*/);
      p.kept[unit] = -1;
    }
    return;
  }
  const int w_eff = min(p.w, L);
  const double prod = r * static_cast<double>(L);
  int m = static_cast<int>(ceil(prod));
  m = max(w_eff, m);
  m = min(L, m);
  const int k = m - w_eff;
  const int P = L - w_eff;
  const float *sc = p.scores + static_cast<size_t>(unit) * p.cap;
  int32_t *idx = p.idx + static_cast<size_t>(unit) * p.cap;

  if (tid == 0) s_bad = 0;
  __syncthreads();

  // Wave `wave` owns positions [wave * 64 * turns, (wave + 1) * 64 * turns).
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int turns = (P + kSelThreads - 1) / kSelThreads;
  const int j0 = wave * turns * kWave + lane;
  const bool held = turns <= kHeld;
  bool bad = false;
  uint32_t kept_bits[kHeld];
  if (held) {
    float x[kHeld];
#pragma unroll
    for (int i = 0; i < kHeld; ++i) x[i] = i < turns && j0 + i * kWave < P ? sc[j0 + i * kWave] : 0.f;
#pragma unroll
    for (int i = 0; i < kHeld; ++i) kept_bits[i] = score_bits(x[i], &bad);
  }
  // f(bits, position) for every position of this lane, in order and by whole
  // waves; positions at or past P come too.
  const auto for_each = [&](auto f) {
    if (held) {
#pragma unroll
      for (int i = 0; i < kHeld; ++i)
        if (i < turns) f(kept_bits[i], j0 + i * kWave);
    } else {
#pragma unroll 4
      for (int i = 0; i < turns; ++i) {
        const int j = j0 + i * kWave;
        f(score_bits(j < P ? sc[j] : 0.f, &bad), j);
      }
    }
  };

  // Validate the prefix scores (one pass, fused with the first histogram when k < P).
  uint32_t prefix = 0, pmask = 0;
  int krem = k;
  if (k > 0 && k < P) {
    const int shifts[3] = {21, 10, 0};
    const int nbits[3] = {11, 11, 10};
    for (int pass = 0; pass < 3; ++pass) {
      const int sh = shifts[pass];
      const int nb = 1 << nbits[pass];
      for (int i = tid; i < nb * kCopies / 4; i += kSelThreads) reinterpret_cast<int4 *>(hist)[i] = make_int4(0, 0, 0, 0);
      __syncthreads();
      for_each([&](uint32_t u, int j) {
        if (j < P && (u & pmask) == prefix) atomicAdd(&hist[((u >> sh) & (nb - 1)) * kCopies + lane % kCopies], 1);
      });
      if (bad) s_bad = 1;
      __syncthreads();
      if (s_bad) break;
      // Find the bin holding the krem-th largest entry: thread t has bins
      // 2t and 2t + 1, or bin t alone.
      static_assert(kCopies == 4 && kMaxBins == 2 * kSelThreads, "one int4 per bin, at most two bins per thread");
      const auto count = [&](int bin) {
        const int4 c = reinterpret_cast<const int4 *>(hist)[bin];
        return c.x + c.y + c.z + c.w;
      };
      const bool two = nb == kMaxBins;
      const int lo = two ? count(2 * tid) : count(tid);
      const int hi = two ? count(2 * tid + 1) : 0;
      const int incl = wave_incl_scan(lo + hi, lane);
      if (lane == kWave - 1) wsum[wave] = incl;
      __syncthreads();
      const int wincl = wave_incl_scan(lane < kSelWaves ? wsum[lane] : 0, lane);
      const int total = __shfl(wincl, kSelWaves - 1, kWave);
      const int before = wave == 0 ? 0 : __shfl(wincl, wave - 1, kWave);
      const int above = total - before - incl;               // entries in the bins of later threads
      if (above < krem && krem <= above + lo + hi) {
        const bool in_hi = krem <= above + hi;
        s_bin = two ? 2 * tid + (in_hi ? 1 : 0) : tid;
        s_krem = krem - above - (in_hi ? 0 : hi);
      }
      __syncthreads();
      prefix |= static_cast<uint32_t>(s_bin) << sh;
      pmask |= static_cast<uint32_t>(nb - 1) << sh;
      krem = s_krem;
    }
  } else {
    for_each([](uint32_t, int) {});
    if (bad) s_bad = 1;
    __syncthreads();
  }
  if (s_bad) {
    if (tid == 0) {
      report(p.dev_err, 3 /*RECO_DEV_BAD_SCORE*/);
      p.kept[unit] = -1;
    }
    return;
  }

  // Keep u > theta, and the first `need` entries with u == theta.
  const uint32_t theta = prefix;
  const int need = krem;
  if (k == 0) {
    // only the window survives
  } else if (k == P) {
    for (int j = tid; j < P; j += kSelThreads) idx[j] = j;
  } else {
    int n_gt = 0, n_eq = 0;                                  // of this wave
    for_each([&](uint32_t u, int j) {
      n_gt += __popcll(__ballot(j < P && u > theta));
      n_eq += __popcll(__ballot(j < P && u == theta));
    });
    if (lane == 0) wcount[wave] = make_int2(n_gt, n_eq);
    __syncthreads();
    int eq = 0, pos = 0;                                     // entries equal to theta, and kept ones, so far
    for (int w = 0; w < wave; ++w) {
      pos += wcount[w].x;
      eq += wcount[w].y;
    }
    pos += min(eq, need);
    const uint64_t below = (1ull << lane) - 1;
    for_each([&](uint32_t u, int j) {
      const bool is_eq = j < P && u == theta;
      const uint64_t eq_mask = __ballot(is_eq);
      const bool keep = (j < P && u > theta) || (is_eq && eq + __popcll(eq_mask & below) < need);
      const uint64_t keep_mask = __ballot(keep);
      if (keep) idx[pos + __popcll(keep_mask & below)] = j;
      pos += __popcll(keep_mask);
      eq += __popcll(eq_mask);
    });
  }
  for (int t = tid; t < w_eff; t += kSelThreads) idx[k + t] = P + t;
  if (tid == 0) p.kept[unit] = m;
}

template <int ROWB>
__global__ __launch_bounds__(kCompThreads) void compact_kernel(SelectParams p) {
  constexpr int kSlices = ROWB / kSliceBytes;
  constexpr int kPerUnit = 2 * kSlices;             // (K or V) x slice workgroups of one unit
  // XCD-aware order: consecutive workgroup ids go to the eight XCDs in turn,
  // so ids are laid out in groups of 8 units x kPerUnit with every workgroup
  // of a unit at the same id mod 8: they share one XCD's L2 and the unit's
  // kept list is fetched from HBM once.  Padding workgroups return at once.
  const int grp8 = static_cast<int>(blockIdx.x) / (8 * kPerUnit);
  const int r8 = static_cast<int>(blockIdx.x) - grp8 * 8 * kPerUnit;
  const int unit = grp8 * 8 + (r8 & 7);
  const int job = r8 >> 3;
  const int slice = job % kSlices;
  const int tensor = job / kSlices;
  if (unit >= p.n_layers * p.batch * p.hkv) return;
  const int per_layer = p.batch * p.hkv;
  const int lc = unit / per_layer;
  const int b = (unit % per_layer) / p.hkv;
  const int h = unit % p.hkv;
  const size_t cunit = (static_cast<size_t>(p.layer0 + lc) * p.batch + b) * p.hkv + h;
  const int m = p.kept[unit];
  if (m < 0) return;
  const int32_t *idx = p.idx + static_cast<size_t>(unit) * p.cap;
  unsigned char *base = reinterpret_cast<unsigned char *>(tensor == 0 ? p.k : p.v) +
                        cunit * static_cast<size_t>(p.cap) * ROWB + slice * kSliceBytes;
  const int sub = (threadIdx.x % kLanesPerRow) * 16;
  const int rrow = threadIdx.x / kLanesPerRow;

  for (int c0 = 0; c0 < m; c0 += kChunkRows) {
    // One 128-bit register per row of the chunk; the whole chunk stays in
    // registers across the barrier.  Rows that do not move (or lie past m)
    // read row 0 of the unit, which is always in bounds.
    typedef unsigned int u32x32 __attribute__((ext_vector_type(4 * kRowsPerThread)));
    u32x32 v;
    unsigned mv = 0;
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) {
      const int pdst = c0 + i * kRowsPerPass + rrow;
      const int s = idx[min(pdst, m - 1)];
      const bool move = pdst < m && s != pdst;
      mv |= (move ? 1u : 0u) << i;
      const uint4 x = *reinterpret_cast<const uint4 *>(base + static_cast<size_t>(move ? s : 0) * ROWB + sub);
      v[4 * i + 0] = x.x;
      v[4 * i + 1] = x.y;
      v[4 * i + 2] = x.z;
      v[4 * i + 3] = x.w;
    }
    __syncthreads();   // every read of this chunk has returned before any row of it is overwritten
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) {
      const int pdst = c0 + i * kRowsPerPass + rrow;
      if (mv & (1u << i))
        *reinterpret_cast<uint4 *>(base + static_cast<size_t>(pdst) * ROWB + sub) =
            make_uint4(v[4 * i + 0], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    }
  }
  if (tensor == 0 && slice == 0 && threadIdx.x == 0) p.len[cunit] = m;
}

}  // namespace

size_t select_workspace_bytes(int units, int capacity, bool need_idx) {
  size_t bytes = (static_cast<size_t>(units) * sizeof(int32_t) + 255) / 256 * 256;
  if (need_idx) bytes += static_cast<size_t>(units) * capacity * sizeof(int32_t);
  return bytes;
}

hipError_t launch_select_compact(const SelectParams &p, int dtype, int head_dim, hipStream_t s) {
  const int units = p.n_layers * p.batch * p.hkv;
  hipLaunchKernelGGL(select_kernel, dim3(units), dim3(kSelThreads), 0, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int rowb = head_dim * (dtype == 0 ? 4 : 2);
  switch (rowb) {
    case 128:
      hipLaunchKernelGGL(compact_kernel<128>, dim3((units + 7) / 8 * 8 * 2 * 1), dim3(kCompThreads), 0, s, p);
      break;
    case 256:
      hipLaunchKernelGGL(compact_kernel<256>, dim3((units + 7) / 8 * 8 * 2 * 2), dim3(kCompThreads), 0, s, p);
      break;
    default:
      hipLaunchKernelGGL(compact_kernel<512>, dim3((units + 7) / 8 * 8 * 2 * 4), dim3(kCompThreads), 0, s, p);
      break;
  }
  return hipGetLastError();
}

}  // namespace reco
