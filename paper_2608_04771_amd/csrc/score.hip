// Window attention-mass scoring of every cached key (Eq. 2), gfx950.
//
// For one unit (layer, sequence, kv head h) the window rows are the G * w
// (query head of h's group, window position) pairs.  Row r = g * w + t is the
// query of head h*G + g at absolute position pos = L - w + t.  Scoring takes
// the softmax normaliser (max, sum) of every window row (a statistics pass
// over K, or the values decode wrote for the window tokens), then the mass
// pass adds exp2(x - max) / sum over all rows of each key.
//
// Both passes are a persistent grid of one eight-wave workgroup (two waves
// per SIMD) per CU.  A workgroup takes an equal share of all units' keys and
// walks it as segments, the pieces inside one unit: it stages the unit's
// window rows in LDS once per segment (in blocks of at most max_rows), and
// every wave then walks its own groups of 32 * KT keys, the group's K
// fragments loaded from global memory straight into registers, with no
// barrier in the loop.
//
// A tile is 32 keys x 32 window rows, S^T = K.Q^T, on the 32x32 MFMAs: a lane
// holds 16 keys of one window row, so a row's (max, sum) is one register per
// lane.  Measured (in-bounds probes, two waves per SIMD): a
// 32x32x16 bf16 MFMA occupies the matrix core for 32 cycles and takes no
// issue cycles from the other wave's VALU work, where a 16x16x32 one takes
// about 4 of its 16; FMA and add take 4 cycles and v_exp_f32 8.  A pair
// (row, key) needs one FMA, one exp2 and one add, so 64 pairs cost 16 cycles
// of VALU and, at head_dim 128, 16 cycles of matrix core: the two pipes are
// balanced, and a pass can reach half the time of doing them in turn only if
// they overlap.  So the tiles are software-pipelined inside each wave: the
// products of the next tile are issued between the exponentials of the
// current one, through two accumulators, and each Q fragment register is
// reloaded from LDS right after its last use.  In a loop of its own the pair
// of waves then takes 750 cycles per 64 keys x 32 rows and wave, against 512
// with perfect overlap: an MFMA takes about 10 cycles of its SIMD's issue.
//
// Measured (both sides in turn): 28 layers x 4 heads x 16,384 keys, 448
// rows, two passes: 538 us with 16x16x32 tiles in turn with their exponentials
// and a row-merge kernel between the passes, now 448 us.  Counters there: the
// VALU issues in 60 to 62% of the cycles, the matrix core is busy in 45 to 47%,
// one or the other in 78 to 80%, so what the two waves of a SIMD do not overlap
// bounds the call.  64 units of 65,536 keys, 160 rows, one pass: 254 us, now
// 249 us (4.3 TB/s of K): there the pipes work in 64% of the cycles and the
// address unit in 56%, as the fragments' 16-byte accesses take 32 bytes of each
// row, with few products to hide behind.  Two fp32 units of 2,048 keys: 97.7 us,
// now 26.8 us (their keys and row tiles spread over 66 CUs instead of 8).
// Slower for the 64 units: the next group's K fragments held in registers a
// group ahead (they spill: 309 us, where reloading each fragment after its last
// use took 245 us), and touching the next group's lines a group ahead (275 us).
#include "reco_device.hpp"
#include "reco_kernels.hpp"

#include <math.h>

namespace reco {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kWave;
constexpr int kTileRows = 32;

typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <typename T, int D>
struct ScoreCfg {
  static constexpr int row_bytes = D * (int)sizeof(T);
  static constexpr int pieces = row_bytes / 32;         // 16-byte pieces per lane of one row (two lanes share a row)
  typedef uint4 frags[pieces];                          // a lane of one 32-row tile
  static constexpr int KT = pieces <= 8 ? 2 : 1;        // 32-key tiles per wave group (64 K registers either way)
  static constexpr int group = 32 * KT;                 // keys per wave group
  static constexpr int q_stride = row_bytes + 16;       // LDS pitch of a window row: eight rows cover all banks
  // Row tiles staged at once: the rows, the per-wave sums and the references must fit the LDS of a CU.
  static constexpr int max_tiles = row_bytes == 128 ? 28 : row_bytes == 256 ? 16 : 8;
  static constexpr int max_rows = max_tiles * kTileRows;
  static constexpr int q_bytes = max_rows * q_stride;
  static constexpr int sum_bytes = kWaves * max_rows * 4;
  static constexpr int stats_lds = q_bytes + sum_bytes + max_rows * 4;
  static constexpr int mass_lds = q_bytes + max_rows * 8;
  static constexpr int lost_keys = 4096;                // longest mass segment of a call with several row blocks
  static_assert(stats_lds <= 160 * 1024 && mass_lds + lost_keys * 4 + kWaves * kWave * 4 + 16 <= 160 * 1024,
                "window rows and statistics fit one CU's LDS");
};

// ---------------------------------------------------------------------------
// Shares of the persistent grid.  The work is the non-empty chunks of
// chunk_keys keys of every unit (ceil(L / chunk_keys) of them), unit-major.
// Workgroup b takes chunks [total * b / grid, total * (b + 1) / grid) of that
// order and walks them as segments, the pieces inside one unit.
// ---------------------------------------------------------------------------
struct Share {
  int b;             // rank of the workgroup in the chunk order
  int unit;          // unit of the next chunk
  int chunk;         // that chunk's index within its unit
  long long n;       // chunks left
  long long before;  // chunks of all units before `unit`
  long long total;   // chunks of all units
};

// A value that is the same in every lane, kept in a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uniform(long long v) {
  const unsigned lo = uniform(static_cast<int>(v)), hi = uniform(static_cast<int>(v >> 32));
  return static_cast<long long>(static_cast<unsigned long long>(hi) << 32 | lo);
}

__device__ __forceinline__ int unit_len(const ScoreParams &p, int unit) {
  const int L = p.len[static_cast<size_t>(p.layer0) * p.batch * p.hkv + unit];
  return L < 0 ? 0 : (L > p.cap ? p.cap : L);
}

__device__ __forceinline__ int unit_chunks(const ScoreParams &p, int unit) {
  return (unit_len(p, unit) + p.chunk_keys - 1) / p.chunk_keys;
}

__device__ __forceinline__ long long share_begin(long long total, int b) {
  return total * b / static_cast<int>(gridDim.x);
}

// Every workgroup scans the units' chunk counts to find where its share
// starts.  `lds`: kWaves + 3 entries of scratch.
__device__ Share find_share(const ScoreParams &p, long long *lds) {
  const int units = p.n_layers * p.batch * p.hkv;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int per_t = (units + kThreads - 1) / kThreads;
  const int u0 = min(units, static_cast<int>(threadIdx.x) * per_t);
  const int u1 = min(units, u0 + per_t);
  long long mine = 0;
  for (int u = u0; u < u1; ++u) mine += unit_chunks(p, u);
  long long incl = mine;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const long long o = __shfl_up(incl, d, kWave);
    if (lane >= d) incl += o;
  }
  if (lane == kWave - 1) lds[wave] = incl;
  if (threadIdx.x == 0) lds[kWaves] = units;       // an empty share starts past the last unit
  __syncthreads();
  long long total = 0, excl = incl - mine;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) excl += lds[w];
    total += lds[w];
  }
  // Consecutive workgroup ids go to the eight XCDs in turn; neighbouring
  // shares (which stage the same units' window rows) are kept on one XCD's L2.
  const int g = static_cast<int>(gridDim.x);
  Share s;
  s.b = g % 8 == 0 ? static_cast<int>(blockIdx.x % 8) * (g / 8) + static_cast<int>(blockIdx.x / 8)
                   : static_cast<int>(blockIdx.x);
  total = uniform(total);
  const long long b0 = share_begin(total, s.b), b1 = share_begin(total, s.b + 1);
  if (b0 < b1 && excl <= b0 && b0 < excl + mine) {
    long long c = excl;
    for (int u = u0; u < u1; ++u) {
      const int nc = unit_chunks(p, u);
      if (b0 < c + nc) {
        lds[kWaves] = u;
        lds[kWaves + 1] = b0 - c;
        lds[kWaves + 2] = c;
        break;
      }
      c += nc;
    }
  }
  __syncthreads();
  s.unit = uniform(static_cast<int>(lds[kWaves]));
  s.chunk = uniform(static_cast<int>(lds[kWaves + 1]));
  s.before = uniform(lds[kWaves + 2]);
  s.n = b1 - b0;
  s.total = total;
  __syncthreads();                                 // the scratch is reused by the caller
  return s;
}

struct Segment {
  int unit, L;
  int k0, k1;              // its keys
  long long before;        // chunks of all units before its unit
};

// Next segment of the share, of at most max_keys keys; false when the share is
// exhausted.
__device__ __forceinline__ bool next_segment(const ScoreParams &p, Share &s, Segment &seg, int max_keys = 1 << 30) {
  const int units = p.n_layers * p.batch * p.hkv;
  while (s.n > 0 && s.unit < units) {
    const int L = unit_len(p, s.unit);
    const int nc = (L + p.chunk_keys - 1) / p.chunk_keys;
    seg.unit = s.unit;
    seg.L = L;
    seg.before = s.before;
    const int c0 = s.chunk;
    if (c0 < nc) {
      const int take =
          min(static_cast<int>(min(static_cast<long long>(nc - c0), s.n)), max_keys / p.chunk_keys);
      seg.k0 = c0 * p.chunk_keys;
      seg.k1 = min(L, (c0 + take) * p.chunk_keys);
      s.n -= take;
      s.chunk += take;
      return true;
    }
    s.chunk = 0;
    s.before += nc;
    ++s.unit;
  }
  return false;
}

// The statistics of workgroup b's segment of a unit go to partial slot b +
// unit: along the chunk order every new segment raises b, the unit or both,
// so the slots of all segments differ, and grid + units - 1 slots hold them.

// ---------------------------------------------------------------------------
// Tiles.  Piece c of lane (l32, half) is the 16 bytes at 32 c + 16 half of its
// row: the contraction order is the same permutation for K and Q.
// ---------------------------------------------------------------------------
__device__ __forceinline__ f32x16_t mma_piece(bf16_t, uint4 k, uint4 q, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, k), __builtin_bit_cast(bf16x8_t, q), c,
                                                 0, 0, 0);
}
__device__ __forceinline__ f32x16_t mma_piece(float, uint4 k, uint4 q, f32x16_t c) {
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(k.x), __uint_as_float(q.x), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(k.y), __uint_as_float(q.y), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(k.z), __uint_as_float(q.z), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(k.w), __uint_as_float(q.w), c, 0, 0, 0);
}

__device__ __forceinline__ f32x16_t zero16() {
  f32x16_t z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}

// Key of accumulator register i of a tile at key kb.
__device__ __forceinline__ int tile_key(int kb, int i, int half) { return kb + 8 * (i >> 2) + 4 * half + (i & 3); }

template <typename T, int D>
struct Keys {
  typename ScoreCfg<T, D>::frags k[ScoreCfg<T, D>::KT];
};
template <typename T, int D>
struct Rows {
  typename ScoreCfg<T, D>::frags q;
};

// Where a wave's K fragments come from: the unit's rows and its length (keys
// at or past it read row 0 and are masked by the caller).
struct KeySource {
  const unsigned char *base;
  int L, l32, half;
};

template <typename T, int D>
__device__ __forceinline__ void load_key_tile(typename ScoreCfg<T, D>::frags &k, const KeySource &src, int kb) {
  const int key = kb + src.l32;
  const unsigned char *row =
      src.base + static_cast<size_t>(key < src.L ? key : 0) * ScoreCfg<T, D>::row_bytes + src.half * 16;
#pragma unroll
  for (int c = 0; c < ScoreCfg<T, D>::pieces; ++c) k[c] = *reinterpret_cast<const uint4 *>(row + c * 32);
}
template <typename T, int D>
__device__ __forceinline__ void load_keys(Keys<T, D> &kf, const KeySource &src, int g0) {
#pragma unroll
  for (int kt = 0; kt < ScoreCfg<T, D>::KT; ++kt) load_key_tile<T, D>(kf.k[kt], src, g0 + kt * 32);
}

// `qrow`: the lane's row of row tile 0 (plus 16 bytes for the upper half).
template <typename T, int D>
__device__ __forceinline__ uint4 q_piece(const unsigned char *qrow, int rt, int c) {
  return *reinterpret_cast<const uint4 *>(qrow + rt * kTileRows * ScoreCfg<T, D>::q_stride + c * 32);
}
template <typename T, int D>
__device__ __forceinline__ void load_rows(Rows<T, D> &r, const unsigned char *qrow, int rt) {
#pragma unroll
  for (int c = 0; c < ScoreCfg<T, D>::pieces; ++c) r.q[c] = q_piece<T, D>(qrow, rt, c);
}

template <typename T, int D>
__device__ __forceinline__ f32x16_t tile_products(const typename ScoreCfg<T, D>::frags &k, const Rows<T, D> &r) {
  f32x16_t s = zero16();
#pragma unroll
  for (int c = 0; c < ScoreCfg<T, D>::pieces; ++c) s = mma_piece(T{}, k[c], r.q[c], s);
  return s;
}

// One pipeline phase: the products of one tile into `s`, and between them the
// work on the previous tile's 16 registers: arg(x), exp2, add(i, e), each step
// one slot after the one before so that no instruction waits for its operand.
// RELOAD replaces each Q fragment by the one of row tile `next` after its last
// use.
template <typename T, int D, bool RELOAD, typename Arg, typename Add>
__device__ __forceinline__ void phase(f32x16_t &s, const typename ScoreCfg<T, D>::frags &k, Rows<T, D> &r,
                                      const unsigned char *qrow, int next, const f32x16_t &prev, Arg arg, Add add) {
  constexpr int P = ScoreCfg<T, D>::pieces;
  constexpr int per = 16 / P;
  float t[16];
  s = zero16();
#pragma unroll
  for (int c = 0; c < P; ++c) {
    s = mma_piece(T{}, k[c], r.q[c], s);
    if constexpr (RELOAD) r.q[c] = q_piece<T, D>(qrow, next, c);
#pragma unroll
    for (int e = 0; e < per; ++e) {
      if (c >= 2) add((c - 2) * per + e, t[(c - 2) * per + e]);
      if (c >= 1) t[(c - 1) * per + e] = fast_exp2(t[(c - 1) * per + e]);
      t[c * per + e] = arg(prev[c * per + e]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int e = 0; e < per; ++e) {
    add((P - 2) * per + e, t[(P - 2) * per + e]);
    t[(P - 1) * per + e] = fast_exp2(t[(P - 1) * per + e]);
  }
#pragma unroll
  for (int e = 0; e < per; ++e) add((P - 1) * per + e, t[(P - 1) * per + e]);
}

// A wave's row tiles rt0, rt0 + step, ... < tiles (at least one) of one group,
// pipelined: begin(rt) before the tile's first use, arg and add(kt, i, e) as in
// phase for register i of key tile kt, end(rt) after its last.  Each K
// fragment is replaced by the one of the group at `next` (none if negative)
// after its last use, so that these loads run under the last tile's
// exponentials and the other wave's work.
template <typename T, int D, typename Begin, typename Arg, typename Add, typename End>
__device__ __forceinline__ void walk_rows(Keys<T, D> &kf, const KeySource &src, int next, const unsigned char *qrow,
                                          int rt0, int step, int tiles, Begin begin, Arg arg, Add add, End end) {
  constexpr int KT = ScoreCfg<T, D>::KT;
  Rows<T, D> r;
  load_rows<T, D>(r, qrow, rt0);
  const auto add0 = [&](int i, float e) { add(0, i, e); };
  const auto add1 = [&](int i, float e) { add(1, i, e); };
  f32x16_t s0, s1;
  s0 = tile_products<T, D>(kf.k[0], r);
  int rt = rt0;
  if constexpr (KT == 2) {
    for (; rt + step < tiles; rt += step) {
      begin(rt);
      phase<T, D, true>(s1, kf.k[1], r, qrow, rt + step, s0, arg, add0);
      phase<T, D, false>(s0, kf.k[0], r, qrow, 0, s1, arg, add1);
      end(rt);
    }
    if (next >= 0) load_key_tile<T, D>(kf.k[0], src, next);
    begin(rt);
    phase<T, D, false>(s1, kf.k[1], r, qrow, 0, s0, arg, add0);
    if (next >= 0) load_key_tile<T, D>(kf.k[1], src, next + 32);
#pragma unroll
    for (int i = 0; i < 16; ++i) add1(i, fast_exp2(arg(s1[i])));
    end(rt);
  } else {
    if (rt0 + step < tiles) load_rows<T, D>(r, qrow, rt0 + step);
    for (; rt + step < tiles; rt += step) {
      begin(rt);
      phase<T, D, true>(s1, kf.k[0], r, qrow, min(rt + 2 * step, tiles - 1), s0, arg, add0);
      end(rt);
      s0 = s1;
    }
    if (next >= 0) load_key_tile<T, D>(kf.k[0], src, next);
    begin(rt);
#pragma unroll
    for (int i = 0; i < 16; ++i) add0(i, fast_exp2(arg(s0[i])));
    end(rt);
  }
}

// How the waves of a workgroup split a segment: row_waves waves share a group's
// row tiles (1 when the segment has a group for every wave; more in small
// calls, whose segments have fewer), the other factor takes different groups.
template <typename T, int D>
__device__ __forceinline__ int row_waves(const Segment &seg, int tiles) {
  const int groups = (seg.k1 - seg.k0 + ScoreCfg<T, D>::group - 1) / ScoreCfg<T, D>::group;
  int rw = 1;
  while (2 * rw * groups <= kWaves && 2 * rw <= tiles) rw *= 2;
  return rw;
}

// threadIdx.x, hidden from the optimiser: addresses derived from it are
// computed where they are used instead of being kept in registers (and
// spilled) across the key loop.
__device__ __forceinline__ int thread_id() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Row block [r0, r0 + 32 * tiles) of the unit's window rows into LDS (rows
// that do not exist are zero).  Loads go out in batches ahead of their stores.
template <typename T, int D>
__device__ __forceinline__ void stage_rows(const ScoreParams &p, const Segment &seg, unsigned char *qs, int r0,
                                           int tiles) {
  using C = ScoreCfg<T, D>;
  constexpr int pieces = C::row_bytes / 16;
  constexpr int kBatch = 7;
  const unsigned char *base = reinterpret_cast<const unsigned char *>(p.q_win) +
                              static_cast<size_t>(seg.unit) * p.rows * C::row_bytes;
  const int n = tiles * kTileRows * pieces;
  const int tid = thread_id();
  for (int i0 = 0; i0 < n; i0 += kBatch * kThreads) {
    uint4 v[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int i = i0 + j * kThreads + tid;
      const int r = r0 + i / pieces;
      const bool ok = i < n && r < p.rows && (seg.L >= p.w || seg.L - p.w + r % p.w >= 0);
      v[j] = ok ? *reinterpret_cast<const uint4 *>(base + static_cast<size_t>(r) * C::row_bytes + (i % pieces) * 16)
                : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int i = i0 + j * kThreads + tid;
      if (i < n) *reinterpret_cast<uint4 *>(qs + (i / pieces) * C::q_stride + (i % pieces) * 16) = v[j];
    }
  }
}

template <typename T, int D>
__device__ __forceinline__ KeySource key_source(const ScoreParams &p, const Segment &seg, int l32, int half) {
  const size_t cunit = static_cast<size_t>(p.layer0) * p.batch * p.hkv + seg.unit;
  return KeySource{reinterpret_cast<const unsigned char *>(p.k) + cunit * p.cap * ScoreCfg<T, D>::row_bytes, seg.L,
                   l32, half};
}

// Row blocks of a unit: the fewest that fit the LDS stage, of equal size.
template <typename T, int D>
__device__ __forceinline__ int block_tiles(const ScoreParams &p) {
  const int tiles = (p.rows + kTileRows - 1) / kTileRows;
  const int blocks = (tiles + ScoreCfg<T, D>::max_tiles - 1) / ScoreCfg<T, D>::max_tiles;
  return (tiles + blocks - 1) / blocks;
}

// Last key that window row r sees (-1 or less: none).
__device__ __forceinline__ int last_visible(const ScoreParams &p, int L, int r) {
  return p.causal ? L - p.w + r % p.w : L - 1;
}

// Keys every valid window row sees: below L, and (causal) up to L - w.
__device__ __forceinline__ int full_end(const ScoreParams &p, int L) { return p.causal ? min(L, L - p.w + 1) : L; }

// ---------------------------------------------------------------------------
// Statistics pass.  Every row has a reference m, the whole number below the
// largest logit among the segment's first 32 keys (finite unless the row sees no
// key of the segment), and sums 2^(x - m) over the segment's keys: no running
// maximum per key, and the largest term is at least 1.  An exponent is rounded
// to its own size, so a group of keys that sums to more than kFarSum in a row is
// done again against its own maxima (the tile's 32 rows at once); being whole
// numbers too, these leave sums that scale to the reference exactly.  A sum past
// kMaxSum, far below fp32's largest value (the sums of the waves and of a row's
// segments are added later), makes the whole segment be done again with its
// exact maxima as references.
//
// Measured: 512 bf16 rows at head_dim 128 over 9,000 keys with logits of
// standard deviation 8 and 16: error of the scores (2-norm) 7.4e-7 and 1.19e-6
// with the first references alone, 6.8e-7 and 9.7e-7 so (with a running maximum
// per key 6.6e-7 and 9.3e-7).  It takes time only where there are such keys: 7B
// 16K two passes 450 -> 453 us at standard deviation 1, 462 -> 461 us at 4,
// 464 -> 634 us at 8, where most groups hold some.  From sums of 2^16 on it
// takes more time (469 and 742 us) for 1 to 2% less error, from 2^24 on less
// (466 and 541 us) for 2% more.
// ---------------------------------------------------------------------------
constexpr float kFarSum = 1048576.f;             // 2^20
constexpr float kMaxSum = 1.2676506e30f;         // 2^100

// Largest visible logit of the lane's row in one tile at key kb (lim: the last
// key the row sees).
__device__ __forceinline__ float tile_max(const ScoreParams &p, const f32x16_t &s, int kb, int lim, int half) {
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) m = fmaxf(m, tile_key(kb, i, half) <= lim ? s[i] * p.scale_log2 : -INFINITY);
  return m;
}

// max over the two lane halves (lanes l and l ^ 32 hold the same row).
__device__ __forceinline__ float half_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float half_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One row tile of the group at g0, against its own maxima where these are above
// the references.
template <typename T, int D>
__device__ __forceinline__ void far_tile(const ScoreParams &p, const Segment &seg, const Keys<T, D> &kf,
                                         const unsigned char *qrow, const float *mref, float *acc, int r0, int rt,
                                         int g0, int l32, int half) {
  constexpr int KT = ScoreCfg<T, D>::KT;
  Rows<T, D> r;
  load_rows<T, D>(r, qrow, rt);
  const int lim = last_visible(p, seg.L, r0 + rt * kTileRows + l32);
  const float ref = mref[rt * kTileRows + l32];
  f32x16_t s[KT];
  float m = ref;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    s[kt] = tile_products<T, D>(kf.k[kt], r);
    m = fmaxf(m, floorf(half_max(tile_max(p, s[kt], g0 + kt * 32, lim, half))));
  }
  float sum = 0.f;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float e = fast_exp2(fmaf(s[kt][i], p.scale_log2, -m));
      sum += tile_key(g0 + kt * 32, i, half) <= lim ? e : 0.f;
    }
  }
  sum = half_sum(sum);
  acc[rt * kTileRows] += m > ref ? __builtin_amdgcn_ldexpf(sum, static_cast<int>(fminf(m - ref, 1024.f))) : sum;
}

// Sums (or, with MAX, maxima) of a wave's groups, per row in `acc`.
template <typename T, int D, bool MAX>
__device__ __forceinline__ void stats_groups(const ScoreParams &p, const Segment &seg, const KeySource &src,
                                             const unsigned char *qrow, const float *mref, float *acc, int r0,
                                             int tiles, int wave, int rw) {
  using C = ScoreCfg<T, D>;
  const int stride = kWaves / rw * C::group;
  const int rt0 = wave % rw;
  const int l32 = src.l32, half = src.half;
  const float c = p.scale_log2;
  const int end = full_end(p, seg.L);
  int g0 = seg.k0 + wave / rw * C::group;
  if (g0 >= seg.k1) return;
  Keys<T, D> kf;
  load_keys<T, D>(kf, src, g0);
  for (; g0 < seg.k1; g0 += stride) {
    const int next = g0 + stride < seg.k1 ? g0 + stride : -1;
    if constexpr (MAX) {
      for (int rt = rt0; rt < tiles; rt += rw) {
        Rows<T, D> r;
        load_rows<T, D>(r, qrow, rt);
        const int lim = last_visible(p, seg.L, r0 + rt * kTileRows + l32);
        float a = acc[rt * kTileRows];
#pragma unroll
        for (int kt = 0; kt < C::KT; ++kt)
          a = fmaxf(a, tile_max(p, tile_products<T, D>(kf.k[kt], r), g0 + kt * 32, lim, half));
        acc[rt * kTileRows] = half_max(a);
      }
      if (next >= 0) load_keys<T, D>(kf, src, next);
    } else {
      float m, z[4], a;
      int lim;
      unsigned far = 0;                            // row tiles to do again
      const auto begin = [&](int rt) {
        m = mref[rt * kTileRows + l32];
        a = acc[rt * kTileRows];
        z[0] = z[1] = z[2] = z[3] = 0.f;
      };
      const auto arg = [&](float x) { return fmaf(x, c, -m); };
      const auto end_tile = [&](int rt) {
        const float sum = half_sum((z[0] + z[1]) + (z[2] + z[3]));
        const bool again = __any(!(sum <= kFarSum));
        far |= again ? 1u << rt : 0u;
        acc[rt * kTileRows] = a + (again ? 0.f : sum);
      };
      if (g0 + C::group <= end) {
        walk_rows<T, D>(kf, src, next, qrow, rt0, rw, tiles, begin, arg,
                        [&](int, int i, float e) { z[i & 3] += e; }, end_tile);
      } else {
        walk_rows<T, D>(
            kf, src, next, qrow, rt0, rw, tiles,
            [&](int rt) {
              begin(rt);
              lim = last_visible(p, seg.L, r0 + rt * kTileRows + l32) - tile_key(g0, 0, half);
            },
            arg, [&](int kt, int i, float e) { z[i & 3] += tile_key(kt * 32, i, 0) <= lim ? e : 0.f; }, end_tile);
      }
      // Out of the way of the loop (small calls run its code cold: 0.5 us of 16 us).
      if (__builtin_expect(far != 0, 0)) {         // their keys again, then the next group's
        load_keys<T, D>(kf, src, g0);
        for (; far != 0; far &= far - 1)
          far_tile<T, D>(p, seg, kf, qrow, mref, acc, r0, __ffs(far) - 1, g0, l32, half);
        if (next >= 0) load_keys<T, D>(kf, src, next);
      }
    }
  }
}

template <typename T, int D>
__global__ __launch_bounds__(kThreads, 1) void score_stats_kernel(ScoreParams p) {
  using C = ScoreCfg<T, D>;
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::stats_lds];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
  const int l32 = lane & 31, half = lane >> 5;
  float *sums = reinterpret_cast<float *>(smem + C::q_bytes);              // [wave][max_rows]
  float *mref = reinterpret_cast<float *>(smem + C::q_bytes + C::sum_bytes);  // [max_rows]
  float *acc = sums + wave * C::max_rows + l32;    // both halves of a row write the same value
  const unsigned char *qrow = smem + l32 * C::q_stride + half * 16;
  const int btiles = block_tiles<T, D>(p);
  Share share = find_share(p, reinterpret_cast<long long *>(smem));
  Segment seg;
  while (next_segment(p, share, seg)) {
    const KeySource src = key_source<T, D>(p, seg, l32, half);
    float *part = p.row_part + static_cast<size_t>(share.b + seg.unit) * p.rows_pad * 2;
    for (int r0 = 0; r0 < p.rows; r0 += btiles * kTileRows) {
      const int tiles = min(btiles, (p.rows - r0 + kTileRows - 1) / kTileRows);
      __syncthreads();                             // the previous rows and sums are consumed
      stage_rows<T, D>(p, seg, smem, r0, tiles);
      for (int rt = 0; rt < tiles; ++rt) acc[rt * kTileRows] = 0.f;
      __syncthreads();
      // References from the segment's first 32 keys, the row tiles dealt to the waves.
      if (wave < tiles) {
        Keys<T, D> kf;
        load_key_tile<T, D>(kf.k[0], src, seg.k0);
        for (int rt = wave; rt < tiles; rt += kWaves) {
          Rows<T, D> r;
          load_rows<T, D>(r, qrow, rt);
          const f32x16_t s = tile_products<T, D>(kf.k[0], r);
          const int lim = last_visible(p, seg.L, r0 + rt * kTileRows + l32);
          const float m = floorf(half_max(tile_max(p, s, seg.k0, lim, half)));
          if (half == 0) mref[rt * kTileRows + l32] = m;
        }
      }
      __syncthreads();
      const int rw = row_waves<T, D>(seg, tiles);
      stats_groups<T, D, false>(p, seg, src, qrow, mref, acc, r0, tiles, wave, rw);
      bool bad = false;
      for (int rt = 0; rt < tiles; ++rt) bad |= !(acc[rt * kTileRows] <= kMaxSum);
      if (__syncthreads_or(bad)) {                 // a sum is too large against its reference
        for (int rt = 0; rt < tiles; ++rt) acc[rt * kTileRows] = -INFINITY;
        stats_groups<T, D, true>(p, seg, src, qrow, mref, acc, r0, tiles, wave, rw);
        __syncthreads();
        for (int r = thread_id(); r < tiles * kTileRows; r += kThreads) {
          float m = -INFINITY;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) m = fmaxf(m, sums[w * C::max_rows + r]);
          mref[r] = floorf(m);
        }
        __syncthreads();
        for (int rt = 0; rt < tiles; ++rt) acc[rt * kTileRows] = 0.f;
        stats_groups<T, D, false>(p, seg, src, qrow, mref, acc, r0, tiles, wave, rw);
        __syncthreads();
      }
      for (int r = thread_id(); r < tiles * kTileRows && r0 + r < p.rows; r += kThreads) {
        float z = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) z += sums[w * C::max_rows + r];
        *reinterpret_cast<float2 *>(part + (r0 + r) * 2) = make_float2(mref[r], z);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Mass pass.
// ---------------------------------------------------------------------------

// The workgroups whose shares hold chunks of the segment's unit, in order.  The
// share of chunk c is the last one that begins at or before it, ceil((c + 1) *
// grid / total) - 1.  With at least one chunk per share these are consecutive;
// with fewer, each chunk has a workgroup of its own and some have none.
struct UnitShares {
  int n;           // how many
  int first;       // dense: the first one
  int chunk0, total, grid;

  __device__ UnitShares(const ScoreParams &p, const Share &s, const Segment &seg) {
    grid = static_cast<int>(gridDim.x);
    const int nc = (seg.L + p.chunk_keys - 1) / p.chunk_keys;
    total = 0;
    if (s.total >= grid) {
      first = static_cast<int>(((seg.before + 1) * grid + s.total - 1) / s.total) - 1;
      n = static_cast<int>(((seg.before + nc) * grid + s.total - 1) / s.total) - first;
    } else {
      total = static_cast<int>(s.total);
      chunk0 = static_cast<int>(seg.before);
      n = nc;
    }
  }
  __device__ __forceinline__ int workgroup(int i) const {
    return total == 0 ? first + i : ((chunk0 + i + 1) * grid + total - 1) / total - 1;
  }
};

// (reference, 1/sum) of row r of the segment's unit, from the statistics partials
// of the unit's segments or the decode statistics (there it is the maximum);
// absent or empty rows get (+inf, 0), so that they add exactly zero.
constexpr int kNearLog2 = 8;
__device__ __forceinline__ float2 row_norm(const ScoreParams &p, const Segment &seg, const UnitShares &u, int r) {
  const bool valid = r < p.rows && (seg.L >= p.w || seg.L - p.w + r % p.w >= 0);
  float2 n = make_float2(INFINITY, 0.f);
  if (!valid) return n;
  if (p.given) {
    const float *st = p.given + (static_cast<size_t>(seg.unit) * p.rows + r) * 2;
    const float m = st[0], z = st[1];
    if (m != -INFINITY && m != INFINITY && z > 0.f) n = make_float2(m, 1.f / z);
    return n;
  }
  const float *part = p.row_part + (static_cast<size_t>(seg.unit) * p.rows_pad + r) * 2;
  constexpr int kBatch = 8;                        // partials requested at once
  float M = -INFINITY;
  double Z = 0.0;
  for (int s0 = 0; s0 < u.n; s0 += kBatch) {
    float m[kBatch], z[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const float *st = part + static_cast<size_t>(u.workgroup(min(s0 + j, u.n - 1))) * p.rows_pad * 2;
      m[j] = st[0];
      z[j] = st[1];
    }
    float mb = M;
#pragma unroll
    for (int j = 0; j < kBatch; ++j) mb = s0 + j < u.n ? fmaxf(mb, m[j]) : mb;
    if (mb == -INFINITY) continue;
    Z *= static_cast<double>(fast_exp2(M - mb));
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (s0 + j < u.n && m[j] != -INFINITY)
        Z += static_cast<double>(z[j]) * static_cast<double>(fast_exp2(m[j] - mb));
    M = mb;
  }
  if (M != -INFINITY && Z > 0.0) {
    // M is a reference, and log2 Z an upper bound of how far above it the row's
    // largest logit lies.  Where that is far, M is raised to near it, by a whole
    // number, so that the exponents of the heavy keys are small in the mass pass.
    const float inv = static_cast<float>(1.0 / Z);
    const float m = M + static_cast<float>(max(126 - kNearLog2 - static_cast<int>(__float_as_uint(inv) >> 23), 0));
    n = make_float2(m, __builtin_amdgcn_ldexpf(inv, static_cast<int>(m - M)));
  }
  return n;
}

// Sum over the 32 lanes of each half, of the 16 * KT registers of a group:
// each step halves the registers and folds one bit of the register index into
// the lane index, so the lane ends with the total of one key (KT = 2), or the
// lane pairs l, l ^ 16 with the same key's (KT = 1).  The lane partner of a
// step differs in the step's bit (and may differ in lower ones, which are
// summed over later).
template <int KT>
__device__ __forceinline__ float fold_keys(float (&a)[KT * 16], int lane) {
  constexpr int kRor8 = 0x128;
  float b[16];
  if constexpr (KT == 2) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {               // key tile <-> lane bit 4
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[i]), __float_as_uint(a[16 + i]), false, false);
      b[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[i]), __float_as_uint(a[i]), false, false);
      b[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {                  // register bit 3 <-> lane bit 3
    const float own = (lane & 8) ? b[8 + i] : b[i], other = (lane & 8) ? b[i] : b[8 + i];
    b[i] = own + dpp<kRor8>(other);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {                  // register bit 2 <-> lane bit 2
    const float own = (lane & 4) ? b[4 + i] : b[i], other = (lane & 4) ? b[i] : b[4 + i];
    b[i] = own + dpp<kDppHalfMirror>(other);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {                  // register bit 1 <-> lane bit 1
    const float own = (lane & 2) ? b[2 + i] : b[i], other = (lane & 2) ? b[i] : b[2 + i];
    b[i] = own + dpp<kDppXor2>(other);
  }
  const float own = (lane & 1) ? b[1] : b[0], other = (lane & 1) ? b[0] : b[1];
  return own + dpp<kDppXor1>(other);
}

// Key of the group that fold_keys leaves in `lane`.
template <int KT>
__device__ __forceinline__ int folded_key(int lane) {
  return (KT == 2 ? (lane & 16) * 2 : 0) + ((lane & 8) << 1) + ((lane & 4) << 1) + ((lane & 32) >> 3) + (lane & 3);
}

// The score of `key` over the row block at r0.  With several blocks the sums
// are added with what each addition rounds off kept aside (in `lost`, by key
// of the segment) and added last, so that the number of blocks costs no
// precision.
__device__ __forceinline__ void add_block(const ScoreParams &p, float *out, float *lost, const Segment &seg, int r0,
                                          int btiles, int key, float tot) {
  if (r0 == 0) {
    out[key] = tot;
    if (p.rows > btiles * kTileRows) lost[key - seg.k0] = 0.f;
    return;
  }
  const float a = out[key], s = a + tot;
  const float b = s - a;
  const float e = lost[key - seg.k0] + ((a - (s - b)) + (tot - b));
  const bool last = r0 + btiles * kTileRows >= p.rows;
  out[key] = last ? s + e : s;
  lost[key - seg.k0] = e;
}

template <typename T, int D>
__global__ __launch_bounds__(kThreads, 1) void score_mass_kernel(ScoreParams p) {
  using C = ScoreCfg<T, D>;
  constexpr int KT = C::KT;
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::mass_lds];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = uniform(static_cast<int>(threadIdx.x) / kWave);
  const int l32 = lane & 31, half = lane >> 5;
  float2 *norm = reinterpret_cast<float2 *>(smem + C::q_bytes);            // [max_rows] (max, 1/sum)
  const unsigned char *qrow = smem + l32 * C::q_stride + half * 16;
  __shared__ int s_next;
  __shared__ float part[kWaves][kWave];
  __shared__ float lost[C::lost_keys];
  const float c = p.scale_log2;
  const int btiles = block_tiles<T, D>(p);
  Share share = find_share(p, reinterpret_cast<long long *>(smem));
  Segment seg;
  const bool blocks = p.rows > btiles * kTileRows;
  while (next_segment(p, share, seg, blocks ? C::lost_keys : 1 << 30)) {
    const KeySource src = key_source<T, D>(p, seg, l32, half);
    float *out = p.scores + static_cast<size_t>(seg.unit) * p.cap;
    const int end = full_end(p, seg.L);
    const UnitShares shares(p, share, seg);
    for (int r0 = 0; r0 < p.rows; r0 += btiles * kTileRows) {
      const int tiles = min(btiles, (p.rows - r0 + kTileRows - 1) / kTileRows);
      const int rw = row_waves<T, D>(seg, tiles);
      int g0 = seg.k0 + wave / rw * C::group;
      Keys<T, D> kf;
      load_keys<T, D>(kf, src, g0 < seg.k1 ? g0 : seg.k0);
      __syncthreads();                             // every wave is done with the previous rows
      if (threadIdx.x == 0) s_next = kWaves;
      stage_rows<T, D>(p, seg, smem, r0, tiles);
      for (int r = thread_id(); r < tiles * kTileRows; r += kThreads)
        norm[r] = row_norm(p, seg, shares, r0 + r);
      __syncthreads();
      // The older wave of a SIMD wins most issue slots and would finish a fixed
      // share early, so the groups after the first are taken from a counter
      // (which wave computes a score does not change it).
      int next;
      for (; g0 >= 0 && g0 < seg.k1; g0 = next) {
        next = -1;
        if (rw == 1) {
          int taken = 0;
          if (lane == 0) taken = atomicAdd(&s_next, 1);
          const int g = seg.k0 + uniform(taken) * C::group;
          if (g < seg.k1) next = g;
        }
        float acc[KT * 16];
#pragma unroll
        for (int i = 0; i < KT * 16; ++i) acc[i] = 0.f;
        float2 n;
        int lim;
        const auto arg = [&](float x) { return fmaf(x, c, -n.x); };
        if (g0 + C::group <= end) {
          walk_rows<T, D>(
              kf, src, next, qrow, wave % rw, rw, tiles, [&](int rt) { n = norm[rt * kTileRows + l32]; }, arg,
              [&](int kt, int i, float e) { acc[kt * 16 + i] = fmaf(e, n.y, acc[kt * 16 + i]); }, [](int) {});
        } else {
          walk_rows<T, D>(
              kf, src, next, qrow, wave % rw, rw, tiles,
              [&](int rt) {
                n = norm[rt * kTileRows + l32];
                lim = last_visible(p, seg.L, r0 + rt * kTileRows + l32) - tile_key(g0, 0, half);
              },
              arg,
              [&](int kt, int i, float e) {
                acc[kt * 16 + i] = fmaf(tile_key(kt * 32, i, 0) <= lim ? e : 0.f, n.y, acc[kt * 16 + i]);
              },
              [](int) {});
        }
        const float tot = fold_keys<KT>(acc, lane);
        const int key = g0 + folded_key<KT>(lane);
        const bool mine = (KT == 2 || !(lane & 16)) && key < seg.k1;
        if (rw == 1) {
          if (mine) add_block(p, out, lost, seg, r0, btiles, key, tot);
        } else {
          part[wave][lane] = tot;                  // one group per wave: summed after the loop
        }
      }
      if (rw > 1) {
        __syncthreads();
        const int key = seg.k0 + wave / rw * C::group + folded_key<KT>(lane);
        if (wave % rw == 0 && (KT == 2 || !(lane & 16)) && key < seg.k1) {
          float tot = part[wave][lane];
          for (int i = 1; i < rw; ++i) tot += part[wave + i][lane];
          add_block(p, out, lost, seg, r0, btiles, key, tot);
        }
      }
    }
  }
}

// Chunks are the unit of load balance over the persistent grid: 512 keys, one
// 64-key group for each wave, when every CU gets many of them; else 64 keys,
// so that mid-sized and small calls spread evenly over the CUs.  Units
// of at most 512 keys stay whole when there is one for every CU: cutting them
// would stage a unit's window rows more than once (480 units of 259 keys, 512
// window rows: 143 us in 64-key chunks, 105 us whole, with one block of rows).
void score_plan(ScoreParams &p, int units, int &grid) {
  p.chunk_keys = kScoreChunk;
  const bool whole_units = p.cap <= kScoreChunk && units >= p.cus;
  if (!whole_units && static_cast<long long>(units) * ((p.cap + p.chunk_keys - 1) / p.chunk_keys) < 8LL * p.cus)
    p.chunk_keys = 64;
  const long long chunks = static_cast<long long>(units) * ((p.cap + p.chunk_keys - 1) / p.chunk_keys);
  long long g = chunks < p.cus ? chunks : p.cus;
  if (!p.given && g > p.part_slots - units + 1) g = p.part_slots - units + 1;   // a slot for every segment
  grid = static_cast<int>(g);
}

template <typename T, int D>
hipError_t launch_typed(const ScoreParams &p0, hipStream_t s) {
  ScoreParams p = p0;
  int grid;
  score_plan(p, p.n_layers * p.batch * p.hkv, grid);
  if (!p.given) {
    hipLaunchKernelGGL((score_stats_kernel<T, D>), dim3(grid), dim3(kThreads), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((score_mass_kernel<T, D>), dim3(grid), dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

}  // namespace

size_t score_min_workspace_bytes(int units, int capacity, int rows) {
  const size_t rows_pad = static_cast<size_t>((rows + 15) / 16 * 16);
  const size_t chunks = static_cast<size_t>((capacity + kScoreChunk - 1) / kScoreChunk);
  return static_cast<size_t>(units) * rows_pad * (chunks + 1) * 2 * sizeof(float);
}

size_t score_workspace_bytes(int units, int capacity, int rows) {
  const size_t rows_pad = static_cast<size_t>((rows + 15) / 16 * 16);
  const size_t slots = (static_cast<size_t>(units) + kScoreMaxGrid) * rows_pad * 2 * sizeof(float);
  const size_t least = score_min_workspace_bytes(units, capacity, rows);
  return slots > least ? slots : least;
}

hipError_t launch_score(const ScoreParams &p, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0) {
    if (head_dim == 64) return launch_typed<float, 64>(p, s);
    return launch_typed<float, 128>(p, s);
  }
  if (head_dim == 64) return launch_typed<bf16_t, 64>(p, s);
  return launch_typed<bf16_t, 128>(p, s);
}

}  // namespace reco
