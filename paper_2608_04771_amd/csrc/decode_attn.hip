// GQA split-K decode attention over ragged per-head KV caches (gfx950).
//
// One "unit" is a (layer, sequence, kv head) with n valid cache rows and G
// query heads.  The grid is (splits, units): workgroup (s, u) walks a
// contiguous range of 32-key tiles of unit u with its waves (four, or eight
// where a CU holds one workgroup that bounds the call) interleaved over the
// tiles, so the workgroup streams one contiguous stretch of K and V.
//
// Per 32-key tile a wave computes, on the matrix cores,
//   S^T = K_tile . Q^T            (M = 16 keys per half, N = 16 padded queries)
//   O^T += V_tile^T . P^T         (M = 16 head-dim rows per d-tile, N = 16 queries)
// The S^T accumulator already holds, per lane, the probabilities the P^T
// operand needs (same lane, same element slot), so P never leaves registers.
// K and V are streamed with coalesced non-temporal 16-byte loads (each 128-byte
// line read whole, nothing allocated in L2) and staged through LDS, one after
// the other through one buffer: K is re-read in the MFMA operand layout, V
// column-wise.  The registers of a staged half tile are refilled at once, and
// tiles inside the cache need no masks and no addresses of their own (a tile
// ahead in a second set of registers, waited for at the end of the same turn,
// against this: 28 one-layer calls in a graph 359 -> 333 us, 128 even units of
// 18,000 rows 191 -> 182 us, 32 fp32 units of 3,000 to 12,000 rows at head_dim
// 64 137 -> 99 us; with two sets used in turn, two tiles ahead, 28 one-layer
// calls take as long and the others 1 to 5% longer: more on its way per CU
// gives nothing).  Softmax is online in the log2 domain with fp32 statistics.
// The waves' (max, sum, O) states are merged through LDS and written as one
// split partial: every store and load of that merge is 16 bytes on a row pitch
// free of bank conflicts (as 4-byte stores on a pitch of D, 16 lanes on one
// bank, it took 2 us of each call: 28 one-layer calls 397 -> 359 us, 256 units
// x 1,100 rows 27.8 -> 26.5 us, 112 units x 9,645 rows 88.2 -> 86.4 us).  A
// second kernel merges the splits of each unit, writes out / lse and commits the
// optional append (so no workgroup of the attention kernel races on len); a unit
// covered by a single workgroup (one split) is finalised by that workgroup, with
// no second launch.  Merging in the last-finishing workgroup instead would need
// device-scope fences, which on this chip write back and invalidate the L2 that
// the streaming workgroups depend on.
#include "reco_device.hpp"
#include "decode_attn.hpp"
#include "decode_plan.hpp"

#include <math.h>

#include <atomic>
#include <mutex>
#include <type_traits>

namespace reco {

namespace {

constexpr int kTile = kDecodeTile;   // keys per wave iteration
constexpr int kMaxSplits = kDecodeMaxSplits;

template <typename T, int D, int NW = 4>
struct DecodeCfg {
  using MF = Mfma<T>;
  static constexpr int kpl = MF::kPerLane;
  static constexpr int dq = D / 4;                  // head-dim elements per lane group for Q.K
  static constexpr int qk_steps = dq / kpl;         // MFMAs per 16-key half
  static constexpr int dtiles = D / 16;             // output head-dim tiles
  static constexpr int pv_ops = kTile / MF::kPerOp;  // MFMAs per d-tile per 32-key tile
  static constexpr int row_bytes = D * (int)sizeof(T);
  static constexpr int lds_stride = row_bytes + 8;  // padded row pitch of the V stage
  static constexpr int k_stride = row_bytes + 16;   // padded, 16-byte aligned pitch of the K stage
  static constexpr int wave_stage = kTile * k_stride;   // K, then V of the same tile (a wave's LDS accesses run in order)
  static constexpr int stage_bytes = NW * wave_stage;
  // Cross-wave merge: a lane's four consecutive outputs are one 16-byte store,
  // and the row pitch shifts the eight rows stored together over all banks.
  static constexpr int merge_pitch = D + 4;
  static constexpr int merge_bytes = NW * 16 * (2 + merge_pitch) * 4;
  static constexpr int smem_bytes = stage_bytes > merge_bytes ? stage_bytes : merge_bytes;
  // Coalesced tile loads: per instruction the wave reads 1 KB of consecutive
  // rows (lane l takes 16 bytes at l * 16), so every 128-byte line is read whole.
  static constexpr int lanes_per_row = row_bytes / 16;
  static constexpr int rows_per_inst = kWave / lanes_per_row;
  static constexpr int v_insts = kTile / rows_per_inst;
  // Two workgroups of four waves per CU (two waves per SIMD) where a tile and the
  // outputs fit in 256 registers; the fp32 head_dim-128 variant needs more.
  static constexpr int min_wgs = (sizeof(T) == 4 && D == 128) || NW == 8 ? 1 : 2;
};

// Registers of one 32-key tile: K and V as coalesced 16-byte pieces bound
// for the LDS stages (K is re-read from LDS in the MFMA operand layout).
template <typename T, int D>
using TileRows = uint4[DecodeCfg<T, D>::v_insts];
template <typename T, int D>
struct TileRegs {
  TileRows<T, D> kreg;
  TileRows<T, D> vreg;
};

// Issue the loads of one tile's K or V rows, starting at key kb.  A tile inside
// the cache is one stretch of memory.  In the last one, key n_cache comes from
// the appended row, and rows past the end read row 0, so that every address
// stays inside the unit; what they bring is masked where it is used, so that
// nothing here waits for a load.
template <typename T, int D>
__device__ __forceinline__ void load_rows(TileRows<T, D> &reg, int kb, int n_cache, bool append,
                                          const T *base, const T *row_new, int lane) {
  using Cfg = DecodeCfg<T, D>;
  if (kb + kTile <= n_cache) {
    const unsigned char *p = reinterpret_cast<const unsigned char *>(base + static_cast<size_t>(kb) * D) + lane * 16;
#pragma unroll
    for (int i = 0; i < Cfg::v_insts; ++i) reg[i] = nt_load_u4(p + i * (kWave * 16));
  } else {
    const int sub = (lane % Cfg::lanes_per_row) * 16;
#pragma unroll
    for (int i = 0; i < Cfg::v_insts; ++i) {
      const int key = kb + i * Cfg::rows_per_inst + lane / Cfg::lanes_per_row;
      const T *row = key == n_cache && append ? row_new : base + (key < n_cache ? static_cast<size_t>(key) * D : 0);
      reg[i] = nt_load_u4(reinterpret_cast<const unsigned char *>(row) + sub);
    }
  }
}

template <typename T>
__device__ __forceinline__ T lds_elem(const unsigned char *p) {
  return *reinterpret_cast<const T *>(p);
}

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;

// Gather the V^T fragment of MFMA `c` for head-dim tile `dt` from the staged
// tile: lane (col, grp) needs, at head-dim column dt*16 + col, the keys of
// element e = c * kpl + j, key (e / 4) * 16 + 4 * grp + (e % 4).
// bf16: two LDS transpose reads.  Within each 16-lane group, lane j supplies
// the 8 bytes at row key0 + j / 4, columns d0 + 4 * (j % 4) .. + 3, and lane i
// receives element i % 4 of the rows supplied by lanes 4r + i / 4, r = 0..3,
// i.e. column d0 + i of rows key0 .. key0 + 3: four consecutive keys of one
// head-dim column, as the operand wants.
template <typename T, int D>
__device__ __forceinline__ typename Mfma<T>::frag vt_frag(const unsigned char *stage, int c, int grp, int dt,
                                                          int col) {
  using Cfg = DecodeCfg<T, D>;
  typename Mfma<T>::frag a;
  if constexpr (Cfg::kpl == 1) {
    const int e = c;
    const int kl = (e >> 2) * 16 + 4 * grp + (e & 3);
    a = lds_elem<float>(stage + kl * Cfg::lds_stride + (dt * 16 + col) * 4);
  } else {
    static_assert(Cfg::lds_stride % 8 == 0, "transpose reads need 8-byte aligned rows");
    const int key0 = 32 * c + 4 * grp + col / 4;
    const int cb = (dt * 16 + 4 * (col % 4)) * 2;
    const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4_t *)(stage + key0 * Cfg::lds_stride + cb));
    const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4_t *)(stage + (key0 + 16) * Cfg::lds_stride + cb));
    const short v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = __builtin_bit_cast(__bf16, v[j]);
  }
  return a;
}

// P^T fragment of MFMA `c`: the probabilities pv[e] for e = c * kpl + j.
template <typename T>
__device__ __forceinline__ typename Mfma<T>::frag pt_frag(const float (&pv)[8], int c) {
  if constexpr (Mfma<T>::kPerLane == 1) {
    return pv[c];
  } else {
    return pack_frag8(pv);
  }
}

// The lengths of a call's units (kDecodeHeldUnits at most), two in a lane.
struct HeldLengths {
  static constexpr int kPer = kDecodeHeldUnits / kWave;
  int len[kPer];

  __device__ __forceinline__ HeldLengths(const DecodeParams &p, int units, int lane) {
    const int32_t *src = p.len + static_cast<size_t>(p.layer0) * p.batch * p.hkv;
#pragma unroll
    for (int i = 0; i < kPer; ++i) len[i] = lane + i * kWave < units ? src[lane + i * kWave] : -1;
  }
  // `unit` is the same in all lanes.
  __device__ __forceinline__ int of(int unit) const {
    static_assert(kPer == 2, "one of two registers");
    return __builtin_amdgcn_readlane(unit < kWave ? len[0] : len[1], unit % kWave);
  }
  // Whether the units take all splits launched: unless they are long and even
  // (the longest less than a quarter above the mean).
  // The first tile waits for this: the folds by the vector unit take 0.35 us less
  // than by shuffles (112 units of 6,000 to 6,256 rows in 16,640: 56.6 -> 56.2 us).
  __device__ __forceinline__ bool all_splits(const DecodeParams &p, int units) const {
    constexpr int kLongRows = 3200;
    if (!__any(max(len[0], len[1]) >= kLongRows)) return true;
    float total = 0.f, top = 0.f;                  // in rows
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const float rows = static_cast<float>(max(min(len[i], p.cap), 0));
      total += rows;
      top = fmaxf(top, rows);
    }
    total = wave_fold(total, [](float a, float b) { return a + b; });
    top = wave_fold(top, [](float a, float b) { return fmaxf(a, b); });
    return __builtin_amdgcn_readfirstlane(4.f * top * static_cast<float>(units) >= 5.f * total);
  }
};

// HELD: the call may launch more splits than long even units take, and the
// workgroups decide.  A form of its own, as its code in front of the others'
// start costs them up to 1% (256 units of 1,100 rows: with it 23.22 us, without
// 23.06 us; two fp32 units of 2,048 at head_dim 64: 8.71 us, 8.62 us).
template <typename T, int D, int NW, bool HELD>
__global__ __launch_bounds__(NW * kWave, (DecodeCfg<T, D, NW>::min_wgs)) void decode_split_kernel(DecodeParams p) {
  using Cfg = DecodeCfg<T, D, NW>;
  constexpr int kThreads = NW * kWave;
  using MF = Mfma<T>;
  using frag = typename MF::frag;
  __shared__ __attribute__((aligned(16))) unsigned char smem[Cfg::smem_bytes];

  const int lane = threadIdx.x & (kWave - 1);
  // the same in all lanes: what follows from it is scalar
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int col = lane & 15;
  const int grp = lane >> 4;
  int split = blockIdx.x, unit = blockIdx.y;
  int active = p.splits;                           // splits that share the unit
  int len_in = 0;
  if constexpr (HELD) {
    // Every workgroup finds the same from the same lengths (no one changes them
    // before the merge kernel: even_splits is 2 or more).  Its own unit's is one
    // of them; a load of its own would come after the decision.
    const int units = static_cast<int>(gridDim.y);
    const HeldLengths held(p, units, lane);
    if (!held.all_splits(p, units)) {
      // The first workgroups take the splits there are, as in a grid of these
      // alone (so that they spread over the XCDs and CUs alike); the others
      // leave empty partials, of which the merge reads the maximum alone (with
      // zeroed outputs written too, 112 units of 9,516 rows on take 84.8 us a
      // call, not 83.5; 128 even units of 20,000 204 us, not 197).
      active = p.even_splits;
      int id = unit * p.splits + split;
      if (id >= units * active) {
        id -= units * active;
        unit = id / (p.splits - active);
        split = active + id - unit * (p.splits - active);
        const size_t pbase = static_cast<size_t>(unit) * p.splits + split;
        if (static_cast<int>(threadIdx.x) < p.group) {
          p.part_ml[pbase * 2 * p.group + threadIdx.x] = -INFINITY;
          p.part_ml[pbase * 2 * p.group + p.group + threadIdx.x] = 0.f;
        }
        return;
      }
      unit = id / active;
      split = id - unit * active;
    }
    len_in = held.of(unit);
  }
  const int per_layer = p.batch * p.hkv;
  const int lc = unit / per_layer;
  const int b = (unit % per_layer) / p.hkv;
  const int h = unit % p.hkv;
  const size_t cunit = (static_cast<size_t>(p.layer0 + lc) * p.batch + b) * p.hkv + h;
  const size_t qunit = static_cast<size_t>(lc) * per_layer + static_cast<size_t>(b) * p.hkv + h;

  if constexpr (!HELD) len_in = p.len[cunit];
  const int n_cache = len_in < 0 ? 0 : (len_in > p.cap ? p.cap : len_in);
  const bool append = p.k_new != nullptr;
  const int n_tot = n_cache + (append ? 1 : 0);
  const T *kbase = reinterpret_cast<const T *>(p.k) + cunit * p.cap * D;
  const T *vbase = reinterpret_cast<const T *>(p.v) + cunit * p.cap * D;
  const T *knew = append ? reinterpret_cast<const T *>(p.k_new) + qunit * D : nullptr;
  const T *vnew = append ? reinterpret_cast<const T *>(p.v_new) + qunit * D : nullptr;

  const int ntiles = (n_tot + kTile - 1) / kTile;
  const int tps = (ntiles + active - 1) / active;
  const int t0 = split * tps;
  const int t1 = min(ntiles, t0 + tps);

  // Q^T operand: lane (query col, group grp) holds head-dim elements grp*dq + c*kpl + j.
  frag qf[Cfg::qk_steps];
  {
    const T *qrow = reinterpret_cast<const T *>(p.q) +
                    ((static_cast<size_t>(lc) * p.batch + b) * p.hq + h * p.group + col) * D + grp * Cfg::dq;
#pragma unroll
    for (int c = 0; c < Cfg::qk_steps; ++c)
      qf[c] = (col < p.group) ? load_frag(qrow + c * Cfg::kpl) : zero_frag(frag{});
  }

  float m_run = -INFINITY;
  float l_run = 0.f;
  f32x4_t o[Cfg::dtiles];
#pragma unroll
  for (int dt = 0; dt < Cfg::dtiles; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  unsigned char *stage = smem + wave * Cfg::wave_stage;           // V, row pitch lds_stride
  unsigned char *kstage = stage;                                    // K, row pitch k_stride

  TileRegs<T, D> cur;
  const auto load_k = [&](int t) { load_rows<T, D>(cur.kreg, t * kTile, n_cache, append, kbase, knew, lane); };
  const auto load_v = [&](int t) { load_rows<T, D>(cur.vreg, t * kTile, n_cache, append, vbase, vnew, lane); };

  // Tile t, from its registers to m_run, l_run and o.  Unless it is the wave's
  // last one, all its keys are valid, and tile t + NW is asked for: K's
  // registers as soon as K is staged, V's as soon as V is, so that one tile per
  // wave is on its way at any time and a tile takes one set of registers.
  const auto attend = [&](int t, auto last_tile) {
    constexpr bool kLast = decltype(last_tile)::value;
    const int kb = t * kTile;
    // K tile -> LDS -> MFMA operand layout (lane holds key hf*16 + col,
    // head-dim slice grp*dq + c*kpl of it).
#pragma unroll
    for (int i = 0; i < Cfg::v_insts; ++i) {
      const int r = i * Cfg::rows_per_inst + lane / Cfg::lanes_per_row;
      *reinterpret_cast<uint4 *>(kstage + r * Cfg::k_stride + (lane % Cfg::lanes_per_row) * 16) = cur.kreg[i];
    }
    if constexpr (!kLast) load_k(t + NW);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    frag kf[2][Cfg::qk_steps];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const T *krow = reinterpret_cast<const T *>(kstage + (hf * 16 + col) * Cfg::k_stride) + grp * Cfg::dq;
#pragma unroll
      for (int c = 0; c < Cfg::qk_steps; ++c) kf[hf][c] = load_frag(krow + c * Cfg::kpl);
    }

    // S^T = K . Q^T for the two 16-key halves.
    f32x4_t s[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      s[hf] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < Cfg::qk_steps; ++c) s[hf] = MF::mma(kf[hf][c], qf[c], s[hf]);
    }

    // Online softmax over this tile (log2 domain).  Lane holds keys
    // kb + hf*16 + 4*grp + i of query col.
    float sv[8];
    float tmax = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int key = kb + (e >> 2) * 16 + 4 * grp + (e & 3);
      float x = s[e >> 2][e & 3] * p.scale_log2;
      if constexpr (kLast) x = key < n_tot ? x : -INFINITY;
      sv[e] = x;
      tmax = fmaxf(tmax, x);
    }
    tmax = group4_max(tmax);
    const float m_new = fmaxf(m_run, tmax);          // finite: the tile holds a valid key
    const float alpha = fast_exp2(m_run - m_new);    // 0 on the first tile
    float pv[8];
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pv[e] = fast_exp2(sv[e] - m_new);
      psum += pv[e];
    }
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int dt = 0; dt < Cfg::dtiles; ++dt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) o[dt][i] *= alpha;
    }

    // Stage V (row-major, padded pitch) and read it back column-wise.
#pragma unroll
    for (int i = 0; i < Cfg::v_insts; ++i) {
      const int r = i * Cfg::rows_per_inst + lane / Cfg::lanes_per_row;
      uint2 *dst = reinterpret_cast<uint2 *>(stage + r * Cfg::lds_stride + (lane % Cfg::lanes_per_row) * 16);
      uint4 x = cur.vreg[i];
      if constexpr (kLast) {                                 // a NaN past the end times 0 would be NaN
        const unsigned keep = kb + r < n_tot ? ~0u : 0u;
        x = make_uint4(x.x & keep, x.y & keep, x.z & keep, x.w & keep);
      }
      dst[0] = make_uint2(x.x, x.y);
      dst[1] = make_uint2(x.z, x.w);
    }
    if constexpr (!kLast) load_v(t + NW);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int dt = 0; dt < Cfg::dtiles; ++dt) {
#pragma unroll
      for (int c = 0; c < Cfg::pv_ops; ++c) {
        const frag a = vt_frag<T, D>(stage, c, grp, dt, col);
        o[dt] = MF::mma(a, pt_frag<T>(pv, c), o[dt]);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };

  const std::integral_constant<bool, false> inner{};
  const std::integral_constant<bool, true> last{};
  int t = t0 + wave;
  if (t < t1) {
    load_k(t);
    load_v(t);
    for (; t + NW < t1; t += NW) attend(t, inner);
    attend(t, last);
  }

  // Total of the per-lane partial sums of query col.
  const float l_tot = group4_sum(l_run);

  // Cross-wave merge through LDS.
  __syncthreads();
  float *mw = reinterpret_cast<float *>(smem);   // [NW][16]
  float *lw = mw + NW * 16;                      // [NW][16]
  float *ow = lw + NW * 16;                      // [NW][16][merge_pitch]
  if (grp == 0) {
    mw[wave * 16 + col] = m_run;
    lw[wave * 16 + col] = l_tot;
  }
#pragma unroll
  for (int dt = 0; dt < Cfg::dtiles; ++dt)
    *reinterpret_cast<float4 *>(ow + (wave * 16 + col) * Cfg::merge_pitch + dt * 16 + 4 * grp) =
        make_float4(o[dt][0], o[dt][1], o[dt][2], o[dt][3]);
  __syncthreads();
  // Four outputs d .. d + 3 of query qi over all waves, with the maximum M and
  // the sum L of the workgroup's softmax.
  const auto merged = [&](int qi, int d, float &M, float &L) {
    M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, mw[w * 16 + qi]);
    L = 0.f;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (M != -INFINITY) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float e = fast_exp2(mw[w * 16 + qi] - M);
        const float4 x = *reinterpret_cast<const float4 *>(ow + (w * 16 + qi) * Cfg::merge_pitch + d);
        acc.x += x.x * e;
        acc.y += x.y * e;
        acc.z += x.z * e;
        acc.w += x.w * e;
        L += lw[w * 16 + qi] * e;
      }
    }
    return acc;
  };

  if (p.splits == 1) {
    // The workgroup holds its unit's whole softmax: it writes out / lse /
    // row_stats and commits the append itself, with the arithmetic of the
    // merge of a single split (weight exp2(0) * 1/L, added to zero).
    const size_t oq0 = (static_cast<size_t>(lc) * p.batch + b) * p.hq + h * p.group;
    for (int idx = threadIdx.x; idx < p.group * (D / 4); idx += kThreads) {
      const int qi = idx / (D / 4);
      const int d = (idx - qi * (D / 4)) * 4;
      float M, L;
      const float4 acc = merged(qi, d, M, L);
      const float inv = L > 0.f ? 1.f / L : 0.f;
      T *dst = reinterpret_cast<T *>(p.out) + (oq0 + qi) * D + d;
      dst[0] = from_f32<T>(fmaf(acc.x, inv, 0.f));
      dst[1] = from_f32<T>(fmaf(acc.y, inv, 0.f));
      dst[2] = from_f32<T>(fmaf(acc.z, inv, 0.f));
      dst[3] = from_f32<T>(fmaf(acc.w, inv, 0.f));
      if (d == 0) {
        if (p.lse) p.lse[oq0 + qi] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
        if (p.row_stats) {
          p.row_stats[(oq0 + qi) * 2 + 0] = M;
          p.row_stats[(oq0 + qi) * 2 + 1] = L;
        }
      }
    }
    // Every wave has finished reading the cache (barrier above); row n_cache
    // is read by no one in this call (the new key comes from k_new).
    if (threadIdx.x == 0 && (len_in < 0 || len_in > p.cap)) report(p.dev_err, 5 /*RECO_DEV_BAD_LENGTH*/);
    if (!append || len_in < 0 || len_in > p.cap) return;
    if (len_in == p.cap) {
      if (threadIdx.x == 0) report(p.dev_err, 1 /*RECO_DEV_APPEND_OVERFLOW*/);
      return;
    }
    for (int d = threadIdx.x; d < D; d += kThreads) {
      reinterpret_cast<T *>(p.k)[(cunit * p.cap + len_in) * D + d] = knew[d];
      reinterpret_cast<T *>(p.v)[(cunit * p.cap + len_in) * D + d] = vnew[d];
    }
    if (threadIdx.x == 0) p.len[cunit] = len_in + 1;
    return;
  }

  const size_t pbase = static_cast<size_t>(unit) * p.splits + split;
  float *po = p.part_o + pbase * p.group * D;
  float *pml = p.part_ml + pbase * 2 * p.group;
  for (int idx = threadIdx.x; idx < p.group * (D / 4); idx += kThreads) {
    const int qi = idx / (D / 4);
    const int d = (idx - qi * (D / 4)) * 4;
    float M, L;
    const float4 acc = merged(qi, d, M, L);
    float *dst = po + qi * D + d;
    dst[0] = acc.x;
    dst[1] = acc.y;
    dst[2] = acc.z;
    dst[3] = acc.w;
    if (d == 0) {
      pml[qi] = M;
      pml[p.group + qi] = L;
    }
  }
}

// Merge the split partials of every (unit, query head), write out / lse and
// commit the append.  One 64-lane wave per (unit, query head): every lane
// fetches all split statistics at once (one memory round trip), derives the
// merge weights itself, then loads its head-dim slice of every split partial
// (a second round trip).  The appended row is fetched up front.
template <typename T, int D>
__global__ __launch_bounds__(kWave) void decode_merge_kernel(DecodeParams p) {
  constexpr int kPer = D / kWave;                  // head-dim elements per lane
  const int unit = blockIdx.x;
  const int qi = blockIdx.y;
  const int lane = threadIdx.x;
  const int per_layer = p.batch * p.hkv;
  const int lc = unit / per_layer;
  const int b = (unit % per_layer) / p.hkv;
  const int h = unit % p.hkv;
  const size_t cunit = (static_cast<size_t>(p.layer0 + lc) * p.batch + b) * p.hkv + h;
  const size_t qunit = static_cast<size_t>(lc) * per_layer + static_cast<size_t>(b) * p.hkv + h;
  const int S = p.splits;
  const bool append = p.k_new != nullptr && qi == 0;

  // Query head 0 of the unit also commits the append: fetch len and the row now.
  const int len_in = qi == 0 ? p.len[cunit] : 0;
  T krow[kPer], vrow[kPer];
  if (append) {
    const T *ksrc = reinterpret_cast<const T *>(p.k_new) + qunit * D;
    const T *vsrc = reinterpret_cast<const T *>(p.v_new) + qunit * D;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      krow[i] = ksrc[lane + i * kWave];
      vrow[i] = vsrc[lane + i * kWave];
    }
  }
  const int G = p.group;
  const float *pml = p.part_ml + static_cast<size_t>(unit) * S * 2 * G;
  const float *po = p.part_o + (static_cast<size_t>(unit) * S * G + qi) * D;
  // The first kPre splits' output slices are requested together with the
  // statistics, so a call with at most kPre splits costs one memory round trip.
  constexpr int kPre = 4;
  float pre[kPre][kPer];
#pragma unroll
  for (int s = 0; s < kPre; ++s) {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      pre[s][i] = s < S ? po[static_cast<size_t>(s) * G * D + lane + i * kWave] : 0.f;
  }
  // Lane s holds split s's statistics, lane s - 64 the rest (S <= kMaxSplits = 128).
  const float m0 = lane < S ? pml[lane * 2 * G + qi] : -INFINITY;
  const float l0 = lane < S ? pml[lane * 2 * G + G + qi] : 0.f;
  const float m1 = lane + kWave < S ? pml[(lane + kWave) * 2 * G + qi] : -INFINITY;
  const float l1 = lane + kWave < S ? pml[(lane + kWave) * 2 * G + G + qi] : 0.f;
  const float M = wave_max(fmaxf(m0, m1));
  float L = 0.f;
  if (M != -INFINITY) L = wave_sum(l0 * fast_exp2(m0 - M) + l1 * fast_exp2(m1 - M));
  const float inv = L > 0.f ? 1.f / L : 0.f;
  // Below 0: nothing in the split, whose outputs may be left unwritten.
  const float w0 = m0 != -INFINITY ? fast_exp2(m0 - M) * inv : -1.f;
  const float w1 = m1 != -INFINITY ? fast_exp2(m1 - M) * inv : -1.f;

  float acc[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) acc[i] = 0.f;
#pragma unroll
  for (int s = 0; s < kPre; ++s) {
    const float wgt = __shfl(w0, s, kWave);       // -1 for s >= S
#pragma unroll
    for (int i = 0; i < kPer; ++i) acc[i] = fmaf(wgt, wgt < 0.f ? 0.f : pre[s][i], acc[i]);
  }
  for (int s = kPre; s < S; ++s) {
    const float wgt = __shfl(s < kWave ? w0 : w1, s & (kWave - 1), kWave);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const float x = po[static_cast<size_t>(s) * G * D + lane + i * kWave];
      acc[i] = fmaf(wgt, wgt < 0.f ? 0.f : x, acc[i]);
    }
  }
  T *out = reinterpret_cast<T *>(p.out) + ((static_cast<size_t>(lc) * p.batch + b) * p.hq + h * p.group + qi) * D;
#pragma unroll
  for (int i = 0; i < kPer; ++i) out[lane + i * kWave] = from_f32<T>(acc[i]);
  const size_t oq = (static_cast<size_t>(lc) * p.batch + b) * p.hq + h * p.group + qi;
  if (p.lse && lane == 0) p.lse[oq] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
  if (p.row_stats && lane == 0) {
    p.row_stats[oq * 2 + 0] = M;
    p.row_stats[oq * 2 + 1] = L;
  }

  if (qi != 0) return;
  if (lane == 0 && (len_in < 0 || len_in > p.cap)) report(p.dev_err, 5 /*RECO_DEV_BAD_LENGTH*/);
  if (!append || len_in < 0 || len_in > p.cap) return;
  if (len_in == p.cap) {
    if (lane == 0) report(p.dev_err, 1 /*RECO_DEV_APPEND_OVERFLOW*/);
    return;
  }
  T *kdst = reinterpret_cast<T *>(p.k) + (cunit * p.cap + len_in) * D;
  T *vdst = reinterpret_cast<T *>(p.v) + (cunit * p.cap + len_in) * D;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    kdst[lane + i * kWave] = krow[i];
    vdst[lane + i * kWave] = vrow[i];
  }
  if (lane == 0) p.len[cunit] = len_in + 1;
}

// Merge for many splits (small calls, e.g. one layer per call): one
// 256-thread workgroup per (unit, query head).  Every split's output slice is
// requested at once (thread group sg loads splits sg, sg + kSG, ... as 16-byte
// pieces) together with the split statistics, so the merge costs one memory
// round trip whatever the split count; the weighted slices meet in LDS.
constexpr int kWideThreads = 256;
constexpr int kWideMinSplits = 9;                  // fewer splits use the one-wave merge

template <typename T, int D>
__global__ __launch_bounds__(kWideThreads) void decode_merge_wide_kernel(DecodeParams p) {
  constexpr int kVec = 4;
  constexpr int kTPS = D / kVec;                   // threads per split slice
  constexpr int kSG = kWideThreads / kTPS;         // split groups
  constexpr int kMaxPer = kMaxSplits / kSG;        // splits per thread at most
  constexpr int kWaves = kWideThreads / kWave;
  __shared__ float s_w[kMaxSplits];
  __shared__ float s_red[kWaves];
  __shared__ __attribute__((aligned(16))) float s_acc[kSG][D];

  const int unit = blockIdx.x;
  const int qi = blockIdx.y;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int per_layer = p.batch * p.hkv;
  const int lc = unit / per_layer;
  const int b = (unit % per_layer) / p.hkv;
  const int h = unit % p.hkv;
  const size_t cunit = (static_cast<size_t>(p.layer0 + lc) * p.batch + b) * p.hkv + h;
  const size_t qunit = static_cast<size_t>(lc) * per_layer + static_cast<size_t>(b) * p.hkv + h;
  const int S = p.splits;
  const bool append = p.k_new != nullptr && qi == 0;

  // Everything this workgroup reads is requested up front.
  const int len_in = qi == 0 ? p.len[cunit] : 0;
  T krow = T{}, vrow = T{};
  if (append && tid < D) {
    krow = reinterpret_cast<const T *>(p.k_new)[qunit * D + tid];
    vrow = reinterpret_cast<const T *>(p.v_new)[qunit * D + tid];
  }
  const int sg = tid / kTPS;
  const int dv = (tid % kTPS) * kVec;
  const int G = p.group;
  const float *po = p.part_o + (static_cast<size_t>(unit) * S * G + qi) * D;
  float4 part[kMaxPer];
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    const int sp = sg + kSG * i;
    part[i] = sp < S ? *reinterpret_cast<const float4 *>(po + static_cast<size_t>(sp) * G * D + dv)
                     : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const float *pml = p.part_ml + static_cast<size_t>(unit) * S * 2 * G;
  const float m_t = tid < S ? pml[tid * 2 * G + qi] : -INFINITY;
  const float l_t = tid < S ? pml[tid * 2 * G + G + qi] : 0.f;

  // M = max of the split maxima, L = sum of the rescaled split sums.
  float v = wave_max(m_t);
  if (lane == 0) s_red[wave] = v;
  __syncthreads();
  float M = s_red[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) M = fmaxf(M, s_red[w]);
  __syncthreads();
  const float e_t = (M != -INFINITY && tid < S) ? fast_exp2(m_t - M) : 0.f;
  v = wave_sum(l_t * e_t);
  if (lane == 0) s_red[wave] = v;
  __syncthreads();
  float L = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) L += s_red[w];
  const float inv = L > 0.f ? 1.f / L : 0.f;
  if (tid < kMaxSplits) s_w[tid] = e_t * inv;
  __syncthreads();

  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < kMaxPer; ++i) {
    const int sp = sg + kSG * i;
    const float wgt = sp < S ? s_w[sp] : 0.f;
    acc.x += wgt * part[i].x;
    acc.y += wgt * part[i].y;
    acc.z += wgt * part[i].z;
    acc.w += wgt * part[i].w;
  }
  *reinterpret_cast<float4 *>(&s_acc[sg][dv]) = acc;
  __syncthreads();

  const size_t oq = (static_cast<size_t>(lc) * p.batch + b) * p.hq + h * p.group + qi;
  if (tid < D) {
    float o = 0.f;
#pragma unroll
    for (int g = 0; g < kSG; ++g) o += s_acc[g][tid];
    reinterpret_cast<T *>(p.out)[oq * D + tid] = from_f32<T>(o);
  }
  if (tid == 0) {
    if (p.lse) p.lse[oq] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
    if (p.row_stats) {
      p.row_stats[oq * 2 + 0] = M;
      p.row_stats[oq * 2 + 1] = L;
    }
  }

  if (qi != 0) return;
  if (tid == 0 && (len_in < 0 || len_in > p.cap)) report(p.dev_err, 5 /*RECO_DEV_BAD_LENGTH*/);
  if (!append || len_in < 0 || len_in > p.cap) return;
  if (len_in == p.cap) {
    if (tid == 0) report(p.dev_err, 1 /*RECO_DEV_APPEND_OVERFLOW*/);
    return;
  }
  if (tid < D) {
    reinterpret_cast<T *>(p.k)[(cunit * p.cap + len_in) * D + tid] = krow;
    reinterpret_cast<T *>(p.v)[(cunit * p.cap + len_in) * D + tid] = vrow;
  }
  if (tid == 0) p.len[cunit] = len_in + 1;
}

template <typename T, int D>
hipError_t launch_typed(const DecodeParams &p, hipStream_t s) {
  const int units = p.n_layers * p.batch * p.hkv;
  // Eight waves where a split holds more tiles than four waves take in one
  // round and nothing else hides the second round: small calls of long units
  // (28 one-layer calls of 4 units x 9,645 rows: four waves 359 us, eight 352 us).
  // With few splits per unit (longer runs of tiles) eight waves only add to the
  // merge (112 units x 9,645 rows: four 86.4 us, eight 88.4 us).
  const int tiles_cap = (p.cap + 1 + kTile - 1) / kTile;
  // fp32 at head_dim 128 needs more than the 256 registers that eight waves
  // leave a lane (808 bytes of scratch).
  constexpr bool kEight = !(sizeof(T) == 4 && D == 128);
  // Rows of 128 bytes make tiles of half the size: with one workgroup on a CU
  // four waves have too little on their way (200 units of 600 to 4,500 rows: four
  // waves 50.6 us, eight 33.7 us; 256 units of 1,100 rows: 19.1 us, 15.5 us).
  // With two on a CU eight are no faster (512 units of 500 to 3,500 rows: 54.5
  // us, 55.1 us).
  const bool thin = sizeof(T) * D == 128 && static_cast<int64_t>(units) * p.splits <= p.cus;
  // Wider rows, one split each: a CU's only workgroup bounds the call where
  // other CUs have none, or shorter ones, and streams faster with eight waves
  // (192 units of 600 to 4,800 rows: four waves 59.8 us, eight 55.3 us; 144 even
  // units of 9,645: 123 us, 115 us; 144 fp32 units of 5,000 at head_dim 64: 75.8
  // us, 67.3 us).  Where even units fill nearly every CU, as one sequence's layers
  // and heads do, four are faster, by what the merge over eight costs (256 units
  // of 1,100 rows: four 24.1 us, eight 25.2 us; of 4,800: 92.0 us, 94.6 us; ragged
  // ones of 600 to 4,800: 68.2 us, 65.0 us).
  const bool alone = p.splits == 1 && 8 * static_cast<int64_t>(units) <= 7 * static_cast<int64_t>(p.cus);
  // (Where uneven units may take more than two splits, two workgroups of four
  // waves share a CU; two of eight do so only at 128 bytes a row.)
  constexpr int kHeldWaves = sizeof(T) * D == 128 ? 8 : 4;
  const dim3 grid(p.splits, units);
  if (p.splits > p.even_splits)
    hipLaunchKernelGGL((decode_split_kernel<T, D, kHeldWaves, true>), grid, dim3(kHeldWaves * kWave), 0, s, p);
  else if (kEight && (p.splits >= kWideMinSplits || thin || alone) && tiles_cap >= 6 * p.splits)
    hipLaunchKernelGGL((decode_split_kernel<T, D, kEight ? 8 : 4, false>), grid, dim3((kEight ? 8 : 4) * kWave), 0, s, p);
  else
    hipLaunchKernelGGL((decode_split_kernel<T, D, 4, false>), grid, dim3(4 * kWave), 0, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.splits == 1) return e;   // one split: finalised in place
  if (p.splits >= kWideMinSplits)
    hipLaunchKernelGGL((decode_merge_wide_kernel<T, D>), dim3(units, p.group), dim3(kWideThreads), 0, s, p);
  else
    hipLaunchKernelGGL((decode_merge_kernel<T, D>), dim3(units, p.group), dim3(kWave), 0, s, p);
  return hipGetLastError();
}

}  // namespace

// Split partials of the allocation-free entry point.  Every device holds its
// own copy of this array at its own address until the process ends.  In host
// code `scratch` names a host-side stand-in for the device symbol, not device
// memory: host code uses only the address hipGetSymbolAddress returns for the
// current device, never the name itself.  The decode kernels write every
// partial they later read, so the array never needs clearing; calls that
// overlap on one device share it and race.
static __device__ __align__(256) unsigned char scratch[kDecodeScratchBytes];

hipError_t decode_scratch(void **ptr) {
  constexpr int kMaxDevices = 64;
  static std::atomic<void *> addr[kMaxDevices];
  static std::mutex mu;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void *p = addr[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> lock(mu);
    p = addr[dev].load(std::memory_order_relaxed);
    if (!p) {
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // with `dev` current
      if (e != hipSuccess) return e;
      if (!p) return hipErrorInvalidSymbol;
      addr[dev].store(p, std::memory_order_release);
    }
  }
  *ptr = p;
  return hipSuccess;
}

hipError_t launch_decode(const DecodeParams &p, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0) {
    if (head_dim == 64) return launch_typed<float, 64>(p, s);
    return launch_typed<float, 128>(p, s);
  }
  if (head_dim == 64) return launch_typed<bf16_t, 64>(p, s);
  return launch_typed<bf16_t, 128>(p, s);
}

}  // namespace reco
