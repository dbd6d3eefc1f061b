// Work split of the decode-attention kernels (decode_attn.hip): how many
// workgroups share one unit's keys, and the bytes of split partials that
// implies.  Host code only; kept apart from the kernel sources so that
// tuning the split rule leaves the kernels' files untouched.
#pragma once

#include <stddef.h>

namespace reco {

constexpr int kDecodeTile = 32;          // keys per wave iteration of the attention kernel
constexpr int kDecodeMaxSplits = 128;    // most splits the merge kernels take
constexpr int kDecodeHeldUnits = 128;    // units whose lengths a wave holds

// Splits per unit that the workspace is sized for; compute_units: CUs of the
// device the call runs on.
int decode_splits(int units, int capacity, int compute_units);
// The splits a call launches per unit, `splits` being those that its partials'
// memory is sized for: that size counts 16 query rows a split, a call writes
// `group` of them, and what this saves holds more splits.  Where two are sized
// for, there is room for two workgroups a compute unit: four or five.  The host
// knows the capacity, the device the rows: the kernel takes them all where the
// units are uneven, so that the compute units that draw short ones help with the
// rest, or all short, where more pieces take less time; long even units take two,
// as the second ramp costs them more than it gives (HeldLengths in
// decode_attn.hip).  Measured, two splits and all: 96 units of 1,200 to 9,645 rows
// 63.4 us, 53.6 us; of 2,500 to 20,000 124 us, 99 us; 128 of 2,500 to 20,000 139
// us, 134 us; 96 even units of 600 rows in 21,000 11.8 us, 11.2 us; of 20,000 144
// us, 149 us; 112 of 9,645 84.0 us, 86.2 us.
// Not where
// - there is one split: more would add the merge kernel, which costs a cache of
//   few rows more than the splits give a full one (256 units of 1,100 rows in a
//   capacity of 8,800: one split 24.5 us, two 28.7 us; 160 units of 100 rows in
//   10,064: one 6.0 us, three 9.2 us; 256 of 600 to 4,800 rows: one 68 us, two
//   66 us);
// - there are three or more: twice as many are a merge of their own, and again
//   cost short units more (48 units of 300 rows in 39,000: five splits 8.0 us, ten
//   12.3 us; of 2,500 to 20,000: 58 us, 55 us);
// - the capacity is below 320 tiles, or only some compute units would get a second
//   workgroup (fewer than 1.5 a compute unit);
// - rows have 128 bytes (eight waves stream them) or 512 (a workgroup has its
//   compute unit to itself) and a fifth of the compute units or less would be
//   idle (96 units of 1,500 to 12,000 rows: 128 bytes 40.2 us, 36.0 us, 512 bytes
//   163 us, 140 us; 128 of these units: 45.0 us, 47.3 us and 180 us, 182 us).
int decode_launch_splits(int splits, int units, int capacity, int group, int head_dim, int elem_bytes,
                         int compute_units);
size_t decode_workspace_bytes(int units, int capacity, int head_dim, int compute_units);

// Size of the allocation-free entry point's static partials array on every
// device (the split partials of one call with at most compute_units units
// need at most compute_units * (16 * head_dim + 32) * 4 bytes: 2.1 MB on a
// 256-CU device at head_dim 128).
constexpr size_t kDecodeScratchBytes = size_t(8) << 20;
// Split count of an allocation-free call: decode_splits, except that a call
// with more units than compute units whose partials would not fit the array
// takes one split per unit.
int decode_scratch_splits(int units, int capacity, int head_dim, int compute_units);
// Bytes of partials that a call of `splits` launched splits per unit writes (0
// for one, which is finalised in place).
size_t decode_partials_bytes(int units, int splits, int group, int head_dim);

}  // namespace reco
