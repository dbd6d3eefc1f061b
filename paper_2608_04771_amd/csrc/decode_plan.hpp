// Work split of the decode-attention kernels (decode_attn.hip): how many
// workgroups share one unit's keys, and the bytes of split partials that
// implies.  Host code only; kept apart from the kernel sources so that
// tuning the split rule leaves the kernels' files untouched.
#pragma once

#include <stddef.h>

namespace reco {

constexpr int kDecodeTile = 32;          // keys per wave iteration of the attention kernel
constexpr int kDecodeMaxSplits = 128;    // most splits the merge kernels take

// compute_units: CUs of the device the call runs on (sets the split count).
int decode_splits(int units, int capacity, int compute_units);
// Splits of one call, `splits` being those that its partials' memory is sized
// for: that size counts 16 query rows a split, a call writes `group` of them,
// and what this saves takes more splits.  Where a split would be long (160 tiles
// or more at capacity), two workgroups a compute unit are taken, of 64 tiles or
// more: the units are ragged more often than not, and the compute units that
// draw short ones then help with the rest (one layer of 32 sequences of 4K to
// 32K rows: two splits each 235 us, four splits 206 us; 128 even units of 18,000
// rows: two 182 us, four 186 us).  Shorter splits cost more in a second ramp than
// they give (112 units of 9,645 rows: two 89.5 us, four 91.3 us), and so do
// splits that give only some compute units a second workgroup: at least 1.5 a
// compute unit.  A call of one split each keeps it whatever its capacity: more
// would add the merge kernel, which costs a cache of few rows more than the
// splits give a full one (256 units of 1,100 rows in a capacity of 8,800: one
// split 24.5 us, two 28.7 us; 160 units of 100 rows in 10,064: one 6.0 us, three
// 9.2 us; 256 of 600 to 4,800 rows: one 68 us, two 66 us).
int decode_call_splits(int splits, int units, int capacity, int group, int head_dim, int compute_units);
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
// Bytes of the array one call uses (0 when every unit is a single split,
// which needs no partials).
size_t decode_scratch_bytes(int units, int capacity, int head_dim, int compute_units);

}  // namespace reco
