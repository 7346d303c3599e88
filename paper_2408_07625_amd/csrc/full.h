// Row sums of the conventional local energy with lanes over rows (full.hip).
#pragma once

#include "internal.h"

namespace eloc {

// Launch shape for `rows` rows of one-word keys; by the table's partitions
// where P.part says so, which then needs S.part.
Plan full_plan(const HamDev& H, int64_t rows, int part_bits);
// The n states in the order perm: keys and hashes; and 16-byte amplitudes.
hipError_t launch_full_order(int64_t n, const int32_t* perm, const uint64_t* keys, const uint64_t* hash,
                             uint64_t* keys_to, uint64_t* hash_to, hipStream_t st);
hipError_t launch_full_vec(int64_t n, const int32_t* perm, const double2* from, double2* to, hipStream_t st);
// S.keys, S.hash: the rows'; `vec` by the table's indices.
hipError_t launch_full_rows(int precision, const HamDev& H, const SampleDev& S, const Plan& P, const double2* vec,
                            const float4* vecf, void* partial, hipStream_t st);

}  // namespace eloc
