// Arguments of the attention kernels (attend.hip, attend_f32.hip).
#pragma once
#include "ltri_internal.h"

namespace ltri {

struct AttArgs {
  Dims D; DevState st; const void* k_arena; const void* v_arena; const void* q;
  void* out; float* lse; int layer; int seq_count; int n_q;
  int n_splits; float* part;             // > 1: the key range is split over workgroups, partial results in part
  int32_t* even_flags;                   // even shares: a flag per workgroup's place in part; fp32 splits: tickets. Zero between launches
  int part_mode;                         // ATT_ALL, or one of the two parts of a two-part step
  const int32_t* loclist; int loc_cap;   // ATT_LOCAL: initial | window tokens per sequence [seq_count][loc_cap]
  const float* lse_a;                    // ATT_RETRIEVED: log-sum-exp of the first part, whose output is in `out`
  BatchPos bp;
};

hipError_t launch_attend_f32(const AttArgs& a, long long n_ctx, hipStream_t s);
size_t attend_f32_part_rows();

}  // namespace ltri
