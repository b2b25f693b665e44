// Optional per-launch timing of the library's heavy kernels with HIP events on the
// caller's stream.  Off by default; when off a launch pays one branch.  Internal.
#pragma once
#include <hip/hip_runtime.h>

namespace fise {

// one kind per kernel family, so that a kind's average can be set against a profiler's per-kernel figure
enum { PROF_IGEMM = 0,          // gathered GEMM over maps (wave_gemm.hip, conv_patch.hip), and 64x64 tiles of igemm.hip
       PROF_IGEMM_GEGLU = 1,    // the GEGLU epilogue
       PROF_ATTENTION = 2,      // active-query attention, both kernels (without the merge launch)
       PROF_IGEMM_WIDE = 3,     // linears of many rows: linear_wide.hip, 64x128 tiles of igemm.hip
       PROF_REDUCE = 4,         // split-K reduce + epilogue
       PROF_IGEMM_THIN = 5,     // 32x128 tiles of igemm.hip (at most 32 rows that wave_gemm.hip does not take)
       PROF_IGEMM_STAGED = 6,   // register-staged gathered GEMM (GroupNorm prologue, 32-wide K steps)
       PROF_ATTENTION_MERGE = 7,
       PROF_EMPTY = 8,          // nothing between the two events: the bracket's own cost
       PROF_ROWS_GEMM = 9,      // products of compact rows (wave_gemm.hip) and behind a normalisation (norm_gemm.hip)
       PROF_KINDS = 10 };

extern bool g_profile_on;
void profile_begin(int kind, double flops, double bytes, hipStream_t st);
void profile_end(hipStream_t st);

struct ProfileScope {
    hipStream_t st; bool on;
    ProfileScope(int kind, double flops, double bytes, hipStream_t s) : st(s), on(g_profile_on) {
        if (on) profile_begin(kind, flops, bytes, st);
    }
    ~ProfileScope() { if (on) profile_end(st); }
};

}  // namespace fise
