// What the two many-row GEMMs (gemm_tile.hip, gemm_wide.hip) share: direct-to-LDS loads' helpers, and which of the two a product takes.
#pragma once
#include <type_traits>

#include "kernels.h"

namespace mdz {

constexpr int kRound = 64;  // features per round of loads

#define MDZ_LDS_ADDR(p) ((uint32_t)(uintptr_t)((__attribute__((address_space(3))) void*)(p)))

__device__ inline float silu_tile(float v) { return v / (1.0f + expf(-v)); }
template <int N, int I = 0, typename F>
__device__ inline __attribute__((always_inline)) void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}
// One wave brings 64 x 16 B from base + off (per lane) to LDS address `lds` + OFF + 16 * lane.  base and lds are wave-uniform.
// The load takes its LDS address from m0, one wait state after a scalar write of it (the compiler inserts that for its own
// loads; it does not look into assembly).  (clang warns that m0 is a reserved register: it is named so that a value the compiler
// itself puts there is not taken to outlive the load.)
// ONCE: the bytes are not wanted again soon (gemm_tile.hip: W is read once per row block, of which there are few), so the load is
// non-temporal (see gemm_mfma.hip).  us, plain / non-temporal W there: steps of 4 layers with 4 sequences on 64 nodes 1026 / 993, 12 on 15
// nodes 948 / 915; of 8 layers with 90 rows 1367 / 1356, 192 rows 1706 / 1678.  gemm_wide.hip keeps plain loads: its many row blocks meet in
// L2 at their own pace (5 layers, 832 rows 3136 / 3193, 640 rows 2925 / 2942, 1024 rows 3617 / 3601).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int OFF, bool ONCE = false>
__device__ inline void load_to_lds(const void* base, uint32_t off, uint32_t lds) {
  if constexpr (ONCE)
    asm volatile("s_add_i32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(off), "s"(base), "n"(OFF)
                 : "memory", "scc", "m0");
  else
    asm volatile("s_add_i32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base), "n"(OFF)
                 : "memory", "scc", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ inline void wait_loads() {  // all but the N youngest loads of this wave have landed
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ inline void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Modelled time of a launch in us, the reading of its partial-sum slots by the consumer included; `slots` (nullable) receives
// their number.
double gemm_tile_cost(int M, int N, int K, int max_split, bool swiglu, int* slots);
double gemm_wide_cost(int M, int N, int K, int max_split, bool swiglu, int* slots);
// the faster of the two by these models
inline bool gemm_wide_preferred(int M, int N, int K, int max_split, bool swiglu) {
  return gemm_wide_cost(M, N, K, max_split, swiglu, nullptr) < gemm_tile_cost(M, N, K, max_split, swiglu, nullptr);
}
struct ManyRowsPlan {
  bool wide;
  int tile_rows, tile_cols, k_splits;
};
ManyRowsPlan gemm_tile_plan(int M, int N, int K, int max_split, bool swiglu);
ManyRowsPlan gemm_wide_plan(int M, int N, int K, int max_split, bool swiglu);
bool gemm_tile_supported(int dtype, int M, int N, int K);
int launch_gemm_wide(int dtype, const void* X, const void* Wp, float* P, int M, int N, int K, int64_t ldp, int64_t part_stride,
                     int max_split, Partials* res, hipStream_t st);
int launch_gemm_wide_swiglu(int dtype, const void* X, const void* Wp, void* U, int M, int N, int K, hipStream_t st);

}  // namespace mdz
