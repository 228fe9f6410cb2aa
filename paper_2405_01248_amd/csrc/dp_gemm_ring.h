// Main loop of the small MFMA tiles: a plain ring of direct-to-LDS stages of 64-deep k-tiles, one barrier per k-tile; several workgroups per
// CU, or the waves of one, hide each other's latencies.
//
// What bounds it is instruction issue: four to eight MFMAs of 32 cycles a k-tile and wave beside everything else that a wave issues, at some four cycles each.  Hence
// a round of the loop is as many k-tiles as make the stages and the two sets of fragments constants, so that what is left beside the eight or twelve reads
// and the copies is a wait, the barrier and a few scalar instructions (per k-tile and wave 95 to 110 instructions before, 40 to 50 now).
// The fragments of k-tile t are read while the products of k-tile t - 1 run.
#pragma once
#include "dp_device.h"
#include <type_traits>

namespace dp {

// acc[TN] += rows row_a .. + 31 of the stage's first part times rows row_b + 32 j .. of its second, k-tiles in ascending order.  Both parts are rows of 128 bytes,
// chunk c of row r at c ^ ((r >> 1) & 7).  issue(t, stage): this wave's LOADS copies of k-tile t; past the last one all the same (the waits count them), from
// outside the buffers.  done(): called behind the products of each k-tile.
template <int STAGES, int STAGE, int A_BYTES, int LOADS, int TN, class Issue, class Done>
__device__ __forceinline__ void ring_main_loop(f32x16 (&acc)[TN], unsigned char* smem, int nk, int row_a, int row_b, int lane, Issue issue, Done done) {
  constexpr int ROUND = STAGES % 2 ? 2 * STAGES : STAGES;
  static_assert(STAGES >= 3 && (STAGES - 1) * LOADS < 64, "pipeline shape");
  const int g = lane >> 5, ra = row_a + (lane & 31), rb = row_b + (lane & 31);
  bf16x8 fa[2][4], fb[2][4][TN];
  auto read = [&](auto stage, auto set) {
    const unsigned char* st = smem + stage * STAGE;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      fa[set][ks] = *reinterpret_cast<const bf16x8*>(st + ra * 128 + ((2 * ks + g) ^ ((ra >> 1) & 7)) * 16);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[set][ks][j] = *reinterpret_cast<const bf16x8*>(st + A_BYTES + (rb + 32 * j) * 128 + ((2 * ks + g) ^ ((rb >> 1) & 7)) * 16);
    }
  };
  auto multiply = [&](auto set) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[j] = mfma32(fa[set][ks], fb[set][ks][j], acc[j]);
    done();
  };
  constexpr std::integral_constant<int, 0> S0{};
  constexpr std::integral_constant<int, 1> S1{};
  static_for<STAGES>([&](auto s) { issue(s, smem + s * STAGE); });
  wait_vmcnt<(STAGES - 1) * LOADS>();
  barrier_nofence();
  read(S0, S0);
  int t = 1;
  auto round = [&](auto self, auto uc) -> bool {      // k-tiles t + u .. of a round; whether there may be more
    constexpr int u = decltype(uc)::value;
    if constexpr (u == ROUND) return true;
    else {
      if (t + u >= nk) return false;
      wait_vmcnt<(STAGES - 2) * LOADS>();
      wait_lgkmcnt0();               // this wave's reads of k-tile t + u - 1 are done
      barrier_nofence();             // k-tile t + u is there for everybody, and nobody reads the one before any more
      issue(t + u + STAGES - 1, smem + u % STAGES * STAGE);
      read(std::integral_constant<int, (u + 1) % STAGES>(), std::integral_constant<int, (u + 1) % 2>());
      multiply(std::integral_constant<int, u % 2>());
      return self(self, std::integral_constant<int, u + 1>());
    }
  };
  while (round(round, S0)) t += ROUND;
  if (nk % 2) multiply(S0);
  else multiply(S1);
  wait_vmcnt<0>();                   // (copies from outside the buffers may still be under way to what the caller puts there)
}

}  // namespace dp
