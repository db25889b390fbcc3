// Which candidate kernel a linear call takes (host code, no HIP).
#pragma once

#include <stdint.h>

namespace rocs {

constexpr int kStreamBM = 256, kStreamBN = 256;   // the streaming kernel's tile

// Tile slots of the streaming kernel: without a request term (R = 0) the tiles
// cover the candidates contiguously, with one none straddles two requests.
inline int64_t stream_slots(int64_t N, int64_t R) { return R + (N + kStreamBN - 1) / kStreamBN; }

// Whether the streaming kernel is the faster one for a call that it can run.
//
// Its workgroups, one per CU, take whole 256 x 256 tiles, so its time is that
// of its rounds; the tiled kernel's smaller tiles pack better but stream K more
// slowly, the more so the longer K is. What decides is the share of the
// rounds' area that the call fills. (At most R - 1 slots come on top of the
// candidates' own.) Measured, us, streaming / tiled:
//   one round, K of 256 and more: share 0.5, 8,192 x 1024, K 512: 15.1 / 14.2,
//     K 4096: 78.8 / 82.3; 0.55, 9,011 x 1024, K 512: 15.4 / 18.3, K 1024: 25.1
//     / 30.7, K 4096: 80.6 / 113; 0.4, 6,553 x 1024, K 4096: 78.7 / 69.1.
//   K below 512: 0.65, 64,324 x 512, K 256: 45 / 35; 0.75, 98,304 x 256, K 256:
//     25.5 / 23.1; 0.8, 26,214 x 1024, K 256: 23.1 / 24.0; 1, 163,840 x 1024,
//     K 256: 107 / 158.
//   K 512: 0.65, 21,299 x 1024: 35.1 / 33.3; 0.67, 8,192 x 8,192: 92 / 117;
//     0.75, 24,576 x 1024: 35.3 / 34.6; 0.8, 26,214 x 1024: 35.8 / 38.6.
//   K 1024: 0.6, 19,660 x 1024: 55.8 / 52.3; 0.65, 21,299 x 1024: 59.0 / 59.5;
//     0.7, 22,937 x 1024: 58.4 / 61.0.
//   K 2048 and more: 0.55, 18,022 x 1024, K 2048: 98 / 96, K 4096: 184 / 188;
//     0.65, 21,299 x 1024, K 2048: 111 / 116, K 4096: 213 / 229.
inline bool stream_pays(int64_t N, int64_t D, int64_t K, int64_t R, int cus) {
  const int64_t tiles = (stream_slots(N, R) - (R > 0)) * ((D + kStreamBM - 1) / kStreamBM);
  const int64_t rounds = (tiles + cus - 1) / cus;
  const double share = (double)N * (double)D / ((double)(rounds * cus) * kStreamBM * kStreamBN);
  if (rounds == 1 && K >= 256) return K < 2048 ? share > 0.5 : share >= 0.5;
  return share >= (K < 512 ? 3.0 / 4 : K < 1024 ? 2.0 / 3 : K < 2048 ? 0.6 : 0.55);
}

}  // namespace rocs
