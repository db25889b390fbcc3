// IKBO fused linear (Eq. glm-linear, two-group case; Section 4.1 decomposition;
// broadcast-add fused into the GEMM epilogue, Section 4.2.1).
//
//   out[n][d] = act( sum_k W_CC[d][k] xc[n][k] + Z[m_n][d] + b[d] ),
//   Z = X^R W_CR^T computed once per request (batch size R).
//
// Two launches on the caller's stream:
//   1. request side: Z (fp32, [R, D]) on the matrix cores, plus the expanded
//      index map ids[n] = m_n, in one grid;
//   2. candidate side: a bf16 MFMA GEMM over the candidate batch whose
//      accumulators start from Z[m_n] + b, so the request term is added in
//      registers and only the final activations are written.
// The general path (fp32, sizes or pointers off the fast path's alignment) runs
// on the fp32 matrix instructions: two steps for large calls, for small ones a
// single launch that takes the request term into the candidates' product.
#include "common.h"
#include "kernels.h"
#include "launch.h"
#include "linear_rule.h"

#include <atomic>
#include <random>

namespace rocs {
namespace {

// ---------------------------------------------------------------------------
// Index map expansion (standalone; also used by rocs_request_ids).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void request_ids_kernel(const int32_t* __restrict__ off, int R,
                                                          int64_t N, int32_t* __restrict__ ids) {
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n < N) ids[n] = owner_of(off, R, n);
}

// ---------------------------------------------------------------------------
// Request-side GEMM, bf16 in: the request table Zb = X^R W_CR^T + b (fp32;
// the bias is folded in here, once per request) and, for a full GLM layer,
// the request-side output Y^R = act(X^R W_RR^T + b^R) (bf16) from the same
// launch: the stacked weight [W_RR; W_CR] of Section 4.1, one GEMM at batch
// size R. One workgroup per 16 x 16 output tile (the W_RR column tiles come
// first); its eight waves split K in 32-wide steps (operands straight from
// global memory into MFMA registers, each lane's 8 consecutive k are one
// 16-byte load) and reduce through LDS in a fixed order. A handful of
// workgroups at batch size R is bound by the latency of a wave's loads: with
// eight waves and eight steps in flight a K of 2048 is one round trip to L2
// (16 requests, 1024 outputs: 7 us), where four waves with four steps in
// flight made four (12 us); a K of 4096, 1024 outputs: 22 -> 12 us. Many
// requests take a wave per tile (request_gemm_many). Workgroups past the tiles
// expand the index map when the candidate GEMM needs it.
// ---------------------------------------------------------------------------
struct RequestOut {          // the optional Y^R part of the stacked weight
  const bf16_t* w;           // W_RR [d, K]
  const float* bias;         // b^R [d] or NULL
  bf16_t* y;                 // Y^R [R, d]
  int d, tiles, relu;        // tiles = ceil(d / 16); 0 when there is no Y^R
};

constexpr int kReqAhead = 8;   // k-steps of a wave in flight
constexpr int kReqMaxBlocks = 1 << 21;   // workgroups of 512 per launch; they loop over more tiles
// ... beside the workgroups that expand a map of up to 2^31 - 1 candidates.
static_assert((int64_t)kReqMaxBlocks * 512 + (int64_t(1) << 31) + 512 < int64_t(1) << 32, "grid");

// One 16 x 16 output tile of the stacked request GEMM, as one wave sees it.
struct RequestTile {
  const bf16_t* x;           // this lane's eight k of its request row ...
  const bf16_t* w;           // ... and of its weight row
  const float* bias;
  int r0, d0, D;             // first request, first column, columns of this output
  bool to_y, rok, dok;       // a tile of Y^R; this lane's rows are inside

  __device__ __forceinline__ RequestTile(const bf16_t* x_in, const bf16_t* w_in,
                                         const float* bias_in, int R, int K, int D_in, int tiles_d,
                                         const RequestOut& yr, int tile, int lane) {
    const int tiles_all = yr.tiles + tiles_d;
    const int t = tile % tiles_all;
    to_y = t < yr.tiles;                          // a column tile of Y^R
    bias = to_y ? yr.bias : bias_in;
    D = to_y ? yr.d : D_in;
    r0 = (tile / tiles_all) * 16;
    d0 = (to_y ? t : t - yr.tiles) * 16;
    const int row = lane & 15, kq = (lane >> 4) * 8;
    dok = d0 + row < D;
    rok = r0 + row < R;
    w = (to_y ? yr.w : w_in) + (int64_t)(d0 + row) * K + kq;
    x = x_in + (int64_t)(r0 + row) * K + kq;
  }
  // s[i] = Z[r0 + lane % 16][d0 + 4 (lane / 16) + i] without the bias.
  __device__ __forceinline__ void store(f32x4 s, float* z, const RequestOut& yr, int lane) const {
    const int row = lane & 15, d = d0 + (lane >> 4) * 4;
    if (!rok || d >= D) return;
    if (bias != nullptr) s += *reinterpret_cast<const f32x4*>(bias + d);
    if (to_y) {
      if (yr.relu) s = f32x4{fmaxf(s[0], 0.f), fmaxf(s[1], 0.f), fmaxf(s[2], 0.f), fmaxf(s[3], 0.f)};
      *reinterpret_cast<u32x2*>(yr.y + (int64_t)(r0 + row) * D + d) =
          u32x2{pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3])};
    } else {
      *reinterpret_cast<f32x4*>(z + (int64_t)(r0 + row) * D + d) = s;
    }
  }
};

// Tile `tile` by a 512-thread workgroup; `red` is 8 KiB of LDS. Returns whether
// it was a Zb tile (the candidate side's input); wave 0 has stored it.
__device__ __forceinline__ bool request_tile(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w_in,
    const float* __restrict__ bias_in, float* __restrict__ z, int R, int K, int D_in,
    int tiles_d, const RequestOut& yr, int tile, ROCS_LDS f32x4* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const RequestTile t(x, w_in, bias_in, R, K, D_in, tiles_d, yr, tile, lane);
  const int kq = (lane >> 4) * 8;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = wave * 32; k0 < K; k0 += 256 * kReqAhead) {
    u32x4 a[kReqAhead], b[kReqAhead];
#pragma unroll
    for (int j = 0; j < kReqAhead; ++j) {
      const int k = k0 + 256 * j;
      const bool kok = k + kq < K;
      a[j] = load16(t.w + k, t.dok && kok);
      b[j] = load16(t.x + k, t.rok && kok);
    }
#pragma unroll
    for (int j = 0; j < kReqAhead; ++j)
      if (k0 + 256 * j < K) acc = mfma16(as_bf16x8(a[j]), as_bf16x8(b[j]), acc);
  }
  red[wave * kWave + lane] = acc;
  __syncthreads();
  if (wave == 0) {
    f32x4 s = red[lane];
#pragma unroll
    for (int w = 1; w < 8; ++w) s += red[w * kWave + lane];
    t.store(s, z, yr, lane);
  }
  return !t.to_y;
}

__global__ __launch_bounds__(512) void request_gemm_bf16(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w_in, const float* __restrict__ bias_in,
    float* __restrict__ z, const int32_t* __restrict__ off, int32_t* __restrict__ ids, int R,
    int64_t N, int K, int D_in, int tiles_d, int z_tiles, int z_blocks, RequestOut yr) {
  if ((int)blockIdx.x >= z_blocks) {
    const int64_t n = (int64_t)(blockIdx.x - z_blocks) * 512 + threadIdx.x;
    if (n < N) ids[n] = owner_of(off, R, n);
    return;
  }
  __shared__ f32x4 red[8 * kWave];
  for (int t = (int)blockIdx.x; t < z_tiles; t += z_blocks) {
    request_tile(x, w_in, bias_in, z, R, K, D_in, tiles_d, yr, t, (ROCS_LDS f32x4*)red);
    __syncthreads();                      // red is free for the next tile
  }
}

// The same tiles, a wave each: the eight slices of K in eight accumulators,
// added in the same order, so the values are the same. For many requests: the
// tiles fill the chip by themselves, and at a short K a workgroup per tile has
// most of its waves without a k-step.
__global__ __launch_bounds__(512) void request_gemm_many(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w_in, const float* __restrict__ bias_in,
    float* __restrict__ z, const int32_t* __restrict__ off, int32_t* __restrict__ ids, int R,
    int64_t N, int K, int D_in, int tiles_d, int z_tiles, int z_blocks, RequestOut yr) {
  if ((int)blockIdx.x >= z_blocks) {
    const int64_t n = (int64_t)(blockIdx.x - z_blocks) * 512 + threadIdx.x;
    if (n < N) ids[n] = owner_of(off, R, n);
    return;
  }
  const int lane = threadIdx.x & 63, kq = (lane >> 4) * 8;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t at = (int64_t)blockIdx.x * 8 + wave; at < z_tiles; at += (int64_t)z_blocks * 8) {
    const RequestTile t(x, w_in, bias_in, R, K, D_in, tiles_d, yr, (int)at, lane);
    f32x4 acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 256) {
      u32x4 a[8], b[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bool kok = k0 + 32 * j + kq < K;
        a[j] = load16(t.w + k0 + 32 * j, t.dok && kok);
        b[j] = load16(t.x + k0 + 32 * j, t.rok && kok);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (k0 + 32 * j < K) acc[j] = mfma16(as_bf16x8(a[j]), as_bf16x8(b[j]), acc[j]);
    }
    f32x4 s = acc[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) s += acc[j];
    t.store(s, z, yr, lane);
  }
}

// Launch of the request GEMM with `ids` expanded beside it (n_ids candidates).
hipError_t launch_request(const LinearArgs& a, int cus, int tiles_d, int req_tiles,
                          int64_t n_ids, const RequestOut& yr, hipStream_t s) {
  // A wave per tile from eight tiles a CU on, more the longer its K is: a wave
  // walks K alone. Whole call (us, workgroup / wave per tile), requests x
  // outputs, K: 256 x 1024 (1,024 tiles), 256: 9.0 / 9.5, K 1024: 13.8 / 19.9;
  // 512 x 1024 (2,048), 64: 11.6 / 7.9, K 1024: 22.2 / 20.4; 300 x 2000 (2,375),
  // 2000: 81 / 93; 2000 x 1024 (8,000), 4096: 232 / 232; 16,384 x 1024 (65,536),
  // 64: 207 / 67, K 256: 235 / 138.
  const bool many = (int64_t)req_tiles * 1024 >= 8 * (int64_t)cus * (a.k_req > 1024 ? a.k_req : 1024);
  const int blocks = many ? (req_tiles + 7) / 8 : req_tiles;
  const int z_blocks = blocks < kReqMaxBlocks ? blocks : kReqMaxBlocks;
  const int id_blocks = (int)((n_ids + 511) / 512);
  return launch_kernel(many ? request_gemm_many : request_gemm_bf16, dim3(z_blocks + id_blocks),
                       dim3(512), s, static_cast<const bf16_t*>(a.x_req),
                       static_cast<const bf16_t*>(a.w_req), a.bias, a.z, a.cand_offsets, a.ids,
                       (int)a.R, a.N, (int)a.k_req, (int)a.d_out, tiles_d, req_tiles, z_blocks, yr);
}

// ---------------------------------------------------------------------------
// Tiled candidate GEMM, bf16 MFMA 32x32x16: any map, any K and D of the fast
// path (multiples of 8 and 4), the pointwise residual input, and calls too
// small for the streaming kernel below.
//
// Matrix-core roles: A = W_CC rows (output features d), B = candidate rows, so
// each lane's accumulator holds, for one candidate, four runs of 4 consecutive
// output features. Workgroup tile BM (features) x BN (candidates), four waves,
// WVM of them along the features; three workgroups share a CU (two of 64 x 64
// with a residual), so one's prologue (index map, request rows, first slabs)
// and epilogue run under the others' products. K arrives in
// BK-wide slabs by LDS DMA, S - 1 slabs ahead of use; 16-byte chunks are
// XOR-swizzled by row so that the 16 rows of a quarter-wave read fall on
// distinct banks. Chunks past K come from a zeroed address, rows past the
// operands repeat the last one and are not stored.
//
// HAS_ADD: the residual's slab travels the same way, and the sum round(x +
// x_add) is formed on the fragments, by every wave along the features again:
// about as much vector work as a pair of matrix instructions takes, so at a
// longer K the waves stand side by side along the candidates (WVM 1).
//
// Epilogue: each candidate's own request row Z[m_n] (or the bias), loaded in
// the prologue, is added after the products (the order of the streaming
// kernel, so the two give the same values), then the activation; the wave's
// block goes through LDS so that a store instruction covers whole row
// segments.
// What bounds it: reads of the two operands through L2 (each 128 x 128 tile
// reads 256 rows of K) and the output stores; the slab depth, the request rows
// in the prologue or the epilogue and two to four waves a SIMD all measured
// within 5% (the residual form gains 10% from the epilogue: 100,000 x 1024,
// K 512: 228 / 252 us). Against register-staged slabs with one slab ahead and
// 8-byte stores: 64,324 x 512, K 256, shuffled: 58 -> 39 us; 407,816 x 552, K
// 104: 310 -> 241; with residual 100,000 x 1024, K 512: 227 -> 205, K 1024: 387
// -> 385, 3,000 x 4096, K 4096: 189 -> 193, 20,011 x 300, K 360: 20.7 -> 19.5.
// ---------------------------------------------------------------------------
__device__ __constant__ u32x4 g_zero_chunk = {0u, 0u, 0u, 0u};

template <int BM, int BN, int BK, int S, bool HAS_ADD, int WVM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void ikbo_gemm_tile(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ xadd, const bf16_t* __restrict__ w,
    const float* __restrict__ z, const int32_t* __restrict__ ids, bf16_t* __restrict__ out,
    int64_t N, int K, int D, int tiles_m, int relu, int R) {
  constexpr int WM = BM / WVM, WN = BN / (4 / WVM);   // wave block
  constexpr int FM = WM / 32, FN = WN / 32;
  constexpr bool ZLATE = HAS_ADD;              // request rows loaded in the epilogue
  constexpr int ZFN = ZLATE ? 1 : FN;
  constexpr int ROWB = 2 * BK;                 // bytes of one slab row
  constexpr int CPR = ROWB / 16;               // its 16-byte chunks
  constexpr int RPI = 1024 / ROWB;             // slab rows per wave-wide DMA load
  constexpr int NA = BM / RPI / 4, NB = BN / RPI / 4;   // DMA loads per wave and slab
  constexpr int NL = NA + (HAS_ADD ? 2 : 1) * NB;
  constexpr int XO = BM * ROWB, AO = XO + BN * ROWB;    // candidates, residual in a stage
  constexpr int STAGE = AO + (HAS_ADD ? BN * ROWB : 0);
  constexpr int ORB = 2 * WM;                  // bytes of one output row of a wave's block
  static_assert(NA >= 1 && NB >= 1 && NL * (S - 1) < 64, "staging does not tile");
  static_assert(S * STAGE >= 4 * 32 * ORB, "the output staging reuses the ring");
  __shared__ __attribute__((aligned(1024))) char lds[S * STAGE];
  ROCS_LDS char* const lds3 = (ROCS_LDS char*)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const uint32_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const int m0 = (int)(tile % (uint32_t)tiles_m) * BM;
  const int64_t n0 = (int64_t)(tile / (uint32_t)tiles_m) * BN;
  const int wm0 = wave % WVM * WM, wn0 = wave / WVM * WN;
  const uint32_t lbase = lds_addr(lds);
  auto swz = [](int row) { return CPR == 8 ? (row >> 1) & 7 : (row >> 2) & 3; };

  // DMA lane map: load i of this wave fills rows RPI (N? wave + i) + lane /
  // CPR, chunk position lane % CPR, with chunk (lane % CPR) ^ swz(row).
  const char* pa[NA];
  const char* pb[NB];
  int chunk_a[NA], chunk_b[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int row = RPI * (NA * wave + i) + lane / CPR;
    chunk_a[i] = 8 * ((lane % CPR) ^ swz(row));
    pa[i] = reinterpret_cast<const char*>(w + (int64_t)min(m0 + row, D - 1) * K + chunk_a[i]);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int row = RPI * (NB * wave + i) + lane / CPR;
    chunk_b[i] = 8 * ((lane % CPR) ^ swz(row));
    pb[i] = reinterpret_cast<const char*>(x + min(n0 + row, N - 1) * K + chunk_b[i]);
  }
  const int64_t to_add = HAS_ADD ? reinterpret_cast<const char*>(xadd) - reinterpret_cast<const char*>(x) : 0;
  const char* const zeros = reinterpret_cast<const char*>(&g_zero_chunk);
  const int nk = (K + BK - 1) / BK;
  auto issue = [&](int s, int slot) __attribute__((always_inline)) {
    const uint32_t dst = lbase + (uint32_t)(slot * STAGE);
    const int64_t at = (int64_t)s * ROWB;
    const int left = K - s * BK;               // valid elements of the slab's rows
#pragma unroll
    for (int i = 0; i < NA; ++i)
      lds_dma16(left >= BK || chunk_a[i] < left ? pa[i] + at : zeros,
                dst + (uint32_t)(1024 * (NA * wave + i)));
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const bool ok = left >= BK || chunk_b[i] < left;
      lds_dma16(ok ? pb[i] + at : zeros, dst + (uint32_t)(XO + 1024 * (NB * wave + i)));
      if constexpr (HAS_ADD)
        lds_dma16(ok ? pb[i] + at + to_add : zeros, dst + (uint32_t)(AO + 1024 * (NB * wave + i)));
    }
  };

  // The request row of each lane's candidates. A request id outside [0, R) (a
  // malformed caller map) is clamped into range: wrong rows, never an access
  // outside Z.
  int rq[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int64_t n = min(n0 + wn0 + 32 * fn + l32, N - 1);
    rq[fn] = ids != nullptr ? (int)min((uint32_t)ids[n], (uint32_t)(R - 1)) : 0;
  }
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < nk) issue(s, s);
  f32x4 zv[ZFN][FM][4];
  auto load_z = [&](int fn) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int d = m0 + wm0 + 32 * fm + 8 * q + 4 * hh;
        zv[fn % ZFN][fm][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (z != nullptr && d < D)
          zv[fn % ZFN][fm][q] = *reinterpret_cast<const f32x4*>(z + (int64_t)rq[fn] * D + d);
      }
  };
  if constexpr (!ZLATE) {
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) load_z(fn);
  }

  // Fragments: row 32 f + l32 of the wave's block, chunk 2 ks + hh; the
  // swizzle turns the k-step into an XOR with 32 ks.
  const uint32_t fr = (uint32_t)(l32 * ROWB + 16 * (hh ^ swz(l32)));
  const uint32_t fa = (uint32_t)(wm0 * ROWB) + fr, fb = (uint32_t)(XO + wn0 * ROWB) + fr;
  f32x16 acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = f32x16{};
  int slot = 0, next = S - 1;
  for (int kt = 0; kt < nk; ++kt) {
    // Slab kt resident: everything but the S - 2 slabs issued after it.
    if (kt + S - 2 < nk) wait_vmcnt<(S - 2) * NL>(); else wait_vmcnt<0>();
    ring_barrier();                            // ... of every wave; slab kt - 1's slot is free
    if (kt + S - 1 < nk) issue(kt + S - 1, next);
    const uint32_t so = (uint32_t)(slot * STAGE);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 af[FM], bfr[FN];
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
        af[fm] = *reinterpret_cast<const ROCS_LDS bf16x8*>(
            lds3 + so + 32 * fm * ROWB + (fa ^ (32u * ks)));
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        bfr[fn] = *reinterpret_cast<const ROCS_LDS bf16x8*>(
            lds3 + so + 32 * fn * ROWB + (fb ^ (32u * ks)));
        if constexpr (HAS_ADD) {
          const u32x4 p = as_u32x4(bfr[fn]);
          const u32x4 q = *reinterpret_cast<const ROCS_LDS u32x4*>(
              lds3 + so + (AO - XO) + 32 * fn * ROWB + (fb ^ (32u * ks)));
          u32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            v[e] = pack_bf16x2(bf16_lo(p[e]) + bf16_lo(q[e]), bf16_hi(p[e]) + bf16_hi(q[e]));
          bfr[fn] = as_bf16x8(v);
        }
      }
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mfma32(af[fm], bfr[fn], acc[fm][fn]);
    }
    slot = slot + 1 == S ? 0 : slot + 1;
    next = next + 1 == S ? 0 : next + 1;
  }
  ring_barrier();                              // the ring is free

  // Element 4 q + i of acc[fm][fn] is feature 32 fm + 8 q + 4 hh + i of
  // candidate 32 fn + l32. After the half-wave swap lane (l32, hh) holds
  // features 32 fm + 16 j + 8 hh .. + 7: one 16-byte chunk of its row in the
  // wave's staging area, at chunk position ^ row.
  const uint32_t st = (uint32_t)(wave * 32 * ORB);
  const int64_t nw = n0 + wn0;
  const int dw = m0 + wm0;
  const uint32_t lo = act_floor(relu);
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    if constexpr (ZLATE) load_z(fn);
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t p[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x16& a = acc[fm][fn];
          const f32x4 zq = zv[fn % ZFN][fm][2 * j + u];
          const int e = 4 * (2 * j + u);
          p[u][0] = pack_bf16x2(a[e] + zq[0], a[e + 1] + zq[1]);
          p[u][1] = pack_bf16x2(a[e + 2] + zq[2], a[e + 3] + zq[3]);
          p[u][0] = act_bf16x2(p[u][0], lo);
          p[u][1] = act_bf16x2(p[u][1], lo);
        }
        const auto s0 = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
        const int ch = (4 * fm + 2 * j + hh) ^ (l32 & (ORB / 16 - 1));
        *reinterpret_cast<ROCS_LDS u32x4*>(lds3 + st + l32 * ORB + 16 * ch) =
            u32x4{s0[0], s1[0], s0[1], s1[1]};
      }
    // Read back row-contiguous; 16-byte stores where the rows allow them.
    if (D % 8 == 0) {
      constexpr int LPR = ORB / 16;            // lanes per row
#pragma unroll
      for (int i = 0; i < 32 * LPR / 64; ++i) {
        const int r = (64 / LPR) * i + lane / LPR, c = lane % LPR;
        const u32x4 v = *reinterpret_cast<const ROCS_LDS u32x4*>(
            lds3 + st + r * ORB + 16 * (c ^ (r & (ORB / 16 - 1))));
        const int64_t n = nw + 32 * fn + r;
        const int d = dw + 8 * c;
        if (n < N && d < D) *reinterpret_cast<u32x4*>(out + n * D + d) = v;
      }
    } else {
      constexpr int LPR = ORB / 8;
#pragma unroll
      for (int i = 0; i < 32 * LPR / 64; ++i) {
        const int r = (64 / LPR) * i + lane / LPR, c = lane % LPR;
        const u32x2 v = *reinterpret_cast<const ROCS_LDS u32x2*>(
            lds3 + st + r * ORB + 16 * ((c >> 1) ^ (r & (ORB / 16 - 1))) + 8 * (c & 1));
        const int64_t n = nw + 32 * fn + r;
        const int d = dw + 4 * c;
        if (n < N && d < D) *reinterpret_cast<u32x2*>(out + n * D + d) = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Streaming candidate GEMM (bf16, K a multiple of 64), the main path.
//
// Persistent workgroups, one per CU, walk the 256 (features) x 256
// (candidates) output tiles with a stride of the grid; eight waves, two per
// SIMD, each own a 64 x 128 block (8 MFMA 32x32 accumulators, 128 of the
// wave's 256 registers), so one wave's stalls (fragment reads, the
// epilogue's stores) leave the SIMD to the other. K arrives in 64-wide slabs
// (128-byte row segments: whole cache lines, which the L2 serves at twice the
// rate of half lines) through LDS rings filled by LDS DMA loads, as one
// stream across tile boundaries: the weight slab (L2-resident) one slab ahead
// of use in a 2-deep ring, the candidate slab (from HBM, longer latency) two
// slabs ahead in a 3-deep ring; together exactly the 160 KiB of LDS. The
// 16-byte chunks of each slab row are XOR-swizzled by (row / 2) % 8, which
// puts the 16 rows read by each quarter-wave on distinct banks; fragments
// are read one k-step ahead.
//
// Producer waves: waves 0-3 issue every DMA load (two pieces between
// consecutive MFMA groups), waves 4-7 none. The two waves of a SIMD do not
// progress alike (the arbiter favours the older one, waves 0-3), so loads
// issued by the slower waves arrived late and the whole workgroup waited at
// the slab barrier for them; the faster waves have that time to spare. Each
// wave waits only for its own loads (the vector-memory counter is per wave),
// so waves 4-7 never wait on a load of the ring.
// IKBO tiling (Section 4.2.1): with a request term, tiles never straddle two
// requests: request r owns tile slots r + floor(off[r] / 256) ... (the last
// one partial), so the whole tile shares one row of the request table
// Zb = X^R W_CR^T + b, added in the epilogue (the broadcast add fused into
// the GEMM). Without a request term the tiles cover the candidate rows
// contiguously and Zb is the bias (or absent).
//
// Epilogue: Zb, activation on packed bf16, then the two wave halves swap
// 8-byte pieces so every lane holds 8 consecutive features of one row. Stored
// from that layout, each instruction would write 32 bytes into each of 32
// rows, and a CU then stores at about a quarter of the rate it reaches with
// whole 128-byte lines (measured on this part: ~38 GB/s against ~150 GB/s
// per CU). So each wave passes its block through 4 KiB of the candidate slot
// the last slab has just released (after a barrier): 32 rows at a time
// written in that layout, read back row-contiguous, and stored as 8 rows x
// 128 bytes per instruction.
//
// Rows past the tile's end are clamped loads whose results are not stored.
// ---------------------------------------------------------------------------
constexpr int kStreamBK = 64;
constexpr int kCpolNT = 2;   // buffer-instruction cache policy bits: NT (the former SLC bit)

struct StreamTile {
  int slot;       // tile slot (candidate block)
  int mb;         // feature block
  int r;          // request of the slot (0 without a request term)
  int64_t n0;     // first candidate row
  int rows;       // candidate rows in the tile
  int m0;         // first output feature
};

// Tiles are numbered slot * tiles_m + mb and a workgroup takes every
// grid-th one; the step is passed split into (slot, mb) parts so that no
// division runs on the device.
struct StreamStep {
  int slots, mbs;                  // grid = slots * tiles_m + mbs, mbs < tiles_m
};

__device__ __forceinline__ void stream_next(StreamTile& c, StreamStep st, int tiles_m) {
  c.slot += st.slots;
  c.mb += st.mbs;
  if (c.mb >= tiles_m) {
    c.mb -= tiles_m;
    ++c.slot;
  }
}

// Move `c` forward (in grid steps) to the first tile that holds candidate
// rows; false when the slots are exhausted. All values are wave-uniform.
template <typename OffPtr>
__device__ __forceinline__ bool stream_seek(StreamTile& c, StreamStep st, int n_slots,
                                            int tiles_m, OffPtr off, int R, int64_t N) {
  for (; c.slot < n_slots; stream_next(c, st, tiles_m)) {
    c.m0 = c.mb * kStreamBM;
    if (off != nullptr) {
      auto base_of = [&](int r) { return (int64_t)r + off[r] / kStreamBN; };   // tile slots
      while (c.r + 1 < R && base_of(c.r + 1) <= c.slot) ++c.r;
      const int64_t end = off[c.r + 1];
      c.n0 = (int64_t)off[c.r] + (c.slot - base_of(c.r)) * kStreamBN;
      if (c.n0 < end) {
        c.rows = (int)(end - c.n0 < kStreamBN ? end - c.n0 : kStreamBN);
        return true;
      }
    } else {
      c.n0 = (int64_t)c.slot * kStreamBN;
      c.rows = (int)(N - c.n0 < kStreamBN ? N - c.n0 : kStreamBN);
      return true;
    }
  }
  return false;
}

// The request side inside the candidate kernel (Section 4.2.3, combined
// request and candidate kernels): the stacked request GEMM's 16 x 16 tiles
// are computed first, by the workgroups taken in ascending order, and each
// Zb tile publishes a completion flag (agent-scope release: the tile's
// stores reach every XCD before the flag does). A workgroup then issues its
// first candidate loads and waits for the flags while they are in flight,
// then fences once (agent-scope acquire); the main loop and the epilogue
// carry no request-side state. Flags hold this call's epoch (a per-process
// random salt and a call counter), so stale flags from earlier calls never
// match and nothing resets them. The wait is bounded: past the limit the
// workgroup computes every tile whose flag is still unset itself (the same
// code, so the same values), so every workgroup always finishes.
struct FusedRequest {
  const bf16_t* x;           // x_req [R, K]
  const bf16_t* w;           // W_CR [D, K]
  const float* bias;         // b [D] or NULL
  float* z;                  // Zb [R, D] (workspace)
  RequestOut yr;             // optional Y^R part of the stacked weight
  uint64_t* flags;           // one per Zb tile: ceil(R / 16) x ceil(D / 16)
  uint64_t epoch;
  int K, tiles_d, n_tiles;   // n_tiles: all request tiles (Y^R and Zb)
};

constexpr int kFlagSpinLimit = 1 << 17;   // polls of about 0.3 us each

// This call's flag value: a per-process random salt in the high word and a
// call counter below it (never zero).
uint64_t next_epoch() {
  static std::atomic<uint64_t> counter{[] {
    std::random_device rd;
    return (uint64_t)rd() << 32 | 1u;
  }()};
  return counter.fetch_add(1, std::memory_order_relaxed);
}

template <bool HAS_ZB, bool RELU, bool FUSED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ikbo_gemm_stream(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                      const float* __restrict__ zb, const int32_t* __restrict__ off_g,
                      bf16_t* __restrict__ out, int R, int64_t N, int K, int D, int tiles_m,
                      int n_slots, StreamStep step_g, FusedRequest fr) {
  constexpr int BM = kStreamBM, BN = kStreamBN, BK = kStreamBK;
  constexpr int NSA = 2, NSB = 3;                // ring depths: weights, candidates
  constexpr int ROWB = BK * 2;                   // bytes of one slab row (128)
  constexpr int RPI = 1024 / ROWB;               // slab rows per wave-wide DMA load (8)
  constexpr int NI = BM / RPI / 8;               // DMA loads per wave and operand (4)
  constexpr int SLAB = BM * ROWB;                // bytes of one operand slab (32 KiB)
  constexpr int BBASE = NSA * SLAB;              // candidate ring after the weight ring
  static_assert(BM == BN && NI * RPI * 8 == BM && ROWB == 128, "tiling");
  static_assert((NSA + NSB) * SLAB <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char lds[(NSA + NSB) * SLAB];
  ROCS_LDS char* const lds3 = (ROCS_LDS char*)lds;
  // The offsets are read-only for the kernel's lifetime: read them through
  // the constant address space (scalar loads).
  const __attribute__((address_space(4))) int32_t* off =
      (const __attribute__((address_space(4))) int32_t*)off_g;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5, h4 = 4 * hh;
  const int wm0 = (wave & 3) * 64, wn0 = (wave >> 2) * 128;
  const int nk = K / BK;
  const int rowb = K * 2;
  const int logical = (int)xcd_remap(blockIdx.x, gridDim.x);
  // Request tiles reduce through the third candidate ring slot, which the
  // prologue leaves empty.
  ROCS_LDS f32x4* const red = (ROCS_LDS f32x4*)(lds3 + BBASE + 2 * SLAB);
  auto run_request_tile = [&](int t) __attribute__((always_inline)) {
    const bool is_zb = request_tile(fr.x, fr.w, fr.bias, fr.z, R, fr.K, D, fr.tiles_d, fr.yr,
                                    t, red);
    if (is_zb && threadIdx.x == 0) {      // wave 0 stored the tile
      const int tiles_all = fr.yr.tiles + fr.tiles_d;
      const int fi = (t / tiles_all) * fr.tiles_d + (t % tiles_all - fr.yr.tiles);
      __hip_atomic_store(fr.flags + fi, fr.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  };
  if constexpr (FUSED) {
    for (int t = logical; t < fr.n_tiles; t += (int)gridDim.x) run_request_tile(t);
  }
  // Candidate tiles: descending for the workgroups that took request tiles
  // (they get the smaller share when the tiles do not divide evenly).
  const int first = FUSED ? (int)gridDim.x - 1 - logical : logical;
  const uint32_t lbase = lds_addr(lds);

  // DMA lane map (producer waves 0-3): load i of this wave fills slab rows
  // RPI (PI wave + i) + lane / 8, chunk position lane % 8, with chunk
  // (lane % 8) ^ ((row / 2) % 8). Rows past the operand's valid rows are
  // clamped to the last valid one.
  constexpr int PI = 2 * NI;                     // DMA loads per producer wave and operand (8)
  const bool producer = wave < 4;
  const int drow0 = RPI * PI * (wave & 3) + (lane >> 3);
  auto dma_piece = [&](const char* src, int rowlim, uint32_t dst, int i) __attribute__((always_inline)) {
    const int row = drow0 + RPI * i;
    const uint32_t chunk = 16u * (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
    lds_dma16_sv(src, __umul24((uint32_t)min(row, rowlim), (uint32_t)rowb) + chunk,
                 dst + (uint32_t)(RPI * (PI * (wave & 3) + i) * ROWB));
  };
  auto dma_all = [&](const char* src, int rowlim, uint32_t dst) __attribute__((always_inline)) {
    if (producer) {
#pragma unroll
      for (int i = 0; i < PI; ++i) dma_piece(src, rowlim, dst, i);
    }
  };

  // The issue cursor walks the slab sequence two slabs ahead of compute and
  // plans the candidate slab; the weight slab of the same position follows
  // one slab later (weights sit in L2, candidates come from HBM).
  StreamTile ic{first / tiles_m, first % tiles_m, 0, 0, 0, 0};
  bool ic_live = stream_seek(ic, step_g, n_slots, tiles_m, off, R, N);
  int ic_s = 0;
  int buf_b = 0, buf_a = 0;              // ring slots of the next loads
  const char* a_next_src = nullptr;      // weight slab queued behind the candidates
  int a_next_lim = 0;
  bool a_queued = false;
  // Loads planned for the current slab: weights of slab g + 1, candidates
  // of slab g + 2. They are issued one at a time between the MFMAs.
  const char* pa_src = nullptr;
  int pa_lim = 0;
  uint32_t pa_dst = 0;
  bool pa_on = false;
  const char* pb_src = nullptr;
  int pb_lim = 0;
  uint32_t pb_dst = 0;
  bool pb_on = false;
  auto plan_b = [&]() __attribute__((always_inline)) {
    const int kb = ic_s * ROWB;
    pb_src = reinterpret_cast<const char*>(x + ic.n0 * K) + kb;
    pb_lim = ic.rows - 1;
    pb_dst = lbase + (uint32_t)(BBASE + buf_b * SLAB);
    pb_on = true;
    buf_b = buf_b == NSB - 1 ? 0 : buf_b + 1;
    a_next_src = reinterpret_cast<const char*>(w + (int64_t)ic.m0 * K) + kb;
    a_next_lim = D - 1 - ic.m0;
    a_queued = true;
    if (++ic_s == nk) {
      ic_s = 0;
      stream_next(ic, step_g, tiles_m);
      ic_live = stream_seek(ic, step_g, n_slots, tiles_m, off, R, N);
    }
  };
  auto plan_a = [&]() __attribute__((always_inline)) {
    pa_src = a_next_src;
    pa_lim = a_next_lim;
    pa_dst = lbase + (uint32_t)(buf_a * SLAB);
    pa_on = true;
    buf_a ^= 1;
    a_queued = false;
  };
  // Group p (0..7) of the planned loads, two pieces each: weights for
  // p < 4, candidates after.
  auto dma_plan_piece = [&](int p) __attribute__((always_inline)) {
    if (!producer) return;
    if (p < NI) {
      if (pa_on) {
        dma_piece(pa_src, pa_lim, pa_dst, 2 * p);
        dma_piece(pa_src, pa_lim, pa_dst, 2 * p + 1);
      }
    } else {
      if (pb_on) {
        dma_piece(pb_src, pb_lim, pb_dst, 2 * (p - NI));
        dma_piece(pb_src, pb_lim, pb_dst, 2 * (p - NI) + 1);
      }
    }
  };

  // Fragment addresses within an operand slab: row 32 f + l32 of the wave's
  // quarter, chunk 2 ks + hh; the swizzle turns the ks step into XOR 32 ks.
  const uint32_t fa0 = (uint32_t)(l32 * ROWB + 16 * (hh ^ ((l32 >> 1) & 7)));
  f32x16 acc[2][4];
  int cbuf_a = 0, cbuf_b = 0;            // ring slots of the slab being computed
  // Fragments, double-buffered across k-steps (slot ks % 2): the reads of
  // step ks + 1 are in flight while the MFMAs of step ks run. The last
  // k-step of a slab that is not a tile's last is deferred: its fragments
  // are read (and waited for) before the slab barrier, and its MFMAs run
  // after the barrier, while the next slab's first fragment reads are in
  // flight; every wave would otherwise start each slab waiting for LDS. The
  // accumulation order is unchanged.
  bf16x8 af[2][2], bfr[2][4];
  auto compute = [&](auto first_slab, auto last_slab) __attribute__((always_inline)) {
    constexpr bool kFirst = decltype(first_slab)::value;
    constexpr bool kLastS = decltype(last_slab)::value;
    constexpr int KSTEPS = BK / 16;
    const uint32_t sa = (uint32_t)(cbuf_a * SLAB) + wm0 * ROWB;
    const uint32_t sb = (uint32_t)(BBASE + cbuf_b * SLAB) + wn0 * ROWB;
    auto load_frags = [&](int ks, int slot) __attribute__((always_inline)) {
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        if (f < 2) af[slot][f] = *reinterpret_cast<const ROCS_LDS bf16x8*>(lds3 + sa + 32 * f * ROWB + (fa0 ^ (32u * ks)));
        bfr[slot][f] = *reinterpret_cast<const ROCS_LDS bf16x8*>(lds3 + sb + 32 * f * ROWB + (fa0 ^ (32u * ks)));
      }
    };
    // DMA group g (0..7) goes with the g-th MFMA group of the slab.
    constexpr int kDeferred = kFirst ? 0 : 2;          // MFMA groups of the previous slab
    load_frags(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!kFirst) {
#pragma unroll
      for (int fm = 0; fm < 2; ++fm) {
#pragma unroll
        for (int fn = 0; fn < 4; ++fn) acc[fm][fn] = mfma32(af[1][fm], bfr[1][fn], acc[fm][fn]);
        dma_plan_piece(fm);
        __builtin_amdgcn_sched_barrier(0x0002 | 0x0004);
      }
    }
    constexpr int KRUN = kLastS ? KSTEPS : KSTEPS - 1;
#pragma unroll
    for (int ks = 0; ks < KRUN; ++ks) {
      const int cur = ks & 1;
      if (ks + 1 < KSTEPS) load_frags(ks + 1, cur ^ 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int fm = 0; fm < 2; ++fm) {
#pragma unroll
        for (int fn = 0; fn < 4; ++fn) {
          if constexpr (kFirst) {
            if (ks == 0) {
              const f32x16 zero = {};
              acc[fm][fn] = mfma32(af[cur][fm], bfr[cur][fn], zero);
              continue;
            }
          }
          acc[fm][fn] = mfma32(af[cur][fm], bfr[cur][fn], acc[fm][fn]);
        }
        if (kDeferred + 2 * ks + fm < 8) dma_plan_piece(kDeferred + 2 * ks + fm);
        // Keep MFMAs and loads in this order; ALU work may move.
        __builtin_amdgcn_sched_barrier(0x0002 | 0x0004);
      }
    }
#pragma unroll
    for (int g = kDeferred + 2 * KRUN; g < 8; ++g) dma_plan_piece(g);
    // The deferred step's fragments are in registers before the barrier
    // hands this slab's ring slots to the next loads.
    if constexpr (!kLastS) wait_lgkmcnt0();
  };

  // Request row Zb[m0 + wm0 + 32 fm + 8 q + h4 .. +3] of the tile, loaded
  // after the tile's last MFMAs (the fragment registers are free then) and
  // added in the epilogue. The buffer's extent is the request's row, so
  // features past D read as zero.
  f32x4 zv[2][4];
  auto load_zb = [&](const StreamTile& c) __attribute__((always_inline)) {
    if constexpr (HAS_ZB) {
      const auto rz = buffer_rsrc(zb + (int64_t)c.r * D, (uint32_t)D * 4u);
      const uint32_t vo = 4u * (uint32_t)(c.m0 + wm0 + h4);
#pragma unroll
      for (int fm = 0; fm < 2; ++fm)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          zv[fm][q] = __builtin_bit_cast(
              f32x4, __builtin_amdgcn_raw_buffer_load_b128(rz, vo + 4u * (32 * fm + 8 * q), 0, 0));
    }
  };

  // Combined kernel: wait (bounded) until every Zb tile's flag carries this
  // call's epoch; past the limit, compute the missing tiles here.
  auto wait_request_side = [&]() __attribute__((always_inline)) {
    const int nflags = ((R + 15) / 16) * fr.tiles_d;
    int spins = 0;
    for (; spins < kFlagSpinLimit; ++spins) {
      bool ok = true;
      for (int i = lane; i < nflags; i += kWave)
        ok &= __hip_atomic_load(fr.flags + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == fr.epoch;
      if (__ballot(!ok) == 0) break;
      __builtin_amdgcn_s_sleep(8);
    }
    // Workgroup-wide verdicts go through one LDS word past the reduction
    // area, so every wave takes the same branch around the tiles' barriers.
    ROCS_LDS int* const verdict = (ROCS_LDS int*)(lds3 + BBASE + 2 * SLAB + 8192);
    if (threadIdx.x == 0) *verdict = 0;
    __syncthreads();
    if (lane == 0 && spins == kFlagSpinLimit) *verdict = 1;
    __syncthreads();
    const bool timed_out = *verdict != 0;
    __syncthreads();
    if (timed_out) {
      const int tiles_all = fr.yr.tiles + fr.tiles_d;
      for (int fi = 0; fi < nflags; ++fi) {
        if (threadIdx.x == 0)
          *verdict = __hip_atomic_load(fr.flags + fi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != fr.epoch;
        __syncthreads();
        const bool run = *verdict != 0;
        __syncthreads();
        if (run) run_request_tile((fi / fr.tiles_d) * tiles_all + fr.yr.tiles + fi % fr.tiles_d);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  };

  // Epilogue. Element 4 q + i of acc[fm][fn] is feature 32 fm + 8 q + h4 + i
  // of candidate 32 fn + l32 (within the wave's block). For q = 2j, 2j + 1
  // the lower half-wave keeps its q = 2j words and takes the upper half's,
  // the upper half keeps q = 2j + 1 and takes the lower half's: then lane
  // (l32, hh) holds features 32 fm + 16 j + 8 hh .. +7, one 16-byte store.
  auto packed = [&](int fm, int fn, int q, uint32_t& lo, uint32_t& hi) __attribute__((always_inline)) {
    const f32x16& a = acc[fm][fn];
    float v0 = a[4 * q], v1 = a[4 * q + 1], v2 = a[4 * q + 2], v3 = a[4 * q + 3];
    if constexpr (HAS_ZB) {
      v0 += zv[fm][q][0];
      v1 += zv[fm][q][1];
      v2 += zv[fm][q][2];
      v3 += zv[fm][q][3];
    }
    lo = pack_bf16x2(v0, v1);
    hi = pack_bf16x2(v2, v3);
    if constexpr (RELU) {
      lo = relu_bf16x2(lo);
      hi = relu_bf16x2(hi);
    }
  };
  auto swapped = [&](int fm, int fn, int j) __attribute__((always_inline)) {
    uint32_t e0, e1, o0, o1;                     // words of q = 2j and q = 2j + 1
    packed(fm, fn, 2 * j, e0, e1);
    packed(fm, fn, 2 * j + 1, o0, o1);
    const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
    const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
    // Lower half: {own q = 2j, partner's q = 2j}; upper: {partner's q = 2j + 1, own}.
    const uint32_t w0 = s0[0], w2 = s0[1], w1 = s1[0], w3 = s1[1];
    return u32x4{w0, w1, w2, w3};
  };
  // A tile inside the row range of the output stores through a buffer
  // whose extent ends after the tile's last candidate row, so stores of rows
  // past it are dropped. A tile that reaches past feature D (D not a
  // multiple of the tile) tests each store.
  // `stage` is this wave's 4 KiB of free LDS. Staging layout: row r (of the
  // 32 candidates of one fn block) at r * 128 bytes, its 16-byte chunk c
  // (features 8 c .. 8 c + 7 of the wave's 64) at position c ^ (r % 8), so
  // both the writes (32 rows at one chunk) and the row-contiguous reads
  // (8 rows x 8 chunks) spread over all banks.
  auto store_tile = [&](const StreamTile& c, uint32_t stage) __attribute__((always_inline)) {
    if (c.m0 + BM <= D) {
      const auto ro = buffer_rsrc(out + c.n0 * D, (uint32_t)c.rows * (uint32_t)D * 2u);
      ROCS_LDS char* const st = lds3 + stage;
      const int rr = lane >> 3, cr = lane & 7;  // read-back: row 8 i + rr, chunk cr
      const uint32_t vo = 2u * ((uint32_t)(wn0 + rr) * (uint32_t)D + (uint32_t)(c.m0 + wm0 + 8 * cr));
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) {
#pragma unroll
        for (int fm = 0; fm < 2; ++fm)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int ch = 4 * fm + 2 * j + hh;
            *reinterpret_cast<ROCS_LDS u32x4*>(st + l32 * 128 + 16 * (ch ^ (l32 & 7))) =
                swapped(fm, fn, j);
          }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 8 * i + rr;
          const u32x4 v = *reinterpret_cast<const ROCS_LDS u32x4*>(st + r * 128 + 16 * (cr ^ (r & 7)));
          // Non-temporal (cache policy NT): the output is not read again by
          // this kernel, so it should not push the candidate slabs and the
          // weights out of L2 before the tile's other feature tiles read them.
          __builtin_amdgcn_raw_buffer_store_b128(
              v, ro, vo + 2u * (uint32_t)(32 * fn + 8 * i) * (uint32_t)D, 0, kCpolNT);
        }
      }
      return;
    }
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) {
      const int rr = wn0 + 32 * fn + l32;
#pragma unroll
      for (int fm = 0; fm < 2; ++fm)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          // The swap is wave-wide: every lane takes part, only valid ones
          // store. D is a multiple of 4: a lane's 8 features are all valid,
          // or only the first 4 (the row's last ones).
          const u32x4 v = swapped(fm, fn, j);
          const int d = c.m0 + wm0 + 32 * fm + 16 * j + 8 * hh;
          if (rr < c.rows && d < D) {
            bf16_t* p = out + (c.n0 + rr) * D + d;
            if (d + 8 <= D) *reinterpret_cast<u32x4*>(p) = v;
            else *reinterpret_cast<u32x2*>(p) = u32x2{v[0], v[1]};
          }
        }
    }
  };

  // Prologue: candidates of slabs 0 and 1, weights of slab 0, all resident.
  if (!ic_live) return;
  StreamTile cc = ic;
  plan_b();
  plan_a();
  dma_all(pb_src, pb_lim, pb_dst);
  dma_all(pa_src, pa_lim, pa_dst);
  if (ic_live) {
    plan_b();
    dma_all(pb_src, pb_lim, pb_dst);
  }
  pa_on = pb_on = false;
  if constexpr (FUSED) wait_request_side();   // while the first slabs load
  wait_vmcnt<0>();
  ring_barrier();

  // One slab. Vector-memory operations retire in issue order (the
  // counter of outstanding ones is decremented in order), and only the
  // producer waves have ring loads in flight. In an inner slab the candidate
  // loads (slab g + 2) follow the weight loads (g + 1), so waiting until only
  // those are in flight makes slab g + 1 resident. In the last slab of a
  // tile the candidates of slab g + 2 wait until after the epilogue, and the
  // Zb loads are issued and drained with the slab; the epilogue stages
  // through the candidate slot the slab has just released, once every wave
  // is done with it.
  auto step = [&](auto first_slab, auto last_slab) __attribute__((always_inline)) {
    constexpr bool kLast = decltype(last_slab)::value;
    const bool a_next = a_queued;
    if (a_next) plan_a();
    const bool b_next = ic_live;
    if (!kLast && b_next) plan_b();
    compute(first_slab, last_slab);
    pa_on = pb_on = false;
    const uint32_t released = (uint32_t)(BBASE + cbuf_b * SLAB);
    cbuf_a ^= 1;
    cbuf_b = cbuf_b == NSB - 1 ? 0 : cbuf_b + 1;
    if constexpr (kLast) {
      ring_barrier();                            // every wave is past the slab's fragments
      load_zb(cc);
      wait_vmcnt<0>();
      store_tile(cc, released + (uint32_t)wave * 4096u);
      if (b_next) {
        plan_b();
        dma_all(pb_src, pb_lim, pb_dst);
        pb_on = false;
      }
    } else {
      if (producer) {
        if (b_next) wait_vmcnt<PI>(); else wait_vmcnt<0>();
      }
    }
    if (a_next) ring_barrier();                  // a next slab exists
  };
  while (true) {
    if (nk == 1) {
      step(std::true_type(), std::true_type());
    } else {
      step(std::true_type(), std::false_type());
      for (int s = 1; s < nk - 1; ++s) step(std::false_type(), std::false_type());
      step(std::false_type(), std::true_type());
    }
    stream_next(cc, step_g, tiles_m);
    if (!stream_seek(cc, step_g, n_slots, tiles_m, off, R, N)) break;
  }
}

// ---------------------------------------------------------------------------
// General path: any dtype, any K / D, no alignment requirements.
//
// One TS x TS output tile (features x rows) per workgroup and step; its four
// waves split K and reduce through LDS in a fixed order. The products run on
// the fp32 matrix instructions (fp32 in, fp32 accumulation; bf16 inputs
// convert exactly), operands straight from global memory: lane (row l % TS,
// group l / TS) loads four consecutive k of its feature row and of its
// candidate row, and the i-th matrix instruction of a step takes the i-th
// element of both, so any k order inside a step is the same for both
// operands. Small calls are bound by latency: the split over waves keeps a
// wave's chain short and 16 x 16 tiles spread a few hundred rows over all
// CUs. At 256 rows, 384 -> 256, fp32, this form takes 4 us where one thread
// per output took 57 us in two launches.
//
// EXT (small calls): the request term is taken as k_req further columns of
// the candidate's own product, w_req and x_req[m_n] read per row, so a call
// is one launch and no request table is formed.
// ---------------------------------------------------------------------------
constexpr int64_t kExtMaxWork = int64_t(1) << 27;   // N d_out k_req up to which EXT runs

template <typename T>
struct GeneralArgs {
  const T* x;              // [N, K]
  const T* xadd;           // [N, K] or NULL
  const T* w;              // [D, K]
  const T* x2;             // EXT: x_req [R, K2]
  const T* w2;             // EXT: w_req [D, K2]
  const float* bias;       // [D] or NULL
  const float* z;          // request table [R, D] or NULL
  const int32_t* off;      // CSR offsets [R + 1], or
  const int32_t* ids;      // a request id per row (with z or EXT)
  void* out;               // [N, D] T, or float when OUTF
  int64_t N;
  int K, K2, D, R, relu, tiles_m;
  int64_t tiles;
};

template <typename T, int TS, bool VEC, bool OUTF, bool EXT>
__global__ __launch_bounds__(256) void linear_general(GeneralArgs<T> a) {
  constexpr int NG = 64 / TS;              // lane groups: k values per matrix instruction
  constexpr int CH = 4 * NG;               // k per step
  constexpr int NA = TS * TS / 64;         // accumulators per lane (4 or 16)
  typedef float acc_t __attribute__((ext_vector_type(NA)));
  __shared__ f32x4 red[NA / 4][4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l = lane % TS, g = lane / TS;
  for (int64_t t = blockIdx.x; t < a.tiles; t += gridDim.x) {
    const int d0 = (int)(t % a.tiles_m) * TS;
    const int64_t n0 = t / a.tiles_m * TS;
    const int d = d0 + l;                  // this lane's feature row of W ...
    const int64_t n = n0 + l;              // ... and its candidate
    const bool dok = d < a.D, nok = n < a.N;
    int r = 0;
    if ((EXT || a.z != nullptr) && nok)
      r = a.ids != nullptr ? (int)min((uint32_t)a.ids[n], (uint32_t)(a.R - 1))
                           : owner_of(a.off, a.R, n);
    acc_t acc;
#pragma unroll
    for (int e = 0; e < NA; ++e) acc[e] = 0.f;
    auto product = [&](const T* xp, const T* xap, const T* wp, int K) __attribute__((always_inline)) {
#pragma unroll 4
      for (int k = CH * wave + 4 * g; k < (K + CH - 1) / CH * CH; k += 4 * CH) {
        const int left = K - k;
        const f32x4 av = load4_f32<T, VEC>(wp + k, dok ? left : 0);
        f32x4 bv = load4_f32<T, VEC>(xp + k, nok ? left : 0);
        if (xap != nullptr) {              // GLM pointwise residual: round(x + x_add)
          bv += load4_f32<T, VEC>(xap + k, nok ? left : 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) bv[i] = (float)from_f32<T>(bv[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (TS == 16) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[i], acc, 0, 0, 0);
          else acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[i], acc, 0, 0, 0);
        }
      }
    };
    product(a.x + n * a.K, a.xadd != nullptr ? a.xadd + n * a.K : nullptr,
            a.w + (int64_t)d * a.K, a.K);
    if constexpr (EXT)
      product(a.x2 + (int64_t)r * a.K2, nullptr, a.w2 + (int64_t)d * a.K2, a.K2);
    // Quad q of the accumulators: features d0 + 4 NG q + 4 g .. + 3 of candidate n.
#pragma unroll
    for (int q = 0; q < NA / 4; ++q)
      red[q][wave][lane] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    __syncthreads();
    for (int q = wave; q < NA / 4; q += 4) {
      f32x4 s = ((red[q][0][lane] + red[q][1][lane]) + red[q][2][lane]) + red[q][3][lane];
      const int df = d0 + 4 * NG * q + 4 * g;
      if (!nok) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (df + i >= a.D) break;
        if (!EXT && a.z != nullptr) s[i] += a.z[(int64_t)r * a.D + df + i];
        if (a.bias != nullptr) s[i] += a.bias[df + i];
        if (a.relu) s[i] = fmaxf(s[i], 0.f);
        const int64_t o = n * a.D + df + i;
        if constexpr (OUTF) static_cast<float*>(a.out)[o] = s[i];
        else static_cast<T*>(a.out)[o] = from_f32<T>(s[i]);
      }
    }
    __syncthreads();                       // red is free for the next tile
  }
}

template <typename T, bool OUTF, bool EXT>
hipError_t launch_general(GeneralArgs<T> g, hipStream_t s) {
  // 32 x 32 tiles read half the operand bytes per product; 16 x 16 tiles while
  // the larger ones would leave CUs without a workgroup.
  const bool small = ((g.N + 31) / 32) * ((g.D + 31) / 32) < 512;
  const int ts = small ? 16 : 32;
  g.tiles_m = (g.D + ts - 1) / ts;
  g.tiles = (g.N + ts - 1) / ts * g.tiles_m;
  const uint32_t grid = (uint32_t)(g.tiles < (1 << 20) ? g.tiles : (1 << 20));
  // Four-element loads need every row of every operand aligned to them.
  auto ok = [](const void* p, int k) {
    return k % 4 == 0 && reinterpret_cast<uintptr_t>(p) % (4 * sizeof(T)) == 0;
  };
  const bool vec = ok(g.x, g.K) && ok(g.xadd, g.K) && ok(g.w, g.K) && ok(g.x2, g.K2) &&
                   ok(g.w2, g.K2);
  auto go = [&](auto kernel) { return launch_kernel(kernel, dim3(grid), dim3(256), s, g); };
  if (small)
    return vec ? go(linear_general<T, 16, true, OUTF, EXT>) : go(linear_general<T, 16, false, OUTF, EXT>);
  return vec ? go(linear_general<T, 32, true, OUTF, EXT>) : go(linear_general<T, 32, false, OUTF, EXT>);
}

template <int BM, int BN, int BK, int S, bool HAS_ADD, int WVM = 2>
hipError_t launch_tile(const LinearArgs& a, hipStream_t s) {
  const int tiles_m = (int)((a.d_out + BM - 1) / BM);
  const int64_t grid = tiles_m * ((a.N + BN - 1) / BN);
  if (!grid_fits(grid, 256)) return hipErrorInvalidConfiguration;
  return launch_kernel(ikbo_gemm_tile<BM, BN, BK, S, HAS_ADD, WVM>, dim3((uint32_t)grid), dim3(256), s,
                       static_cast<const bf16_t*>(a.x_cand),
                       static_cast<const bf16_t*>(a.x_cand_add),
                       static_cast<const bf16_t*>(a.w_cand), a.k_req > 0 ? a.z : a.bias,
                       a.k_req > 0 ? a.ids : nullptr, static_cast<bf16_t*>(a.out), a.N,
                       (int)a.k_cand, (int)a.d_out, tiles_m, (int)a.relu, (int)a.R);
}

template <typename T>
hipError_t launch_generic(const LinearArgs& a, hipStream_t s) {
  GeneralArgs<T> g{};
  g.x = static_cast<const T*>(a.x_cand);
  g.xadd = static_cast<const T*>(a.x_cand_add);
  g.w = static_cast<const T*>(a.w_cand);
  g.bias = a.bias;
  g.out = a.out;
  g.N = a.N;
  g.K = (int)a.k_cand;
  g.D = (int)a.d_out;
  g.R = (int)a.R;
  g.relu = (int)a.relu;
  if (a.k_req == 0) return launch_general<T, false, false>(g, s);
  g.off = a.cand_offsets;
  g.ids = a.ids_given ? a.ids : nullptr;
  // The request term inside the candidate product costs N / R times the
  // request table's work, the table a launch of its own (5 us and more).
  if (a.N * a.d_out <= kExtMaxWork / a.k_req) {
    g.x2 = static_cast<const T*>(a.x_req);
    g.w2 = static_cast<const T*>(a.w_req);
    g.K2 = (int)a.k_req;
    return launch_general<T, false, true>(g, s);
  }
  GeneralArgs<T> r{};
  r.x = static_cast<const T*>(a.x_req);
  r.w = static_cast<const T*>(a.w_req);
  r.out = a.z;
  r.N = a.R;
  r.K = (int)a.k_req;
  r.D = (int)a.d_out;
  const hipError_t e = launch_general<T, true, false>(r, s);
  if (e != hipSuccess) return e;
  g.z = a.z;
  return launch_general<T, false, false>(g, s);
}

}  // namespace

hipError_t launch_request_ids(const int32_t* off, int64_t R, int64_t N, int32_t* ids,
                              hipStream_t s) {
  if (!grid_fits((N + 255) / 256, 256)) return hipErrorInvalidConfiguration;
  return launch_kernel(request_ids_kernel, dim3((uint32_t)((N + 255) / 256)), dim3(256), s,
                       off, (int)R, N, ids);
}

hipError_t launch_request_table(const LinearArgs& a, hipStream_t s) {
  const int tiles_d = (int)((a.d_out + 15) / 16);
  if (!grid_fits((int64_t)tiles_d * ((a.R + 15) / 16), 256)) return hipErrorInvalidConfiguration;
  const int req_tiles = tiles_d * (int)((a.R + 15) / 16);
  const RequestOut none{nullptr, nullptr, nullptr, 0, 0, 0};
  int cus = 0;
  const hipError_t e = current_cu_count(&cus);
  if (e != hipSuccess) return e;
  return launch_request(a, cus, tiles_d, req_tiles, 0, none, s);
}

hipError_t launch_linear(const LinearArgs& a, bool fast, hipStream_t s) {
  if (!fast) {
    if (a.y_req != nullptr) {
      // Y^R on the general path: the plain linear over the R request rows.
      LinearArgs r{};
      r.x_cand = a.x_req; r.w_cand = a.w_rr; r.bias = a.b_rr;
      r.N = a.R; r.k_cand = a.k_req; r.d_out = a.d_req; r.R = 1;
      r.bf16 = a.bf16; r.relu = a.relu; r.out = a.y_req;
      const hipError_t e = a.bf16 ? launch_generic<bf16_t>(r, s) : launch_generic<float>(r, s);
      if (e != hipSuccess || a.N == 0) return e;
    }
    return a.bf16 ? launch_generic<bf16_t>(a, s) : launch_generic<float>(a, s);
  }
  // The streaming kernel needs request-aligned tiles, i.e. CSR offsets; a
  // caller's per-candidate map takes the kernel with per-row request lookup.
  // (K and D bounds: the kernel's per-lane load and store offsets within a
  // 256-row tile are 32-bit.)
  int cus = 0;
  const hipError_t ce = current_cu_count(&cus);
  if (ce != hipSuccess) return ce;
  const int64_t tiles_m256 = (a.d_out + kStreamBM - 1) / kStreamBM;
  const int64_t slots = stream_slots(a.N, a.k_req > 0 ? a.R : 0);
  const bool can_stream = !a.ids_given && a.x_cand_add == nullptr && a.k_cand % kStreamBK == 0 &&
                      a.k_cand < (int64_t(1) << 22) && a.d_out < (int64_t(1) << 22) &&
                      slots * tiles_m256 < (int64_t(1) << 31);
  // On request, the streaming kernel also runs the request side (combined
  // kernel); otherwise the request GEMM is a launch of its own. Separate
  // launches are the default on this part: the cross-XCD release / acquire
  // the combined kernel needs (an L2 write-back per request tile, an L2
  // invalidate per workgroup) costs more than the launch it saves.
  const bool fused = a.combined && can_stream && a.k_req > 0 && a.N > 0;
  const bool stream = can_stream &&
                      (fused || stream_pays(a.N, a.d_out, a.k_cand, a.k_req > 0 ? a.R : 0, cus));
  RequestOut yr{static_cast<const bf16_t*>(a.w_rr), a.b_rr, static_cast<bf16_t*>(a.y_req),
                (int)a.d_req, a.y_req != nullptr ? (int)((a.d_req + 15) / 16) : 0, (int)a.relu};
  // No candidates: only the Y^R tiles (the request table has no reader).
  const int tiles_d = a.N > 0 ? (int)((a.d_out + 15) / 16) : 0;
  if (a.k_req > 0 && !grid_fits((int64_t)(yr.tiles + tiles_d) * ((a.R + 15) / 16) +
                                    (a.N + 255) / 256, 256))
    return hipErrorInvalidConfiguration;
  const int req_tiles = (yr.tiles + tiles_d) * (int)((a.R + 15) / 16);
  if (a.k_req > 0 && !fused) {
    const hipError_t e = launch_request(a, cus, tiles_d, req_tiles,
                                        stream || a.ids_given ? 0 : a.N, yr, s);
    if (e != hipSuccess) return e;
  }
  if (a.N == 0) return hipSuccess;      // request-side output only
  if (stream) {
    const int tiles_m = (int)tiles_m256;
    const int64_t n_tiles = slots * tiles_m;
    const int grid = (int)(n_tiles < cus ? n_tiles : cus);
    const StreamStep step{grid / tiles_m, grid % tiles_m};
    const float* zb = a.k_req > 0 ? a.z : a.bias;
    const int32_t* off = a.k_req > 0 ? a.cand_offsets : nullptr;
    const bf16_t* x = static_cast<const bf16_t*>(a.x_cand);
    const bf16_t* w = static_cast<const bf16_t*>(a.w_cand);
    bf16_t* o = static_cast<bf16_t*>(a.out);
    FusedRequest fr{};
    if (fused) {
      fr.x = static_cast<const bf16_t*>(a.x_req);
      fr.w = static_cast<const bf16_t*>(a.w_req);
      fr.bias = a.bias;
      fr.z = a.z;
      fr.yr = yr;
      fr.flags = reinterpret_cast<uint64_t*>(a.ids);   // the index map's slot is free here
      fr.epoch = next_epoch();
      fr.K = (int)a.k_req;
      fr.tiles_d = tiles_d;
      fr.n_tiles = req_tiles;
    }
    auto go = [&](auto kernel) {
      return launch_kernel(kernel, dim3((uint32_t)grid), dim3(512), s, x, w, zb, off, o,
                           (int)a.R, a.N, (int)a.k_cand, (int)a.d_out, tiles_m, (int)slots, step,
                           fr);
    };
    if (fused)
      return a.relu ? go(ikbo_gemm_stream<true, true, true>) : go(ikbo_gemm_stream<true, false, true>);
    if (zb != nullptr)
      return a.relu ? go(ikbo_gemm_stream<true, true, false>) : go(ikbo_gemm_stream<true, false, false>);
    return a.relu ? go(ikbo_gemm_stream<false, true, false>) : go(ikbo_gemm_stream<false, false, false>);
  }
  // 64 x 64 tiles while 128 x 128 ones would leave CUs without a workgroup
  // (613 x 1024, K 256: 3.7 against 6.0 us; 2,000 x 1024, K 512: 10.3 / 12.9;
  // 8,192 x 512, K 2048, 256 tiles: 41.5 / 37.8).
  const bool small = ((a.d_out + 127) / 128) * ((a.N + 127) / 128) < cus;
  // Residual: four waves side by side along the candidates form each sum once,
  // two by two waves twice. Two by two / side by side, us: 200,000 x 256, K 64:
  // 27.5 / 28.6; 50,000 x 512, K 256: 32.3 / 31.1; 100,000 x 1024, K 512: 216 /
  // 205; 8,000 x 1024, K 4096: 119 / 109.
  if (a.x_cand_add != nullptr) {
    if (small) return launch_tile<64, 64, 64, 3, true>(a, s);
    return a.k_cand >= 256 ? launch_tile<128, 128, 32, 2, true, 1>(a, s)
                           : launch_tile<128, 128, 32, 2, true>(a, s);
  }
  return small ? launch_tile<64, 64, 64, 3, false>(a, s) : launch_tile<128, 128, 32, 3, false>(a, s);
}

}  // namespace rocs
