// Two stacked IKBO linear layers with the hidden layer kept on chip
// (Section 3.1, closure under composition; Eq. glm-linear for each layer;
// Section 4.1 decomposition of the first layer).
//
//   H_n   = act1(W1_CC X^C_n + Zb_{m_n})     Zb = W1_CR X^R + b1, once per request
//   Y^C_n = act2(W2 H_n + b2)
//
// Run as two launches of the linear kernel, H makes a round trip through HBM
// (written once, read once: 2 d_hidden bytes per candidate each way, four
// times the 2 k_cand + 2 d_out bytes the pair needs at the retrieval shape).
// Here a persistent workgroup (one per CU, eight waves, two per SIMD) walks
// 128-candidate tiles with the tile's X^C rows in registers and the hidden
// layer in chunks of 64 units: the chunk's 64 rows of W1_CC and 64 columns of
// W2 come through a two-slot LDS ring (DMA loads, one chunk ahead, as one
// stream across tiles since every tile needs the same weights). Per chunk
//   1. the waves, as 2 hidden blocks x 4 candidate blocks of 32, compute H^T
//      on the matrix cores on top of the Zb values of each lane's own request,
//      apply the activation and write bf16 H to LDS;
//   2. the waves, as 4 output quarters x 2 candidate halves of 64, add
//      W2 H to their accumulators.
// Chunk c's step 1 and chunk c - 1's step 2 share one barrier interval.
// What bounds it: LDS, which per chunk is read 272 KiB of fragments and
// written 64 KiB of weights (2600 cycles at 128 bytes a cycle), beside 2048
// cycles of matrix instructions a SIMD. Measured per call, request table
// included, against one wave per SIMD that kept H in its registers (as many
// LDS reads, nothing to overlap them): 64 requests, 64,324 candidates, 256 ->
// 512 -> 256: 53.5 -> 49.3 us; 9 requests, 6,025 candidates, 128 -> 960 ->
// 256: 33.4 -> 24.5 us; one request of 500: 24.7 -> 21.5 us. Four waves of 64
// candidates (a third fewer LDS reads, 400 registers) copy operands through
// the accumulation registers: 99 us. Without the DMA: 46 us.
//
// Matrix-core roles (32x32x16 bf16 MFMA): both products are computed
// transposed, hidden / output units on the M side and candidates on the N
// side, so that a lane's accumulator holds one candidate's runs of four
// consecutive units:
//   H^T[h][n]  = sum_k W1_CC[h][k] X^C[n][k]    A = W1 rows (LDS), B = X^C rows
//   Y^T[o][n] += sum_h W2[o][h] H[n][h]         A = W2 rows (LDS), B = H (LDS)
// One half-wave swap gives 16 contiguous bytes per lane of H and of the output.
//
// Tiles cover the candidates contiguously, whatever requests they belong to.
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace rocs {
namespace {

constexpr int kMlpBM = 128;          // candidates per tile
constexpr int kMlpHC = 64;           // hidden units per chunk
constexpr int kMlpMaxHidden = 1024;
constexpr int kMlpSmall = 32;        // candidates per workgroup of the small kernel

// Chunk position of 16-byte chunk c of an LDS row: c ^ swizzle(row). With
// 16 or more chunks per row the 16 rows read by a quarter-wave at one chunk
// land on 16 distinct 16-byte bank groups (the row stride is a multiple of
// 256 bytes); with 8 chunks per row (128-byte rows) two rows share a 256-byte
// bank span, so the row's low bit selects the half and (row / 2) % 8 the
// chunk.
template <int CPR>
__device__ __forceinline__ int mlp_swizzle(int row) {
  static_assert(CPR == 8 || CPR >= 16, "row width");
  if constexpr (CPR >= 16) return row & 15;
  else return (row >> 1) & 7;
}

// Four fp32 accumulator values of one lane (units u .. u + 3 of one
// candidate) with their activation (act_floor), as two packed bf16 pairs.
__device__ __forceinline__ void pack4(const f32x16& acc, int q, uint32_t lo, uint32_t& p0,
                                      uint32_t& p1) {
  p0 = act_bf16x2(pack_bf16x2(acc[4 * q], acc[4 * q + 1]), lo);
  p1 = act_bf16x2(pack_bf16x2(acc[4 * q + 2], acc[4 * q + 3]), lo);
}

// Accumulator rows 8 q + 4 hh + i (q = 2 s, 2 s + 1) of one 32-unit block,
// packed, exchanged between the wave halves: afterwards lane (l32, hh) holds
// units 16 s + 8 hh .. + 7 of its candidate, in order.
__device__ __forceinline__ u32x4 swap_halves(const uint32_t (&p)[4][2], int s) {
  const auto s0 = __builtin_amdgcn_permlane32_swap(p[2 * s][0], p[2 * s + 1][0], false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(p[2 * s][1], p[2 * s + 1][1], false, false);
  return u32x4{s0[0], s1[0], s0[1], s1[1]};
}

// Owner of candidate n (the largest r < R with off[r] <= n), with the
// offsets read through the scalar cache: the search is wave-uniform.
__device__ __forceinline__ int owner_scalar(const __attribute__((address_space(4))) int32_t* off,
                                            int R, int64_t n) {
  int lo = 0, hi = R - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((int64_t)off[mid] <= n) lo = mid; else hi = mid - 1;
  }
  return lo;
}

template <int KC, int DO>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ikbo_mlp2_bf16(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w1,
                    const float* __restrict__ zb, int64_t zb_stride,
                    const bf16_t* __restrict__ w2, const float* __restrict__ b2,
                    const int32_t* __restrict__ off_g, int R, int64_t N, int DH, int relu1,
                    int relu2, bf16_t* __restrict__ out) {
  constexpr int BM = kMlpBM, HC = kMlpHC;
  constexpr int ROWB1 = 2 * KC;                 // bytes of one W1 row
  constexpr int CPR1 = ROWB1 / 16;              // its 16-byte chunks
  constexpr int ROWB2 = 2 * HC;                 // bytes of one W2 (or H) row segment (128)
  constexpr int W1B = HC * ROWB1;               // W1 part of a ring slot
  constexpr int W2B = DO * ROWB2;               // W2 part of a ring slot
  constexpr int W2O = 2 * W1B;                  // W2 slots after the two W1 slots
  constexpr int HO = W2O + 2 * W2B;             // H of a chunk, [candidate][64], two buffers
  constexpr int HB = BM * ROWB2;
  constexpr int KS = KC / 16;                   // k-steps of the first product
  constexpr int OBW = DO / 128;                 // 32-unit output blocks per wave
  constexpr int I1 = W1B / 1024, I2 = W2B / 1024;   // wave-wide DMA loads per chunk
  static_assert(I1 % 8 == 0 && I2 % 8 == 0, "chunk loads split over eight waves");
  static_assert(HO + 2 * HB <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char lds[HO + 2 * HB];
  ROCS_LDS char* const lds3 = (ROCS_LDS char*)lds;
  // The offsets are read-only for the kernel's lifetime: scalar loads.
  const __attribute__((address_space(4))) int32_t* off =
      (const __attribute__((address_space(4))) int32_t*)off_g;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const int hb = wave & 1, cb = wave >> 1;      // first product: hidden and candidate block
  const int og = wave & 3, cg = wave >> 2;      // second: output quarter, candidate half
  const int row = 32 * cb + l32;                // this lane's candidate (first product)
  const int n_tiles = (int)((N + BM - 1) / BM);
  const uint32_t lbase = lds_addr(lds);

  // Chunk c of W1 (rows 64 c .. 64 c + 63, contiguous in memory) and of W2
  // (columns 64 c .. 64 c + 63 of every output row) into their ring slots.
  // Load i of the chunk fills 1 KiB of the slot in lane order.
  auto issue_w1 = [&](int c, int slot) __attribute__((always_inline)) {
    const char* s1 = reinterpret_cast<const char*>(w1 + (int64_t)c * HC * KC);
#pragma unroll
    for (int j = 0; j < I1 / 8; ++j) {
      const int i = wave + 8 * j, p = 64 * i + lane;
      const int r = p / CPR1, pos = p % CPR1;
      lds_dma16_sv(s1, (uint32_t)(r * ROWB1 + 16 * (pos ^ mlp_swizzle<CPR1>(r))),
                   lbase + (uint32_t)(slot * W1B) + 1024u * i);
    }
  };
  auto issue_w2 = [&](int c, int slot) __attribute__((always_inline)) {
    const char* s2 = reinterpret_cast<const char*>(w2 + (int64_t)c * HC);
#pragma unroll
    for (int j = 0; j < I2 / 8; ++j) {
      const int i = wave + 8 * j, p = 64 * i + lane;
      const int o = p >> 3, pos = p & 7;
      lds_dma16_sv(s2, (uint32_t)(o * DH * 2 + 16 * (pos ^ mlp_swizzle<8>(o))),
                   lbase + (uint32_t)(W2O + slot * W2B) + 1024u * i);
    }
  };
  // This lane's candidate rows of tile t as B fragments (row l32 of the block,
  // features 16 s + 8 hh ..); rows past the end are clamped, never stored.
  bf16x8 xf[KS];
  auto load_x = [&](int t) __attribute__((always_inline)) {
    const int64_t n = min((int64_t)t * BM + row, N - 1);
    const bf16_t* xp = x + n * KC + 8 * hh;
#pragma unroll
    for (int s = 0; s < KS; ++s) xf[s] = *reinterpret_cast<const bf16x8*>(xp + 16 * s);
  };
  // The Zb row of this lane's candidate: one scalar search per tile, then a
  // walk over the tile's request boundaries (a tile of many small requests
  // searches per lane instead).
  auto find_request = [&](int t) __attribute__((always_inline)) -> const float* {
    if (off == nullptr) return zb;
    const int64_t n0 = (int64_t)t * BM, last = min(n0 + BM, N) - 1, n = min(n0 + row, last);
    int r = owner_scalar(off, R, n0);
    int at = r, steps = 0;
    for (; at + 1 < R && (int64_t)off[at + 1] <= last && steps < 8; ++steps) {
      ++at;
      if (n >= (int64_t)off[at]) r = at;
    }
    if (steps == 8) r = owner_of(off_g, R, n);
    return zb + (int64_t)r * zb_stride;
  };
  const float* zrow;
  // The first product's accumulators start at units 64 c + 32 hb + 8 q + 4 hh
  // .. + 3 of that row. Loaded straight into them, between the packing of one
  // chunk's H and the next chunk's products, while the second product runs
  // (a second register set, loaded a whole chunk ahead, was no faster).
  f32x16 acc1;
  auto load_z = [&](int c) __attribute__((always_inline)) {
    if (zb == nullptr) {
      acc1 = f32x16{};
      return;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 z = *reinterpret_cast<const f32x4*>(zrow + HC * c + 32 * hb + 8 * q + 4 * hh);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc1[4 * q + i] = z[i];
    }
  };

  int t = (int)blockIdx.x;
  issue_w1(0, 0);
  load_x(t);
  zrow = find_request(t);
  load_z(0);
  // Make the candidate rows resident here: the compiler does not count the
  // DMA loads, so its own waits for them would include the DMA issued later.
  auto resident = [&]() __attribute__((always_inline)) {
    wait_vmcnt<0>();
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" :: "v"(as_u32x4(xf[s])));
  };
  resident();
  ring_barrier();

  // Fragment addresses: row l32 of a 32-row block, chunk 2 s + hh; the
  // swizzle turns the s step into an XOR with 32 s.
  const uint32_t fa1 = (uint32_t)((32 * hb + l32) * ROWB1 + 16 * (hh ^ mlp_swizzle<CPR1>(l32)));
  const uint32_t f2 = (uint32_t)(l32 * ROWB2 + 16 * (hh ^ mlp_swizzle<8>(l32)));
  const uint32_t fa2 = (uint32_t)(W2O + 32 * OBW * og * ROWB2) + f2;
  const uint32_t fh = (uint32_t)(HO + 64 * cg * ROWB2) + f2;
  const uint32_t lo1 = act_floor(relu1), lo2 = act_floor(relu2);
  const int nch = DH / HC;
  f32x16 acc2[OBW][2];
  // First product of the chunk in W1 slot `par`, on top of acc1; W1 fragments
  // three k-steps ahead.
  auto first = [&](int par) __attribute__((always_inline)) {
    const uint32_t sl = (uint32_t)(par * W1B);
    bf16x8 af[4];
    auto load_a = [&](int s) __attribute__((always_inline)) {
      af[s % 4] = *reinterpret_cast<const ROCS_LDS bf16x8*>(lds3 + sl + (fa1 ^ (32u * s)));
    };
    load_a(0);
    load_a(1);
    load_a(2);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s + 3 < KS) load_a(s + 3);
      __builtin_amdgcn_sched_barrier(0);
      acc1 = mfma32(af[s % 4], xf[s], acc1);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Activation, bf16, into H buffer `par`.
  auto put_h = [&](int par) __attribute__((always_inline)) {
    uint32_t p[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q) pack4(acc1, q, lo1, p[q][0], p[q][1]);
#pragma unroll
    for (int s = 0; s < 2; ++s)
      *reinterpret_cast<ROCS_LDS u32x4*>(
          lds3 + HO + par * HB + row * ROWB2 + 16 * ((4 * hb + 2 * s + hh) ^ mlp_swizzle<8>(row))) =
          swap_halves(p, s);
  };
  // Second product of the chunk in W2 slot and H buffer `par`.
  bf16x8 wf[2][OBW], hf[2][2];
  auto load_2 = [&](int par, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int ob = 0; ob < OBW; ++ob)
      wf[s & 1][ob] = *reinterpret_cast<const ROCS_LDS bf16x8*>(
          lds3 + par * W2B + 32 * ob * ROWB2 + (fa2 ^ (32u * s)));
#pragma unroll
    for (int j = 0; j < 2; ++j)
      hf[s & 1][j] = *reinterpret_cast<const ROCS_LDS bf16x8*>(
          lds3 + par * HB + 32 * j * ROWB2 + (fh ^ (32u * s)));
  };
  auto second = [&](int par) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (s + 1 < 4) load_2(par, s + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ob = 0; ob < OBW; ++ob)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc2[ob][j] = mfma32(wf[s & 1][ob], hf[s & 1][j], acc2[ob][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int par = 0;                   // ring slot and H buffer of the chunk in the first product
  while (true) {
    const int tn = t + (int)gridDim.x;
    const bool live = tn < n_tiles;
    // Chunk 0: its first product alone. W1 of the next chunk and W2 of this
    // one load meanwhile.
    issue_w2(0, par);
    if (nch > 1 || live) issue_w1(nch > 1 ? 1 : 0, par ^ 1);
#pragma unroll
    for (int ob = 0; ob < OBW; ++ob)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4 b = {0.f, 0.f, 0.f, 0.f};
        if (b2 != nullptr)
          b = *reinterpret_cast<const f32x4*>(b2 + 32 * (OBW * og + ob) + 8 * q + 4 * hh);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc2[ob][0][4 * q + i] = acc2[ob][1][4 * q + i] = b[i];
      }
    const float* znext = live ? find_request(tn) : zb;   // in this light interval
    first(par);
    put_h(par);
    if (nch > 1) load_z(1);
    wait_lgkmcnt0();
    wait_vmcnt<0>();
    ring_barrier();
    par ^= 1;
    // Chunk c's first product with chunk c - 1's second: one barrier a chunk.
    for (int c = 1; c < nch; ++c) {
      const bool last = c + 1 == nch;
      issue_w2(c, par);
      if (!last || live) issue_w1(last ? 0 : c + 1, par ^ 1);
      first(par);
      load_2(par ^ 1, 0);
      put_h(par);
      if (!last) load_z(c + 1);
      second(par ^ 1);
      wait_lgkmcnt0();
      wait_vmcnt<0>();          // the next chunk's W1, this one's W2, the next Zb values
      ring_barrier();           // every wave's loads in, H complete, the other slots free
      par ^= 1;
    }
    // The last chunk's second product; the next tile's rows load meanwhile
    // (the candidate registers are free).
    if (live) {
      load_x(tn);
      zrow = znext;
      load_z(0);
    }
    load_2(par ^ 1, 0);
    second(par ^ 1);

    // Epilogue: activation, bf16; after the swaps four lanes store 64
    // contiguous bytes of one candidate.
    const int l16 = lane & 15, q4 = lane >> 4;
    const int64_t n0 = (int64_t)t * BM + 64 * cg + l16;
    bf16_t* op = out + n0 * DO + 32 * OBW * og + 16 * (q4 & 1) + 8 * hh;
#pragma unroll
    for (int ob = 0; ob < OBW; ++ob)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t p[4][2];
#pragma unroll
        for (int q = 0; q < 4; ++q) pack4(acc2[ob][j], q, lo2, p[q][0], p[q][1]);
        const u32x4 s0 = swap_halves(p, 0), s1 = swap_halves(p, 1);
        u32x4 o[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto w = __builtin_amdgcn_permlane16_swap(s0[e], s1[e], false, false);
          o[0][e] = w[0];
          o[1][e] = w[1];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (n0 + 32 * j + 16 * i < N)
            *reinterpret_cast<u32x4*>(op + (int64_t)(32 * j + 16 * i) * DO + 32 * ob) = o[i];
      }
    if (!live) break;
    resident();
    ring_barrier();             // every wave is past the last chunk's W2 and H
    t = tn;
  }
}

// Few candidates: the persistent kernel's 128-candidate tiles would leave most
// CUs idle, each walking the chunks behind a barrier. Here a workgroup (eight
// waves) takes 32 candidates and the whole hidden layer at once:
//   1. wave w forms the 32-unit blocks w, w + 8, .. of H^T, X^C rows in
//      registers, and writes them to LDS as bf16;
//   2. after one barrier, wave w adds a 32-unit output block over all of H;
//      with 128 outputs the two wave quartets split H and add up in LDS.
// Each wave streams its weights through a private two-slot LDS ring of DMA
// units (32 rows x 64 columns), one stream over both products. Bound by the
// latency and the L2 reads of the weights. One request of 500 candidates, 256
// -> 512 -> 256, request table included: 11.3 us (persistent kernel 21.6; the
// weights loaded straight into registers, 32 lines touched per load: 29.5).
template <int KC, int DO>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void ikbo_mlp2_small(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w1,
                     const float* __restrict__ zb, int64_t zb_stride,
                     const bf16_t* __restrict__ w2, const float* __restrict__ b2,
                     const int32_t* __restrict__ off, int R, int64_t N, int DH, int relu1,
                     int relu2, bf16_t* __restrict__ out) {
  constexpr int KS = KC / 16, JU = KC / 64, SPLIT = 256 / DO;
  constexpr int ROWX = 2 * KC, CPRX = ROWX / 16;
  constexpr int UB = 32 * 128;                    // bytes of a unit
  // H rows are 16 bytes longer than the hidden layer: the rows that a
  // quarter-wave reads at one chunk start in distinct 16-byte bank groups.
  constexpr int HB = kMlpSmall * (2 * kMlpMaxHidden + 16);
  static_assert(HB % 1024 == 512 && HB >= kMlpSmall * ROWX && HB >= 16 * 1024, "LDS plan");
  constexpr int RO = HB + 512;                    // the rings, 1 KiB aligned
  __shared__ __attribute__((aligned(1024))) char lds[RO + 8 * 2 * UB];
  const uint32_t lbase = lds_addr(lds);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const int64_t n0 = (int64_t)blockIdx.x * kMlpSmall, n_at = n0 + l32;
  const int64_t n = min(n_at, N - 1);             // rows past the end are never stored
  const int stride = 2 * DH + 16;
  const int blocks = DH / 32;
  const int ob = SPLIT == 1 ? wave : wave & 3, half = SPLIT == 1 ? 0 : wave >> 2;

  // The wave's units: its hidden blocks' JU each, then its 64-column units of W2.
  const int n1 = wave < blocks ? (blocks - wave + 7) / 8 * JU : 0;
  const int first2 = half == 0 ? 0 : (DH / 64 + 1) / 2;
  const int last2 = SPLIT == 2 && half == 0 ? (DH / 64 + 1) / 2 : DH / 64;
  const int units = n1 + last2 - first2;
  const uint32_t ring = (uint32_t)(RO + wave * 2 * UB);
  auto issue = [&](int u) __attribute__((always_inline)) {
    const bool one = u < n1;
    const bf16_t* rows = one ? w1 + (int64_t)32 * (wave + 8 * (u / JU)) * KC
                             : w2 + (int64_t)32 * ob * DH;
    const int col = one ? u % JU : first2 + u - n1;
    const uint32_t rowb = one ? 2 * KC : 2 * DH;
    const char* base = uniform_ptr(reinterpret_cast<const char*>(rows + 64 * col));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 8 * i + (lane >> 3);
      lds_dma16_sv(base, (uint32_t)r * rowb + 16u * ((lane & 7) ^ mlp_swizzle<8>(r)),
                   lbase + ring + (uint32_t)((u & 1) * UB) + 1024u * i);
    }
  };
  // X^C rows through H's place, while the first units are on the way.
#pragma unroll
  for (int i = wave; i < kMlpSmall * ROWX / 1024; i += 8) {
    const int p = 64 * i + lane, r = p / CPRX, pos = p % CPRX;
    lds_dma16_sv(uniform_ptr(reinterpret_cast<const char*>(x + n0 * KC)),
                 (uint32_t)((int)(min(n0 + r, N - 1) - n0) * ROWX + 16 * (pos ^ mlp_swizzle<CPRX>(r))),
                 lbase + 1024u * i);
  }
  if (units > 0) issue(0);
  if (units > 1) issue(1);
  const float* zrow = zb;
  if (off != nullptr) zrow = zb + (int64_t)owner_of(off, R, n) * zb_stride;
  wait_vmcnt<0>();
  __syncthreads();
  bf16x8 xf[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k)
    xf[k] = *reinterpret_cast<const bf16x8*>(
        lds + l32 * ROWX + 16 * ((2 * k + hh) ^ mlp_swizzle<CPRX>(l32)));
  __syncthreads();                                // H's place is free

  // Unit u's fragments; the next unit stays in flight, the one after starts.
  bf16x8 wf[4];
  auto take = [&](int u) __attribute__((always_inline)) {
    if (u + 1 < units) wait_vmcnt<4>(); else wait_vmcnt<0>();
    asm volatile("" ::: "memory");                // no read above the wait
    const char* slot = lds + ring + (u & 1) * UB + l32 * 128;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      wf[k] = *reinterpret_cast<const bf16x8*>(slot + 16 * ((2 * k + hh) ^ mlp_swizzle<8>(l32)));
    asm volatile("" ::: "memory");                // no read below the next one
    wait_lgkmcnt0();                              // the slot has been read
    asm volatile("" ::: "memory");
    if (u + 2 < units) issue(u + 2);
  };

  const uint32_t lo1 = act_floor(relu1);
  int u = 0;
  for (int hb = wave; hb < blocks; hb += 8) {
    f32x16 acc = f32x16{};
    if (zb != nullptr) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 z = *reinterpret_cast<const f32x4*>(zrow + 32 * hb + 8 * q + 4 * hh);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[4 * q + i] = z[i];
      }
    }
#pragma unroll
    for (int j = 0; j < JU; ++j, ++u) {
      take(u);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc = mfma32(wf[k], xf[4 * j + k], acc);
    }
    uint32_t p[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q) pack4(acc, q, lo1, p[q][0], p[q][1]);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      *reinterpret_cast<u32x4*>(lds + l32 * stride + 2 * (32 * hb + 16 * j + 8 * hh)) =
          swap_halves(p, j);
  }

  f32x16 acc = f32x16{};
  if (b2 != nullptr && half == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(b2 + 32 * ob + 8 * q + 4 * hh);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[4 * q + i] = b[i];
    }
  }
  __syncthreads();                                // H is whole
  for (int c = first2; c < last2; ++c, ++u) {
    bf16x8 hf[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      hf[k] = *reinterpret_cast<const bf16x8*>(lds + l32 * stride + 128 * c + 32 * k + 16 * hh);
    take(u);
#pragma unroll
    for (int k = 0; k < 4; ++k) acc = mfma32(wf[k], hf[k], acc);
  }
  if constexpr (SPLIT == 2) {
    __syncthreads();                              // H has been read: its place is free
    // 64 lanes x 64 bytes a wave, 16 KiB in all; the shortest H takes 4.5 KiB
    // of the same array, whose size does not depend on it.
    f32x4* part = reinterpret_cast<f32x4*>(lds) + ob * 256;
    if (half == 1) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        part[64 * q + lane] = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    }
    __syncthreads();
    if (half == 1) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 v = part[64 * q + lane];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[4 * q + i] += v[i];
    }
  }
  const uint32_t lo2 = act_floor(relu2);
  uint32_t p[4][2];
#pragma unroll
  for (int q = 0; q < 4; ++q) pack4(acc, q, lo2, p[q][0], p[q][1]);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const u32x4 v = swap_halves(p, j);            // every lane takes part in the swap
    if (n_at < N)
      *reinterpret_cast<u32x4*>(out + n_at * DO + 32 * ob + 16 * j + 8 * hh) = v;
  }
}

template <int KC, int DO>
hipError_t launch_fused(const Mlp2Args& a, const float* zb, int64_t zb_stride,
                        const int32_t* off, hipStream_t s) {
  int cus = 0;
  const hipError_t e = current_cu_count(&cus);
  if (e != hipSuccess) return e;
  // Up to two rounds of 32-candidate workgroups (one fits a CU) beat the
  // persistent kernel's weight stream through barriers. Persistent / small, us:
  // 8,000 candidates, 256 -> 512 -> 256: 22.4 / 12.8, 128 -> 960 -> 256: 25.8 /
  // 16.0; 12,000: 23.9 / 21.0, 27.0 / 26.9; 16,384: 25.0 / 22.5, 28.6 / 28.3.
  // A round adds about 10 us, the persistent kernel's step to 24,000 0.3.
  if (a.N <= (int64_t)2 * kMlpSmall * cus) {
    return launch_kernel(ikbo_mlp2_small<KC, DO>, dim3((uint32_t)((a.N + kMlpSmall - 1) / kMlpSmall)),
                         dim3(512), s, static_cast<const bf16_t*>(a.x_cand),
                         static_cast<const bf16_t*>(a.w1_cand), zb, zb_stride,
                         static_cast<const bf16_t*>(a.w2), a.b2, off, (int)a.R, a.N,
                         (int)a.d_hidden, (int)a.relu1, (int)a.relu2,
                         static_cast<bf16_t*>(a.out));
  }
  const int64_t tiles = (a.N + kMlpBM - 1) / kMlpBM;
  const int grid = (int)(tiles < cus ? tiles : cus);
  return launch_kernel(ikbo_mlp2_bf16<KC, DO>, dim3((uint32_t)grid), dim3(512), s,
                       static_cast<const bf16_t*>(a.x_cand),
                       static_cast<const bf16_t*>(a.w1_cand), zb, zb_stride,
                       static_cast<const bf16_t*>(a.w2), a.b2, off, (int)a.R, a.N,
                       (int)a.d_hidden, (int)a.relu1, (int)a.relu2,
                       static_cast<bf16_t*>(a.out));
}

}  // namespace

bool mlp2_fused_shape(int64_t R, int64_t k_cand, int64_t d_hidden, int64_t d_out) {
  // Request tables of 4 GiB and more take the two-launch form.
  return (k_cand == 128 || k_cand == 256) && (d_out == 128 || d_out == 256) &&
         d_hidden >= kMlpHC && d_hidden % kMlpHC == 0 && d_hidden <= kMlpMaxHidden &&
         R * d_hidden * 4 < (int64_t(1) << 32);
}

hipError_t launch_mlp2(const Mlp2Args& a, bool fused, hipStream_t s) {
  if (a.N == 0) return hipSuccess;
  LinearArgs l1{};
  l1.x_req = a.x_req; l1.x_cand = a.x_cand; l1.w_req = a.w1_req; l1.w_cand = a.w1_cand;
  l1.bias = a.b1; l1.cand_offsets = a.cand_offsets;
  l1.R = a.R; l1.N = a.N; l1.k_req = a.k_req; l1.k_cand = a.k_cand; l1.d_out = a.d_hidden;
  l1.bf16 = a.bf16; l1.relu = a.relu1; l1.z = a.z; l1.ids = a.ids;
  if (fused) {
    // The request table Zb = X^R W1_CR^T + b1 at batch size R, then the
    // fused candidate kernel.
    const float* zb = a.b1;
    int64_t stride = 0;
    const int32_t* off = nullptr;
    if (a.k_req > 0) {
      const hipError_t e = launch_request_table(l1, s);
      if (e != hipSuccess) return e;
      zb = a.z;
      stride = a.d_hidden;
      off = a.cand_offsets;
    }
    if (a.k_cand == 256)
      return a.d_out == 256 ? launch_fused<256, 256>(a, zb, stride, off, s)
                            : launch_fused<256, 128>(a, zb, stride, off, s);
    return a.d_out == 256 ? launch_fused<128, 256>(a, zb, stride, off, s)
                          : launch_fused<128, 128>(a, zb, stride, off, s);
  }
  // Two launches of the linear kernel, H through the workspace.
  l1.out = a.h;
  hipError_t e = launch_linear(l1, a.linear_fast, s);
  if (e != hipSuccess) return e;
  LinearArgs l2{};
  l2.x_cand = a.h; l2.w_cand = a.w2; l2.bias = a.b2;
  l2.R = 1; l2.N = a.N; l2.k_cand = a.d_hidden; l2.d_out = a.d_out;
  l2.bf16 = a.bf16; l2.relu = a.relu2; l2.out = a.out;
  return launch_linear(l2, a.linear_fast, s);
}

}  // namespace rocs
