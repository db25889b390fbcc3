// IKBO Deep Cross Attention (Section 3.2, Eq. dca-attention; Section 4.3).
//
// Candidate n of request r = m_n attends over r's history rows
// kv_offsets[r] .. kv_offsets[r+1]-1 of the request-batched K/V. IKBO form
// (Section 4.3.1): a workgroup owns one (head, request, tile of that
// request's query rows) and streams the request's K/V through LDS once; every
// candidate row in the tile reuses it, so K/V are read once per request tile
// instead of once per candidate, and no candidate-batched copy exists.
//
// Stacking candidates: with few query tokens per candidate (one, in the
// retrieval and ranking workloads) a tile of 128 or 256 query rows holds that
// many / T_q candidates of the same request, which fills the matrix cores the way one
// long query sequence would (the paper co-processes 2-4 candidates per CTA for
// the same reason, Section 4.3.2).
//
// Work order (the paper's grid reorder for L2 locality, Section 4.3.1, done
// the MI355X way): workgroup ids are renumbered so that consecutive ones run
// on the same XCD, and the work list is ordered (head, request, tile), so the
// tiles of one (request, head) run together on one XCD and share its L2.
#include "common.h"
#include "kernels.h"
#include "launch.h"

#include <type_traits>

namespace rocs {
namespace {

constexpr int kTileKeys = 64;    // history rows per K/V stage
constexpr int kGroupMaxRequests = 16384;            // LDS counters of the grouping kernels
constexpr int64_t kGroupMaxHist = int64_t(1) << 20;  // per-block counts scanned by one workgroup

size_t align_up256(size_t n) { return (n + 255) & ~size_t(255); }
// Online softmax bound. A stage's weights, taken against the running max as
// it stands, are accepted as they are while their per-lane sum is at most
// 2^64. Otherwise the stage takes its row max, and the running max moves to
// it only if it lies more than kLazyRescale above the running max; either
// way every accepted weight is then at most 2^64 (it may sit just under the
// bound on all 32 keys of a lane, so an accepted per-lane stage sum is at
// most 32 * 2^64). Row sums therefore stay below L * 2^64 and outputs below
// L * 2^64 * max|v|: finite in fp32 (and in bf16, which has fp32's exponent
// range) for any history shorter than 2^60 rows.
constexpr float kLazyRescale = 64.0f;     // log2 of the largest unnormalised weight
constexpr float kWeightBound = 0x1p64f;   // per-lane stage sum accepted without a row max

// Eight packed bf16 pairs added elementwise in fp32 and rounded back (RNE).
__device__ __forceinline__ u32x4 add_bf16x8(u32x4 a, u32x4 b) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = __builtin_bit_cast(float, a[i] << 16) + __builtin_bit_cast(float, b[i] << 16);
    const float hi = __builtin_bit_cast(float, a[i] & 0xffff0000u) +
                     __builtin_bit_cast(float, b[i] & 0xffff0000u);
    r[i] = pack_bf16x2(lo, hi);
  }
  return r;
}

// ---------------------------------------------------------------------------
// bf16 MFMA kernel (32x32x16 shape), head_dim D in {64, 128}.
//
// Workgroup: 4 waves x 32 query rows = one 128-row tile. With 32 rows a wave
// needs under 256 VGPRs (under 168 at head_dim 64), and each workgroup's K/V
// staging fits in 64 KiB of LDS (32 KiB at head_dim 64), so two workgroups
// share a CU (three at head_dim 64): each SIMD runs one wave of each. The two
// waves are not held in step by a common barrier, so one's softmax (VALU)
// overlaps the other's matrix-core work, and one workgroup's prologue (request
// lookup, query and first K/V loads) and epilogue run while the other is in
// its main loop. (A 256-row workgroup of 8 waves, one per CU, reuses each K/V
// stage for twice the rows but leaves those fixed costs exposed: 4% slower at
// a history of 2048.)
//
// Scores are computed transposed, S^T = K Q^T (A = K rows from LDS, B = the
// wave's query rows held in registers for the whole history), so each lane's
// accumulator holds 16 keys of one query row: the row max needs only one
// exchange between the two wave halves. O^T = V^T P^T reuses the
// probabilities straight from registers as the B operand (the order of the
// 16 keys inside one MFMA step is a fixed permutation applied to both P and
// V^T).
//
// K/V staging: history rows go from HBM/L2 straight into LDS with the DMA
// form of the global load (no VGPR round trip, no LDS store instructions),
// ahead of use through two 2-slot rings in LDS, one for K and one for V (K of
// stage t + 2 and V of stage t + 1 load while stage t is processed). Rows keep
// their HBM layout in
// LDS, with the 16-byte chunks of each row XOR-swizzled by the row index so
// that both fragment reads are conflict-free; V^T fragments come out of the
// row-major V stage through the transposing LDS read (ds_read_b64_tr_b16).
//
// Online softmax in the exp2 domain, scale * log2(e) folded into one FMA.
// Weights are taken against the running max as it stands; the max (and the
// accumulator rescale) is only computed when a stage's weights could pass
// 2^kLazyRescale, which the per-lane sum of the weights detects, so after the
// first stage almost no stage needs a row max (the final division by the row
// sum is exact in the algebra). Row sums are accumulated per wave half from
// the bf16-rounded weights the PV product uses, and combined at the end.
//
// Loads never branch: history and query row indices are clamped into range,
// and the keys past the history's end are masked (weight 0) in the last,
// ragged stage only.
// ---------------------------------------------------------------------------
template <int D> constexpr int attn_waves() { return 4; }  // query rows / 32 per workgroup
// Slots per K (and per V) ring: 4 stages in LDS, 64 KiB at head_dim 128, so
// two workgroups share a CU; 32 KiB at head_dim 64, where three workgroups
// share a CU (each wave within 168 registers). (At head_dim 64 a single
// 4-slot ring holding K and V of a stage together, loaded three stages
// ahead, measured 5% slower on ranking-sized histories; three-slot K and V
// rings loaded two steps ahead need runtime slot offsets, spill at 168
// registers and ran 1.5x slower.)
constexpr int kRingSlots = 2;

// MAPPED: the candidates arrive grouped by request through a permutation
// (Section 4.3.1 with a general map m): cand_off are the offsets of the
// grouped order and grouped position p holds candidate order[p], so query
// rows are gathered and output rows scattered through `order`; everything
// else is the CSR kernel.
// QPROJ: the queries are projected in the prologue (Q = round(X W_q^T), see
// below) instead of read: `q` is then X [N, T_q, kProjIn] and `wq` is W_q
// [H D, kProjIn].
constexpr int kProjIn = 256;   // input width of the fused query projection

// Tile plan (launch_attention_plan): an int32 array. Header: mode (1 =
// sorted, 0 = use the built-in order), T (tiles over all heads), R, H, T_q,
// rows per tile; then from kPlanHeader the request ids sorted by history
// length, longest first (lengths from 2^20 - 1 on count as equal; ties by
// id), and their tile offsets P[0..R]
// (P[i+1] - P[i] = H * ceil(n_r T_q / rows per tile) for the i-th request r;
// all heads of one request are consecutive, each head's tiles in order).
// Workgroup b takes tile t of that list, in chunks of kPlanChunk consecutive
// tiles per XCD: t = ((b / 8) / C * 8 + b % 8) C + (b / 8) % C, so the chunks
// of the longest histories are spread over all XCDs first and a chunk (a
// request's tiles, sharing its K/V) stays on one L2.
constexpr int kPlanHeader = 8;
constexpr int kPlanChunk = 16;
constexpr int kAttnTileRows = 128;   // query rows per tile (4 waves x 32) at head_dim 64 and 128

// Largest g in [0, n) with P[g] <= t, given P[0] <= t and P non-decreasing;
// wave-parallel like request_of_slot. Call with every lane of the wave active.
__device__ __forceinline__ int plan_group_of(const int32_t* __restrict__ P, int n, int64_t t) {
  const int lane = (int)(threadIdx.x & 63);
  int lo = 0;
  while (n > 1) {
    const int step = (n + 63) / 64;
    const int g = lo + lane * step;
    const bool ok = g < lo + n && (int64_t)P[g] <= t;
    const uint64_t m = __ballot(ok);
    const int k = 63 - __builtin_clzll(m);
    lo += k * step;
    n = min(step, n - k * step);
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

template <int D, int W, bool MAPPED, bool QPROJ>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2))) void dca_attn_bf16(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const int32_t* __restrict__ cand_off, const int32_t* __restrict__ kv_off,
    bf16_t* __restrict__ out, int R, int Tq, int H, int64_t kv_stride, float scale_log2,
    int64_t slots_per_head, const int32_t* __restrict__ order, const bf16_t* __restrict__ res,
    bf16_t* __restrict__ out_sum, const bf16_t* __restrict__ wq,
    const int32_t* __restrict__ plan) {
  constexpr int NT = 64 * W;
  constexpr int TR = 32 * W;           // query rows per tile
  static_assert(TR == kAttnTileRows, "the tile plan assumes 128-row tiles");
  constexpr int KB = kTileKeys / 32;   // 32-key blocks per stage
  constexpr int KS = D / 16;           // MFMA steps over head_dim
  constexpr int DB = D / 32;           // 32-wide output column blocks
  constexpr int PS = kTileKeys / 16;   // MFMA steps over the stage's keys
  constexpr int ROWB = 2 * D;          // bytes of one history row of one head
  constexpr int CR = D / 8;            // 16-byte chunks per row
  constexpr int STAGE = kTileKeys * ROWB;             // bytes of one K (or V) stage
  constexpr int KPI = 1024 / ROWB;                    // rows per wave-wide DMA load
  constexpr int NI = kTileKeys / (KPI * W);           // DMA loads per wave, operand, stage
  static_assert(NI >= 1 && kTileKeys % (KPI * W) == 0, "staging does not tile");
  static_assert(CR * 16 == ROWB, "layout");
  constexpr int kStages = kRingSlots;
  static_assert(kStages * STAGE <= 65536, "LDS offsets must fit the 16-bit immediate");
  __shared__ __attribute__((aligned(1024))) char lds[2 * kStages * STAGE];  // K ring, V ring
  ROCS_LDS char* const lds3 = (ROCS_LDS char*)lds;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  // This workgroup's (head, request, tile of the request): from the
  // caller's plan when it matches this launch, else the built-in order
  // (head-major slots R + ceil(N T_q / TR) per head, XCD-remapped). The
  // planned grid is rounded up to whole chunk rounds; surplus workgroups
  // exit. A plan never moves an access out of range: its request ids are
  // clamped and a tile past its request's rows is idle.
  int h, r;
  int64_t j;
  const uint32_t b = blockIdx.x;
  const int64_t n_work = slots_per_head * H;
  if (plan != nullptr && plan[0] == 1 && plan[2] == R && plan[3] == H && plan[4] == Tq &&
      plan[5] == TR) {
    const uint32_t xi = b / kNumXcd;
    const int64_t t = ((int64_t)(xi / kPlanChunk) * kNumXcd + b % kNumXcd) * kPlanChunk +
                      xi % kPlanChunk;
    if (t >= plan[1]) return;
    const int32_t* P = plan + kPlanHeader + R;
    const int g = plan_group_of(P, R, t);
    r = (int)min((uint32_t)plan[kPlanHeader + g], (uint32_t)(R - 1));
    const int p0 = P[g];
    const int per_head = (P[g + 1] - p0) / H;
    if (per_head < 1) return;
    const int off = (int)(t - p0);
    h = off / per_head;
    j = off - (int64_t)h * per_head;
    if (h >= H) return;
  } else {
    if ((int64_t)b >= n_work) return;
    const uint32_t work = xcd_remap(b, (uint32_t)n_work);
    h = (int)(work / (uint64_t)slots_per_head);
    const int64_t slot = (int64_t)(work % (uint64_t)slots_per_head);
    r = request_of_slot(cand_off, R, slot, Tq, TR);
    j = slot - tile_base(cand_off, r, Tq, TR);
  }
  const int64_t rend = (int64_t)cand_off[r + 1] * Tq;
  const int64_t row0 = (int64_t)cand_off[r] * Tq + j * TR;
  if (row0 >= rend) return;                               // idle slot
  const int rows = (int)(rend - row0 < TR ? rend - row0 : TR);
  const int64_t kv0 = kv_off[r];
  const int L = kv_off[r + 1] - (int)kv0;
  const int64_t qs = (int64_t)H * D;                      // q / out row stride
  // Query / output row of the tile's row i (i < rows): row0 + i directly,
  // or through the grouped order (grouped candidate p = row / T_q holds
  // candidate order[p]).
  auto src_row = [&](int i) -> int64_t {
    const int64_t gr = row0 + i;
    if constexpr (MAPPED) {
      const int64_t p = gr / Tq;
      return (int64_t)order[p] * Tq + (gr - p * Tq);
    } else {
      return gr;
    }
  };
  const bf16_t* qh = q + (int64_t)h * D;

  if (L == 0) {                                  // empty history: zeros (and out_sum = res)
    for (int c = tid; c < rows * (D / 8); c += NT) {
      const int rr = c / (D / 8), dc = (c % (D / 8)) * 8;
      const int64_t o = src_row(rr) * qs + (int64_t)h * D + dc;
      *reinterpret_cast<u32x4*>(out + o) = u32x4{0u, 0u, 0u, 0u};
      if (res != nullptr)
        *reinterpret_cast<u32x4*>(out_sum + o) = *reinterpret_cast<const u32x4*>(res + o);
    }
    return;
  }

  // This wave's 32 query rows as B fragments: lane holds Q[row l32][16 ks + 8 hh .. +7].
  const int wrow0 = wave * 32;
  const bool active = wrow0 < rows;
  const int qrow = min(wrow0 + l32, rows - 1);            // clamped; extra rows never stored
  bf16x8 qf[KS];
  if constexpr (!QPROJ) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks] = *reinterpret_cast<const bf16x8*>(qh + src_row(qrow) * qs + 16 * ks + 8 * hh);
  } else {
    // The query projection of this head, fused (the candidate side of the
    // DCA query generator): Q^T = W_q,h X^T on the matrix cores, with the
    // same operand roles and k order as the streaming GEMM, so Q is
    // bit-identical to projecting first. W_q,h (D rows of 512 bytes) is
    // staged in the K/V ring before the ring's first stage; chunk c of row
    // d sits at position c ^ (d % 16), so the 16 rows read by a quarter-wave
    // fall on distinct banks. This wave's 32 rows of X are B fragments.
    static_assert(D == 64 && 2 * kStages * STAGE >= D * kProjIn * 2, "projection staging");
    constexpr int PK = kProjIn / 16;                      // k-steps (16)
    constexpr int PRB = kProjIn * 2;                      // bytes of one W_q row (512)
    constexpr int PNI = D * PRB / 1024 / W;               // DMA loads per wave (8)
    const char* wsrc = reinterpret_cast<const char*>(wq + (int64_t)h * D * kProjIn);
    const uint32_t lb = lds_addr(lds);
#pragma unroll
    for (int i = 0; i < PNI; ++i) {
      const int blk = wave * PNI + i;                     // 1 KiB: rows 2 blk, 2 blk + 1
      const int prow = 2 * blk + (lane >> 5), pos = lane & 31;
      lds_dma16_sv(wsrc, (uint32_t)(prow * PRB + 16 * (pos ^ (prow & 15))), lb + 1024u * blk);
    }
    const bf16_t* xr = q + src_row(qrow) * kProjIn + 8 * hh;
    bf16x8 xq[PK];
#pragma unroll
    for (int s2 = 0; s2 < PK; ++s2) xq[s2] = *reinterpret_cast<const bf16x8*>(xr + 16 * s2);
    wait_vmcnt<0>();
    ring_barrier();
    f32x16 pacc[2];
#pragma unroll
    for (int s2 = 0; s2 < PK; ++s2)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int prow = 32 * b + l32;
        const bf16x8 a = *reinterpret_cast<const ROCS_LDS bf16x8*>(
            lds3 + prow * PRB + 16 * ((2 * s2 + hh) ^ (prow & 15)));
        if (s2 == 0) {
          const f32x16 zero = {};
          pacc[b] = mfma32(a, xq[0], zero);
        } else {
          pacc[b] = mfma32(a, xq[s2], pacc[b]);
        }
      }
    // Round to bf16 and exchange halves: lane (l32, hh) then holds dims
    // 32 b + 16 jj + 8 hh .. + 7 of its row, i.e. qf[2 b + jj].
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const f32x16& pa = pacc[b];
        const uint32_t e0 = pack_bf16x2(pa[8 * jj], pa[8 * jj + 1]);
        const uint32_t e1 = pack_bf16x2(pa[8 * jj + 2], pa[8 * jj + 3]);
        const uint32_t o0 = pack_bf16x2(pa[8 * jj + 4], pa[8 * jj + 5]);
        const uint32_t o1 = pack_bf16x2(pa[8 * jj + 6], pa[8 * jj + 7]);
        const auto t0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
        const auto t1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
        qf[2 * b + jj] = as_bf16x8(u32x4{t0[0], t1[0], t0[1], t1[1]});
      }
    ring_barrier();                                       // W_q's LDS goes to the K/V ring
  }

  // DMA staging. Load i of wave w fills LDS rows KPI (NI w + i) .. +KPI-1 of
  // the stage, 16 bytes per lane in lane order: lane -> row KPI (NI w + i) +
  // lane / CR, chunk position lane % CR, so the lane fetches chunk
  // (lane % CR) ^ kv_swizzle(row) of that history row.
  const char* kbase = reinterpret_cast<const char*>(k + kv0 * kv_stride + (int64_t)h * D);
  const char* vbase = reinterpret_cast<const char*>(v + kv0 * kv_stride + (int64_t)h * D);
  const int64_t rowstride = kv_stride * 2;                // bytes
  int skey[NI];
  uint32_t schunk[NI], soff[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    skey[i] = KPI * (NI * wave + i) + lane / CR;
    schunk[i] = 16u * (uint32_t)((lane % CR) ^ kv_swizzle<D>(skey[i]));
    soff[i] = (uint32_t)(skey[i] * rowstride) + schunk[i];
  }
  const uint32_t lds_base = lds_addr(lds);
  // Stage t of one operand (K: ring 0, V: ring 1) into slot t % kStages.
  auto issue_op = [&](int t, int ring) {
    const int base = t * kTileKeys;
    const char* src = ring == 0 ? kbase : vbase;
    const uint32_t dst = lds_base + (uint32_t)((ring * kStages + t % kStages) * STAGE);
    if (base + kTileKeys <= L) {
      const char* ss = src + base * rowstride;
#pragma unroll
      for (int i = 0; i < NI; ++i) lds_dma16_sv(ss, soff[i], dst + KPI * (NI * wave + i) * ROWB);
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int64_t o = (int64_t)min(base + skey[i], L - 1) * rowstride + schunk[i];
        lds_dma16(src + o, dst + KPI * (NI * wave + i) * ROWB);
      }
    }
  };
  auto issue = [&](int t) {
    issue_op(t, 0);
    issue_op(t, 1);
  };

  // LDS fragment addresses (bytes, stage 0). K: row 32 kb + l32, chunk
  // 2 ks + hh; the swizzle turns the ks step into an XOR with 32 ks.
  const uint32_t ka0 = (uint32_t)(l32 * ROWB + 16 * (hh ^ kv_swizzle<D>(l32)));
  // V, transposing read r of step ps: 16-lane group g = lane / 16 reads rows
  // 16 ps + 4 (g / 2) + 8 r + (lane % 16) / 4, dims 32 db + 16 (g % 2) +
  // 4 (lane % 4) .. +3; the db step is an XOR with 64 db.
  uint32_t va0[2];
#pragma unroll
  for (int rr = 0; rr < 2; ++rr) {
    const int g = lane >> 4, jl = lane & 15;
    const int key = 4 * (g >> 1) + 8 * rr + (jl >> 2);
    const int chunk0 = 2 * (g & 1) + ((jl & 3) >> 1);
    va0[rr] = (uint32_t)(kStages * STAGE + key * ROWB + 16 * (chunk0 ^ kv_swizzle<D>(key)) +
                         8 * (jl & 1));
  }

  const int ntiles = (L + kTileKeys - 1) / kTileKeys;
  const int last_valid = L - (ntiles - 1) * kTileKeys;    // keys in the last stage
  float m_run = -INFINITY, l_part = 0.f;
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;

  // Scores of one stage: S^T for the 64 keys in LDS buffer `buf`. Element
  // 4 qq + i of sacc[kb] is S[key 32 kb + 8 qq + 4 hh + i][row l32].
  auto qk = [&](int buf, f32x16 (&sacc)[KB]) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[kb][e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const bf16x8 a = *reinterpret_cast<const ROCS_LDS bf16x8*>(
            lds3 + ((ka0 ^ (32u * ks)) + buf * STAGE + kb * 32 * ROWB));
        sacc[kb] = mfma32(a, qf[ks], sacc[kb]);
      }
      // Keep at most two steps of K fragments in flight (register budget for
      // two waves per SIMD); the other wave on the SIMD covers the latency.
      if (ks % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Row max of one stage (masking the keys past the history's end in the
  // last stage) and the move of the running max: only when the stage max
  // exceeds it by more than 2^kLazyRescale (always on the first stage).
  auto row_max = [&](f32x16 (&sacc)[KB], auto masked, int valid) {
    if constexpr (decltype(masked)::value) {
      // One 16-key group at a time: issued all at once, the 32 compares would
      // hold 32 lane masks (64 scalar registers) and push values to scratch.
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (32 * kb + 8 * qq + 4 * hh + i >= valid) sacc[kb][4 * qq + i] = -INFINITY;
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    // Row max: 32 keys per lane, then across the two wave halves.
    float mx = sacc[0][0];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sacc[kb][e]);
    mx = max_across_halves(mx) * scale_log2;
    const bool need = mx > m_run + kLazyRescale;
    if (__ballot(need) != 0) {
      const float m_new = need ? mx : m_run;
      const float alpha = exp2f(m_run - m_new);            // 0 on the first stage
      m_run = m_new;
      l_part *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
    }
  };

  // Weights of MFMA step ps as packed bf16 B fragments: step ps covers keys
  // 16 ps + 4 hh + {0..3} and 16 ps + 8 + 4 hh + {0..3}, elements
  // 8 (ps % 2) .. +7 of sacc[ps / 2]. Each packed pair is a scalar of its
  // own: the row-sum dot2 must not read its operand out of a vector register
  // tuple (the gfx950 code generator has been seen to feed the same tuple
  // element to every dot2 in that form). `lst` sums the bf16-rounded weights
  // the PV product uses.
  auto exp_block = [&](const f32x16 (&sacc)[KB], int ps, uint32_t (&pk)[4], float& lst) {
    const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float s0 = sacc[ps / 2][8 * (ps % 2) + 2 * w];
      const float s1 = sacc[ps / 2][8 * (ps % 2) + 2 * w + 1];
      pk[w] = pack_bf16x2(__builtin_amdgcn_exp2f(fmaf(s0, scale_log2, -m_run)),
                          __builtin_amdgcn_exp2f(fmaf(s1, scale_log2, -m_run)));
      lst = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk[w]), ones, lst, false);
    }
  };
  // O^T += V^T P^T for step ps: the A lane holds V^T[32 db + l32][the same
  // 8 keys], read transposed out of the row-major V stage.
  auto pv_block = [&](int buf, int ps, const uint32_t (&pk)[4]) {
    const bf16x8 pf = as_bf16x8(u32x4{pk[0], pk[1], pk[2], pk[3]});
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const uint32_t off = buf * STAGE + ps * 16 * ROWB;
      const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (ROCS_LDS i16x4*)(lds3 + ((va0[0] ^ (64u * db)) + off))));
      const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (ROCS_LDS i16x4*)(lds3 + ((va0[1] ^ (64u * db)) + off))));
      oacc[db] = mfma32(as_bf16x8(u32x4{lo[0], lo[1], hi[0], hi[1]}), pf, oacc[db]);
    }
  };
  // One stage of the software pipeline: the scores of the next stage (LDS
  // buffer nbuf) on the matrix cores, interleaved step by step with the
  // weights of this stage on the VALU; then this stage's PV product. The
  // weights use the running max as it stands; their per-lane sum bounds each
  // of them, so a stage whose sum stays below 2^kLazyRescale needs no max at
  // all. Otherwise (first stage, a jump of the scores, inf or NaN) the stage
  // takes the row max and recomputes its weights.
  auto stage = [&](int nbuf, f32x16 (&snext)[KB], int buf, f32x16 (&sacc)[KB]) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) snext[kb][e] = 0.f;
    uint32_t pk[PS][4];
    float lst = 0.f;
#pragma unroll
    for (int ps = 0; ps < PS; ++ps) {
#pragma unroll
      for (int ks = (KS / PS) * ps; ks < (KS / PS) * (ps + 1); ++ks)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          const bf16x8 a = *reinterpret_cast<const ROCS_LDS bf16x8*>(
              lds3 + ((ka0 ^ (32u * ks)) + nbuf * STAGE + kb * 32 * ROWB));
          snext[kb] = mfma32(a, qf[ks], snext[kb]);
        }
      exp_block(sacc, ps, pk[ps], lst);
      // head_dim 128: the compiler's own interleave of these MFMAs with the
      // next step's weights measured 1.3% faster than this fixed order.
      if constexpr (D == 64) __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_expect(__ballot(!(lst <= kWeightBound)) != 0, 0)) {
      row_max(sacc, std::false_type(), kTileKeys);
      lst = 0.f;
#pragma unroll
      for (int ps = 0; ps < PS; ++ps) exp_block(sacc, ps, pk[ps], lst);
    }
    l_part += lst;
    // The PV products run at raised wave priority, so the SIMD's other wave
    // (of the other workgroup) fills their gaps with its own work instead of
    // delaying them (about 1% at head_dim 128).
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ps = 0; ps < PS; ++ps) {
      pv_block(buf, ps, pk[ps]);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  // The last (possibly ragged) stage: masked row max, weights, PV.
  auto last_stage = [&](int buf, f32x16 (&sacc)[KB]) {
    row_max(sacc, std::true_type(), last_valid);
    uint32_t pk[PS][4];
    float lst = 0.f;
#pragma unroll
    for (int ps = 0; ps < PS; ++ps) exp_block(sacc, ps, pk[ps], lst);
    l_part += lst;
#pragma unroll
    for (int ps = 0; ps < PS; ++ps) pv_block(buf, ps, pk[ps]);
  };

  // Software pipeline over stages: while the matrix cores compute the scores
  // of stage t + 1, the VALU runs the softmax of stage t, then stage t's PV
  // product follows. Meanwhile K of stage t + 2 and V of stage t + 1 are
  // loaded; one barrier per stage hands the ring slots around.
  issue(0);
  if (ntiles > 1) issue_op(1, 0);
  // Everything resident, the query fragments included: from here on the
  // only vector-memory operations in flight are the ring's DMA loads, which
  // the compiler does not track, so it adds no waits of its own in the loop.
  wait_vmcnt<0>();
  ring_barrier();
  f32x16 s_a[KB], s_b[KB];
  auto step = [&](int kt, f32x16 (&s_cur)[KB], f32x16 (&s_next)[KB]) {
    // This step reads K of stage kt + 1 and V of stage kt; their other slots
    // (K of kt, V of kt - 1) were released by the last barrier.
    if (kt + 2 < ntiles) issue_op(kt + 2, 0);
    if (kt + 1 < ntiles) issue_op(kt + 1, 1);
    if (active) stage((kt + 1) % kStages, s_next, kt % kStages, s_cur);
    wait_vmcnt<0>();                                        // K of kt + 2, V of kt + 1
    ring_barrier();
  };
  if (active) qk(0, s_a);
  // Step 0 reloads K slot 0, which qk(0) has just read.
  ring_barrier();
  int kt = 0;
  for (; kt + 2 < ntiles; kt += 2) {        // unrolled by two: the score buffers swap roles
    step(kt, s_a, s_b);
    step(kt + 1, s_b, s_a);
  }
  if (kt + 1 < ntiles) {
    step(kt, s_a, s_b);
    if (active) {                              // one call site for the last stage
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) s_a[kb] = s_b[kb];
    }
  }
  if (active) last_stage((ntiles - 1) % kStages, s_a);

  // Epilogue through LDS. Once every wave is past its last stage the K/V
  // ring is idle; each wave writes its 32 normalised output rows there
  // (16 contiguous bytes per lane after a half-wave swap, row-swizzled) and
  // reads them back row-contiguous, so each store instruction covers whole
  // 2D-byte row segments instead of 16 bytes of 32 different rows.
  ring_barrier();
  if (!active) return;
  // The epilogue's addresses come from a laundered copy of the lane index:
  // derived from `lane` directly, the compiler computes them at the start
  // and holds them through the main loop, where the registers are short.
  int lane_e = lane;
  asm volatile("" : "+v"(lane_e));
  const int l32e = lane_e & 31, hhe = lane_e >> 5;
  // Element 4 qq + i of oacc[db] is O[row l32][dim 32 db + 8 qq + 4 hh + i];
  // after the swap lane (l32, hh) holds dims 32 db + 16 j + 8 hh .. +7
  // (16-byte chunk 4 db + 2 j + hh of the row).
  const float inv = 1.0f / sum_across_halves(l_part);
  const uint32_t obase = (uint32_t)(wave * 32 * ROWB);
  auto out_swz = [](int row) { return CR == 16 ? (row & 15) : ((row >> 1) & 7); };
  // Read-back layout: store instruction i covers rows RPS i .. RPS i + RPS - 1
  // of the wave's 32, lane -> row RPS i + lane / CR, chunk lane % CR. With a
  // residual, its matching 16-byte pieces are loaded first, so their latency
  // runs under the LDS round trip and no load waits behind an output store.
  constexpr int RPS = 1024 / ROWB;            // output rows per store instruction
  constexpr int NST = 32 / RPS;
  auto out_off = [&](int i) -> int64_t {
    const int row = RPS * i + lane_e / CR;
    return src_row(min(wrow0 + row, rows - 1)) * qs + (int64_t)h * D + 8 * (lane_e % CR);
  };
  u32x4 rv[NST];
  if (res != nullptr) {
#pragma unroll
    for (int i = 0; i < NST; ++i) rv[i] = *reinterpret_cast<const u32x4*>(res + out_off(i));
  }
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x16& o = oacc[db];
      const uint32_t e0 = pack_bf16x2(o[8 * j] * inv, o[8 * j + 1] * inv);
      const uint32_t e1 = pack_bf16x2(o[8 * j + 2] * inv, o[8 * j + 3] * inv);
      const uint32_t o0 = pack_bf16x2(o[8 * j + 4] * inv, o[8 * j + 5] * inv);
      const uint32_t o1 = pack_bf16x2(o[8 * j + 6] * inv, o[8 * j + 7] * inv);
      const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
      const int chunk = (4 * db + 2 * j + hhe) ^ out_swz(l32e);
      *reinterpret_cast<ROCS_LDS u32x4*>(lds3 + obase + l32e * ROWB + 16 * chunk) =
          u32x4{s0[0], s1[0], s0[1], s1[1]};
    }
#pragma unroll
  for (int i = 0; i < NST; ++i) {
    const int row = RPS * i + lane_e / CR;
    const u32x4 v = *reinterpret_cast<const ROCS_LDS u32x4*>(
        lds3 + obase + row * ROWB + 16 * ((lane_e % CR) ^ out_swz(row)));
    if (wrow0 + row < rows) {
      const int64_t o = out_off(i);
      *reinterpret_cast<u32x4*>(out + o) = v;
      if (res != nullptr) *reinterpret_cast<u32x4*>(out_sum + o) = add_bf16x8(v, rv[i]);
    }
  }
}

// ---------------------------------------------------------------------------
// The same attention for calls of few tiles (bf16, head_dim 64 or 128): a
// workgroup takes 32 query rows of one head and its four waves split the
// history, wave w taking stages w, w + 4, ... of 64 keys. With 128-row tiles
// such a call leaves most CUs idle, and each workgroup walks the whole history
// alone; here there are four times the workgroups, each a quarter of the walk.
// Every wave stages K and V in LDS of its own (DMA, the next K under the
// softmax, the next V under the next scores), so the waves meet only for the
// first stage's row max and to merge their partial softmaxes at the end. The
// layouts, the weights rounded to bf16, the row sums taken from them and the
// running max are those of the tiled kernel: all four waves start from the row
// max of the history's first stage and move it under the same rule, so a
// weight is rounded against the same max in both kernels and their results
// differ only by the order of fp32 sums (after a jump of the scores by more
// than 2^kLazyRescale also by that max: a wave knows its own stages' alone).
// What bounds it: the latency of a wave's chain of stages. At one request of
// 203 candidates, history 613, 4 heads x 64 it takes 6.4 us (128-row tiles:
// 11.7 us), at 16 requests of 32 query rows, history 1024: 7.7 us (15.4 us).
// ---------------------------------------------------------------------------
constexpr int kSplitRows = 32;

template <int D, bool MAPPED, bool QPROJ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void dca_attn_split(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    const int32_t* __restrict__ cand_off, const int32_t* __restrict__ kv_off,
    bf16_t* __restrict__ out, int R, int Tq, int H, int64_t kv_stride, float scale_log2,
    int slots_per_head, const int32_t* __restrict__ order, const bf16_t* __restrict__ res,
    bf16_t* __restrict__ out_sum, const bf16_t* __restrict__ wq) {
  constexpr int W = 4, TR = kSplitRows;
  constexpr int KB = kTileKeys / 32, KS = D / 16, DB = D / 32, PS = kTileKeys / 16;
  constexpr int ROWB = 2 * D, CR = D / 8;
  constexpr int STAGE = kTileKeys * ROWB;             // bytes of one K (or V) stage
  constexpr int KPI = 1024 / ROWB;                    // rows per wave-wide DMA load
  constexpr int NI = kTileKeys / KPI;                 // DMA loads per stage and operand
  constexpr int OP = D + 4;                           // floats of one partial output row
  static_assert(TR * OP * 4 <= 2 * STAGE, "a wave's partial output takes its staging");
  __shared__ __attribute__((aligned(1024))) char lds[W * 2 * STAGE];
  __shared__ float pm[W][TR], pl[W][TR], m0[TR];
  ROCS_LDS char* const lds3 = (ROCS_LDS char*)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const uint32_t work = xcd_remap(blockIdx.x, gridDim.x);
  const int h = __builtin_amdgcn_readfirstlane((int)(work / (uint32_t)slots_per_head));
  const int64_t slot = work - (uint32_t)h * (uint32_t)slots_per_head;
  const int r = request_of_slot(cand_off, R, slot, Tq, TR);
  const int64_t rend = (int64_t)cand_off[r + 1] * Tq;
  const int64_t row0 = (int64_t)cand_off[r] * Tq + (slot - tile_base(cand_off, r, Tq, TR)) * TR;
  if (row0 >= rend) return;                               // idle slot
  const int rows = (int)(rend - row0 < TR ? rend - row0 : TR);
  const int64_t kv0 = kv_off[r];
  const int L = kv_off[r + 1] - (int)kv0;
  const int64_t qs = (int64_t)H * D;
  auto src_row = [&](int i) -> int64_t {
    const int64_t gr = row0 + i;
    if constexpr (MAPPED) {
      const int64_t p = gr / Tq;
      return (int64_t)order[p] * Tq + (gr - p * Tq);
    } else {
      return gr;
    }
  };
  // DMA lane map of a stage: load i fills rows KPI i + lane / CR, chunk
  // position lane % CR, with chunk (lane % CR) ^ kv_swizzle(row).
  const char* kbase = reinterpret_cast<const char*>(k + kv0 * kv_stride + (int64_t)h * D);
  const char* vbase = reinterpret_cast<const char*>(v + kv0 * kv_stride + (int64_t)h * D);
  const int64_t rowstride = kv_stride * 2;
  const uint32_t kdst = lds_addr(lds) + (uint32_t)(wave * 2 * STAGE);
  auto issue = [&](const char* src, int t, uint32_t dst) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int row = KPI * i + lane / CR;
      lds_dma16(src + (int64_t)min(t * kTileKeys + row, L - 1) * rowstride +
                    16 * ((lane % CR) ^ kv_swizzle<D>(row)),
                dst + 1024u * i);
    }
  };
  // Query rows as B fragments, all waves the same 32 (projected as in the
  // tiled kernel, W_q,h staged in the K/V area first).
  const int qrow = min(l32, rows - 1);                    // clamped; extra rows never stored
  const int ntiles = (L + kTileKeys - 1) / kTileKeys;
  bf16x8 qf[KS];
  if constexpr (!QPROJ) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks] = *reinterpret_cast<const bf16x8*>(q + (int64_t)h * D + src_row(qrow) * qs + 16 * ks + 8 * hh);
  } else {
    constexpr int PK = kProjIn / 16, PRB = kProjIn * 2, PNI = D * PRB / 1024 / W;
    static_assert(D == 64 && W * 2 * STAGE >= D * PRB, "projection staging");
    const char* wsrc = uniform_ptr(reinterpret_cast<const char*>(wq + (int64_t)h * D * kProjIn));
    const uint32_t lb = lds_addr(lds);
#pragma unroll
    for (int i = 0; i < PNI; ++i) {
      const int blk = wave * PNI + i;                     // 1 KiB: rows 2 blk, 2 blk + 1
      const int prow = 2 * blk + (lane >> 5), pos = lane & 31;
      lds_dma16_sv(wsrc, (uint32_t)(prow * PRB + 16 * (pos ^ (prow & 15))), lb + 1024u * blk);
    }
    const bf16_t* xr = q + src_row(qrow) * kProjIn + 8 * hh;
    bf16x8 xq[PK];
#pragma unroll
    for (int s2 = 0; s2 < PK; ++s2) xq[s2] = *reinterpret_cast<const bf16x8*>(xr + 16 * s2);
    wait_vmcnt<0>();
    ring_barrier();
    f32x16 pacc[2] = {};
#pragma unroll
    for (int s2 = 0; s2 < PK; ++s2)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int prow = 32 * b + l32;
        const bf16x8 a = *reinterpret_cast<const ROCS_LDS bf16x8*>(
            lds3 + prow * PRB + 16 * ((2 * s2 + hh) ^ (prow & 15)));
        pacc[b] = mfma32(a, xq[s2], pacc[b]);
      }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const f32x16& pa = pacc[b];
        const uint32_t e0 = pack_bf16x2(pa[8 * jj], pa[8 * jj + 1]);
        const uint32_t e1 = pack_bf16x2(pa[8 * jj + 2], pa[8 * jj + 3]);
        const uint32_t o0 = pack_bf16x2(pa[8 * jj + 4], pa[8 * jj + 5]);
        const uint32_t o1 = pack_bf16x2(pa[8 * jj + 6], pa[8 * jj + 7]);
        const auto t0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
        const auto t1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
        qf[2 * b + jj] = as_bf16x8(u32x4{t0[0], t1[0], t0[1], t1[1]});
      }
    wait_lgkmcnt0();
    ring_barrier();                                       // W_q's LDS goes to K and V
  }
  // The query rows resident before the first DMA load: the stage loop then
  // has only DMA loads in flight, which the waits below count.
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" :: "v"(as_u32x4(qf[ks])));

  const uint32_t kb0 = (uint32_t)(wave * 2 * STAGE);
  const uint32_t ka0 = kb0 + (uint32_t)(l32 * ROWB + 16 * (hh ^ kv_swizzle<D>(l32)));
  uint32_t va0[2];
#pragma unroll
  for (int rr = 0; rr < 2; ++rr) {
    const int g = lane >> 4, jl = lane & 15;
    const int key = 4 * (g >> 1) + 8 * rr + (jl >> 2);
    const int chunk0 = 2 * (g & 1) + ((jl & 3) >> 1);
    va0[rr] = kb0 + (uint32_t)(STAGE + key * ROWB + 16 * (chunk0 ^ kv_swizzle<D>(key)) + 8 * (jl & 1));
  }
  float m = -INFINITY, l_part = 0.f;
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) oacc[db] = f32x16{};
  if (wave < ntiles) {
    issue(kbase, wave, kdst);
    issue(vbase, wave, kdst + STAGE);
  } else {
    ring_barrier();                                       // the first stage's row max, below
  }
  for (int t = wave; t < ntiles; t += W) {
    const bool more = t + W < ntiles;
    wait_vmcnt<NI>();                                     // K of t (V of t may be in flight)
    asm volatile("" ::: "memory");
    f32x16 sacc[KB] = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const bf16x8 a = *reinterpret_cast<const ROCS_LDS bf16x8*>(
            lds3 + ((ka0 ^ (32u * ks)) + kb * 32 * ROWB));
        sacc[kb] = mfma32(a, qf[ks], sacc[kb]);
      }
    wait_lgkmcnt0();                                      // K's fragments are in registers
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (more) issue(kbase, t + W, kdst);
    if (t == ntiles - 1) {                                // keys past the history's end
      const int valid = L - t * kTileKeys;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (32 * kb + 8 * (e / 4) + 4 * hh + e % 4 >= valid) sacc[kb][e] = -INFINITY;
    }
    // Row max: 32 keys per lane in two chains, then across the wave halves.
    auto row_max = [&]() __attribute__((always_inline)) {
      float mx[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        mx[kb] = sacc[kb][0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx[kb] = fmaxf(mx[kb], sacc[kb][e]);
      }
      static_assert(KB == 2, "two chains");
      return max_across_halves(fmaxf(mx[0], mx[1])) * scale_log2;
    };
    if (t < W) {                                          // every wave's first stage
      if (t == 0) {
        const float mx = row_max();
        if (hh == 0) m0[l32] = mx;
        wait_lgkmcnt0();
      }
      ring_barrier();
      m = m0[l32];
    }
    // Each packed pair is a scalar of its own (see exp_block above); a sum per
    // 16 keys, so that the test of the weights waits for a short chain.
    uint32_t pk[PS][4];
    auto weights = [&](float ms) __attribute__((always_inline)) {
      const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
      float part[PS];
#pragma unroll
      for (int ps = 0; ps < PS; ++ps) {
        part[ps] = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float s0 = sacc[ps / 2][8 * (ps % 2) + 2 * w];
          const float s1 = sacc[ps / 2][8 * (ps % 2) + 2 * w + 1];
          pk[ps][w] = pack_bf16x2(__builtin_amdgcn_exp2f(fmaf(s0, scale_log2, -ms)),
                                  __builtin_amdgcn_exp2f(fmaf(s1, scale_log2, -ms)));
          part[ps] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk[ps][w]), ones,
                                                     part[ps], false);
        }
      }
      static_assert(PS == 4, "four sums");
      return (part[0] + part[1]) + (part[2] + part[3]);
    };
    float lst = weights(m);
    if (__builtin_expect(__ballot(!(lst <= kWeightBound)) != 0, 0)) {
      const float mx = row_max();
      const bool need = mx > m + kLazyRescale;
      const float alpha = need ? exp2f(m - mx) : 1.f;
      if (need) m = mx;
      l_part *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
      lst = weights(m == -INFINITY ? 0.f : m);            // no finite score yet: weights 0
    }
    l_part += lst;
    if (more) wait_vmcnt<NI>(); else wait_vmcnt<0>();     // V of t (K of t + 4 in flight)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int ps = 0; ps < PS; ++ps) {
      const bf16x8 pf = as_bf16x8(u32x4{pk[ps][0], pk[ps][1], pk[ps][2], pk[ps][3]});
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const uint32_t off = ps * 16 * ROWB;
        const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (ROCS_LDS i16x4*)(lds3 + ((va0[0] ^ (64u * db)) + off))));
        const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (ROCS_LDS i16x4*)(lds3 + ((va0[1] ^ (64u * db)) + off))));
        oacc[db] = mfma32(as_bf16x8(u32x4{lo[0], lo[1], hi[0], hi[1]}), pf, oacc[db]);
      }
    }
    wait_lgkmcnt0();                                      // V's fragments are in registers
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (more) issue(vbase, t + W, kdst + STAGE);
  }
  // This wave's partial softmax into its staging area: element 4 qq + i of
  // oacc[db] is O[row l32][dim 32 db + 8 qq + 4 hh + i].
  const float l_sum = sum_across_halves(l_part);
  if (hh == 0) {
    pm[wave][l32] = m;
    pl[wave][l32] = l_sum;
  }
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int qq = 0; qq < 4; ++qq)
      *reinterpret_cast<ROCS_LDS f32x4*>(lds3 + kb0 + 4 * (l32 * OP + 32 * db + 8 * qq + 4 * hh)) =
          f32x4{oacc[db][4 * qq], oacc[db][4 * qq + 1], oacc[db][4 * qq + 2], oacc[db][4 * qq + 3]};
  __syncthreads();
  for (int c = tid; c < rows * CR; c += 256) {            // one 16-byte piece of an output row
    const int i = c / CR, d0 = 8 * (c % CR);
    const float mx = fmaxf(fmaxf(pm[0][i], pm[1][i]), fmaxf(pm[2][i], pm[3][i]));
    const float ms = mx == -INFINITY ? 0.f : mx;
    float l = 0.f;
    f32x4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float f = exp2f(pm[w][i] - ms);
      const ROCS_LDS char* src = lds3 + w * 2 * STAGE + 4 * (i * OP + d0);
      l += pl[w][i] * f;
      y0 += *reinterpret_cast<const ROCS_LDS f32x4*>(src) * f;
      y1 += *reinterpret_cast<const ROCS_LDS f32x4*>(src + 16) * f;
    }
    const float inv = L > 0 ? 1.0f / l : 0.f;             // empty history: zeros
    const u32x4 y = {pack_bf16x2(y0[0] * inv, y0[1] * inv), pack_bf16x2(y0[2] * inv, y0[3] * inv),
                     pack_bf16x2(y1[0] * inv, y1[1] * inv), pack_bf16x2(y1[2] * inv, y1[3] * inv)};
    const int64_t o = src_row(i) * qs + (int64_t)h * D + d0;
    *reinterpret_cast<u32x4*>(out + o) = y;
    if (res != nullptr)
      *reinterpret_cast<u32x4*>(out_sum + o) = add_bf16x8(y, *reinterpret_cast<const u32x4*>(res + o));
  }
}

// ---------------------------------------------------------------------------
// General kernel: any dtype, head_dim <= 256, any stride.
//
// A workgroup takes up to 16 consecutive query rows of one head; its four
// waves split the history in blocks of 16 keys and merge their partial
// softmaxes through LDS. Scores and outputs run on the fp32 matrix
// instructions (fp32 in, fp32 accumulation; bf16 inputs convert exactly): S^T =
// K Q^T leaves lane (l16, g) with keys 4 g .. + 3 of query row l16, which is
// the B operand of O^T = V^T P^T as it stands, so the weights never leave the
// registers. Rows of other requests in the tile (a request's edge, or a
// caller's map in any order) take a pass of their own over their request's
// history; a pass hands on only its own rows.
// A score is summed in 4 CB accumulators, added pairwise: one chain over
// head_dim would be less exact than a lane tree. Error against float64 (fp32,
// 256 rows x 2 heads; a lane tree with keys in order / one chain / as here):
// head_dim 32, history 32: 1.67e-7 / 1.80e-7 / 1.36e-7; 128, 32: 1.69e-7 /
// 3.01e-7 / 1.38e-7; 256, 5: 9.05e-8 / 2.12e-7 / 9.03e-8; 64, 2000: 1.04e-6 /
// 5.0e-7 / 4.3e-7. (bf16 inputs: four, the output's rounding hides the rest.)
// What bounds it: the latency of a wave's loads. They are clamped and selected
// rather than skipped, so that a block's K and V are in flight together, and
// the registers leave room for two workgroups a CU: 8,192 rows x 2 heads x 128,
// history 200, fp32: 104 -> 60 us; 64 rows x 4 heads x 64, history 5000: 335 ->
// 117 us; 256 rows x 2 heads x 32, history 32: 4.9 -> 4.2 us (one wave per
// query row: 809, 4018 and 20.5). fp32 at head_dim 256 needs one workgroup a CU
// and K's loads in turn: 100 rows x 2 heads, history 700: 174 us, 236 with them
// all in flight.
// ---------------------------------------------------------------------------
constexpr int kGenRows = 16;   // at most

// Dims d .. d + 3 of a row of D, zeros past its end. The loads are clamped, not
// skipped: a branch around each would keep them from being in flight together.
template <typename T, bool VEC>
__device__ __forceinline__ f32x4 dims4(const T* row, int d, int D) {
  if constexpr (VEC) {                     // D is a multiple of four, and so is d
    const f32x4 v = load4_f32<T, true>(row + min(d, D - 4), 4);
    return d < D ? v : f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = load_f32(row + min(d + i, D - 1));
      v[i] = d + i < D ? x : 0.f;
    }
    return v;
  }
}

// DP: head_dim rounded up to 32, 64, 128 or 256. VEC: every row of q, k, x and
// w_q is aligned to four elements and head_dim (and d_in) a multiple of four.
template <typename T, int DP, bool VEC>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(DP == 256 && sizeof(T) == 4 ? 1 : 2))) void dca_attn_generic(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const int32_t* __restrict__ cand_off, const int32_t* __restrict__ kv_off,
    T* __restrict__ out, int R, int Tq, int64_t n_rows, int tile_rows, int H, int D,
    int64_t kv_stride, float scale, const int32_t* __restrict__ ids, const T* __restrict__ res,
    T* __restrict__ out_sum, const T* __restrict__ wq, int d_in) {
  constexpr int NB = DP / 16;              // 16-dim blocks
  constexpr int CB = sizeof(T) == 2 || DP == 32 ? 1 : DP == 64 ? 4 : 8;
  constexpr int LP = DP + 4;               // LDS row (floats), padded against bank conflicts
  __shared__ __attribute__((aligned(16))) float po[4][kGenRows][LP];   // O, per wave (also Q)
  __shared__ float pm[4][kGenRows], pl[4][kGenRows];                   // running max, row sum
  __shared__ int has_keys[kGenRows];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int h = blockIdx.y;
  const int64_t row0 = (int64_t)blockIdx.x * tile_rows;
  const int rows = (int)(n_rows - row0 < tile_rows ? n_rows - row0 : tile_rows);
  const int64_t row = row0 + min(l16, rows - 1);         // clamped; extra rows never stored
  // The row's request: from the caller's per-candidate map (clamped into
  // [0, R), so a malformed map gives wrong rows, never an access outside the
  // offsets), else from the CSR offsets.
  const int rq = ids != nullptr ? (int)min((uint32_t)ids[row / Tq], (uint32_t)(R - 1))
                                : owner_of(cand_off, R, row / Tq);
  // Query fragments: dims 16 b + 4 g + i of row l16.
  f32x4 qf[NB];
  if (wq == nullptr) {
    const T* qr = q + (row * H + h) * D;
#pragma unroll
    for (int b = 0; b < NB; ++b) qf[b] = dims4<T, VEC>(qr, 16 * b + 4 * g, D);
  } else {
    // The fused query projection q = x W_q^T for this head's dims, rounded to
    // T as a separate projection would store it; the waves share the blocks.
    const T* xr = q + row * d_in;
    for (int b = wave; b < NB; b += 4) {
      const int dim = 16 * b + l16;
      const T* wr = wq + ((int64_t)h * D + dim) * d_in;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int kk = 4 * g; kk < (d_in + 15) / 16 * 16; kk += 16) {
        const f32x4 av = load4_f32<T, VEC>(wr + kk, dim < D ? d_in - kk : 0);
        const f32x4 bv = load4_f32<T, VEC>(xr + kk, d_in - kk);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[i], acc, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = (float)from_f32<T>(acc[i]);
      *reinterpret_cast<f32x4*>(&po[0][l16][16 * b + 4 * g]) = acc;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) qf[b] = *reinterpret_cast<const f32x4*>(&po[0][l16][16 * b + 4 * g]);
    __syncthreads();
  }
  uint32_t todo = (1u << rows) - 1u;       // rows whose request has had no pass yet
  while (todo != 0) {
    const int r = __builtin_amdgcn_readlane(rq, __builtin_ctz(todo));
    const bool mine = rq == r;
    todo &= ~(uint32_t)(__ballot(mine) & 0xffffu);
    const int64_t a = kv_off[r];
    const int L = kv_off[r + 1] - (int)a;
    float m = -INFINITY, lsum = 0.f;
    f32x4 o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kb = 16 * wave; kb < L; kb += 64) {
      const T* kr = k + (a + min(kb + l16, L - 1)) * kv_stride + (int64_t)h * D;
      const T* vr[4];                                    // clamped: no load waits for a branch
#pragma unroll
      for (int i = 0; i < 4; ++i)
        vr[i] = v + (a + min(kb + 4 * g + i, L - 1)) * kv_stride + (int64_t)h * D;
      f32x4 part[CB][4] = {};
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const f32x4 kf = DP == 256 ? load4_f32<T, VEC>(kr + 16 * b + 4 * g, D - 16 * b - 4 * g)
                                   : dims4<T, VEC>(kr, 16 * b + 4 * g, D);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          part[b % CB][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i], qf[b][i], part[b % CB][i],
                                                                 0, 0, 0);
      }
#pragma unroll
      for (int c = 1; c < CB; c *= 2)                    // pairwise
#pragma unroll
        for (int b = 0; b + c < CB; b += 2 * c)
#pragma unroll
          for (int i = 0; i < 4; ++i) part[b][i] += part[b + c][i];
      f32x4 s4 = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]);
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s4[i] = kb + 4 * g + i < L ? s4[i] * scale : -INFINITY;
        mx = fmaxf(mx, s4[i]);
      }
      const float mn = fmaxf(m, max_across_rows(mx));
      const float ms = mn == -INFINITY ? 0.f : mn;       // no finite score yet: weights 0
      const float alpha = expf(m - ms);
      f32x4 p;
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = expf(s4[i] - ms);
      lsum = lsum * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
      m = mn;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int dim = 16 * b + l16;
        o[b] *= alpha;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float vf = load_f32(vr[i] + min(dim, D - 1));
          o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kb + 4 * g + i < L && dim < D ? vf : 0.f, p[i],
                                                      o[b], 0, 0, 0);
        }
      }
    }
    lsum = sum_across_rows(lsum);
    if (mine) {
      if (g == 0) {
        pm[wave][l16] = m;
        pl[wave][l16] = lsum;
        if (wave == 0) has_keys[l16] = L > 0;
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
        *reinterpret_cast<f32x4*>(&po[wave][l16][16 * b + 4 * g]) = o[b];
    }
  }
  __syncthreads();
  // Merge the four partial softmaxes of each row. An empty history gives zeros.
  // Four dims a step: a row's four factors are formed once for them.
  for (int idx = threadIdx.x; idx < rows * (DP / 4); idx += 256) {
    const int i = idx / (DP / 4), d0 = 4 * (idx % (DP / 4));
    if (d0 >= D) continue;
    const float mx = fmaxf(fmaxf(pm[0][i], pm[1][i]), fmaxf(pm[2][i], pm[3][i]));
    const float ms = mx == -INFINITY ? 0.f : mx;
    float l = 0.f;
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = expf(pm[w][i] - ms);
      l += pl[w][i] * f;
      y += *reinterpret_cast<const f32x4*>(&po[w][i][d0]) * f;
    }
    const float inv = 1.0f / l;
    const int64_t at = ((row0 + i) * H + h) * D + d0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (d0 + e >= D) break;
      const T yt = from_f32<T>(has_keys[i] ? y[e] * inv : 0.f);
      out[at + e] = yt;
      if (res != nullptr) out_sum[at + e] = from_f32<T>(load_f32(&yt) + load_f32(res + at + e));
    }
  }
}

// ---------------------------------------------------------------------------
// Grouping a per-candidate request map by request, a stable counting sort,
// so that the tiled kernel also serves a general map (Section 4.3.1: resolve
// m_i, then share the request's K/V). order[p] lists request 0's candidates
// first, then request 1's, ..., each request's candidates in their original
// order; grp_off[R + 1] are the CSR offsets of that order. The candidates
// are cut into nb blocks of G; hist[r * nb + b] counts request r in block b,
// and its exclusive scan in that (request-major) order is the grouped
// position of request r's first candidate in block b. Ids outside [0, R)
// are clamped into range, as the other kernels do.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int clamp_request(int32_t m, int R) {
  return (int)min((uint32_t)m, (uint32_t)(R - 1));
}

__global__ __launch_bounds__(1024) void group_count(const int32_t* __restrict__ ids, int64_t N,
                                                    int R, int64_t G, int nb,
                                                    int32_t* __restrict__ hist) {
  __shared__ int cnt[kGroupMaxRequests];
  const int b = blockIdx.x;
  for (int r = threadIdx.x; r < R; r += 1024) cnt[r] = 0;
  __syncthreads();
  const int64_t lo = (int64_t)b * G, hi = min(lo + G, N);
  for (int64_t i = lo + threadIdx.x; i < hi; i += 1024) atomicAdd(&cnt[clamp_request(ids[i], R)], 1);
  __syncthreads();
  for (int r = threadIdx.x; r < R; r += 1024) hist[(int64_t)r * nb + b] = cnt[r];
}

// One workgroup: exclusive scan of hist[0 .. total) in place (each thread
// owns a contiguous run; the run sums are scanned in LDS), then the grouped
// offsets grp_off[r] = scan[r * nb], grp_off[R] = N.
__global__ __launch_bounds__(1024) void group_scan(int32_t* __restrict__ hist, int64_t total,
                                                   int R, int nb, int64_t N,
                                                   int32_t* __restrict__ grp_off) {
  __shared__ int part[1024];
  const int t = threadIdx.x;
  const int64_t per = (total + 1023) / 1024;
  const int64_t lo = min((int64_t)t * per, total), hi = min(lo + per, total);
  int sum = 0;
  for (int64_t i = lo; i < hi; ++i) sum += hist[i];
  part[t] = sum;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {                    // inclusive scan of the run sums
    const int add = t >= d ? part[t - d] : 0;
    __syncthreads();
    part[t] += add;
    __syncthreads();
  }
  int acc = part[t] - sum;                                // exclusive
  for (int64_t i = lo; i < hi; ++i) {
    const int c = hist[i];
    hist[i] = acc;
    acc += c;
  }
  __threadfence_block();
  __syncthreads();
  for (int r = t; r < R; r += 1024) grp_off[r] = hist[(int64_t)r * nb];
  if (t == 0) grp_off[R] = (int)N;
}

// One workgroup per block, each of its waves owning a contiguous share of the
// block's candidates: the waves count their shares, a prefix over the waves
// turns the counts into each wave's cursors, then every wave walks its share
// in order 64 candidates at a time. Lanes holding the same request are found
// by one ballot per bit of the request id and take consecutive slots in lane
// order, so the order within a request is the original one. The time is the
// length of a wave's serial walk: 16 waves take 13 us for 8192 candidates of
// 16 requests, counting included, where one wave per 4096 candidates visiting
// the requests of its 64 lanes one by one took 150 us (and 13 us to count).
// WHOLE (one block, N up to kGroupWholeCands): the counts are scanned here
// too and the grouped offsets written, in one launch instead of three.
constexpr int kGroupCounters = 32768;              // per-wave request counters in LDS (128 KiB)
constexpr int64_t kGroupWholeCands = 8192;
constexpr int kGroupAhead = 8;                     // rounds of 64 ids in flight

template <bool WHOLE>
__global__ __launch_bounds__(1024) void group_scatter(const int32_t* __restrict__ ids, int64_t N,
                                                      int R, int64_t G, int nb, int key_bits,
                                                      const int32_t* __restrict__ base,
                                                      int32_t* __restrict__ grp_off,
                                                      int32_t* __restrict__ order) {
  __shared__ int cnt[kGroupCounters];               // [wave][R]
  __shared__ int part[16];
  volatile int* const cursors = cnt;                // written by other lanes of the wave
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int NT = blockDim.x, W = NT / 64;
  for (int i = tid; i < W * R; i += NT) cnt[i] = 0;
  __syncthreads();
  const int64_t lo = (int64_t)b * G, hi = min(lo + G, N);
  const int64_t share = ((hi - lo + W - 1) / W + 63) / 64 * 64;
  const int64_t wlo = min(lo + wave * share, hi), whi = min(wlo + share, hi);
  // Ids are loaded kGroupAhead rounds at a time: one memory latency for all.
  for (int64_t c = wlo + lane; c < whi; c += 64 * kGroupAhead) {
    int key[kGroupAhead];
#pragma unroll
    for (int j = 0; j < kGroupAhead; ++j)
      key[j] = c + 64 * j < whi ? clamp_request(ids[c + 64 * j], R) : -1;
#pragma unroll
    for (int j = 0; j < kGroupAhead; ++j)
      if (key[j] >= 0) atomicAdd(&cnt[wave * R + key[j]], 1);
  }
  __syncthreads();
  // Counts -> cursors: the request's first position (its scan over the
  // requests, or the caller's), then a prefix over the waves.
  int run = 0;
  if constexpr (WHOLE) {
    // Requests in rounds of one per thread, scanned over the workgroup.
    for (int r0 = 0; r0 < R; r0 += NT) {
      const int r = r0 + tid;
      int sum = 0;
      if (r < R)
        for (int w = 0; w < W; ++w) sum += cnt[w * R + r];
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
      }
      if (lane == 63) part[wave] = incl;
      __syncthreads();
      int at = run + incl - sum, total = 0;
      for (int w = 0; w < W; ++w) {
        if (w < wave) at += part[w];
        total += part[w];
      }
      run += total;
      if (r < R) {
        grp_off[r] = at;
        for (int w = 0; w < W; ++w) {
          const int c = cnt[w * R + r];
          cnt[w * R + r] = at;
          at += c;
        }
      }
      __syncthreads();                              // part is free for the next round
    }
    if (tid == 0) grp_off[R] = (int)N;
  } else {
    for (int r = tid; r < R; r += NT) {
      int at = base[(int64_t)r * nb + b];
      for (int w = 0; w < W; ++w) {
        const int c = cnt[w * R + r];
        cnt[w * R + r] = at;
        at += c;
      }
    }
    __syncthreads();
  }
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int64_t c = wlo; c < whi; c += 64 * kGroupAhead) {
    int keys[kGroupAhead];
#pragma unroll
    for (int j = 0; j < kGroupAhead; ++j)
      keys[j] = c + 64 * j + lane < whi ? clamp_request(ids[c + 64 * j + lane], R) : -1;
#pragma unroll
    for (int j = 0; j < kGroupAhead; ++j) {
      const int key = keys[j];
      uint64_t same = __ballot(key >= 0);
      for (int bit = 0; bit < key_bits; ++bit) {
        const uint64_t m = __ballot((key >> bit) & 1);
        same &= (key >> bit) & 1 ? m : ~m;
      }
      if (key >= 0) {
        const int at = cursors[wave * R + key];     // read by every lane first ...
        order[at + __builtin_popcountll(same & below)] = (int)(c + 64 * j + lane);
        if ((same & below) == 0)                    // ... then advanced by the group's first
          cursors[wave * R + key] = at + __builtin_popcountll(same);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Tile plan for one batch (one workgroup of 256 threads, one wave per SIMD):
// every request's history length and tile count are read in one pass; the
// requests are sorted by (history length descending, index) as 32-bit keys
// in LDS (kPlanLenBits bits of clamped length, 12 bits of index): up to 256
// requests by counting each key's rank, more with a bitonic sort; an
// exclusive scan of the tile counts in that order gives P. Beyond
// kAttnPlanMaxSort requests only the header is written (mode 0: the kernel
// keeps its built-in order).
// ---------------------------------------------------------------------------
constexpr int kPlanThreads = 256;
constexpr int kPlanIdBits = 12;
constexpr int kPlanLenBits = 32 - kPlanIdBits;   // lengths beyond 2^20 - 1 tie
static_assert(kAttnPlanMaxSort == (1 << kPlanIdBits), "plan key layout");

__global__ __launch_bounds__(kPlanThreads) void attn_plan_kernel(
    const int32_t* __restrict__ cand_off, const int32_t* __restrict__ kv_off, int R, int Tq,
    int H, int32_t* __restrict__ plan) {
  constexpr int PER = (int)kAttnPlanMaxSort / kPlanThreads;   // sorted positions per thread
  constexpr uint32_t kLenMax = (1u << kPlanLenBits) - 1;
  __shared__ __attribute__((aligned(16))) uint32_t key[kAttnPlanMaxSort];
  __shared__ int32_t tiles[kAttnPlanMaxSort];
  __shared__ int32_t wsum[kPlanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (R > kAttnPlanMaxSort) {
    if (tid < kPlanHeader) plan[tid] = tid == 2 ? R : 0;   // mode 0
    return;
  }
  int32_t* ids = plan + kPlanHeader;
  int32_t* P = ids + R;
  if (R <= kPlanThreads) {
    // Up to one request per thread: its sorted position is the number of
    // smaller keys (keys are distinct), counted over the LDS copy four keys
    // per read; then the tile counts are scanned in sorted order.
    uint32_t kk = ~0u;
    int tl = 0;
    if (tid < R) {
      const uint32_t L = (uint32_t)max(kv_off[tid + 1] - kv_off[tid], 0);
      const int64_t rows = (int64_t)max(cand_off[tid + 1] - cand_off[tid], 0) * Tq;
      kk = ((kLenMax - min(L, kLenMax)) << kPlanIdBits) | (uint32_t)tid;
      tl = (int)((rows + kAttnTileRows - 1) / kAttnTileRows) * H;
    }
    key[tid] = kk;                                         // padding: ~0, never smaller
    __syncthreads();
    int rank = 0;
    const uint4* k4 = reinterpret_cast<const uint4*>(key);
#pragma unroll 8
    for (int c = 0; c < kPlanThreads / 4; ++c) {
      const uint4 q = k4[c];
      rank += (q.x < kk) + (q.y < kk) + (q.z < kk) + (q.w < kk);
    }
    if (tid < R) {
      tiles[rank] = tl;
      ids[rank] = tid;
    }
    __syncthreads();
    const int t = tid < R ? tiles[tid] : 0;
    int incl = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int run = incl - t;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    if (tid < R) P[tid] = run;
    if (tid == R - 1) {
      P[R] = run + t;
      plan[1] = run + t;
    }
    if (tid == 0) {
      if (R == 0) {
        P[0] = 0;
        plan[1] = 0;
      }
      plan[0] = 1;
      plan[2] = R;
      plan[3] = H;
      plan[4] = Tq;
      plan[5] = kAttnTileRows;
      plan[6] = 0;
      plan[7] = 0;
    }
    return;
  }
  int n = 1;
  while (n < R) n <<= 1;
  for (int i = tid; i < n; i += kPlanThreads) {
    uint32_t kk = ~0u;                                     // padding sorts last
    if (i < R) {
      const uint32_t L = (uint32_t)max(kv_off[i + 1] - kv_off[i], 0);
      const int64_t rows = (int64_t)max(cand_off[i + 1] - cand_off[i], 0) * Tq;
      kk = ((kLenMax - min(L, kLenMax)) << kPlanIdBits) | (uint32_t)i;
      tiles[i] = (int)((rows + kAttnTileRows - 1) / kAttnTileRows) * H;
    }
    key[i] = kk;
  }
  __syncthreads();
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = tid; i < n / 2; i += kPlanThreads) {
        const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
        const uint32_t x = key[lo], y = key[hi];
        if ((x > y) == ((lo & size) == 0)) {
          key[lo] = y;
          key[hi] = x;
        }
      }
      __syncthreads();
    }
  }
  // Thread tid owns sorted positions PER tid .. PER tid + PER - 1.
  int cnt[PER], rid[PER], tsum = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int i = PER * tid + e;
    rid[e] = i < R ? (int)(key[i] & ((1u << kPlanIdBits) - 1)) : 0;
    cnt[e] = i < R ? tiles[rid[e]] : 0;
    tsum += cnt[e];
  }
  // Block exclusive scan of the per-thread sums.
  int incl = tsum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int run = incl - tsum;
  for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int i = PER * tid + e;
    if (i < R) {
      ids[i] = rid[e];
      P[i] = run;
    }
    run += cnt[e];
  }
  if (tid == kPlanThreads - 1) {
    P[R] = run;
    plan[0] = 1;
    plan[1] = run;
    plan[2] = R;
    plan[3] = H;
    plan[4] = Tq;
    plan[5] = kAttnTileRows;
    plan[6] = 0;
    plan[7] = 0;
  }
}

template <int D, bool MAPPED, bool QPROJ = false>
hipError_t launch_fast(const AttentionArgs& a, const int32_t* cand_off, const int32_t* order,
                       hipStream_t s) {
  constexpr int W = attn_waves<D>(), TR = 32 * W;
  const int64_t slots = a.R + (a.N * a.q_len + TR - 1) / TR;
  // Few rows: 32-row tiles with the history split over the waves, while those
  // tiles fit the CUs at once (two workgroups a CU at head_dim 64, one at 128)
  // and the requests alone would not fill them (then 128-row tiles stream the
  // histories better). Measured (us, 128-row / split): one request of 203,
  // history 613, 4 x 64: 11.7 / 6.4; 16 x 200, 600, 4 x 64 (400 tiles of 32
  // rows): 12.4 / 9.5; 32 x 200 (800): 16.5 / 16.7; 1000, 2048, 8 x 128 (250):
  // 36.8 / 24.9; 64 rows x 4, 1000, 8 x 128 (512): 21.5 / 26.0; 100 requests
  // of 32 rows, 500, 4 x 64: 12.8 / 15.4.
  int cus = 0;
  const hipError_t ce = current_cu_count(&cus);
  if (ce != hipSuccess) return ce;
  if (a.N * a.q_len * a.heads <= (int64_t)kSplitRows * cus * (D == 64 ? 2 : 1) &&
      a.R * a.heads <= cus) {
    const int64_t slots32 = a.R + (a.N * a.q_len + kSplitRows - 1) / kSplitRows;
    return launch_kernel(dca_attn_split<D, MAPPED, QPROJ>, dim3((uint32_t)(slots32 * a.heads)),
                         dim3(256), s, static_cast<const bf16_t*>(a.q),
                         static_cast<const bf16_t*>(a.k), static_cast<const bf16_t*>(a.v), cand_off,
                         a.kv_offsets, static_cast<bf16_t*>(a.out), (int)a.R, a.q_len, a.heads,
                         a.kv_stride, a.scale * 1.4426950408889634f, (int)slots32, order,
                         static_cast<const bf16_t*>(a.residual), static_cast<bf16_t*>(a.out_sum),
                         static_cast<const bf16_t*>(a.proj_w));
  }
  constexpr int64_t kRound = (int64_t)kNumXcd * kPlanChunk;
  const int32_t* plan = MAPPED ? nullptr : a.plan;
  const int64_t grid = plan != nullptr ? (slots * a.heads + kRound - 1) / kRound * kRound
                                       : slots * a.heads;
  const float scale_log2 = a.scale * 1.4426950408889634f;
  if (!grid_fits(grid, 64 * W)) return hipErrorInvalidConfiguration;
  return launch_kernel(dca_attn_bf16<D, W, MAPPED, QPROJ>, dim3((uint32_t)grid), dim3(64 * W), s,
                       static_cast<const bf16_t*>(a.q), static_cast<const bf16_t*>(a.k),
                       static_cast<const bf16_t*>(a.v), cand_off, a.kv_offsets,
                       static_cast<bf16_t*>(a.out), (int)a.R, a.q_len, a.heads, a.kv_stride,
                       scale_log2, slots, order, static_cast<const bf16_t*>(a.residual),
                       static_cast<bf16_t*>(a.out_sum), static_cast<const bf16_t*>(a.proj_w),
                       plan);
}

// The mapped form on the tiled kernel: group, then attend in grouped order.
template <int D>
hipError_t launch_fast_mapped(const AttentionArgs& a, hipStream_t s) {
  int64_t G = 0;
  int nb = 0;
  if (!mapped_grouping_plan(a.R, a.N, &G, &nb)) return hipErrorInvalidValue;
  char* ws = static_cast<char*>(a.workspace);
  int32_t* grp_off = reinterpret_cast<int32_t*>(ws);
  int32_t* order = reinterpret_cast<int32_t*>(ws + align_up256((size_t)(a.R + 1) * 4));
  int32_t* hist = reinterpret_cast<int32_t*>(ws + align_up256((size_t)(a.R + 1) * 4) +
                                             align_up256((size_t)a.N * 4));
  int waves = 16, key_bits = 0;
  while (waves > 1 && waves * a.R > kGroupCounters) waves /= 2;
  while ((int64_t(1) << key_bits) < a.R) ++key_bits;
  const int32_t* base = hist;
  hipError_t e;
  // One launch while its waves' walks (N / 16 candidates each) take no longer
  // than the two launches it saves, and every request has its counters in all
  // 16 waves. Whole call (us, one launch / three), 16 requests: 4,096: 13.7 /
  // 17.7; 8,192: 18.9 / 21.1; 10,000: 19.1 / 18.2; 16,384: 23.2 / 19.5; 32,768:
  // 36.5 / 22.0; 512 requests, 8,192: 21.8 / 25.2, 10,000: 28.1 / 25.6.
  if (a.N <= kGroupWholeCands && waves == 16) {
    e = launch_kernel(group_scatter<true>, dim3(1), dim3(1024), s, a.ids, a.N, (int)a.R, a.N, 1,
                      key_bits, base, grp_off, order);
  } else {
    e = launch_kernel(group_count, dim3((uint32_t)nb), dim3(1024), s, a.ids, a.N, (int)a.R, G, nb,
                      hist);
    if (e == hipSuccess)
      e = launch_kernel(group_scan, dim3(1), dim3(1024), s, hist, a.R * (int64_t)nb, (int)a.R, nb,
                        a.N, grp_off);
    if (e == hipSuccess)
      e = launch_kernel(group_scatter<false>, dim3((uint32_t)nb), dim3(64 * waves), s, a.ids, a.N,
                        (int)a.R, G, nb, key_bits, base, grp_off, order);
  }
  if (e != hipSuccess) return e;
  return launch_fast<D, true>(a, grp_off, order, s);
}

template <typename T>
hipError_t launch_generic(const AttentionArgs& a, hipStream_t s) {
  const int64_t rows = a.N * a.q_len;
  // Rows per workgroup. Sixteen share every K and V read, but a tile takes one
  // pass per request in it, one after the other: where its rows are of many
  // requests and the chip has room, smaller tiles run the passes side by side.
  // A map in any order mixes its requests: two rows from 8 requests on. CSR
  // offsets mix them where a request has fewer than four rows: four rows, and
  // also while even those leave CUs idle. Measured (us, 16 / 4 / 2 rows, fp32,
  // 2 heads): map, 1,000 rows of 16 requests x 32, history 100: 27.9 / 15.8 /
  // 15.1; 3,000 of 1,000 x 48, 30: 40.9 / 27.3 / 29.5; 256 of 8 x 256, 5: 51.4 /
  // 26.5 / 15.1; 8,192 of 16 x 64, 200: 170 / 206 / 218; 4,000 of 16 x 256, 100:
  // 316 / 443 / 464. CSR, 4 heads: 500 of 500 x 64, 200: 94 / 42 / 49; 2 heads:
  // 1,000 of 16 x 32, 100 (126 tiles): 8.3 / 9.4; 256 of 1 x 32, 32: 4.2 / 3.7.
  int cus = 0;
  const hipError_t ce = current_cu_count(&cus);
  if (ce != hipSuccess) return ce;
  const int64_t tiles16 = (rows + 15) / 16 * a.heads;
  const bool room = a.head_dim <= 128 ? tiles16 <= 2 * cus : 2 * tiles16 <= cus;
  int tile_rows = 16;
  if (a.ids != nullptr) {
    if (a.R >= 8 && room) tile_rows = 2;
  } else if ((rows < 4 * a.R && room) || 4 * tiles16 <= cus) {
    tile_rows = 4;
  }
  const int64_t blocks = (rows + tile_rows - 1) / tile_rows;
  if (!grid_fits(blocks, 256) || a.heads > 65535) return hipErrorInvalidConfiguration;
  auto ok = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % (4 * sizeof(T)) == 0; };
  const bool vec = a.head_dim % 4 == 0 && a.kv_stride % 4 == 0 && ok(a.q) && ok(a.k) &&
                   (a.proj_w == nullptr || (ok(a.proj_w) && a.proj_in % 4 == 0));
  auto go = [&](auto kernel) {
    return launch_kernel(kernel, dim3((uint32_t)blocks, (uint32_t)a.heads), dim3(256), s,
                         static_cast<const T*>(a.q), static_cast<const T*>(a.k),
                         static_cast<const T*>(a.v), a.cand_offsets, a.kv_offsets,
                         static_cast<T*>(a.out), (int)a.R, a.q_len, rows, tile_rows, a.heads,
                         a.head_dim,
                         a.kv_stride, a.scale, a.ids, static_cast<const T*>(a.residual),
                         static_cast<T*>(a.out_sum), static_cast<const T*>(a.proj_w), a.proj_in);
  };
  if (a.head_dim <= 32) return vec ? go(dca_attn_generic<T, 32, true>) : go(dca_attn_generic<T, 32, false>);
  if (a.head_dim <= 64) return vec ? go(dca_attn_generic<T, 64, true>) : go(dca_attn_generic<T, 64, false>);
  if (a.head_dim <= 128) return vec ? go(dca_attn_generic<T, 128, true>) : go(dca_attn_generic<T, 128, false>);
  return vec ? go(dca_attn_generic<T, 256, true>) : go(dca_attn_generic<T, 256, false>);
}

}  // namespace

bool mapped_grouping_plan(int64_t R, int64_t N, int64_t* G, int* nb) {
  if (R < 1 || R > kGroupMaxRequests || N < 1) return false;
  int64_t g = 4096;
  while (R * ((N + g - 1) / g) > kGroupMaxHist && g < (int64_t(1) << 24)) g *= 2;
  const int64_t blocks = (N + g - 1) / g;
  if (R * blocks > kGroupMaxHist || blocks >= (int64_t(1) << 31)) return false;
  *G = g;
  *nb = (int)blocks;
  return true;
}

size_t mapped_grouping_bytes(int64_t R, int64_t N) {
  int64_t G = 0;
  int nb = 0;
  if (!mapped_grouping_plan(R, N, &G, &nb)) return 0;
  return align_up256((size_t)(R + 1) * 4) + align_up256((size_t)N * 4) +
         align_up256((size_t)R * (size_t)nb * 4);
}

size_t attention_plan_bytes(int64_t R) {
  return align_up256((size_t)(kPlanHeader + 2 * R + 1) * sizeof(int32_t));
}

hipError_t launch_attention_plan(const int32_t* cand_off, const int32_t* kv_off, int64_t R,
                                 int q_len, int heads, int32_t* plan, hipStream_t s) {
  return launch_kernel(attn_plan_kernel, dim3(1), dim3(kPlanThreads), s, cand_off, kv_off,
                       (int)R, q_len, heads, plan);
}

hipError_t launch_attention(const AttentionArgs& a, bool fast, hipStream_t s) {
  // The tiled kernel runs on request-contiguous candidates: the CSR offsets,
  // or a caller's per-candidate map grouped by request first (that needs the
  // grouping workspace); otherwise the general kernel runs.
  if (a.proj_w != nullptr) {
    // Fused query projection: the tiled kernel for head_dim 64 and a
    // projection input of kProjIn, the general kernel otherwise.
    if (fast && a.ids == nullptr && a.head_dim == 64 && a.proj_in == kProjIn)
      return launch_fast<64, false, true>(a, a.cand_offsets, nullptr, s);
    return a.bf16 ? launch_generic<bf16_t>(a, s) : launch_generic<float>(a, s);
  }
  if (fast && a.ids == nullptr)
    return a.head_dim == 128 ? launch_fast<128, false>(a, a.cand_offsets, nullptr, s)
                             : launch_fast<64, false>(a, a.cand_offsets, nullptr, s);
  if (fast && a.workspace != nullptr)
    return a.head_dim == 128 ? launch_fast_mapped<128>(a, s) : launch_fast_mapped<64>(a, s);
  return a.bf16 ? launch_generic<bf16_t>(a, s) : launch_generic<float>(a, s);
}

}  // namespace rocs
