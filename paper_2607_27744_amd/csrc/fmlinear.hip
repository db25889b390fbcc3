// GLM FM interaction fused into the operand of the GLM linear that consumes it
// (Eq. glm-fm-two-groups feeding Eq. glm-linear; Section 3.1, closure under
// composition; Section 4.1 decomposition of both).
//
//   Y^R_r = X^R_r (X^R_r)^T                                 once per request
//   Zb_r  = W_CR vec(Y^R_r) + b                              once per request
//   out_n = act(W_CC vec([X^C_n (X^R_{m_n})^T | X^C_n (X^C_n)^T]) + Zb_{m_n})
//
// As two operators the candidate interaction Y^C (F_c (F_r + F_c) values per
// candidate) is written to HBM and read back by the linear. Here it lives in
// LDS for one block of 32 candidates. The call is bound by memory (2 KiB of
// X^C in, 2 d_out bytes out per candidate), so the kernel is built to keep
// loads in flight all the time and everything else off the memory path:
//   - persistent workgroups, one per CU, of eight waves (two per SIMD), each
//     walking a contiguous run of 32-candidate blocks of one request each;
//   - X^C blocks (64 KiB) arrive by LDS DMA in a two-slot ring, so 64 to
//     128 KiB per CU are in flight; the block's X^R_r and Zb_r rows (from L2)
//     come the same way, one block ahead;
//   - W_CC stays in the registers of the eight waves for the whole run (64 of
//     up to 512 features a wave: 160 registers), so the linear reads only the
//     block's Y^C from LDS and no weights move after the prologue;
//   - the matrix cores do both interactions: wave i the request-candidate
//     products of field i, and two candidates' Gram blocks at a time (16 rows,
//     of which the two 8 x 8 diagonal blocks are kept).
// At 128 ragged requests, 65,536 candidates, d_out 512 the kernel takes 58 us
// (3.5 TB/s; 8 us of it the weights' way into the registers, 4.7 TB/s at d_out
// 128), where 128-candidate tiles that loaded, then computed, one workgroup
// per CU, took 105 us. A copy without any matrix instruction takes 55 us.
// Fast shape: F_r = 32, F_c = 8, E = 128 (the interaction workload), d_out a
// multiple of 64.
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace rocs {
namespace {

constexpr int kFlBN = 32;            // candidates per block
constexpr int kFlFR = 32, kFlFC = 8, kFlE = 128;
constexpr int kFlK = kFlFC * (kFlFR + kFlFC);   // 320 interaction features
constexpr int kFlSlice = 512;        // features whose weights eight waves hold
constexpr int kFlMaxD = 4096;

// Accumulator rows 8 q + 4 hh + i (q = 2 s, 2 s + 1) of one 32-row block,
// packed to bf16 and exchanged between the wave halves: afterwards lane
// (l32, hh) holds rows 16 s + 8 hh .. + 7 of its column, in order.
__device__ __forceinline__ u32x4 fl_swap(const f32x16& acc, int s) {
  const uint32_t e0 = pack_bf16x2(acc[8 * s], acc[8 * s + 1]);
  const uint32_t e1 = pack_bf16x2(acc[8 * s + 2], acc[8 * s + 3]);
  const uint32_t o0 = pack_bf16x2(acc[8 * s + 4], acc[8 * s + 5]);
  const uint32_t o1 = pack_bf16x2(acc[8 * s + 6], acc[8 * s + 7]);
  const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
  const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
  return u32x4{s0[0], s1[0], s0[1], s1[1]};
}

// One block of candidates. Request r owns block slots r + floor(off[r] / 32)
// .. (tile_base); all values are wave-uniform.
struct FlBlock {
  int slot, r, n0, rows;
  bool live;
};

// Move `c` forward to the first slot below `end` that holds candidates.
__device__ __forceinline__ void fl_seek(FlBlock& c, int end,
                                        const __attribute__((address_space(4))) int32_t* off,
                                        int R) {
  for (; c.slot < end; ++c.slot) {
    while (c.r + 1 < R && c.r + 1 + off[c.r + 1] / kFlBN <= c.slot) ++c.r;
    const int first = off[c.r], stop = off[c.r + 1];
    const int at = first + (c.slot - c.r - first / kFlBN) * kFlBN;
    if (at < stop) {
      c.n0 = at;
      c.rows = min(kFlBN, stop - at);
      c.live = true;
      return;
    }
  }
  c.live = false;
}

// FB: 32-feature blocks per wave (2: slices of up to 512 features, 1: up to
// 256). Workgroup b works on feature slice b % n_slices (slice_w features, a
// multiple of 64) and on run b / n_slices of the block slots.
template <int FB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void glm_fm_linear_bf16(const bf16_t* __restrict__ xr, const bf16_t* __restrict__ xc,
                        const float* __restrict__ zb, const bf16_t* __restrict__ w,
                        const int32_t* __restrict__ off_g, int R, int D, int slice_w,
                        int n_slices, int n_slots, int relu, bf16_t* __restrict__ out) {
  constexpr int FC = kFlFC, E = kFlE, K = kFlK;
  constexpr int XROW = FC * E * 2;              // bytes of one candidate (2048)
  constexpr int XB = kFlBN * XROW;              // one X^C ring slot (64 KiB)
  constexpr int YROW = K * 2;                   // bytes of one Y^C row (640)
  constexpr int YO = 2 * XB;                    // Y^C of the block
  constexpr int RO = YO + kFlBN * YROW;         // X^R of the block's request
  constexpr int ZO = RO + kFlFR * E * 2;        // Zb slice, two buffers by block parity
  constexpr int ZB = 4 * kFlSlice;
  constexpr int KQ = K / 16;                    // k-steps of the linear (20)
  constexpr int NX = XB / 1024 / 8;             // X^C DMA loads per wave and block (8)
  static_assert(ZO + 2 * ZB <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char lds[ZO + 2 * ZB];
  ROCS_LDS char* const lds3 = (ROCS_LDS char*)lds;
  const __attribute__((address_space(4))) int32_t* off =
      (const __attribute__((address_space(4))) int32_t*)off_g;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5, l16 = lane & 15, g4 = lane >> 4;
  const uint32_t lbase = lds_addr(lds);
  // Runs next to each other, and a run's slices, share an XCD.
  const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
  const int runs = (int)gridDim.x / n_slices, run = b / n_slices;
  const int f0 = (b % n_slices) * slice_w;                  // the slice's first feature
  const int fw = f0 + 32 * FB * wave;                       // this wave's first feature
  const bool active = fw < min(f0 + slice_w, D);
  FlBlock cur{(int)((int64_t)n_slots * run / runs), 0, 0, 0, false};
  const int slot_end = (int)((int64_t)n_slots * (run + 1) / runs);
  if (cur.slot >= slot_end) return;
  cur.r = request_of_slot(off_g, R, cur.slot, 1, kFlBN);
  fl_seek(cur, slot_end, off, R);
  if (!cur.live) return;

  // DMA. X^C: wave w fills candidates 4 w .. 4 w + 3, half a candidate per
  // load; 16-byte chunk ch of field f of candidate c sits at chunk position
  // ch ^ (c % 16) ^ 2 f of its 256-byte field row, so that both the 16
  // candidates of one field and the 16 field rows of two candidates fall on
  // distinct banks at one chunk. Candidates past the block's end repeat the
  // last one.
  auto issue_x = [&](const FlBlock& c, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      const int cand = 4 * wave + j / 2;
      const int f = 4 * (j % 2) + g4;
      const char* src = reinterpret_cast<const char*>(xc) +
                        (int64_t)(c.n0 + min(cand, c.rows - 1)) * XROW;
      lds_dma16_sv(src, (uint32_t)(f * 256 + 16 * (l16 ^ (cand & 15) ^ (2 * f))),
                   lbase + (uint32_t)(buf * XB + cand * XROW + 1024 * (j % 2)));
    }
  };
  // X^R_r (rows swizzled by row % 16) and this wave's part of the Zb slice.
  auto issue_request = [&](const FlBlock& c, int par) __attribute__((always_inline)) {
    const int row = 4 * wave + g4;
    lds_dma16_sv(xr + (int64_t)c.r * kFlFR * E, (uint32_t)(row * 256 + 16 * (l16 ^ (row & 15))),
                 lbase + (uint32_t)(RO + 1024 * wave));
    if (active && lane < 8 * FB)
      lds_dma16_sv(zb + (int64_t)c.r * D + fw, (uint32_t)(16 * lane),
                   lbase + (uint32_t)(ZO + par * ZB + 128 * FB * wave));
  };

  // Weights: rows fw + 32 fm + l32, features 16 q + 8 hh .. of Y^C. Resident
  // before the ring starts: the loop then has no load that the compiler
  // tracks, so it adds no waits of its own there.
  bf16x8 wf[FB][KQ];
  if (active) {
#pragma unroll
    for (int fm = 0; fm < FB; ++fm)
#pragma unroll
      for (int q = 0; q < KQ; ++q)
        wf[fm][q] = *reinterpret_cast<const bf16x8*>(w + (int64_t)(fw + 32 * fm + l32) * K +
                                                     16 * q + 8 * hh);
  }
  issue_x(cur, 0);
  issue_request(cur, 0);
  FlBlock nxt = cur;
  ++nxt.slot;
  fl_seek(nxt, slot_end, off, R);
  if (nxt.live) issue_x(nxt, 1);
  if (active) {
#pragma unroll
    for (int fm = 0; fm < FB; ++fm)
#pragma unroll
      for (int q = 0; q < KQ; ++q) asm volatile("" :: "v"(as_u32x4(wf[fm][q])));
  }
  if (nxt.live) wait_vmcnt<NX>(); else wait_vmcnt<0>();
  const uint32_t lo = act_floor(relu);
  int buf = 0, par = 0;
  while (true) {
    ring_barrier();            // X^C, X^R, Zb of `cur` in; Y^C free
    // The loop's LDS addresses come from a laundered lane index: derived from
    // `lane`, they would be hoisted and held beside the 160 weight registers.
    int lz = lane;
    asm volatile("" : "+v"(lz));
    const int c32 = lz & 31, h2 = lz >> 5, c16 = lz & 15, q4 = lz >> 4;
    const uint32_t ysw = (uint32_t)((c32 >> 1) & 7);        // Y^C rows: chunk ^ (row / 2 % 8)
    const uint32_t yrow = (uint32_t)(YO + c32 * YROW);
    {
      // Request-candidate products of field `wave`: P^T[j][c] = <x^R_j, x^C_c>.
      // A k-step is an XOR with 32 s within the 256-byte field row.
      const uint32_t ra = (uint32_t)(RO + c32 * 256 + 16 * (h2 ^ (c32 & 15)));
      const uint32_t xa = (uint32_t)(buf * XB + c32 * XROW + wave * 256 +
                                     16 * (h2 ^ (c32 & 15) ^ (2 * wave)));
      f32x16 p = {};
#pragma unroll
      for (int s = 0; s < E / 16; ++s) {
        const bf16x8 a = *reinterpret_cast<const ROCS_LDS bf16x8*>(lds3 + (ra ^ (32u * s)));
        const bf16x8 x = *reinterpret_cast<const ROCS_LDS bf16x8*>(lds3 + (xa ^ (32u * s)));
        p = mfma32(a, x, p);
      }
      // Gram blocks of candidates 4 wave .. 4 wave + 3, two at a time.
      f32x4 cc[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = 4 * wave + 2 * u + (c16 >> 3), f = c16 & 7;
        const uint32_t ga = (uint32_t)(buf * XB + c * XROW + f * 256 +
                                       16 * (q4 ^ (c & 15) ^ (2 * f)));
        cc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < E / 32; ++s) {
          const bf16x8 x = *reinterpret_cast<const ROCS_LDS bf16x8*>(lds3 + (ga ^ (64u * s)));
          cc[u] = mfma16(x, x, cc[u]);
        }
      }
      // Features 40 wave + 16 s + 8 hh .. of candidate l32: one 16-byte chunk.
#pragma unroll
      for (int s = 0; s < 2; ++s)
        *reinterpret_cast<ROCS_LDS u32x4*>(
            lds3 + yrow + 16 * ((uint32_t)(5 * wave + 2 * s + h2) ^ ysw)) = fl_swap(p, s);
      // cc[u][i] = <field 4 (q4 % 2) + i, field c16 % 8> where both rows are
      // one candidate's: features 40 (c16 % 8) + 32 + 4 (q4 % 2) ..
      if ((q4 >> 1) == (c16 >> 3)) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int c = 4 * wave + 2 * u + (c16 >> 3);
          *reinterpret_cast<ROCS_LDS u32x2*>(
              lds3 + YO + c * YROW + 16 * ((5 * (c16 & 7) + 4) ^ ((c >> 1) & 7)) + 8 * (q4 & 1)) =
              u32x2{pack_bf16x2(cc[u][0], cc[u][1]), pack_bf16x2(cc[u][2], cc[u][3])};
        }
      }
    }
    wait_lgkmcnt0();
    ring_barrier();            // Y^C complete; this X^C slot and X^R free
    FlBlock nn = nxt;
    if (nxt.live) {
      issue_request(nxt, par ^ 1);
      ++nn.slot;
      fl_seek(nn, slot_end, off, R);
      if (nn.live) issue_x(nn, buf);
    }
    if (active) {
      f32x16 acc[FB];
#pragma unroll
      for (int fm = 0; fm < FB; ++fm)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 z = *reinterpret_cast<const ROCS_LDS f32x4*>(
              lds3 + ZO + par * ZB + 128 * FB * wave + 16 * h2 + 4 * (32 * fm + 8 * q));
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[fm][4 * q + i] = z[i];
        }
      // Chunk 2 q + hh of the row: its low three bits swizzled, the rest a
      // constant offset.
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        const bf16x8 y = *reinterpret_cast<const ROCS_LDS bf16x8*>(
            lds3 + yrow + 16 * ((uint32_t)(2 * (q & 3) + h2) ^ ysw) + 128 * (q >> 2));
#pragma unroll
        for (int fm = 0; fm < FB; ++fm) acc[fm] = mfma32(wf[fm][q], y, acc[fm]);
      }
      // bf16, activation, stores. fl_swap leaves the lanes of one candidate
      // with 16-byte pieces 32 bytes apart; exchanging 16-lane rows between
      // the two pieces puts four lanes on 64 contiguous bytes (1 us less at
      // 65,536 candidates). Store i takes candidates 16 i .. + 15, and is
      // skipped where there are none: the waits below count them.
      bf16_t* op = out + (int64_t)(cur.n0 + c16) * D + fw + 16 * (q4 & 1) + 8 * h2;
#pragma unroll
      for (int fm = 0; fm < FB; ++fm) {
        const u32x4 s0 = fl_swap(acc[fm], 0), s1 = fl_swap(acc[fm], 1);
        u32x4 o[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const auto t = __builtin_amdgcn_permlane16_swap(act_bf16x2(s0[e], lo),
                                                          act_bf16x2(s1[e], lo), false, false);
          o[0][e] = t[0];
          o[1][e] = t[1];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (16 * i + c16 < cur.rows)
            *reinterpret_cast<u32x4*>(op + (int64_t)(16 * i) * D + 32 * fm) = o[i];
      }
    }
    if (!nxt.live) break;
    // The next block's X^C, X^R and Zb: everything but the loads of the block
    // after it and this block's stores, which were issued later.
    if (!nn.live) {
      wait_vmcnt<0>();
    } else if (!active) {
      wait_vmcnt<NX>();
    } else if (cur.rows > 16) {
      wait_vmcnt<NX + 2 * FB>();
    } else {
      wait_vmcnt<NX + FB>();
    }
    cur = nxt;
    nxt = nn;
    buf ^= 1;
    par ^= 1;
  }
}

// ---------------------------------------------------------------------------
// Request side in one launch: Y^R = X^R (X^R)^T (rounded to bf16) and Zb =
// W_CR vec(Y^R) + b. One workgroup per 16 requests x 16 features: its four
// waves form the 16 requests' Y^R in LDS (one 32 x 32 product over E each, the
// same registers as both operands), then split its 1024 features as the K of
// the Zb tile and reduce through LDS in a fixed order. Every feature tile
// forms Y^R again (128 KiB of X^R from L2): at 128 requests, d_out 512, that
// costs less than the second launch it saves (8 us against 4.5 + 6 and a gap).
// The first feature tile writes Y^R out.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fm_request_bf16(
    const bf16_t* __restrict__ xr, const bf16_t* __restrict__ w, const float* __restrict__ bias,
    bf16_t* __restrict__ y_req, float* __restrict__ z, int R, int D) {
  constexpr int E = kFlE, K = kFlFR * kFlFR, ROW = 2 * K;
  constexpr int KS = K / 128;              // 32-wide k-steps per wave
  __shared__ __attribute__((aligned(16))) char ly[16 * ROW];
  __shared__ f32x4 red[4 * kWave];
  ROCS_LDS char* const y3 = (ROCS_LDS char*)ly;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, hh = lane >> 5, l16 = lane & 15, g4 = lane >> 4;
  const int tiles_d = D / 16;
  const int r0 = ((int)blockIdx.x / tiles_d) * 16, d0 = ((int)blockIdx.x % tiles_d) * 16;
  bf16x8 wf[KS];                           // W_CR row d0 + l16, k = 128 s + 32 wave + 8 g4 ..
  const bf16_t* wp = w + (int64_t)(d0 + l16) * K + 32 * wave + 8 * g4;
#pragma unroll
  for (int s = 0; s < KS; ++s) wf[s] = *reinterpret_cast<const bf16x8*>(wp + 128 * s);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int rr = 4 * wave + u;
    const bf16_t* xp = xr + (int64_t)min(r0 + rr, R - 1) * kFlFR * E + l32 * E + 8 * hh;
    bf16x8 x[E / 16];
#pragma unroll
    for (int s = 0; s < E / 16; ++s) x[s] = *reinterpret_cast<const bf16x8*>(xp + 16 * s);
    f32x16 p = {};
#pragma unroll
    for (int s = 0; s < E / 16; ++s) p = mfma32(x[s], x[s], p);
    // Y^R[l32][16 s + 8 hh ..] (symmetric): 16-byte chunk 4 l32 + 2 s + hh of
    // the request's row, at chunk position ^ rr.
#pragma unroll
    for (int s = 0; s < 2; ++s)
      *reinterpret_cast<ROCS_LDS u32x4*>(y3 + rr * ROW + 16 * ((4 * l32 + 2 * s + hh) ^ rr)) =
          fl_swap(p, s);
  }
  __syncthreads();
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const bf16x8 y = *reinterpret_cast<const ROCS_LDS bf16x8*>(
        y3 + l16 * ROW + 16 * ((16 * s + 4 * wave + g4) ^ l16));
    acc = mfma16(wf[s], y, acc);           // acc[i] = Zb[r0 + l16][d0 + 4 g4 + i]
  }
  red[wave * kWave + lane] = acc;
  if (d0 == 0) {
    for (int c = threadIdx.x; c < 16 * (K / 8); c += 256) {
      const int rr = c / (K / 8), ch = c % (K / 8);
      if (r0 + rr < R)
        *reinterpret_cast<u32x4*>(y_req + (int64_t)(r0 + rr) * K + 8 * ch) =
            *reinterpret_cast<const ROCS_LDS u32x4*>(y3 + rr * ROW + 16 * (ch ^ rr));
    }
  }
  __syncthreads();
  if (wave == 0 && r0 + l16 < R) {
    f32x4 s = ((red[lane] + red[kWave + lane]) + red[2 * kWave + lane]) + red[3 * kWave + lane];
    const int d = d0 + 4 * g4;
    if (bias != nullptr) s += *reinterpret_cast<const f32x4*>(bias + d);
    *reinterpret_cast<f32x4*>(z + (int64_t)(r0 + l16) * D + d) = s;
  }
}

}  // namespace

bool fm_linear_fused_shape(int f_req, int f_cand, int emb, int64_t d_out) {
  return f_req == kFlFR && f_cand == kFlFC && emb == kFlE && d_out % 64 == 0 &&
         d_out <= kFlMaxD;
}

hipError_t launch_fm_linear(const FmLinearArgs& a, bool fused, hipStream_t s) {
  if (!fused) {
    InteractionArgs ia{};
    ia.x_req = a.x_req; ia.x_cand = a.x_cand; ia.cand_offsets = a.cand_offsets;
    ia.R = a.R; ia.N = a.N; ia.f_req = a.f_req; ia.f_cand = a.f_cand; ia.emb = a.emb;
    ia.bf16 = a.bf16; ia.y_req = a.y_req; ia.y_cand = a.y_cand;
    const hipError_t e = launch_interaction(ia, a.interaction_fast, s);
    if (e != hipSuccess) return e;
    LinearArgs l{};
    l.x_req = a.y_req; l.x_cand = a.y_cand; l.w_req = a.w_req; l.w_cand = a.w_cand;
    l.bias = a.bias; l.cand_offsets = a.cand_offsets;
    l.R = a.R; l.N = a.N; l.k_req = (int64_t)a.f_req * a.f_req;
    l.k_cand = (int64_t)a.f_cand * (a.f_req + a.f_cand); l.d_out = a.d_out;
    l.bf16 = a.bf16; l.relu = a.relu; l.out = a.out; l.z = a.z; l.ids = a.ids;
    return launch_linear(l, a.linear_fast, s);
  }
  const int64_t req_tiles = (a.R + 15) / 16 * (a.d_out / 16);
  if (!grid_fits(req_tiles, 256)) return hipErrorInvalidConfiguration;
  hipError_t e = launch_kernel(fm_request_bf16, dim3((uint32_t)req_tiles), dim3(256), s,
                               static_cast<const bf16_t*>(a.x_req),
                               static_cast<const bf16_t*>(a.w_req), a.bias,
                               static_cast<bf16_t*>(a.y_req), a.z, (int)a.R, (int)a.d_out);
  if (e != hipSuccess || a.N == 0) return e;
  int cus = 0;
  e = current_cu_count(&cus);
  if (e != hipSuccess) return e;
  const int64_t slots = a.R + (a.N + kFlBN - 1) / kFlBN;
  if (slots >= (int64_t(1) << 31)) return hipErrorInvalidConfiguration;
  // Slices of at most 512 features (the registers of one workgroup), equal to
  // within 64; every slice reads X^C again, at about the same time on the
  // same XCD. A call of few blocks takes more slices while CUs are idle: a
  // workgroup's first 512 features of weights take 8 us, as long as two blocks.
  int ns = (int)((a.d_out + kFlSlice - 1) / kFlSlice);
  while (slots * ns * 2 <= cus && a.d_out / (ns * 2) >= 64) ns *= 2;
  const int sw = (int)((a.d_out / 64 + ns - 1) / ns * 64);
  const int64_t runs = cus / ns < 1 ? 1 : cus / ns;
  const int grid = (int)(slots < runs ? slots : runs) * ns;
  auto go = [&](auto kernel) {
    return launch_kernel(kernel, dim3((uint32_t)grid), dim3(512), s,
                         static_cast<const bf16_t*>(a.x_req), static_cast<const bf16_t*>(a.x_cand),
                         static_cast<const float*>(a.z), static_cast<const bf16_t*>(a.w_cand),
                         a.cand_offsets, (int)a.R, (int)a.d_out, sw, ns, (int)slots,
                         (int)a.relu, static_cast<bf16_t*>(a.out));
  };
  return sw > kFlSlice / 2 ? go(glm_fm_linear_bf16<2>) : go(glm_fm_linear_bf16<1>);
}

}  // namespace rocs
