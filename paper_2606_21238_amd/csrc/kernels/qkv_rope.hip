// Producer of the computed tokens' Q/K/V: projection of their hidden states and rotary
// position embedding (the attention inputs of a prefill; the paper serves Qwen3-14B, Sec. 4,
// and the layer details follow its public configuration).
//
//   y = x W^T            x [T][H] bf16, W [(Hq + 2 Hkv) D][H] bf16, y rounded to bf16
//   q, k = rotary(y_q, y_k) at each token's absolute position; v = y_v
//
// One kernel does the projection and the rotation, so y never goes to memory:
//  * qkv_gemm_rope_kernel (prefill batches): 256-, 192- or 128-token x 256-output tiles, 4 waves,
//    one per SIMD, rotation in registers;
//  * qkv_ksplit_kernel (decode steps, short questions): 32- or 64-token x 32- or 64-output tiles
//    whose waves split H.
// Both use v_mfma_f32_32x32x16_bf16 and stream x and W global -> LDS with 16-byte direct loads
// (SGPR base + 32-bit lane offsets) in stages of 64 columns of H, so that every load instruction
// takes whole 128-byte lines of 8 rows (stages of 32 columns, half lines, measured 53 us against
// 41 for 16 tokens x 8192 x 10240, where W comes from HBM).  A row's 16-byte chunk c is stored at
// c ^ ((row / 2) % 8), so 16 lanes of an operand read hit 16 different 16-byte slots of the banks.
// The (cos, sin) pairs of a token (D/2 angles p * theta^(-2i/D), in fp64 reduced mod 2 pi, then
// fp32 sine and cosine) come from a small pre-pass into the caller's workspace for the first
// kernel; the second computes its tile's own.  A token's position is found from cu_q / seq_lens
// (suffix token i of request r sits at L_r - S_r + i).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "../host/internal.hpp"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kTN = 256;        // outputs per work-group tile of the prefill kernel
constexpr int kKC = 64;         // columns of H per stage (the last stage may hold 32)
constexpr int kGroupTokens = 1024;   // tokens per group of the tile order

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {  // nearest even; inputs finite
  const uint32_t u = __builtin_bit_cast(uint32_t, f);
  return static_cast<uint16_t>((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {  // nearest even, one instruction
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __builtin_bit_cast(float, static_cast<uint32_t>(b) << 16);
}

// 16 bytes per lane from global memory straight into LDS: lane l reads base + ofs_l and
// writes LDS bytes [M0 + 16 l, M0 + 16 l + 16); the kernel counts these loads itself with
// vmcnt.  The SGPR base + 32-bit offset form halves the address traffic of 64-bit lane
// addresses.
__device__ __forceinline__ void load_lds16(const void* base, uint32_t ofs, lds_void* l) {
  const uint32_t m = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(l));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(ofs), "s"(base), "s"(m)
               : "memory", "m0");
}

// 4 bytes per lane from global memory (a 64-bit address per lane) into LDS bytes [M0 + 4 l, + 4).
__device__ __forceinline__ void load_lds4(const void* g, lds_void* l) {
  const uint32_t m = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(l));
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(g), "s"(m) : "memory", "m0");
}

// (cos, sin) of every token's D/2 rotary angles: tab[t][i], i < D/2.  A work-group computes
// the D/2 frequencies once (fp64 pow) and then walks tokens grid-stride, 256 / (D/2) at a
// time; the angle p f is reduced mod 2 pi in fp64 (k = floor(a / 2 pi), a - 2 pi k in one
// fma), then fp32 sine and cosine.
constexpr int kTableBlocks = 1024;
template <int D>
__global__ __launch_bounds__(256) void rope_table_kernel(int64_t n_tokens, const int32_t* __restrict__ cu_q,
                                                          const int32_t* __restrict__ seq_lens, int n_reqs,
                                                          double theta, float2* __restrict__ tab) {
  constexpr int HALF = D / 2;
  constexpr int kTokPer = 256 / HALF;     // tokens per pass of the work-group
  constexpr double kTwoPi = 6.283185307179586476925;
  __shared__ double freq[HALF];
  if (threadIdx.x < HALF) freq[threadIdx.x] = std::pow(theta, -2.0 * static_cast<int>(threadIdx.x) / D);
  __syncthreads();
  const int i = threadIdx.x % HALF;
  const double f = freq[i];
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * kTokPer + threadIdx.x / HALF; t < n_tokens;
       t += static_cast<int64_t>(gridDim.x) * kTokPer) {
    int lo = 0, hi = n_reqs - 1;          // request of token t: the last r with cu_q[r] <= t
    while (lo < hi) {
      const int mid = (lo + hi + 1) / 2;
      if (cu_q[mid] <= t) lo = mid; else hi = mid - 1;
    }
    const int64_t p = static_cast<int64_t>(seq_lens[lo]) - (cu_q[lo + 1] - cu_q[lo]) + (t - cu_q[lo]);
    const double a = static_cast<double>(p) * f;
    const double r = std::fma(-std::floor(a / kTwoPi), kTwoPi, a);
    float sn, cs;
    sincosf(static_cast<float>(r), &sn, &cs);
    tab[t * HALF + i] = make_float2(cs, sn);
  }
}

// Stores a finished TM x TN tile of y (bf16 in LDS at ep, [token][output], rows `pitch` bytes
// apart): every thread takes 16-byte chunks of a token's head and stores them whole.  ROT: the
// tile is not rotated yet; query and key chunks are rotated here against the chunk `partner`
// local columns away.  col(o): the output (head * D + dim) of local column o (chunks of 8 are
// consecutive outputs); cs_of(row, i): the (cos, sin) pairs of dims i .. i + 7 of tile row `row`.
// POOL: K and V go straight into the paged pools (layout V1; k_out and v_out are then the
// pools) at the tile's slots (tslot, -1 past the last token) instead of into [token][head][dim]
// rows: K rows as 16-byte chunks, V (dim-major blocks) as 8 consecutive tokens of one dim per
// 16-byte store where the 8 tokens hold 8 aligned consecutive slots, else one 2-byte store per
// token.  Slots outside [0, n_slots) are skipped, as the scatter does.
template <int D, bool POOL, bool ROT, int TM, int TN, int THREADS, class Col, class Cs>
__device__ __forceinline__ void store_tile(const char* ep, int pitch, int t0, int n_tokens, Col col, int n_out,
                                           int partner, Cs cs_of, const int32_t* tslot, int hq, int hkv,
                                           uint16_t* __restrict__ q_out, uint16_t* __restrict__ k_out,
                                           uint16_t* __restrict__ v_out, int64_t n_slots) {
  const int tid = threadIdx.x;
  const int nrot = (hq + hkv) * D;
#pragma unroll 4
  for (int qc = tid; qc < TM * TN / 8; qc += THREADS) {
    const int row = qc / (TN / 8), o = (qc % (TN / 8)) * 8;
    const int t = t0 + row, n = col(o);
    if (t >= n_tokens || n >= n_out) continue;
    if (POOL && n >= nrot) continue;               // V: the pass below
    const int head = n / D, i0 = n % D;
    const u32x4_t own = *reinterpret_cast<const u32x4_t*>(ep + row * pitch + o * 2);
    u32x4_t res = own;
    if (ROT && n < nrot) {
      const bool lo = i0 < D / 2;
      const u32x4_t par = *reinterpret_cast<const u32x4_t*>(ep + row * pitch + (lo ? o + partner : o - partner) * 2);
      const float4* cs = cs_of(row, lo ? i0 : i0 - D / 2);
      const float sg = lo ? -1.f : 1.f;      // lo: a c - b s; hi: a c + b s (a own, b partner)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 c2 = cs[j];             // (cos, sin) of elements 2j and 2j + 1
        const float a0 = bf16_to_f32(own[j] & 0xFFFF), a1 = bf16_to_f32(own[j] >> 16);
        const float b0 = bf16_to_f32(par[j] & 0xFFFF), b1 = bf16_to_f32(par[j] >> 16);
        const uint32_t o0 = f32_to_bf16(a0 * c2.x + sg * (b0 * c2.y));
        const uint32_t o1 = f32_to_bf16(a1 * c2.z + sg * (b1 * c2.w));
        res[j] = o0 | (o1 << 16);
      }
    }
    uint16_t* dst;
    if (head < hq) {
      dst = q_out + (static_cast<int64_t>(t) * hq + head) * D + i0;
    } else if (head < hq + hkv) {
      if constexpr (POOL) {
        const int32_t sl = tslot[row];
        if (sl < 0 || sl >= n_slots) continue;
        dst = k_out + ((static_cast<int64_t>(sl >> 4) * hkv + head - hq) * 16 + (sl & 15)) * D + i0;
      } else {
        dst = k_out + (static_cast<int64_t>(t) * hkv + head - hq) * D + i0;
      }
    } else {
      dst = v_out + (static_cast<int64_t>(t) * hkv + head - hq - hkv) * D + i0;
    }
    *reinterpret_cast<u32x4_t*>(dst) = res;
  }
  if constexpr (POOL) {
    // V columns of the tile into the dim-major pool: item p is 8 tokens (rows 8 g .. 8 g + 7)
    // of one output column; consecutive threads take consecutive columns of the same tokens.
    if (col(TN - 1) >= nrot) {                                    // uniform
#pragma unroll 2
      for (int p = tid; p < (TM / 8) * TN; p += THREADS) {
        const int g = p / TN, oc = p % TN;
        const int n = col(oc), tf = t0 + 8 * g;
        if (n < nrot || n >= n_out || tf >= n_tokens) continue;
        const int vh = (n - nrot) / D, dim = (n - nrot) % D;
        int32_t sl[8];
        uint16_t val[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          sl[j] = tslot[8 * g + j];                               // -1 past the last token
          val[j] = *reinterpret_cast<const uint16_t*>(ep + (8 * g + j) * pitch + oc * 2);
        }
        bool run = (sl[0] & 7) == 0 && sl[0] >= 0 && sl[0] + 7 < n_slots;
#pragma unroll
        for (int j = 1; j < 8; ++j) run = run && sl[j] == sl[0] + j;
        if (run) {     // 8 aligned consecutive slots: one block, one 16-byte row segment
          u32x4_t v;
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = static_cast<uint32_t>(val[2 * j]) | (static_cast<uint32_t>(val[2 * j + 1]) << 16);
          *reinterpret_cast<u32x4_t*>(v_out + ((static_cast<int64_t>(sl[0] >> 4) * hkv + vh) * D + dim) * 16 +
                                      (sl[0] & 15)) = v;
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (sl[j] >= 0 && sl[j] < n_slots)
              v_out[((static_cast<int64_t>(sl[j] >> 4) * hkv + vh) * D + dim) * 16 + (sl[j] & 15)] = val[j];
        }
      }
    }
  }
}

// Prefill batches.  A work-group of 4 waves, one per SIMD, computes TM = 64 MB tokens x 256
// outputs of y, each wave 32 MB tokens x 128 outputs.  What bounds it: LDS traffic and the load
// latency first, the chip's power then (1.8 GHz under this load).  128 x 128 wave tiles read 0.5
// KiB of operands per MFMA (the 64 x 128 tiles of an 8-wave work-group 0.75 KiB, which with the
// tile writes took every LDS cycle the MFMAs left); with one wave per SIMD the accumulators
// (256 registers) and two sets of operands fit, so a step's MFMAs run with the next step's
// operand reads and the loads between them, one barrier per 64 columns.  x tiles have a ring
// of three stages; W tiles of WS = 2 at TM = 256 (160 KiB in all) and 192 (136 KiB), where a stage
// takes as long as a load, and of 3 at TM = 128 (144 KiB): its stages are half as long, and W
// requested 3/4 of a stage ahead bound them (907 tokens x 5120 x 7168: 91.7 us with 2, 80.7 with 3;
// 512 x 8192 x 10240: 129 and 112).
//
// Stage s, four steps of 16 columns (the operands of a step are read during the step before):
//   step 0       requests x(s + 2), into the buffer of x(s - 1)
//   after step 2 this wave's reads of stage s have returned and its loads of stage s + 1 are
//                complete (x(s + 2), and W(s + 2) with WS = 3, may be pending); barrier
//   step 3       requests W(s + WS), into the buffer of W(s); reads step 0 of stage s + 1
// Stages past the end are requested as copies of the last one, into buffers nobody reads any
// more, which keeps the counts constant.
//
// W is the MFMA's first operand, so a lane holds one token and its registers run over the
// outputs: both members of a rotary pair are in one lane, the rotation needs no exchange, and
// four consecutive outputs go to LDS as one 8-byte write.  The tile then leaves as whole
// 16-byte chunks of contiguous rows.  (With the tile rounded and written by 2-byte stores and
// rotated on the way out, the epilogue took 37 us of a tile's 129.)
template <int D, bool POOL, int MB>
__global__ __launch_bounds__(256, 1) void qkv_gemm_rope_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ w, int n_tokens, int hidden,
    int n_out, int hq, int hkv, const float2* __restrict__ tab, uint16_t* __restrict__ q_out,
    uint16_t* __restrict__ k_out, uint16_t* __restrict__ v_out, const int32_t* __restrict__ slots,
    int64_t n_slots) {
  constexpr int TM = 64 * MB;
  constexpr int XB = TM * kKC * 2, WB = kTN * kKC * 2;  // bytes of an x and of a W stage
  constexpr int XL = TM / 32, WL = kTN / 32;            // 1 KiB loads per wave of each (8 rows)
  static_assert(XL <= 2 * MB, "every x load has its place in step 0");
  constexpr int kPitch = kTN * 2 + 16;
  constexpr int WS = MB == 2 ? 3 : 2;                   // stages of the W ring
  constexpr int kRing = 3 * XB + WS * WB, kEnd = TM * kPitch + TM * 4;
  __shared__ __attribute__((aligned(1024))) char smem[kRing > kEnd ? kRing : kEnd];  // rings, then y and slots
  // Tile order.  Work-groups are dealt to the 8 XCDs in turn (b -> XCD b % 8) and each XCD has
  // its own L2, so logical tile L = (b % 8) * (G / 8) + b / 8 gives every XCD a contiguous run
  // of tiles; runs go over groups of kGroupTokens tokens output-tile by output-tile, so the
  // ~32 tiles one XCD holds at a time share their x tiles and 8 (4) W tiles in its L2.
  constexpr int kGroupM = kGroupTokens / TM;
  const int n_tiles_n = n_out / kTN + (n_out % kTN ? 1 : 0);
  const int n_tiles_m = n_tokens / TM + (n_tokens % TM ? 1 : 0);
  const int b = blockIdx.x, full = gridDim.x & ~7;
  const int L = b < full ? (b % 8) * (full / 8) + b / 8 : b;
  const int group = L / (kGroupM * n_tiles_n), in_group = L % (kGroupM * n_tiles_n);
  const int first_m = group * kGroupM, gm = min(n_tiles_m - first_m, kGroupM);
  const int tile_m = first_m + in_group % gm, tile_n = in_group / gm;
  const int t0 = tile_m * TM, n0 = tile_n * kTN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hg = lane >> 5;
  const int row0 = (wave & 1) * (32 * MB);              // the wave's tokens of the tile
  const int col0 = (wave >> 1) * 128;                   // the wave's 128 outputs

  // ---- loads: piece i of a wave covers rows 32 i + 8 wave .. + 7 of a tile --------------------
  uint32_t xofs[XL], wofs[WL];                          // byte offsets from the tile's first row
  const int c_ld = (lane % 8) ^ (((8 * wave + lane / 8) >> 1) & 7);   // chunk of the row (the same for every i)
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int t = min(t0 + 32 * i + 8 * wave + lane / 8, n_tokens - 1) - t0;
    xofs[i] = static_cast<uint32_t>(t * hidden + c_ld * 8) * 2u;
  }
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int n = min(n0 + 32 * i + 8 * wave + lane / 8, n_out - 1) - n0;
    wofs[i] = static_cast<uint32_t>(n * hidden + c_ld * 8) * 2u;
  }
  const uint16_t* xbase = x + static_cast<int64_t>(t0) * hidden;
  const uint16_t* wbase = w + static_cast<int64_t>(n0) * hidden;
  const int n_full = hidden / kKC, n_st = (hidden + kKC - 1) / kKC;
  // the last stage of a hidden size that is no multiple of 64 holds 32 columns: its upper chunks
  // repeat the lower ones (never used), so no lane reads past a row's end
  const uint32_t hi64 = c_ld >= 4 ? 64u : 0u;
  auto back = [&](int s) -> uint32_t { return s >= n_full ? hi64 : 0u; };
  auto issue_x = [&](int s, int buf, int i) __attribute__((always_inline)) {
    const int sc = min(s, n_st - 1);
    load_lds16(xbase + sc * kKC, xofs[i] - back(sc), (lds_void*)(smem + buf * XB + (32 * i + 8 * wave) * 128));
  };
  auto issue_w = [&](int s, int buf, int i) __attribute__((always_inline)) {
    const int sc = min(s, n_st - 1);
    load_lds16(wbase + sc * kKC, wofs[i] - back(sc),
               (lds_void*)(smem + 3 * XB + buf * WB + (32 * i + 8 * wave) * 128));
  };

  f32x16_t acc[MB][4];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = f32x16_t{};
  uint32_t xa[4], wa[4];                                // LDS bytes of this lane's operands of step ks
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const uint32_t c = ((2 * ks + hg) ^ ((l32 >> 1) & 7)) * 16;
    xa[ks] = (row0 + l32) * 128 + c;
    wa[ks] = 3 * XB + (col0 + l32) * 128 + c;
  }
  constexpr int NOP = MB + 4;                           // operands of a step: W blocks 0-3, then x blocks
  bf16x8_t op[2][NOP];
  auto rd = [&](int xo, int wo, int ks, int i) __attribute__((always_inline)) -> bf16x8_t {
    return *reinterpret_cast<const bf16x8_t*>(smem + (i < 4 ? wa[ks] + wo + i * 4096 : xa[ks] + xo + (i - 4) * 4096));
  };
  // operands in the order the next step's MFMAs need them: the first x block, W, the other x blocks
  constexpr int kOrder[8] = {4, 0, 1, 2, 3, 5, 6, 7};
  // one step: 4 MB MFMAs, one operand read every other MFMA and, after that one, a load
  auto step = [&](int cur, auto read, auto load) __attribute__((always_inline)) {
    constexpr int N = 4 * MB, EV = N / NOP >= 2 ? 2 : 1;   // MFMAs per operand read
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int mb = n / 4, nb = n % 4;
      acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[cur][nb], op[cur][4 + mb], acc[mb][nb], 0, 0, 0);
      if (n % EV == 0 && n / EV < NOP) op[cur ^ 1][kOrder[n / EV]] = read(kOrder[n / EV]);
      if (n % 2 == 1) load(n / 2);
    }
#pragma unroll
    for (int n = 0; n < NOP; ++n) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (EV == 2) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  };
#pragma unroll
  for (int i = 0; i < WL; ++i) issue_w(0, 0, i);
#pragma unroll
  for (int i = 0; i < XL; ++i) issue_x(0, 0, i);
#pragma unroll
  for (int i = 0; i < XL; ++i) issue_x(1, 1, i);
#pragma unroll
  for (int k = 1; k < WS; ++k)
#pragma unroll
    for (int i = 0; i < WL; ++i) issue_w(k, k, i);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(XL + (WS - 1) * WL) : "memory");
#pragma unroll
  for (int i = 0; i < NOP; ++i) op[0][i] = rd(0, 0, 0, i);
  int x3 = 0;                                           // s % 3
  for (int s = 0; s < n_full; ++s) {
    const int xn = x3 == 2 ? 0 : x3 + 1;
    const int wb = WS == 3 ? x3 : s & 1;
    const int xo = x3 * XB, wo = wb * WB, wn = (WS == 3 ? xn : wb ^ 1) * WB;
    auto no_load = [](int) {};
    step(0, [&](int i) __attribute__((always_inline)) { return rd(xo, wo, 1, i); },
         [&](int i) __attribute__((always_inline)) { if (i < XL) issue_x(s + 2, x3 == 0 ? 2 : x3 - 1, i); });
    step(1, [&](int i) __attribute__((always_inline)) { return rd(xo, wo, 2, i); }, no_load);
    step(0, [&](int i) __attribute__((always_inline)) { return rd(xo, wo, 3, i); }, no_load);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(XL + (WS - 2) * WL) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    step(1, [&](int i) __attribute__((always_inline)) { return rd(xn * XB, wn, 0, i); },
         [&](int i) __attribute__((always_inline)) {
#pragma unroll
           for (int k = i * WL / (2 * MB); k < (i + 1) * WL / (2 * MB); ++k) issue_w(s + WS, wb, k);
         });
    __builtin_amdgcn_sched_barrier(0);
    x3 = xn;
  }
  if (n_st > n_full) {                                  // 32 columns left: two steps
    const int xo = x3 * XB, wo = (WS == 3 ? x3 : n_full & 1) * WB;
    step(0, [&](int i) __attribute__((always_inline)) { return rd(xo, wo, 1, i); }, [](int) {});
    step(1, [&](int i) __attribute__((always_inline)) { return op[0][i]; }, [](int) {});
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // no LDS write or read is in flight

  // ---- epilogue: round, rotate, y tile to LDS ([token][output]) --------------------------------
  // acc[mb][nb] register r: token row0 + 32 mb + l32, output col0 + 32 nb + 8 (r / 4) + 4 hg + r % 4
  int32_t* tslot = reinterpret_cast<int32_t*>(smem + TM * kPitch);
  if constexpr (POOL)
    for (int e = tid; e < TM; e += 256) tslot[e] = t0 + e < n_tokens ? slots[t0 + e] : -1;
  constexpr int PB = D / 64;                            // blocks of half a head: a pair is (nb, nb + PB)
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int row = row0 + 32 * mb + l32;
    const float4* cs = reinterpret_cast<const float4*>(tab + static_cast<int64_t>(min(t0 + row, n_tokens - 1)) * (D / 2));
    char* dst = smem + row * kPitch + (col0 + 4 * hg) * 2;
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {                    // the two pairs of blocks
      const int lo = D == 128 ? pr : 2 * pr, hi = lo + PB;
      const int i0 = D == 128 ? 32 * pr : 0;            // first angle of block lo
      const bool rot = (n0 + col0 + 32 * lo) / D < hq + hkv;   // uniform
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        uint32_t a[2], c[2];                            // y of dims i .. i + 3 and of their partners
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          a[j] = pack_bf16(acc[mb][lo][4 * q4 + 2 * j], acc[mb][lo][4 * q4 + 2 * j + 1]);
          c[j] = pack_bf16(acc[mb][hi][4 * q4 + 2 * j], acc[mb][hi][4 * q4 + 2 * j + 1]);
        }
        if (rot) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float4 c2 = cs[(i0 + 8 * q4 + 4 * hg) / 2 + j];   // (cos, sin) of two angles
            const float a0 = bf16_to_f32(a[j] & 0xFFFF), a1 = bf16_to_f32(a[j] >> 16);
            const float b0 = bf16_to_f32(c[j] & 0xFFFF), b1 = bf16_to_f32(c[j] >> 16);
            a[j] = pack_bf16(a0 * c2.x - b0 * c2.y, a1 * c2.z - b1 * c2.w);
            c[j] = pack_bf16(b0 * c2.x + a0 * c2.y, b1 * c2.z + a1 * c2.w);
          }
        }
        *reinterpret_cast<uint2*>(dst + (32 * lo + 8 * q4) * 2) = make_uint2(a[0], a[1]);
        *reinterpret_cast<uint2*>(dst + (32 * hi + 8 * q4) * 2) = make_uint2(c[0], c[1]);
      }
    }
  }
  __syncthreads();
  store_tile<D, POOL, false, TM, kTN, 256>(
      smem, kPitch, t0, n_tokens, [&](int o) { return n0 + o; }, n_out, 0, [](int, int) -> const float4* { return nullptr; },
      tslot, hq, hkv, q_out, k_out, v_out, n_slots);
}

// Decode steps and short questions.  The 256-token tiles would leave most compute units idle
// (up to 256 tokens are 24 to 40 work-groups).  What bounds these calls is reading W once, so a
// tile is narrow in outputs (TN = 32 NB) and tall enough for the tokens (TM = 32 MB), and its WV
// waves split H: wave w takes the 64-column stages w, w + WV, ..  Every byte staged in LDS is read
// by one wave only: each wave owns a ring of RING stages (its x and W rows) and waits for its
// own loads, with no barrier in the loop; two to three work-groups of four waves share a
// compute unit.  The partial sums (fp32) meet in LDS: the upper half of the waves hand theirs to
// the lower half, whose sums are added in order.  A tile's columns are TN/2 dims below D/2 of
// one head and their rotary partners D/2 above, so the rotation needs this tile only.  The
// (cos, sin) pairs of the tile are computed here too, while the first stages are in flight: no
// table pass.  64 tokens x 4096 x 6144: 14.9 us (3.4 TB/s of W), from 73.
constexpr int kMetaMax = 256;     // cu_q entries staged in LDS; batches of more requests search global memory
template <int D, bool POOL, int MB, int NB, int WV, int RING>
__global__ __launch_bounds__(64 * WV, 2) void qkv_ksplit_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ w, int n_tokens, int hidden, int n_out, int hq,
    int hkv, const int32_t* __restrict__ cu_q, const int32_t* __restrict__ seq_lens, int n_reqs, double log2_theta,
    uint16_t* __restrict__ q_out, uint16_t* __restrict__ k_out, uint16_t* __restrict__ v_out,
    const int32_t* __restrict__ slots, int64_t n_slots) {
  constexpr int TM = 32 * MB, TN = 32 * NB, ROWS = TM + TN, KC = kKC;
  constexpr int STAGE = ROWS * KC * 2;               // bytes of one wave's stage: x rows, then W rows
  constexpr int LOADS = STAGE / 1024;                 // 16-byte direct loads per thread per stage (8 rows each)
  constexpr int kThr = 64 * WV, NS = WV / 2;          // NS: partial sums held in LDS at the end
  constexpr int PP = TN + 4;                          // row pitch of the partial sums (floats)
  constexpr int YP = TN * 2 + 16;                     // row pitch of the y tile (bytes)
  constexpr int YOFS = NS * TM * PP * 4;              // after the loop: partial sums, y tile, (cos, sin)
  constexpr int COFS = YOFS + TM * YP;
  constexpr int END = COFS + TM * (TN / 2) * 8;
  constexpr int RING_BYTES = WV * RING * STAGE;
  constexpr int SMEM = END > RING_BYTES ? END : RING_BYTES;
  constexpr int NCS = TM * (TN / 2) / kThr;           // (cos, sin) pairs per thread
  static_assert(NCS * kThr == TM * (TN / 2) && COFS % 16 == 0, "(cos, sin) split");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  __shared__ int32_t meta[2][kMetaMax];               // cu_q, seq_lens
  __shared__ int32_t tslot[TM];
  const int n_tiles_n = n_out / TN, n_tiles_m = (n_tokens + TM - 1) / TM;
  // every XCD (b % 8) gets a contiguous run of tiles, token tiles fastest: tiles that share W rows
  // run on one XCD
  const int b = blockIdx.x, full = gridDim.x & ~7;
  const int L = b < full ? (b % 8) * (full / 8) + b / 8 : b;
  const int tile_n = L / n_tiles_m, tile_m = L % n_tiles_m;
  if (tile_n >= n_tiles_n) return;
  const int t0 = tile_m * TM;
  const int head = tile_n / (D / TN), part = tile_n % (D / TN);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hg = lane >> 5;
  // dim of local column o within the head: o < TN/2 below D/2, its partner TN/2 columns further on
  auto dim_of = [&](int o) { return o < TN / 2 ? part * (TN / 2) + o : D / 2 + part * (TN / 2) + o - TN / 2; };

  // piece i of a stage covers its rows 8 i .. 8 i + 7: the tile's tokens, then its W rows
  uint32_t ofs[LOADS];                                // byte offsets of this lane's 16 bytes at column 0
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int row = 8 * i + lane / 8;
    const int c = (lane % 8) ^ ((row >> 1) & 7);
    const int r = row < TM ? min(t0 + row, n_tokens - 1) - t0 : dim_of(row - TM);
    ofs[i] = static_cast<uint32_t>(r * hidden + c * 8) * 2u;
  }
  const uint16_t* xbase = x + static_cast<int64_t>(t0) * hidden;
  const uint16_t* wbase = w + static_cast<int64_t>(head) * D * hidden;
  char* ring = smem + wave * (RING * STAGE);
  const int n_full = hidden / KC, n_st = (hidden + KC - 1) / KC;
  const int cnt = n_st > wave ? (n_st - wave + WV - 1) / WV : 0;    // this wave's stages: wave, wave + WV, ..
  auto issue = [&](int j) {
    char* st = ring + (j % RING) * STAGE;
    const int s = j * WV + wave;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      // a last stage of 32 columns: its upper chunks repeat the lower ones (never used)
      const int c = (lane % 8) ^ (((8 * i + lane / 8) >> 1) & 7);
      load_lds16((i < TM / 8 ? xbase : wbase) + s * KC, ofs[i] - (s >= n_full && c >= 4 ? 64u : 0u),
                 (lds_void*)(st + i * 1024));
    }
  };

  // ---- the batch's request boundaries to LDS, then the first stages ------------------------
  const bool rot = head < hq + hkv;                   // uniform: Q or K
  const bool staged = n_reqs < kMetaMax;              // cu_q has n_reqs + 1 entries
  if (rot && staged) {
    if (wave < kMetaMax / 64) {
      const int e = wave * 64 + lane;
      load_lds4(cu_q + min(e, n_reqs), (lds_void*)(&meta[0][wave * 64]));
      load_lds4(seq_lens + min(e, n_reqs - 1), (lds_void*)(&meta[1][wave * 64]));
    }
  }
#pragma unroll
  for (int j = 0; j < RING; ++j)
    if (j < cnt) issue(j);
  float2 cs_reg[NCS];
  if (rot) {
    // the boundaries were requested first: they are here once at most the ring's loads are pending
    if (cnt >= RING) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(RING * LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    constexpr double kTwoPi = 6.283185307179586476925;
#pragma unroll
    for (int k = 0; k < NCS; ++k) {
      const int e = tid + k * kThr;
      const int row = e / (TN / 2), i = e % (TN / 2);
      const int t = min(t0 + row, n_tokens - 1);
      auto cu = [&](int r) { return staged ? meta[0][r] : cu_q[r]; };
      int lo = 0, hi = n_reqs - 1;                    // request of token t: the last r with cu_q[r] <= t
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (cu(mid) <= t) lo = mid; else hi = mid - 1;
      }
      const int64_t len = staged ? meta[1][lo] : seq_lens[lo];
      const int64_t p = len - (cu(lo + 1) - cu(lo)) + (t - cu(lo));
      // theta^(-2 i / D) as a power of two: its rounding (exponents up to ~2^5) moves an angle by
      // under 1e-14 of itself, far below the fp32 sine and cosine
      const double f = exp2(log2_theta * (-2.0 * (part * (TN / 2) + i) / D));
      const double a = static_cast<double>(p) * f;
      const double r = std::fma(-std::floor(a / kTwoPi), kTwoPi, a);
      float sn, cs;
      sincosf(static_cast<float>(r), &sn, &cs);
      cs_reg[k] = make_float2(cs, sn);
    }
  }

  // ---- the loop over this wave's columns -----------------------------------------------------
  f32x16_t acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x16_t{};
  for (int j = 0; j < cnt; ++j) {
    // stage j is complete when at most the RING - 1 newer stages are pending (loads return in order)
    if (j + RING <= cnt) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 1) * LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const char* st = ring + (j % RING) * STAGE;
    bf16x8_t a[KC / 16][MB], bq[KC / 16][NB];
#pragma unroll
    for (int ks = 0; ks < KC / 16; ++ks) {
      const int c = (ks * 2 + hg) ^ ((l32 >> 1) & 7);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) a[ks][mb] = *reinterpret_cast<const bf16x8_t*>(st + (mb * 32 + l32) * 128 + c * 16);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        bq[ks][nb] = *reinterpret_cast<const bf16x8_t*>(st + (TM + nb * 32 + l32) * 128 + c * 16);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // the stage is read: it may be overwritten
    if (j + RING < cnt) issue(j + RING);
    const int n_ks = j * WV + wave < n_full ? KC / 16 : KC / 32;
#pragma unroll
    for (int ks = 0; ks < KC / 16; ++ks)
      if (ks < KC / 32 || ks < n_ks)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][mb], bq[ks][nb], acc[mb][nb], 0, 0, 0);
  }
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");   // no wave's ring is in use any more

  // ---- sum over the waves: the upper half into the lower, then those sums in order -----------
  float* sums = reinterpret_cast<float*>(smem) + (wave % NS) * (TM * PP);
  auto each = [&](auto f) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          f(sums[(mb * 32 + (r / 4) * 8 + hg * 4 + (r % 4)) * PP + nb * 32 + l32], acc[mb][nb][r]);
  };
  float2* cs_tab = reinterpret_cast<float2*>(smem + COFS);
  if (rot)
#pragma unroll
    for (int k = 0; k < NCS; ++k) cs_tab[tid + k * kThr] = cs_reg[k];
  if (wave >= NS) each([](float& s, float v) { s = v; });
  if constexpr (POOL)
    if (tid < TM) tslot[tid] = t0 + tid < n_tokens ? slots[t0 + tid] : -1;
  __syncthreads();
  if (wave < NS) each([](float& s, float v) { s = v + s; });
  __syncthreads();
  const float* s0 = reinterpret_cast<const float*>(smem);
  for (int e = tid; e < TM * TN / 4; e += kThr) {
    const int row = e / (TN / 4), c = (e % (TN / 4)) * 4;
    f32x4_t v = *reinterpret_cast<const f32x4_t*>(s0 + row * PP + c);
#pragma unroll
    for (int g = 1; g < NS; ++g) v += *reinterpret_cast<const f32x4_t*>(s0 + g * (TM * PP) + row * PP + c);
    uint2 y;
    y.x = pack_bf16(v[0], v[1]);
    y.y = pack_bf16(v[2], v[3]);
    *reinterpret_cast<uint2*>(smem + YOFS + row * YP + c * 2) = y;
  }
  __syncthreads();
  store_tile<D, POOL, true, TM, TN, kThr>(
      smem + YOFS, YP, t0, n_tokens, [&](int o) { return head * D + dim_of(o); }, n_out, TN / 2,
      [&](int row, int i) { return reinterpret_cast<const float4*>(&cs_tab[row * (TN / 2) + i - part * (TN / 2)]); },
      tslot, hq, hkv, q_out, k_out, v_out, n_slots);
}

}  // namespace

namespace {

// Which kernel and tile a call takes, by its sizes alone (never by where K and V go, so that
// arckv_qkv_rope and arckv_qkv_rope_to_pool give the same bits).  us per call, 32 / 8 heads of
// 128 and hidden 4096 unless stated, against the 256 x 256 tiles that served every size before:
//   T <= 32   eight waves per 32 x 32 tile when every tile has its own compute unit: 11.0 at T =
//             32 (four waves, two tiles per unit: 11.9; before: 69); else four waves: hidden
//             8192, 320 tiles: 44.7 against 46.1
//   T <= 64   four waves, 32 x 32: 14.9 at T = 64 (64 x 32: 15.8; before: 73).  From T = 33 on two
//             token tiles read every W row; with W out of the caches, T = 33 and 64: 17.6 and 20.7 (64 x
//             32: 18.7, 20.3), hidden 1024 6.6 and 7.1 (9.4, 9.7), hidden 5120 23.1 and 28.5 (23.3, 26.0),
//             hidden 8192 44.4 and 55.4 (47.7, 58.4; 64 x 64: 43.9, 49.9; before: 138, 146)
//   up to 3.5 64 x 64 tiles per compute unit: 64 x 64 where they fill most of the chip and H is
//             long enough to outweigh their reduction (T = 256: 30.7, hidden 5120: 38.7 against
//             46.9 with 64 x 32; before 97 and 137), else 64 x 32 (hidden 1024, 3072 outputs,
//             T = 256: 10.2 against 13.5; between the two, hidden 2048, 8192 outputs: 29.6 against 23.7
//             at T = 256, 16.6 and 17.4 at T = 80).  Past that the prefill kernel's reuse wins: hidden 8192,
//             T = 512 (5 tiles per unit): 112 against 149; hidden 5120, T = 450 (3.5): 78 against 76
//   prefill   the tile height whose rounds of the chip take least, a round of 128-, 192- and
//             256-token tiles counted as 3, 4 and 5 (T = 907: 58, 70 and 84 us, one round each).
//             T = 1500: 112 us with 128 (2 rounds), 80 with 192 (1), 86 with 256 (1; the tiles before
//             84); T = 2000 (2, 2, 1): 117, 153 and 98; T = 2600 (2, 2, 2): 132, 157, 191; T = 3300 (3, 2,
//             2): 181, 164, 194; hidden 1024, 3072 outputs, T = 3300 (2, 1, 1): 43, 34 and 38 (before: 36).
//             Not 192 where its last tiles pad the tokens by over 10 % more than 256 does: hidden
//             8192, T = 1004 (1152 and 1024 tokens, one round each): 157 and 154
enum class QkvRoute { kK32x32Wide, kK32x32, kK64x32, kK64x64, kG128, kG192, kG256 };
constexpr int64_t kUnits = 256;   // compute units of a whole MI355X (on a part of one another tile may be faster)
QkvRoute qkv_route(int64_t n_tokens, int64_t hidden, int64_t n_out) {
  auto tiles = [&](int64_t m, int64_t n) { return ((n_tokens + m - 1) / m) * ((n_out + n - 1) / n); };
  if (n_tokens <= 32 && tiles(32, 32) <= kUnits) return QkvRoute::kK32x32Wide;
  if (n_tokens <= 64) return QkvRoute::kK32x32;
  if (2 * tiles(64, 64) <= 7 * kUnits)
    return hidden > 2048 && 4 * tiles(64, 64) >= 3 * kUnits ? QkvRoute::kK64x64 : QkvRoute::kK64x32;
  auto time = [&](int64_t m, int64_t each) { return each * ((tiles(m, kTN) + kUnits - 1) / kUnits); };
  const int64_t t128 = time(128, 3), t192 = time(192, 4), t256 = time(256, 5);
  const bool pads = 192 * tiles(192, kTN) * 10 > 256 * tiles(256, kTN) * 11;
  if (t256 <= t128 && (t256 <= t192 || pads)) return QkvRoute::kG256;
  return t192 <= t128 && !pads ? QkvRoute::kG192 : QkvRoute::kG128;
}

// Shared by arckv_qkv_rope and arckv_qkv_rope_to_pool: pool == true writes K and V into the
// pools k_dst / v_dst (num_blocks blocks) at slots.
int32_t qkv_rope_launch(const char* fn, const void* x, const void* w_qkv, int64_t n_tokens, int32_t hidden,
                        int32_t num_q_heads, int32_t num_kv_heads, int32_t head_dim, const int32_t* cu_q,
                        const int32_t* seq_lens, int32_t n_reqs, double rope_theta, void* workspace,
                        int64_t ws_bytes, void* q_out, void* k_dst, void* v_dst, bool pool, int64_t num_blocks,
                        const int32_t* slots, void* stream) {
  if (n_tokens < 0 || hidden < 1 || num_q_heads < 1 || num_kv_heads < 1 || n_reqs < 0 ||
      num_q_heads % num_kv_heads != 0 || !(rope_theta > 1.0) || !std::isfinite(rope_theta))
    return arckv::fail(ARCKV_EINVAL, "%s: bad sizes or theta", fn);
  if (head_dim != 64 && head_dim != 128)
    return arckv::fail(ARCKV_EUNSUPPORTED, "%s: head_dim %d not in {64,128}", fn, head_dim);
  const int64_t n_out = static_cast<int64_t>(num_q_heads + 2 * num_kv_heads) * head_dim;
  if (hidden % 32 != 0 || hidden > (1 << 22) || n_out % 128 != 0)   // (32-bit load offsets in a tile)
    return arckv::fail(ARCKV_EUNSUPPORTED,
                       "%s: hidden %d must be a multiple of %d (at most 2^22) and the %lld outputs of 128",
                       fn, hidden, 32, (long long)n_out);
  if (pool && (num_blocks < 1 || num_blocks > (int64_t{1} << 27)))
    return arckv::fail(ARCKV_EINVAL, "%s: num_blocks %lld", fn, (long long)num_blocks);
  if (n_tokens == 0) return ARCKV_OK;
  if (n_tokens > INT32_MAX - 256 || n_out > INT32_MAX || n_reqs < 1 ||
      static_cast<int64_t>(hidden) * n_tokens > (int64_t{1} << 40))
    return arckv::fail(ARCKV_EINVAL, "%s: %lld tokens, %lld outputs, %d requests", fn,
                       (long long)n_tokens, (long long)n_out, n_reqs);
  if (x == nullptr || w_qkv == nullptr || cu_q == nullptr || seq_lens == nullptr ||
      workspace == nullptr || q_out == nullptr || k_dst == nullptr || v_dst == nullptr ||
      (pool && slots == nullptr))
    return arckv::fail(ARCKV_EINVAL, "%s: NULL pointer", fn);
  for (const void* p : {x, w_qkv, static_cast<const void*>(workspace), static_cast<const void*>(q_out),
                        static_cast<const void*>(k_dst), static_cast<const void*>(v_dst)})
    if (reinterpret_cast<uintptr_t>(p) % 16 != 0)
      return arckv::fail(ARCKV_EINVAL, "%s: x, w_qkv, workspace and outputs must be 16-byte aligned", fn);
  const int64_t tab_bytes = n_tokens * (head_dim / 2) * static_cast<int64_t>(sizeof(float2));
  if (ws_bytes < tab_bytes)
    return arckv::fail(ARCKV_ENOSPC, "%s: workspace %lld bytes < %lld", fn, (long long)ws_bytes,
                       (long long)tab_bytes);
  auto* s = static_cast<hipStream_t>(stream);
  auto* tab = static_cast<float2*>(workspace);
  const dim3 tgrid(static_cast<unsigned>(std::min<int64_t>(kTableBlocks, (n_tokens * (head_dim / 2) + 255) / 256)));
  auto* xp = static_cast<const uint16_t*>(x);
  auto* wp = static_cast<const uint16_t*>(w_qkv);
  auto* q = static_cast<uint16_t*>(q_out);
  auto* k = static_cast<uint16_t*>(k_dst);
  auto* v = static_cast<uint16_t*>(v_dst);
  const int T = static_cast<int>(n_tokens), N = static_cast<int>(n_out);
  const int64_t n_slots = pool ? num_blocks * 16 : 0;
  auto go = [&](auto d_tag, auto pool_tag) {
    constexpr int D = decltype(d_tag)::value;
    constexpr bool P = decltype(pool_tag)::value;
    auto ksplit = [&](auto mb, auto nb, auto wv, auto ring) {
      constexpr int MB = decltype(mb)::value, NB = decltype(nb)::value, WV = decltype(wv)::value;
      const dim3 grid(static_cast<unsigned>((n_out / (32 * NB)) * ((n_tokens + 32 * MB - 1) / (32 * MB))));
      hipLaunchKernelGGL((qkv_ksplit_kernel<D, P, MB, NB, WV, decltype(ring)::value>), grid, dim3(64 * WV), 0, s, xp,
                         wp, T, hidden, N, num_q_heads, num_kv_heads, cu_q, seq_lens, n_reqs, std::log2(rope_theta), q, k,
                         v, slots, n_slots);
    };
    auto gemm = [&](auto mb) {
      constexpr int MB = decltype(mb)::value;
      const dim3 grid(static_cast<unsigned>(((n_out + kTN - 1) / kTN) * ((n_tokens + 64 * MB - 1) / (64 * MB))));
      hipLaunchKernelGGL(rope_table_kernel<D>, tgrid, dim3(256), 0, s, n_tokens, cu_q, seq_lens, n_reqs, rope_theta, tab);
      hipLaunchKernelGGL((qkv_gemm_rope_kernel<D, P, MB>), grid, dim3(256), 0, s, xp, wp, T, hidden, N,
                         num_q_heads, num_kv_heads, tab, q, k, v, slots, n_slots);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    using I8 = std::integral_constant<int, 8>;
    switch (qkv_route(n_tokens, hidden, n_out)) {
      case QkvRoute::kK32x32Wide: ksplit(I1{}, I1{}, I8{}, I2{}); break;
      case QkvRoute::kK32x32: ksplit(I1{}, I1{}, I4{}, I2{}); break;
      case QkvRoute::kK64x32: ksplit(I2{}, I1{}, I4{}, I1{}); break;
      case QkvRoute::kK64x64: ksplit(I2{}, I2{}, I4{}, I1{}); break;
      case QkvRoute::kG128: gemm(I2{}); break;
      case QkvRoute::kG192: gemm(I3{}); break;
      case QkvRoute::kG256: gemm(I4{}); break;
    }
  };
  using D64 = std::integral_constant<int, 64>;
  using D128 = std::integral_constant<int, 128>;
  if (head_dim == 64) {
    if (pool) go(D64{}, std::true_type{}); else go(D64{}, std::false_type{});
  } else {
    if (pool) go(D128{}, std::true_type{}); else go(D128{}, std::false_type{});
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return arckv::fail(ARCKV_EDEVICE, "%s: %s", fn, hipGetErrorString(e));
  return ARCKV_OK;
}

}  // namespace

extern "C" int32_t arckv_test_qkv_tiles(int64_t n_tokens, int32_t hidden, int64_t n_out, int32_t* tile_tokens,
                                        int32_t* tile_outputs, int32_t* split_waves) {
  if (n_tokens < 1 || n_tokens > INT32_MAX || hidden < 1 || n_out < 1 || n_out > INT32_MAX ||
      tile_tokens == nullptr || tile_outputs == nullptr || split_waves == nullptr)
    return arckv::fail(ARCKV_EINVAL, "test_qkv_tiles: bad arguments");
  auto set = [&](int32_t m, int32_t n, int32_t w) { *tile_tokens = m; *tile_outputs = n; *split_waves = w; };
  switch (qkv_route(n_tokens, hidden, n_out)) {
    case QkvRoute::kK32x32Wide: set(32, 32, 8); break;
    case QkvRoute::kK32x32: set(32, 32, 4); break;
    case QkvRoute::kK64x32: set(64, 32, 4); break;
    case QkvRoute::kK64x64: set(64, 64, 4); break;
    case QkvRoute::kG128: set(128, kTN, 0); break;
    case QkvRoute::kG192: set(192, kTN, 0); break;
    case QkvRoute::kG256: set(256, kTN, 0); break;
  }
  return ARCKV_OK;
}

extern "C" int32_t arckv_qkv_rope(const void* x, const void* w_qkv, int64_t n_tokens, int32_t hidden,
                                  int32_t num_q_heads, int32_t num_kv_heads, int32_t head_dim,
                                  const int32_t* cu_q, const int32_t* seq_lens, int32_t n_reqs,
                                  double rope_theta, void* workspace, int64_t ws_bytes, void* q_out,
                                  void* k_out, void* v_out, void* stream) {
  return qkv_rope_launch("qkv_rope", x, w_qkv, n_tokens, hidden, num_q_heads, num_kv_heads, head_dim, cu_q,
                         seq_lens, n_reqs, rope_theta, workspace, ws_bytes, q_out, k_out, v_out, false, 0,
                         nullptr, stream);
}

extern "C" int32_t arckv_qkv_rope_to_pool(const void* x, const void* w_qkv, int64_t n_tokens, int32_t hidden,
                                          int32_t num_q_heads, int32_t num_kv_heads, int32_t head_dim,
                                          const int32_t* cu_q, const int32_t* seq_lens, int32_t n_reqs,
                                          double rope_theta, void* workspace, int64_t ws_bytes, void* q_out,
                                          void* k_pool, void* v_pool, int64_t num_blocks,
                                          const int32_t* slot_mapping, void* stream) {
  return qkv_rope_launch("qkv_rope_to_pool", x, w_qkv, n_tokens, hidden, num_q_heads, num_kv_heads, head_dim,
                         cu_q, seq_lens, n_reqs, rope_theta, workspace, ws_bytes, q_out, k_pool, v_pool, true,
                         num_blocks, slot_mapping, stream);
}
