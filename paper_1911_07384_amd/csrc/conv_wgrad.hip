// Weight gradient of the convolution on the gfx950 FP16 matrix cores.
//
// GEMM view: dW[k][col] = sum_pix dy[pix][k] * X[pix][col],
//   pix = (image, p, q) over the output grid (the reduction, length N*P*Q),
//   col = (r, s, c) with c fastest (the KRSC filter row),
//   X[pix][(r,s,c)] = x[image][p*sh - ph + r][q*sw - pw + s][c] (zero outside).
// Both operands are channel-contiguous in memory but the reduction runs over
// pixels: they are DMA'd pixel-major into LDS and the MFMA operands come from
// gfx950's transposing LDS read.
//
// The pixel range is split across workgroups (split-K).  Each split writes
// its float32 partial tile to the workspace; a second kernel adds the splits
// in a fixed order and rounds once to binary16, so the result is
// deterministic.

#include "kernels.hpp"

#include <stdio.h>

#include <type_traits>

namespace fp16k {
namespace {

constexpr int BKP = 64;  // pixels per k-step

// For K and C multiples of 8 (where C is not a multiple of 64, each lane's
// 8-channel chunk carries its own filter tap).  Each stage covers 64 pixels:
// the dy rows (BM channels) and the x patch rows (BN filter columns, 64 per
// tap and channel block) are DMA'd pixel-major straight into LDS, in 8 KB
// sub-tiles of 64 pixel rows x 128 bytes (16-byte chunks XOR-swizzled by
// pixel row).  The MFMA operands, which need 8 consecutive pixels per lane,
// come from the transposing LDS read of gfx950 (ds_read_b64_tr_b16: within
// each 16-lane group, lane b*4+a receives element a of the 8-byte rows that
// lanes b, b+4, b+8 and b+12 address), two reads per operand.  S stages in a
// ring, operand reads one k sub-step ahead, as in the implicit-GEMM kernels;
// four waves, or eight with one workgroup per CU (see wgrad_choice).

typedef short short4v __attribute__((ext_vector_type(4)));

// One 16-byte-per-lane DMA from a buffer resource into LDS (1 KB per wave).
__device__ __forceinline__ void wdma16(__amdgpu_buffer_rsrc_t rs, char* lds_dst, uint32_t voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)lds_dst, 16,
                                           voff, 0, 0, 0);
}

__device__ __forceinline__ void wbarrier() { __asm__ volatile("s_barrier" ::: "memory"); }

// The transposing read, issued from inline assembly at an LDS byte address
// plus a constant offset.  Through the compiler's builtin, every such read
// waits for all LDS DMAs in flight (the compiler cannot tell the buffers
// apart), so the stage just issued had to land before the next stage could be
// read; from assembly the ring keeps its stages in flight (5-15 % faster on
// the ResNet-50 shapes, bit-identical partials).  The compiler then neither
// orders the read after the DMAs nor waits for its result: the loop orders
// the DMAs by its own vmcnt wait and barrier, and each result by lds_ready()
// before the MFMAs that use it.  Nothing may read the destination registers
// before that wait (not even a register copy); a host-side test checks the
// built code for it.
template <int OFF>
__device__ __forceinline__ short4v ldtr_asm(uint32_t addr) {
  short4v r;
  __asm__ volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFF));
  return r;
}
// Waits until at most N LDS reads of this wave are in flight; the fragment is
// tied to the wait so that no use of it is scheduled before.
template <int N>
__device__ __forceinline__ void lds_ready(half8& v) {
  __asm__ volatile("s_waitcnt lgkmcnt(%1)" : "+v"(v) : "i"(N));
}
__device__ __forceinline__ void lds_tie(half8& v) { __asm__ volatile("" : "+v"(v)); }

template <int BM, int BN, int WM, int WN, int S>
struct WCfg7 {
  static constexpr int SA = BM / 64, SB = BN / 64;  // 64-channel sub-tiles
  static constexpr int NW = WM * WN;                // waves: 4 or 8
  static constexpr int NI = (SA + SB) * 8;          // DMA instructions per stage
  static constexpr int IW = NI / NW;                // per wave
  static constexpr int H = 8 / NW;                  // pixel rows per lane and sub-tile
  static constexpr int STAGE = (SA + SB) * 8192;    // bytes
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int TM = WTM / 32, TN = WTN / 32;
};

template <int BM, int BN, int WM, int WN, int S, bool CGEN = false>
__global__ __launch_bounds__(64 * WM * WN) void wgrad7_kernel(const WgradArgs a) {
  using K = WCfg7<BM, BN, WM, WN, S>;
  constexpr int SA = K::SA, SB = K::SB, IW = K::IW, H = K::H, TM = K::TM, TN = K::TN,
                WTM = K::WTM, WTN = K::WTN;
  static_assert((K::NW == 4 || K::NW == 8) && TM >= 1 && TN >= 1 && S >= 2, "tile shape");
  static_assert(IW * (S - 1) < 64, "vmcnt range");
  // with a third stage the next loads go out between the MFMAs of a step, a
  // few per sub-step, instead of in a burst behind its barrier
  constexpr bool SPREAD = S >= 3;
  __shared__ __attribute__((aligned(1024))) char lds[S * K::STAGE];

  const int Nw = a.R * a.S * a.C;
  const int tiles_n = (Nw + BN - 1) / BN;
  // Workgroups are dealt to the 8 XCDs round-robin in launch order.  Each
  // XCD gets a contiguous run of the split-major order instead, so the tiles
  // that share a pixel range (and so its dy and x rows) share one L2: the
  // layers with 28x28 and larger grids at batch 128 went 1.1-1.9x faster.
  int tile, split;
  {
    const int total = gridDim.x * gridDim.y;
    const int L = blockIdx.y * gridDim.x + blockIdx.x;
    const int q = total >> 3, r = total & 7, xcd = L & 7;
    const int Lg = xcd * q + (xcd < r ? xcd : r) + (L >> 3);
    tile = Lg % gridDim.x;
    split = Lg / gridDim.x;
  }
  const int m0 = (tile / tiles_n) * BM;
  const int n0 = (tile % tiles_n) * BN;
  const int npix = a.N * a.P * a.Q;  // < 2^30
  const int pbeg = split * a.pix_per_split;
  const int pend = npix - pbeg < a.pix_per_split ? npix : pbeg + a.pix_per_split;
  const int KT = pend > pbeg ? (pend - pbeg + 63) / 64 : 0;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  constexpr uint32_t OOB = 0x80000000u;
  const int dy_bytes = (int)((int64_t)npix * a.K * 2);
  const int x_bytes = (int)((int64_t)a.N * a.H * a.W * a.C * 2);

  // DMA roles: instruction i of this wave fills sub-tile i/H, pixel rows
  // rb*8 .. rb*8+7 with rb = 4*(i%H) + wave; a lane covers pixel row
  // rb*8 + lane/8 and physical chunk lane%8, holding logical chunk
  // (lane%8) ^ swz(row), swz(row) = 2*(row%4).  A transposing read takes
  // 32 bytes (chunks 2i, 2i+1) from each of 4 consecutive rows per 16-lane
  // group; with this swizzle the 4 rows' pairs land on distinct chunk
  // positions, and the two groups served together (the other channel
  // half) on the rest, so the reads are bank-conflict free.
  // Per pixel row: the next step's pixel (relative to pend), its output row
  // and column as the input position of tap (0, 0), and the byte offsets of
  // its chunk in dy and of tap (0, 0) in x (wrapping below zero in the
  // padding): a DMA then costs an add and its range checks.
  const int lc = (lane & 7) ^ (((lane >> 3) & 3) << 1);  // (rows 8 apart share it)
  bool av[SA];  // the lane's chunk of each dy sub-tile is inside K
#pragma unroll
  for (int u = 0; u < SA; ++u) av[u] = m0 + u * 64 + lc * 8 < a.K;
  int left[H], ih0[H], iw0[H];
  uint32_t dyo[H], xo[H];
  const int dq = 64 % a.Q, dp = (64 / a.Q) % a.P, dimg = 64 / (a.P * a.Q);
  const uint32_t pix_bytes = (uint32_t)a.C * 2u, row_bytes = (uint32_t)a.W * pix_bytes,
                 img_bytes = (uint32_t)a.H * row_bytes;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int pix = pbeg + (4 * h + wave) * 8 + (lane >> 3);
    const int PQ = a.P * a.Q;
    const int img = pix / PQ;
    const int rem = pix - img * PQ;
    const int p = rem / a.Q, q = rem - p * a.Q;
    left[h] = pend - pix;
    ih0[h] = p * a.sh - a.ph;
    iw0[h] = q * a.sw - a.pw;
    dyo[h] = (uint32_t)pix * (uint32_t)a.K * 2u + (uint32_t)(m0 + lc * 8) * 2u;
    xo[h] = (uint32_t)img * img_bytes + (uint32_t)ih0[h] * row_bytes +
            (uint32_t)iw0[h] * pix_bytes;
  }
  // the filter tap of each x sub-tile (and its channel base): uniform; with
  // CGEN (C a multiple of 8 but not of 64) a 64-column block spans several
  // taps and each lane's 8-channel chunk has a tap of its own (none past Nw)
  int tr[SB], ts[SB];
  uint32_t to[SB];
  bool tv[SB];
#pragma unroll
  for (int b = 0; b < SB; ++b) {
    const int col = n0 + b * 64 + (CGEN ? lc * 8 : 0);
    const int tap = col / a.C;
    const int c0 = col - tap * a.C;
    tr[b] = tap / a.S;
    ts[b] = tap - tr[b] * a.S;
    tv[b] = col < Nw;
    to[b] = (uint32_t)tr[b] * row_bytes + (uint32_t)ts[b] * pix_bytes +
            (uint32_t)(c0 + (CGEN ? 0 : lc * 8)) * 2u;
  }

  auto dma = [&](char* buf, int i) {
    const int h = i % H, sub = i / H;
    char* dst = buf + sub * 8192 + (4 * h + wave) * 1024;
    if (sub < SA) {
      const __amdgpu_buffer_rsrc_t rs_dy = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<h16*>(a.dy), (short)0, dy_bytes, 0x00020000);
      const bool v = left[h] > 0 && av[sub];
      wdma16(rs_dy, dst, v ? dyo[h] + (uint32_t)sub * 128u : OOB);
    } else {
      const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<h16*>(a.x), (short)0, x_bytes, 0x00020000);
      const int b = sub - SA;
      const bool v = left[h] > 0 && tv[b] && (unsigned)(ih0[h] + tr[b]) < (unsigned)a.H &&
                     (unsigned)(iw0[h] + ts[b]) < (unsigned)a.W;
      wdma16(rs_x, dst, v ? xo[h] + to[b] : OOB);
    }
  };
  // the pixel rows 64 further
  auto advance = [&]() {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      left[h] -= 64;
      dyo[h] += 128u * (uint32_t)a.K;
      int iw = iw0[h] + dq * a.sw;
      const bool c1 = iw + a.pw >= a.Q * a.sw;
      iw -= c1 ? a.Q * a.sw : 0;
      int ih = ih0[h] + (dp + (c1 ? 1 : 0)) * a.sh;
      const bool c2 = ih + a.ph >= a.P * a.sh;
      ih -= c2 ? a.P * a.sh : 0;
      xo[h] += (uint32_t)(dimg + (c2 ? 1 : 0)) * img_bytes +
               (uint32_t)(ih - ih0[h]) * row_bytes + (uint32_t)(iw - iw0[h]) * pix_bytes;
      ih0[h] = ih;
      iw0[h] = iw;
    }
  };
  auto issue = [&](char* buf) {
#pragma unroll
    for (int i = 0; i < IW; ++i) dma(buf, i);
    advance();
  };

  const int wm = wave / WN, wn = wave % WN;
  const int g = lane >> 4, j = lane & 15;
  // transposing-read address pieces of this lane: pixel row within a k16
  // sub-step, and channel quad within a 32-row operand
  const int kr_l = 8 * (g >> 1) + (j >> 2);
  const int ch_l = 16 * (g & 1) + 4 * (j & 3);
  floatx16 acc[TM][TN];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[tm][tn][e] = 0.0f;

  half8 af[2][TM], bf[2][TN];
  auto mma = [&](const half8 (&fa)[TM], const half8 (&fb)[TN]) {
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = mfma32x32x16(fa[tm], fb[tn], acc[tm][tn]);
  };

  if (KT > 0) {
    // lane part of each operand's read address (the swizzle depends on the
    // pixel row mod 4, which k sub-steps of 16 rows and the +4 row of the
    // second read leave unchanged): sub-step ks of a stage is at +2048*ks,
    // the second read at +512
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    uint32_t oa[TM], ob[TN];
    auto lane_part = [&](int c) {
      const int ch = (c & 63) + ch_l;
      return (uint32_t)((c >> 6) * 8192 + kr_l * 128 + (((ch >> 3) ^ ((kr_l & 3) << 1)) << 4) +
                        ((ch >> 2) & 1) * 8);
    };
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) oa[tm] = lds0 + lane_part(wm * WTM + tm * 32);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) ob[tn] = lds0 + SA * 8192 + lane_part(wn * WTN + tn * 32);
    constexpr int NR = 2 * (TM + TN);  // reads per sub-step
    static_assert(NR <= 15, "lgkmcnt range");
    auto afetch = [&](auto ks, uint32_t sbase, half8(&fa)[TM], half8(&fb)[TN]) {
      constexpr int KS = decltype(ks)::value;
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) {
        const short4v v0 = ldtr_asm<KS * 2048>(oa[tm] + sbase);
        const short4v v1 = ldtr_asm<KS * 2048 + 512>(oa[tm] + sbase);
        fa[tm] = __builtin_bit_cast(half8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
      }
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        const short4v v0 = ldtr_asm<KS * 2048>(ob[tn] + sbase);
        const short4v v1 = ldtr_asm<KS * 2048 + 512>(ob[tn] + sbase);
        fb[tn] = __builtin_bit_cast(half8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    };
    // the fragments of one sub-step are complete once at most NR reads (those
    // of the next sub-step, issued after them) are in flight
    auto ready = [&](half8(&fa)[TM], half8(&fb)[TN]) {
      lds_ready<NR>(fa[0]);
#pragma unroll
      for (int tm = 1; tm < TM; ++tm) lds_tie(fa[tm]);
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) lds_tie(fb[tn]);
    };
    constexpr int PRE = SPREAD ? S - 1 : S;  // stages loaded ahead of the loop
#pragma unroll
    for (int s = 0; s < PRE; ++s) issue(lds + s * K::STAGE);
    constexpr int ALLOW0 = IW * (PRE - 1);
    constexpr int WAIT0 = (0x0 << 8) | (0x7 << 4) | (ALLOW0 & 0xF) | ((ALLOW0 >> 4) << 14);
    constexpr int ALLOW = IW * (S - 2);
    constexpr int WAIT = (0x0 << 8) | (0x7 << 4) | (ALLOW & 0xF) | ((ALLOW >> 4) << 14);
    __builtin_amdgcn_s_waitcnt(WAIT0);
    wbarrier();
    afetch(std::integral_constant<int, 0>(), 0u, af[0], bf[0]);
    int rd = 0, wr = S - 1;
    constexpr int P = (IW + 2) / 3;
    auto part = [&](int q0, int q1) {  // SPREAD: some of stage kt+2's loads
      if (SPREAD) {
#pragma unroll
        for (int i = q0; i < (q1 < IW ? q1 : IW); ++i) dma(lds + wr * K::STAGE, i);
      }
    };
    auto fence = [&]() {
      if (SPREAD) __builtin_amdgcn_sched_barrier(0);
    };
    for (int kt = 0; kt < KT; ++kt) {
      const uint32_t cur = (uint32_t)(rd * K::STAGE);
      afetch(std::integral_constant<int, 1>(), cur, af[1], bf[1]);
      part(0, P);
      ready(af[0], bf[0]);
      mma(af[0], bf[0]);
      fence();
      afetch(std::integral_constant<int, 2>(), cur, af[0], bf[0]);
      part(P, 2 * P);
      ready(af[1], bf[1]);
      mma(af[1], bf[1]);
      fence();
      afetch(std::integral_constant<int, 3>(), cur, af[1], bf[1]);
      part(2 * P, 3 * P);
      ready(af[0], bf[0]);
      mma(af[0], bf[0]);
      if (SPREAD) advance();
      fence();
      // every read of this stage is complete (lgkmcnt 0) and stage kt+1 has
      // landed (vmcnt) in every wave before the buffer is refilled
      __builtin_amdgcn_s_waitcnt(WAIT);
      wbarrier();
      if (!SPREAD) issue(lds + rd * K::STAGE);
      rd = rd + 1 == S ? 0 : rd + 1;
      wr = wr + 1 == S ? 0 : wr + 1;
      afetch(std::integral_constant<int, 0>(), (uint32_t)(rd * K::STAGE), af[0], bf[0]);
      ready(af[1], bf[1]);
      mma(af[1], bf[1]);
      fence();
    }
    __builtin_amdgcn_s_waitcnt(0);
  }

  // float32 partial tile of this split
  float* out = a.partial + (int64_t)split * a.K * Nw;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = m0 + wm * WTM + tm * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      if (m >= a.K) continue;
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        const int n = n0 + wn * WTN + tn * 32 + (lane & 31);
        if (n < Nw) out[(int64_t)m * Nw + n] = acc[tm][tn][e];
      }
    }
  }
}

// dw = rne16(sum over splits), written KRSC or KCRS with the real C.  A block
// of 256 threads owns 64 consecutive outputs; its four waves each add every
// fourth split (in order), and the four subtotals are added in a fixed order,
// so the result is deterministic.
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const float* __restrict__ partial,
                                                           int splits, int K, int Kp, int R, int S,
                                                           int C, int Cp, int layout,
                                                           h16* __restrict__ dw) {
  __shared__ float red[4][64];
  const int64_t Nw = (int64_t)R * S * Cp;
  const int64_t total = (int64_t)K * R * S * C;
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;  // enumerates KRSC with the real C
  int64_t src = 0;
  int k = 0, r = 0, s = 0, c = 0;
  if (i < total) {
    c = (int)(i % C);
    int64_t t = i / C;
    s = (int)(t % S);
    t /= S;
    r = (int)(t % R);
    k = (int)(t / R);
    src = (int64_t)k * Nw + ((int64_t)r * S + s) * Cp + c;
  }
  // splits grp, grp+4, grp+8, ... added in that order; eight loads are
  // issued before their adds so the loop is not a chain of load latencies
  float sum = 0.0f;
  if (i < total) {
    const int64_t stride = (int64_t)Kp * Nw;
    const float* p = partial + src;
    int sp = grp;
    for (; sp + 28 < splits; sp += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(sp + 4 * u) * stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) sum += v[u];
    }
    for (; sp < splits; sp += 4) sum += p[(int64_t)sp * stride];
  }
  red[grp][lane] = sum;
  __syncthreads();
  if (grp == 0 && i < total) {
    const float v = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    const int64_t dst = layout == 0 ? i : (((int64_t)k * C + c) * R + r) * S + s;
    dw[dst] = to_h16(v);
  }
}

// Few splits, KRSC output with unpadded channels (the partial rows are then
// the output rows): each thread adds four consecutive outputs over all splits
// in split order (16-byte loads, four splits in flight), and rounds once.
__global__ __launch_bounds__(256) void wgrad_reduce_vec_kernel(const float* __restrict__ partial,
                                                               int splits, int64_t total,
                                                               int64_t stride, h16* __restrict__ dw) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= total) return;
  const floatx4* p = reinterpret_cast<const floatx4*>(partial + i);
  const int64_t st4 = stride / 4;
  floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  int sp = 0;
  for (; sp + 4 <= splits; sp += 4) {
    const floatx4 v0 = p[(sp + 0) * st4], v1 = p[(sp + 1) * st4];
    const floatx4 v2 = p[(sp + 2) * st4], v3 = p[(sp + 3) * st4];
    acc += v0;
    acc += v1;
    acc += v2;
    acc += v3;
  }
  for (; sp < splits; ++sp) acc += p[sp * st4];
  union {
    h16 h[4];
    uint2 u;
  } o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o.h[e] = to_h16(acc[e]);
  *reinterpret_cast<uint2*>(dw + i) = o.u;
}

// Tile configuration shared by the plan and the launch.
struct WCfg {
  int BM, BN;
  int S = 2;   // stages of the DMA ring
  int NW = 4;  // waves
};
// From 65 output channels and 65 filter columns on: eight waves, one workgroup
// per CU, the tile of the least
//   rounds * k-steps of a split * area * 0.62 + splits * K * Nw * 8 / 4e6  (us)
// among 128 x 128 and, where those come in a count that divides 256 badly,
// 256 x 128 and 128 x 256 (area 2), with 256 / tiles splits: a 128 x 128 k-step
// takes 0.62 us at full load, and each partial sum moves 8 bytes at 4 TB/s.
// Measured with the reduction, batch 128: 14x14 256 -> 256 3x3 55.5 -> 42.0 us
// (four waves on 128 x 64, two workgroups per CU, 576 of them for 512 slots),
// 28x28 128 -> 128 47.3 -> 42.3, 7x7 512 -> 512 53.4 -> 41.7 (256 x 128; 54 on
// 128 x 128), 56x56 256 -> 512 1x1/2 49.8 -> 40.8, 14x14 256 -> 1024 28.6 ->
// 26.1.
// Fewer channels or columns: four waves, the tile that pads the columns less
// (64 x 192 tiles cover a 3x3 64-channel filter's 576 columns exactly, where
// 64 x 256 tiles left a quarter of the third empty: conv2_x 60.4 -> 53.5 us).
inline WCfg wgrad_choice(int K, int Nw, int64_t npix) {
  if (K > 64 && Nw > 64) {
    // a few k-steps of many tiles are the writing of partial sums, better by two
    // workgroups per CU (432 pixels, 1024 x 4608: 26.9 -> 24.2 us)
    if (npix <= 8 * BKP && ceil_div(K, 128) * ceil_div(Nw, 128) > 256) return {128, 64, 3};
    static constexpr int kShapes[3][2] = {{128, 128}, {256, 128}, {128, 256}};
    WCfg best{128, 128, 3, 8};
    double cost = 1e30;
    for (const auto& t : kShapes) {
      const int64_t tiles = (int64_t)ceil_div(K, t[0]) * ceil_div(Nw, t[1]);
      const int64_t splits = tiles < 256 ? 256 / tiles : 1;
      const int64_t steps = ceil_div64(ceil_div64(npix, BKP), splits);
      const double c = (double)ceil_div64(tiles * splits, 256) * (double)steps * 0.62 *
                           (t[0] * t[1] / 16384) +
                       (double)splits * K * Nw * 8.0 / 4.0e6;
      if (c < cost) {
        cost = c;
        best.BM = t[0];
        best.BN = t[1];
      }
    }
    return best;
  }
  if (K > 64) return {128, 64, 3};
  if (Nw <= 64) return {64, 64};
  if (Nw <= 128) return {64, 128};
  return ceil_div(Nw, 192) * 192 < ceil_div(Nw, 256) * 256 ? WCfg{64, 192} : WCfg{64, 256, 3, 8};
}

template <bool CGEN>
void launch_wgrad7(const WCfg& cfg, dim3 grid, hipStream_t st, const WgradArgs& a) {
  if (cfg.NW == 8) {
    if (cfg.BM == 256)
      hipLaunchKernelGGL((wgrad7_kernel<256, 128, 4, 2, 3, CGEN>), grid, dim3(512), 0, st, a);
    else if (cfg.BM == 64)
      hipLaunchKernelGGL((wgrad7_kernel<64, 256, 2, 4, 3, CGEN>), grid, dim3(512), 0, st, a);
    else if (cfg.BN == 256)
      hipLaunchKernelGGL((wgrad7_kernel<128, 256, 2, 4, 3, CGEN>), grid, dim3(512), 0, st, a);
    else
      hipLaunchKernelGGL((wgrad7_kernel<128, 128, 4, 2, 3, CGEN>), grid, dim3(512), 0, st, a);
    return;
  }
  if (cfg.BM == 128)
    hipLaunchKernelGGL((wgrad7_kernel<128, 64, 2, 2, 3, CGEN>), grid, dim3(256), 0, st, a);
  else if (cfg.BN == 192)
    hipLaunchKernelGGL((wgrad7_kernel<64, 192, 2, 2, 2, CGEN>), grid, dim3(256), 0, st, a);
  else if (cfg.BN == 128)
    hipLaunchKernelGGL((wgrad7_kernel<64, 128, 2, 2, 2, CGEN>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((wgrad7_kernel<64, 64, 2, 2, 2, CGEN>), grid, dim3(256), 0, st, a);
}

}  // namespace

void wgrad_plan(int K, int Cp, int R, int S, int64_t npix, int target, int64_t room, int* splits,
                int* pix_per_split) {
  const int Nw = R * S * Cp;
  const WCfg cfg = wgrad_choice(K, Nw, npix);
  const int64_t tiles = (int64_t)ceil_div(K, cfg.BM) * ceil_div(Nw, cfg.BN);
  // one workgroup per CU for the eight-wave kernel and for 1x1 filters, which
  // are bound by reading x and dy (56x56 64 -> 256 at batch 128: 44 us with 256
  // workgroups, 51 with 512); never more than the target, where a few more
  // than the slots cost a round (14x14: 576 workgroups for 512 slots)
  if ((cfg.NW == 8 || R * S == 1) && target > 256) target = 256;
  int64_t want = target / tiles;
  const int64_t steps = ceil_div64(npix, BKP);
  // k-steps of a split: four or more, or two where that leaves most CUs idle
  // (9 steps, 256 x 176: 8.2 -> 7.4 us)
  int64_t max_splits = ceil_div64(steps, 4);
  if (max_splits * tiles < 64) max_splits = min(ceil_div64(steps, 2), ceil_div64(64, tiles));
  if (want > max_splits) want = max_splits;
  // eight or more on the eight-wave kernel if that still fills half the CUs: fewer
  // partial sums (14x14 256 -> 1024 1x1 at batch 32, 6 steps a split on 16 splits
  // 21.6 us, 12 steps on 8 splits 18.3; 3x3 128 -> 128 over 6,272 pixels 17.0 and
  // 15.0; with 12 steps a split and more the longer ones lose)
  const int64_t half = 128 / tiles;
  if (cfg.NW == 8 && want > half && want * 8 > steps) want = max(half, steps / 8);
  if (want < 1) want = 1;
  auto per_split = [&](int64_t n) { return ceil_div64(ceil_div64(npix, n), BKP) * BKP; };
  int64_t pps = per_split(want);
  const int64_t n = ceil_div64(npix, pps);
  if (n > room && room >= 1) {
    const int64_t t4 = K >= 128 ? (int64_t)ceil_div(K, 128) * ceil_div(Nw, 64)
                                : (int64_t)ceil_div(K, 64) * ceil_div(Nw, Nw >= 128 ? 128 : 64);
    const int64_t w4 = min(ceil_div64(kWgradWorkgroups, t4), ceil_div64(npix, 2 * BKP));
    if (ceil_div64(npix, per_split(w4)) <= room) pps = per_split(room);
  }
  *pix_per_split = (int)pps;
  *splits = (int)((npix + pps - 1) / pps);
  if (*splits < 1) *splits = 1;
}

void wgrad_name(int K, int Cp, int R, int S, int64_t npix, char* out, size_t bytes) {
  const WCfg c = wgrad_choice(K, R * S * Cp, npix);
  snprintf(out, bytes, "%dx%d %d waves%s", c.BM, c.BN, c.NW, Cp % 64 != 0 ? " taps" : "");
}

hipError_t launch_wgrad_partial(const WgradArgs& a, hipStream_t st) {
  const int Nw = a.R * a.S * a.C;
  const WCfg cfg = wgrad_choice(a.K, Nw, (int64_t)a.N * a.P * a.Q);
  const int tiles = ceil_div(a.K, cfg.BM) * ceil_div(Nw, cfg.BN);
  const dim3 grid(tiles, a.splits);
  // channel counts that are not multiples of 64 take per-lane filter taps
  if (a.C % 64 != 0)
    launch_wgrad7<true>(cfg, grid, st, a);
  else
    launch_wgrad7<false>(cfg, grid, st, a);
  return hipGetLastError();
}

// Split-K partial sums folded in place: block (b, g) adds, for the 64
// float4 columns [64b, 64b + 64) of the split rows (row4 float4 each), the
// splits [g*kFoldGs, (g+1)*kFoldGs) of group g and writes the sum over the
// group's first split.  Wave w takes the group's splits w, w + 4, ... in
// order (all of its loads in flight; a split past the last is loaded
// clamped, in bounds, and not added), then the four wave sums are added in
// order.  Only this block reads or writes these elements of these splits.
constexpr int kFoldGs = 16;

__global__ __launch_bounds__(256) void wgrad_fold_kernel(float* part, int splits, int64_t row4) {
  __shared__ float4 red[3][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t col = (int64_t)blockIdx.x * 64 + lane;
  const bool live = col < row4;
  const int64_t cc = live ? col : 0;
  const int g0 = blockIdx.y * kFoldGs;
  float4* p = reinterpret_cast<float4*>(part);
  constexpr int U = kFoldGs / 4;
  float4 v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int sp = g0 + w + 4 * u;
    v[u] = p[(int64_t)(sp < splits ? sp : splits - 1) * row4 + cc];
  }
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (g0 + w + 4 * u < splits) {
      acc.x += v[u].x;
      acc.y += v[u].y;
      acc.z += v[u].z;
      acc.w += v[u].w;
    }
  }
  if (w > 0) red[w - 1][lane] = acc;
  __syncthreads();
  if (w != 0 || !live) return;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    acc.x += red[i][lane].x;
    acc.y += red[i][lane].y;
    acc.z += red[i][lane].z;
    acc.w += red[i][lane].w;
  }
  p[(int64_t)g0 * row4 + col] = acc;
}

// The stem's weight gradient computed as a 4x4 stride-1 convolution over the
// 2x2 space-to-depth image (16 channels, (dh*2 + dw)*3 + c): original tap
// (r, s, c) is s2d tap ((r+1)/2, (s+1)/2) at channel (((r+1)%2)*2 + (s+1)%2)*3
// + c.  dw[k][r][s][c] (KRSC, 7x7x3) = rne16(sum over the groups, in order, of
// the folded partial[g * kFoldGs][k][(r'*4 + s')*16 + ch]).
__global__ __launch_bounds__(256) void wgrad_reduce_s2d3_kernel(const float* __restrict__ partial,
                                                                 int groups, int64_t stride,
                                                                 int K, h16* __restrict__ dw) {
  const int i = blockIdx.x * 256 + threadIdx.x;  // enumerates k, r, s, c
  if (i >= K * 147) return;
  const int c = i % 3, rs = (i / 3) % 49, k = i / 147;
  const int r = rs / 7, s = rs % 7;
  const int rp = (r + 1) >> 1, sp = (s + 1) >> 1;
  const int ch = (((r + 1) & 1) * 2 + ((s + 1) & 1)) * 3 + c;
  const float* p = partial + (int64_t)k * 256 + (rp * 4 + sp) * 16 + ch;
  constexpr int U = 8;
  float acc = 0.0f;
  for (int g0 = 0; g0 < groups; g0 += U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = p[(int64_t)(g0 + u < groups ? g0 + u : groups - 1) * stride];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g0 + u < groups) acc += v[u];
  }
  dw[i] = to_h16(acc);
}

hipError_t launch_wgrad_reduce_s2d3(float* partial, int splits, int K, h16* dw, hipStream_t st) {
  const int64_t row4 = (int64_t)K * 256 / 4;
  const int groups = (splits + kFoldGs - 1) / kFoldGs;
  hipLaunchKernelGGL(wgrad_fold_kernel, dim3((unsigned)((row4 + 63) / 64), groups), dim3(256), 0,
                     st, partial, splits, row4);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(wgrad_reduce_s2d3_kernel, dim3((K * 147 + 255) / 256), dim3(256), 0, st,
                     partial, groups, (int64_t)kFoldGs * K * 256, K, dw);
  return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const float* partial, int splits, int K, int Kp, int R, int S, int C,
                               int Cp, int layout, h16* dw, hipStream_t st) {
  const int64_t total = (int64_t)K * R * S * C;
  if (layout == 0 && C == Cp && splits <= 32) {
    const int64_t threads = total / 4;  // C % 8 == 0 here
    hipLaunchKernelGGL(wgrad_reduce_vec_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0,
                       st, partial, splits, total, (int64_t)Kp * R * S * Cp, dw);
    return hipGetLastError();
  }
  const int64_t blocks = (total + 63) / 64;
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, st, partial, splits,
                     K, Kp, R, S, C, Cp, layout, dw);
  return hipGetLastError();
}

}  // namespace fp16k
