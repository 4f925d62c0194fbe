// Fused +/- adapted GEMM for few tokens (gfx950): the depth split over workgroups.
//
// Same contraction as the 256 x 256 persistent schedule (k_gemm_4w64.hip): y[h] = x[h] W^T +
// b + p[h] C_h^T, W read once for both halves.  Where 2 T tokens give fewer 256 x 256 tiles
// than the chip has compute units, that schedule leaves most of the chip idle and every busy
// workgroup walks the whole depth; the time is then depth x stage time whatever T is.  Here:
//
//  * a workgroup owns 128 features x NB 16-token blocks (NB = 2, 4 or 8).  Blocks are counted
//    over both halves (each half padded to whole blocks), so one tile holds both halves of a
//    short batch and W crosses L2 -> LDS once for them;
//  * the depth is split over S workgroups (slices of whole 64-deep stages); each stores its
//    fp32 accumulators, and a second kernel adds the slices in the order 0 .. S - 1 and runs
//    the epilogue.  The slices depend on (T, N, K) and the workspace only, so the halves, the
//    shared-input form and the INT4 form of a call give the same bits as each other;
//  * 64-deep stages through LDS: three 16 KB W slots and two x slots (80 KB at NB = 8), so two
//    workgroups share a CU and hide each other's waits.  W of stage S + 2 is requested during
//    the first sub-step of stage S, x of S + 2 during the second, one barrier per stage.
//    INT4 weights travel packed (4 KB and the scales per stage) and are dequantised in the
//    registers of the one wave that multiplies them.
//
// What bounds it: at 16 to 64 tokens the W bytes from HBM; above, the L2 -> LDS rate (13 to 14
// TB/s over the chip whatever the occupancy, ring depth or store kind).  Measured with a workspace
// and weights from HBM against the 256 x 256 schedule with its split tail (us, bf16, 16 / 64 / 256
// / 512 / 768 / 1024 tokens per half; "=": that schedule is the one chosen):
//   q|k|v 4096 -> 6144    18 / 23 / 43 / 58 / = / =         42 / 42 / 46 / 74 / 82 / 87
//   o 4096 -> 4096        16 / 19 / 31 / 43 / 59 / 65       36 / 37 / 39 / 52 / 72 / 76
//   gate|up 4096 -> 28672 56 / 62 / = / = / = / =           88 / 91 / 102 / 200 / 287 / 371
//   down 14336 -> 4096    38 / 42 / 69 / 118 / 182 / 211    65 / 65 / 74 / 110 / 158 / 191
//   out 5120 -> 5120      23 / 30 / 43 / 86 / 80 / =        42 / 43 / 49 / 78 / 96 / 101
//   fc2 20480 -> 5120     66 / 69 / 115 / 307 / 290 / =     117 / 119 / 138 / 220 / 329 / 382
// and INT4 against its whole tiles: o 19 / 24 / 38 / 56 / 81 / 82 (101 to 106 throughout), down 42 /
// 42 / 81 / 143 / 253 / 262 (331 to 336).
#include <algorithm>
#include <type_traits>

#include "gemm_4w_epi.hpp"

namespace zoact {

namespace {

using namespace gemm;

constexpr int NT = 256;

// LDS of one variant: per stage a W slot (bf16: 128 rows x 128 bytes; INT4: the packed rows, 32
// bytes each, and one 4-byte scale slot for each of 4 x 64 lanes) and an x slot; XR stages of
// x and XR + 1 of W.
constexpr int w_slot(bool i4) { return i4 ? 128 * 32 + 1024 : 128 * 128; }
constexpr int lds_bytes(int nb, int xr, bool i4) { return (xr + 1) * w_slot(i4) + xr * nb * 2048; }

// Tiles and slices of one launch.
struct SPlan {
  int32_t nbt;      // 16-token blocks per half
  int32_t tiles_m;  // token tiles over both halves (one half's, shared input)
  int32_t tiles_n;  // 128-feature tiles
  int32_t nslice;   // depth slices S
  int32_t n_begin;  // first feature
};

// Byte offset of (row, 16-byte chunk c) in a 64-deep operand tile (rows of 128 bytes).
__device__ __forceinline__ int swz64(int row, int c) { return (row << 7) + ((c ^ (row & 7)) << 4); }

template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Direct-to-LDS load of 16 bytes per lane: lane l lands at dst + 16 l.  (A function of its own:
// called inside a template the builtin stops the host pass from emitting the kernel's stub.)
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rs, char* dst, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)dst, 16, voff, soff, 0, 0);
}

__device__ __forceinline__ void dma2(__amdgpu_buffer_rsrc_t rs, char* dst, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)dst, 2, voff, soff, 0, 0);
}

// Half and first token of 16-token block b.
template <bool SHARED>
__device__ __forceinline__ void block_pos(const SPlan& pl, int b, int& half, int& t0) {
  half = (!SHARED && b >= pl.nbt) ? 1 : 0;
  t0 = (b - half * pl.nbt) * 16;
}

// Depth slice s of S over NS stages: [NS s / S, NS (s + 1) / S).
__device__ __forceinline__ int slice_begin(int NS, int s, int S) { return NS * s / S; }

// fp32 accumulators of one tile and slice: [wave][i * NJ + j][lane] x float4.  Slices of a tile
// lie together; with a shared input slice 0 (which carries the correction) has one copy per
// half, the others one for both.
template <int NB, bool SHARED>
__device__ __forceinline__ floatx4* part_slot(const GemmArgs& a, const SPlan& pl, int tile, int slice, int half,
                                              int wave) {
  const int per = SHARED ? pl.nslice + 1 : pl.nslice;
  const int idx = SHARED ? (slice == 0 ? half : slice + 1) : slice;
  return reinterpret_cast<floatx4*>(a.tail_ws) + (((int64_t)tile * per + idx) * 4 + wave) * (NB * 2) * 64;
}

// Rank-r correction of half h added to the blocks j with half_j[j] == h (all of them with a
// shared input): ceil(r/32) 32-deep steps on p[h] and C_h from global memory, columns past r
// and rows past T or N zero.
template <bool PERM, bool SHARED, int NI, int NJ>
__device__ __forceinline__ void correct(const GemmArgs& a, floatx4 (&acc)[NI][NJ], const int (&half_j)[NJ],
                                        const int (&tok_j)[NJ], int h, int64_t nw, int lane) {
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t plen = a.plain_end - a.plain_begin;
  const int64_t cw = nw >= a.plain_end ? nw - plen : nw;   // coefficient row of feature nw
  const int64_t crows = a.N - plen;
  const uint16_t* cb = a.ch + (int64_t)h * a.ch_stride;
  const uint16_t* pb = a.p + (SHARED ? 0 : (int64_t)h * a.T * a.r);
  const int r = a.r;
  // 16-byte loads where rows of 8 start on them (a caller's p may be less aligned)
  const bool vec = (r & 7) == 0 && ((reinterpret_cast<uintptr_t>(cb) | reinterpret_cast<uintptr_t>(pb)) & 15) == 0;
  auto frag = [&](const uint16_t* base, int64_t row, bool in, int col) -> bf16x8 {
    uint4 u = make_uint4(0u, 0u, 0u, 0u);
    if (in && col < r) {
      if (vec) {
        u = *reinterpret_cast<const uint4*>(base + row * r + col);
      } else {
        uint16_t e[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) e[q] = col + q < r ? base[row * r + col + q] : (uint16_t)0;
        u = make_uint4(pack2(e[0], e[1]), pack2(e[2], e[3]), pack2(e[4], e[5]), pack2(e[6], e[7]));
      }
    }
    return __builtin_bit_cast(bf16x8, u);
  };
  for (int col0 = 0; col0 < r; col0 += 32) {
    const int col = col0 + lk * 8;
    bf16x8 fa[NI], fb[NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int64_t row = cw + (PERM ? (i >> 1) * 32 + (lr >> 2) * 8 + (i & 1) * 4 + (lr & 3) : i * 16 + lr);
      fa[i] = frag(cb, row, row < crows, col);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) fb[j] = frag(pb, tok_j[j] + lr, tok_j[j] + lr < a.T, col);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (!SHARED && half_j[j] != h) continue;   // uniform
#pragma unroll
      for (int i = 0; i < NI; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
  }
}

// WF: waves along the features (4 / WF along the tokens).
// XR: stages of x in LDS.
template <int EPI, bool OUT_F32, int NB, int WF, int XR, bool SHARED, bool I4>
__global__ void __launch_bounds__(NT, (lds_bytes(NB, XR, I4) <= 81920 ? 2 : 1)) gemm_s_kernel(GemmArgs a, SPlan pl) {
  constexpr bool PERM = epi_perm(EPI);
  constexpr int WT = 4 / WF, NI = 8 / WF, NJ = NB / WT;
  constexpr int X_SLOT = NB * 16 * 128, WR = XR + 1;
  constexpr int W_SLOT = w_slot(I4);
  constexpr int WL = I4 ? 2 : 4, XL = NB / 2;   // direct-to-LDS loads per wave and stage
  extern __shared__ __align__(16) uint16_t lds[];
  char* const lw = reinterpret_cast<char*>(lds);
  char* const lx = lw + WR * W_SLOT;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, lk = lane >> 4;

  // token tiles of one (feature tile, slice) are consecutive workgroups of one XCD, so its W
  // is fetched into one L2; feature tiles of a slice come next (they share x's slice)
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const int q = (local / pl.tiles_m) * 8 + xcd, tm = local % pl.tiles_m;
  if (q >= pl.tiles_n * pl.nslice) return;
  const int tn = q % pl.tiles_n, slice = q / pl.tiles_n;
  const int NS = (int)(a.K >> 6);
  const int s0 = slice_begin(NS, slice, pl.nslice), nst = slice_begin(NS, slice + 1, pl.nslice) - s0;
  const int64_t n0 = pl.n_begin + (int64_t)tn * 128;
  const int wn0 = (wave % WF) * (NI * 16), wm0 = (wave / WF) * (NJ * 16);

  // per-lane byte offsets of this wave's loads (row and swizzled chunk; OFF_NONE for rows past
  // the ends, which then read zeros); the depth goes in the scalar offset
  const __amdgpu_buffer_rsrc_t wrs = buffer_rsrc(a.w, (uint32_t)(I4 ? a.N * (a.K >> 1) : a.N * a.K * 2));
  const __amdgpu_buffer_rsrc_t srs = buffer_rsrc(a.wsc, (uint32_t)(I4 ? a.N * (a.K >> 7) * 2 : 0));
  const __amdgpu_buffer_rsrc_t xrs = buffer_rsrc(a.x, (uint32_t)((SHARED ? 1 : 2) * a.T * a.K * 2));
  const int chunk = ((lane & 7) ^ (lane >> 3)) << 4;
  int wo[WL], xo[XL];
  if constexpr (I4) {
    // a wave's 32 rows lie in LDS in the order their fragments are read (block, then row): its
    // packed load moves two 16-byte halves per row, its scale load one value per row
    auto grow = [&](int r) -> int64_t {
      const int f = r & 15, h = r >> 4;
      return n0 + wave * 32 + (PERM ? (f >> 2) * 8 + h * 4 + (f & 3) : r);
    };
    const int64_t np = grow(lane >> 1), ns = grow(lane & 31);
    wo[0] = np < a.N ? (int)(np * (a.K >> 1)) + (lane & 1) * 16 : OFF_NONE;
    wo[1] = lane < 32 && ns < a.N ? (int)(ns * (a.K >> 7) * 2) : OFF_NONE;
  } else {
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int64_t n = n0 + wave * 32 + i * 8 + (lane >> 3);
      wo[i] = n < a.N ? (int)(n * a.K * 2) + chunk : OFF_NONE;
    }
  }
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int rr = wave * (NB * 4) + i * 8;
    int half, t0;
    block_pos<SHARED>(pl, tm * NB + (rr >> 4), half, t0);
    const int64_t t = t0 + (rr & 15) + (lane >> 3);
    xo[i] = t < a.T ? (int)((half * a.T + t) * a.K * 2) + chunk : OFF_NONE;
  }
  // stage st of this slice (st >= nst: nothing is fetched, zeros land in a slot nobody reads)
  auto load_w = [&](int st, int slot) {
    const bool in = st < nst;
    if constexpr (I4) {
      dma16(wrs, lw + slot * W_SLOT + wave * 1024, in ? wo[0] : OFF_NONE, in ? (s0 + st) * 32 : 0);
      dma2(srs, lw + slot * W_SLOT + 4096 + wave * 256, in ? wo[1] : OFF_NONE, in ? ((s0 + st) >> 1) * 2 : 0);
    } else {
      const int k = in ? (s0 + st) * 128 : 0;
#pragma unroll
      for (int i = 0; i < WL; ++i)
        dma16(wrs, lw + slot * W_SLOT + (wave * 32 + i * 8) * 128, in ? wo[i] : OFF_NONE, k);
    }
  };
  auto load_x = [&](int st, int slot) {
    const int k = st < nst ? (s0 + st) * 128 : 0;
#pragma unroll
    for (int i = 0; i < XL; ++i)
      dma16(xrs, lx + slot * X_SLOT + (wave * (NB * 4) + i * 8) * 128, st < nst ? xo[i] : OFF_NONE, k);
  };

  // W fragment of block i, k-half kh, as it lies in LDS (rows interleaved per block pair with
  // PERM): 8 bf16 values, or 8 packed ones and the row's scale, dequantised when used
  using wraw = std::conditional_t<I4, uint2, bf16x8>;
  const int prow = (lr >> 2) * 8 + (lr & 3);
  auto wfrag = [&](int slot, int i, int kh) -> wraw {
    if constexpr (I4) {
      const int grp = (wn0 >> 5) + (i >> 1), r = (i & 1) * 16 + lr;
      const char* b = lw + slot * W_SLOT;
      return make_uint2(*reinterpret_cast<const uint32_t*>(b + grp * 1024 + r * 32 + kh * 16 + lk * 4),
                        *reinterpret_cast<const uint32_t*>(b + 4096 + grp * 256 + r * 4));
    } else {
      const int row0 = wn0 + (PERM ? (i >> 1) * 32 : i * 16);
      const int fo = PERM ? swz64(prow + (i & 1) * 4, 4 * kh + lk) : swz64(lr, 4 * kh + lk);
      return *reinterpret_cast<const bf16x8*>(lw + slot * W_SLOT + row0 * 128 + fo);
    }
  };
  auto wval = [&](const wraw& w) -> bf16x8 {
    if constexpr (I4) return __builtin_bit_cast(bf16x8, dequant8(w.x, bf2f((uint16_t)w.y)));
    else return w;
  };
  auto xfrag = [&](int slot, int j, int kh) -> bf16x8 {
    return *reinterpret_cast<const bf16x8*>(lx + slot * X_SLOT + (wm0 + j * 16) * 128 + swz64(lr, 4 * kh + lk));
  };

  floatx4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  wraw fa0[NI], fa1[NI];
  bf16x8 fb0[NJ], fb1[NJ];

#pragma unroll
  for (int st = 0; st < XR; ++st) {
    load_w(st, st);
    load_x(st, st);
  }
  wait_vm<(XR - 1) * (WL + XL)>();
  barrier();
#pragma unroll
  for (int i = 0; i < NI; ++i) fa0[i] = wfrag(0, i, 0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) fb0[j] = xfrag(0, j, 0);

  // issue order of a sub-step: each memory instruction right after an MFMA, in whose shadow
  // its issue cycles fall (nv loads, then the NI + NJ fragment reads)
  auto interleave = [&](auto nv_) {
    constexpr int nv = decltype(nv_)::value;
    constexpr int nm = NI * NJ, nd = NI + NJ;
    if constexpr (!I4 && nm >= nv + nd) {
#pragma unroll
      for (int k = 0; k < nd; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
#pragma unroll
      for (int k = 0; k < nv; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, nm - nv - nd, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  using LoadsW = std::integral_constant<int, WL>;
  using LoadsX = std::integral_constant<int, XL>;
  __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
  int ws = 0, xs = 0;   // slots of the current stage
  const int nsub = 2 * nst;
  for (int sub = 0; sub < nsub; sub += 2) {
    const int st = sub >> 1;
    const int ws1 = ws == WR - 1 ? 0 : ws + 1, wsl = ws == 0 ? WR - 1 : ws - 1;
    // first sub-step: k-half 0; W of stage st + XR into the slot stage st - 1 has left
    load_w(st + XR, wsl);
#pragma unroll
    for (int i = 0; i < NI; ++i) fa1[i] = wfrag(ws, i, 1);
#pragma unroll
    for (int j = 0; j < NJ; ++j) fb1[j] = xfrag(xs, j, 1);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const bf16x8 w = wval(fa0[i]);
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, fb0[j], acc[i][j], 0, 0, 0);
    }
    interleave(LoadsW{});
    // stage st + 1 has landed (what was requested after it may stay in flight), and every wave holds its last
    // fragments of stage st
    wait_vm<(XR - 1) * WL + (XR - 2) * XL>();
    __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
    barrier();
    // second sub-step: k-half 1; x of stage st + XR into this stage's slot
    if (sub + 1 < nsub) {   // (always: written as a test, the accumulators stay in place)
      load_x(st + XR, xs);
      xs = xs == XR - 1 ? 0 : xs + 1;
#pragma unroll
      for (int i = 0; i < NI; ++i) fa0[i] = wfrag(ws1, i, 0);
#pragma unroll
      for (int j = 0; j < NJ; ++j) fb0[j] = xfrag(xs, j, 0);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const bf16x8 w = wval(fa1[i]);
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, fb1[j], acc[i][j], 0, 0, 0);
      }
      interleave(LoadsX{});
      __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
      __builtin_amdgcn_sched_barrier(0);
    }
    ws = ws1;
  }
  // the loads past the last stage land (as zeros) before the workgroup ends
  __builtin_amdgcn_s_waitcnt(WAIT_VM0);

  int half_j[NJ], tok_j[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) block_pos<SHARED>(pl, tm * NB + (wm0 >> 4) + j, half_j[j], tok_j[j]);
  const int64_t nw = n0 + wn0;
  const bool corr = a.r > 0 && slice == 0 && !(n0 >= a.plain_begin && n0 < a.plain_end);
  const int tile = tm * pl.tiles_n + tn;
  const bool split = pl.nslice > 1;

  auto out = [&](const floatx4 (&c)[NI][NJ], int h) {   // h: the half (shared input), else per block
    if (split) {
      floatx4* slot = part_slot<NB, SHARED>(a, pl, tile, slice, h, wave);
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) slot[(i * NJ + j) * 64 + lane] = c[i][j];
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        floatx4 v[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) v[i] = c[i][j];
        emit<EPI, OUT_F32, NI>(a, v, SHARED ? h : half_j[j], tok_j[j] + lr, nw, lk);
      }
    }
  };
  if constexpr (SHARED) {
    if (corr || !split) {
      floatx4 a0[NI][NJ];
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) a0[i][j] = acc[i][j];
      if (corr) correct<PERM, true, NI, NJ>(a, a0, half_j, tok_j, 0, nw, lane);
      out(a0, 0);
      if (corr) correct<PERM, true, NI, NJ>(a, acc, half_j, tok_j, 1, nw, lane);
      out(acc, 1);
    } else if (slice == 0) {
      out(acc, 0);
      out(acc, 1);
    } else {
      out(acc, 0);
    }
  } else {
    if (corr) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        bool any = false;
#pragma unroll
        for (int j = 0; j < NJ; ++j) any = any || half_j[j] == h;
        if (any) correct<PERM, false, NI, NJ>(a, acc, half_j, tok_j, h, nw, lane);
      }
    }
    out(acc, 0);
  }
}

// Adds a tile's slices (0 first) and runs the epilogue: one wave per 32 features x 16 tokens
// (block pair q, token block j of a wave tile) and half.
template <int EPI, bool OUT_F32, int NB, int WF, bool SHARED>
__global__ void __launch_bounds__(NT) combine_s_kernel(GemmArgs a, SPlan pl, int nunits) {
  constexpr int WT = 4 / WF, NI = 8 / WF, NJ = NB / WT, NQ = NI / 2;
  const int lane = threadIdx.x & 63;
  const int u = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (u >= nunits) return;
  const int q = u % NQ, j = (u / NQ) % NJ, wave = (u / (NQ * NJ)) & 3, rest = u / (NQ * NJ * 4);
  const int ntile = pl.tiles_m * pl.tiles_n;
  const int tile = rest % ntile, h = rest / ntile;   // (h: the half, shared input only)
  const int tm = tile / pl.tiles_n, tn = tile % pl.tiles_n;
  int half, t0;
  block_pos<SHARED>(pl, tm * NB + (wave / WF) * NJ + j, half, t0);
  if (SHARED) half = h;
  if (t0 >= a.T) return;   // a block past the last (uniform)
  floatx4 v[2];
  const int o0 = (2 * q * NJ + j) * 64 + lane, o1 = o0 + NJ * 64;
  const floatx4* s0 = part_slot<NB, SHARED>(a, pl, tile, 0, half, wave);
  v[0] = s0[o0], v[1] = s0[o1];
#pragma unroll 8
  for (int s = 1; s < pl.nslice; ++s) {
    const floatx4* sp = part_slot<NB, SHARED>(a, pl, tile, s, 0, wave);
    v[0] += sp[o0], v[1] += sp[o1];
  }
  emit<EPI, OUT_F32, 2>(a, v, half, t0 + (lane & 15),
                        pl.n_begin + (int64_t)tn * 128 + (wave % WF) * (NI * 16) + q * 32, lane >> 4);
}

template <int EPI, bool OUT_F32, int NB, int WF, int XR, bool SHARED, bool I4>
hipError_t launch_s(const GemmArgs& a, const SPlan& pl, hipStream_t s) {
  constexpr int LDS = lds_bytes(NB, XR, I4);
  static bool attr_set = false;  // benign race: every thread sets the same value
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_s_kernel<EPI, OUT_F32, NB, WF, XR, SHARED, I4>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int nq = pl.tiles_n * pl.nslice;
  const unsigned grid = (unsigned)((nq + 7) / 8 * 8 * pl.tiles_m);
  gemm_s_kernel<EPI, OUT_F32, NB, WF, XR, SHARED, I4><<<dim3(grid), dim3(NT), LDS, s>>>(a, pl);
  if (pl.nslice > 1) {
    const int units = pl.tiles_m * pl.tiles_n * 4 * NB * (SHARED ? 2 : 1);   // 32 features x 16 tokens each
    combine_s_kernel<EPI, OUT_F32, NB, WF, SHARED><<<dim3((unsigned)(units / 4)), dim3(NT), 0, s>>>(a, pl, units);
  }
  return hipGetLastError();
}

// Token blocks per tile (0: the 256 x 256 schedule) and depth slices for T tokens per half.
//
// The line between the schedules, and the slices, come from the time each form is bound by, in
// bytes per microsecond, fitted to a sweep over the Llama-3-8B and OPT-13B layer shapes at 16 to
// 2048 tokens per half (96 shapes).  The other side of the line is that schedule's whole tiles
// (1.2 us a stage): its split tail, which a workspace allows with bf16 weights, is not priced, and
// from about 512 tokens per half it is the faster form at some shapes that are kept here (the table
// above: down at 512 to 1024, out and fc2 at 512).  INT4 weights are charged as bf16 bytes:
//  * one workgroup moves at most 55 KB/us from L2 to LDS, all of them 14 TB/s (the L2 rate, which
//    also bounds the 256 x 256 schedule: 64 KB per 1.2 us stage and CU), and W comes from HBM at
//    5 TB/s;
//  * slices cost their partial sums' way out and back (0.3 us per MB) and a second launch.
// The slices depend on (T, N, K) and the workspace only, never on the form of the call, so that
// forms with equal bits keep them.
struct Choice {
  int nb, nslice;
};
Choice choose(int64_t T, int64_t N, int64_t K, int64_t ws_bytes, int ncu) {
  const int NS = (int)(K >> 6);
  const int64_t big_tiles = 2 * ((T + 255) / 256) * ((N + 255) / 256);
  const int64_t rounds = (big_tiles + ncu - 1) / ncu;
  if (rounds > 2) return {0, 1};   // the chip is full with 256 x 256 tiles
  Choice best{0, 1};
  double t_best = 3.0 + (double)rounds * NS * 1.2;
  const int64_t nblk = 2 * ((T + 15) / 16), tn = (N + 127) / 128;
  for (int nb = 2; nb <= 16; nb *= 2) {
    const int64_t tiles = (nblk + nb - 1) / nb * tn;
    const int resident = (nb <= 8 ? 2 : 1) * ncu;
    const double bytes = 16384.0 + 2048.0 * nb;   // per workgroup and stage
    for (int S = 1; S <= 16 && (S == 1 || S * 4 <= NS); ++S) {   // (slices of at least 4 stages)
      const int64_t part = tiles * nb * 8192;
      if (S > 1 && (S + 1) * part > ws_bytes) break;
      const int64_t n = tiles * S;
      const double nst = (NS + S - 1) / S;
      double t = (double)((n + resident - 1) / resident) * nst * bytes / 55e3;
      const double t_l2 = (double)n * nst * bytes / 14e6 * (256.0 / ncu), t_w = (double)N * K * 2 / 5e6;
      t = t > t_l2 ? t : t_l2;
      t = (t > t_w ? t : t_w) + 2.0;
      if (S > 1) t += 2.0 + 0.3e-6 * (double)S * (double)part;
      if (t < t_best) t_best = t, best = {nb, S};
    }
  }
  return best;
}

}  // namespace

// hipErrorNotSupported where the 256 x 256 schedule is the one to use, and outside this
// schedule's coverage: that of the 256 x 256 one (bf16 weights, or INT4 in whole scale groups;
// C_h precomputed or r = 0), plain, ReLU or SwiGLU outputs, both halves of x below 2 GiB.
hipError_t launch_linear_pm_s(const GemmArgs& a, int w_dtype, int epi, bool out_f32, bool shared, hipStream_t s) {
  const bool i4 = w_dtype == ZOACT_INT4_G128;
  if (!i4 && w_dtype != ZOACT_BF16) return hipErrorNotSupported;
  if (a.r > 0 && a.ch == nullptr) return hipErrorNotSupported;
  if (a.r > 256 || (a.K % 64) != 0 || a.K < 128) return hipErrorNotSupported;
  if (2 * a.T * a.K * 2 >= (int64_t(1) << 31) || a.N * a.K * 2 >= (int64_t(1) << 31)) return hipErrorNotSupported;
  if (shared && (i4 || a.r < 8 || a.r > 32 || (a.r & 7) != 0)) return hipErrorNotSupported;
  if (i4 && (a.wsc == nullptr || (a.K % 128) != 0 || a.K < 256)) return hipErrorNotSupported;
  if (a.plain_end > a.plain_begin && (shared || (a.plain_begin & 255) != 0 || (a.plain_end & 255) != 0))
    return hipErrorNotSupported;
  const int ncu = cu_count();
  if (ncu <= 0) return hipErrorInvalidDevice;
  // (the sweep the cost is fitted to had 256 KB per compute unit)
  const int64_t wsb = a.tail_ws ? std::min<int64_t>(a.tail_ws_bytes, (int64_t)ncu * 256 * 1024) : 0;
  const Choice c = choose(a.T, a.N, a.K, wsb, ncu);
  if (c.nb == 0) return hipErrorNotSupported;
  SPlan pl{};
  pl.nbt = (int32_t)((a.T + 15) / 16);
  pl.tiles_m = ((shared ? 1 : 2) * pl.nbt + c.nb - 1) / c.nb;
  pl.tiles_n = (int32_t)((a.N + 127) / 128);
  pl.nslice = c.nslice;
#define ZO_S(EP, OF, SH, I)                                                     \
  if (epi == EP && out_f32 == OF && shared == SH && i4 == I) {                  \
    if (c.nb == 16) return launch_s<EP, OF, 16, I ? 4 : 2, 3, SH, I>(a, pl, s); \
    if (c.nb == 8) return launch_s<EP, OF, 8, I ? 4 : 2, I ? 3 : 2, SH, I>(a, pl, s); \
    if (c.nb == 4) return launch_s<EP, OF, 4, I ? 4 : 2, I ? 5 : 2, SH, I>(a, pl, s); \
    return launch_s<EP, OF, 2, 4, I ? 6 : 3, SH, I>(a, pl, s);                  \
  }
  ZO_S(0, false, false, false)
  ZO_S(0, true, false, false)
  ZO_S(ZOACT_EPI_SWIGLU, false, false, false)
  ZO_S(ZOACT_EPI_RELU, false, false, false)
  ZO_S(0, false, true, false)
  ZO_S(0, true, true, false)
  ZO_S(ZOACT_EPI_RELU, false, true, false)
  ZO_S(0, false, false, true)
  ZO_S(0, true, false, true)
  ZO_S(ZOACT_EPI_SWIGLU, false, false, true)
  ZO_S(ZOACT_EPI_RELU, false, false, true)
#undef ZO_S
  return hipErrorNotSupported;
}

}  // namespace zoact
