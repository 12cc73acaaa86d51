// Device half of libcw for gfx950 (MI355X): the suffix QKV projection with
// rotary embedding, fused with the KV append.
//
// Paper Sec. 1 and 2.1: a prefix hit removes every per-layer prefill step of
// the cached tokens; for the suffix tokens the layer still projects each
// hidden state to its query, key and value heads, rotates queries and keys by
// their absolute position, and stores the new keys and values in the
// request's cache blocks. This kernel does those three steps in one pass:
//
//   y = x W^T (+ b)          x [T, hidden], W [(Hq + 2 Hkv) D, hidden]
//   q, k = rope(y_q, y_k)    rotate-half form at position P_r + i
//   q -> q_out [T, Hq, D];  k -> K cache [blk][g][slot][d];
//   v -> V cache [blk][g][slot][d]
//
// Seven tile shapes serve batches from one token to tens of thousands (kShapes:
// which, and why). The largest, persistent workgroups of 8 wavefronts, one per
// CU, walking tiles of 256 features x 256 tokens:
//  * The product is formed as C^T = W x^T with v_mfma_f32_16x16x32_bf16:
//    A = 16 rows of W, B = 16 token rows of x, 32 hidden per instruction. In
//    the 16x16 accumulator a lane holds one token and 4 consecutive features,
//    so everything the epilogue needs per element (position, block, slot) is
//    per lane. This shape sustains a higher rate than 32x32x16 on random data
//    (the card's power limit lowers the clock less for it).
//  * A wave owns features {j0 .. j0 + 31} and {j0 + D/2 .. + 31} of one head
//    (four 16-row blocks) and 128 tokens (eight 16-token blocks). The two
//    halves are rotary pairs (j, j + D/2) in the same lane and register of two
//    accumulators: the rotation needs no data exchange. The rows of a pair of
//    blocks are staged interleaved (staged_feature), so that a lane's elements
//    of both are 8 consecutive features: one 16-byte store.
//  * Hidden is walked in steps of 64 (two MFMA k-steps). LDS is a ring of five
//    32 KB slots that hold the W rows and the x rows of a step in turn (256
//    rows of one 128-byte line each), filled by load-to-LDS copies (no
//    registers) about two steps ahead; the copies run on across tiles, so the
//    next tile's first steps arrive during a tile's epilogue. Each copy brings
//    8 whole lines (half-line copies run at a fraction of the rate). The
//    16-byte chunk c of LDS row r holds global chunk c ^ ((r >> 1) & 7), so the
//    16 rows read by one operand load hit distinct banks.
//  * The two waves of a SIMD (w and w + 4) alternate: while one issues the 32
//    products of a k-step, the other reads its next operands from LDS and
//    issues copies; a workgroup barrier ends each interval, and the second
//    group runs one interval behind the first. The matrix pipe then always has
//    one wave feeding it, instead of waiting at each step's barrier for every
//    wave's first operands. Both k-steps' W operands are read in the first
//    interval (16 and 8 operand loads), which frees the W slot a step early.
//  * Tiles are numbered XCD-major (workgroup b runs on XCD b % 8), and within
//    an XCD feature tiles vary fastest in groups of 8, so the workgroups that
//    run together on one L2 share their W and x rows.
//  * fp32 accumulation; bias, rotation (fp32 cos/sin from a table the host
//    computes in fp64) and one bf16 rounding in the epilogue.
// Smaller tiles (below) keep this staging, operand layout and epilogue.
// Bound: the matrix pipe under the card's power limit (the clock falls to about
// 1.7 GHz on random data, 2.39 on zeros). T = 16,128, hidden 4,096, 6,144
// features (812 GFLOP), back to back: 567 us, 1.43 PFLOP/s; with one barrier per
// step for all waves, a 2-stage ring and one workgroup per tile 672 us (same card).
// A tile takes 138 k cycles for its 64 steps (131 k of them products of the two
// waves of a SIMD) and 9 k for its epilogue.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <type_traits>

#include "cw_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) int32_t cint32_t;

constexpr int kThreads = 512;                  // 8 wavefronts
constexpr int kTileF = 256;                    // output features per tile
constexpr int kTileT = 256;                    // tokens per tile
constexpr int kStep = 64;                      // hidden elements per pipeline step
constexpr int kRow = kStep * 2;                // bytes of one staged row (one 128-byte line)
constexpr int kSlot = 256 * kRow;              // 32 KB: the W rows or the x rows of a step
constexpr int kSlots = 5;
constexpr int kOwn = kSlot / 8;                // a wave's part of a slot
constexpr int kGroupF = 8;                     // feature tiles per XCD group
constexpr int kBs = cw::kBlockSize;
static_assert(kTileF == 256 && kTileT == 256, "32 W and 32 x rows per wave, four 8-row copies each");
static_assert(kSlots * kSlot <= 160 * 1024, "LDS of one CU");

struct QkvArgs {
  const uint8_t* x;
  const uint8_t* w;
  const uint16_t* bias;
  const float* rope;
  uint16_t* q_out;
  uint16_t* k_cache;
  uint16_t* v_cache;
  const int32_t* bt;
  const int32_t* cu;
  const int32_t* plen;
  int T, hidden, n_feat, bt_stride, batch, hq, hkv, num_blocks;
  int n_ftiles, n_ttiles, per_xcd;
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

__device__ __forceinline__ float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xFFFF0000u); }

// One load-to-LDS copy: lane l's 16 bytes at base + off land at dst + 16 l
// (base and dst wave-uniform, dst through M0). The compiler does not count it:
// the kernel's own waits complete it.
__device__ __forceinline__ void copy16_to_lds(const uint8_t* base, uint32_t off, uint32_t dst) {
  const uint64_t b = reinterpret_cast<uintptr_t>(base);
  const uint64_t bu = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(b >> 32)))) << 32) |
                      uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(b))));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(off), "s"(bu), "s"(__builtin_amdgcn_readfirstlane(dst)) : "memory");
}

// s_waitcnt immediates (gfx9 encoding): vmcnt(n) with lgkmcnt(0), expcnt untouched.
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | (7 << 4) | ((n >> 4) << 14); }

// Chunk swizzle of staged row r (128-byte rows, eight 16-byte chunks): the
// 16 rows of an operand load, two per 256 bytes of banks, take 8 distinct
// positions per row parity.
__device__ __forceinline__ int row_swz(int r) { return (r >> 1) & 7; }

// Feature staged at LDS row s: within each 32 rows, block b = s / 16 of the
// MFMA's 16 rows holds features 8 g + 4 b + e at row 4 g + e, so that a lane's
// accumulator elements of blocks 0 and 1 are 8 consecutive features.
__device__ __forceinline__ int staged_feature(int s) {
  return (s & ~31) | ((s & 12) << 1) | ((s & 16) >> 2) | (s & 3);
}

// Workgroup barrier that no memory access or instruction group moves across.
__device__ __forceinline__ void interval_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Bias, rotation, rounding and stores of one wave's results: features j0 ..
// j0 + 16 FH - 1 of head hf and their partners at + D/2, for the NTB 16-token
// blocks from token tw on (tokens before t_own are another tile's). Element e
// of acc[fa][tb] is feature j0 + 4 FH g + 4 (fa % FH) + e (+ D/2 for fa >= FH)
// of token tw + 16 tb + l16, with g = lane / 16, l16 = lane % 16. `own`: 1 KB x
// 2 FH of LDS no other wave uses.
//
// Lane l first works out position and destination of tokens tw + 64 i + l: the
// requests of the first and last token by bisection over cu (scalar loads), then
// one after the other those in between, or where these are more than kWalk a
// bisection per lane between the two: a longer chain than a few scalar loads,
// but it does not grow with the requests. 6,144 features: 600 tokens of two
// requests with 20,000 empty ones between them, hidden 4,096: 1,855 us by walking
// alone, 68 now; 8,192 one-token requests, hidden 256: 144 / 74; 1,000 requests of
// 3 tokens (42 in a wave's tokens), hidden 4,096: 166 by walking, 169 with 16
// walked and the rest by bisection. The rotation's cos/sin rows
// are loaded whole, one token block ahead (128 FH contiguous bytes per token: a
// load that takes each lane's own 16 bytes touches four times as many lines
// per instruction, and the loads' line rate bounds the epilogue: 11 k cycles
// against 9 k), and reach their lanes through `own`.
template <int D, int FH, int NTB>
__device__ __forceinline__ void store_results(const QkvArgs& a, f32x4 (&acc)[2 * FH][NTB], int hf, int j0, int tw,
                                              int t_own, uint8_t* own, int lane) {
  if (hf >= a.hq + 2 * a.hkv) return;
  cint32_t* const cu = reinterpret_cast<cint32_t*>(reinterpret_cast<uintptr_t>(a.cu));
  cint32_t* const plen = reinterpret_cast<cint32_t*>(reinterpret_cast<uintptr_t>(a.plen));
  const int l16 = lane & 15, g4 = lane >> 4;
  const int kind = hf < a.hq ? 0 : (hf < a.hq + a.hkv ? 1 : 2);   // q, k, v
  const int g = kind == 1 ? hf - a.hq : hf - a.hq - a.hkv;
  constexpr int NM = (NTB + 3) / 4;   // tokens per lane
  const int t_last = max(tw, min(tw + 16 * NTB, a.T) - 1);
  int lo = 0, lo1 = a.batch - 1, hi = 0, hi1 = a.batch - 1;   // requests of tokens tw and t_last
  while (lo < lo1 || hi < hi1) {
    const int m0 = (lo + lo1 + 1) >> 1, m1 = (hi + hi1 + 1) >> 1;
    const int c0 = cu[m0], c1 = cu[m1];
    if (c0 <= tw) lo = m0;
    else lo1 = m0 - 1;
    if (c1 <= t_last) hi = m1;
    else hi1 = m1 - 1;
  }
  constexpr int kWalk = 48;
  int req[NM], shift[NM];   // request, and its position minus token
  if (hi - lo <= kWalk) {
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      req[i] = lo;
      shift[i] = plen[lo] - cu[lo];
    }
    for (int r = lo + 1; r <= hi; ++r) {
      const int c = cu[r];
      const int sh = plen[r] - c;
#pragma unroll
      for (int i = 0; i < NM; ++i)
        if (tw + 64 * i + lane >= c) {
          req[i] = r;
          shift[i] = sh;
        }
    }
  } else {
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      const int t = min(tw + 64 * i + lane, t_last);
      int b0 = lo, b1 = hi;
      while (b0 < b1) {
        const int mid = (b0 + b1 + 1) >> 1;
        if (a.cu[mid] <= t) b0 = mid;
        else b1 = mid - 1;
      }
      req[i] = b0;
      shift[i] = a.plen[b0] - a.cu[b0];
    }
  }
  int pos[NM];        // position, -1 where nothing is written
  uint64_t dst[NM];   // address of the token's row of head hf
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    const int t = tw + 64 * i + lane;
    const int p = min(t, a.T - 1) + shift[i];
    bool ok = t < a.T && t >= t_own;
    if (kind == 0) {
      dst[i] = reinterpret_cast<uintptr_t>(a.q_out) + (uint64_t(uint32_t(t)) * uint32_t(a.hq) + uint32_t(hf)) * (2 * D);
    } else {
      const int blk = ok ? a.bt[int64_t(req[i]) * a.bt_stride + p / kBs] : -1;
      ok = blk >= 0 && blk < a.num_blocks;
      dst[i] = reinterpret_cast<uintptr_t>(kind == 1 ? a.k_cache : a.v_cache) +
               ((uint64_t(uint32_t(blk)) * uint32_t(a.hkv) + uint32_t(g)) * kBs + (p & (kBs - 1))) * (2 * D);
    }
    pos[i] = ok ? p : -1;
  }
  const int j = j0 + 4 * FH * g4;   // the lane's first feature
  if (a.bias) {
#pragma unroll
    for (int fa = 0; fa < 2 * FH; ++fa) {
      const uint16_t* bp = a.bias + int64_t(hf) * D + (fa / FH) * (D / 2) + j + 4 * (fa % FH);
      const uint64_t v = *reinterpret_cast<const uint64_t*>(bp);
      const f32x4 b{bf16_lo(uint32_t(v)), bf16_hi(uint32_t(v)), bf16_lo(uint32_t(v >> 32)), bf16_hi(uint32_t(v >> 32))};
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb) acc[fa][tb] += b;
    }
  }
  auto finish = [&](auto rotate) __attribute__((always_inline)) {
    constexpr bool kRotate = decltype(rotate)::value;
    constexpr int CH = 8 * FH;   // 16-byte chunks of a token's cos/sin pairs
    f32x4 nx[2 * FH], cs[2 * FH];
    auto load_cs = [&](int tb) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 2 * FH; ++i) {
        const int p = max(__shfl(pos[tb >> 2], (tb & 3) * 16 + (64 / CH) * i + lane / CH), 0);
        nx[i] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const uint8_t*>(a.rope) +
                                                uint64_t(uint32_t(p)) * (4 * D) + (j0 * 8 + (lane % CH) * 16));
      }
    };
    if constexpr (kRotate) load_cs(0);
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) {
      if constexpr (kRotate) {
        // chunk c of token r at position c ^ (r % CH) of its row
#pragma unroll
        for (int i = 0; i < 2 * FH; ++i) {
          const int r = (64 / CH) * i + lane / CH;
          *reinterpret_cast<f32x4*>(own + r * (16 * CH) + (((lane % CH) ^ (r % CH)) << 4)) = nx[i];
        }
        asm volatile("" ::: "memory");   // other lanes' writes: not to be forwarded past
        if (tb + 1 < NTB) load_cs(tb + 1);
#pragma unroll
        for (int i = 0; i < 2 * FH; ++i)
          cs[i] = *reinterpret_cast<const f32x4*>(own + l16 * (16 * CH) + (((2 * FH * g4 + i) ^ (l16 % CH)) << 4));
        asm volatile("" ::: "memory");
      }
      const int ps = __shfl(pos[tb >> 2], (tb & 3) * 16 + l16);
      const uint32_t dlo = __shfl(uint32_t(dst[tb >> 2]), (tb & 3) * 16 + l16);
      const uint32_t dhi = __shfl(uint32_t(dst[tb >> 2] >> 32), (tb & 3) * 16 + l16);
      uint32_t o0[2 * FH], o1[2 * FH];
#pragma unroll
      for (int e = 0; e < 2 * FH; ++e) {
        float a0 = acc[e >> 1][tb][(e & 1) * 2], a1 = acc[e >> 1][tb][(e & 1) * 2 + 1];
        float b0 = acc[FH + (e >> 1)][tb][(e & 1) * 2], b1 = acc[FH + (e >> 1)][tb][(e & 1) * 2 + 1];
        if constexpr (kRotate) {
          const f32x4 r = cs[e];   // cos, sin of two rotary indices
          const float ra = fmaf(a0, r[0], -(b0 * r[1])), rb = fmaf(b0, r[0], a0 * r[1]);
          const float sa = fmaf(a1, r[2], -(b1 * r[3])), sb = fmaf(b1, r[2], a1 * r[3]);
          a0 = ra;
          b0 = rb;
          a1 = sa;
          b1 = sb;
        }
        o0[e] = pack_bf16x2(a0, a1);
        o1[e] = pack_bf16x2(b0, b1);
      }
      if (ps >= 0) {
        uint32_t* dp = reinterpret_cast<uint32_t*>(((uint64_t(dhi) << 32) | dlo) + 2 * j);
        typedef uint32_t vec_t __attribute__((ext_vector_type(2 * FH)));
        vec_t v0, v1;
#pragma unroll
        for (int e = 0; e < 2 * FH; ++e) {
          v0[e] = o0[e];
          v1[e] = o1[e];
        }
        *reinterpret_cast<vec_t*>(dp) = v0;
        *reinterpret_cast<vec_t*>(dp + D / 4) = v1;
      }
    }
  };
  if (kind != 2) finish(std::true_type{});
  else finish(std::false_type{});
}

// First feature and token of tile L: feature tiles vary fastest in groups of
// kGroupF, the token tiles within a group.
__device__ __forceinline__ void tile_origin(const QkvArgs& a, int L, int tile_f, int tile_t, int& f0, int& t0) {
  const int grp = L / (kGroupF * a.n_ttiles);
  const int gf = min(kGroupF, a.n_ftiles - grp * kGroupF);
  const int rem = L - grp * kGroupF * a.n_ttiles;
  t0 = (rem / gf) * tile_t;
  f0 = (grp * kGroupF + rem % gf) * tile_f;
}

// Byte offset in a row of W or x of plane p (64 hidden) of `planes`. Past the last
// plane: that plane again, which nothing uses. A last plane of 32 hidden is moved
// back to the row's last 64.
__device__ __forceinline__ int64_t plane_offset(int p, int planes, bool half_last) {
  const int q = min(p, planes - 1);
  return int64_t(q) * kRow - ((half_last && q == planes - 1 && q > 0) ? kRow / 2 : 0);
}

template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void qkv_rope_append_kernel(const QkvArgs a) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kSlots * kSlot];
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));

  // ---- this workgroup's tiles: every 32nd tile of its XCD's range
  const int xcd = blockIdx.x & 7, wg_per_xcd = gridDim.x >> 3;
  const int tile_end = min((xcd + 1) * a.per_xcd, a.n_ftiles * a.n_ttiles);
  int tile = xcd * a.per_xcd + (blockIdx.x >> 3);
  if (tile >= tile_end) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- copy cursor: the tile and step whose rows are copied next. A tile that
  // would reach past the last row of W or x is moved back to end there (its
  // first rows are then another tile's, and not stored), so the lane offsets
  // are the same for every tile.
  const int64_t hb = int64_t(a.hidden) * 2;   // bytes per row of W and x
  const int nk = (a.hidden + kStep - 1) / kStep;
  // the last step holds 32 hidden: it is moved back to the row's last 64 and
  // uses their upper half (a row of 32 has both halves copied from it)
  const bool half_last = (a.hidden % kStep) != 0;
  const int f_max = max(a.n_feat - kTileF, 0), t_max = max(a.T - kTileT, 0);
  int c_tile = tile, c_step = 0;
  const uint8_t *c_w, *c_x;
  uint32_t offw[4], offx[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 32 * wave + 8 * i + (lane >> 3);
    int c = ((lane & 7) ^ row_swz(row)) * 16;
    if (a.hidden < kStep) c &= ~64;
    offw[i] = uint32_t(min(staged_feature(row), a.n_feat - 1)) * uint32_t(hb) + c;
    offx[i] = uint32_t(min(row, a.T - 1)) * uint32_t(hb) + c;
  }
  auto cursor_tile = [&]() __attribute__((always_inline)) {
    int f0, t0;
    tile_origin(a, c_tile, kTileF, kTileT, f0, t0);
    c_w = a.w + int64_t(min(f0, f_max)) * hb;
    c_x = a.x + int64_t(min(t0, t_max)) * hb;
  };
  cursor_tile();
  // the W (x) rows of the cursor's step into ring slot `slot`
  auto issue4 = [&](const uint8_t* base, const uint32_t (&off)[4], int slot) __attribute__((always_inline)) {
    const uint32_t dst = lds0 + slot * kSlot + wave * kOwn;
#pragma unroll
    for (int i = 0; i < 4; ++i) copy16_to_lds(base, off[i], dst + i * 1024);
  };
  auto cursor_next = [&]() __attribute__((always_inline)) {
    if (++c_step < nk) {
      const int d = (half_last && c_step == nk - 1) ? kRow / 2 : kRow;
      c_w += d;
      c_x += d;
    } else if (c_tile + wg_per_xcd < tile_end) {
      c_tile += wg_per_xcd;
      c_step = 0;
      cursor_tile();
    }   // past the last tile: its last step again, which nothing reads
  };

  // ---- operand rows of this wave
  constexpr int kWavesPerHead = D / 64;
  const int wf = wave & 3, wt = wave >> 2;
  const int head_l = wf / kWavesPerHead;
  const int j0 = (wf % kWavesPerHead) * 32;
  const int arow0 = head_l * D + j0;
  const int brow = wt * 128;
  const int l16 = lane & 15;
  const int g4 = lane >> 4;
  // 16-row block starting at a multiple of 16 rows, k-step ks of the slot:
  // lane reads row l16, chunk 4 ks + g4 (swizzled)
  const int so0 = l16 * kRow + ((g4 ^ row_swz(l16)) << 4);
  const int so1 = l16 * kRow + (((4 + g4) ^ row_swz(l16)) << 4);
  // feature blocks: fa = 0, 1 -> rows j0 + 16 fa; fa = 2, 3 -> j0 + D/2 + 16 (fa - 2)
  auto arow = [&](int fa) { return arow0 + (fa >> 1) * (D / 2) + (fa & 1) * 16; };
  auto ld = [&](int addr) __attribute__((always_inline)) -> bf16x8 {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(lds + addr));
  };

  f32x4 acc[4][8];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int fa = 0; fa < 4; ++fa)
#pragma unroll
      for (int tb = 0; tb < 8; ++tb) acc[fa][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();

  // ---- the first two steps' copies; the second is left in flight
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    issue4(c_w, offw, 2 * i);
    issue4(c_x, offx, 2 * i + 1);
    cursor_next();
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(8));
  interval_barrier();
  if (wt == 1) interval_barrier();   // the second group runs one interval behind

  // Slots: step s (counted over all tiles) keeps its W rows in slot 2 s % 5 and
  // its x rows in slot (2 s + 1) % 5. Numbering the intervals so that group 0
  // reads in intervals 4 s and 4 s + 2 of step s and group 1 in 4 s + 1 and
  // 4 s + 3:
  //  - the W copies of step s + 2 go out from interval 4 s on, into the slot of
  //    x of step s - 1, last read (by group 1) in interval 4 s - 1;
  //  - the x copies of step s + 2 go out from interval 4 s + 2 on, into the slot
  //    of W of step s, last read in interval 4 s + 1;
  //  - a wave's copies of step s + 1 have landed at the end of its second
  //    reading interval of step s (8 younger copies stay in flight), at most
  //    4 s + 3; the barrier after it lets interval 4 s + 4 read them.
  // A reading interval ends with lgkmcnt(0), so its reads are complete at its
  // barrier.
  int slot = 0, free_slot = 0;
  auto inc = [](int v) { return v + 1 == kSlots ? 0 : v + 1; };
  for (; tile < tile_end; tile += wg_per_xcd) {
    for (int k = 0; k < nk; ++k) {
      const int sx = inc(slot), s2 = inc(sx), s4 = inc(inc(s2));
      const int wst = slot * kSlot, xst = sx * kSlot;
      bf16x8 af[2][4], bx[8];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (c == 0) {
#pragma unroll
          for (int fa = 0; fa < 4; ++fa) {
            af[0][fa] = ld(wst + arow(fa) * kRow + so0);
            af[1][fa] = ld(wst + arow(fa) * kRow + so1);
          }
        }
#pragma unroll
        for (int tb = 0; tb < 8; ++tb) bx[tb] = ld(xst + (brow + 16 * tb) * kRow + (c ? so1 : so0));
        if (c == 0) {
          issue4(c_w, offw, s4);
        } else {
          issue4(c_x, offx, slot);
          cursor_next();
        }
        __builtin_amdgcn_sched_barrier(0);
        if (c == 0) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));
        else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(8));
        interval_barrier();
        __builtin_amdgcn_s_setprio(1);
        if (!(half_last && k == nk - 1 && c == 0)) {
#pragma unroll
          for (int tb = 0; tb < 8; ++tb)
#pragma unroll
            for (int fa = 0; fa < 4; ++fa)
              acc[fa][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[c][fa], bx[tb], acc[fa][tb], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(0);
        interval_barrier();
      }
      free_slot = sx;
      slot = s2;
    }
    // ---- epilogue. The slot of the last step's x rows is free until the next
    // tile's first step, whose copies into a wave's part of it are that wave's.
    int f0, t0;
    tile_origin(a, tile, kTileF, kTileT, f0, t0);
    const int hf = min(f0, f_max) / D + head_l;
    if (hf * D >= f0)
      store_results<D, 2, 8>(a, acc, hf, j0, min(t0, t_max) + brow, t0, lds + free_slot * kSlot + wave * kOwn, lane);
    clear();
  }
  if (wt == 0) interval_barrier();
  // the copies past the last tile must not outlive the workgroup's LDS
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
}

// ---------------------------------------------------------------------------
// Fewer tokens: one smaller tile per workgroup, so that more CUs work on the
// batch. Same staging, operand layout and epilogue as above, and the same order
// of every sum: each accumulator takes the steps of 32 hidden one after the other
// in one wave, in every kernel of this file, so a token's results do not depend
// on the tile that computes it, nor on the rest of its batch.
//
// 256 features x 128 tokens, alternating wave groups as above with one reading
// and one product interval (both k-steps) per step. Wave (w4, gr) owns 64
// features and 64 tokens. A ring of three stages (W and x rows of a step).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void qkv_tile_kernel(const QkvArgs a) {
  constexpr int TF = 256, TT = 128;
  constexpr int W_BYTES = TF * kRow, STAGE = W_BYTES + TT * kRow;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[3 * STAGE];
  static_assert(3 * STAGE <= 160 * 1024, "LDS of one CU");
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int tile = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
  if (tile >= a.n_ftiles * a.n_ttiles) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w4 = wave & 3, gr = wave >> 2;

  int f_own, t_own;
  tile_origin(a, tile, TF, TT, f_own, t_own);
  // (a tile past the last row of W or x is moved back, as above)
  const int f0 = min(f_own, max(a.n_feat - TF, 0)), t0 = min(t_own, max(a.T - TT, 0));

  // ---- staging: planes of 64 hidden, one per step
  const int64_t hb = int64_t(a.hidden) * 2;
  const int nk = (a.hidden + kStep - 1) / kStep;
  const bool half_last = (a.hidden % kStep) != 0;
  const uint8_t* const wb = a.w + int64_t(f0) * hb;
  const uint8_t* const xb = a.x + int64_t(t0) * hb;
  uint32_t offw[4], offx[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 32 * wave + 8 * i + (lane >> 3);
    int c = ((lane & 7) ^ row_swz(row)) * 16;
    if (a.hidden < kStep) c &= ~64;
    offw[i] = uint32_t(min(staged_feature(row), a.n_feat - 1)) * uint32_t(hb) + c;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 16 * wave + 8 * i + (lane >> 3);
    int c = ((lane & 7) ^ row_swz(row)) * 16;
    if (a.hidden < kStep) c &= ~64;
    offx[i] = uint32_t(min(row, a.T - 1)) * uint32_t(hb) + c;
  }
  auto issue = [&](int s, uint32_t dst) __attribute__((always_inline)) {
    const int64_t o = plane_offset(s, nk, half_last);
#pragma unroll
    for (int i = 0; i < 4; ++i) copy16_to_lds(wb + o, offw[i], dst + (32 * wave + 8 * i) * kRow);
#pragma unroll
    for (int i = 0; i < 2; ++i) copy16_to_lds(xb + o, offx[i], dst + W_BYTES + (16 * wave + 8 * i) * kRow);
  };

  // ---- operand rows of this wave
  constexpr int kWavesPerHead = D / 64;
  const int head_l = w4 / kWavesPerHead;
  const int j0 = (w4 % kWavesPerHead) * 32;
  const int arow0 = head_l * D + j0;
  const int brow = 64 * gr;
  const int l16 = lane & 15;
  const int g4 = lane >> 4;
  const int so[2] = {l16 * kRow + ((g4 ^ row_swz(l16)) << 4), l16 * kRow + (((4 + g4) ^ row_swz(l16)) << 4)};
  auto ld = [&](int addr) __attribute__((always_inline)) -> bf16x8 {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(lds + addr));
  };
  f32x4 acc[4][4];
#pragma unroll
  for (int fa = 0; fa < 4; ++fa)
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) acc[fa][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Step s is in stage s % 3. Group 0 reads it in interval 2 s, group 1 in 2 s + 1:
  // step s + 2 goes into the stage of step s - 1, last read (by group 1) in
  // interval 2 s - 1, when a group reads step s; a wave's copies of step s + 1
  // have landed at the end of interval 2 s + 1.
  constexpr int kFly = 6;   // copies of one step
  issue(0, lds0);
  issue(1, lds0 + STAGE);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kFly));
  interval_barrier();
  if (gr == 1) interval_barrier();
  int stage = 0;
  for (int s = 0; s < nk; ++s) {
    const int wst = stage * STAGE, xst = wst + W_BYTES;
    bf16x8 af[2][4], bx[2][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int fa = 0; fa < 4; ++fa)
        af[ks][fa] = ld(wst + (arow0 + (fa >> 1) * (D / 2) + (fa & 1) * 16) * kRow + so[ks]);
#pragma unroll
      for (int tb = 0; tb < 4; ++tb) bx[ks][tb] = ld(xst + (brow + 16 * tb) * kRow + so[ks]);
    }
    issue(s + 2, lds0 + (stage == 0 ? 2 : stage - 1) * STAGE);
    __builtin_amdgcn_sched_barrier(0);
    if (gr == 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kFly));
    else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));
    interval_barrier();
    __builtin_amdgcn_s_setprio(1);
    const bool half = half_last && s == nk - 1;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      if (!(half && ks == 0)) {
#pragma unroll
        for (int tb = 0; tb < 4; ++tb)
#pragma unroll
          for (int fa = 0; fa < 4; ++fa)
            acc[fa][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks][fa], bx[ks][tb], acc[fa][tb], 0, 0, 0);
      }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (gr == 0) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kFly));
    interval_barrier();
    stage = stage == 2 ? 0 : stage + 1;
  }
  if (gr == 0) interval_barrier();
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
  interval_barrier();   // every wave's copies have landed: the ring is free
  const int hf = f0 / D + head_l;
  if (hf * D >= f_own) store_results<D, 2, 4>(a, acc, hf, j0, t0 + brow, t_own, lds + wave * 4096, lane);
}

// ---------------------------------------------------------------------------
// 128 features x 128 tokens. Waves 0-3 multiply (64 features and 64 tokens each,
// the operand reads of a k-step under the products of the one before), waves 4-7,
// one on each SIMD beside them, copy; at the end they finish half of the tokens.
// (Eight multiplying waves of 64 x 32 would read half as much again from LDS,
// which bounds the kernel: 96 KB a step read and written at 128 bytes a cycle, 768
// cycles, against 512 of products. 6,144 features, hidden 4,096, T = 576: 32.6
// us. With the wave groups on alternate steps and their sums added at the end,
// another order of the sums than the other tiles', it took 33.9.)
// A ring of five stages of 32 KB, W rows then x rows. At the barrier that starts
// step s the planes up to s + 1 have landed; step s reads the second k-step of
// plane s and the first of plane s + 1. The copies that go out after it (plane
// s + 4) replace plane s - 1, whose last reads fed products before that barrier.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void qkv_block_kernel(const QkvArgs a) {
  constexpr int TF = 128, TT = 128, W_BYTES = TF * kRow, STAGE = W_BYTES + TT * kRow, ST = 5;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[ST * STAGE];
  static_assert(ST * STAGE <= 160 * 1024, "LDS of one CU");
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int tile = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
  if (tile >= a.n_ftiles * a.n_ttiles) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w4 = wave & 3;
  const bool copier = wave >= 4;

  int f_own, t_own;
  tile_origin(a, tile, TF, TT, f_own, t_own);
  // (a tile past the last row of W or x is moved back, as above)
  const int f0 = min(f_own, max(a.n_feat - TF, 0)), t0 = min(t_own, max(a.T - TT, 0));
  const int nk = (a.hidden + kStep - 1) / kStep;
  const bool half_last = (a.hidden % kStep) != 0;

  constexpr int kWavesPerHead = D / 64;
  const int wf = w4 & 1;
  const int head_l = wf / kWavesPerHead;
  const int j0 = (wf % kWavesPerHead) * 32;
  const int brow = 64 * (w4 >> 1);
  f32x4 acc[4][4];
#pragma unroll
  for (int fa = 0; fa < 4; ++fa)
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) acc[fa][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (copier) {
    const int64_t hb = int64_t(a.hidden) * 2;
    const uint8_t* const wb = a.w + int64_t(f0) * hb;
    const uint8_t* const xb = a.x + int64_t(t0) * hb;
    uint32_t offw[4], offx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 32 * w4 + 8 * i + (lane >> 3);
      int c = ((lane & 7) ^ row_swz(row)) * 16;
      if (a.hidden < kStep) c &= ~64;
      offw[i] = uint32_t(min(staged_feature(row), a.n_feat - 1)) * uint32_t(hb) + c;
      offx[i] = uint32_t(min(row, a.T - 1)) * uint32_t(hb) + c;
    }
    auto issue = [&](int s, int stage) __attribute__((always_inline)) {
      const int64_t o = plane_offset(s, nk, half_last);
      const uint32_t dst = lds0 + stage * STAGE + 32 * w4 * kRow;
#pragma unroll
      for (int i = 0; i < 4; ++i) copy16_to_lds(wb + o, offw[i], dst + 8 * i * kRow);
#pragma unroll
      for (int i = 0; i < 4; ++i) copy16_to_lds(xb + o, offx[i], dst + W_BYTES + 8 * i * kRow);
    };
#pragma unroll
    for (int i = 0; i < ST - 1; ++i) issue(i, i);
    int stage = ST - 1;
    for (int s = 0; s < nk; ++s) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(16));   // all but the planes s + 2 and s + 3
      interval_barrier();
      issue(s + ST - 1, stage);
      stage = stage == ST - 1 ? 0 : stage + 1;
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
  } else {
    const int arow0 = head_l * D + j0;
    const int l16 = lane & 15;
    const int g4 = lane >> 4;
    const int so[2] = {l16 * kRow + ((g4 ^ row_swz(l16)) << 4), l16 * kRow + (((4 + g4) ^ row_swz(l16)) << 4)};
    // operand i of a k-step: feature blocks 0 .. 3, then token blocks 0 .. 3
    bf16x8 op[2][8];
    auto read = [&](int st, int ks, int i) __attribute__((always_inline)) {
      const int row = i < 4 ? arow0 + (i >> 1) * (D / 2) + (i & 1) * 16 : TF + brow + 16 * (i - 4);
      op[ks][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(lds + st + row * kRow + so[ks]));
    };
    // The products of k-step ks, with the reads of the k-step after it (the other
    // register set; stage `st`) between them: two products, one read.
    auto products = [&](int ks, int st) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int n = 2 * i + u, tb = n >> 2, fa = n & 3;
          acc[fa][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[ks][fa], op[ks][4 + tb], acc[fa][tb], 0, 0, 0);
        }
        read(st, ks ^ 1, i);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    int stage = 0;
    for (int s = 0; s < nk; ++s) {
      interval_barrier();
      const int next = stage == ST - 1 ? 0 : stage + 1;
      if (s == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) read(0, 0, i);
      }
      if (half_last && s == nk - 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) read(stage * STAGE, 1, i);
      } else {
        products(0, stage * STAGE);
      }
      products(1, next * STAGE);
      stage = next;
    }
  }
  interval_barrier();   // every wave's copies have landed: the ring is free
  // waves 4-7 finish token blocks 2 and 3 of the waves beside them
  f32x4 fin[4][2];
  if (!copier) {
#pragma unroll
    for (int fa = 0; fa < 4; ++fa)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        *reinterpret_cast<f32x4*>(lds + w4 * 8192 + (fa * 2 + i) * 1024 + lane * 16) = acc[fa][2 + i];
        fin[fa][i] = acc[fa][i];
      }
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));
  interval_barrier();
  if (copier) {
#pragma unroll
    for (int fa = 0; fa < 4; ++fa)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        fin[fa][i] = *reinterpret_cast<const f32x4*>(lds + w4 * 8192 + (fa * 2 + i) * 1024 + lane * 16);
  }
  const int hf = f0 / D + head_l;
  if (hf * D >= f_own)
    store_results<D, 2, 2>(a, fin, hf, j0, t0 + brow + (copier ? 32 : 0), t_own, lds + 4 * 8192 + wave * 4096, lane);
}

// ---------------------------------------------------------------------------
// Fewest tokens: a workgroup takes 16 FH rotary pairs (2 x 16 FH rows of W) and
// 16 TB tokens and streams its rows through a ring of ST stages of PL planes
// (64 hidden each). All eight waves copy; WF x WT of them multiply, each its
// share of the 2 FH feature and TB token blocks over all k-steps in order.
// Bound by the read of W: the ring keeps ST - 1 stages (up to 128 KB) in flight
// per CU, and the products hide under it.
// ---------------------------------------------------------------------------
// f(R), f(R - 1), .. f(0), the argument a compile-time constant.
template <int R, class F>
__device__ __forceinline__ void countdown(F&& f) {
  f(std::integral_constant<int, R>{});
  if constexpr (R > 0) countdown<R - 1>(f);
}

template <int FH, int TB, int PL, int ST, int WF, int WT>
struct StreamGeom {
  static constexpr int TF = 32 * FH, TT = 16 * TB, ROWS = TF + TT;
  static constexpr int FB = 2 * FH, FW = FB / WF, NB = TB / WT;   // feature blocks; feature and token blocks per wave
  static constexpr int PLANE = ROWS * kRow, STAGE = PL * PLANE;
  static constexpr int COPIES = STAGE / 1024, NC = COPIES / 8;   // 8-row copies per stage, per wave
  static constexpr int SUMS = TB * FB * 1024;
  static constexpr int TAIL = SUMS + TB * FH * 2048;   // sums and cos/sin rows, after the ring is done
  static constexpr int LDS = ST * STAGE > TAIL ? ST * STAGE : TAIL;
  static_assert(COPIES % 8 == 0 && WF * FW == FB && WT * NB == TB && WF * WT <= 8, "even shares");
  static_assert(LDS <= 160 * 1024, "LDS of one CU");
};

template <int D, int FH, int TB, int PL, int ST, int WF, int WT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void qkv_stream_kernel(const QkvArgs a) {
  using G = StreamGeom<FH, TB, PL, ST, WF, WT>;
  constexpr int FB = G::FB, FW = G::FW, NB = G::NB, NC = G::NC;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[G::LDS];
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int tile = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
  if (tile >= a.n_ftiles * a.n_ttiles) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  constexpr int kUnits = D / G::TF;   // tiles per head
  int ft, t0;
  tile_origin(a, tile, 1, G::TT, ft, t0);
  const int hf = ft / kUnits, j0 = (ft % kUnits) * (16 * FH);

  const int64_t hb = int64_t(a.hidden) * 2;
  const int planes = (a.hidden + kStep - 1) / kStep;
  const int nk = (planes + PL - 1) / PL;
  const bool half_last = (a.hidden % kStep) != 0;
  // Copy i of this wave: rows 8 (c % (ROWS / 8)) .. + 7 of plane c / (ROWS / 8),
  // c = wave + 8 i; W rows of the two halves of the pairs first, then x rows.
  const uint8_t* base[NC];
  uint32_t off[NC];
  int pl[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = wave + 8 * i;
    pl[i] = c / (G::ROWS / 8);
    const int r8 = 8 * (c % (G::ROWS / 8));
    const int row = r8 + (lane >> 3);
    int ch = ((lane & 7) ^ row_swz(row)) * 16;
    if (a.hidden < kStep) ch &= ~64;
    if (r8 < G::TF) {
      const int half = row / (16 * FH), r = row % (16 * FH);
      base[i] = a.w + (int64_t(hf) * D + j0) * hb;
      off[i] = uint32_t(half * (D / 2) + (FH == 2 ? staged_feature(r) : r)) * uint32_t(hb) + ch;
    } else {
      base[i] = a.x + int64_t(t0) * hb;
      off[i] = uint32_t(min(row - G::TF, a.T - 1 - t0)) * uint32_t(hb) + ch;
    }
  }
  auto issue = [&](int s, int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NC; ++i)
      copy16_to_lds(base[i] + plane_offset(PL * s + pl[i], planes, half_last), off[i],
                    lds0 + stage * G::STAGE + (wave + 8 * i) * 1024);
  };

  const int wf = wave % WF, wt = wave / WF;   // (a wave with wt >= WT only copies)
  const int so[2] = {l16 * kRow + ((g4 ^ row_swz(l16)) << 4), l16 * kRow + (((4 + g4) ^ row_swz(l16)) << 4)};
  const int arow = 16 * FW * wf, brow = G::TF + 16 * NB * wt;
  f32x4 acc[FW][NB];
#pragma unroll
  for (int fa = 0; fa < FW; ++fa)
#pragma unroll
    for (int tb = 0; tb < NB; ++tb) acc[fa][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int s, int stage) __attribute__((always_inline)) {
    if (wt >= WT) return;
    const uint8_t* st = lds + stage * G::STAGE;
    // k-steps of the stage: those of missing planes, and the first of a plane
    // that holds 32 hidden, are read and not multiplied
    const int first_half = half_last && (planes - 1) / PL == s ? (planes - 1) % PL : PL;
    const int np = min(planes - PL * s, PL);
    bf16x8 af[2 * PL][FW], bx[2 * PL][NB];
#pragma unroll
    for (int u = 0; u < 2 * PL; ++u) {
      const uint8_t* p = st + (u >> 1) * G::PLANE + so[u & 1];
#pragma unroll
      for (int fa = 0; fa < FW; ++fa) af[u][fa] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p + (arow + 16 * fa) * kRow));
#pragma unroll
      for (int tb = 0; tb < NB; ++tb) bx[u][tb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p + (brow + 16 * tb) * kRow));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 2 * PL; ++u)
      if ((u >> 1) < np && !((u & 1) == 0 && (u >> 1) == first_half)) {
#pragma unroll
        for (int fa = 0; fa < FW; ++fa)
#pragma unroll
          for (int tb = 0; tb < NB; ++tb)
            acc[fa][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[u][fa], bx[u][tb], acc[fa][tb], 0, 0, 0);
      }
  };
  // Stage s % ST holds step s. At the barrier of step s every wave's copies of
  // step s have landed (ST - 2 younger steps stay in flight) and every wave's
  // reads of step s - 1 are complete, so step s + ST - 1 goes into its stage.
#pragma unroll
  for (int i = 0; i < ST - 1; ++i)
    if (i < nk) issue(i, i);
  int stage = 0, s = 0;
  for (; s + ST - 1 < nk; ++s) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(NC * (ST - 2)));
    interval_barrier();
    issue(s + ST - 1, stage == 0 ? ST - 1 : stage - 1);
    compute(s, stage);
    stage = stage == ST - 1 ? 0 : stage + 1;
  }
  countdown<ST - 2>([&](auto younger) __attribute__((always_inline)) {   // the last steps
    constexpr int R = decltype(younger)::value;
    if (nk - 1 - s != R) return;
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(NC * R));
    interval_barrier();
    compute(s, stage);
    stage = stage == ST - 1 ? 0 : stage + 1;
    ++s;
  });
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
  interval_barrier();   // every wave is done with the ring
  // ---- wave tb finishes token block tb: its sums from the waves that hold them
  if (wt < WT) {
#pragma unroll
    for (int fa = 0; fa < FW; ++fa)
#pragma unroll
      for (int tb = 0; tb < NB; ++tb)
        *reinterpret_cast<f32x4*>(lds + ((wt * NB + tb) * FB + wf * FW + fa) * 1024 + lane * 16) = acc[fa][tb];
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));
  interval_barrier();
  if (wave >= TB) return;
  f32x4 sum[FB][1];
#pragma unroll
  for (int fa = 0; fa < FB; ++fa) sum[fa][0] = *reinterpret_cast<const f32x4*>(lds + (wave * FB + fa) * 1024 + lane * 16);
  const int tfirst = t0 + 16 * wave;
  store_results<D, FH, 1>(a, sum, hf, j0, tfirst, tfirst, lds + G::SUMS + wave * FH * 2048, lane);
}

cw_status check_launch(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return cw::fail(CW_EHIP, std::string(what) + ": " + hipGetErrorString(e));
  return cw::ok();
}

// The tile shapes, and what a call costs with each: `tiles` tiles in rounds of
// one per CU, a round fixed + planes * us (planes = hidden / 64), where us goes
// from `light` (few CUs busy) to `full` (all busy). The shape with the smallest
// estimate is taken; all give the same bits. The constants are fits to calls in
// captured graphs at 180 sizes: T = 1 .. 8,000 tokens, 384 .. 10,240 features,
// hidden 256 .. 8,192, all shapes at each (profiles/qkv_tile_shapes.txt). The
// estimate's choice is within 2.6 % of the best shape everywhere and 0.05 % on
// average. Leaving out any one shape costs 13 % (256 x 256) to 63 % (128 x 128)
// at its sizes; a 64 x 128 tile was the best by more than 1 % at two of the 180
// (by 4 and 9 %, 0.3 and 0.6 us) and is left out. Examples, in us, 6,144 features
// and hidden 4,096, 256 x 256 tile against the chosen one: T = 64: 67.2 / 16.7
// (32 x 64); 128: 68.3 / 20.9 (64 x 64); 256: 70.4 / 27.2 (128 x 128); 576: 72.1
// / 32.6 (128 x 128); 1,024: 72.6 / 50.8 (256 x 128); 1,536: 77.0 (128 x 128: 85.5).
struct QkvShape {
  int tile_f, tile_t;
  bool persistent;
  double fixed, light, full;   // us
  void (*kernel128)(QkvArgs);
  void (*kernel64)(QkvArgs);
};
const QkvShape kShapes[] = {
    {256, 256, true, 13.4, 0.768, 1.297, qkv_rope_append_kernel<128>, qkv_rope_append_kernel<64>},
    {256, 128, false, 6.97, 0.529, 0.754, qkv_tile_kernel<128>, qkv_tile_kernel<64>},
    {128, 128, false, 5.52, 0.296, 0.400, qkv_block_kernel<128>, qkv_block_kernel<64>},
    {64, 64, false, 4.11, 0.255, 0.242, qkv_stream_kernel<128, 2, 4, 2, 5, 2, 2>, qkv_stream_kernel<64, 2, 4, 2, 5, 2, 2>},
    {32, 64, false, 3.88, 0.187, 0.182, qkv_stream_kernel<128, 1, 4, 2, 6, 2, 2>, qkv_stream_kernel<64, 1, 4, 2, 6, 2, 2>},
    {32, 32, false, 3.45, 0.129, 0.122, qkv_stream_kernel<128, 1, 2, 4, 5, 2, 2>, qkv_stream_kernel<64, 1, 2, 4, 5, 2, 2>},
    {32, 16, false, 3.52, 0.100, 0.092, qkv_stream_kernel<128, 1, 1, 4, 6, 2, 1>, qkv_stream_kernel<64, 1, 1, 4, 6, 2, 1>},
};

const QkvShape& pick_shape(int64_t rows, int64_t n_feat, int64_t hidden) {
  const double planes = double((hidden + kStep - 1) / kStep);
  const QkvShape* best = nullptr;
  double best_us = 0;
  for (const QkvShape& s : kShapes) {
    const int64_t tiles = ((n_feat + s.tile_f - 1) / s.tile_f) * ((rows + s.tile_t - 1) / s.tile_t);
    const int64_t rounds = tiles / cw::kNumCu, rest = tiles % cw::kNumCu;
    double us = double(rounds) * (s.fixed + planes * s.full);
    if (rest > 0) us += s.fixed + planes * (s.light + (s.full - s.light) * double(rest) / cw::kNumCu);
    if (!best || us < best_us) {
      best = &s;
      best_us = us;
    }
  }
  return *best;
}

}  // namespace

extern "C" cw_status cw_qkv_rope_append(const void* x, const void* w, const void* bias, const float* rope,
                                        int32_t rope_len, int32_t hidden, void* q_out, void* k_cache,
                                        void* v_cache, const int32_t* block_table, int32_t bt_stride,
                                        const int32_t* cu_suffix_dev, const int32_t* prefix_len_dev,
                                        const int32_t* cu_suffix_host, const int32_t* prefix_len_host,
                                        int32_t batch, int32_t num_q_heads, int32_t num_kv_heads,
                                        int32_t head_dim, int32_t block_size, int32_t num_blocks, void* stream) {
  const char* what = "qkv_rope_append";
  if (!w || !rope || !k_cache || !v_cache || !block_table || !cu_suffix_dev || !prefix_len_dev)
    return cw::fail(CW_EINVAL, std::string(what) + ": a required pointer is NULL");
  if (num_q_heads < 1 || num_kv_heads < 1 || num_q_heads % num_kv_heads != 0)
    return cw::fail(CW_EINVAL, std::string(what) + ": num_q_heads must be a positive multiple of num_kv_heads");
  if (num_blocks < 1) return cw::fail(CW_EINVAL, std::string(what) + ": num_blocks must be >= 1");
  if (head_dim != 64 && head_dim != 128)
    return cw::fail(CW_EUNSUPPORTED, std::string(what) + ": head_dim must be 64 or 128");
  if (block_size != kBs) return cw::fail(CW_EUNSUPPORTED, std::string(what) + ": block_size must be 16");
  if (hidden < kStep / 2 || hidden % (kStep / 2) != 0 || hidden > (1 << 20))
    return cw::fail(CW_EUNSUPPORTED, std::string(what) + ": hidden must be a multiple of 32 in [32, 2^20]");
  if (rope_len < 0) return cw::fail(CW_EINVAL, std::string(what) + ": rope_len must be >= 0");
  int64_t rows = 0;
  cw_status st = cw::check_batch(cu_suffix_host, prefix_len_host, batch, block_size, bt_stride, &rows);
  if (st != CW_OK) return st;
  int64_t max_pos = -1;   // largest position of a suffix row
  for (int32_t r = 0; r < batch; ++r)
    if (cu_suffix_host[r + 1] > cu_suffix_host[r])
      max_pos = std::max<int64_t>(max_pos, int64_t(prefix_len_host[r]) + cu_suffix_host[r + 1] - cu_suffix_host[r] - 1);
  if (max_pos >= rope_len)
    return cw::fail(CW_EINVAL, std::string(what) + ": the rotary table holds " + std::to_string(rope_len) +
                                   " positions, position " + std::to_string(max_pos) + " is needed");
  if (rows == 0) return cw::ok();
  if (!x || !q_out) return cw::fail(CW_EINVAL, std::string(what) + ": x and q_out are required");
  if (rows > INT32_MAX - kTileT) return cw::fail(CW_EUNSUPPORTED, std::string(what) + ": too many suffix rows");
  const int64_t n_feat = int64_t(num_q_heads + 2 * num_kv_heads) * head_dim;
  const QkvShape& sh = pick_shape(rows, n_feat, hidden);
  const int64_t n_ftiles = (n_feat + sh.tile_f - 1) / sh.tile_f;
  const int64_t n_ttiles = (rows + sh.tile_t - 1) / sh.tile_t;
  const int64_t per_xcd = (n_ftiles * n_ttiles + cw::kNumXcd - 1) / cw::kNumXcd;
  if (per_xcd * cw::kNumXcd > INT32_MAX) return cw::fail(CW_EUNSUPPORTED, std::string(what) + ": too many tiles");
  auto* s = static_cast<hipStream_t>(stream);
  const dim3 grid(unsigned((sh.persistent ? std::min<int64_t>(per_xcd, cw::kNumCu / cw::kNumXcd) : per_xcd) * cw::kNumXcd));
  QkvArgs a;
  a.x = static_cast<const uint8_t*>(x);
  a.w = static_cast<const uint8_t*>(w);
  a.bias = static_cast<const uint16_t*>(bias);
  a.rope = rope;
  a.q_out = static_cast<uint16_t*>(q_out);
  a.k_cache = static_cast<uint16_t*>(k_cache);
  a.v_cache = static_cast<uint16_t*>(v_cache);
  a.bt = block_table;
  a.cu = cu_suffix_dev;
  a.plen = prefix_len_dev;
  a.T = int(rows);
  a.hidden = hidden;
  a.n_feat = int(n_feat);
  a.bt_stride = bt_stride;
  a.batch = batch;
  a.hq = num_q_heads;
  a.hkv = num_kv_heads;
  a.num_blocks = num_blocks;
  a.n_ftiles = int(n_ftiles);
  a.n_ttiles = int(n_ttiles);
  a.per_xcd = int(per_xcd);
  hipLaunchKernelGGL(head_dim == 128 ? sh.kernel128 : sh.kernel64, grid, dim3(kThreads), 0, s, a);
  return check_launch("qkv_rope_append launch");
}
