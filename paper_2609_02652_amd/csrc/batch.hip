// Batched GEMV on the matrix cores for gfx950, for the batches that the narrow
// launches of gemv_kernel_mx do not take (narrow_batch in kernels.hip: up to four
// activations, up to eight in some shapes): Y[b] = W X[b] with W in the Planes14
// layout (§6 "Batching": one decode of each weight serves several activations).
//
// Arithmetic.  A block's 24 decoded weights meet an activation in six chained
// binary16 MFMAs of four products each, with an f32 result per (row,
// activation); the block's factor scale · 2^24 · centroid / (4√m) then
// multiplies that result in f32.  No sum crosses a block inside the matrix core
// and no weight is rounded.  The shapes 4×4×4 (16 blocks; gemv_kernel_mx), 16×16×4
// (4 blocks) and 32×32×4 (2 blocks) give the same bits (measured over 262,144 dot
// products; shapes that sum eight products at a time do not), and in all of
// them a lane supplies a column of its own: the block it has decoded, with no
// exchange between lanes.
//
// Order.  gemv_kernel_mx's: wave w takes the units (lane_cols = C columns) w, w +
// 8, ... one after the other and keeps one partial sum per column of the unit;
// these are added in pairs, and the waves' sums one after the other.  So Y[b] is
// the same bits for any batch size, position in the batch and tile shape.
//
// Work split.  A workgroup owns RW = 16, 32 or 64 consecutive rows (whatever the
// layout's tiles) and NB = 16, 32 or 64 activations; its eight waves take their
// units each and meet once, in LDS, at the end.  A step of a wave decodes 64
// blocks, one a lane: RW rows × 64 / RW columns.  The activations go through LDS
// in pair order, a few columns at a time, in a region of the wave's own: nothing
// in the loop waits for another wave, and Kpad does not bound the batch.  What
// bounds it: up to 16 activations the vector instructions of the decode (about
// 75 a step), above that the matrix cores (384 cycles a step and 32
// activations).

#include <algorithm>
#include <cstdint>
#include <string>
#include <type_traits>

#include "batch.h"
#include "device_common.h"

namespace leech {
namespace {

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x32 __attribute__((ext_vector_type(32)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int64_t kMaxGroups = 0xFFFFFFFFll / kThreads;   // a launch has fewer than 2^32 threads
constexpr uint32_t kOutOfRange = 0x7FFFFFF0u;   // buffer offset past any descriptor's end

struct BatchArgs {
  const uint8_t* main;
  const DevClass* table;
  const uint16_t* scale;
  const uint16_t* x;
  float* y;
  float cen0, cen1;
  uint64_t main_bytes;
  int64_t ldx, ldy;
  uint32_t M;
  int nb, R, batch;
  int groups;                 // units of a tile
  uint32_t inv_r;             // 65536 / R, rounded up
  uint32_t inv_r32, inv_t32;  // 2^32 / R and 2^32 / batch tiles, rounded up
  int row_blocks, batch_tiles;
};

// n / d for the reciprocal inv = ⌈2^32 / d⌉ (d ≥ 2): exact, or one too large
// where n · (inv · d − 2^32) ≥ 2^32.
__device__ __forceinline__ uint32_t divide(uint32_t n, uint32_t d, uint32_t inv) {
  const uint32_t q = __umulhi(n, inv);
  return q * d > n ? q - 1 : q;
}

__device__ __forceinline__ void swap32(float& a, float& b) {
  // a's upper 32 lanes and b's lower 32 lanes change places
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]);
  b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ void swap16(float& a, float& b) {
  // the odd 16-lane rows of a and the even ones of b change places
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a),
                                                  __builtin_bit_cast(uint32_t, b), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]);
  b = __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Orders the wave's own LDS writes and reads of other lanes' data; the LDS
// serves a wave's operations in order, so this is for the compiler alone.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The products of the lane's decoded block h with the activations x (the
// lane's activation row in pair order): six chained MFMAs of a shape.
struct Acts {
  u32x4a v[3];
};
__device__ __forceinline__ half4_t pairs(uint32_t lo, uint32_t hi) {
  return __builtin_bit_cast(half4_t, u32x2a{lo, hi});
}
#define LEECH_CHAIN(MFMA)                                                             \
  d = MFMA(pairs(x.v[0].x, x.v[0].y), pairs(h[0], h[1]), d, 0, 0, 0);                 \
  d = MFMA(pairs(x.v[0].z, x.v[0].w), pairs(h[2], h[3]), d, 0, 0, 0);                 \
  d = MFMA(pairs(x.v[1].x, x.v[1].y), pairs(h[4], h[5]), d, 0, 0, 0);                 \
  d = MFMA(pairs(x.v[1].z, x.v[1].w), pairs(h[6], h[7]), d, 0, 0, 0);                 \
  d = MFMA(pairs(x.v[2].x, x.v[2].y), pairs(h[8], h[9]), d, 0, 0, 0);                 \
  d = MFMA(pairs(x.v[2].z, x.v[2].w), pairs(h[10], h[11]), d, 0, 0, 0);
__device__ __forceinline__ void products(const Acts& x, const uint32_t h[12], f32x16& d) {
  LEECH_CHAIN(__builtin_amdgcn_mfma_f32_16x16x4f16)
}
__device__ __forceinline__ void products(const Acts& x, const uint32_t h[12], f32x32& d) {
  LEECH_CHAIN(__builtin_amdgcn_mfma_f32_32x32x4f16)
}
#undef LEECH_CHAIN

// Activation columns staged at a time (whole units, or a whole part of one),
// and the LDS bytes of one activation's share of them: 16 bytes of padding make it
// an odd number of 16-byte words, which puts 16 consecutive activations' 16-byte
// reads on distinct banks.  (With three columns a stage, C = 3 with 64 rows, it is
// 10 words, and such reads conflict two ways.)
__host__ __device__ constexpr int x_cols(int C, int RW, int NB) {
  return C == 3 ? (RW == 64 ? 3 : 6) : NB > 32 ? 2 : 4;
}
__host__ __device__ constexpr int x_stride(int C, int RW, int NB) {
  return x_cols(C, RW, NB) * 48 + 16;
}
__host__ __device__ constexpr int red_batch(int NB) { return NB < 32 ? NB : 32; }
__host__ __device__ constexpr size_t lds_bytes(int C, int RW, int NB) {
  const size_t x = (size_t)kWaves * NB * x_stride(C, RW, NB);
  const size_t red = (size_t)kWaves * red_batch(NB) * RW * 4;
  return kTableBytes + (x > red ? x : red);
}

// C: the layout's lane_cols; RW rows × NB activations a workgroup; D steps'
// records in flight a wave; WPS waves a SIMD the registers are held to.
template <int C, int RW, int NB, int D, int WPS>
__global__ __launch_bounds__(kThreads, WPS) void batch_kernel(BatchArgs a) {
  constexpr int XC = x_cols(C, RW, NB), XS = x_stride(C, RW, NB);
  constexpr int SC = 64 / RW;                          // columns a step
  constexpr int SPS = XC / SC;                         // steps a stage of activations
  constexpr int XB = (NB * XC + 63) / 64;              // activation blocks a lane stages
  constexpr int NACC = RW * NB / 64;                   // outputs a lane holds
  constexpr bool kAligned = C % SC == 0 || SC % C == 0;
  static_assert(XC % SC == 0 && D % SPS == 0 && D * SC % C == 0, "ring sizes");
  static_assert(XC % C == 0 || C % XC == 0, "stages hold whole units or parts of one");
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  LdsEntry* const ts = (LdsEntry*)smem;

  // Workgroup -> (row block, batch tile): the batch tiles of a row block run
  // one after the other on one XCD (workgroups go to the 8 XCDs in turn), so
  // that its records come from HBM once and from that XCD's L2 afterwards.
  uint32_t rblk = blockIdx.x, btile = 0;
  if (a.batch_tiles > 1) {
    const uint32_t local = rblk >> 3, grp = divide(local, (uint32_t)a.batch_tiles, a.inv_t32);
    btile = local - grp * (uint32_t)a.batch_tiles;
    rblk = grp * 8 + (rblk & 7u);
    if (rblk >= (uint32_t)a.row_blocks) return;
  }
  const uint32_t row0 = rblk * RW;
  const int b0 = (int)btile * NB, nbat = min(NB, a.batch - b0);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = a.nb;
  // The wave's columns in its order: the n-th is column n % C of its unit n / C,
  // which is unit g = wave + 8 (n / C) of the tile, column j = g·C + n % C of the
  // matrix.  Past its last unit, j ≥ nb.
  const int units = wave < a.groups ? (a.groups - 1 - wave) / kWaves + 1 : 0;
  const int steps = (units * C + SC - 1) / SC;
  auto column = [&](int n) { return (wave + kWaves * (n / C)) * C + n % C; };

  // class records first, then activations, then weight records: loads return
  // in order
  u32x4a tr = {0, 0, 0, 0};
  if (wave * 64 < kBallClasses)
    tr = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(a.table, kBallClasses * sizeof(DevClass)),
                                               tid * (int)sizeof(DevClass), 0, 0);

  // Activations: lane block idx = lane + 64 k is (activation idx / XC, column
  // idx % XC) of the stage.  Activations past the batch repeat its last one
  // (their products are not written); columns past nb repeat the last column
  // and are written as zeros.
  const uint8_t* xrow[XB];
  uint32_t xdst[XB];
  int xcol[XB];
  uint8_t* const xs = smem + kTableBytes + wave * (NB * XS);
#pragma unroll
  for (int k = 0; k < XB; ++k) {
    const int idx = lane + 64 * k, b = idx / XC, c = idx % XC;
    xrow[k] = (const uint8_t*)(a.x + (int64_t)(b0 + min(b, nbat - 1)) * a.ldx);
    xcol[k] = C < XC ? c / C * (kWaves * C) + c % C : c;
    xdst[k] = (uint32_t)(b * XS + c * 48);
  }
  XBlock xr[XB];
  auto load_x = [&](int step) {      // the stage that starts at this step
    const int j = column(step * SC);
#pragma unroll
    for (int k = 0; k < XB; ++k) {
      const uint32_t off = step < steps ? __umul24((uint32_t)min(j + xcol[k], nb - 1), 48u) : 0u;
      xr[k] = load_x_block((const uint16_t*)(xrow[k] + off));
    }
  };
  auto store_x = [&](int step) {
    const int j = column(step * SC);
    if (j + (C < XC ? (XC / C - 1) * (kWaves * C) + C : XC) > nb) {
#pragma unroll
      for (int k = 0; k < XB; ++k)
        if (j + xcol[k] >= nb) xr[k].v0 = xr[k].v1 = xr[k].v2 = u32x4a{0, 0, 0, 0};
    }
#pragma unroll
    for (int k = 0; k < XB; ++k)
      if (NB * XC % 64 == 0 || lane + 64 * k < NB * XC)
        store_x_block(xr[k], (uint32_t*)(xs + xdst[k]));
  };
  load_x(0);

  // Records.  A lane's row of the row block (past the matrix: its last row,
  // whose stand-in results are not written) and column p of the step.  Block
  // (row, j) of tile t = row / R is at
  //   t·R·nb + g·R_t·C + (row % R)·cols(g) + j % C
  //   = t·R·nb + (row % R)·C + g·(R_t − 1)·C + j − (row % R)·(C − cols(g))
  // for its column group g = j / C, R_t rows in the tile, cols(g) columns in
  // the group; the descriptors start at the row block's first tile.  Where R_t
  // is one number for the row block and the wave has no narrower group, this is
  // a lane constant plus a scalar: no vector instruction but the choice of the
  // constant by the scalar's parity, which decides on which half of a word the
  // 14-byte record starts.
  const uint32_t R = (uint32_t)a.R;
  const uint32_t tile0 = divide(row0, R, a.inv_r32);
  const uint64_t blk0 = (uint64_t)tile0 * (R * (uint32_t)nb);
  const uint64_t blocks = (uint64_t)a.M * (uint32_t)nb;
  const __amdgpu_buffer_rsrc_t rs_rec = make_rsrc(
      a.main + blk0 * kPlanes14Bytes,
      min(a.main_bytes - blk0 * kPlanes14Bytes, (uint64_t)0x40000000u));
  const __amdgpu_buffer_rsrc_t rs_sc =
      make_rsrc(a.scale + blk0, min((blocks - blk0) * 2, (uint64_t)0x40000000u));
  const int p = RW == 64 ? 0 : lane / RW;
  const int glast = a.groups - 1, cols_last = nb - glast * C;
  const uint32_t t_last = (min(row0 + RW, a.M) - 1 - tile0 * R) * a.inv_r >> 16;
  const uint32_t group = (min(R, a.M - tile0 * R) - 1) * C;      // (R_t − 1)·C of one height
  const bool plain = kAligned && (t_last == 0 || (tile0 + t_last + 1) * R <= a.M) &&
                     (cols_last == C || glast % kWaves != wave) && units * C % SC == 0;
  uint32_t lane_row, lane_skip, lane_group, rec_even, rec_odd, sh_even, sh_odd, vscale;
  {
    const uint32_t in0 = min(row0 + (uint32_t)(lane & (RW - 1)), a.M - 1) - tile0 * R;
    const uint32_t t = in0 * a.inv_r >> 16, rr = in0 - t * R;
    lane_row = t * (R * (uint32_t)nb) + rr * C;
    lane_skip = rr * (uint32_t)(C - cols_last);
    lane_group = (min(R, a.M - (tile0 + t) * R) - 1) * C;
    // the step's columns lie in one unit, or are whole units
    const uint32_t lb = lane_row + (C < SC ? p / C * kWaves * (group + C) + p % C : (uint32_t)p);
    rec_even = lb * kPlanes14Bytes & ~3u;
    rec_odd = rec_even + (lb & 1u) * 4u;
    sh_even = (lb & 1u) * 16u;
    sh_odd = sh_even ^ 16u;
    vscale = lb * 2u;
  }
  struct Slot {
    u32x4a w;
    uint32_t scale, sh;
  };
  Slot slot[D];
  // PLAIN: the lane constant plus a scalar
  auto load_rec = [&](Slot& s, int step, auto plain_t) {
    const int n = step * SC;
    uint32_t vo, vs, so, ss;
    if constexpr (decltype(plain_t)::value) {
      const uint32_t u = (uint32_t)(wave + kWaves * (n / C)) * (group + C) + (uint32_t)(n % C);
      const bool odd = u & 1u;
      vo = odd ? rec_odd : rec_even;
      s.sh = odd ? sh_odd : sh_even;
      so = u * kPlanes14Bytes & ~3u;
      vs = vscale;
      ss = u * 2u;
    } else {
      const uint32_t nl = (uint32_t)(n + p), k = nl / C;
      const uint32_t g = (uint32_t)wave + kWaves * k, j = g * C + (nl - k * C);
      const uint32_t idx = __umul24(g, lane_group) + lane_row + j - ((int)g == glast ? lane_skip : 0u);
      // Past the last column: a scale of zero, zero activations, and a record of
      // zeros, which nothing is read for (so the class factors have to be
      // finite, see launch_batch_mx), or in the 32 × 16 tile of three columns the
      // buffer's first record: it takes the general path for every step, and
      // spills four registers with the other choice (5120×17408, 16 activations:
      // 24.7 µs here, 27.5; other tiles lose up to 5% this way).
      const bool live = (int)j < nb;
      uint32_t off = __umul24(idx, (uint32_t)kPlanes14Bytes);
      if constexpr (C == 3 && NB == 16) {
        off = live ? off : 0u;
        vo = step < steps ? off & ~3u : kOutOfRange;
      } else {
        vo = live ? off & ~3u : kOutOfRange;
      }
      s.sh = (off & 2u) << 3;
      vs = live ? idx * 2u : kOutOfRange;
      so = ss = 0;
    }
    s.w = __builtin_amdgcn_raw_buffer_load_b128(rs_rec, (int)vo, (int)so, 0);
    s.scale = __builtin_amdgcn_raw_buffer_load_b16(rs_sc, (int)vs, (int)ss, 0);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) {
    load_rec(slot[d], d, std::false_type{});
    __builtin_amdgcn_sched_barrier(0);
  }

  if (tid < kBallClasses) {
    LdsEntry e;
    e.tlo = tr.x;
    e.thi = tr.y;
    e.aux = 0u;
    const float f = __builtin_bit_cast(float, (uint32_t)tr.z) * kTwo24;
    e.factor = f * a.cen0;
    ts[tid] = e;
    e.factor = f * a.cen1;
    ts[tid + 512] = e;
  }
  __syncthreads();

  // one set of accumulators per column of a unit
  float acc[C][NACC];
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[c][i] = 0.0f;

  // the lane's activation of a product's x operand, in its own column
  constexpr int kActs = NB == 16 ? 16 : 32;      // rows of the operand
  const uint8_t* const xa = xs + (lane & (kActs - 1)) * XS + p * 48;
  auto read_x = [&](int set, int col) {
    const u32x4a* s = (const u32x4a*)__builtin_assume_aligned(xa + set * (kActs * XS) + col * 48, 16);
    return Acts{{s[0], s[1], s[2]}};
  };

  // One step: the 64 blocks of slot s, whose first column is column c0 of its
  // unit and column col of the stage; refill requests the slot's next records
  // while the products run.
  auto process = [&](Slot& s, int c0, int col, auto refill) {
    uint32_t words[3], h[12], e16;
    p14_record(s.w.x, s.w.y, s.w.z, s.w.w, s.sh, (s.sh + 28u) & 31u, words, e16);
    const LdsEntry te = *(const LdsEntry*)__builtin_assume_aligned(smem + e16, 16);
    p14_core(words, te.tlo, te.thi, h);
    const float f0 = (float)as_half(s.scale) * te.factor;
    // A product's result block q (of lanes 64/Q·q..) belongs to column c0 + q·SC/Q
    // of the step, Q blocks; f[q] are their factors, in every lane.
    constexpr int Q = NB == 16 ? 4 : 2, P = 64 / Q;
    float f[4];
    f[0] = f[2] = f0;
    swap32(f[0], f[2]);
    if constexpr (Q == 4) {
      f[1] = f[0];
      swap16(f[0], f[1]);
      f[3] = f[2];
      swap16(f[2], f[3]);
    } else {
      f[1] = f[2];
    }
    typedef std::conditional_t<Q == 4, f32x16, f32x32> Result;
    constexpr int NI = Q == 4 ? 4 : 16;          // results a lane per block
    Result d[NB / kActs];
#pragma unroll
    for (int g = 0; g < NB / kActs; ++g) {
#pragma unroll
      for (int i = 0; i < Q * NI; ++i) d[g][i] = 0.0f;
      products(read_x(g, col), h, d[g]);
    }
    __builtin_amdgcn_sched_barrier(0);     // the record's registers are free: refill them
    refill();
    // d[g][NI·q + i] of a lane: the block of lane P·q + lane % P
#pragma unroll
    for (int g = 0; g < NB / kActs; ++g)
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float& s2 = acc[(c0 + q * P / RW) % C][(g * (RW / P > 0 ? RW / P : 1) + q * P % RW / P) * NI + i];
          s2 = __builtin_fmaf(f[q], d[g][NI * q + i], s2);
        }
    // holds the accumulators' updates in the step: left alone they sink to the
    // loop's end, with every step's products alive
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int i = 0; i < NACC; ++i) asm("" : "+v"(acc[c][i]));
  };
  auto stage = [&](int step) {
    wave_lds_fence();
    store_x(step);
    load_x(step + SPS);
    wave_lds_fence();
  };
  // while every record the loop requests is one of the wave's, at a lane
  // constant plus a scalar
  int step = 0;
  if (plain)
    for (; step + 2 * D <= steps; step += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (d % SPS == 0) stage(step + d);
        process(slot[d], d * SC % C, d % SPS * SC,
                [&] { load_rec(slot[d], step + d + D, std::true_type{}); });
      }
    }
  for (; step < steps; step += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (step + d >= steps) break;
      if (d % SPS == 0) stage(step + d);
      process(slot[d], d * SC % C, d % SPS * SC,
              [&] { load_rec(slot[d], step + d + D, std::false_type{}); });
    }
  }

  // The columns' sums in pairs, then the waves' sums in the activation area, 32
  // activations at a time.
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    if constexpr (C == 3) {
      acc[0][i] = (acc[0][i] + acc[1][i]) + acc[2][i];
    } else {
#pragma unroll
      for (int w = 1; w < C; w <<= 1)
#pragma unroll
        for (int c = 0; c + w < C; c += 2 * w) acc[c][i] += acc[c + w][i];
    }
  }
  constexpr int NR = red_batch(NB), NG = NB / NR;
  float* const red = (float*)(smem + kTableBytes);
  float* const mine = red + wave * (NR * RW);
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NACC / NG; ++i) {
      int act, row;       // of accumulator i of the group
      if (NB == 16) {
        act = 4 * (lane >> 4) + i % 4;
        row = 16 * (i / 4) + (lane & 15);
      } else {
        act = 8 * (i % 16 / 4) + 4 * (lane >> 5) + i % 4;
        row = 32 * (i / 16) + (lane & 31);
      }
      mine[act * RW + row] = acc[0][g * (NACC / NG) + i];
    }
    __syncthreads();
    for (int o = tid; o < NR * RW; o += kThreads) {
      const int b = NR * g + o / RW;
      const uint32_t row = row0 + (uint32_t)(o % RW);
      if (b < nbat && row < a.M) {
        float y = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) y += red[w * (NR * RW) + o];
        a.y[(int64_t)(b0 + b) * a.ldy + row] = y;
      }
    }
  }
}

template <int C, int RW, int NB, int D, int WPS>
int launch_tile(BatchArgs a, hipStream_t st) {
  const void* fn = (const void*)batch_kernel<C, RW, NB, D, WPS>;
  constexpr size_t shmem = lds_bytes(C, RW, NB);
  static_assert(shmem <= 160 * 1024, "LDS of a workgroup");
  if (shmem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess)
      return set_error(LEECH_E_HIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
  }
  const int64_t row_blocks = ((int64_t)a.M + RW - 1) / RW;
  if (row_blocks > kMaxGroups) return set_error(LEECH_E_SHAPE, "matrix too large for one launch");
  // As many batch tiles a launch as it can hold; a launch of several has a
  // multiple of eight row blocks.
  const int64_t padded = (row_blocks + 7) / 8 * 8;
  const int64_t most = std::max<int64_t>(1, kMaxGroups / padded) * NB;
  const uint16_t* const x = a.x;
  float* const y = a.y;
  const int64_t batch = a.batch;
  a.row_blocks = (int)row_blocks;
  for (int64_t b0 = 0; b0 < batch; b0 += most) {
    a.x = x + b0 * a.ldx;
    a.y = y + b0 * a.ldy;
    a.batch = (int)std::min(most, batch - b0);
    const int64_t batch_tiles = ((int64_t)a.batch + NB - 1) / NB;
    a.batch_tiles = (int)batch_tiles;
    a.inv_t32 = (uint32_t)(((1ull << 32) + batch_tiles - 1) / batch_tiles);
    const int64_t grid = batch_tiles > 1 ? padded * batch_tiles : row_blocks;
    hipLaunchKernelGGL((batch_kernel<C, RW, NB, D, WPS>), dim3((unsigned)grid), dim3(kThreads),
                       shmem, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
      return set_error(LEECH_E_HIP, std::string("batch launch: ") + hipGetErrorString(e));
  }
  return LEECH_OK;
}

// The tiles of each lane_cols, widest first: (rows, activations) as RW · 100 +
// NB.  Wider tiles decode and stage less per product; a unit of C columns
// keeps C sets of accumulators, which bounds them.
struct Tiles {
  int C, tile[4];
};
constexpr Tiles kTiles[] = {{1, {6464, 6432, 6416, 3216}}, {2, {6432, 3232, 3216, 0}},
                            {3, {6432, 3232, 3216, 0}},    {4, {6432, 3232, 3216, 1616}},
                            {8, {3232, 3216, 1616, 0}},    {16, {3216, 1616, 0, 0}}};

// The widest tile that makes at least 160 workgroups for the 256 CUs, wider than
// 16 activations only where the batch is more than half as wide, else the
// narrowest.  (What the batch's last tile holds beside that does not count: 65
// activations may take two 64-wide tiles.)  Measured (µs a
// launch, 160 and more workgroups against fewer): 4096×4104 (4 × 16), 16
// activations: 16 rows 8.0, 32 rows (128 workgroups) 9.1; 32: 32 × 16 9.5, 32 ×
// 32 (128) 12.2; 64: 32 × 32 13.1, 64 × 32 (128) 17.5; 128: 64 × 32 18.8, 32 × 32
// 23.4; 5120×17424 (3 × 20), 32: 32 × 32 (160) 45.4, 64 × 32 (80) 68.7;
// 14336×4104 (1 × 64), 64: 64 × 64 31.7, 64 × 32 38.4.
int choose_tile(int C, int64_t M, int64_t batch) {
  int best = 0;
  for (const Tiles& t : kTiles)
    if (t.C == C)
      for (int tile : t.tile) {
        if (!tile) break;
        best = tile;
        const int64_t rw = tile / 100, nb = tile % 100;
        if ((nb == 16 || 2 * batch > nb) && (M + rw - 1) / rw * ((batch + nb - 1) / nb) >= 160)
          break;
      }
  return best;
}

}  // namespace

int launch_batch_mfma(const BatchCall& c, hipStream_t st) {
  BatchArgs a;
  a.main = c.main;
  a.table = c.table;
  a.scale = c.scale;
  a.x = c.x;
  a.y = c.y;
  a.cen0 = c.cen0;
  a.cen1 = c.cen1;
  a.main_bytes = c.main_bytes;
  a.M = (uint32_t)c.M;
  a.ldx = c.ldx;
  a.ldy = c.ldy;
  a.nb = (int)c.nb;
  a.R = c.R;
  a.batch = c.batch;
  a.groups = (int)((c.nb + c.C - 1) / c.C);
  a.inv_r = (uint32_t)((65536 + c.R - 1) / c.R);
  a.inv_r32 = (uint32_t)(((1ull << 32) + c.R - 1) / c.R);
  a.inv_t32 = 0;
  a.row_blocks = a.batch_tiles = 0;
  switch (c.C * 10000 + choose_tile(c.C, c.M, c.batch)) {
    case 16464: return launch_tile<1, 64, 64, 4, 2>(a, st);
    case 16432: return launch_tile<1, 64, 32, 4, 2>(a, st);
    case 16416: return launch_tile<1, 64, 16, 4, 4>(a, st);
    case 13216: return launch_tile<1, 32, 16, 4, 4>(a, st);
    case 26432: return launch_tile<2, 64, 32, 4, 2>(a, st);
    case 23232: return launch_tile<2, 32, 32, 4, 2>(a, st);
    case 23216: return launch_tile<2, 32, 16, 4, 4>(a, st);
    case 36432: return launch_tile<3, 64, 32, 3, 2>(a, st);
    case 33232: return launch_tile<3, 32, 32, 3, 2>(a, st);
    case 33216: return launch_tile<3, 32, 16, 3, 4>(a, st);
    case 46432: return launch_tile<4, 64, 32, 4, 2>(a, st);
    case 43232: return launch_tile<4, 32, 32, 4, 2>(a, st);
    case 43216: return launch_tile<4, 32, 16, 4, 4>(a, st);
    case 41616: return launch_tile<4, 16, 16, 4, 4>(a, st);
    case 83232: return launch_tile<8, 32, 32, 4, 2>(a, st);
    case 83216: return launch_tile<8, 32, 16, 4, 2>(a, st);
    case 81616: return launch_tile<8, 16, 16, 4, 4>(a, st);
    case 163216: return launch_tile<16, 32, 16, 8, 2>(a, st);
    case 161616: return launch_tile<16, 16, 16, 4, 2>(a, st);
    default: return set_error(LEECH_E_ARG, "no such batch tile");
  }
}

}  // namespace leech
