// Load-time transcoder on gfx950 (§2.2 "Unfolding at load time": the 47-bit
// index is never decoded in the matvec; each block is expanded once, at load
// time, into its decoded-field record).  Format-v1 block codes -> the Planes14
// main stream, byte for byte what the host expansion writes.
//
// Geometry.  A lane owns one record: a wavefront takes runs of 64 storage slots
// (896 bytes of the stream), puts its records together in LDS of its own and
// writes them with 56 aligned 16-byte stores.  Each lane maps its slot back to
// its (row, column block) in the wave-tile order, reads that block's 8-byte code
// and decodes it.  A workgroup first lays the index table out in LDS (61 KB: two
// workgroups a CU), with what the decode would otherwise compute per block:
// reciprocals of the radices, the binomials, and the class that each run of 2^37
// indices starts in, which leaves the class search a step or two.
//
// Decode.  The lanes of a wave hold blocks of different classes, so the
// longest lane's trip counts hold for all.  Even and odd classes therefore
// take one path: a level's positions come from the support or from the rest
// (odd classes: everything is support), with the two sides' digits and free
// positions selected per lane.  Digits are taken in double precision: all values
// are below 2^47, the quotient by a rounded reciprocal is within one of the true
// one, and the remainder is exact.  The record's words follow from the level-code
// planes and the sign mask by one 4×4 bit transpose and nibble moves.
//
// What bounds it: the vector instructions of the positions' scans (colex
// unranking), not memory (22 bytes a block); and their latency, which is why a
// lane holds one record and not several: with eight records a thread, a 5120 ×
// 5136 matrix made 268 workgroups of 512 threads, one a CU, and took 200 µs.

#include <hip/hip_runtime.h>

#include <string>

#include "index_core.h"
#include "leech_internal.h"

namespace leech {
namespace {

constexpr int kTcThreads = 1024;
constexpr int kTcWaves = kTcThreads / 64;
constexpr int kTcBlocksPerCu = 2;     // two workgroups (each with its LDS table) per CU
constexpr int kRunBytes = 64 * kPlanes14Bytes;   // 896 = 56 × 16
constexpr int kBucketBits = 37;
constexpr int kBuckets = 1 << (kIndexBits - kBucketBits);
constexpr int kTcClasses = 304;       // the ball's 301 classes, rounded up
static_assert(kTcClasses >= kBallClasses, "every class has its LDS entry");

typedef uint32_t u32x4t __attribute__((ext_vector_type(4)));

// Everything a decode reads, in LDS.
struct alignas(16) TcTable {
  uint64_t offset[kTcClasses];
  double A[kTcClasses], B[kTcClasses], rcpA[kTcClasses], rcpB[kTcClasses];
  double rcp[25][32];               // 1 / C(n, k)
  uint32_t binom[25][32];           // C(n, k)
  uint32_t shape[kTcClasses];       // f0 | f2 << 5 | codeword base << 10 | odd << 31
  uint32_t counts[kTcClasses];      // 5 bits a level
  uint32_t levels[kTcClasses];      // side | zero << 5 | mag3 << 10 | sum8 << 15
  uint32_t codeword[2 * 4096];      // by weight; from 4096 on by value
  uint16_t bucket[kBuckets + 2];    // class of index b << 37
};
constexpr size_t kTcLds = sizeof(TcTable) + kTcWaves * kRunBytes;
static_assert(sizeof(TcTable) % 16 == 0 && kTcBlocksPerCu * kTcLds <= 160 * 1024,
              "two workgroups' tables and runs fit in LDS");

struct TranscodeArgs {
  const IdxTable* T;
  const uint64_t* code;
  uint8_t* main;
  uint32_t* bad;
  uint64_t main_bytes, runs;
  uint64_t n;                       // blocks
  uint64_t tile_blocks;             // blocks of a full tile
  uint64_t nb, tiles;
  uint32_t C, R, rows_last;
  uint32_t inv_tile, inv_unit, inv_unit_last;   // 2^32 / d, rounded up
};

// n / d for the reciprocal inv = min(⌈2^32 / d⌉, 2^32 − 1), n < 2^32: before the
// correction at most one too large, or (d = 1) one too small.
__device__ __forceinline__ uint32_t divide(uint32_t n, uint32_t d, uint32_t inv) {
  const uint32_t q = __umulhi(n, inv);
  const int r = (int)(n - q * d);
  return r < 0 ? q - 1 : r >= (int)d ? q + 1 : q;
}

// a / d and a mod d of whole numbers below 2^47, rcp the rounded 1 / d: the
// truncated product is within one of the quotient, and a − q·d is exact.
__device__ __forceinline__ double divmod(double a, double d, double rcp, double* rem) {
  double q = __builtin_trunc(a * rcp);
  double r = __builtin_fma(-q, d, a);
  if (r < 0.0) {
    q -= 1.0;
    r += d;
  } else if (r >= d) {
    q += 1.0;
    r -= d;
  }
  *rem = r;
  return q;
}

__device__ __forceinline__ uint32_t bits_at(uint32_t v, int from, int to, int n) {
  // n bits of v from bit `from`, at bit `to`
  return (v >> from & ((1u << n) - 1)) << to;
}

// Record words of a block from its level-code planes and non-negative mask.
// In pair order a word holds eight coordinates' nibbles, (code, pos) of the four
// pairs' first coordinates and then of their second ones, with the pos bits
// moved up by eight (see planes14_words).
__device__ __forceinline__ void record_words(const uint32_t planes[3], uint32_t pos, uint32_t w[3]) {
  // 4×4 bit transposes: nibble g of n[r] = the four bits of coordinate 4g + r
  const uint32_t mC = 0xCCCCCCCCu, mA = 0xAAAAAAAAu;
  const uint32_t q0 = planes[0], q1 = planes[1], q2 = planes[2], q3 = pos;
  const uint32_t a0 = (q0 & ~mC) | (q2 << 2 & mC), a2 = (q0 >> 2 & ~mC) | (q2 & mC);
  const uint32_t a1 = (q1 & ~mC) | (q3 << 2 & mC), a3 = (q1 >> 2 & ~mC) | (q3 & mC);
  const uint32_t n0 = (a0 & ~mA) | (a1 << 1 & mA), n1 = (a0 >> 1 & ~mA) | (a1 & mA);
  const uint32_t n2 = (a2 & ~mA) | (a3 << 1 & mA), n3 = (a2 >> 1 & ~mA) | (a3 & mA);
  // nibbles, lowest first: (0,4,8,1 | 16,20,12,17), (5,9,2,6 | 21,13,18,22),
  // (10,3,7,11 | 14,19,23,15)
  const uint32_t v[3] = {
      bits_at(n0, 0, 0, 12) | bits_at(n1, 0, 12, 4) | bits_at(n0, 16, 16, 8) |
          bits_at(n0, 12, 24, 4) | bits_at(n1, 16, 28, 4),
      bits_at(n1, 4, 0, 8) | bits_at(n2, 0, 8, 8) | bits_at(n1, 20, 16, 4) |
          bits_at(n1, 12, 20, 4) | bits_at(n2, 16, 24, 8),
      bits_at(n2, 8, 0, 4) | bits_at(n3, 0, 4, 12) | bits_at(n2, 12, 16, 4) |
          bits_at(n3, 16, 20, 8) | bits_at(n3, 12, 28, 4)};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t p = v[k] & 0x88888888u;
    w[k] = (v[k] & 0x77777777u) | p << 8 | p >> 24;
  }
}

// Record words of a 48-bit code (index_core.h: the order of the index): its
// three pair words and class | gain << 9; false if it is not a code.
__device__ __forceinline__ bool decode_code(const TcTable& T, uint64_t n_points, uint64_t code,
                                            uint32_t w[4]) {
  const uint64_t idx = code & kIndexMask;
  const bool ok = code >> 48 == 0 && idx < n_points;
  if (!ok) {
    w[0] = w[1] = w[2] = w[3] = 0;
    return false;
  }
  const uint32_t b = (uint32_t)(idx >> kBucketBits);
  int ci = T.bucket[b];
  for (int hi = T.bucket[b + 1]; ci < hi;) {      // largest class with offset ≤ idx
    const int mid = (ci + hi + 1) >> 1;
    if (T.offset[mid] <= idx) ci = mid;
    else hi = mid - 1;
  }
  uint64_t r = idx - T.offset[ci];
  const uint32_t shape = T.shape[ci], counts = T.counts[ci], lev = T.levels[ci];
  const uint32_t f0 = shape & 31u, f2 = shape >> 5 & 31u;
  const bool odd = shape >> 31;
  const uint32_t s_sup = (uint32_t)r & ((1u << f2) - 1);
  r >>= f2;
  const uint32_t s_off = (uint32_t)r & ((1u << f0) - 1);
  r >>= f0;
  double a_off, a_sup;
  double q = divmod((double)r, T.B[ci], T.rcpB[ci], &a_off);
  q = divmod(q, T.A[ci], T.rcpA[ci], &a_sup);
  const uint32_t cw = T.codeword[(shape >> 10 & 0x1FFFu) + (uint32_t)q];

  // digits, last level first: of the support's levels from a_sup, of the others
  // from a_off
  uint32_t free_s = odd ? 0xFFFFFFu : cw, free_o = ~free_s & 0xFFFFFFu;
  int n_s = idx_popc(free_s), n_o = 24 - n_s;
  const uint32_t* const binom = &T.binom[0][0];
  const double* const rcp = &T.rcp[0][0];
  int at[kMaxLevels];                // the level's binomial C(free, count)
  uint32_t digit[kMaxLevels];
  {
    int ls = n_s, lo = n_o;
#pragma unroll
    for (int k = 0; k < kMaxLevels; ++k) {
      const int c = counts >> (5 * k) & 31u;
      const bool on = lev >> k & 1u;
      at[k] = (on ? ls : lo) * 32 + c;
      ls -= on ? c : 0;
      lo -= on ? 0 : c;
    }
#pragma unroll
    for (int k = kMaxLevels - 1; k >= 0; --k) {
      const bool on = lev >> k & 1u;
      const uint32_t radix = binom[at[k]];
      double rem = 0.0;
      if (radix > 1) {
        const double rest = divmod(on ? a_sup : a_off, (double)radix, rcp[at[k]], &rem);
        a_sup = on ? rest : a_sup;
        a_off = on ? a_off : rest;
      }
      digit[k] = (uint32_t)rem;
    }
  }
  uint32_t planes[3] = {0, 0, 0}, zero = 0, mag3 = 0;
#pragma unroll
  for (int k = 0; k < kMaxLevels; ++k) {
    const int c = counts >> (5 * k) & 31u;
    const bool on = lev >> k & 1u;
    const uint32_t free = on ? free_s : free_o;
    const int nfree = on ? n_s : n_o;
    uint32_t take = 0;
    if (c == nfree) {
      take = c ? free : 0u;
    } else {
      // colex unranking: from the top free position down, the j-th member lies
      // at the highest place q with C(q, j) ≤ what is left of the digit
      uint32_t d = digit[k], scan = free;
      int cell = (nfree - 1) * 32 + c;       // of C(q, j)
      for (int j = c; j > 0;) {
        const uint32_t bit = 1u << idx_top(scan), bn = binom[cell];
        const bool here = bn <= d;
        d -= here ? bn : 0u;
        take |= here ? bit : 0u;
        j -= here ? 1 : 0;
        cell -= here ? 33 : 32;
        scan ^= bit;
      }
    }
    const int level = level_code(k);
#pragma unroll
    for (int p = 0; p < 3; ++p)
      if (level >> p & 1) planes[p] |= take;
    zero |= lev >> (5 + k) & 1u ? take : 0u;
    mag3 |= lev >> (10 + k) & 1u ? take : 0u;
    free_s &= on ? ~take : ~0u;
    free_o &= on ? ~0u : ~take;
    n_s -= on ? c : 0;
    n_o -= on ? 0 : c;
  }
  uint32_t neg = cw ^ mag3;          // odd classes: the codeword forces the signs
  if (!odd) {
    // even classes: see idx_decode for the last support sign
    const uint32_t top = cw ? 1u << idx_top(cw) : 0u;
    neg = idx_deposit(s_off, ~zero & ~cw & 0xFFFFFFu) | idx_deposit(s_sup, cw & ~top);
    if (top && (((lev >> 15) + 4 * idx_popc(neg & cw)) & 7)) neg |= top;
  }
  record_words(planes, ~neg & 0xFFFFFFu, w);
  w[3] = (uint32_t)ci | (uint32_t)(code >> kIndexBits & 1) << 9;
  return true;
}

// Block (row-major) of the storage slot `lane` places after slot s0 of tile t0.
__device__ __forceinline__ uint64_t block_of_slot(const TranscodeArgs& a, uint64_t t0, uint64_t s0,
                                                  int lane) {
  if (a.tile_blocks >> 31) {        // a tile of 2^31 blocks: 64-bit divisions
    uint64_t o = s0 + lane, t = t0;
    if (o >= a.tile_blocks) {
      o -= a.tile_blocks;
      ++t;
    }
    const uint64_t unit = (uint64_t)(t + 1 == a.tiles ? a.rows_last : a.R) * a.C;
    const uint64_t g = o / unit;
    const uint32_t u = (uint32_t)(o - g * unit), cols = (uint32_t)min((uint64_t)a.C, a.nb - g * a.C);
    return (t * a.R + u / cols) * a.nb + g * a.C + u % cols;
  }
  uint32_t o = (uint32_t)s0 + lane;
  const uint32_t tb = (uint32_t)a.tile_blocks, nb = (uint32_t)a.nb;
  const uint32_t dt = divide(o, tb, a.inv_tile);
  o -= dt * tb;
  const uint64_t t = t0 + dt;
  const bool last = t + 1 == a.tiles;
  const uint32_t unit = (last ? a.rows_last : a.R) * a.C;
  const uint32_t g = divide(o, unit, last ? a.inv_unit_last : a.inv_unit);
  const uint32_t u = o - g * unit;
  const uint32_t cols = min(a.C, nb - g * a.C);
  const uint32_t r = u / cols;
  return (t * a.R + r) * nb + g * a.C + (u - r * cols);
}

__global__ __launch_bounds__(kTcThreads) void transcode_planes14_kernel(TranscodeArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  TcTable& T = *reinterpret_cast<TcTable*>(smem);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t n_points = a.T->n_points;
  const int n_classes = (int)min(a.T->n_classes, (uint32_t)kTcClasses);
  for (int i = tid; i < kTcClasses; i += kTcThreads) {
    if (i < n_classes) {
      const IdxClass& c = a.T->cls[i];
      T.offset[i] = c.offset;
      T.A[i] = (double)c.A;
      T.B[i] = (double)c.B;
      T.rcpA[i] = 1.0 / (double)c.A;
      T.rcpB[i] = 1.0 / (double)c.B;
      uint32_t counts = 0, zero = 0, mag3 = 0;
      for (int k = 0; k < c.n_levels; ++k) {
        counts |= (uint32_t)c.count[k] << (5 * k);
        zero |= (uint32_t)(c.mag[k] == 0) << k;
        mag3 |= (uint32_t)((c.mag[k] & 3) == 3) << k;
      }
      const bool odd = c.parity;
      T.shape[i] = (uint32_t)c.f0 | (uint32_t)c.f2 << 5 |
                   (odd ? 4096u : a.T->weight_start[c.w]) << 10 | (uint32_t)odd << 31;
      T.counts[i] = counts;
      T.levels[i] = (uint32_t)c.side | zero << 5 | mag3 << 10 | (uint32_t)c.sum8 << 15;
    } else {
      T.offset[i] = ~0ull;
    }
  }
  for (int i = tid; i < 25 * 32; i += kTcThreads) {
    const uint32_t v = (&a.T->binom[0][0])[i];
    (&T.binom[0][0])[i] = v;
    (&T.rcp[0][0])[i] = v ? 1.0 / (double)v : 0.0;
  }
  for (int i = tid; i < 4096; i += kTcThreads) {
    T.codeword[i] = a.T->cw_weight[i];
    T.codeword[4096 + i] = a.T->cw_value[i];
  }
  __syncthreads();
  for (int b = tid; b < kBuckets + 2; b += kTcThreads) {
    const uint64_t first = (uint64_t)b << kBucketBits;
    int lo = 0, hi = n_classes - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (T.offset[mid] <= first) lo = mid;
      else hi = mid - 1;
    }
    T.bucket[b] = (uint16_t)lo;
  }
  __syncthreads();

  // the workgroup's runs, evenly cut, its waves in turn
  const uint64_t run_end = a.runs * (blockIdx.x + 1) / gridDim.x;
  uint8_t* const stage = smem + sizeof(TcTable) + wave * kRunBytes;
  for (uint64_t run = a.runs * blockIdx.x / gridDim.x + wave; run < run_end; run += kTcWaves) {
    const uint64_t s0 = run * 64;
    const uint64_t t0 = s0 / a.tile_blocks;
    uint32_t w[4] = {0, 0, 0, 0};
    if (s0 + lane < a.n) {
      const uint64_t at = block_of_slot(a, t0, s0 - t0 * a.tile_blocks, lane);
      if (!decode_code(T, n_points, a.code[at], w)) atomicAdd(a.bad, 1u);
    }
    // the run's records, put together in the wave's own LDS: a record starts on
    // an even half word, so every piece is a half word (the LDS serves a wave's
    // operations in order; the fences are for the compiler)
    uint16_t* const rec = reinterpret_cast<uint16_t*>(stage) + 7 * lane;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < 7; ++k) rec[k] = (uint16_t)(w[k / 2] >> (16 * (k & 1)));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane < kRunBytes / 16) {
      const uint64_t out = run * kRunBytes + 16 * lane;
      const u32x4t v = reinterpret_cast<const u32x4t*>(stage)[lane];
      if (out + 16 <= a.main_bytes) {
        *reinterpret_cast<u32x4t*>(a.main + out) = v;
      } else {
        for (int e = 0; e < 16 && out + e < a.main_bytes; ++e)
          a.main[out + e] = (uint8_t)(v[e / 4] >> (8 * (e % 4)));
      }
    }
  }
}

__global__ void clear_u32_kernel(uint32_t* p) { *p = 0; }

// The block scales in storage order: a thread a slot, from slot `first` on, so
// the writes are contiguous and the reads gather; bound by its launch (11 MB of
// scales and less in real matrices).
__global__ __launch_bounds__(256) void scale_order_kernel(TranscodeArgs a, uint64_t first,
                                                          const uint16_t* __restrict__ in,
                                                          uint16_t* __restrict__ out) {
  const uint64_t s0 = first + (uint64_t)blockIdx.x * 256;
  const uint64_t t0 = s0 / a.tile_blocks;
  const int k = threadIdx.x;
  if (s0 + k < a.n) out[s0 + k] = in[block_of_slot(a, t0, s0 - t0 * a.tile_blocks, k)];
}

int tc_fail(const char* what, hipError_t e) {
  return set_error(LEECH_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

}  // namespace
}  // namespace leech

namespace leech {
namespace {
// The slot arithmetic of a matrix in a geometry.
TranscodeArgs slot_args(const Geometry& geo) {
  TranscodeArgs a = {};
  a.n = (uint64_t)geo.M * (uint64_t)geo.nb;
  a.tile_blocks = (uint64_t)geo.R * (uint64_t)geo.nb;
  a.nb = (uint64_t)geo.nb;
  a.C = (uint32_t)geo.C;
  a.R = (uint32_t)geo.R;
  a.tiles = (uint64_t)geo.tiles;
  a.rows_last = (uint32_t)geo.rows_in_tile(geo.tiles - 1);
  auto reciprocal = [](uint64_t d) {
    return (uint32_t)std::min<uint64_t>(((1ull << 32) + d - 1) / d, 0xFFFFFFFFu);
  };
  a.inv_tile = reciprocal(a.tile_blocks);
  a.inv_unit = reciprocal((uint64_t)a.R * a.C);
  a.inv_unit_last = reciprocal((uint64_t)a.rows_last * a.C);
  return a;
}
int check_geometry(const leech_layout_desc* desc) {
  if (desc->M <= 0 || desc->Kpad <= 0 || desc->Kpad % kDim || desc->nb != desc->Kpad / kDim ||
      !geometry_ok(desc->lane_cols, desc->tile_rows))
    return set_error(LEECH_E_SHAPE, "descriptor shape is not valid");
  return LEECH_OK;
}
}  // namespace
}  // namespace leech

using namespace leech;

extern "C" int leech_layout_scales_device(const leech_layout_desc* desc,
                                          const uint16_t* d_scale_rowmajor, uint16_t* d_scale_out,
                                          void* stream) {
  clear_error();
  if (!desc || !d_scale_rowmajor || !d_scale_out) return set_error(LEECH_E_ARG, "NULL argument");
  int rc = check_geometry(desc);
  if (rc) return rc;
  if (((uintptr_t)d_scale_rowmajor & 1) || ((uintptr_t)d_scale_out & 1))
    return set_error(LEECH_E_ARG, "misaligned device pointer");
  const TranscodeArgs a =
      slot_args(Geometry(desc->M, desc->nb, desc->lane_cols, desc->tile_rows));
  const uint64_t most = 0xFFFFFF00ull;      // a launch has fewer than 2^32 threads
  for (uint64_t first = 0; first < a.n; first += most) {
    const uint64_t blocks = (std::min(most, a.n - first) + 255) / 256;
    hipLaunchKernelGGL(scale_order_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       (hipStream_t)stream, a, first, d_scale_rowmajor, d_scale_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return tc_fail("scale order launch", e);
  }
  return LEECH_OK;
}

extern "C" int leech_transcode_planes14(const leech_layout_desc* desc, const void* d_index_table,
                                        const uint64_t* d_code, void* d_main, uint32_t* d_bad,
                                        void* stream) {
  clear_error();
  if (!desc || !d_index_table || !d_code || !d_main || !d_bad)
    return set_error(LEECH_E_ARG, "NULL argument");
  if (desc->layout != LEECH_PLANES14)
    return set_error(LEECH_E_LAYOUT, "the transcoder writes the Planes14 layout only");
  int rc = check_geometry(desc);
  if (rc) return rc;
  const int64_t n = desc->M * desc->nb;
  if (desc->main_bytes != (uint64_t)n * kPlanes14Bytes + kPadBytes)
    return set_error(LEECH_E_SHAPE, "descriptor size is not the Planes14 size of its shape");
  if (((uintptr_t)d_main & 15) || ((uintptr_t)d_code & 7) || ((uintptr_t)d_index_table & 15))
    return set_error(LEECH_E_ARG, "misaligned device pointer");
  TranscodeArgs a = slot_args(Geometry(desc->M, desc->nb, desc->lane_cols, desc->tile_rows));
  a.T = (const IdxTable*)d_index_table;
  a.code = d_code;
  a.main = (uint8_t*)d_main;
  a.bad = d_bad;
  a.main_bytes = desc->main_bytes;
  a.runs = (desc->main_bytes + kRunBytes - 1) / kRunBytes;
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess)
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const uint64_t blocks = std::min<uint64_t>((a.runs + kTcWaves - 1) / kTcWaves,
                                             (uint64_t)kTcBlocksPerCu * (uint64_t)std::max(cus, 1));
  hipError_t e = hipFuncSetAttribute((const void*)transcode_planes14_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTcLds);
  if (e != hipSuccess) return tc_fail("hipFuncSetAttribute", e);
  hipLaunchKernelGGL(clear_u32_kernel, dim3(1), dim3(1), 0, (hipStream_t)stream, d_bad);
  hipLaunchKernelGGL(transcode_planes14_kernel, dim3((unsigned)blocks), dim3(kTcThreads), kTcLds,
                     (hipStream_t)stream, a);
  e = hipGetLastError();
  if (e != hipSuccess) return tc_fail("transcode launch", e);
  return LEECH_OK;
}
