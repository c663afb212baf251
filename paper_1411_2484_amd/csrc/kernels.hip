// gfx950 kernels for the Pohlig-Hellman parameter-split generator:
//   - skip-prefix table segments (eq. (7b) building blocks),
//   - width-64 tile starts, from the 64-bit table for instances that stay
//     in its range, else from the requests' own skip sums (reduce, then a
//     scan per instance); both commit the instance's message,
//   - batched generation (algorithm (9)) as a persistent work-stealing grid
//     or as one plain grid per request,
//   - width-64 positioning and jumps (eq. (7) sums on the device),
//   - the fixed scratch of the allocation-free entry point.
//
// Width-32 tiles are 2048 consecutive draws of one instance whose starting
// state index is a multiple of 2048 within the skip period: the universal
// table holds the skip-prefix sum U and the skip a^r there.  Width-64 tiles
// are 1024 draws, starting at multiples of 1024 skip logarithms (table
// entries) or counted from the first draw of their request (reduce and
// scan).  One wave computes a tile in
// three passes over its LDS row block:
//   A. lane l steps the skip generator over its run of draws, keeps the
//      skips in LDS and sums them;
//   B. a wave scan of the run sums gives each lane its starting message; the
//      lane accumulates its run's messages into LDS (eq. (3a));
//   C. lanes read the messages back in draw order (lane l takes draws
//      i*64 + l), encrypt (eq. (1)), form R and store both coalesced.
// A chunk is a run of consecutive tiles of one request; a wave carries the
// state from one tile to the next within a chunk.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "arith.hpp"
#include "kernels.hpp"
#include "layout.hpp"

namespace phprng {

constexpr int kRow32 = kRun32 + 1;  // padded LDS rows (conflict-free for both access orders)
constexpr int kRow64 = kRun64 + 1;
static_assert((kTilesPerPeriod32 & (kTilesPerPeriod32 - 1)) == 0, "tiles per period is a power of two");
constexpr int kTileShift32 = 20;
static_assert((1ull << kTileShift32) == kTilesPerPeriod32, "tile shift");
// LDS words (64-bit) per wave: 64 rows of the tile and, before them, the last
// row of the tile before it; the width-32 block, or the larger width-64 one.
constexpr int kLdsWords32 = (65 * kRow32 + 1) / 2;  // 1073
constexpr int kLdsWords64 = 65 * kRow64;            // 1105
// The rows of a tile are shifted back to output elements that are multiples of
// these, so that they start at whole 128-byte lines of an array that starts at
// one (32 4-byte or 16 8-byte elements).
constexpr uint32_t kAlign32 = 32, kAlign64 = 16;
static_assert(kAlign32 <= kRun32 && kAlign64 <= kRun64, "one row of the tile before holds the shifted draws");

// ---------------------------------------------------------------------------
// skip-prefix table segments
// ---------------------------------------------------------------------------

// Segment i: start skip a^{i*stride} and the sum of the next `stride` skips.
__global__ void __launch_bounds__(256) table_segments32(uint64_t nseg, uint64_t *seg_sum, uint32_t *seg_start) {
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nseg) return;
  uint32_t s = dev::powmod_p31(kA32, i * kTableStride);
  seg_start[i] = s;
  uint64_t sum = 0;
  for (uint64_t j = 0; j < kTableStride; ++j) {
    s = dev::fold_p31(dev::step_p31(s));
    sum += s;
  }
  seg_sum[i] = sum;
}

__global__ void __launch_bounds__(256) table_segments64(uint64_t nseg, uint64_t *seg_lo, uint64_t *seg_hi,
                                                        uint64_t *seg_start) {
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nseg) return;
  uint64_t s = dev::powmod_p61(kA64, i * kTab64Stride);
  seg_start[i] = s;
  uint64_t lo = 0, hi = 0;
  for (uint64_t j = 0; j < kTab64Stride; ++j) {
    s = dev::step_p61(s);
    uint64_t t = lo + s;
    hi += (t < lo) ? 1 : 0;
    lo = t;
  }
  seg_lo[i] = lo;
  seg_hi[i] = hi;
}

// ---------------------------------------------------------------------------
// instance seeding on the device
// ---------------------------------------------------------------------------

// flags[i] = 1 when output j0 + i of the seeding stream, read as a candidate
// modulus (lo + x mod 2^w) | 1 of the width's range, is prime.
__global__ void __launch_bounds__(256) seed_prime_flags(uint64_t seed, uint64_t j0, uint64_t count, int width,
                                                        uint8_t *flags) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint64_t x = dev::splitmix64_at(seed, j0 + i);
  bool p;
  if (width == 32) {
    const uint32_t n = (uint32_t)((1ull << 31) + (x & ((1ull << 31) - 1))) | 1u;
    p = dev::is_prime32_dev(n);
  } else {
    const uint64_t n = ((1ull << 62) + (x & ((1ull << 62) - 1))) | 1ull;
    p = dev::is_prime64_dev(n);
  }
  flags[i] = p ? 1 : 0;
}

// Instance records for base-state instances (m_0 = 0, s_0 = 1) of one width:
// the same constants the host computes (Montgomery inverse, R^2, R^e, the
// full-period skip sum times R^2, binary64 n + 1 and its reciprocal).
__global__ void __launch_bounds__(256) build_records(const uint64_t *n_arr, const uint64_t *e_arr, uint64_t count,
                                                     int width, InstRec *out) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint64_t n = n_arr[i], e = e_arr[i];
  InstRec rec;
  memset(&rec, 0, sizeof rec);
  rec.n = n;
  rec.e = e;
  rec.width = (uint32_t)width;
  int eb = 0;
  for (uint64_t v = e; v; v >>= 1) ++eb;
  rec.ebits = (uint32_t)eb;
  rec.ekind = (e == 3 || e == 5 || e == 9 || e == 17) ? (uint32_t)e : 0u;
  rec.sched = kSchedSkipLcg;
  rec.den = (double)(n + 1);
  if (width == 32) {
    const uint32_t n32 = (uint32_t)n, ninv = dev::inv32(n32);
    const uint32_t one = 0u - n32;
    uint32_t r2 = one;
    for (int k = 0; k < 32; ++k) r2 = dev::addmod32(r2, r2, n32);
    // R^e: the Montgomery power of R (Montgomery form R^2) is R^{e+1}; one more REDC
    const uint32_t re1 = dev::mpow32(r2, e, one, n32, ninv);
    rec.ninv = ninv;
    rec.r2 = r2;
    rec.kcorr = n32 - dev::mont32(re1, 1u, n32, ninv);
    // p(p-1)/2 mod n, then times R^2: mont(b, R^3) with R^3 = mont(R^2, R^2)
    const uint64_t full = ((uint64_t)kP32 * ((uint64_t)kP32 - 1)) / 2;
    const uint32_t b = dev::mont32(dev::redc32(full, n32, ninv), r2, n32, ninv);
    rec.br2 = dev::mont32(b, dev::mont32(r2, r2, n32, ninv), n32, ninv);
    rec.rcp = 1.0 / rec.den;
  } else {
    const uint64_t ninv = dev::inv64(n);
    uint64_t one = 0ull - n;
    while (one >= n) one -= n;
    uint64_t r2 = one;
    for (int k = 0; k < 64; ++k) r2 = dev::addmod64(r2, r2, n);
    const uint64_t re1 = dev::mpow64(r2, e, one, n, ninv);
    rec.ninv = ninv;
    rec.r2 = r2;
    rec.kcorr = n - dev::mont64(re1, 1ull, n, ninv);
    rec.br2 = 0;
    rec.rcp = 1.0 / rec.den;
  }
  rec.rcp_lo = __builtin_fma(-rec.den, rec.rcp, 1.0) / rec.den;  // the fma is exact
  out[i] = rec;
}

// ---------------------------------------------------------------------------
// width-64 skip sums from the positioning table (eq. (7b))
// ---------------------------------------------------------------------------

// U(t) mod n for t < kTab64Range: the table entry at or below t plus at most
// kTab64Stride - 1 steps of the skip generator, then the 128-bit sum reduced
// mod n.
__device__ uint64_t table_prefix64(const uint64_t *u_lo, const uint64_t *u_hi, const uint64_t *u_s, uint64_t t,
                                   uint64_t n, uint64_t ninv, uint64_t r2) {
  const uint64_t i = t / kTab64Stride;
  uint64_t lo = u_lo[i], hi = u_hi[i], s = u_s[i];
  for (uint64_t x = i * kTab64Stride; x < t; ++x) {
    s = dev::step_p61(s);
    const uint64_t v = lo + s;
    hi += v < lo ? 1 : 0;
    lo = v;
  }
  // hi < 2^30 < n, so REDC applies; times R^2 undoes the 2^-64
  dev::W128 w;
  w.lo = lo;
  w.hi = hi;
  return dev::mont64(dev::redc64(w, n, ninv), r2, n, ninv);
}

// m64[ids[i]] = m0[i] + U(ta[i]) - U(tb[i]) mod n, for skip logarithms
// ta, tb < kTab64Range (one thread per instance).  With ta = t0 + k0 and
// tb = t0 this is the message at position k0 of an instance whose state at
// position 0 is (m0, a^t0) (eq. (7b)); a jump by d from skip log t takes
// ta = t + d, tb = t (backward: ta = t - d).
__global__ void __launch_bounds__(256) position64_kernel(const InstRec *inst, const uint32_t *ids, const uint64_t *m0,
                                                         const uint64_t *ta, const uint64_t *tb, uint64_t count,
                                                         const uint64_t *u_lo, const uint64_t *u_hi,
                                                         const uint64_t *u_s, uint64_t *m64) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const InstRec &I = inst[ids[i]];
  const uint64_t n = I.n, ninv = I.ninv, r2 = I.r2;
  const uint64_t a = ta ? ta[i] : 0, b = tb ? tb[i] : 0;
  const uint64_t ua = a ? table_prefix64(u_lo, u_hi, u_s, a, n, ninv, r2) : 0;
  const uint64_t ub = b ? table_prefix64(u_lo, u_hi, u_s, b, n, ninv, r2) : 0;
  const uint64_t m = dev::addmod64(m0 ? m0[i] : 0, ua, n);
  m64[ids[i]] = m >= ub ? m - ub : m + (n - ub);
}

// ---------------------------------------------------------------------------
// width-64 tile starts: reduce, then scan per instance
// ---------------------------------------------------------------------------

// Wave-cooperative search over a sorted key: the last index r in [0, nreq)
// with key(r) <= c (the last such r when empty requests share a key).
template <typename Key>
__device__ __forceinline__ uint64_t wave_search(uint64_t nreq, uint64_t c, uint32_t lane, Key key) {
  uint64_t lo = 0, hi = nreq;
  while (hi - lo > 1) {
    const uint64_t step = (hi - lo + 63) / 64;
    const uint64_t idx = lo + (uint64_t)lane * step;
    const bool le = idx < hi && key(idx) <= c;
    const uint64_t mask = __ballot(le);
    const uint64_t k = (uint64_t)__popcll(mask);
    lo = lo + (k - 1) * step;
    hi = min(lo + step, hi);
  }
  return lo;
}

// The batch's planned requests: the kernel's own arguments for a small batch.
// (GenArgs is every kernel's first parameter.)
using ArgPtr = const __attribute__((address_space(4))) char *;
__device__ __forceinline__ const ReqRec *requests(const GenArgs &A) {
  const ArgPtr args = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  return A.nreq <= kInlineReqs ? (const ReqRec *)(args + offsetof(GenArgs, inline_req)) : A.req;
}

// The kernel arguments, read again from the scalar cache: for a loop whose
// body would otherwise hold all of them in scalar registers (and spill them).
__device__ __forceinline__ const GenArgs &args_again() {
  ArgPtr args = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  return *(const GenArgs *)args;
}

// Start of the call, from the kernel that is its first.
__device__ __forceinline__ void stamp_begin(const GenArgs &A) {
  if (A.stamp && A.stamp_start && blockIdx.x == 0 && threadIdx.x == 0) A.stamp[0] = (uint64_t)wall_clock64();
}

// End of wave w of the generation kernel, its stores included.
__device__ __forceinline__ void stamp_end(const GenArgs &A, uint32_t w, uint32_t lane) {
  if (!A.stamp) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (lane == 0) A.stamp[1 + w] = (uint64_t)wall_clock64();
}

// Sum, mod n, of the skips of lane `lane`'s run of kRun64 draws in a tile
// that starts with skip s_tile and holds `len` draws; every lane gets the
// tile total.
__device__ __forceinline__ uint64_t tile_skip_sum64(uint64_t s_tile, uint64_t lane_mul, uint32_t len, uint64_t n,
                                                    uint32_t lane) {
  uint64_t s = dev::mulmod_p61(s_tile, lane_mul);
  uint64_t sum = 0;
  const uint32_t first = lane * kRun64;
#pragma unroll 4
  for (int i = 0; i < kRun64; ++i) {
    s = dev::step_p61(s);
    if (first + (uint32_t)i < len) sum = dev::addmod64(sum, s, n);
  }
  return dev::wave_sum_mod(sum, n);
}

// Draws in tile j of a width-64 request: 1024, or what is left in its last
// tile.  Written with a 32-bit test of the tile index: a wave-uniform 64-bit
// "rem < 1024 ? rem : 1024" has been compiled for gfx950 into a select that
// reads a stale SCC after the branch on the same comparison, which gave 1024
// for every last tile.
__device__ __forceinline__ uint32_t tile_len64(const ReqRec &R, uint32_t j, uint32_t head = 0) {
  // one past the request's last draw, counted from the first tile's start
  const uint32_t last = (uint32_t)(R.count + head - (uint64_t)(R.ntiles - 1) * kTile64);
  return j + 1 == R.ntiles ? last : (uint32_t)kTile64;
}

// One wave per reduce unit (grid-stride): up to A.reduce_tiles consecutive
// tiles of one width-64 request.  For each tile j of a request starting at
// skip log t it writes the skip before the tile, a^{t + 1024 j} mod p (a
// power for the unit's first tile, then carried from tile to tile), and the
// sum of the tile's skips mod n.
__global__ void __launch_bounds__(256) reduce64_kernel(GenArgs A) {
  const uint32_t lane = dev::lane_id();
  const uint32_t wave = dev::uniform_u32(threadIdx.x / 64);
  stamp_begin(A);
  const ReqRec *const req = requests(A);
  const uint64_t units = A.units64, nreq64 = A.nreq64;
  const uint32_t rt = A.reduce_tiles;
  const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x / 64);
  const uint64_t lane_mul = A.lanemul->m64[lane];
  const uint64_t pm1 = kP64 - 1;
  for (uint64_t u = (uint64_t)blockIdx.x * (blockDim.x / 64) + wave; u < units; u += nwaves) {
    const uint64_t r =
        dev::uniform_u64(wave_search(nreq64, u, lane, [&](uint64_t i) { return req[i].rbase; }));
    const ReqRec R = dev::const_load(req + r);
    const uint64_t n = dev::const_load(&A.inst[R.inst].n);
    const uint32_t j0 = (uint32_t)(u - R.rbase) * rt;
    const uint32_t j1 = R.ntiles - j0 > rt ? j0 + rt : R.ntiles;
    uint64_t lg = R.x + (uint64_t)j0 * kTile64;  // x < p - 1 and j * 1024 < 2^42: one subtraction wraps it
    if (lg >= pm1) lg -= pm1;
    uint64_t s_tile = dev::wave_pow_p61(A.lanemul->pow64, lg, lane);
    const uint64_t a8 = A.lanemul->pow64[3];  // a^8
    for (uint32_t j = j0; j < j1; ++j) {
      const uint32_t len = tile_len64(R, j);
      uint64_t sum;
      uint64_t s = dev::mulmod_p61(s_tile, lane_mul);  // skip before the lane's run
      if (len == kTile64) {
        // The run as two independent chains of 8 skips (more work in flight
        // per lane).  Eight skips below 2^61 sum below 2^64 < 4n, so each
        // chain is summed in plain 64-bit adds and reduced once.
        uint64_t s2 = dev::mulmod_p61(s, a8);
        uint64_t g1 = 0, g2 = 0;
#pragma unroll
        for (int i = 0; i < kRun64 / 2; ++i) {
          s = dev::step_p61(s);
          s2 = dev::step_p61(s2);
          g1 += s;
          g2 += s2;
        }
        sum = dev::addmod64(dev::mod_below_4n(g1, n), dev::mod_below_4n(g2, n), n);
        s = s2;
      } else {
        // the request's last tile: only draws below len count
        const uint32_t first = lane * kRun64;
        sum = 0;
#pragma unroll 4
        for (int i = 0; i < kRun64; ++i) {
          s = dev::step_p61(s);
          if (first + (uint32_t)i < len) sum = dev::addmod64(sum, s, n);
        }
      }
      sum = dev::wave_sum_mod(sum, n);
      if (lane == 0) {
        A.t64.s[R.g1 + j] = s_tile;
        A.t64.sum[R.g1 + j] = sum;
      }
      s_tile = dev::shfl_u64(s, 63);  // the skip after the tile's last draw
    }
  }
}

// ---------------------------------------------------------------------------
// width-64 tile starts from the table (batches whose draws all lie below
// kTab64Range)
// ---------------------------------------------------------------------------

// A table entry U(i * kTab64Stride) (128 bits, read as w) reduced mod n:
// U < 2^95 < n 2^64, so one REDC and a product with R^2 give it.  n is the
// same in every lane of the wave.
__device__ __forceinline__ uint64_t table_u_mod64(dev::W128 w, uint64_t n, uint64_t ninv, uint64_t r2) {
  return dev::mont64_uniform(dev::redc64_uniform(w, n, ninv), r2, n, ninv);
}

// U(x) mod n and U(y) mod n for x, y < kTab64Range by the whole wave: the
// entry at or below each plus the (at most kTab64Stride - 1) skips after
// it, lane l taking the 16 skip indices from T + 16 l + 1.  The table reads
// of both positions are issued before either is used, and the two skip
// chains run side by side.  Every lane gets both results.
__device__ void wave_prefix64_pair(const SkipTables &T, uint64_t x, uint64_t y, uint64_t n, uint64_t ninv,
                                   uint64_t r2, uint64_t lane_mul, uint32_t lane, uint64_t *ux, uint64_t *uy) {
  const uint64_t ix = x / kTab64Stride, iy = y / kTab64Stride;
  const uint32_t rx = (uint32_t)(x - ix * kTab64Stride), ry = (uint32_t)(y - iy * kTab64Stride);
  const uint64_t sx0 = dev::const_load(T.s64 + ix), sy0 = dev::const_load(T.s64 + iy);
  const dev::W128 wx{dev::const_load(T.u64lo + ix), dev::const_load(T.u64hi + ix)};
  const dev::W128 wy{dev::const_load(T.u64lo + iy), dev::const_load(T.u64hi + iy)};
  uint64_t sx = dev::mulmod_p61(sx0, lane_mul), sy = dev::mulmod_p61(sy0, lane_mul);
  uint64_t sumx = 0, sumy = 0;
  const uint32_t first = lane * kRun64;
#pragma unroll 4
  for (int k = 0; k < kRun64; ++k) {
    sx = dev::step_p61(sx);
    sy = dev::step_p61(sy);
    if (first + (uint32_t)k < rx) sumx = dev::addmod64(sumx, sx, n);
    if (first + (uint32_t)k < ry) sumy = dev::addmod64(sumy, sy, n);
  }
  *ux = dev::addmod64(table_u_mod64(wx, n, ninv, r2), dev::wave_sum_mod(sumx, n), n);
  *uy = dev::addmod64(table_u_mod64(wy, n, ninv, r2), dev::wave_sum_mod(sumy, n), n);
}

// One wave per width-64 request; the first request of each instance in the
// batch whose tiles start at table entries (seg count > 0 and kSegTable)
// serves all of that instance's requests.  With m the
// instance's committed message at skip log x (its first request's start),
// mbase = m - U(x) mod n gives the message at any skip log t of the range as
// mbase + U(t) (eq. (7b)).  Each tile of the requests starts at a table
// entry, so its skip a^t and message come straight from the table.  The
// wave then commits the message after the instance's last draw in the batch.
__global__ void __launch_bounds__(64) tab64_kernel(GenArgs A) {
  const uint32_t lane = dev::lane_id();
  stamp_begin(A);
  const ReqRec *const req = requests(A);
  const ReqRec R0 = dev::const_load(req + blockIdx.x);
  const uint32_t seg = R0.seg & kSegCount;
  if (seg == 0 || !(R0.seg & kSegTable)) return;
  const InstRec &I = A.inst[R0.inst];
  const uint64_t n = dev::const_load(&I.n), ninv = dev::const_load(&I.ninv), r2 = dev::const_load(&I.r2);
  const uint64_t lane_mul = A.lanemul->m64[lane];
  const uint64_t m0 = dev::uniform_u64(A.m64[R0.inst]);
  // U at the instance's first and last positions in the batch
  const ReqRec RL = dev::const_load(req + blockIdx.x + seg - 1);
  uint64_t u0, ue;
  wave_prefix64_pair(A.tab, R0.x, RL.x + RL.count, n, ninv, r2, lane_mul, lane, &u0, &ue);
  const uint64_t mbase = m0 >= u0 ? m0 - u0 : m0 + (n - u0);
  for (uint32_t q = 0; q < seg; ++q) {
    const ReqRec R = dev::const_load(req + blockIdx.x + q);
    const uint64_t e0 = R.x / kTab64Stride;
    // the table reads of kTabGroup tiles per lane are issued before any of
    // them is used, so their latencies overlap (a long request has up to
    // 16 tiles per lane)
    constexpr int kTabGroup = 8;
    for (uint32_t j0 = 0; j0 < R.ntiles; j0 += 64 * kTabGroup) {
      // lanes past the request's last tile compute on zeros and store nothing
      uint64_t sv[kTabGroup] = {}, ulo[kTabGroup] = {}, uhi[kTabGroup] = {};
#pragma unroll
      for (int k = 0; k < kTabGroup; ++k) {
        const uint32_t j = j0 + 64 * k + lane;
        if (j < R.ntiles) {
          sv[k] = dev::const_load(A.tab.s64 + e0 + j);
          ulo[k] = dev::const_load(A.tab.u64lo + e0 + j);
          uhi[k] = dev::const_load(A.tab.u64hi + e0 + j);
        }
      }
      uint64_t mv[kTabGroup];
#pragma unroll
      for (int k = 0; k < kTabGroup; ++k) {
        // mbase + U(1024 e) mod n
        mv[k] = dev::addmod64(mbase, table_u_mod64({ulo[k], uhi[k]}, n, ninv, r2), n);
      }
#pragma unroll
      for (int k = 0; k < kTabGroup; ++k) {
        const uint32_t j = j0 + 64 * k + lane;
        if (j < R.ntiles) {
          A.t64.s[R.g1 + j] = sv[k];
          A.t64.m[R.g1 + j] = mv[k];
        }
      }
    }
  }
  if (lane == 0) A.m64[R0.inst] = dev::addmod64(mbase, ue, n);
}

// Scan per instance: one workgroup per width-64 request; the first request
// of each instance in the batch (seg > 0) turns the tile sums of all of that
// instance's requests into tile-start messages, starting from the
// instance's committed message, and commits the message after the last
// draw.  The instance's requests hold consecutive tiles.
constexpr int kScanThreads = 256;
constexpr int kScanPer = 4;

__global__ void __launch_bounds__(kScanThreads) scan64_kernel(GenArgs A) {
  __shared__ uint64_t wtot[kScanThreads / 64];
  const uint64_t r = blockIdx.x;
  stamp_begin(A);
  const ReqRec *const req = requests(A);
  const ReqRec R = dev::const_load(req + r);
  const uint32_t seg = R.seg & kSegCount;
  if (seg == 0 || (R.seg & kSegTable)) return;
  const ReqRec L = dev::const_load(req + r + seg - 1);
  const uint64_t n = dev::const_load(&A.inst[R.inst].n);
  const uint64_t t0 = R.g1, t1 = L.g1 + L.ntiles;
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint64_t carry = A.m64[R.inst];
  for (uint64_t base = t0; base < t1; base += (uint64_t)kScanThreads * kScanPer) {
    const uint64_t first = base + (uint64_t)tid * kScanPer;
    uint64_t v[kScanPer];
    uint64_t tot = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      v[q] = first + q < t1 ? A.t64.sum[first + q] : 0;
      tot = dev::addmod64(tot, v[q], n);
    }
    // exclusive prefix of the thread totals over the workgroup
    const uint64_t ex = dev::wave_exclusive_mod(tot, n);
    if (lane == 63) wtot[w] = dev::addmod64(ex, tot, n);
    __syncthreads();
    uint64_t before = carry, all = carry;
#pragma unroll
    for (int k = 0; k < kScanThreads / 64; ++k) {
      if (k < (int)w) before = dev::addmod64(before, wtot[k], n);
      all = dev::addmod64(all, wtot[k], n);
    }
    __syncthreads();
    uint64_t m = dev::addmod64(before, ex, n);
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      if (first + q < t1) A.t64.m[first + q] = m;
      m = dev::addmod64(m, v[q], n);
    }
    carry = all;
  }
  if (tid == 0) A.m64[R.inst] = carry;
}

// ---------------------------------------------------------------------------
// width-64 jumps off the table: sum of `count` consecutive skips
// ---------------------------------------------------------------------------

// partial[w] = sum, mod n, of the skips a^{t+1+i} mod p for the blocks of
// 1024 draws i in [1024 b, 1024 (b + 1)) ∩ [0, count) that wave w takes
// (b = w, w + nwaves, ...).
__global__ void __launch_bounds__(256) skip_total64_kernel(uint64_t t, uint64_t count, uint64_t n,
                                                           const LaneMul *lm, uint64_t *partial) {
  const uint32_t lane = dev::lane_id();
  const uint32_t wave = dev::uniform_u32(threadIdx.x / 64);
  const uint64_t w = (uint64_t)blockIdx.x * (blockDim.x / 64) + wave;
  const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x / 64);
  const uint64_t pm1 = kP64 - 1;
  const uint64_t lane_mul = lm->m64[lane];
  const uint64_t nblk = (count + kTile64 - 1) / kTile64;
  uint64_t acc = 0;
  for (uint64_t b = w; b < nblk; b += nwaves) {
    const uint64_t off = (b * kTile64) % pm1;
    uint64_t lg = t + off;
    if (lg >= pm1) lg -= pm1;
    const uint64_t s0 = dev::wave_pow_p61(lm->pow64, lg, lane);
    // the last block holds what is left (an equality test: see tile_len64)
    const uint32_t len = b + 1 == nblk ? (uint32_t)(count - (nblk - 1) * kTile64) : (uint32_t)kTile64;
    acc = dev::addmod64(acc, tile_skip_sum64(s0, lane_mul, len, n, lane), n);
  }
  if (lane == 0) partial[w] = acc;
}

// *m = *m + sign * (sum of the partials + extra) mod n (one wave).
__global__ void __launch_bounds__(64) skip_total64_apply(const uint64_t *partial, uint64_t nparts, uint64_t n,
                                                         uint64_t extra, int sign, uint64_t *m) {
  const uint32_t lane = threadIdx.x;
  uint64_t acc = 0;
  for (uint64_t i = lane; i < nparts; i += 64) acc = dev::addmod64(acc, partial[i], n);
  acc = dev::wave_sum_mod(acc, n);
  acc = dev::addmod64(acc, extra, n);
  if (lane == 0) {
    const uint64_t v = *m;
    *m = sign > 0 ? dev::addmod64(v, acc, n) : (v >= acc ? v - acc : v + (n - acc));
  }
}

// ---------------------------------------------------------------------------
// tiles
// ---------------------------------------------------------------------------

// Which outputs a pass writes (bit 0: ciphertexts, bit 1: uniforms).
enum { kOutC = 1, kOutR = 2 };

struct Enc32 {
  uint32_t n, ninv, kc;
  uint64_t e;
  int ebits;
  double rcp, rcp_lo;
};

// What a draw stores: its ciphertext and its uniform.
template <class C>
struct Draw {
  C c;
  double r;
};

// The draw of one message of a width-32 tile (x = n - m).
template <int EK, int OUT>
__device__ __forceinline__ Draw<uint32_t> draw32(uint32_t x, const Enc32 &K) {
  Draw<uint32_t> d{};
  if constexpr (OUT & kOutC) {
    d.c = dev::encrypt32<EK>(x, K.n, K.ninv, K.kc, K.e, K.ebits);
    if constexpr (OUT & kOutR) d.r = dev::uniform32(d.c + 1u, K.rcp, K.rcp_lo);
  } else {
    d.r = dev::uniform32(dev::encrypt32<EK, 1>(x, K.n, K.ninv, K.kc, K.e, K.ebits), K.rcp, K.rcp_lo);
  }
  return d;
}

template <int OUT, class C>
__device__ __forceinline__ void put_draw(const Draw<C> &d, C *c, double *r) {
  if constexpr (OUT & kOutC) *c = d.c;
  if constexpr (OUT & kOutR) *r = d.r;
}

// Pass C works on rows of 64 consecutive draws, one per lane.  The rows of a
// tile are shifted back by `shift` draws, so that row r holds the draws
// t = 64 r + lane - shift and its stores cover whole 128-byte lines whatever
// the request's output offset, in arrays that start at a line (rows that
// straddle lines cost 6% of the store rate for uniforms and 10% with
// ciphertexts).  u = t + shift counts from the
// first row; the pass writes u in [u_lo, u_hi): whole rows in groups of UNROLL
// (all messages, then all encryptions, then all stores of a group), the rows
// at either end masked one at a time.  get(k) gives this lane's message of the
// k-th row from the current one, calc(x) what is stored for it, put(k, v)
// stores it, and next(n) makes the n-th row from here the current one (the
// first is row u_lo / 64).
template <int UNROLL, class Get, class Calc, class Put, class Next>
__device__ __forceinline__ void row_loop(uint32_t u_lo, uint32_t u_hi, uint32_t lane, Get get, Calc calc, Put put,
                                         Next next) {
  const uint32_t whole_end = u_hi >> 6, end = (u_hi + 63) >> 6;
  uint32_t r = u_lo >> 6;
  for (;;) {
    // masked rows: the first when u_lo cuts it, and what is left at the end
    while (r < end && ((r << 6) < u_lo || r + UNROLL > whole_end)) {
      if ((r << 6) + lane - u_lo < u_hi - u_lo) put(0, calc(get(0)));
      next(1);
      ++r;
    }
    if (r >= end) break;
    for (; r + UNROLL <= whole_end; r += UNROLL) {
      decltype(get(0)) x[UNROLL];
      decltype(calc(get(0))) v[UNROLL];
#pragma unroll
      for (int k = 0; k < UNROLL; ++k) x[k] = get(k);
#pragma unroll
      for (int k = 0; k < UNROLL; ++k) v[k] = calc(x[k]);
#pragma unroll
      for (int k = 0; k < UNROLL; ++k) put(k, v[k]);
      next(UNROLL);
    }
  }
}

// The part of a tile's rows that wave `part` of the 2^split waves which share
// the tile writes (each computes the whole tile's messages).
__device__ __forceinline__ void part_of_rows(uint32_t split, uint32_t part, uint32_t tile, uint32_t *u_lo,
                                             uint32_t *u_hi) {
  const uint32_t span = tile >> split;
  const uint32_t lo = max(*u_lo, part * span);
  *u_hi = max(lo, (part + 1) >> split ? *u_hi : min(*u_hi, (part + 1) * span));
  *u_lo = lo;
}

// Calls f with the exponent chain and the outputs as compile-time constants.
template <int V>
struct Const {
  static constexpr int value = V;
};
template <int EK, class F>
__device__ __forceinline__ void with_outputs(bool c, bool r, F f) {
  if (c && r) f(Const<EK>(), Const<kOutC | kOutR>());
  else if (r) f(Const<EK>(), Const<kOutR>());
  else if (c) f(Const<EK>(), Const<kOutC>());
}
template <class F>
__device__ __forceinline__ void with_chain(int ekind, bool c, bool r, F f) {
  switch (ekind) {
    case 9: with_outputs<9>(c, r, f); break;
    case 17: with_outputs<17>(c, r, f); break;
    case 3: with_outputs<3>(c, r, f); break;
    case 5: with_outputs<5>(c, r, f); break;
    default: with_outputs<0>(c, r, f); break;
  }
}

template <int UNROLL>
__device__ void run_chunk32(const GenArgs &A, const InstRec &I, const ReqRec &R, uint64_t chunk, uint32_t part,
                            uint32_t *L, uint32_t lane) {
  const uint32_t n = (uint32_t)I.n, ninv = (uint32_t)I.ninv, kc = (uint32_t)I.kcorr, r2 = (uint32_t)I.r2;
  const uint32_t br2 = (uint32_t)I.br2;
  const uint64_t e = I.e;
  const int ebits = (int)I.ebits, ekind = (int)I.ekind;
  const Enc32 K{n, ninv, kc, e, ebits, I.rcp, I.rcp_lo};
  const uint64_t pm1 = (uint64_t)kP32 - 1;
  const uint32_t lane_mul = A.lanemul->m32[lane];
  const uint32_t one = dev::opaque_one();

  const uint64_t g_begin = R.g1 + chunk * A.tiles_per_chunk;
  const uint64_t g_end = min(g_begin + A.tiles_per_chunk, R.g1 + R.ntiles);
  uint32_t *const T = L + kRow32;  // the tile's rows; the row before holds the last 32 messages of the tile before
  uint32_t m_t = 0, s_t = 0;
  bool carried = false;
  bool deferred = false;  // the tile before left its last `shift` draws to this one
  uint32_t u_next = 0;    // and this is where the request begins among its rows
  for (uint64_t g = g_begin; g < g_end; ++g) {
    const uint64_t q = g >> kTileShift32;
    const uint32_t j = (uint32_t)(g & (kTilesPerPeriod32 - 1));
    const uint64_t x0 = q * pm1 + (uint64_t)j * kTile32;
    if (!carried || j == 0) {
      // state at x0 from the universal table (eq. (7)):
      // m = mbase + q p(p-1)/2 + U(j*2048) mod n,  s = a^{j*2048} mod p
      const uint64_t u = A.tab.u32[j];
      s_t = A.tab.s32[j];
      uint32_t mu = dev::mont32(dev::redc32(u + I.mbase, n, ninv), r2, n, ninv);
      uint32_t mq = dev::mont32(dev::redc32(q, n, ninv), br2, n, ninv);
      m_t = dev::addmod32(mu, mq, n);
    }
    // ---- pass A: skips of this lane's run, their sum (two skips < 2^31 add
    // below 2^32 before they enter the 64-bit sum)
    uint32_t *row = T + lane * kRow32;
    uint32_t s = dev::mulmod_p31(s_t, lane_mul);
    uint64_t sum = 0;
#pragma unroll 4
    for (int i = 0; i < kRun32; i += 2) {
      const uint32_t v0 = dev::step_p31(s);
      const uint32_t v1 = dev::step_p31(v0);
      const uint32_t s0 = dev::fold_p31(v0);
      s = dev::fold_p31(v1);
      row[i] = s0;
      row[i + 1] = s;
      sum = dev::acc_u32(sum, s0 + s, one);
    }
    // ---- pass B: exclusive wave scan of run sums -> run start message,
    // carried as x = n - m: the encryption takes the sign back (kcorr), and
    // x - s mod n is one instruction shorter than m + s mod n
    const uint64_t incl = dev::wave_inclusive_sum(sum);
    uint32_t x = n - dev::mont32(dev::redc32(incl - sum + m_t, n, ninv), r2, n, ninv);
#pragma unroll 8
    for (int i = 0; i < kRun32; ++i) {
      x = dev::submod32(x, row[i], n);
      row[i] = x;
    }
    // state at the end of the tile (lane 63's last message and skip)
    m_t = n - (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
    s_t = (uint32_t)__builtin_amdgcn_readlane((int)s, 63);
    carried = true;
    dev::wave_lds_sync();
    // ---- pass C: encrypt in draw order.  Draw t of this tile comes from
    // state index x0 + t; a tile before another one of its chunk and period
    // leaves its last `shift` draws to that tile's first row.
    const uint64_t last = j + 1 == kTilesPerPeriod32 ? pm1 - (uint64_t)j * kTile32 : (uint64_t)kTile32;
    const bool flush = g + 1 == g_end || j + 1 == kTilesPerPeriod32;
    const int64_t base = (int64_t)R.out_off + (int64_t)(x0 - R.x);  // output element of draw 0
    const uint32_t shift = (uint32_t)base & (kAlign32 - 1);
    uint32_t u_lo = deferred ? u_next : shift + (R.x > x0 ? (uint32_t)(R.x - x0) : 0u);
    uint32_t u_hi = flush ? shift + (uint32_t)min(R.x + R.count - x0, last) : (uint32_t)kTile32;
    if (A.split) part_of_rows(A.split, part, kTile32, &u_lo, &u_hi);
    const int t0 = (int)lane - (int)shift;
    const uint32_t *src = T + (t0 >> 5) * kRow32 + (t0 & 31);
    const int64_t at = base - (int64_t)shift + (int64_t)(u_lo & ~63u) + (int64_t)lane;
    uint32_t *cp = A.out_c32 + at;
    double *rp = A.out_r + at;
    const uint32_t *sp = src + (u_lo >> 6) * (2 * kRow32);
    with_chain(ekind, A.out_c32 != nullptr, A.out_r != nullptr, [&](auto ek, auto out) {
      constexpr int EK = decltype(ek)::value, OUT = decltype(out)::value;
      row_loop<UNROLL>(
          u_lo, u_hi, lane, [&](int k) { return sp[k * (2 * kRow32)]; },
          [&](uint32_t v) { return draw32<EK, OUT>(v, K); },
          [&](int k, const Draw<uint32_t> &d) { put_draw<OUT>(d, cp + k * 64, rp + k * 64); },
          [&](int k) {
            sp += k * (2 * kRow32);
            cp += k * 64;
            rp += k * 64;
          });
    });
    deferred = !flush;
    u_next = u_lo > (uint32_t)kTile32 ? u_lo - (uint32_t)kTile32 : 0u;  // all of this tile's draws deferred
    if (deferred && lane < 32) L[lane] = T[63 * kRow32 + lane];
    dev::wave_lds_sync();
  }
}

struct Enc64 {
  uint64_t n, ninv, kc, e;
  int ebits;
  double den, rcp, rcp_lo;
};

// The draw of one message of a width-64 tile (x = n - m).
template <int EK, int OUT>
__device__ __forceinline__ Draw<uint64_t> draw64(uint64_t x, const Enc64 &K) {
  Draw<uint64_t> d{};
  if constexpr (OUT & kOutC) {
    d.c = dev::encrypt64<EK>(x, K.n, K.ninv, K.kc, K.e, K.ebits);
    if constexpr (OUT & kOutR) d.r = dev::uniform64(d.c + 1, K.den, K.rcp, K.rcp_lo);
  } else {
    d.r = dev::uniform64(dev::encrypt64<EK, 1>(x, K.n, K.ninv, K.kc, K.e, K.ebits), K.den, K.rcp, K.rcp_lo);
  }
  return d;
}

// Width 64: tile j of the request covers its draws [1024 j, 1024 (j + 1)),
// or, when the instance's tiles start at table entries, the skip logarithms
// (1024 (e0 + j), 1024 (e0 + j + 1)] with e0 = x / 1024, of which the first
// tile skips the part before the request.  The state before the chunk's
// first tile comes from the scan or the table kernel; later tiles continue
// from lane 63's last state.
template <int UNROLL>
__device__ void run_chunk64(const GenArgs &A, const InstRec &I, const ReqRec &R, uint64_t chunk, uint32_t part,
                            uint64_t *L, uint32_t lane) {
  const uint64_t n = I.n, ninv = I.ninv, kc = I.kcorr;
  const uint64_t e = I.e;
  const int ebits = (int)I.ebits, ekind = (int)I.ekind;
  const uint64_t lane_mul = A.lanemul->m64[lane];

  const uint32_t j_begin = (uint32_t)chunk * A.tiles_per_chunk;
  const uint32_t j_end = min(j_begin + A.tiles_per_chunk, R.ntiles);
  const bool tab = (R.seg & kSegTable) != 0;
  // draw t of tile j is request draw (first draw of tile j) + t; at table
  // entries the first tile starts x mod 1024 draws before the request
  const uint32_t head = tab ? (uint32_t)(R.x & (kTab64Stride - 1)) : 0u;
  // messages are carried as x = n - m (the encryption takes the sign back)
  uint64_t x_t = n - dev::uniform_u64(dev::const_load(A.t64.m + R.g1 + j_begin));
  uint64_t s_t = dev::uniform_u64(dev::const_load(A.t64.s + R.g1 + j_begin));
  uint64_t *const T = L + kRow64;  // the tile's rows; the row before holds the last 16 messages of the tile before
  const Enc64 K{n, ninv, kc, e, ebits, I.den, I.rcp, I.rcp_lo};
  // draw 0 of tile j is output element base + 1024 j, so the shift that
  // aligns its rows is the same for all tiles of the request.  Uniforms alone
  // (8 bytes for some 110 VALU cycles) are far from the store rate, and the
  // one more row that a shifted chunk takes is not won back: 283 against
  // 286 us for 200 streams x 300,007.
  const int64_t base = (int64_t)R.out_off - (int64_t)head;
  const uint32_t shift = A.out_c64 ? (uint32_t)base & (kAlign64 - 1) : 0u;
  const int t0 = (int)lane - (int)shift;
  const uint64_t *src = T + (t0 >> 4) * kRow64 + (t0 & 15);
  uint32_t u_lo = shift + (j_begin == 0 ? head : 0u);
  for (uint32_t j = j_begin; j < j_end; ++j) {
    // ---- pass A
    uint64_t *row = T + lane * kRow64;
    uint64_t s = dev::mulmod_p61(s_t, lane_mul);
    // eight skips below 2^61 sum below 2^64 < 4n: plain adds, one reduction per half run
    uint64_t g1 = 0, g2 = 0;
#pragma unroll 4
    for (int i = 0; i < kRun64 / 2; ++i) {
      s = dev::step_p61(s);
      row[i] = s;
      g1 += s;
    }
#pragma unroll 4
    for (int i = kRun64 / 2; i < kRun64; ++i) {
      s = dev::step_p61(s);
      row[i] = s;
      g2 += s;
    }
    const uint64_t sum = dev::addmod64(dev::mod_below_4n(g1, n), dev::mod_below_4n(g2, n), n);
    // ---- pass B
    uint64_t x = dev::submod64(x_t, dev::wave_exclusive_mod(sum, n), n);
#pragma unroll 4
    for (int i = 0; i < kRun64; ++i) {
      x = dev::submod64(x, row[i], n);
      row[i] = x;
    }
    x_t = dev::lane_u64<63>(x);
    s_t = dev::lane_u64<63>(s);
    dev::wave_lds_sync();
    // ---- pass C: a tile before another one of its chunk leaves its last
    // `shift` draws to that tile's first row
    const bool flush = j + 1 == j_end;
    uint32_t u_hi = flush ? shift + tile_len64(R, j, head) : (uint32_t)kTile64;
    if (A.split) part_of_rows(A.split, part, kTile64, &u_lo, &u_hi);
    const int64_t first = base + (int64_t)j * kTile64 - (int64_t)shift;
    const int64_t at = first + (int64_t)(u_lo & ~63u) + (int64_t)lane;
    uint64_t *cp = A.out_c64 + at;
    double *rp = A.out_r + at;
    const uint64_t *sp = src + (u_lo >> 6) * (4 * kRow64);
    with_chain(ekind, A.out_c64 != nullptr, A.out_r != nullptr, [&](auto ek, auto out) {
      constexpr int EK = decltype(ek)::value, OUT = decltype(out)::value;
      row_loop<UNROLL>(
          u_lo, u_hi, lane, [&](int k) { return sp[k * (4 * kRow64)]; },
          [&](uint64_t v) { return draw64<EK, OUT>(v, K); },
          [&](int k, const Draw<uint64_t> &d) { put_draw<OUT>(d, cp + k * 64, rp + k * 64); },
          [&](int k) {
            sp += k * (4 * kRow64);
            cp += k * 64;
            rp += k * 64;
          });
    });
    if (!flush && lane < 16) L[lane] = T[63 * kRow64 + lane];
    u_lo = u_lo > (uint32_t)kTile64 ? u_lo - (uint32_t)kTile64 : 0u;  // where the request begins in the next tile's rows
    dev::wave_lds_sync();
  }
}

// ---------------------------------------------------------------------------
// constant / unit skip (Sec. II): m at state index x is mbase + x b mod n, so
// the lanes of a row start at consecutive states and step by 64 b mod n from
// row to row; no skip generator, no prefix, no LDS.  Every tile is shifted
// back to the outputs' lines as a whole (its states follow from the index
// alone), and a request's last tile takes the draws that the shift leaves.
// ---------------------------------------------------------------------------

// Rows of tile g of a constant-skip request: the pass writes u in
// [u_lo, u_hi), and row u_lo / 64 starts at state index `state` + lane (one
// row later, `state` + 64 + lane, when that row would start before state 0).
// At the other end a row may run past the last state, 2^64 - 1: the lanes in
// use lie below it, and arithmetic modulo 2^64 gives them their indexes.
struct RowsCS {
  uint32_t u_lo, u_hi;
  uint64_t state;
  bool later;
  int64_t first;  // output element of row 0
};

__device__ __forceinline__ RowsCS rows_cs(const ReqRec &R, uint64_t g, uint32_t align, uint32_t split, uint32_t part) {
  const uint64_t x0 = g * kTileCS;
  const int64_t base = (int64_t)R.out_off + (int64_t)(x0 - R.x);  // output element of draw 0
  const uint32_t shift = (uint32_t)base & (align - 1);
  RowsCS W;
  const bool last = g + 1 == R.g1 + R.ntiles;
  // the request begins in its first tile's rows, or, when the shift moves all
  // of that tile's draws on, in those of its second
  const int64_t begin = (int64_t)(R.x - x0) + shift;
  W.u_lo = begin > 0 ? (uint32_t)begin : 0u;
  W.u_hi = last ? shift + (uint32_t)(R.x + R.count - x0) : (uint32_t)kTileCS;
  if (split) part_of_rows(split, part, kTileCS, &W.u_lo, &W.u_hi);
  const uint64_t r0 = W.u_lo & ~63u;
  W.later = g == 0 && r0 < shift;  // (x0 + r0 is 0 modulo 2^64 past the last tile, too)
  W.state = x0 + r0 + 1 - shift;
  W.first = base - (int64_t)shift;
  return W;
}

template <int UNROLL>
__device__ void run_chunk32_cs(const GenArgs &A, const InstRec &I, const ReqRec &R, uint64_t chunk, uint32_t part,
                               uint32_t lane) {
  const uint32_t n = (uint32_t)I.n, ninv = (uint32_t)I.ninv;
  const Enc32 K{n, ninv, (uint32_t)I.kcorr, I.e, (int)I.ebits, I.rcp, I.rcp_lo};
  const uint32_t bR2 = (uint32_t)I.bR2, step = (uint32_t)I.b64, mbase = (uint32_t)I.mbase;
  const uint64_t g_begin = R.g1 + chunk * A.tiles_per_chunk;
  const uint64_t g_end = min(g_begin + A.tiles_per_chunk, R.g1 + R.ntiles);
  for (uint64_t g = g_begin; g < g_end; ++g) {
    const RowsCS W = rows_cs(R, g, kAlign32, A.split, part);
    // v b mod n by Montgomery: bring hi(v) below n, then REDC(v) times b R^2
    const uint64_t v = W.state + lane + (W.later ? 64 : 0);
    uint32_t vh = (uint32_t)(v >> 32);
    vh = vh >= n ? vh - n : vh;
    const uint64_t vr = ((uint64_t)vh << 32) | (uint32_t)v;
    uint32_t x = n - dev::addmod32(mbase, dev::mont32(dev::redc32(vr, n, ninv), bR2, n, ninv), n);
    if (W.later) x = dev::addmod32(x, step, n);
    uint32_t y = x;  // message of the row last taken
    const int64_t at = W.first + (int64_t)(W.u_lo & ~63u) + (int64_t)lane;
    uint32_t *cp = A.out_c32 + at;
    double *rp = A.out_r + at;
    with_chain((int)I.ekind, A.out_c32 != nullptr, A.out_r != nullptr, [&](auto ek, auto out) {
      constexpr int EK = decltype(ek)::value, OUT = decltype(out)::value;
      row_loop<UNROLL>(
          W.u_lo, W.u_hi, lane, 
          [&](int k) {  // called in row order
            y = k == 0 ? x : dev::submod32(y, step, n);
            return y;
          },
          [&](uint32_t v) { return draw32<EK, OUT>(v, K); },
          [&](int k, const Draw<uint32_t> &d) { put_draw<OUT>(d, cp + k * 64, rp + k * 64); },
          [&](int k) {
            x = dev::submod32(k == 1 ? x : y, step, n);
            cp += k * 64;
            rp += k * 64;
          });
    });
  }
}

template <int UNROLL>
__device__ void run_chunk64_cs(const GenArgs &A, const InstRec &I, const ReqRec &R, uint64_t chunk, uint32_t part,
                               uint32_t lane) {
  const uint64_t n = I.n, ninv = I.ninv;
  const Enc64 K{n, ninv, I.kcorr, I.e, (int)I.ebits, I.den, I.rcp, I.rcp_lo};
  const uint64_t g_begin = R.g1 + chunk * A.tiles_per_chunk;
  const uint64_t g_end = min(g_begin + A.tiles_per_chunk, R.g1 + R.ntiles);
  for (uint64_t g = g_begin; g < g_end; ++g) {
    const RowsCS W = rows_cs(R, g, kAlign64, A.split, part);
    dev::W128 v;
    v.lo = W.state + lane + (W.later ? 64 : 0);  // hi word 0 < n, so REDC applies
    v.hi = 0;
    uint64_t x = n - dev::addmod64(I.mbase, dev::mont64(dev::redc64(v, n, ninv), I.bR2, n, ninv), n);
    if (W.later) x = dev::addmod64(x, I.b64, n);
    uint64_t y = x;  // message of the row last taken
    const int64_t at = W.first + (int64_t)(W.u_lo & ~63u) + (int64_t)lane;
    uint64_t *cp = A.out_c64 + at;
    double *rp = A.out_r + at;
    with_chain((int)I.ekind, A.out_c64 != nullptr, A.out_r != nullptr, [&](auto ek, auto out) {
      constexpr int EK = decltype(ek)::value, OUT = decltype(out)::value;
      row_loop<UNROLL>(
          W.u_lo, W.u_hi, lane, 
          [&](int k) {  // called in row order
            y = k == 0 ? x : dev::submod64(y, I.b64, n);
            return y;
          },
          [&](uint64_t v) { return draw64<EK, OUT>(v, K); },
          [&](int k, const Draw<uint64_t> &d) { put_draw<OUT>(d, cp + k * 64, rp + k * 64); },
          [&](int k) {
            x = dev::submod64(k == 1 ? x : y, I.b64, n);
            cp += k * 64;
            rp += k * 64;
          });
    });
  }
}

// One chunk of request r.
template <int UNROLL, bool HAS64>
__device__ __forceinline__ void run_chunk(const GenArgs &A, const ReqRec &R, uint64_t chunk, uint64_t *L,
                                          uint32_t lane) {
  const uint32_t part = (uint32_t)chunk & ((1u << A.split) - 1);
  chunk >>= A.split;
  const InstRec I = dev::const_load(A.inst + R.inst);
  if (I.sched == kSchedConstant) {
    if (HAS64 && I.width == 64) run_chunk64_cs<UNROLL>(A, I, R, chunk, part, lane);
    else run_chunk32_cs<UNROLL>(A, I, R, chunk, part, lane);
  } else if (HAS64 && I.width == 64) {
    run_chunk64<UNROLL>(A, I, R, chunk, part, L, lane);
  } else {
    run_chunk32<UNROLL>(A, I, R, chunk, part, reinterpret_cast<uint32_t *>(L), lane);
  }
}

template <int BLOCK, int UNROLL, bool HAS64>
__global__ void __launch_bounds__(BLOCK) gen_persistent(GenArgs A) {
  __shared__ uint64_t lds[BLOCK / 64][HAS64 ? kLdsWords64 : kLdsWords32];
  const uint32_t lane = dev::lane_id();
  const uint32_t wave = dev::uniform_u32(threadIdx.x / 64);  // wave-uniform: keeps chunk math scalar
  uint64_t *L = lds[wave];
  stamp_begin(A);
  const uint64_t total = A.total_chunks;
  // The blocks of group g take the chunks g, g + ngroups, g + 2 ngroups, ...:
  // chunk k of the group is chunk g + k ngroups of the batch.  The first chunk
  // of every wave is its index among the group's waves; later chunks come from
  // the group's counter, offset by the number of its waves.  Small batches
  // therefore need no atomics, and large ones avoid the start-up burst.
  // A large batch keeps one group: its chunks are long enough that one
  // counter keeps up, and it hands them out in the order of their output, which
  // writes memory 1 to 2.5% faster (2048 ragged streams, c + R: 2623 against
  // 2690 us; 4096 x 2^18 uniforms: 1615 against 1637 us).  Below kOneGroupChunks
  // chunks per wave the single counter is the bound (116 M draws of 1024
  // requests: 402 against 233 us; 200 width-64 streams x 300,007: 411 against
  // 275 us).
  const uint32_t ngroups =
      total >= (uint64_t)kOneGroupChunks * gridDim.x * (BLOCK / 64) ? 1u : min(gridDim.x, kWorkGroups);
  const uint32_t g = blockIdx.x % ngroups;
  const uint32_t nwaves = ((gridDim.x - g + ngroups - 1) / ngroups) * (BLOCK / 64);
  const uint64_t mine = total > g ? (total - g + ngroups - 1) / ngroups : 0;
  uint64_t k = (uint64_t)(blockIdx.x / ngroups) * (BLOCK / 64) + wave;
  // Every wave grabs until a grab fails, so there are mine - nwaves
  // successful grabs and one failed grab per wave: the grabs return
  // 0 .. mine - 1, and the one returning mine - 1 is the last of all.  Its
  // wave puts the counter back to zero for the next launch.  A group with no
  // more chunks than waves never touches its counter.  (One call site of
  // run_chunk: a second one gets the whole chunk code outlined into a call.)
  const bool grab = mine > nwaves;
  for (;;) {
    if (k >= mine) break;
    const GenArgs &B = args_again();
    const uint64_t c = g + k * ngroups;
    const ReqRec *const req = requests(B);
    const uint64_t r =
        B.nreq == 1 ? 0
                    : dev::uniform_u64(wave_search(B.nreq, c, lane, [&](uint64_t i) { return req[i].chunk_base; }));
    const ReqRec R = dev::const_load(req + r);
    run_chunk<UNROLL, HAS64>(B, R, c - R.chunk_base, L, lane);
    if (!grab) break;
    uint32_t next = 0;
    if (lane == 0) {
      uint32_t *const counter = &args_again().ctr->group[g].counter;
      next = atomicAdd(counter, 1u);
      if ((uint64_t)next == mine - 1) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    k = (uint64_t)nwaves + dev::uniform_u32((uint32_t)__shfl((int)next, 0, 64));
  }
  stamp_end(args_again(), blockIdx.x * (BLOCK / 64) + wave, lane);
}

// Planned requests from the kernel's arguments to device memory, a 64-bit word
// per thread and step.
struct PutArgs {
  ReqRec req[kPutReqs];
  ReqRec *dst;
  uint32_t count;  // of the requests in use
};
static_assert(sizeof(PutArgs) <= 4096, "kernel arguments stay within 4 KB");
__global__ void __launch_bounds__(256) put_requests_kernel(PutArgs P) {
  constexpr uint32_t kWords = sizeof(ReqRec) / sizeof(uint64_t);
  using WordPtr = const __attribute__((address_space(4))) uint64_t *;
  const WordPtr src = (WordPtr)((ArgPtr)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(PutArgs, req));
  uint64_t *const dst = reinterpret_cast<uint64_t *>(P.dst);
  for (uint32_t i = threadIdx.x; i < P.count * kWords; i += 256) dst[i] = src[i];
}

// One grid per request: block b (one wave) takes chunk b of request `r`.
template <int UNROLL, bool HAS64>
__global__ void __launch_bounds__(64) gen_plain(GenArgs A, uint64_t r) {
  __shared__ uint64_t lds[HAS64 ? kLdsWords64 : kLdsWords32];
  const uint32_t lane = dev::lane_id();
  const ReqRec R = dev::const_load(requests(A) + r);
  if ((uint64_t)blockIdx.x >= R.nchunks) return;
  run_chunk<UNROLL, HAS64>(A, R, blockIdx.x, lds, lane);
}

// ---------------------------------------------------------------------------
// fixed scratch of the allocation-free entry point
// ---------------------------------------------------------------------------

// One copy per device, held until the process ends.  Host code never passes
// this name to a kernel: it takes the device address once per device
// (scratch_address) and uses that.
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

__global__ void __launch_bounds__(64) clear_words(uint32_t *p, uint32_t nwords) {
  for (uint32_t i = threadIdx.x; i < nwords; i += 64) p[i] = 0;
}

hipError_t scratch_address(int device, void **ptr) {
  clear_launch_error();
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices || !ptr) return hipErrorInvalidValue;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[device]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    // the work counter must start at zero; every launch leaves it so
    hipLaunchKernelGGL(clear_words, dim3(1), dim3(64), 0, nullptr, static_cast<uint32_t *>(p),
                       (uint32_t)(kScratchClearBytes / 4));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipDeviceSynchronize()) != hipSuccess) return e;
    addr[device] = p;
  }
  *ptr = addr[device];
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------

hipError_t launch_table_segments32(uint64_t nseg, uint64_t *seg_sum, uint32_t *seg_start, hipStream_t st) {
  clear_launch_error();
  unsigned blocks = (unsigned)((nseg + 255) / 256);
  hipLaunchKernelGGL(table_segments32, dim3(blocks), dim3(256), 0, st, nseg, seg_sum, seg_start);
  return hipGetLastError();
}

hipError_t launch_table_segments64(uint64_t nseg, uint64_t *seg_lo, uint64_t *seg_hi, uint64_t *seg_start,
                                   hipStream_t st) {
  clear_launch_error();
  unsigned blocks = (unsigned)((nseg + 255) / 256);
  hipLaunchKernelGGL(table_segments64, dim3(blocks), dim3(256), 0, st, nseg, seg_lo, seg_hi, seg_start);
  return hipGetLastError();
}

hipError_t launch_seed_prime_flags(uint64_t seed, uint64_t j0, uint64_t count, int width, uint8_t *flags,
                                   hipStream_t st) {
  clear_launch_error();
  unsigned blocks = (unsigned)((count + 255) / 256);
  hipLaunchKernelGGL(seed_prime_flags, dim3(blocks), dim3(256), 0, st, seed, j0, count, width, flags);
  return hipGetLastError();
}

hipError_t launch_build_records(const uint64_t *n, const uint64_t *e, uint64_t count, int width, InstRec *out,
                                hipStream_t st) {
  clear_launch_error();
  unsigned blocks = (unsigned)((count + 255) / 256);
  hipLaunchKernelGGL(build_records, dim3(blocks), dim3(256), 0, st, n, e, count, width, out);
  return hipGetLastError();
}

hipError_t launch_position64(const InstRec *inst, const uint32_t *ids, const uint64_t *m0, const uint64_t *ta,
                             const uint64_t *tb, uint64_t count, const uint64_t *u_lo, const uint64_t *u_hi,
                             const uint64_t *u_s, uint64_t *m64, hipStream_t st) {
  clear_launch_error();
  if (count == 0) return hipSuccess;
  unsigned blocks = (unsigned)((count + 255) / 256);
  hipLaunchKernelGGL(position64_kernel, dim3(blocks), dim3(256), 0, st, inst, ids, m0, ta, tb, count, u_lo, u_hi, u_s,
                     m64);
  return hipGetLastError();
}

hipError_t launch_tiles64_reduce(const GenArgs &A, uint64_t units64, unsigned max_blocks, hipStream_t st,
                                 LaunchEvents ev) {
  clear_launch_error();
  if (units64 == 0) return hipErrorInvalidValue;
  const uint64_t want = (units64 + 3) / 4;
  const unsigned blocks = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(want, max_blocks));
  return launch_with(ev, reduce64_kernel, blocks, 256, st, A);
}

hipError_t launch_tiles64_table(const GenArgs &A, uint64_t nreq64, hipStream_t st, LaunchEvents ev) {
  clear_launch_error();
  if (nreq64 == 0 || nreq64 > 0x7fffffffull) return hipErrorInvalidValue;
  return launch_with(ev, tab64_kernel, (unsigned)nreq64, 64, st, A);
}

hipError_t launch_tiles64_scan(const GenArgs &A, uint64_t nreq64, hipStream_t st, LaunchEvents ev) {
  clear_launch_error();
  if (nreq64 == 0 || nreq64 > 0x7fffffffull) return hipErrorInvalidValue;
  return launch_with(ev, scan64_kernel, (unsigned)nreq64, kScanThreads, st, A);
}

hipError_t launch_skip_total64(uint64_t t, uint64_t count, uint64_t n, const LaneMul *lm, uint64_t *partial,
                               unsigned blocks, uint64_t extra, int sign, uint64_t *m, hipStream_t st) {
  clear_launch_error();
  if (blocks == 0) return hipErrorInvalidValue;
  if (count > 0) {
    hipLaunchKernelGGL(skip_total64_kernel, dim3(blocks), dim3(256), 0, st, t, count, n, lm, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(skip_total64_apply, dim3(1), dim3(64), 0, st, partial, count > 0 ? (uint64_t)blocks * 4 : 0, n,
                     extra, sign, m);
  return hipGetLastError();
}

template <int BLOCK, bool HAS64>
static hipError_t launch_pu(const GenArgs &A, unsigned grid, int unroll, hipStream_t st, LaunchEvents ev) {
  switch (unroll) {
    case 1: return launch_with(ev, gen_persistent<BLOCK, 1, HAS64>, grid, BLOCK, st, A);
    case 2: return launch_with(ev, gen_persistent<BLOCK, 2, HAS64>, grid, BLOCK, st, A);
    case 4: return launch_with(ev, gen_persistent<BLOCK, 4, HAS64>, grid, BLOCK, st, A);
    default: return hipErrorInvalidValue;
  }
}

template <bool HAS64>
static hipError_t launch_pb(const GenArgs &A, unsigned grid, int block, int unroll, hipStream_t st, LaunchEvents ev) {
  switch (block) {
    case 64: return launch_pu<64, HAS64>(A, grid, unroll, st, ev);
    case 128: return launch_pu<128, HAS64>(A, grid, unroll, st, ev);
    case 256: return launch_pu<256, HAS64>(A, grid, unroll, st, ev);
    case 512: return launch_pu<512, HAS64>(A, grid, unroll, st, ev);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_persistent(const GenArgs &A, unsigned grid, int block, int unroll, bool has64, hipStream_t st,
                             LaunchEvents ev) {
  clear_launch_error();
  return has64 ? launch_pb<true>(A, grid, block, unroll, st, ev) : launch_pb<false>(A, grid, block, unroll, st, ev);
}

hipError_t launch_put_requests(const ReqRec *reqs, uint64_t count, ReqRec *dst, hipStream_t st) {
  clear_launch_error();
  PutArgs P;
  memset(&P, 0, sizeof P);
  for (uint64_t i = 0; i < count; i += kPutReqs) {
    P.count = (uint32_t)std::min<uint64_t>(count - i, kPutReqs);
    P.dst = dst + i;
    memcpy(P.req, reqs + i, P.count * sizeof(ReqRec));
    const hipError_t e = launch_with({}, put_requests_kernel, dim3(1), dim3(256), st, P);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool HAS64>
static hipError_t launch_plain_u(const GenArgs &A, uint64_t r, unsigned grid, int unroll, hipStream_t st,
                                 LaunchEvents ev) {
  switch (unroll) {
    case 4: return launch_with(ev, gen_plain<4, HAS64>, grid, 64, st, A, r);
    case 2: return launch_with(ev, gen_plain<2, HAS64>, grid, 64, st, A, r);
    default: return launch_with(ev, gen_plain<1, HAS64>, grid, 64, st, A, r);
  }
}

hipError_t launch_plain(const GenArgs &A, uint64_t r, unsigned grid, int unroll, bool has64, hipStream_t st,
                        LaunchEvents ev) {
  clear_launch_error();
  if (grid == 0) return hipErrorInvalidValue;
  return has64 ? launch_plain_u<true>(A, r, grid, unroll, st, ev) : launch_plain_u<false>(A, r, grid, unroll, st, ev);
}

}  // namespace phprng
