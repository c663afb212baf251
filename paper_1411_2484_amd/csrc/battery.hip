// gfx950 kernels of the statistical battery (the chi-square tests of the
// paper's Tests section): histograms of the frequency, serial, poker,
// collision, runs and Fourier tests over blocks of 2^20 uniforms, the
// chi-square reduction, and the interstream interleave.
#include "battery.hpp"

#include <algorithm>

#include "arith.hpp"
#include "wavefft.hpp"

namespace phprng {
namespace bat {

namespace {

// Bin of a uniform among B equal bins, clamped so that R = 1.0 (possible for
// 64-bit moduli) falls in the last one.  (The conversion truncates, and the
// product is not negative.)
__device__ __forceinline__ uint32_t bin_of(double x, uint32_t b) {
  const uint32_t u = (uint32_t)(x * (double)b);
  return u < b ? u : b - 1;
}

// Poker hand category from the number of equal pairs among the five digits:
// 0 all different, 1 one pair, 2 two pairs, 3 three of a kind, 4 full house,
// 6 four of a kind, 10 five of a kind.
__device__ __forceinline__ uint32_t poker_cat(const uint32_t d[5]) {
  uint32_t pairs = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int k = i + 1; k < 5; ++k) pairs += d[i] == d[k];
  return pairs <= 4 ? pairs : (pairs == 6 ? 5u : 6u);
}

// Registers per thread for the keys of one tile: 8 + 4 + 3 + 2 + 2.
constexpr int kT = (int)kHistThreads;
constexpr int key_slots(int d) { return ((int)kHistTile / d + kT - 1) / kT; }
constexpr int key_base(int d) { return d == 1 ? 0 : key_base(d - 1) + key_slots(d - 1); }
constexpr int kKeys = key_base(6);
// the test (tuple size) of a key slot, and its first item; plain expressions
// of constants, which fold wherever the slot is one
constexpr int kB2 = key_base(2), kB3 = key_base(3), kB4 = key_base(4), kB5 = key_base(5);
__device__ __forceinline__ uint32_t key_test(int slot) {
  return 1u + (slot >= kB2) + (slot >= kB3) + (slot >= kB4) + (slot >= kB5);
}
__device__ __forceinline__ uint32_t key_first(int slot) {
  return (uint32_t)(slot - (slot >= kB5 ? kB5 : slot >= kB4 ? kB4 : slot >= kB3 ? kB3 : slot >= kB2 ? kB2 : 0)) *
         kHistThreads;
}

// Whether a thread has a key in a slot: FULL (a whole tile of kHistTile
// uniforms) by the wave's first thread `wbase` alone, since every test has a
// multiple of 64 tuples.
template <bool FULL>
__device__ __forceinline__ bool has_key(int slot, uint32_t len, uint32_t wbase) {
  const uint32_t d = key_test(slot), first = key_first(slot);
  if constexpr (FULL) {
    static_assert(kHistTile % (64 * 60) == 0, "whole waves of tuples of every size");
    return first + kHistThreads <= kHistTile / d || first + wbase < kHistTile / d;
  } else {
    return first + threadIdx.x < len / d;
  }
}

// Keys of one test for one tile, held in registers for the partitioned
// histogram: item j = threadIdx.x + it * kHistThreads is the j-th D-tuple of
// the tile (D = 1: the j-th uniform), its key the partition-space offset of
// the test plus its cell (first element most significant).  The cells come
// from each uniform's bins, found once per uniform: b20 among 2^20 bins, whose
// top 10, 5 and 4 bits are the bins among 1024, 32 and 16 (x 2^k is exact, so
// floor(x 2^k) = floor(x 2^20) >> (20 - k)), and b100 among 100, in the low
// byte of dec (b10, among 10, is the high byte).
template <int D, bool FULL>
__device__ __forceinline__ void tuple_keys(const uint32_t *b20, const uint8_t *dec, uint32_t len, uint32_t wbase,
                                           uint32_t key0, uint32_t *key) {
  static_assert(kFreqBins == 1u << 20 && kAxis2 == 1024 && kAxis3 == 100 && kAxis4 == 32 && kAxis5 == 16,
                "bins derived from the 2^20 bin");
  constexpr int kSlots = key_slots(D), kBase = key_base(D);
#pragma unroll
  for (int it = 0; it < kSlots; ++it) {
    const uint32_t j = threadIdx.x + it * kHistThreads;
    uint32_t cell = 0;
    if (has_key<FULL>(kBase + it, len, wbase)) {
      if constexpr (D == 1) {
        cell = b20[j];
      } else if constexpr (D == 3) {
        cell = (dec[6 * j] * 100u + dec[6 * j + 2]) * 100u + dec[6 * j + 4];
      } else {
        constexpr int kShift = D == 2 ? 10 : (D == 4 ? 15 : 16), kBits = 20 - kShift;
#pragma unroll
        for (int i = 0; i < D; ++i) cell = (cell << kBits) | (b20[j * D + i] >> kShift);
      }
    }
    key[kBase + it] = key0 + cell;
  }
}

// One tile of one block: frequency and serial D = 2..5 keys into the
// partitioned histograms, the poker histogram, and the bits R > 1/2 packed
// one 64-bit word per 64 uniforms (for the runs test).
struct HistShared {
  // the tile's bins (b20 among 2^20; 16 bits with b100 among 100 and b10 among
  // 10, the poker digits), later reused as the key staging area of the scatter
  uint32_t buf[kKeys * kHistThreads];
  uint32_t poker[kPokerCats];
  uint32_t cnt[kMaxParts], poff[kMaxParts], base[kMaxParts];
};
static_assert(kKeys * kHistThreads * 4 >= kHistTile * 6, "staging area must hold the tile's bins");

template <bool FULL>
__device__ __forceinline__ void hist_tile(const double *__restrict__ r, const ph::PartSet &P, const BatteryParts &bp,
                                          unsigned long long *poker_hist, uint64_t *__restrict__ bits,
                                          uint64_t base_i, uint32_t len, HistShared &S) {
  uint32_t *b20 = S.buf;
  uint16_t *dec = reinterpret_cast<uint16_t *>(S.buf + kHistTile);
  const uint8_t *dec8 = reinterpret_cast<const uint8_t *>(dec);
  if (threadIdx.x < kPokerCats) S.poker[threadIdx.x] = 0;
  // all of the thread's loads in flight at once (a loop that waits for each
  // load before the next pays the memory latency every step), then the LDS
  // copy and the run bits; len is a multiple of 64, so the bounds test is
  // uniform over a wave and every wave covers 64 consecutive uniforms per step
  constexpr uint32_t kPer = (kHistTile + kHistThreads - 1) / kHistThreads;
  static_assert(kHistTile % 64 == 0 && (kBlock % kHistTile) % 64 == 0, "whole wave steps");
  const uint32_t lane = threadIdx.x & 63, wbase = dev::uniform_u32(threadIdx.x - lane);
  double x[kPer];
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k)
    x[k] = wbase + kHistThreads * k < len ? r[base_i + threadIdx.x + kHistThreads * k] : 0.0;
  // the wave's k-th run-bit word is kept by lane k and all are stored at the
  // end with one instruction: a store inside the loop would make every later
  // step wait for it
  uint32_t mine_lo = 0, mine_hi = 0;
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    const uint32_t i = threadIdx.x + kHistThreads * k;
    if (wbase + kHistThreads * k < len) {
      b20[i] = bin_of(x[k], kFreqBins);
      dec[i] = (uint16_t)(bin_of(x[k], kAxis3) | bin_of(x[k], 10) << 8);
      const uint64_t word = __ballot(x[k] > 0.5);
      mine_lo = lane == k ? (uint32_t)word : mine_lo;
      mine_hi = lane == k ? (uint32_t)(word >> 32) : mine_hi;
    }
  }
  if (lane < kPer && wbase + kHistThreads * lane < len)
    bits[(base_i + wbase + kHistThreads * lane) >> 6] = (uint64_t)mine_hi << 32 | mine_lo;
  __syncthreads();
  // poker: a wave counts its hands per category with ballots and adds each
  // count once (an LDS atomic per hand queued on the seven addresses)
  const uint32_t nhand = len / 5;
  uint32_t wcount[kPokerCats];
#pragma unroll
  for (uint32_t c = 0; c < kPokerCats; ++c) wcount[c] = 0;
  for (uint32_t j0 = wbase; j0 < nhand; j0 += kHistThreads) {  // wave-uniform bound
    const uint32_t j = j0 + lane;
    uint32_t cat = kPokerCats;  // lanes past the last hand count nowhere
    if (FULL || j < nhand) {
      uint32_t d[5];
#pragma unroll
      for (int i = 0; i < 5; ++i) d[i] = dec8[10 * j + 2 * i + 1];
      cat = poker_cat(d);
    }
#pragma unroll
    for (uint32_t c = 0; c < kPokerCats; ++c) wcount[c] += (uint32_t)__popcll(__ballot(cat == c));
  }
  if (lane < kPokerCats) {
    uint32_t v = 0;
#pragma unroll
    for (uint32_t c = 0; c < kPokerCats; ++c) v = lane == c ? wcount[c] : v;
    if (v) atomicAdd(&S.poker[lane], v);
  }
  // all five tests' keys of the tile in registers, then one scatter over the
  // partition space (its first barrier orders the last reads of the tile
  // before the staging area is overwritten)
  uint32_t key[kKeys];
  tuple_keys<1, FULL>(b20, dec8, len, wbase, bp.p0[0] << ph::kPartBits, key);
  tuple_keys<2, FULL>(b20, dec8, len, wbase, bp.p0[1] << ph::kPartBits, key);
  tuple_keys<3, FULL>(b20, dec8, len, wbase, bp.p0[2] << ph::kPartBits, key);
  tuple_keys<4, FULL>(b20, dec8, len, wbase, bp.p0[3] << ph::kPartBits, key);
  tuple_keys<5, FULL>(b20, dec8, len, wbase, bp.p0[4] << ph::kPartBits, key);
  ph::scatter_staged<kHistThreads, kKeys>(key, P, 0, P.npart, S.cnt, S.poff, S.base, S.buf,
                                          [&](int slot) { return has_key<FULL>(slot, len, wbase); });
  if (threadIdx.x < kPokerCats && S.poker[threadIdx.x])
    atomicAdd(&poker_hist[(blockIdx.x % kRep) * kPokerCats + threadIdx.x], (unsigned long long)S.poker[threadIdx.x]);
}

// The last tile of a block (4096 of its 2^20 uniforms) tests every key; the
// 136 whole ones before it know theirs by the wave.  2^26 uniforms: 238 us (79
// vector instructions per uniform, and about half of the LDS turns), against
// 266 with a test per key in every tile (99).
__global__ __launch_bounds__(kHistThreads, 8) void hist_kernel(const double *__restrict__ r, ph::PartSet P,
                                                               BatteryParts bp, unsigned long long *poker_hist,
                                                               uint64_t *__restrict__ bits) {
  __shared__ __align__(16) HistShared S;
  const uint32_t tile = blockIdx.x % kHistTilesPerBlock;
  const uint64_t base_i = (uint64_t)(blockIdx.x / kHistTilesPerBlock) * kBlock + tile * kHistTile;
  if (tile + 1 < kHistTilesPerBlock)
    hist_tile<true>(r, P, bp, poker_hist, bits, base_i, kHistTile, S);
  else
    hist_tile<false>(r, P, bp, poker_hist, bits, base_i, kBlock - tile * kHistTile, S);
}

// Sum of v over the wave, in lane 63 (all lanes active).
__device__ __forceinline__ uint32_t wave_total(uint32_t v) {
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

constexpr uint32_t kCollGroups = 256;  // one per compute unit

// Collision trials: 2^14 uniforms into 2^20 urns held as a 128 KB bitmap in
// LDS; a ball that finds its bit already set is a collision (their number does
// not depend on the order).  The bitmap leaves room for one workgroup per
// compute unit, so a workgroup goes from trial to trial and has the next
// trial's loads in flight while it works on the one before (2^26 uniforms:
// 105 us, 5.1 TB/s; a workgroup per trial waited for its loads, 117 us).
__global__ __launch_bounds__(1024) void collision_kernel(const double *__restrict__ r, uint32_t trials,
                                                         unsigned long long *hist) {
  __shared__ __align__(16) uint32_t bm[kCollUrns / 32];
  __shared__ uint32_t total;
  constexpr uint32_t kPer = kCollBalls / 1024 / 2;
  double2 x[kPer];
  const double2 *src = reinterpret_cast<const double2 *>(r) + (uint64_t)blockIdx.x * (kCollBalls / 2);
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) x[k] = src[threadIdx.x + 1024 * k];
  for (uint32_t trial = blockIdx.x; trial < trials; trial += gridDim.x) {
    for (uint32_t i = threadIdx.x; i < kCollUrns / 128; i += 1024) reinterpret_cast<uint4 *>(bm)[i] = make_uint4(0, 0, 0, 0);
    if (threadIdx.x == 0) total = 0;
    uint32_t urn[2 * kPer];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      urn[2 * k] = bin_of(x[k].x, kCollUrns);
      urn[2 * k + 1] = bin_of(x[k].y, kCollUrns);
    }
    if (trial + gridDim.x < trials) {
      src += (uint64_t)gridDim.x * (kCollBalls / 2);
#pragma unroll
      for (uint32_t k = 0; k < kPer; ++k) x[k] = src[threadIdx.x + 1024 * k];
    }
    __syncthreads();
    uint32_t coll = 0;
#pragma unroll
    for (uint32_t k = 0; k < 2 * kPer; ++k) {
      const uint32_t bit = 1u << (urn[k] & 31);
      const uint32_t old = atomicOr(&bm[urn[k] >> 5], bit);
      coll += (old & bit) ? 1u : 0u;
    }
    coll = wave_total(coll);
    if ((threadIdx.x & 63) == 63) atomicAdd(&total, coll);
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint32_t c = total < kCollLo ? kCollLo : (total > kCollHi ? kCollHi : total);
      atomicAdd(&hist[(trial % kRep) * kCollCats + (c - kCollLo)], 1ull);
    }
    __syncthreads();  // the total is read before it is cleared
  }
}

// Interior runs: kRunsWords 64-bit words of run bits per thread, 256 words
// apart.  Position i of the block changes when its bit differs from the one
// before; a run starts at a change and ends at the next one, so the starts
// whose next L positions do not change are t & ~(ch >> 1) & ... & ~(ch >> L),
// counted with two population counts per L for all 64 positions at once
// (measuring run by run took 65 us per 2^26 uniforms, this 13).  The block's
// first position never changes, and its last change starts a run that the
// block's end cuts: neither is counted.
constexpr uint32_t kRunsWords = 4;
__global__ __launch_bounds__(256) void runs_kernel(const uint64_t *__restrict__ bits, unsigned long long *hist) {
  static_assert(kRunsMax < 32, "the look-ahead is the low half of the next word's changes");
  static_assert(kWordsPerBlock % (256 * kRunsWords) == 0, "a workgroup's words lie in one block");
  __shared__ uint32_t h[kRunsCats];
  if (threadIdx.x < kRunsCats) h[threadIdx.x] = 0;
  __syncthreads();
  uint64_t word[kRunsWords], next[kRunsWords];
  uint32_t prev[kRunsWords], wi[kRunsWords];
  const uint64_t w0 = (uint64_t)blockIdx.x * (256 * kRunsWords) + threadIdx.x;
#pragma unroll
  for (uint32_t k = 0; k < kRunsWords; ++k) {
    const uint64_t w = w0 + 256 * k;
    wi[k] = (uint32_t)(w & (kWordsPerBlock - 1));
    word[k] = bits[w];
    prev[k] = wi[k] ? (uint32_t)(bits[w - 1] >> 63) : (uint32_t)word[k] & 1;
    next[k] = wi[k] + 1 < kWordsPerBlock ? bits[w + 1] : 0;
  }
  uint32_t cnt[kRunsMax + 1] = {};  // cnt[L]: starts whose next L positions do not change
#pragma unroll
  for (uint32_t k = 0; k < kRunsWords; ++k) {
    uint64_t ch = word[k] ^ ((word[k] << 1) | prev[k]);
    uint64_t ahead = wi[k] + 1 < kWordsPerBlock ? next[k] ^ ((next[k] << 1) | (word[k] >> 63)) : 0;
    uint64_t t = ch;
    if (ch && !ahead) {
      // no change in the next word: is there any later one in the block?
      bool later = false;
      uint64_t pw = next[k];
      for (uint32_t wj = wi[k] + 2; wj < kWordsPerBlock && !later; ++wj) {
        const uint64_t nw = bits[w0 + 256 * k + (wj - wi[k])];
        later = (nw ^ ((nw << 1) | (pw >> 63))) != 0;
        pw = nw;
      }
      if (!later) t &= ~(1ull << (63 - __builtin_clzll(ch)));
    }
    uint32_t look = (uint32_t)ahead;
    cnt[0] += (uint32_t)__popcll(t);
#pragma unroll
    for (uint32_t L = 1; L <= kRunsMax; ++L) {
      ch = (ch >> 1) | ((uint64_t)look << 63);
      look >>= 1;
      t &= ~ch;
      cnt[L] += (uint32_t)__popcll(t);
    }
  }
#pragma unroll
  for (uint32_t L = 0; L <= kRunsMax; ++L) {
    const uint32_t tot = wave_total(cnt[L]);
    // cnt[L - 1] - cnt[L] runs have length L; the last category holds the rest
    if ((threadIdx.x & 63) == 63 && tot) {
      atomicAdd(&h[L], tot);
      if (L > 0) atomicSub(&h[L - 1], tot);
    }
  }
  __syncthreads();
  if (threadIdx.x < kRunsCats && h[threadIdx.x])
    atomicAdd(&hist[(blockIdx.x % kRep) * kRunsCats + threadIdx.x], (unsigned long long)h[threadIdx.x]);
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Pass-1 LDS layout: column c of a workgroup's 8 columns at c * kP1Stride
// (double2); 529 = 16 * 33 + 1 holds the column and then, in place, the
// wave transform's transpose, and spreads the columns over the banks.
constexpr int kP1Stride = 529;

// Pass 1 of the four-step transform of z_n = (x_2n - 1/2) + i (x_2n+1 - 1/2),
// n = 1024 j1 + j2: the 512-point transforms over j1 of kFftCols columns j2
// (two per wave, one per half-wave), times exp(2 pi i j2 k1 / 2^19), written
// as rows Y[k1][j2].
__global__ __launch_bounds__(256) void fft_pass1_kernel(const double *__restrict__ r, double2 *__restrict__ y,
                                                        Twiddles tw) {
  __shared__ double2 st[kFftCols * kP1Stride];
  const uint64_t blk = blockIdx.x / kFftPass1Groups;
  const uint32_t c0 = (blockIdx.x % kFftPass1Groups) * kFftCols;
  const double2 *src = reinterpret_cast<const double2 *>(r + blk * kBlock);
  // the thread's 16 loads in flight at once, then into the columns
  constexpr uint32_t kPer = kFftCols * kFftN1 / 256;
  double2 in[kPer];
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    const uint32_t e = threadIdx.x + 256 * k, j1 = e / kFftCols, col = e % kFftCols;
    in[k] = src[(uint64_t)j1 * kFftN2 + c0 + col];
  }
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    const uint32_t e = threadIdx.x + 256 * k, j1 = e / kFftCols, col = e % kFftCols;
    st[col * kP1Stride + j1] = make_double2(in[k].x - 0.5, in[k].y - 0.5);
  }
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63, l = lane & 31;
  const uint32_t col = 2 * (threadIdx.x >> 6) + (lane >> 5);
  double2 *cs = st + col * kP1Stride;
  double2 v[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m] = cs[l + 32 * m];
  wf::wave_fft<32>(v, cs, tw.w1024, l);
  // v[kb] = F[k1], k1 = k_a + 16 kb + 256 q; times the twiddle, back to the
  // column in frequency order
  const uint32_t ka = l >> 1, q = wf::wave_fft_q<32>(l);
  const uint32_t j2 = c0 + col;
  dev::wave_lds_sync();
  // w_N^{j2 k1} = w_N^{j2 (ka + 256 q)} (w_N^{16 j2})^kb: two roots loaded, then products
  const uint32_t t0 = j2 * (ka + 256 * q), t1 = 16 * j2;  // < 2^19
  double2 wt = cmul(tw.fineN[t0 & 1023], tw.w1024[2 * (t0 >> 10)]);
  const double2 ws = cmul(tw.fineN[t1 & 1023], tw.w1024[2 * (t1 >> 10)]);
#pragma unroll
  for (int kb = 0; kb < 16; ++kb) {
    cs[ka + 16 * kb + 256 * q] = cmul(v[kb], wt);
    wt = cmul(wt, ws);
  }
  __syncthreads();
  double2 *dst = y + blk * (uint64_t)kFftN;
  for (uint32_t e = threadIdx.x; e < kFftCols * kFftN1; e += 256) {
    const uint32_t k1 = e / kFftCols, c = e % kFftCols;
    dst[(uint64_t)k1 * kFftN2 + c0 + c] = st[c * kP1Stride + k1];
  }
}

// Category of a coefficient's part, less kFourierHalf + 1 (a value that is not
// a number falls in the first).
__device__ __forceinline__ int fourier_bin(double v, double scale) {
  const int u = (int)fmax(floor(v * scale), (double)(-kFourierHalf - 1));
  return min(u, kFourierHalf);
}

// Pass 2: the 1024-point transforms of rows k1 and 512 - k1 (rows 0 and 256
// pair with themselves), one wave per row, which give F_k for
// k = k1 + 512 k2 and the partner N - k of each; then the real-input split
//   E = (F_k + conj F_{N-k}) / 2,  O = (F_k - conj F_{N-k}) / (2i),
//   X_k = E + w_M^k O,  X_{N-k} = conj(E - w_M^k O),
// scaled by 1/sqrt(M), and the categories of their real and imaginary parts.
// split_and_bin takes A = F_k, B = F_{N-k} and wk = w_M^k.  The categories are
// counted in kFourierRep copies, lane by lane: a third of the coefficients
// fall in eight categories, and lanes that count in one of them queue.
constexpr int kFourierRep = 4;
__device__ __forceinline__ void add_fourier(unsigned long long *hist, const uint32_t *h) {
  if (threadIdx.x >= kFourierCats) return;
  uint32_t v = 0;
#pragma unroll
  for (int k = 0; k < kFourierRep; ++k) v += h[threadIdx.x * kFourierRep + k];
  if (v) atomicAdd(&hist[(blockIdx.x % kRep) * kFourierCats + threadIdx.x], (unsigned long long)v);
}
__device__ __forceinline__ void split_and_bin(double2 A, double2 B, double2 wk, uint32_t k, double scale,
                                              uint32_t *h, double *cb) {
  h += (kFourierHalf + 1) * kFourierRep + (threadIdx.x & (kFourierRep - 1));
  const double fs = 1.0 / 1024.0;  // 1 / sqrt(M), exact
  const double ar = A.x, ai = A.y, br = B.x, bi = B.y;
  const double er = (ar + br) * 0.5, ei = (ai - bi) * 0.5;
  const double orr = (ai + bi) * 0.5, oi = (br - ar) * 0.5;
  const double tr = orr * wk.x - oi * wk.y, ti = orr * wk.y + oi * wk.x;
  const double xr = (er + tr) * fs, xi = (ei + ti) * fs;
  atomicAdd(&h[fourier_bin(xr, scale) * kFourierRep], 1u);
  atomicAdd(&h[fourier_bin(xi, scale) * kFourierRep], 1u);
  if (cb) {
    cb[2 * k] = xr;
    cb[2 * k + 1] = xi;
  }
  const uint32_t kp = (kFftN - k) % kFftN;
  if (kp != k) {  // the partner coefficient, unless it is the same one (k = 0 or N/2)
    const double pr = (er - tr) * fs, pi = -(ei - ti) * fs;
    atomicAdd(&h[fourier_bin(pr, scale) * kFourierRep], 1u);
    atomicAdd(&h[fourier_bin(pi, scale) * kFourierRep], 1u);
    if (cb) {
      cb[2 * kp] = pr;
      cb[2 * kp + 1] = pi;
    }
  }
}

// Row pairs (k1, 512 - k1) with 1 <= k1 <= 255.  Each wave transforms its row
// with the split transpose (half the LDS of a complex one, so more
// workgroups fit on a CU), then the two waves swap half of their
// coefficients through the same areas.  Lane t holds F[c], c = ka + 16 kb +
// 256 q (ka = t / 4, q its output index); the mirror index 1023 - c of the
// other row sits in lane 63 - t of the other wave, register 15 - kb.  Wave 0
// (row k1) takes the pairs whose row-k1 index has kb < 8, wave 1 the pairs
// whose row-(512 - k1) index has kb < 8: every pair once.
constexpr int kP2Half = 16 * 65;  // doubles per wave
constexpr uint32_t kP2PairRows = kFftN1 / 2 - 1;
__global__ __launch_bounds__(128) void fft_pass2_pairs_kernel(const double2 *__restrict__ y, unsigned long long *hist,
                                                              double *__restrict__ coef, Twiddles tw, double scale) {
  constexpr int L = kFftN2;
  __shared__ __align__(16) double buf[2 * kP2Half];
  static_assert(8 * 64 * 2 <= kP2Half && (kP2Half * 8) % 16 == 0, "swap slots fit the area");
  __shared__ uint32_t h[kFourierCats * kFourierRep];
  const uint64_t blk = blockIdx.x / kP2PairRows;
  const uint32_t ra = 1 + blockIdx.x % kP2PairRows, rb = kFftN1 - ra;
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (uint32_t i = threadIdx.x; i < kFourierCats * kFourierRep; i += 128) h[i] = 0;
  const double2 *row = y + blk * (uint64_t)kFftN + (uint64_t)(w ? rb : ra) * L;
  double *area = buf + w * kP2Half;
  double2 v[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m] = row[lane + 64 * m];
  wf::wave_fft_split<64>(v, area, tw.w1024, lane);
  // registers 8..15 to the other wave: slot j * 64 + t holds v[8 + j] of lane t
  double2 *mine = reinterpret_cast<double2 *>(area);
  wf::wave_lds_fence();
#pragma unroll
  for (int j = 0; j < 8; ++j) mine[j * 64 + lane] = v[8 + j];
  __syncthreads();
  const double2 *other = reinterpret_cast<const double2 *>(buf + (1 - w) * kP2Half);
  double *cb = coef ? coef + blk * (uint64_t)kBlock : nullptr;
  // k = ra + 512 k2: w_M^k = fineM[ra + 512 (k2 & 1)] w_1024^{k2 >> 1}, with
  // k2 >> 1 = c0 + 8 kb (wave 0) or 511 - c0 - 8 kb (wave 1): one loaded root
  // and its products with w_1024^{+-8}
  const uint32_t ka = lane >> 2, q = wf::wave_fft_q<64>(lane);
  const uint32_t c0 = (ka >> 1) + 128 * q;
  const double2 fine = tw.fineM[ra + 512 * ((ka & 1) ^ w)];
  const double2 s8 = tw.w1024[8];
  const double2 step = w ? make_double2(s8.x, -s8.y) : s8;
  double2 wc = tw.w1024[w ? 511 - c0 : c0];
#pragma unroll
  for (int kb = 0; kb < 8; ++kb) {
    const uint32_t cown = ka + 16 * kb + 256 * q;
    const uint32_t k2 = w ? 1023 - cown : cown;
    const double2 pv = other[(7 - kb) * 64 + (63 - lane)];
    // A = row ra at k2, B = row rb at 1023 - k2
    split_and_bin(w ? pv : v[kb], w ? v[kb] : pv, cmul(fine, wc), ra + kFftN1 * k2, scale, h, cb);
    wc = cmul(wc, step);
  }
  __syncthreads();
  add_fourier(hist, h);
}

// Rows 0 and 256, each paired with itself: one wave per copy of the row,
// the coefficients in frequency order in LDS (one pad slot every 256).
constexpr int kP2Area = 16 * 65;
__device__ __forceinline__ uint32_t p2_slot(uint32_t k2) { return k2 + (k2 >> 8); }

__global__ __launch_bounds__(128) void fft_pass2_self_kernel(const double2 *__restrict__ y, unsigned long long *hist,
                                                             double *__restrict__ coef, Twiddles tw, double scale) {
  constexpr int L = kFftN2;
  __shared__ double2 buf[2 * kP2Area];
  __shared__ uint32_t h[kFourierCats * kFourierRep];
  const uint64_t blk = blockIdx.x >> 1;
  const uint32_t ra = (blockIdx.x & 1) ? kFftN1 / 2 : 0u;
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (uint32_t i = threadIdx.x; i < kFourierCats * kFourierRep; i += 128) h[i] = 0;
  const double2 *row = y + blk * (uint64_t)kFftN + (uint64_t)ra * L;
  double2 *area = buf + w * kP2Area;
  double2 v[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m] = row[lane + 64 * m];
  wf::wave_fft<64>(v, area, tw.w1024, lane);
  const uint32_t ka = lane >> 2, q = wf::wave_fft_q<64>(lane);
  dev::wave_lds_sync();
#pragma unroll
  for (int kb = 0; kb < 16; ++kb) area[p2_slot(ka + 16 * kb + 256 * q)] = v[kb];
  __syncthreads();
  double *cb = coef ? coef + blk * (uint64_t)kBlock : nullptr;
  // row 0: k2 = 0..512 with partner 1024 - k2; row 256: k2 = 0..511 with
  // partner 1023 - k2 (in the second wave's copy of the row)
  const uint32_t nk2 = ra == 0 ? 513u : 512u;
  const double2 fine0 = tw.fineM[ra], fine1 = tw.fineM[ra + 512];
  for (uint32_t k2 = threadIdx.x; k2 < nk2; k2 += 128) {
    const uint32_t pa = p2_slot(k2);
    const uint32_t pb = ra == 0 ? p2_slot((1024 - k2) & 1023) : kP2Area + p2_slot(1023 - k2);
    const double2 wk = cmul((k2 & 1) ? fine1 : fine0, tw.w1024[k2 >> 1]);
    split_and_bin(buf[pa], buf[pb], wk, ra + kFftN1 * k2, scale, h, cb);
  }
  __syncthreads();
  add_fourier(hist, h);
}

// One workgroup per category of the four small histograms: dst[c] += sum of
// its kRep replicas, which are cleared, one replica per thread (a thread that
// walked the replicas of its category took 30 us per histogram).
__global__ __launch_bounds__(kRep) void fold_kernel(SmallHists S) {
  __shared__ unsigned long long part[kRep / 64];
  uint32_t c = blockIdx.x, t = 0;
  while (c >= S.ncat[t]) c -= S.ncat[t++];
  unsigned long long *const src = S.rep[t] + (uint64_t)threadIdx.x * S.ncat[t] + c;
  unsigned long long v = *src;
  *src = 0;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v += dev::shfl_xor_u64(v, d);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (uint32_t i = 1; i < kRep / 64; ++i) v += part[i];
    if (v) S.dst[t][c] += v;
  }
}

// Exact sums of the counts and of their squares over slice blockIdx.x of
// large histogram blockIdx.y (its cells are equally likely, so these two
// integers give its chi^2); the workgroups of row kPartTests copy the small
// histograms.  The results go to host memory.  64 workgroups per histogram
// read the 42 MB in parallel (one per histogram, which read it twice, took
// 671 us).
__global__ __launch_bounds__(256) void moments_kernel(MomentJobs J, Moments *out, unsigned long long *small_out) {
  if (blockIdx.y == kPartTests) {
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < J.nsmall; i += kMomentSlices * 256) small_out[i] = J.small[i];
    return;
  }
  const unsigned long long *counts = J.counts[blockIdx.y];
  const uint32_t n = J.ncat[blockIdx.y];
  const uint32_t lo = (uint32_t)((uint64_t)n * blockIdx.x / kMomentSlices);
  const uint32_t hi = (uint32_t)((uint64_t)n * (blockIdx.x + 1) / kMomentSlices);
  unsigned long long sum = 0;
  unsigned __int128 sq = 0;
  constexpr uint32_t kU = 8;  // loads in flight per thread
  for (uint32_t i0 = lo + threadIdx.x; i0 < hi; i0 += 256 * kU) {
    unsigned long long o[kU];
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) o[u] = i0 + 256 * u < hi ? counts[i0 + 256 * u] : 0;
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
      sum += o[u];
      sq += (unsigned __int128)o[u] * o[u];
    }
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    sum += dev::shfl_xor_u64(sum, d);
    const uint64_t l = dev::shfl_xor_u64((uint64_t)sq, d), h = dev::shfl_xor_u64((uint64_t)(sq >> 64), d);
    sq += ((unsigned __int128)h << 64) | l;
  }
  __shared__ Moments part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = {sum, (uint64_t)sq, (uint64_t)(sq >> 64)};
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      sum += part[w].sum;
      sq += ((unsigned __int128)part[w].sq_hi << 64) | part[w].sq_lo;
    }
    out[blockIdx.y * kMomentSlices + blockIdx.x] = {sum, (uint64_t)sq, (uint64_t)(sq >> 64)};
  }
}

// A small histogram to mapped host memory (a copy to pageable memory takes
// the host 25 us, this launch and the wait for it 12).
__global__ __launch_bounds__(256) void counts_out_kernel(const unsigned long long *src, uint32_t n,
                                                         unsigned long long *out) {
  for (uint32_t i = threadIdx.x; i < n; i += 256) out[i] = src[i];
}

// out[t * S + a] = in[a * L + t] through a 64 x 64 LDS tile.  PAIRS: S and L
// even and both arrays at 16-byte addresses, so that a whole tile moves two
// uniforms per access with all of a thread's loads in flight; the tiles at the
// ends, and any other shape, move one at a time.
template <bool PAIRS>
__global__ __launch_bounds__(256) void interleave_kernel(const double *__restrict__ in, double *__restrict__ out,
                                                         uint64_t S, uint64_t L) {
  __shared__ double tile[64][65];
  const uint64_t t0 = (uint64_t)blockIdx.x * 64, a0 = (uint64_t)blockIdx.y * 64;
  if (PAIRS && a0 + 64 <= S && t0 + 64 <= L) {
    const uint32_t p = 2 * (threadIdx.x & 31), q = threadIdx.x >> 5;
    double2 v[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const double2 *>(in + (a0 + q + 8 * k) * L + t0 + p);
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      tile[q + 8 * k][p] = v[k].x;
      tile[q + 8 * k][p + 1] = v[k].y;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)
      *reinterpret_cast<double2 *>(out + (t0 + q + 8 * k) * S + a0 + p) =
          make_double2(tile[p][q + 8 * k], tile[p + 1][q + 8 * k]);
    return;
  }
  const uint32_t x = threadIdx.x & 63, y = threadIdx.x >> 6;
  for (uint32_t j = y; j < 64; j += 4) {
    const uint64_t a = a0 + j, t = t0 + x;
    if (a < S && t < L) tile[j][x] = in[a * L + t];
  }
  __syncthreads();
  for (uint32_t j = y; j < 64; j += 4) {
    const uint64_t t = t0 + j, a = a0 + x;
    if (a < S && t < L) out[t * S + a] = tile[x][j];
  }
}

}  // namespace

hipError_t launch_hist(const double *r, uint64_t nblocks, const ph::PartSet &P, const BatteryParts &bp,
                       unsigned long long *poker, uint64_t *bits, hipStream_t st, LaunchEvents ev) {
  clear_launch_error();
  return launch_with(ev, hist_kernel, dim3((unsigned)(nblocks * kHistTilesPerBlock)), dim3(kHistThreads), st, r, P, bp,
                     poker, bits);
}

hipError_t launch_collision(const double *r, uint64_t nblocks, unsigned long long *coll, hipStream_t st,
                            LaunchEvents ev) {
  clear_launch_error();
  const uint32_t trials = (uint32_t)(nblocks * (kBlock / kCollBalls));
  return launch_with(ev, collision_kernel, dim3(std::min(trials, kCollGroups)), dim3(1024), st, r, trials, coll);
}

hipError_t launch_runs(const uint64_t *bits, uint64_t nblocks, unsigned long long *runs, hipStream_t st,
                       LaunchEvents ev) {
  clear_launch_error();
  const uint64_t nwords = nblocks * kWordsPerBlock;
  return launch_with(ev, runs_kernel, dim3((unsigned)(nwords / (256 * kRunsWords))), dim3(256), st, bits, runs);
}

hipError_t launch_fft_pass1(const double *r, uint64_t nblocks, double2 *y, Twiddles tw, hipStream_t st,
                            LaunchEvents ev) {
  clear_launch_error();
  return launch_with(ev, fft_pass1_kernel, dim3((unsigned)(nblocks * kFftPass1Groups)), dim3(256), st, r, y, tw);
}

hipError_t launch_fft_pass2(const double2 *y, uint64_t nblocks, unsigned long long *fourier, double *coef,
                            Twiddles tw, double scale, hipStream_t st, LaunchEvents ev) {
  clear_launch_error();
  const hipError_t e = launch_with({}, fft_pass2_pairs_kernel, dim3((unsigned)(nblocks * kP2PairRows)),
                                   dim3(128), st, y, fourier, coef, tw, scale);
  if (e != hipSuccess) return e;
  return launch_with(ev, fft_pass2_self_kernel, dim3((unsigned)(nblocks * 2)), dim3(128), st, y,
                     fourier, coef, tw, scale);
}

hipError_t launch_fold(const SmallHists &S, hipStream_t st) {
  clear_launch_error();
  uint32_t cats = 0;
  for (uint32_t n : S.ncat) cats += n;
  fold_kernel<<<dim3(cats), dim3(kRep), 0, st>>>(S);
  return hipGetLastError();
}

hipError_t launch_counts_out(const unsigned long long *src, uint32_t n, unsigned long long *out, hipStream_t st) {
  clear_launch_error();
  counts_out_kernel<<<dim3(1), dim3(256), 0, st>>>(src, n, out);
  return hipGetLastError();
}

hipError_t launch_moments(const MomentJobs &J, Moments *out, unsigned long long *small_out, hipStream_t st) {
  clear_launch_error();
  moments_kernel<<<dim3(kMomentSlices, kPartTests + 1), dim3(256), 0, st>>>(J, out, small_out);
  return hipGetLastError();
}

hipError_t launch_interleave(const double *in, double *out, uint64_t nstreams, uint64_t length, hipStream_t st) {
  clear_launch_error();
  const bool pairs = ((nstreams | length) & 1) == 0 &&
                     ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
  const dim3 grid((unsigned)((length + 63) / 64), (unsigned)((nstreams + 63) / 64));
  if (pairs)
    interleave_kernel<true><<<grid, dim3(256), 0, st>>>(in, out, nstreams, length);
  else
    interleave_kernel<false><<<grid, dim3(256), 0, st>>>(in, out, nstreams, length);
  return hipGetLastError();
}

}  // namespace bat
}  // namespace phprng
