// Stable counting sort of particles by cell (or tile-major cell) key: an LSD
// radix sort with as few passes as digits of up to 9 bits need.  Each pass:
// per-block digit histograms, one exclusive scan over (digit, block), and a
// scatter in which every wave ranks its own keys stably (wave ballots, LDS
// counters of its own), so that a block meets at five barriers and not at
// three per 256 keys.  Deterministic: no atomics decide an order.
//
// Blocks are dealt to the XCDs in contiguous ranges (blockIdx mod 8 picks the
// XCD): a digit's output of one block continues that of the block before, and
// with both on one XCD its L2 joins their pieces into whole lines.  Measured
// for 33.5 M keys of 24 bits, us per pass: 303 with 4096 keys a block in plain
// order, ranked in step by the whole block (as this sort began); 315 with 8192
// keys a block ranked wave by wave (2 waves per SIMD); 205 with 4096.  Digits
// of 11 bits save a pass from 19 bits on, but cost 250 us a pass for 16.7 M
// keys against 105 with 8 (the histograms and their scan grow by 8).
#include <algorithm>

#include "dust_device.h"
#include "dust_launch.h"
#include "dust_particle.h"

namespace dust {

static constexpr int BIN_THREADS = 256;
static constexpr int BIN_WAVES = BIN_THREADS / 64;
static constexpr int BIN_MAX_BITS = 9;
// Below this many keys, blocks of 1024 instead of 4096, which would leave
// CUs idle.  A sort of random tile keys, us with 1024 and 4096: 62 and 82 at
// 2^19 keys, 92 and 107 at 2^21, 142 and 124 at 2^22, 445 and 340 at 2^24.
static constexpr int64_t BIN_FEW = 3 << 20;
// Up to this many blocks, a pass without a scan: 26 and 41 us with one at 64
// blocks, 29 and 41 at 128, 50 and 58 at 256, 65 and 60 at 384.
static constexpr int64_t BIN_DIRECT = 256;

// Sort keys from the cells, KEYS_PER particles of a thread (their loads
// issue together).
static constexpr int KEYS_PER = 4;
__global__ void __launch_bounds__(BIN_THREADS)
    k_make_keys(const int32_t* __restrict__ cell, int64_t n, const Box* __restrict__ boxes, int nbox,
                uint32_t nbins, int key_mode, TileShape ts, uint32_t* __restrict__ key) {
  const int64_t i0 = (int64_t)blockIdx.x * (BIN_THREADS * KEYS_PER) + threadIdx.x;
  int32_t c[KEYS_PER];
#pragma unroll
  for (int q = 0; q < KEYS_PER; ++q) {
    const int64_t i = i0 + q * BIN_THREADS;
    c[q] = i < n ? cell[i] : -1;
  }
#pragma unroll
  for (int q = 0; q < KEYS_PER; ++q) {
    const int64_t i = i0 + q * BIN_THREADS;
    uint32_t k = nbins;
    if (c[q] >= 0 && (uint32_t)c[q] < nbins) {
      k = (uint32_t)c[q];
      if (key_mode == DUST_BIN_TILE) {
        // one box (the common case): its descriptor is uniform
        if (nbox == 1) {
          k = tile_key(boxes[0], c[q], ts);
        } else {
          const Box& B = boxes[find_box(boxes, nbox, c[q])];
          k = tile_key(B, c[q] - B.cell_base, ts);
        }
      }
    }
    if (i < n) key[i] = k;
  }
}

// The block of keys of a workgroup (see the head of the file).
__device__ __forceinline__ uint32_t bin_block(uint32_t nblocks) {
  const uint32_t xcd = blockIdx.x & 7u, per = nblocks >> 3, rem = nblocks & 7u;
  return xcd * per + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
}

// Digit histogram of every block of BIN_THREADS * ITEMS keys: hist[digit *
// nblocks + block], with DIRECT hist[block * NDIG + digit].  Only the first lane of a run of equal digits adds (keys
// that are nearly sorted would queue on one counter).
template <int NDIG, int ITEMS, bool DIRECT>
__global__ void __launch_bounds__(BIN_THREADS)
    k_digit_hist(const uint32_t* __restrict__ key, uint32_t n, int shift, int nbits, uint32_t* __restrict__ hist,
                 uint32_t nblocks) {
  __shared__ uint32_t h[NDIG];
  const int t = threadIdx.x, lane = t & 63;
  const uint32_t ndig = 1u << nbits, mask = ndig - 1;
  const uint32_t b = bin_block(nblocks);
  for (uint32_t d = t; d < (DIRECT ? NDIG : ndig); d += BIN_THREADS) h[d] = 0;
  __syncthreads();
  const uint32_t base = b * (uint32_t)(BIN_THREADS * ITEMS);
  uint32_t k[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const uint32_t l = c * BIN_THREADS + t;
    k[c] = l < n - base ? key[base + l] : 0u;
  }
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const bool valid = (uint32_t)(c * BIN_THREADS + t) < n - base;   // (valid lanes come first)
    const uint32_t d = (k[c] >> shift) & mask;
    const uint32_t prev = __shfl_up(d, 1);
    const uint64_t all = __ballot(valid);
    const uint64_t heads = __ballot(valid && (lane == 0 || d != prev));
    if ((heads >> lane) & 1u) {
      // lanes up to the next head, or the last valid one
      const uint64_t above = lane == 63 ? 0ull : heads >> (lane + 1);
      const uint32_t len = above ? (uint32_t)__ffsll((unsigned long long)above) : (uint32_t)__popcll(all) - lane;
      atomicAdd(&h[d], len);
    }
  }
  __syncthreads();
  if constexpr (DIRECT) {
    for (uint32_t d = t; d < NDIG; d += BIN_THREADS) hist[(size_t)b * NDIG + d] = h[d];
  } else {
    for (uint32_t d = t; d < ndig; d += BIN_THREADS) hist[(size_t)d * nblocks + b] = h[d];
  }
}

// One radix pass of one block: every wave ranks its 64 * ITEMS consecutive
// keys among its own (round by round of 64, ballots for lanes with equal
// digits, counters of its own for the rounds), the counters of the waves
// become places in stable digit order, the keys and then the values are put
// there in LDS and written out run by run.  offs: the scanned histogram; with
// DIRECT the histogram itself, which every block sums for its own places.
// val_in = nullptr: values are the element indices (first pass).
template <int NDIG, int ITEMS, bool DIRECT>
__global__ void __launch_bounds__(BIN_THREADS)
    k_digit_scatter(const uint32_t* __restrict__ key_in, const uint32_t* __restrict__ val_in, uint32_t n, int shift,
                    int nbits, const uint32_t* __restrict__ offs, uint32_t nblocks, uint32_t* __restrict__ key_out,
                    uint32_t* __restrict__ val_out) {
  constexpr int KEYS = BIN_THREADS * ITEMS;
  constexpr int P = NDIG / BIN_THREADS;   // digits of a thread
  static_assert(KEYS < 65536 && NDIG % BIN_THREADS == 0 && NDIG <= (1 << BIN_MAX_BITS), "16-bit places");
  __shared__ uint32_t stage[KEYS];
  __shared__ uint32_t goff[NDIG];
  __shared__ uint16_t cnt[BIN_WAVES][NDIG];
  __shared__ uint32_t wsum[BIN_WAVES];
  __shared__ __align__(16) uint32_t part[2][DIRECT ? BIN_WAVES : 1][DIRECT ? NDIG : 4];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t ndig = 1u << nbits, mask = ndig - 1;
  const uint32_t b = bin_block(nblocks), base = b * (uint32_t)KEYS;
  const int nloc = (int)(n - base < (uint32_t)KEYS ? n - base : (uint32_t)KEYS);
  const int l0 = wv * 64 * ITEMS + lane;   // this lane's first key of the block
  uint32_t k[ITEMS], v[ITEMS];
  uint16_t r[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int l = l0 + 64 * c;
    k[c] = l < nloc ? key_in[base + l] : 0u;
  }
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int l = l0 + 64 * c;
    v[c] = l < nloc ? (val_in ? val_in[base + l] : base + l) : 0u;
  }
  for (int d = t; d < BIN_WAVES * NDIG; d += BIN_THREADS) (&cnt[0][0])[d] = 0;
  // DIRECT: keys of this thread's digits in the blocks before this one (gpre)
  // and in all; then, with the keys of lower digits, the first place of each
  uint32_t gpre[P];
  if constexpr (DIRECT) {
    // a wave takes every fourth block, a lane four digits of it, U blocks
    // whose loads issue together (one block after another, a thread per
    // digit, was slower from some 100 blocks on than the scan)
    constexpr int Q = NDIG / 256, U = 16 / Q;
    const uint4* rows = reinterpret_cast<const uint4*>(offs) + lane;
    uint4 all4[Q] = {}, bef4[Q] = {};
    for (uint32_t q = wv; q < nblocks; q += BIN_WAVES * U) {
      uint4 x[U][Q];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < Q; ++j)
          x[u][j] = q + BIN_WAVES * u < nblocks ? rows[(size_t)(q + BIN_WAVES * u) * (NDIG / 4) + 64 * j]
                                                : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          const bool lower = q + BIN_WAVES * u < b;
          const uint4 y = x[u][j];
          all4[j].x += y.x, all4[j].y += y.y, all4[j].z += y.z, all4[j].w += y.w;
          bef4[j].x += lower ? y.x : 0u, bef4[j].y += lower ? y.y : 0u;
          bef4[j].z += lower ? y.z : 0u, bef4[j].w += lower ? y.w : 0u;
        }
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      reinterpret_cast<uint4*>(part[0][wv])[64 * j + lane] = all4[j];
      reinterpret_cast<uint4*>(part[1][wv])[64 * j + lane] = bef4[j];
    }
    __syncthreads();
    uint32_t before[P] = {}, all[P] = {}, sum = 0;
#pragma unroll
    for (int j = 0; j < P; ++j)
      for (int w = 0; w < BIN_WAVES; ++w) {
        all[j] += part[0][w][t * P + j];
        before[j] += part[1][w][t * P + j];
      }
#pragma unroll
    for (int j = 0; j < P; ++j) sum += all[j];
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t low = incl - sum;
    for (int w = 0; w < wv; ++w) low += wsum[w];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      gpre[j] = before[j] + low;
      low += all[j];
    }
  }
  __syncthreads();
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const bool valid = l0 + 64 * c < nloc;
    const uint32_t d = (k[c] >> shift) & mask;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bt = 0; bt < BIN_MAX_BITS; ++bt) {
      if (bt >= nbits) break;   // (uniform)
      const bool one = (d >> bt) & 1u;
      const uint64_t m = __ballot(one);
      peers &= one ? m : ~m;
    }
    const uint32_t rank = (uint32_t)__popcll(peers & lt);
    const uint32_t old = cnt[wv][d];
    if (valid && rank == 0) cnt[wv][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
    r[c] = (uint16_t)(old + rank);
  }
  __syncthreads();
  // places: exclusive scan over (digit, wave)
  uint32_t tot[P], mine = 0;
#pragma unroll
  for (int j = 0; j < P; ++j) {
    tot[j] = 0;
#pragma unroll
    for (int w = 0; w < BIN_WAVES; ++w) tot[j] += cnt[w][t * P + j];
    mine += tot[j];
  }
  uint32_t incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(incl, o);
    if (lane >= o) incl += u;
  }
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  uint32_t start = incl - mine;
  for (int w = 0; w < wv; ++w) start += wsum[w];
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const uint32_t d = (uint32_t)(t * P + j);
    // a place p of digit d goes to goff[d] + p
    if constexpr (DIRECT) goff[d] = gpre[j] - start;
    else goff[d] = (d < ndig ? offs[(size_t)d * nblocks + b] : 0u) - start;
    uint32_t q = start;
#pragma unroll
    for (int w = 0; w < BIN_WAVES; ++w) {
      const uint32_t x = cnt[w][d];
      cnt[w][d] = (uint16_t)q;
      q += x;
    }
    start += tot[j];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    r[c] = (uint16_t)(cnt[wv][(k[c] >> shift) & mask] + r[c]);
    if (l0 + 64 * c < nloc) stage[r[c]] = k[c];
  }
  __syncthreads();
  // the keys run by run; where each went, for the values
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int p = c * BIN_THREADS + t;
    const uint32_t kk = stage[p];   // (past nloc: not used)
    const uint32_t o = goff[(kk >> shift) & mask] + (uint32_t)p;
    if (p < nloc) key_out[o] = kk;
    k[c] = o;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (l0 + 64 * c < nloc) stage[r[c]] = v[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int p = c * BIN_THREADS + t;
    if (p < nloc) val_out[k[c]] = stage[p];
  }
}

// Exclusive scan of uint32 in place, three-phase with recursion.
static constexpr int SCAN_THREADS = 256;
static constexpr int SCAN_ITEMS = 8;
static constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

__global__ void __launch_bounds__(SCAN_THREADS) k_scan_block(uint32_t* a, int64_t n,
                                                             uint32_t* block_sums) {
  __shared__ uint32_t s[SCAN_THREADS];
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  uint32_t v[SCAN_ITEMS], tot = 0;
  for (int k = 0; k < SCAN_ITEMS; ++k) {
    v[k] = base + k < n ? a[base + k] : 0u;
    uint32_t x = v[k];
    v[k] = tot;
    tot += x;
  }
  s[threadIdx.x] = tot;
  __syncthreads();
  for (int off = 1; off < SCAN_THREADS; off <<= 1) {
    uint32_t x = threadIdx.x >= off ? s[threadIdx.x - off] : 0u;
    __syncthreads();
    s[threadIdx.x] += x;
    __syncthreads();
  }
  uint32_t excl = s[threadIdx.x] - tot;
  for (int k = 0; k < SCAN_ITEMS; ++k)
    if (base + k < n) a[base + k] = v[k] + excl;
  if (threadIdx.x == SCAN_THREADS - 1 && block_sums) block_sums[blockIdx.x] = s[threadIdx.x];
}

__global__ void k_scan_add(uint32_t* a, int64_t n, const uint32_t* block_offs) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] += block_offs[i / SCAN_TILE];
}

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// A sort's passes: ITEMS keys of a thread (few where the launch would not
// fill the chip), and as few passes as the histogram's room allows.
// direct: no scan (three launches); every block of the scatter sums the
// histogram's columns, which are then block by block.
struct BinPlan {
  int items, npass, nbits;   // nbits: of every pass but the last, which has the rest
  int64_t nblocks;
  bool direct;
};
static BinPlan bin_plan(int64_t n, int64_t nbins, size_t hist_words) {
  int bits = 1;
  while (bits < 32 && ((uint64_t)1 << bits) <= (uint64_t)nbins) ++bits;
  BinPlan p{};
  p.npass = (bits + BIN_MAX_BITS - 1) / BIN_MAX_BITS;
  p.items = n >= BIN_FEW ? 16 : 4;
  for (;;) {
    p.nbits = (bits + p.npass - 1) / p.npass;
    p.nblocks = ceil_div(n, BIN_THREADS * p.items);
    p.direct = p.items == 4 && p.nblocks <= BIN_DIRECT &&
               (size_t)p.nblocks * (p.nbits <= 8 ? 256 : 512) <= hist_words;
    if (((size_t)p.nblocks << p.nbits) <= hist_words) return p;
    if (p.items == 4) p.items = 16;   // larger blocks, then digits of 8 bits: these always fit
    else ++p.npass;
  }
}

// Room of the histogram for n keys: the largest digits in the blocks that
// bin_plan takes (fixed: the least that a sort needs, 8-bit digits in blocks
// of 4096).
size_t bin_hist_words(int64_t n, bool fixed) {
  const size_t least = (size_t)256 * ceil_div(n, BIN_THREADS * 16);
  if (fixed) return least;
  // (also for fewer keys later, in their smaller blocks)
  const size_t few = (size_t)ceil_div(std::min(n, BIN_FEW), BIN_THREADS * 4) << BIN_MAX_BITS;
  return std::max({least, few, (size_t)ceil_div(n, BIN_THREADS * 16) << BIN_MAX_BITS});
}

size_t bin_scan_tmp_words(int64_t m) {
  size_t words = 0;
  while (m > SCAN_TILE) {
    m = ceil_div(m, SCAN_TILE);
    words += (size_t)m;
  }
  return words + 1;
}

static void scan_exclusive(uint32_t* a, int64_t m, uint32_t* tmp, hipStream_t st) {
  if (m <= 0) return;
  if (m <= SCAN_TILE) {
    hipLaunchKernelGGL(k_scan_block, dim3(1), dim3(SCAN_THREADS), 0, st, a, m, (uint32_t*)nullptr);
    return;
  }
  int64_t nb = ceil_div(m, SCAN_TILE);
  hipLaunchKernelGGL(k_scan_block, dim3((unsigned)nb), dim3(SCAN_THREADS), 0, st, a, m, tmp);
  scan_exclusive(tmp, nb, tmp + nb, st);
  hipLaunchKernelGGL(k_scan_add, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, a, m, tmp);
}

__global__ void k_bin_starts(const uint32_t* key, int64_t n, uint32_t nbins, int64_t* start) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int64_t k = key[i];
  int64_t kp = i == 0 ? -1 : (int64_t)key[i - 1];
  for (int64_t b = kp + 1; b <= k && b <= (int64_t)nbins; ++b) start[b] = i;
  if (i == n - 1)
    for (int64_t b = k + 1; b <= (int64_t)nbins; ++b) start[b] = n;
}

__global__ void k_fill_i64(int64_t* a, int64_t n, int64_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

__global__ void k_copy_perm(const uint32_t* v, int64_t n, int32_t* perm) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) perm[i] = (int32_t)v[i];
}

int launch_bin(const int32_t* cell, int64_t n, const Box* boxes_dev, int nbox, int64_t nbins,
               int key_mode, TileShape tile, BinWork& w, int32_t* perm_out,
               int64_t* bin_start_out, bool keys_ready, hipStream_t st) {
  if (n == 0) {
    if (bin_start_out)
      hipLaunchKernelGGL(k_fill_i64, dim3((unsigned)ceil_div(nbins + 1, 256)), dim3(256), 0, st,
                         bin_start_out, nbins + 1, (int64_t)0);
    return 0;
  }
  if (!keys_ready)
    hipLaunchKernelGGL(k_make_keys, dim3((unsigned)ceil_div(n, BIN_THREADS * KEYS_PER)), dim3(BIN_THREADS), 0, st,
                       cell, n, boxes_dev, nbox, (uint32_t)nbins, key_mode, tile, w.key[0]);
  const BinPlan plan = bin_plan(n, nbins, w.hist_words);
  int bits = 1;
  while (bits < 32 && ((uint64_t)1 << bits) <= (uint64_t)nbins) ++bits;
  const dim3 grid((unsigned)plan.nblocks), block(BIN_THREADS);
  int cur = 0;
  for (int p = 0; p < plan.npass; ++p) {
    const int shift = p * plan.nbits, nb = std::min(plan.nbits, bits - shift);
    const uint32_t* vin = p == 0 ? nullptr : w.val[cur];
    auto pass = [&](auto hist_kern, auto scatter_kern) {
      hipLaunchKernelGGL(hist_kern, grid, block, 0, st, (const uint32_t*)w.key[cur], (uint32_t)n, shift, nb, w.hist,
                         (uint32_t)plan.nblocks);
      if (!plan.direct) scan_exclusive(w.hist, (int64_t)plan.nblocks << nb, w.scan_tmp, st);
      hipLaunchKernelGGL(scatter_kern, grid, block, 0, st, (const uint32_t*)w.key[cur], vin, (uint32_t)n, shift, nb,
                         (const uint32_t*)w.hist, (uint32_t)plan.nblocks, w.key[1 - cur], w.val[1 - cur]);
    };
    if (plan.direct && plan.nbits <= 8) pass(k_digit_hist<256, 4, true>, k_digit_scatter<256, 4, true>);
    else if (plan.direct) pass(k_digit_hist<512, 4, true>, k_digit_scatter<512, 4, true>);
    else if (plan.nbits <= 8 && plan.items == 4) pass(k_digit_hist<256, 4, false>, k_digit_scatter<256, 4, false>);
    else if (plan.nbits <= 8) pass(k_digit_hist<256, 16, false>, k_digit_scatter<256, 16, false>);
    else if (plan.items == 4) pass(k_digit_hist<512, 4, false>, k_digit_scatter<512, 4, false>);
    else pass(k_digit_hist<512, 16, false>, k_digit_scatter<512, 16, false>);
    cur = 1 - cur;
  }
  if (perm_out)
    hipLaunchKernelGGL(k_copy_perm, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, w.val[cur], n,
                       perm_out);
  if (bin_start_out)
    hipLaunchKernelGGL(k_bin_starts, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, st, w.key[cur], n,
                       (uint32_t)nbins, bin_start_out);
  return cur;
}

template <int BYTES> struct Blob { unsigned char b[BYTES]; };

template <typename T>
__global__ void k_permute(const T* in, T* out, const uint32_t* perm, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[perm[i]];
}

void launch_permute(const void* in, void* out, const uint32_t* perm, int64_t n, int bytes,
                    hipStream_t st) {
  if (n == 0) return;
  unsigned g = (unsigned)ceil_div(n, 256);
  if (bytes == 1)
    hipLaunchKernelGGL(k_permute<uint8_t>, dim3(g), dim3(256), 0, st, (const uint8_t*)in,
                       (uint8_t*)out, perm, n);
  else if (bytes == 4)
    hipLaunchKernelGGL(k_permute<uint32_t>, dim3(g), dim3(256), 0, st, (const uint32_t*)in,
                       (uint32_t*)out, perm, n);
  else
    hipLaunchKernelGGL(k_permute<uint64_t>, dim3(g), dim3(256), 0, st, (const uint64_t*)in,
                       (uint64_t*)out, perm, n);
}

}  // namespace dust
