// Photon-event binning and small utility kernels (gfx950, wave64).
#include "nlos_internal.hpp"

#include <algorithm>

namespace nlos {

__global__ __launch_bounds__(256) void fill_u32(uint32_t* __restrict__ p, size_t n, uint32_t v) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 256;
  for (; i < n; i += stride) p[i] = v;
}

__global__ __launch_bounds__(256) void u32_to_f32(const uint32_t* __restrict__ in, float* __restrict__ out,
                                                  size_t n) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 256;
  for (; i < n; i += stride) out[i] = (float)in[i];
}

hipError_t launch_u32_to_f32(const uint32_t* in, float* out, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(u32_to_f32, dim3((unsigned)blocks), dim3(256), 0, s, in, out, n);
  return hipGetLastError();
}

// out[c][r] = in[r][c]: 32 x 32 tiles through LDS, both sides coalesced
__global__ __launch_bounds__(256) void transpose_f32(const float* __restrict__ in, float* __restrict__ out,
                                                     long long rows, int cols) {
  __shared__ float t[32][33];
  const long long r0 = (long long)blockIdx.y * 32;
  const int c0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = ty; k < 32; k += 8) {
    const long long r = r0 + k;
    const int c = c0 + tx;
    if (r < rows && c < cols) t[k][tx] = in[r * cols + c];
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int c = c0 + k;
    const long long r = r0 + tx;
    if (r < rows && c < cols) out[(long long)c * rows + r] = t[tx][k];
  }
}

hipError_t launch_transpose_f32(const float* in, float* out, long long rows, int cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const long long by = (rows + 31) / 32;
  if (by > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(transpose_f32, dim3((unsigned)((cols + 31) / 32), (unsigned)by), dim3(256), 0, s, in, out,
                     rows, cols);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t value, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, value);
  return hipGetLastError();
}

// One event per lane, grid-stride over wave-sized chunks so that every lane of a
// wave takes the same trip count.  Lanes that target the same bin are merged for
// a few rounds (leader lane adds the popcount of its ballot); the remaining lanes
// add 1 each.  Integer atomics make the result exact and order independent.
__global__ __launch_bounds__(256) void bin_events(const uint2* __restrict__ ev, unsigned long long n,
                                                  uint32_t* __restrict__ hist,
                                                  unsigned long long* __restrict__ dropped, int npix,
                                                  int nt, uint32_t bin_ps, uint32_t t0) {
  const int lane = threadIdx.x & 63;
  const unsigned long long stride = (unsigned long long)gridDim.x * 256ull;
  unsigned int drop = 0;
  for (unsigned long long base = (unsigned long long)blockIdx.x * 256ull + (threadIdx.x & ~63u);
       base < n; base += stride) {
    const unsigned long long k = base + lane;
    long long key = -1;
    if (k < n) {
      const uint2 e = ev[k];
      const int pixel = (int)e.x;
      const uint32_t t = e.y;
      if (pixel >= 0 && pixel < npix && t >= t0) {
        const uint32_t b = (t - t0) / bin_ps;
        if (b < (uint32_t)nt) key = (long long)pixel * nt + b;
      }
      if (key < 0) ++drop;
    }
    bool pending = key >= 0;
#pragma unroll
    for (int round = 0; round < 4; ++round) {
      const unsigned long long m = __ballot(pending);
      if (m == 0ull) break;
      const int leader = __ffsll((long long)m) - 1;
      const long long lk = __shfl(key, leader);
      const bool same = pending && key == lk;
      const unsigned long long sm = __ballot(same);
      if (lane == leader) atomicAdd(hist + lk, (uint32_t)__popcll(sm));
      if (same) pending = false;
    }
    if (pending) atomicAdd(hist + key, 1u);
  }
  if (dropped != nullptr) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) drop += __shfl_xor(drop, off, 64);
    if (lane == 0 && drop != 0) atomicAdd(dropped, (unsigned long long)drop);
  }
}

hipError_t launch_bin(const void* events, unsigned long long n, uint32_t* hist,
                      unsigned long long* dropped, int npix, int nt, uint32_t bin_ps, uint32_t t0,
                      hipStream_t s) {
  if (n == 0) return hipSuccess;
  unsigned long long blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(bin_events, dim3((unsigned)blocks), dim3(256), 0, s,
                     static_cast<const uint2*>(events), n, hist, dropped, npix, nt, bin_ps, t0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// binning by pixel tiles
// ---------------------------------------------------------------------------
//
// The histogram (8 MiB at 64 x 64 x 512) is far larger than LDS, and device-scope atomics
// each reach the memory side, so the counters are privatised per tile of tp pixels (tp nt
// counters, at most 16 KB of LDS), in two passes with no global atomics:
// (1) each block takes a chunk of events and sorts it by tile in LDS (per-tile counts, their
//     scan, placement), then writes it back as runs of 16-bit codes (pixel in tile) nt + bin,
//     one run per tile, with the start of every run in a table start[chunk][tile]
//     (start[chunk][ntiles]: the chunk's valid events);
// (2) one block per tile gathers its runs from every chunk, histograms them in LDS and
//     writes the tile's rows with plain stores (all of them, so no clearing pass).
// Events are read once; all adds are integer adds, so the histogram is exact and does not
// depend on the order in which the LDS atomics land.  Both passes wait on latency (the loads,
// the LDS atomics) more than on the 108 MB they move at 1e7 events and 64 x 64 x 512: 28 and
// 23 us, 51 in all against 108 before with scattered reflecting points (the gather searched
// and walked a flat range of all runs per element; see also count_dropped).

constexpr int kBinThreads = 256;
// tp nt <= kBinTileWords (codes fit 16 bits).  Tiles of 2048 words are slower (63 us against 50
// for 1e7 events at 64 x 64 x 512, 137 against 50 for 3e6 at 200 x 200 x 512: beyond kBinMaxTiles
// tiles the atomics).  8192 words take the same 50 us at both and less where a tile holds few
// pixels or few events (42 -> 35 us for 5e6 at 64 x 64 x 1024, 22 -> 19 for 1e6 at 128 x 128 x 256).
constexpr int kBinTileWords = 4096;
constexpr int kBinMaxTiles = 8192;
constexpr int kBinGatherThreads = 1024;

// Quotient of a u32 by a divisor fixed for the launch: a multiply-high and two shifts with
// constants computed on the host (Granlund and Montgomery's division by invariant integers,
// the round-down form with the add fix-up), exact for every 32-bit dividend.
struct U32Div {
  uint32_t m;
  int s1, s2;
};
U32Div u32_div(uint32_t d) {
  int l = 0;
  while (l < 32 && (1ull << l) < d) ++l;
  U32Div r;
  r.m = (uint32_t)((((unsigned __int128)1 << 32) * ((1ull << l) - d)) / d + 1);
  r.s1 = l < 1 ? l : 1;
  r.s2 = l > 1 ? l - 1 : 0;
  return r;
}
__device__ __forceinline__ uint32_t u32_quot(uint32_t n, U32Div d) {
  const uint32_t t = __umulhi(n, d.m);
  return (t + ((n - t) >> d.s1)) >> d.s2;
}

// pixel of a valid event (-1 otherwise) and its bin
__device__ __forceinline__ int bin_event(uint2 e, int npix, int nt, U32Div bin_ps, uint32_t t0, int* b) {
  const int pixel = (int)e.x;
  if (pixel < 0 || pixel >= npix || e.y < t0) return -1;
  const uint32_t bb = u32_quot(e.y - t0, bin_ps);
  if (bb >= (uint32_t)nt) return -1;
  *b = (int)bb;
  return pixel;
}

// LDS atomic add of 1 per lane to cnt[key] (key < 0: none); returns the counter's value
// before this lane's add.  When every active lane of the wave has the same key (sorted
// events, a hot bin) one atomic adds them all; otherwise each lane adds its own (random
// keys rarely coincide within a wave, and the LDS resolves the few conflicts).  Every lane
// of the wave must call it.
__device__ __forceinline__ uint32_t lds_count(uint32_t* cnt, int key) {
  const int lane = threadIdx.x & 63;
  const unsigned long long act = __ballot(key >= 0);
  if (act == 0ull) return 0;
  const int leader = __builtin_amdgcn_readfirstlane(__ffsll((long long)act) - 1);
  const int lk = __builtin_amdgcn_readlane(key, leader);
  if (__ballot(key >= 0 && key == lk) == act) {
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(cnt + lk, (uint32_t)__popcll(act));
    base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
    return base + (uint32_t)__popcll(act & ((1ull << lane) - 1ull));
  }
  return key >= 0 ? atomicAdd(cnt + key, 1u) : 0u;
}

// In-place exclusive scan of a[0..m) in LDS by a block of NT threads, each taking a
// contiguous run; wsum holds NT / 64 words.  The caller synchronises before and after.
template <int NT>
__device__ __forceinline__ void block_exclusive_scan(uint32_t* a, int m, uint32_t* wsum) {
  const int per = (m + NT - 1) / NT;
  const int lo = threadIdx.x * per;
  const int hi = lo + per < m ? lo + per : m;
  uint32_t s = 0;
  for (int i = lo; i < hi; ++i) s += a[i];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = s;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint32_t run = x - s;
  for (int k = 0; k < w; ++k) run += wsum[k];
  for (int i = lo; i < hi; ++i) {
    const uint32_t v = a[i];
    a[i] = run;
    run += v;
  }
}

// Pass 1: chunk blockIdx.x of kBinThreads PT events -> runs[chunk][.] (16-bit codes
// (pixel in tile) stride + bin, sorted by tile) and start[chunk][tile].
template <int PT>
__global__ __launch_bounds__(kBinThreads) void bin_chunk_sort(const uint2* __restrict__ ev, unsigned long long n,
                                                             int npix, int nt, U32Div bin_ps, uint32_t t0, int tp,
                                                             int stride, U32Div tp_div,
                                                             int ntiles, uint16_t* __restrict__ runs,
                                                             uint16_t* __restrict__ start) {
  extern __shared__ uint32_t sh[];
  uint32_t* cnt = sh;  // ntiles + 1 counters, then their exclusive scan
  uint16_t* sorted = reinterpret_cast<uint16_t*>(sh + ntiles + 1);  // the codes
  __shared__ uint32_t wsum[kBinThreads / 64];
  for (int i = threadIdx.x; i <= ntiles; i += kBinThreads) cnt[i] = 0;
  __syncthreads();
  const unsigned long long beg = (unsigned long long)blockIdx.x * (kBinThreads * PT);
  uint32_t code[PT];  // tile << 16 | (pixel in tile) nt + bin; ~0u: none
  uint32_t pos[PT];   // place in the tile's run
  constexpr int kLoads = PT < 16 ? PT : 16;  // loads in flight per lane
#pragma unroll
  for (int r = 0; r < PT; r += kLoads) {
    uint2 e[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const unsigned long long k = beg + (unsigned long long)(r + j) * kBinThreads + threadIdx.x;
      e[j] = k < n ? ev[k] : make_uint2(0xffffffffu, 0u);  // (pixel -1: no event)
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      uint32_t c = ~0u;
      int b = 0;
      const int px = bin_event(e[j], npix, nt, bin_ps, t0, &b);
      if (px >= 0) {
        const int tile = (int)u32_quot((uint32_t)px, tp_div);
        c = ((uint32_t)tile << 16) | (uint32_t)((px - tile * tp) * stride + b);
      }
      code[r + j] = c;
      pos[r + j] = lds_count(cnt, c == ~0u ? -1 : (int)(c >> 16));
    }
  }
  __syncthreads();
  block_exclusive_scan<kBinThreads>(cnt, ntiles + 1, wsum);
  __syncthreads();
  for (int i = threadIdx.x; i <= ntiles; i += kBinThreads)
    start[(size_t)blockIdx.x * (ntiles + 1) + i] = (uint16_t)cnt[i];
#pragma unroll
  for (int j = 0; j < PT; ++j)
    if (code[j] != ~0u) sorted[cnt[code[j] >> 16] + pos[j]] = (uint16_t)(code[j] & 0xffffu);
  __syncthreads();
  const uint32_t nv = cnt[ntiles];
  uint16_t* out = runs + (size_t)blockIdx.x * (kBinThreads * PT);
  for (uint32_t i = threadIdx.x; i < nv; i += kBinThreads) out[i] = sorted[i];
}

// Pass 2 for one tile and a block of NT threads: counts its codes of every chunk's run in the
// tile's histogram h (`words` counters in LDS, cleared here).  Groups of 1 << lw lanes take a
// run each, kBinRuns runs in flight: their bounds, then their codes, then the counts.
constexpr int kBinRuns = 4;
template <int NT>
__device__ __forceinline__ void gather_tile(const uint16_t* __restrict__ runs, const uint16_t* __restrict__ start,
                                            int ntiles, int nchunks, int chunk, int t, uint32_t* h, int words, int lw) {
  for (int i = threadIdx.x; i < words; i += NT) h[i] = 0;
  __syncthreads();
  const int W = 1 << lw, groups = NT >> lw;
  const int g = threadIdx.x >> lw, l = threadIdx.x & (W - 1);
  for (int k0 = 0; k0 < nchunks; k0 += groups * kBinRuns) {
    uint32_t i[kBinRuns], e[kBinRuns];
    const uint16_t* run[kBinRuns];
#pragma unroll
    for (int u = 0; u < kBinRuns; ++u) {
      const int k = k0 + u * groups + g;
      const int kc = k < nchunks ? k : 0;
      const uint16_t* st = start + (size_t)kc * (ntiles + 1) + t;
      i[u] = st[0] + l;
      e[u] = k < nchunks ? st[1] : 0;
      run[u] = runs + (size_t)kc * chunk;
    }
    bool more = true;
    while (more) {  // (the wave's longest run)
      uint32_t v[kBinRuns];
      more = false;
#pragma unroll
      for (int u = 0; u < kBinRuns; ++u) {
        v[u] = i[u] < e[u] ? run[u][i[u]] : 0xffffu;
        i[u] += W;
        more |= i[u] < e[u];
      }
#pragma unroll
      for (int u = 0; u < kBinRuns; ++u) lds_count(h, v[u] == 0xffffu ? -1 : (int)v[u]);
      more = __ballot(more) != 0ull;
    }
  }
  __syncthreads();
}

// Invalid events: n less the chunks' valid ones, by the block of tile 0 (an atomic per wave of
// pass 1 on the one counter took 45 us of 1e7 events).
template <int NT>
__device__ __forceinline__ void count_dropped(const uint16_t* __restrict__ start, int ntiles, int nchunks,
                                              unsigned long long n, unsigned long long* dropped, int accumulate) {
  if (blockIdx.x != 0 || dropped == nullptr) return;
  __shared__ unsigned int part[NT / 64];
  unsigned int v = 0;  // n < 2^31
  for (int k = threadIdx.x; k < nchunks; k += NT) v += start[(size_t)k * (ntiles + 1) + ntiles];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x != 0) return;
  unsigned long long d = n;
  for (int w = 0; w < NT / 64; ++w) d -= part[w];
  if (accumulate) atomicAdd(dropped, d);  // (a counter that other streams may be adding to)
  else *dropped = d;
}

template <int NT>
__global__ __launch_bounds__(NT) void bin_tile_gather(const uint16_t* __restrict__ runs,
                                                      const uint16_t* __restrict__ start, int ntiles, int nchunks,
                                                      int chunk, int npix, int nt, int tp, int lw,
                                                      uint32_t* __restrict__ hist, int accumulate,
                                                      unsigned long long n, unsigned long long* dropped) {
  extern __shared__ uint32_t h[];  // tp nt counters
  const int words = tp * nt;
  count_dropped<NT>(start, ntiles, nchunks, n, dropped, accumulate);
  gather_tile<NT>(runs, start, ntiles, nchunks, chunk, blockIdx.x, h, words, lw);
  const long long first = (long long)blockIdx.x * tp * nt;
  const long long last = (long long)npix * nt;
  for (int i = threadIdx.x; i < words && first + i < last; i += NT) {
    uint32_t* g = hist + first + i;
    *g = accumulate ? *g + h[i] : h[i];
  }
}

// Pass 2 of phasor binning: the tile's histogram as above, which stays in LDS, then its DFT at
// the nf bins on the matrix cores (FP32): rows are the (re, im) parts of the frequencies in
// blocks of 16, columns the tile's pixels in blocks of 16, the contraction runs over the time
// bins, 4 a step.  The twiddles come as operands from the plan's table
// tab[row block][step][lane] (lane l: part (l % 16) of the block at bin 4 step + l / 16), the
// counts from the histogram, whose rows are `stride` = 4 mod 64 words apart so that 16 pixels
// x 4 bins fall on 64 banks.  Few blocks split the bins over the waves and add up in LDS.
// Every sum has a fixed order.  The same DFT on the vector units took 45 us of 61 at
// 64 x 64 x 512 with 39 frequencies (7 instructions per count and frequency).
typedef float bin_f4 __attribute__((ext_vector_type(4)));
constexpr int kPhasorWaves = kBinGatherThreads / 64;
__global__ __launch_bounds__(kBinGatherThreads) void bin_tile_phasor(const uint16_t* __restrict__ runs,
                                                                    const uint16_t* __restrict__ start, int ntiles,
                                                                    int nchunks, int chunk, int npix, int nt, int tp,
                                                                    int lw, int stride, const float* __restrict__ tab,
                                                                    int nf, float* __restrict__ P, int accumulate,
                                                                    unsigned long long n,
                                                                    unsigned long long* dropped) {
  extern __shared__ uint32_t h[];  // tp stride counters, later the partial sums [wave][256]
  const int words = tp * stride;
  float* red = reinterpret_cast<float*>(h);
  count_dropped<kBinGatherThreads>(start, ntiles, nchunks, n, dropped, accumulate);
  gather_tile<kBinGatherThreads>(runs, start, ntiles, nchunks, chunk, blockIdx.x, h, words, lw);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, kq = lane >> 4;
  const int pix0 = blockIdx.x * tp;
  const int npx = npix - pix0 < tp ? npix - pix0 : tp;
  const int nsteps = (nt + 3) / 4;
  const int nrb = (2 * nf + 15) / 16;
  const int units = nrb * ((npx + 15) / 16);
  const int ks = units >= kPhasorWaves ? 1 : kPhasorWaves / units;  // parts of the contraction
  const int per = (nsteps + ks - 1) / ks;
  auto put = [&](int u, bin_f4 d) {  // lane: rows 4 kq + v, column c16
    const int px = (u / nrb) * 16 + c16, row = (u % nrb) * 16 + 4 * kq;
    if (px >= npx) return;
    float* o = P + (long long)(pix0 + px) * 2 * nf + row;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (row + v < 2 * nf) {
        if (accumulate) unsafeAtomicAdd(o + v, d[v]);  // (phasors that other streams may be adding to)
        else o[v] = d[v];
      }
  };
  bin_f4 d;
  for (int s0 = 0; s0 < units * ks; s0 += kPhasorWaves) {
    const int slot = s0 + wv;
    d = bin_f4{0.f, 0.f, 0.f, 0.f};
    if (slot < units * ks) {
      const int u = slot / ks, q0 = (slot % ks) * per;
      const int q1 = q0 + per < nsteps ? q0 + per : nsteps;
      const int px = (u / nrb) * 16 + c16;
      const uint32_t* row = h + (px < tp ? px : tp - 1) * stride + kq;
      const float* t = tab + (long long)(u % nrb) * nsteps * 64 + lane;
#pragma unroll 8
      for (int q = q0; q < q1; ++q) d = __builtin_amdgcn_mfma_f32_16x16x4f32(t[q * 64], (float)row[4 * q], d, 0, 0, 0);
      if (ks == 1) put(u, d);
    }
  }
  if (ks == 1) return;
  // one slot per wave (units ks <= kPhasorWaves); every histogram read is done
  __syncthreads();
  *reinterpret_cast<bin_f4*>(red + wv * 256 + 4 * lane) = d;
  __syncthreads();
  if (wv < units) {
    d = *reinterpret_cast<const bin_f4*>(red + wv * ks * 256 + 4 * lane);
    for (int i = 1; i < ks; ++i) d += *reinterpret_cast<const bin_f4*>(red + (wv * ks + i) * 256 + 4 * lane);
    put(wv, d);
  }
}

// Events per thread of pass 1 (a chunk is kBinThreads times as many): short jobs want more blocks
// (1e4 events at 64 x 64 x 512: 11, 13 and 18 us with 8, 16 and 32), long ones longer runs
// (1e7: 72, 58 and 54; 3e6 at 200 x 200 x 512: 85, 61 and 52)
int bin_per_thread(unsigned long long n) { return n < 400000 ? 8 : n < 1500000 ? 16 : 32; }

// Tile layout of a binning job: tp pixels of `stride` words per tile (tp stride <= words), or
// false when the tiled path does not apply (then the per-event atomic kernel runs).
// Small images keep at least `least` pixels a tile, for blocks enough to fill the device.
bool bin_tiles(int npix, int stride, unsigned long long n, int words, int least, int* tp, int* ntiles) {
  if (stride > words || n >= (1ull << 31)) return false;
  *tp = std::min(words / stride, std::max(npix / 512, least));
  if (*tp > npix) *tp = npix;
  *ntiles = (npix + *tp - 1) / *tp;
  return *ntiles <= kBinMaxTiles;
}
// Phasor binning: 16 pixels a tile (the columns of a matrix product) up to 1024 bins, fewer
// beyond (two blocks of 66 KB of LDS per CU), more below 512; and the row stride of
// bin_tile_phasor
int phasor_words(int stride) { return std::min(std::max(16 * 516, 16 * stride), 16 * 1028); }
int phasor_stride(int nt) { return (nt + 59) / 64 * 64 + 4; }

size_t bin_runs_bytes(unsigned long long n, int ntiles) {
  const size_t chunk = (size_t)kBinThreads * bin_per_thread(n);
  const size_t nchunks = (size_t)((n + chunk - 1) / chunk);
  const size_t bytes = 2 * nchunks * chunk + 2 * (size_t)(ntiles + 1) * nchunks;
  return bytes > 0 ? bytes : 256;  // never zero: zero means "not tiled"
}
size_t bin_workspace_bytes(int npix, int nt, unsigned long long n) {
  int tp = 0, nti = 0;
  return bin_tiles(npix, nt, n, kBinTileWords, 1, &tp, &nti) ? bin_runs_bytes(n, nti) : 0;
}
size_t phasor_workspace_bytes(int npix, int nt, unsigned long long n) {
  int tp = 0, nti = 0;
  return bin_tiles(npix, phasor_stride(nt), n, phasor_words(phasor_stride(nt)), 16, &tp, &nti) ? bin_runs_bytes(n, nti) : 0;
}

namespace {
// The tiles of a job and its sorted runs in ws (pass 1 launched)
struct BinRuns {
  int tp, ntiles, nchunks, chunk;
  int lw;           // log2 of the lanes that gather a run: about its mean length, 4 .. 64
  uint16_t* runs;   // [chunk][.]
  uint16_t* start;  // [chunk][tile], ntiles + 1 a row
};
hipError_t bin_sort(const void* events, unsigned long long n, int npix, int nt,
                    int stride, int words, int least, uint32_t bin_ps, uint32_t t0, void* ws, hipStream_t s,
                    BinRuns* r) {
  if (!bin_tiles(npix, stride, n, words, least, &r->tp, &r->ntiles)) return hipErrorInvalidValue;
  const int pt = bin_per_thread(n);
  r->chunk = kBinThreads * pt;
  r->nchunks = (int)((n + r->chunk - 1) / r->chunk);
  r->runs = static_cast<uint16_t*>(ws);
  r->start = r->runs + (size_t)r->nchunks * r->chunk;
  r->lw = 2;
  while (r->lw < 6 && r->chunk / r->ntiles >= (2 << r->lw)) ++r->lw;
  if (r->nchunks == 0) return hipSuccess;
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, dim3((unsigned)r->nchunks), dim3(kBinThreads),
                       (size_t)4 * (r->ntiles + 1) + (size_t)2 * r->chunk, s, static_cast<const uint2*>(events), n,
                       npix, nt, u32_div(bin_ps), t0, r->tp, stride, u32_div((uint32_t)r->tp), r->ntiles, r->runs, r->start);
    return hipGetLastError();
  };
  return pt == 32 ? go(bin_chunk_sort<32>) : pt == 16 ? go(bin_chunk_sort<16>) : go(bin_chunk_sort<8>);
}
}  // namespace

hipError_t launch_bin_tiled(const void* events, unsigned long long n, uint32_t* hist, unsigned long long* dropped,
                            int npix, int nt, uint32_t bin_ps, uint32_t t0, int accumulate, void* ws, hipStream_t s) {
  BinRuns r;
  const hipError_t e = bin_sort(events, n, npix, nt, nt, kBinTileWords, 1, bin_ps, t0, ws, s, &r);
  if (e != hipSuccess) return e;
  auto go = [&](auto k, int threads) {
    hipLaunchKernelGGL(k, dim3((unsigned)r.ntiles), dim3(threads), (size_t)4 * r.tp * nt, s, r.runs, r.start, r.ntiles,
                       r.nchunks, r.chunk, npix, nt, r.tp, r.lw, hist, accumulate, n, dropped);
    return hipGetLastError();
  };
  return r.ntiles >= 1024 && n / r.ntiles < 4096 ? go(bin_tile_gather<256>, 256) : go(bin_tile_gather<kBinGatherThreads>, kBinGatherThreads);
}

size_t phasor_table(int nt, int nf, const int* bins, const float2* lut, float* tab) {
  const int nsteps = (nt + 3) / 4, nrb = (2 * nf + 15) / 16;
  if (tab != nullptr)
    for (int rb = 0; rb < nrb; ++rb)
      for (int q = 0; q < nsteps; ++q)
        for (int l = 0; l < 64; ++l) {
          const int c = rb * 16 + l % 16, b = 4 * q + l / 16;
          const float2 w = c < 2 * nf && b < nt ? lut[((long long)bins[c / 2] * b) % nt] : make_float2(0.f, 0.f);
          *tab++ = c % 2 ? w.y : w.x;
        }
  return (size_t)nrb * nsteps * 64;
}

hipError_t launch_phasor_tiled(const void* events, unsigned long long n, float2* P, unsigned long long* dropped,
                               int npix, int nt, uint32_t bin_ps, uint32_t t0, const float* tab, int nf,
                               int accumulate, void* ws, hipStream_t s) {
  const int stride = phasor_stride(nt);
  BinRuns r;
  const hipError_t e = bin_sort(events, n, npix, nt, stride, phasor_words(stride), 16, bin_ps, t0, ws, s, &r);
  if (e != hipSuccess) return e;
  const size_t lds = std::max((size_t)4 * r.tp * stride, (size_t)1024 * kPhasorWaves);
  hipLaunchKernelGGL(bin_tile_phasor, dim3((unsigned)r.ntiles), dim3(kBinGatherThreads), lds, s, r.runs, r.start,
                     r.ntiles, r.nchunks, r.chunk, npix, nt, r.tp, r.lw, stride, tab, nf, reinterpret_cast<float*>(P), accumulate,
                     n, dropped);
  return hipGetLastError();
}

// Phasors straight from photon records (Section 4.1, phasor binning; the paper's warp
// per photon becomes a wave64 per photon): a wave loads 64 events, then takes them one
// at a time, its lanes striding over the frequencies; lane f adds the unit phasor
// W_nt^(k_f b) of the event's bin b (from an LDS copy of the FP64-built table) to
// P[pixel][f] with hardware float atomics.  Float sums in arbitrary order: equal to the
// DFT of the histogram up to rounding.
__global__ __launch_bounds__(256) void phasor_bin(const uint2* __restrict__ ev, unsigned long long n,
                                                  float2* __restrict__ P, unsigned long long* __restrict__ dropped,
                                                  int npix, int nt, uint32_t bin_ps, uint32_t t0,
                                                  const float2* __restrict__ lut, const int* __restrict__ bins,
                                                  int nf) {
  __shared__ float2 slut[2048];
  for (int i = threadIdx.x; i < nt; i += 256) slut[i] = lut[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const unsigned long long stride = (unsigned long long)gridDim.x * 256ull;
  unsigned int drop = 0;
  for (unsigned long long base = (unsigned long long)blockIdx.x * 256ull + (threadIdx.x & ~63u);
       base < n; base += stride) {
    const unsigned long long k = base + lane;
    int pix = -1, b = 0;
    if (k < n) {
      const uint2 e = ev[k];
      const int pixel = (int)e.x;
      const uint32_t t = e.y;
      if (pixel >= 0 && pixel < npix && t >= t0) {
        const uint32_t bb = (t - t0) / bin_ps;
        if (bb < (uint32_t)nt) {
          pix = pixel;
          b = (int)bb;
        }
      }
      if (pix < 0) ++drop;
    }
    const unsigned long long valid = __ballot(pix >= 0);
    for (unsigned long long m = valid; m != 0ull; m &= m - 1ull) {
      const int j = __ffsll((long long)m) - 1;  // next valid event of the wave (uniform)
      const int pj = __shfl(pix, j), bj = __shfl(b, j);
      float2* row = P + (long long)pj * nf;
      for (int f = lane; f < nf; f += 64) {
        const float2 w = slut[(int)(((long long)bins[f] * bj) % nt)];
        unsafeAtomicAdd(&row[f].x, w.x);
        unsafeAtomicAdd(&row[f].y, w.y);
      }
    }
  }
  if (dropped != nullptr) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) drop += __shfl_xor(drop, off, 64);
    if (lane == 0 && drop != 0) atomicAdd(dropped, (unsigned long long)drop);
  }
}

hipError_t launch_phasor_bin(const void* events, unsigned long long n, float2* P, unsigned long long* dropped,
                             int npix, int nt, uint32_t bin_ps, uint32_t t0, const float2* lut, const int* bins,
                             int nf, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (nt < 1 || nt > 2048 || nf < 1) return hipErrorInvalidValue;
  unsigned long long blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(phasor_bin, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<const uint2*>(events), n, P,
                     dropped, npix, nt, bin_ps, t0, lut, bins, nf);
  return hipGetLastError();
}

// Coherence-weighted merging (Section 4.4, Eq. 8-9) over the most recent `count` frames:
// S = sum f_j, A = sum |f_j| (oldest first), C = |S| / (eps + A), merged = C |S| / count.
// The new frame is stored into its ring slot in the same pass.
__global__ __launch_bounds__(256) void merge_frames(const float2* __restrict__ frame, float2* __restrict__ ring,
                                                    long long n, int window, int slot, int first, int count,
                                                    float eps, float* __restrict__ merged,
                                                    float* __restrict__ coherence) {
  for (long long v = (long long)blockIdx.x * 256 + threadIdx.x; v < n; v += (long long)gridDim.x * 256) {
    const float2 f = frame[v];
    ring[(long long)slot * n + v] = f;
    float2 S = make_float2(0.f, 0.f);
    float A = 0.f;
    for (int k = 0; k < count; ++k) {
      int r = first + k;
      if (r >= window) r -= window;
      const float2 g = (r == slot) ? f : ring[(long long)r * n + v];
      S.x += g.x;
      S.y += g.y;
      A += sqrtf(g.x * g.x + g.y * g.y);
    }
    const float s = sqrtf(S.x * S.x + S.y * S.y);
    const float C = s / (eps + A);
    merged[v] = C * s / (float)count;
    if (coherence) coherence[v] = C;
  }
}

hipError_t launch_merge(const float2* frame, float2* ring, long long n, int window, int slot, int first,
                        int count, float eps, float* merged, float* coherence, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (window < 1 || slot < 0 || slot >= window || first < 0 || first >= window || count < 1 || count > window)
    return hipErrorInvalidValue;
  long long blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(merge_frames, dim3((unsigned)blocks), dim3(256), 0, s, frame, ring, n, window, slot, first,
                     count, eps, merged, coherence);
  return hipGetLastError();
}

}  // namespace nlos
