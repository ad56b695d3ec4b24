// Radial RSD propagation (Section 4.3 propagation sum, Listing 3 lookup, Algorithm 4
// inner loop) for gfx950.
//
//   C[pix][d] = sum_f w_f P^[pix][f] a(pix) lerp(K_r[., f, d], rho~(pix))
//             = sum_f (wa w_f P^) K_r[i0][f][d] + (wb w_f P^) K_r[i0+1][f][d]
//
// The plan sorts the pixels by their lower radial bin i0 and groups them into chunks of
// up to 64 that share i0.  On FP32 FMAs (rsd_propagate, on request only; the matrix cores below
// are the default) one wave64 takes a chunk, one pixel per lane, and a slice of kDepths depths:
// the kernel rows K_r[i0][f][d0..d0+kDepths) and K_r[i0+1][f][...] have the same address in
// every lane, each value read from its plane or planes and put together (load_kr) once per 64
// pixels.  The lane's own phasor P^[pix][f] is read from its contiguous frequency row.  Every C
// element is produced by one lane in a fixed frequency order.
#include <hip/hip_fp16.h>

#include <algorithm>
#include <type_traits>

#include "mfma_fft.hpp"
#include "nlos_internal.hpp"

namespace nlos {

constexpr int kGroupPix = 64;   // pixels per chunk (one per lane; matches the plan)
constexpr int kDepths = 8;      // depths per wave
constexpr int kWavesPerBlock = 4;

// K_r[i][f][d] from the plan's table (see RsdPropArgs::Kr); FP32 is the sum of its three
// bfloat16 planes times 2^kr_exp
template <int SP>
__device__ __forceinline__ float2 load_kr(const RsdPropArgs& a, int i, int f, int d) {
  constexpr int FL = SP == SP_F32 ? 4 : 2;
  const int ng = 8 / FL * ((a.Nf + 7) / 8);
  const long long o = (((long long)i * ng + f / FL) * a.Nd + d) * FL + f % FL;
  const unsigned int* kr = static_cast<const unsigned int*>(a.Kr);
  if constexpr (SP == SP_F32) {
    using M = Mfma<SP_BF16>;
    const float2 k0 = M::unpack(kr[o]), k1 = M::unpack(kr[o + a.kr_plane]), k2 = M::unpack(kr[o + 2 * a.kr_plane]);
    const float2 k = make_float2((k2.x + k1.x) + k0.x, (k2.y + k1.y) + k0.y);
    return a.kr_exp == 0 ? k : make_float2(ldexpf(k.x, a.kr_exp), ldexpf(k.y, a.kr_exp));
  } else {
    return Mfma<SP>::unpack(kr[o]);
  }
}

// acc += pa K0 + pb K1 (complex), fixed operation order
__device__ __forceinline__ void cmac2(float2& acc, float2 pa, float2 k0, float2 pb, float2 k1) {
  acc.x = fmaf(pa.x, k0.x, fmaf(-pa.y, k0.y, fmaf(pb.x, k1.x, fmaf(-pb.y, k1.y, acc.x))));
  acc.y = fmaf(pa.x, k0.y, fmaf(pa.y, k0.x, fmaf(pb.x, k1.y, fmaf(pb.y, k1.x, acc.y))));
}

// One frequency f of the lane's pixel: tap-weighted phasors, then the ND depths of the
// wave's slice (kernel rows o0, o1 are wave-uniform).
template <int SP, int ND>
__device__ __forceinline__ void rsd_freq(float2* acc, float2 p, float2 wf, float wa, float wb, const RsdPropArgs& a,
                                         int i0, int i1, int f, int d0) {
  const float2 pw = make_float2(p.x * wf.x - p.y * wf.y, p.x * wf.y + p.y * wf.x);
  const float2 pa = make_float2(pw.x * wa, pw.y * wa);
  const float2 pb = make_float2(pw.x * wb, pw.y * wb);
#pragma unroll
  for (int j = 0; j < ND; ++j) 
    cmac2(acc[j], pa, load_kr<SP>(a, i0, f, d0 + j), pb, load_kr<SP>(a, i1, f, d0 + j));
}

// The last pass takes its maxima over several blocks of a pixel: the image is cleared here,
// one value per thread (a launch less).
__device__ __forceinline__ void clear_image(const RsdPropArgs& a) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t < a.img_n) a.img[t] = 0.f;
}

template <int SP>
__global__ __launch_bounds__(256) void rsd_propagate(RsdPropArgs a) {
  clear_image(a);
  const int lane = threadIdx.x & 63;
  // wave-uniform work index: chunk g, depth slice starting at d0
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nds = (a.Nd + kDepths - 1) / kDepths;
  const long long w = (long long)blockIdx.x * kWavesPerBlock + wib;
  if (w >= a.nchunks * nds) return;
  const long long g = w / nds;
  const int d0 = (int)(w % nds) * kDepths;
  const int Nf = a.Nf, Nd = a.Nd;
  const int i0 = a.chunk_i0[g];
  const int pix = a.chunk_pix[g * kGroupPix + lane];
  float2 acc[kDepths];
#pragma unroll
  for (int j = 0; j < kDepths; ++j) acc[j] = make_float2(0.f, 0.f);
  if (i0 >= 0) {
    const int i1 = i0 + 1 < a.cut_idx ? i0 + 1 : a.cut_idx;
    // unused slots have wa = wb = 0 and read pixel 0's row
    const float wa = a.chunk_wa[g * kGroupPix + lane];
    const float wb = a.chunk_wb[g * kGroupPix + lane];
    const float2* __restrict__ ph = static_cast<const float2*>(a.Ph) + (long long)(pix >= 0 ? pix : 0) * a.ph_stride;
    if (d0 + kDepths <= Nd) {
      int f = 0;
      // eight phasor loads in flight per lane
      for (; f + 8 <= Nf; f += 8) {
        float2 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = ph[f + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          rsd_freq<SP, kDepths>(acc, p[u], a.w[f + u], wa, wb, a, i0, i1, f + u, d0);
        }
      }
      for (; f < Nf; ++f) {
        rsd_freq<SP, kDepths>(acc, ph[f], a.w[f], wa, wb, a, i0, i1, f, d0);
      }
    } else {
      // last, partial depth slice
      const int nd = Nd - d0;
      for (int f = 0; f < Nf; ++f) {
        const float2 p = ph[f], wf = a.w[f];
        const float2 pw = make_float2(p.x * wf.x - p.y * wf.y, p.x * wf.y + p.y * wf.x);
        const float2 pa = make_float2(pw.x * wa, pw.y * wa);
        const float2 pb = make_float2(pw.x * wb, pw.y * wb);
#pragma unroll
        for (int j = 0; j < kDepths; ++j)
          if (j < nd) cmac2(acc[j], pa, load_kr<SP>(a, i0, f, d0 + j), pb, load_kr<SP>(a, i1, f, d0 + j));
      }
    }
  }
  if (pix < 0) return;
  float2* out = static_cast<float2*>(a.C) + (long long)pix * a.c_stride + d0;
#pragma unroll
  for (int j = 0; j < kDepths; ++j)
    if (d0 + j < Nd) out[j] = acc[j];
}

// ---------------------------------------------------------------------------
// matrix-core propagation
// ---------------------------------------------------------------------------
//
// For one chunk the sum is a complex matrix product: rows = the chunk's pixels, the
// contraction runs over (tap, frequency), columns = depths.  As a real product on (re, im)
// pairs it maps onto v_mfma_f32_32x32x16 (FP32 accumulation): a 16-wide K step is 8
// frequencies of one tap (FP32 kernels; lane l holds frequencies 8 s + 4 (l / 32) + 0..3 of
// row or column l % 32) or 4 frequencies x 2 taps (FP16 / BF16; 4 s + 2 (l / 32) + 0..1).  The
// kernel operands come as stored pairs from the plan's table, one 16- or 8-byte load a tap and
// step; the phasors enter as (re, -im) for the real part of the output and (im, re) for the
// imaginary.
// A wave takes half a chunk (32 pixels) and DT 32-depth tiles; the loads of the next step are
// in flight during a step (unconditional, clamped: a frequency beyond Nf has a zero weight, a
// depth beyond Nd only feeds columns that are not stored).
//
// FP16 / BF16 kernels: the phasors w_f P^ (wa | wb) of each tap are rounded to the kernel's
// format, FP16 after scaling by 2^e, e per half chunk from the largest |w_f P^| max(wa, wb)
// of its pixels (a first pass over their rows) so that every component stays below 2^14; the
// FP32 result is multiplied by 2^-e.  BF16 has FP32's exponent range and takes no scale.
// DATA4: P^ and C are stored in the kernel's four-byte format too (FP16 P^ times 2^e_ph, FP16
// C at depth d written times 2^e_c[d]), the exponents folded into one final ldexp.
//
// FP32 kernels (the splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", 2019): an FP32 value is the sum of
// three bfloat16 values x0 + x1 + x2 (each the rounded remainder of the previous; 3 x 8 bits), so
// a product is the sum of the six bfloat16 products of order below 2^-24: a0 b0, a0 b1, a1 b0,
// a0 b2, a1 b1, a2 b0 (the dropped a1 b2 + a2 b1 are about 2^-26 of it, of random sign).  The
// kernel's planes come with the plan, the phasors are split in registers; each tap has its own
// accumulators and the tap weights come last, so the split is paid once.  The sums take 3/8 of
// the time of FP32 matrix instructions and round less often (once per 16-wide product sum instead
// of per 2-wide): over the volume within the error of the FP32 instructions against 64 bits.
// The split is exact, and no partial product is lost, only well inside FP32's range: below 2^-109
// the third part leaves bfloat16's normal numbers, above 2^128 - 2^119 the first rounds to
// infinity.  The plan scales the kernel there (RsdPropArgs::kr_exp), and a wave sees from its
// sums, at no cost to its steps, whether its phasors were: sums below kSplitMin (with |K_r| up to
// 2^12 and 2048 terms, phasors of 2^-93 give at most 2^-70), above kSplitMax or not a number make
// it start again with FP32 instructions (propagate_f32).  The largest of the wave
// counts: what smaller phasors lose is below 2^-30 of it.
//
// 128 x 128 x 1024 (129 frequencies, 64 depths; 8.7 GFLOP): FP32 131 -> 76 us, BF16 77 -> 47 us
// against one 64-pixel chunk per wave with FP32 matrix instructions and scattered operand
// loads.  The matrix cores are busy 32 % and the vector units (the splits) 27 % of it.
template <int KSP>
struct PropFmt {  // matrix-core format and planes of a kernel's storage
  static constexpr int SP = KSP == SP_F32 ? (int)SP_BF16 : KSP;
  static constexpr int NPL = KSP == SP_F32 ? 3 : 1;
  static constexpr int NT = KSP == SP_F32 ? 2 : 1;  // accumulator sets: one per tap
  static constexpr int FL = KSP == SP_F32 ? 4 : 2;  // frequencies per lane and step
};

// (re, im) pairs of one K step as the A operands of the real and the imaginary part
__device__ __forceinline__ mf_u4 prop_re(mf_u4 a) { return a ^ 0x80000000u; }
__device__ __forceinline__ mf_u4 prop_im(mf_u4 a) {
  return mf_u4{__builtin_amdgcn_alignbit(a[0], a[0], 16), __builtin_amdgcn_alignbit(a[1], a[1], 16),
               __builtin_amdgcn_alignbit(a[2], a[2], 16), __builtin_amdgcn_alignbit(a[3], a[3], 16)};
}

constexpr float kSplitMin = 0x1p-70f, kSplitMax = 0x1p100f;

// A half chunk's sum with an FP32 kernel on v_mfma_f32_32x32x2f32: a step is one (frequency,
// tap), lane l holds part l / 32 (re or im) of the tap-weighted phasor of its row and the kernel
// value of its column as (re, -im) for the real part of the output, (im, re) for the imaginary.
// Only for phasors beyond the split's range: plain loads, nothing in flight ahead.
// (Everything is worked out anew from the lane number, behind a barrier to the optimiser, so that
// none of it occupies registers during the steps of the split.)
template <int DT>
__device__ __forceinline__ void propagate_f32(const RsdPropArgs& a, const float2* ws, long long gh, int d0, int i0,
                                              int i1, mf_acc (*acc)[2]) {
  int ln = threadIdx.x & 63;
  asm volatile("" : "+v"(ln));
  const bool im = ln >= 32;
  const int c = ln & 31, pix = a.chunk_pix[gh * 32 + c];
  const float wa = a.chunk_wa[gh * 32 + c], wb = a.chunk_wb[gh * 32 + c];
  const float2* row = static_cast<const float2*>(a.Ph) + (long long)(pix >= 0 ? pix : 0) * a.ph_stride;
#pragma unroll
  for (int q = 0; q < DT; ++q)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[q][0][v] = acc[q][1][v] = 0.f;
#pragma unroll 1
  for (int f = 0; f < a.Nf; ++f) {
    const float2 p = row[f], wf = ws[f];
    const float z = im ? p.x * wf.y + p.y * wf.x : p.x * wf.x - p.y * wf.y;
    const float A[2] = {wa * z, wb * z};
#pragma unroll
    for (int q = 0; q < DT; ++q)
#pragma unroll
      for (int tap = 0; tap < 2; ++tap) {
        const float2 k = load_kr<SP_F32>(a, tap == 0 ? i0 : i1, f, min(d0 + 32 * q + c, a.Nd - 1));
        acc[q][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(A[tap], im ? -k.y : k.x, acc[q][0], 0, 0, 0);
        acc[q][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(A[tap], im ? k.x : k.y, acc[q][1], 0, 0, 0);
      }
  }
}

// A half chunk whose every phasor w_f P^ is zero
__device__ __forceinline__ bool all_zero(const RsdPropArgs& a, const float2* ws, long long gh) {
  int ln = threadIdx.x & 63;
  asm volatile("" : "+v"(ln));
  const int pix = a.chunk_pix[gh * 32 + (ln & 31)];
  const float2* row = static_cast<const float2*>(a.Ph) + (long long)(pix >= 0 ? pix : 0) * a.ph_stride;
  for (int f0 = 0; f0 < a.Nf; f0 += 2) {  // (a frequency per half of the wave, which stays together)
    const int f = min(f0 + (ln >> 5), a.Nf - 1);
    const float2 p = row[f], wf = ws[f];
    if (__ballot(p.x * wf.x - p.y * wf.y != 0.f || p.x * wf.y + p.y * wf.x != 0.f) != 0ull) return false;
  }
  return true;
}

template <int KSP, int DT, bool DATA4>
__global__ __launch_bounds__(256, KSP == SP_F32 && DT == 1 ? 3 : 1) void rsd_propagate_mfma(RsdPropArgs a) {
  using F = PropFmt<KSP>;
  using M = Mfma<F::SP>;
  constexpr int NPL = F::NPL, NT = F::NT, FL = F::FL, FS = 2 * FL;
  extern __shared__ float2 ws[];  // weights w_f, zero from Nf to the last step's end
  clear_image(a);
  const int lane = threadIdx.x & 63;
  const int hl = lane >> 5, c32 = lane & 31;
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int Nf = a.Nf, Nd = a.Nd;
  const int ns = (Nf + FS - 1) / FS;
  for (int f = threadIdx.x; f < FS * ns; f += 256) ws[f] = f < Nf ? a.w[f] : make_float2(0.f, 0.f);
  __syncthreads();
  const int nds = (Nd + 32 * DT - 1) / (32 * DT);
  // blocks go round-robin over the 8 XCDs: those of the active chunks (the first nactive) are
  // dealt so that an XCD's L2 sees neighbouring chunks, which share kernel rows
  unsigned b = blockIdx.x;
  const unsigned nb8 = (unsigned)(2 * a.nactive * nds / kWavesPerBlock) & ~7u;
  if (b < nb8) b = (b & 7u) * (nb8 >> 3) + (b >> 3);
  const long long w = (long long)b * kWavesPerBlock + wib;
  if (w >= 2 * a.nchunks * nds) return;
  const long long gh = w / nds;  // half chunk
  const int d0 = (int)(w % nds) * 32 * DT;
  const int i0 = a.chunk_i0[gh >> 1];
  const int* pixs = a.chunk_pix + gh * 32;
  if (pixs[0] < 0) return;  // slots fill in order: an empty half
  const int pix = pixs[c32];
  float wa = a.chunk_wa[gh * 32 + c32], wb = a.chunk_wb[gh * 32 + c32];
  mf_acc acc[NT][DT][2];  // [tap][depth tile][re | im]
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < DT; ++q)
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][q][o][v] = 0.f;
  int out_exp = 0;  // C = acc 2^out_exp (before its own storage scale)
  if (i0 >= 0) {
    const int i1 = i0 + 1 < a.cut_idx ? i0 + 1 : a.cut_idx;
    using PRaw = typename std::conditional<DATA4, unsigned int, float2>::type;
    const PRaw* row = static_cast<const PRaw*>(a.Ph) + (long long)(pix >= 0 ? pix : 0) * a.ph_stride;
    auto cvp = [&](PRaw r) {
      if constexpr (DATA4) return M::unpack(r);
      else return r;
    };
    auto cm = [](float2 p, float2 wf) { return make_float2(p.x * wf.x - p.y * wf.y, p.x * wf.y + p.y * wf.x); };
    float ta = wa, tb = wb;  // tap weights ahead of the rounding (times 2^e)
    if constexpr (KSP == SP_F16) {
      float m = 0.f;
      constexpr int U = 8;  // loads in flight per lane (a repeated last frequency does not change
                            // the maximum); the two lane halves take a part of the row each
      for (int f0 = hl * U; f0 < Nf; f0 += 2 * U) {
        PRaw p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) p[u] = row[min(f0 + u, Nf - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float2 z = cm(cvp(p[u]), ws[min(f0 + u, Nf - 1)]);
          m = fmaxf(m, fmaxf(fabsf(z.x), fabsf(z.y)));
        }
      }
      m *= fmaxf(wa, wb);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
      int ex = 0;
      if (m > 0.f) (void)frexpf(m, &ex);  // m < 2^ex
      // clamped so that the scaled tap weights (<= 1) and 2^-e stay finite normal floats
      const int e = min(max(14 - ex, -100), 100);
      out_exp = -e;
      ta = ldexpf(wa, e);
      tb = ldexpf(wb, e);
    }
    // the lane's kernel operands (groups of FL frequencies): plane pl, depth tile q
    typedef unsigned int bv __attribute__((ext_vector_type(FL)));
    const bv* kr = static_cast<const bv*>(a.Kr);
    const long long npl = a.kr_plane / FL;
    const int ng = 2 * ((Nf + 7) / 8) * (4 / FL);  // groups in a row of the table
    const long long k0 = ((long long)i0 * ng + hl) * Nd, k1 = ((long long)i1 * ng + hl) * Nd;
    int dq[DT];
#pragma unroll
    for (int q = 0; q < DT; ++q) dq[q] = min(d0 + 32 * q + c32, Nd - 1);
    struct Step {
      PRaw p[FL];
      bv b[2][NPL][DT];  // [tap][plane][depth tile]
    };
    auto load = [&](int s) {
      Step t;
      s = min(s, ns - 1);
#pragma unroll
      for (int j = 0; j < FL; ++j) t.p[j] = row[min(FS * s + FL * hl + j, Nf - 1)];
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl)
#pragma unroll
        for (int q = 0; q < DT; ++q) {
          t.b[0][pl][q] = kr[pl * npl + k0 + (long long)(2 * s) * Nd + dq[q]];
          t.b[1][pl][q] = kr[pl * npl + k1 + (long long)(2 * s) * Nd + dq[q]];
        }
      return t;
    };
    auto mul = [&](mf_u4 A, mf_u4 B, mf_acc* c) {
      c[0] = M::mma(prop_re(A), B, c[0]);
      c[1] = M::mma(prop_im(A), B, c[1]);
    };
    auto step = [&](const Step& t, int s) {
      float2 z[FL];
#pragma unroll
      for (int j = 0; j < FL; ++j) z[j] = cm(cvp(t.p[j]), ws[FS * s + FL * hl + j]);
      if constexpr (NPL == 3) {
        mf_u4 A[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            A[pl][j] = M::pack(z[j].x, z[j].y);
            if (pl < 2) {
              const float2 r = M::unpack(A[pl][j]);
              z[j] = make_float2(z[j].x - r.x, z[j].y - r.y);
            }
          }
        constexpr int pa[6] = {2, 1, 0, 1, 0, 0}, pb[6] = {0, 1, 2, 0, 1, 0};  // the small products first
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
          for (int tap = 0; tap < 2; ++tap)
#pragma unroll
            for (int q = 0; q < DT; ++q) mul(A[pa[i]], t.b[tap][pb[i]][q], acc[tap][q]);
      } else {
        const mf_u4 A = {M::pack(z[0].x * ta, z[0].y * ta), M::pack(z[0].x * tb, z[0].y * tb),
                         M::pack(z[1].x * ta, z[1].y * ta), M::pack(z[1].x * tb, z[1].y * tb)};
#pragma unroll
        for (int q = 0; q < DT; ++q) {
          const bv b0 = t.b[0][0][q], b1 = t.b[1][0][q];
          mul(A, mf_u4{b0[0], b1[0], b0[1], b1[1]}, acc[0][q]);
        }
      }
    };
    Step b0 = load(0), b1 = load(1);
    // (both steps of a round unconditional: loads that feed a conditional step are moved into
    // it, next to their use)
    for (int s = 0; s + 1 < ns; s += 2) {
      step(b0, s);
      b0 = load(s + 2);
      __builtin_amdgcn_sched_barrier(0);  // (the loads stay ahead of the step they overlap)
      step(b1, s + 1);
      b1 = load(s + 3);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (ns & 1) step(b0, ns - 1);
    if constexpr (NPL == 3) {
      float m = 0.f;  // the lane's largest sum in magnitude (NaN if one is)
#pragma unroll
      for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int q = 0; q < DT; ++q)
#pragma unroll
          for (int t = 0; t < 2; ++t)
            m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, fabsf(acc[t][q][0][v])), fabsf(acc[t][q][1][v]));
      bool whole = __ballot(!(m <= kSplitMax)) != 0ull;
      if (!whole && __ballot(m >= kSplitMin) == 0ull)  // (all sums zero: of zeros, or too small for any product)
        whole = __ballot(m > 0.f) != 0ull || !all_zero(a, ws, gh);
      const float sc = ldexpf(1.f, a.kr_exp);
      wa *= sc;
      wb *= sc;
      if (whole) {
#pragma unroll
        for (int q = 0; q < DT; ++q)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[1][q][0][v] = acc[1][q][1][v] = 0.f;
        propagate_f32<DT>(a, ws, gh, d0, i0, i1, acc[0]);
        wa = 1.f;  // (acc[0] is the whole sum)
        wb = 0.f;
      }
    }
  }
  // D lane layout: rows 8(v/4) + 4 hl + v%4 of the tile, column c32
  int qexp[DT];  // final exponent per depth tile column: the half chunk's scale, and for FP16
                 // data the stored P^ scale (undone) and C's storage scale at that depth
#pragma unroll
  for (int q = 0; q < DT; ++q) {
    const int d = min(d0 + 32 * q + c32, Nd - 1);
    qexp[q] = out_exp;
    if constexpr (DATA4 && KSP == SP_F16) qexp[q] += a.e_c[d] - a.e_ph[0];
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = 8 * (v >> 2) + 4 * hl + (v & 3);
    const int pp = __shfl(pix, r, 64);
    const float ra = NT == 2 ? __shfl(wa, r, 64) : 0.f, rb = NT == 2 ? __shfl(wb, r, 64) : 0.f;
#pragma unroll
    for (int q = 0; q < DT; ++q) {
      const int d = d0 + 32 * q + c32;
      float re = acc[0][q][0][v], im = acc[0][q][1][v];
      if constexpr (NT == 2) {
        re = fmaf(ra, re, rb * acc[1][q][0][v]);
        im = fmaf(ra, im, rb * acc[1][q][1][v]);
      } else if constexpr (KSP == SP_F16) {
        re = ldexpf(re, qexp[q]);
        im = ldexpf(im, qexp[q]);
      }
      if (pp >= 0 && d < Nd) {
        const long long o = (long long)pp * a.c_stride + d;
        if constexpr (DATA4) static_cast<unsigned int*>(a.C)[o] = M::pack(re, im);
        else static_cast<float2*>(a.C)[o] = make_float2(re, im);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// FP16 storage scales of the RSD intermediates
// ---------------------------------------------------------------------------
//
// L = sum |tau| bounds every phasor |P[f]| (a DFT of one pixel's line), and so also the x
// and y DFTs of the padded phasor planes (sums over pixels).  The propagated plane at
// depth d is bounded by L kappa_d with kappa_d = sum_f |w_f| max_i |K_r[i][f][d]| (the
// tap weights are at most 1), and its unnormalised y-IFFT by My L kappa_d.  Each is stored
// times 2^(14 - k) with bound = f 2^k, f in [0.5, 1), so stored magnitudes stay below
// 2^14: one exponent for P, X and P^, one per depth plane for C and for D.  L is summed in
// a fixed order, so the scales, and the results, are deterministic.

__global__ __launch_bounds__(256) void rsd_l1_partial(const float2* __restrict__ tau, long long n2,
                                                      float* __restrict__ partials) {
  __shared__ float red[4];
  float acc = 0.f;
  const long long stride = (long long)gridDim.x * 256;
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  for (; i + 3 * stride < n2; i += 4 * stride) {  // four loads in flight per thread
    const float2 v0 = tau[i], v1 = tau[i + stride], v2 = tau[i + 2 * stride], v3 = tau[i + 3 * stride];
    acc += ((fabsf(v0.x) + fabsf(v0.y)) + (fabsf(v1.x) + fabsf(v1.y))) +
           ((fabsf(v2.x) + fabsf(v2.y)) + (fabsf(v3.x) + fabsf(v3.y)));
  }
  for (; i < n2; i += stride) acc += fabsf(tau[i].x) + fabsf(tau[i].y);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__device__ __forceinline__ int rsd_storage_exponent(float bound) {
  if (!(bound > 0.f) || !(bound <= 3.0e38f)) return 0;
  int k = 0;
  (void)frexpf(bound, &k);
  return min(max(14 - k, -120), 120);
}

__global__ __launch_bounds__(256) void rsd_scale_exponents(const float* __restrict__ partials, int np,
                                                           const float* __restrict__ kappa, int nd, int l_my,
                                                           int* __restrict__ exps) {
  __shared__ float red[4];
  float acc = 0.f;
  for (int j = threadIdx.x; j < np; j += 256) acc += partials[j];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  const float L = (red[0] + red[1]) + (red[2] + red[3]);
  if (threadIdx.x == 0) exps[0] = rsd_storage_exponent(L);
  for (int d = threadIdx.x; d < nd; d += 256) {
    const int ec = rsd_storage_exponent(L * kappa[d]);
    exps[1 + d] = ec;
    exps[1 + nd + d] = ec - l_my;
  }
}

hipError_t launch_rsd_scales(const float* tau, long long n, float* partials, const float* kappa, int nd, int l_my,
                             int* exps, hipStream_t s) {
  if (n % 2 != 0 || nd < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rsd_l1_partial, dim3(kScaleBlocks), dim3(256), 0, s, reinterpret_cast<const float2*>(tau),
                     n / 2, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(rsd_scale_exponents, dim3(1), dim3(256), 0, s, partials, kScaleBlocks, kappa, nd, l_my, exps);
  return hipGetLastError();
}

hipError_t launch_rsd_propagate(const RsdPropArgs& a, hipStream_t s) {
  if (a.data_sp != SP_F32 && (a.data_sp != a.kernel_sp || !a.mfma)) return hipErrorInvalidValue;
  if (a.mfma) {
    // 32-depth tiles per wave: FP32 kernels 1 (three waves per SIMD; 76 us against 80 with two at
    // 128 x 128 x 1024), FP16 / BF16 2 (47 against 53)
    int dt = a.kernel_sp == SP_F32 ? 1 : 2;
    if (a.mfma == 2) dt = 3 - dt;
    if (a.Nd <= 32) dt = 1;
    const long long waves = 2 * a.nchunks * ((a.Nd + 32 * dt - 1) / (32 * dt));
    const long long blocks = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = sizeof(float2) * 8 * (size_t)((a.Nf + 7) / 8);
    auto go = [&](auto k) {
      hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), lds, s, a);
      return hipGetLastError();
    };
    const bool d4 = a.data_sp != SP_F32;
    if (a.kernel_sp == SP_F32) return dt == 1 ? go(rsd_propagate_mfma<SP_F32, 1, false>) : go(rsd_propagate_mfma<SP_F32, 2, false>);
    if (a.kernel_sp == SP_F16) {
      if (d4) return dt == 1 ? go(rsd_propagate_mfma<SP_F16, 1, true>) : go(rsd_propagate_mfma<SP_F16, 2, true>);
      return dt == 1 ? go(rsd_propagate_mfma<SP_F16, 1, false>) : go(rsd_propagate_mfma<SP_F16, 2, false>);
    }
    if (d4) return dt == 1 ? go(rsd_propagate_mfma<SP_BF16, 1, true>) : go(rsd_propagate_mfma<SP_BF16, 2, true>);
    return dt == 1 ? go(rsd_propagate_mfma<SP_BF16, 1, false>) : go(rsd_propagate_mfma<SP_BF16, 2, false>);
  }
  const long long nds = (a.Nd + kDepths - 1) / kDepths;
  const long long waves = a.nchunks * nds;
  const long long blocks = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  if (a.kernel_sp == SP_F16)
    hipLaunchKernelGGL(rsd_propagate<SP_F16>, dim3((unsigned)blocks), dim3(256), 0, s, a);
  else if (a.kernel_sp == SP_BF16)
    hipLaunchKernelGGL(rsd_propagate<SP_BF16>, dim3((unsigned)blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(rsd_propagate<SP_F32>, dim3((unsigned)blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace nlos
