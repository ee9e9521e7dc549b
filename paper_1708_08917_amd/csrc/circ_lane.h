// FC forward for short blocks (K = 4..32) and more than two vectors, in one launch: every transform
// lives in the registers of one lane.
//
// A block of K <= 32 values is short enough for one lane to hold and transform, and the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32 wants, per lane, exactly one element of a 4-deep slab of the
// reduction: lane l supplies A(m = l % 16, k = l / 16) and B(k = l / 16, n = l % 16).  So a wave takes
// 16 output block rows x 16 batch rows and walks over the input blocks four at a time: lane (n, kk) takes
// block j = 4s + kk of batch row n (K consecutive values), transforms it, and what it then holds
// is its B operand of every frequency - no exchange between the passes of a transform, no operand rows in LDS
// and no barrier before the end of the reduction.  The weight operand of a step is one complex value per frequency
// and lane, from the plain spectrum sections.  Per step one product of 16x16x4 for each of the
// two real bins and four for each of the K/2 - 1 complex ones: 2 + 4 (K/2 - 1) instructions of 32 cycles.
//
// The W waves of a workgroup own the same tile and take every W-th step of the reduction; their
// sums meet in LDS once, at the end, added in wave order, and one thread per (block row, batch row)
// inverts its spectrum in registers, adds the bias, applies the ReLU and stores K consecutive values.
//
// What bounds it: fp32 matrix instructions and vector instructions of a SIMD, which take turns (counters at
// 64 x 2048 blocks of 8, batch 64: matrix cores busy 45 %, and a step measures the sum of the two whatever
// their order in the code): 448 + 184 cycles per step at K = 8, 960 + 470 at 16, 1984 + 1250 at 32 (the vector part
// with a half-length complex transform; RealFft, circ_fftreg.h, has fewer additions: 2 to 4 % of a call).  Hence
//  - x by 16-byte pieces along the rows and a transposition through LDS: a lane per batch row, straight
//    from memory, costs a cache access per lane (29 per instruction; 18.2 -> 16.5 us at 125 x 512 blocks of 8,
//    batch 256),
//  - buffer descriptors instead of pointers (16.4 -> 14.8 us: the address arithmetic was a third of the
//    vector instructions),
//  - two tiles of block rows per workgroup where there are enough of them: the transform of x then serves
//    twice the products (32 x 1024 blocks of 16, batch 512: 59.5 -> 31.4 us),
//  - slices of the reduction in a second launch where there are few (64 x 2048 blocks of 8, batch 64:
//    42.9 -> 13.8 us; 125 x 512 batch 256: 14.8 -> 12.7 us).
// Dropped: the transform of step t+1 between the matrix instructions of step t (no faster, twice the code).
#pragma once

#include <hip/hip_runtime.h>

#include "circ_fused.h"
#include "circ_kernels.h"

namespace circ {

typedef float lanefx4 __attribute__((ext_vector_type(4)));
typedef unsigned laneux2 __attribute__((ext_vector_type(2)));
typedef unsigned laneux4 __attribute__((ext_vector_type(4)));

constexpr int kBufferFlags = 0x00027000;   // raw buffer descriptor, 32-bit data

// K block size; W waves per workgroup.
template <int K, int MI>
struct LaneShape {
  static constexpr int W = K == 32 || MI == 2 ? 4 : 8;
  static constexpr bool TWO_W = K * MI < 32;      // two sets of weight registers
  static constexpr int NT = 64 * W;
  // sums in LDS: [wave][component][lane][4 rows], the four 16-lane groups of a component 16 words apart
  // (mod 64), so that both the 16-byte stores and the reads of the last stage (16 block rows x 4
  // batch rows per wave) touch every bank once
  static constexpr int CW = 4 * 64 + 3 * 16;
  // (the staging buffers of x, 2 x 16 rows x 4 blocks per wave, are the smaller use of the same memory)
  static constexpr size_t lds_bytes() { return size_t(W) * K * CW * sizeof(float); }
  static_assert(CW >= 2 * 16 * 4, "staging buffers fit");
};

// Inverse transform, bias and ReLU of one output block (block row io of batch row bo) from its spectrum
// (in the order of RealFft).
template <int K, int HM>
__device__ __forceinline__ void lane_store(const float (&Y)[K], const float* __restrict__ bias, void* __restrict__ yv, int p, int bo,
                                           int io, int relu) {
  float v[K];
  RealFft<K>::inverse(Y, v);
  constexpr float scale = HM != 0 ? 1.0f / float(K) : 1.0f;    // (fp32 spectra carry the 1/K)
  const long long dst = (long long)bo * ((long long)p * K) + (long long)io * K;
#pragma unroll
  for (int u = 0; u < K / 4; ++u) {
    float4 t = make_float4(scale * v[4 * u], scale * v[4 * u + 1], scale * v[4 * u + 2], scale * v[4 * u + 3]);
    if (bias) {
      const float4 bb = reinterpret_cast<const float4*>(bias + (long long)io * K)[u];
      t.x += bb.x;
      t.y += bb.y;
      t.z += bb.z;
      t.w += bb.w;
    }
    if (relu) {
      t.x = fmaxf(t.x, 0.f);
      t.y = fmaxf(t.y, 0.f);
      t.z = fmaxf(t.z, 0.f);
      t.w = fmaxf(t.w, 0.f);
    }
    if constexpr (HM != 0) store_half4<HM == 2>(static_cast<unsigned short*>(yv) + dst + 4 * u, t);
    else reinterpret_cast<float4*>(static_cast<float*>(yv) + dst)[u] = t;
  }
}

// LDS accesses of a wave execute in program order; this keeps the compiler to that order across lanes.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// W^: fp32 (HM == 0) the spectrum section [f][j][i], which carries the 1/K; 16-bit storage (HM 1: fp16, 2:
// bfloat16) the section of the other direction, conj(W^)[f][j][i] as 16-bit pairs, not normalised: i is the
// fastest index of either, so a step's weights of one frequency are four runs of 16 values.
// x [B][q*K], y [B][p*K].  MI: tiles of 16 block rows per workgroup.  nt: steps per wave.
// Grid: (tiles, slices of the reduction).  With more than one slice `part` receives each slice's sums,
// [slice][tile][component][batch row][block row] (MI = 1), which lane_finish_kernel adds in order.
//
// x and W^ are read through buffer descriptors: a scalar base and a 32-bit offset per lane that one addition
// moves to the next step, and x of the input blocks past q reads as zero by the descriptor's bounds
// check.  The host keeps 16 rows of x and the spectrum section below 2^31 bytes.
template <int K, int MI, int HM>
__global__ __launch_bounds__((LaneShape<K, MI>::NT)) void fc_lane_kernel(const void* __restrict__ Wv, const void* __restrict__ xv,
                                                                   const float* __restrict__ bias, void* __restrict__ yv, int p, int q,
                                                                   int B, FusedTileMap tm, int relu, float* __restrict__ part, int nt) {
  using Sh = LaneShape<K, MI>;
  constexpr int W = Sh::W, CW = Sh::CW, NF = K / 2 + 1;
  constexpr bool BF = HM == 2;
  using WT = typename std::conditional<HM != 0, unsigned, laneux2>::type;
  constexpr unsigned ESZ = HM != 0 ? 2 : 4;                     // bytes of a value of x
  constexpr int CPR = K * int(ESZ) / 4, NL = CPR / 4;           // 16-byte pieces per row and step, loads per lane and step
  extern __shared__ __attribute__((aligned(16))) float lane_smem[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned xcd = blockIdx.x & 7u, local = blockIdx.x >> 3;
  const unsigned lq = tm.ni > 1 ? __umulhi(local, tm.ni_magic) : local;
  const int it = int(xcd & ((1u << tm.xa_shift) - 1u)) * tm.ni + int(local - lq * unsigned(tm.ni));
  const int bt = int(xcd >> tm.xa_shift) * tm.nb + int(lq);
  if (int(lq) >= tm.nb || it >= tm.n_it || bt >= tm.n_bt) return;
  const int i0 = it * (16 * MI), b0 = bt * 16;
  const int n16 = lane & 15, kk = lane >> 4;

  // Weights: lane (m, kk) takes block row i0 + m of input block 4s + kk.  Block rows and input blocks past
  // the edge are clamped: the sums of the former are never stored, the latter meet an x of zero.
  const unsigned wplane = unsigned(p) * unsigned(q) * unsigned(sizeof(WT));   // bytes of one frequency
  const auto wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(Wv), short(0), int(wplane * NF), kBufferFlags);
  const int j0 = 4 * (int(blockIdx.y) * nt * W + wave);         // first input block of this wave
  unsigned woff[MI], wlast[MI];
#pragma unroll
  for (int m = 0; m < MI; ++m) {
    const unsigned i = unsigned(min(i0 + 16 * m + n16, p - 1));
    woff[m] = (unsigned(j0 + kk) * unsigned(p) + i) * unsigned(sizeof(WT));
    wlast[m] = (unsigned(q - 1) * unsigned(p) + i) * unsigned(sizeof(WT));
  }
  const unsigned wstep = 4u * W * unsigned(p) * unsigned(sizeof(WT));
  struct WStep {
    WT w[MI][NF];
  };
  auto load_w = [&](WStep& s) {                                 // this wave's next step
#pragma unroll
    for (int m = 0; m < MI; ++m) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const unsigned o = min(woff[m], wlast[m]);
        if constexpr (HM != 0) s.w[m][f] = __builtin_amdgcn_raw_buffer_load_b32(wrsrc, int(o), int(f * wplane), 0);
        else s.w[m][f] = __builtin_amdgcn_raw_buffer_load_b64(wrsrc, int(o), int(f * wplane), 0);
      }
      woff[m] += wstep;
    }
  };

  // x: a step's 16 rows x 4 blocks are 16 runs of CPR 16-byte pieces.  Lanes load along the runs (a lane per
  // batch row, as the matrix instruction wants them, would cost one cache access per lane) and
  // transpose through a buffer of the wave's own; the pieces of row r lie in the order slot = piece ^
  // (r mod CPR), so that neither the stores nor the reads conflict.
  const unsigned xrow = unsigned(q) * K * ESZ;                  // bytes of a row
  const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(static_cast<const char*>(xv)) + (long long)b0 * xrow, short(0), int(unsigned(min(16, B - b0)) * xrow), kBufferFlags);
  unsigned xoff[NL], xend[NL];                                  // xend: byte of the row from which block j >= q
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    const unsigned r = unsigned(u * 64 + lane) / CPR, piece = (unsigned(u * 64 + lane) % CPR) ^ (r & (CPR - 1));
    xoff[u] = r * xrow + piece * 16 + unsigned(j0) * (K * ESZ);
    xend[u] = (r + 1) * xrow;
  }
  auto load_x = [&](laneux4 (&s)[NL]) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      s[u] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, int(xoff[u] < xend[u] ? xoff[u] : 0x80000000u), 0, 0);
      xoff[u] += 4 * K * ESZ * W;
    }
  };
  laneux4* xbuf = reinterpret_cast<laneux4*>(lane_smem) + wave * (2 * 64 * NL);
  auto stage_x = [&](const laneux4 (&s)[NL], int half) {
#pragma unroll
    for (int u = 0; u < NL; ++u) xbuf[half * (64 * NL) + u * 64 + lane] = s[u];
  };
  auto transform = [&](int half, float (&X)[K]) {
    float v[K];
    const laneux4* row = xbuf + half * (64 * NL) + n16 * CPR;
#pragma unroll
    for (int u = 0; u < CPR / 4; ++u) {
      const laneux4 c = row[(kk * (CPR / 4) + u) ^ (n16 & (CPR - 1))];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (HM != 0) {
          const float2 a = unpack_pair16<BF>(c[e]);
          v[8 * u + 2 * e] = a.x;
          v[8 * u + 2 * e + 1] = a.y;
        } else {
          v[4 * u + e] = __uint_as_float(c[e]);
        }
      }
    }
    RealFft<K>::forward(v, X);
  };

  // fp32, longest blocks: the products with the imaginary part of the weights have sums of their own (acc2), joined with
  // the others at the end: half as long chains, whose rounding errors are smaller.  The fused kernel, which this one
  // replaces at K = 32, sums the same way: relative error against float64 1.62e-7 there, 1.70e-7 here in one chain, 1.58e-7
  // apart (2112 -> 1280, batch 700; 0.5 us of 18 for the longer start and end).  Shorter blocks replace the three-kernel
  // route, whose one chain is longer.
  constexpr bool APART = K == 32 && HM == 0;
  lanefx4 acc[MI][K], acc2[APART ? MI : 1][APART ? K : 1];
#pragma unroll
  for (int m = 0; m < MI; ++m)
#pragma unroll
    for (int c = 0; c < K; ++c) {
      acc[m][c] = lanefx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (APART) acc2[m][c] = lanefx4{0.f, 0.f, 0.f, 0.f};
    }
  auto multiply = [&](const WStep& s, const float (&X)[K]) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
      for (int m = 0; m < MI; ++m) {
        lanefx4(&a)[K] = acc[m];
        float wr, wi;
        if constexpr (HM != 0) {
          const float2 c = unpack_pair16<BF>(s.w[m][f]);
          wr = c.x;
          wi = c.y;
        } else {
          wr = __uint_as_float(s.w[m][f][0]);
          wi = __uint_as_float(s.w[m][f][1]);
        }
        if (f == 0) {
          a[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr, X[0], a[0], 0, 0, 0);
        } else if (f == K / 2) {
          a[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr, X[1], a[1], 0, 0, 0);
        } else {
          // (wr + i wi) X, or (wr - i wi) X where the section holds conjugates
          a[2 * f] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr, X[2 * f], a[2 * f], 0, 0, 0);
          a[2 * f + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr, X[2 * f + 1], a[2 * f + 1], 0, 0, 0);
          if constexpr (APART) {
            lanefx4(&b)[K] = acc2[m];
            b[2 * f] = __builtin_amdgcn_mfma_f32_16x16x4f32(wi, X[2 * f + 1], b[2 * f], 0, 0, 0);
            b[2 * f + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wi, X[2 * f], b[2 * f + 1], 0, 0, 0);
            continue;
          }
          a[2 * f] = __builtin_amdgcn_mfma_f32_16x16x4f32(wi, HM != 0 ? X[2 * f + 1] : -X[2 * f + 1], a[2 * f], 0, 0, 0);
          a[2 * f + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wi, HM != 0 ? -X[2 * f] : X[2 * f], a[2 * f + 1], 0, 0, 0);
        }
      }
    }
  };

  // Step t: x of step t+1 into LDS, the loads of x of step t+2 and of the weights of step t+1 (longest
  // blocks: of step t, with the transform in front of their use), spectra of step t from LDS, products.
  laneux4 xs[NL];
  auto step = [&](const WStep& cur, WStep& next, int half) {
    load_w(next);
    stage_x(xs, half ^ 1);
    load_x(xs);
    wave_fence();
    float X[K];
    transform(half, X);
    // longest blocks: unpacked weights and spectra of the two parts together would not fit the registers (192 moves
    // between the two register files per step without this)
    if constexpr (K == 32) __builtin_amdgcn_sched_barrier(0);
    multiply(cur, X);
  };
  load_x(xs);
  if constexpr (Sh::TWO_W) {
    WStep w0, w1;
    load_w(w0);
    stage_x(xs, 0);
    load_x(xs);
#pragma unroll 1
    for (int t = 0; t < nt; t += 2) {
      step(w0, w1, 0);
      if (t + 1 >= nt) break;
      step(w1, w0, 1);
    }
  } else {
    WStep w0;
    stage_x(xs, 0);
    load_x(xs);
#pragma unroll 1
    for (int t = 0; t < nt; ++t) step(w0, w0, t & 1);
  }

  // The sums of the waves, one tile of 16 block rows after the other.
#pragma unroll
  for (int m = 0; m < MI; ++m) {
    if constexpr (APART) {
#pragma unroll
      for (int f = 1; f < K / 2; ++f) {
        acc[m][2 * f] -= acc2[m][2 * f];
        acc[m][2 * f + 1] += acc2[m][2 * f + 1];
      }
    }
    __syncthreads();                                            // the staging buffers / the tile before have been read
    float* mine = lane_smem + wave * (K * CW) + lane * 4 + kk * 16;
#pragma unroll
    for (int c = 0; c < K; ++c) *reinterpret_cast<lanefx4*>(mine + c * CW) = acc[m][c];
    __syncthreads();
    const int i = tid & 15, b = tid >> 4;                       // C layout: row i = 4 * (lane / 16) + r, column b = lane % 16
    const int io = i0 + 16 * m + i, bo = b0 + b;
    if (tid < 256 && io < p && bo < B) {
      const float* src = lane_smem + (i >> 2) * 80 + b * 4 + (i & 3);
      float Y[K];
#pragma unroll
      for (int c = 0; c < K; ++c) Y[c] = src[c * CW];
#pragma unroll 1
      for (int w = 1; w < W; ++w) {
        src += K * CW;
#pragma unroll
        for (int c = 0; c < K; ++c) Y[c] += src[c * CW];
      }
      if (part) {
        float* dst = part + ((size_t(blockIdx.y) * (unsigned(tm.n_it) * unsigned(tm.n_bt)) + unsigned(bt) * unsigned(tm.n_it) + unsigned(it)) * K) * 256;
#pragma unroll
        for (int c = 0; c < K; ++c) dst[c * 256 + tid] = Y[c];
        return;
      }
      lane_store<K, HM>(Y, bias, yv, p, bo, io, relu);
    }
  }
}

// The sums of nparts slices, added in order; inverse transform and epilogue.  Grid (tiles), 256 threads.
template <int K, int HM>
__global__ __launch_bounds__(256) void lane_finish_kernel(const float* __restrict__ part, const float* __restrict__ bias,
                                                          void* __restrict__ yv, int p, int B, int n_it, int nparts, int relu) {
  const int tid = threadIdx.x, bt = int(blockIdx.x) / n_it, it = int(blockIdx.x) - bt * n_it;
  const int io = it * 16 + (tid & 15), bo = bt * 16 + (tid >> 4);
  if (io >= p || bo >= B) return;
  const float* src = part + size_t(blockIdx.x) * (K * 256) + tid;
  float Y[K];
#pragma unroll
  for (int c = 0; c < K; ++c) Y[c] = src[c * 256];
  const size_t ps = size_t(gridDim.x) * (K * 256);
  // A tile has one workgroup, so the loads have to overlap: U slices, 64 values, are requested before the first of them is
  // added, then the rest in smaller groups (left to itself the compiler waits for every value at K = 32: 16 slices
  // 35.6 us, about 8 in this form).
  constexpr int U = 64 / K;
  int s = 1;
  auto add = [&](auto count) {
    constexpr int N = decltype(count)::value;
    float t[N][K];
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int c = 0; c < K; ++c) t[u][c] = (src + size_t(s + u) * ps)[c * 256];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int c = 0; c < K; ++c) Y[c] += t[u][c];
    s += N;
  };
  while (s + U <= nparts) add(std::integral_constant<int, U>{});
  if constexpr (U > 8) { if (s + 8 <= nparts) add(std::integral_constant<int, 8>{}); }
  if constexpr (U > 4) { if (s + 4 <= nparts) add(std::integral_constant<int, 4>{}); }
  if constexpr (U > 2) { if (s + 2 <= nparts) add(std::integral_constant<int, 2>{}); }
  if (s < nparts) add(std::integral_constant<int, 1>{});
  lane_store<K, HM>(Y, bias, yv, p, bo, io, relu);
}

}  // namespace circ
