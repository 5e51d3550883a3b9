// HIP kernels for gfx950 (CDNA4) of the vectorised per-object training step.
//
// Work decomposition. A batch holds the rays of many objects, segmented by CSR offsets. Each
// object's rays are cut into tiles of `rays_per_tile` consecutive rays; a tile never straddles
// two objects and its boundaries are relative to the object's first ray, so an object's result
// does not depend on the other objects in the batch. One workgroup processes one tile at a time
// (grid-stride, so the launch may be persistent). Inside a tile, each 64-lane wave takes
// sub-tiles of floor(64 / S) whole rays: the S samples of a ray occupy S consecutive lanes.
//
// Per sub-tile a wave of the width-32 kernel runs, without leaving registers except for the weight
// gradients' operands, which pass through LDS (hidden 64 and 128 in BF16 have kernels of their own,
// hidden 256 and up a chain of launches):
//   1. point normalisation in FP64, rounded once to FP32, and Gaussian Fourier features
//      (object-level encoding, supplement Sec. B);
//   2. the MLP on MFMA, both passes of 32 samples together, features on the M axis and samples
//      on the N axis, so each layer's accumulator layout is directly the next layer's B operand (the K axis
//      is permuted consistently in the weights instead of moving data);
//   3. occupancy rendering of Eq. 3 with ray-segmented wavefront scans: an exclusive
//      multiplicative scan of (1 - o) and additive scans for the rendered sums;
//   4. the masked L1 losses of Eqs. 4-7;
//   5. the adjoint of rendering: with g_i the derivative of the loss with respect to the
//      termination probability T_i, dL/do_i = P_i g_i - R_i / (1 - o_i) where R_i = sum over the
//      ray's later samples of g_j T_j (a reverse scan); the logit's adjoint
//      o_i ((1 - o_i) g_i P_i - R_i) needs no division;
//   6. the MLP backward: dX products on MFMA from the accumulator layout, dW products on MFMA
//      after an LDS transpose, accumulated in registers across the wave's sub-tiles.
// The waves of a workgroup then add their gradients in a fixed order and write one partial
// per tile; a second kernel sums each object's tile partials in tile order (no float atomics,
// bitwise reproducible), and a third applies Adam per object.
//
// Precision. Both modes use the sine/cosine of vmap_math.h (error below 2.5e-7; the hardware
// v_sin/v_cos approximations were tried for BF16 and moved enough features across BF16 rounding
// boundaries to show in the gradients) and the hardware exp2 and reciprocal for the logistic.
// FP32 mode uses v_mfma_f32_32x32x2f32. BF16 mode rounds weights, activations and
// back-propagated deltas to BF16 (round to nearest even) where they enter a product and uses
// v_mfma_f32_32x32x16_bf16 with FP32 accumulation; encoding, head activations, rendering,
// losses, reductions and Adam stay FP32.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "vmap_internal.h"
#include "vmap_math.h"
#include "vmap_bf16.h"

namespace vmapi {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Accumulator row held in register r (0..15) by lanes of half h (0, 1) of a 32x32 MFMA tile.
// The same map orders the K axis: K slot (h, r) of a block carries feature rowof(r, h).
__host__ __device__ constexpr int rowof(int r, int h) { return ((r >> 2) << 3) + (h << 2) + (r & 3); }
// Position of feature c (0..31) of a block in the permuted weight-column order.
__host__ __device__ constexpr int colpos(int c) { return (((c >> 2) & 1) << 4) + ((c >> 3) << 2) + (c & 3); }

__device__ __forceinline__ void wave_lds_sync() {
  // Orders this wave's LDS accesses across lanes: the compiler may not move LDS loads or stores
  // across it, and the wave waits until its own LDS operations have completed.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  asm volatile("" ::: "memory");
}

// Keeps the compiler from moving LDS accesses across it. A wave's LDS instructions execute in
// order, so its reads see its own earlier writes (any lane's) without a wait.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

// BF16 operand tiles of the weight-gradient products are staged sample-major: row s (a sample)
// holds the tile's features, TR_STRIDE elements apart. A lane writes its accumulator-layout
// values as 8-byte runs of four consecutive features, and ds_read_b64_tr_b16 regroups them: in
// each group of 16 lanes, lane 4a + b receives element b of the 8-byte chunks addressed by lanes
// a, a + 4, a + 8 and a + 12 of its group (checked on the device), so four lanes that address
// four consecutive rows at the same feature offset hand each of their readers one feature's four
// consecutive samples.
constexpr int kTrStride = 36;  // BF16 elements per staged row (32 features + 4: 8-byte rows)

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));

// Eight BF16 (two transposing reads, the second four rows further down) as one MFMA operand.
__device__ __forceinline__ bf16x8 tr_read8(const __bf16* p) {
  typedef __attribute__((address_space(3))) v4i16 lds_v4;
  const v4i16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p));
  const v4i16 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p + 4 * kTrStride));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Elements 0-3 of v to p and elements 4-7 to p + 8 (two 8-byte stores).
__device__ __forceinline__ void write_runs(__bf16* p, bf16x8 v) {
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u2w __attribute__((ext_vector_type(2)));
  const u4 w = __builtin_bit_cast(u4, v);
  *reinterpret_cast<u2w*>(p) = (u2w){w[0], w[1]};
  *reinterpret_cast<u2w*>(p + 8) = (u2w){w[2], w[3]};
}

// First tile of a workgroup. Workgroups are dealt to the eight XCDs in turn (workgroup b runs on
// XCD b mod 8, each with its own L2); when the grid has a workgroup per tile, the first n_tiles
// workgroups of one XCD take consecutive tiles, so that an object's tiles (its weights, rays and
// samples) share one L2 instead of being fetched into all eight. Workgroups past n_tiles (the
// last dispatched) stay without a tile. Otherwise tile = workgroup index (b of `blocks`).
__device__ __forceinline__ int first_tile_of_block(int b, int blocks, int n_tiles) {
  constexpr int kXcds = 8;
  if (blocks < n_tiles || b >= n_tiles) return b;
  const int x = b % kXcds;
  int start = 0;
  for (int y = 0; y < x; ++y) start += (n_tiles - y + kXcds - 1) / kXcds;  // workgroups of XCD y
  return start + b / kXcds;
}

// Unit and block of this workgroup in a one-dimensional grid of 8 ceil(units / 8) nblk
// workgroups (workgroups are dealt to the eight XCDs in turn by index): unit u goes to XCD u mod 8,
// and each XCD takes its units' nblk blocks one unit after another, so that the blocks of a unit
// (which share its rows and its object's weights) share one L2, and the units that exist (the
// first ones of a bound with slack) are spread evenly over the XCDs.
__device__ __forceinline__ void xcd_unit_block(int b, int nblk, int& unit, int& blk) {
  const int x = b & 7, s = b >> 3;
  unit = x + 8 * (s / nblk);
  blk = s % nblk;
}

// Logistic sigmoid from the hardware exponential and reciprocal (about 1 ulp each; an IEEE
// division costs a dozen instructions). exp(-z) overflows to +inf for z < -88, giving 0.
__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// sigma(z) and sigma(-z) = 1 - sigma(z) from one exponential e = exp(-z) (as 2^(-z log2 e), the
// hardware v_exp_f32): sigma(z) = 1 / (1 + e); sigma(-z) = e sigma(z) for z > 0 (e < 1) and
// 1 - sigma(z) for z <= 0 (sigma(z) <= 1/2, so no cancellation). e = inf for very negative z
// gives sigma(z) = 0 and sigma(-z) = 1.
__device__ __forceinline__ void sigm_pair(float z, float& sp, float& sn) {
  const float e = __builtin_amdgcn_exp2f(-z * 1.44269504088896341f);
  sp = __builtin_amdgcn_rcpf(1.0f + e);
  sn = (z > 0.f) ? e * sp : 1.0f - sp;
}

// Reads of a wide object's weight image in device memory through a buffer resource: the lane
// part of an offset sits in one VGPR and the block's constant part in an SGPR or the immediate,
// so unrolled loops need no 64-bit address per load.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t image_rsrc(const unsigned char* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), (short)0, bytes, 0x00020000);
}
__device__ __forceinline__ bf16x8 img_b128(__amdgpu_buffer_rsrc_t r, int lane_off, int off) {
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0));
}
__device__ __forceinline__ f32x4 img_f4(__amdgpu_buffer_rsrc_t r, int lane_off, int off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0));
}
__device__ __forceinline__ float img_f1(__amdgpu_buffer_rsrc_t r, int lane_off, int off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_off, off, 0));
}

// Activations of one 32-sample pass: NL + 1 layers (encoding first), H/32 blocks, D layout.
template <int H, bool BF>
struct Acts;
template <int H>
struct Acts<H, false> {
  float v[kLayers + 1][H / 32][16];
  __device__ __forceinline__ float get(int l, int b, int r) const { return v[l][b][r]; }
  __device__ __forceinline__ void set(int l, int b, int r, float x) { v[l][b][r] = x; }
  // registers r and r + 1 (r even)
  __device__ __forceinline__ void set2(int l, int b, int r, float x, float y) {
    v[l][b][r] = x;
    v[l][b][r + 1] = y;
  }
};
template <int H>
struct Acts<H, true> {
  bf16x8 v[kLayers + 1][H / 32][2];
  __device__ __forceinline__ float get(int l, int b, int r) const { return (float)v[l][b][r >> 3][r & 7]; }
  __device__ __forceinline__ void set(int l, int b, int r, float x) { v[l][b][r >> 3][r & 7] = (__bf16)x; }
  // registers r and r + 1 (r even), rounded as one packed pair
  __device__ __forceinline__ void set2(int l, int b, int r, float x, float y) {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    u4 w = __builtin_bit_cast(u4, v[l][b][r >> 3]);
    w[(r & 7) >> 1] = pack2(x, y);
    v[l][b][r >> 3] = __builtin_bit_cast(bf16x8, w);
  }
};

// Back-propagated deltas of one 32-sample pass in the accumulator layout. In BF16 mode they only
// ever enter products and LDS staging rounded to BF16, so they are kept rounded.
template <int H, bool BF>
struct Deltas;
template <int H>
struct Deltas<H, false> {
  float v[H / 32][16];
  __device__ __forceinline__ void set(int b, int r, float x) { v[b][r] = x; }
};
template <int H>
struct Deltas<H, true> {
  bf16x8 v[H / 32][2];
  __device__ __forceinline__ void set(int b, int r, float x) { v[b][r >> 3][r & 7] = (__bf16)x; }
};

// ---------------------------------------------------------------------------------------------
// Weight staging: object k's parameters -> LDS (permuted columns; BF16 in BF16 mode, plus the
// transposed copies that the backward's input-gradient products read as A operands). Threads
// tid, tid + nt, ... of the caller share the work; the destination may also be a weight image in
// device memory (wide models).

// Where stage_weights puts parameter p (value w) of a width-H object: the same bytes, one
// parameter at a time (BF16: with its transposed copy, or its bias's three pieces). The
// optimiser kernels keep the weight images current with it after each update.
template <int H, bool BF>
__device__ __forceinline__ void place_param(unsigned char* img, int p, float w) {
  constexpr LdsLayout L = lds_layout(H, BF, 1);
  using WT = typename std::conditional<BF, __bf16, float>::type;
  int off = 0;
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    const int K = (l == 0) ? kEnc : H;
    if (p < off + H * K) {
      const int e = p - off, row = e / K, col = e - row * K;
      reinterpret_cast<WT*>(img + L.w_off[l])[row * L.w_stride[l] + (col & ~31) + colpos(col & 31)] = (WT)w;
      if constexpr (BF && H == 32) {
        if (l > 0)
          reinterpret_cast<__bf16*>(img + L.wt_off[l])[col * (H + 8) + (row & ~31) + colpos(row & 31)] = (__bf16)w;
      }
      return;
    }
    off += H * K;
    if (p < off + H) {
      const int row = p - off;
      reinterpret_cast<float*>(img + L.b_off)[l * H + row] = w;
      if constexpr (BF && !weights_global(H)) {
        const __bf16 hi = (__bf16)w;
        const __bf16 mid = (__bf16)(w - (float)hi);
        const __bf16 lo = (__bf16)((w - (float)hi) - (float)mid);
        __bf16* dst = reinterpret_cast<__bf16*>(img + L.bA_off) + (size_t)(l * H + row) * 16;
        dst[0] = hi;
        dst[1] = mid;
        dst[2] = lo;
      }
      return;
    }
    off += H;
  }
  if (p < off + kOut * H) {
    const int e = p - off, c = e / H, col = e - c * H;
    if constexpr (BF) {
      reinterpret_cast<__bf16*>(img + L.whb_off)[c * (H + 8) + (col & ~31) + colpos(col & 31)] = (__bf16)w;
      reinterpret_cast<__bf16*>(img + L.whtb_off)[col * kOut + c] = (__bf16)w;
    } else {
      reinterpret_cast<float*>(img + L.wh_off)[c * (H + 4) + (col & ~31) + colpos(col & 31)] = w;
    }
    return;
  }
  off += kOut * H;
  reinterpret_cast<float*>(img + L.bh_off)[p - off] = w;
}

// A weight image fetched into LDS without registers: each wave's 64 lanes move 1 KiB blocks
// (global_load_lds_dwordx4: lane l's 16 bytes land at the wave-uniform LDS address + 16 l); the
// part past the last whole block goes through registers. The LDS writes complete under vmcnt, so
// readers wait for it (s_waitcnt) and a barrier.
__device__ __forceinline__ void fetch_image_lds(const unsigned char* src, unsigned char* dst, int bytes,
                                                int lane, int wave, int nw) {
  const int blocks = bytes >> 10;
  for (int b = wave; b < blocks; b += nw)
    __builtin_amdgcn_global_load_lds(src + (b << 10) + 16 * lane,
                                     (__attribute__((address_space(3))) void*)(dst + (b << 10)), 16, 0, 0);
  const int tail = (bytes - (blocks << 10)) >> 4;  // 16-byte pieces left
  if (wave == nw - 1 && lane < tail) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    *reinterpret_cast<u32x4*>(dst + (blocks << 10) + 16 * lane) =
        *reinterpret_cast<const u32x4*>(src + (blocks << 10) + 16 * lane);
  }
}

// src_hidden: the object's own width; an object of hidden 16 staged at H = 32 reads each slot of
// the width-32 layout from its own parameters (padded_index), zero for the padding.
template <int H, bool BF>
__device__ __forceinline__ void stage_weights(const float* __restrict__ th, unsigned char* smem, int tid, int nt,
                                              int src_hidden = H) {
  constexpr LdsLayout L = lds_layout(H, BF, 1);
  using WT = typename std::conditional<BF, __bf16, float>::type;
  const bool padded = (H == 32 && src_hidden == 16);
  auto param = [&](int q) -> float {
    if (padded) {
      const int p = unpadded_index16(q);
      return p >= 0 ? th[p] : 0.f;
    }
    return th[q];
  };
  int off = 0;
  float* bias = reinterpret_cast<float*>(smem + L.b_off);
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    const int K = (l == 0) ? kEnc : H;
    WT* W = reinterpret_cast<WT*>(smem + L.w_off[l]);
    const int ws = L.w_stride[l];
    for (int e = tid; e < H * K; e += nt) {
      const int row = e / K, col = e - row * K;
      const WT w = (WT)param(off + e);
      W[row * ws + (col & ~31) + colpos(col & 31)] = w;
      if constexpr (BF && H == 32) {
        if (l > 0) {  // W^T[col][row], rows of the transpose permuted like the forward's K axis
          __bf16* Wt = reinterpret_cast<__bf16*>(smem + L.wt_off[l]);
          Wt[col * (H + 8) + (row & ~31) + colpos(row & 31)] = w;
        }
      }
    }
    off += H * K;
    for (int e = tid; e < H; e += nt) bias[l * H + e] = param(off + e);
    off += H;
  }
  for (int e = tid; e < kOut * H; e += nt) {
    const int c = e / H, col = e - c * H;
    if constexpr (BF) {
      const __bf16 w = (__bf16)param(off + e);
      reinterpret_cast<__bf16*>(smem + L.whb_off)[c * (H + 8) + (col & ~31) + colpos(col & 31)] = w;
      reinterpret_cast<__bf16*>(smem + L.whtb_off)[col * kOut + c] = w;
    } else {
      reinterpret_cast<float*>(smem + L.wh_off)[c * (H + 4) + (col & ~31) + colpos(col & 31)] = param(off + e);
    }
  }
  off += kOut * H;
  float* bh = reinterpret_cast<float*>(smem + L.bh_off);
  for (int e = tid; e < kOut; e += nt) bh[e] = param(off + e);
  if constexpr (BF && !weights_global(H)) {
    // bias as an MFMA operand: b = hi + mid + lo exactly (three BF16 pieces of 8 bits each)
    __bf16* bA = reinterpret_cast<__bf16*>(smem + L.bA_off);
    int boff[kLayers];
    int o2 = 0;
#pragma unroll
    for (int l = 0; l < kLayers; ++l) {
      const int K = (l == 0) ? kEnc : H;
      boff[l] = o2 + H * K;
      o2 += H * K + H;
    }
    for (int e = tid; e < kLayers * H; e += nt) {
      const int l = e / H, row = e - l * H;
      const float b = param(boff[l] + row);
      const __bf16 hi = (__bf16)b;
      const __bf16 mid = (__bf16)(b - (float)hi);
      const __bf16 lo = (__bf16)((b - (float)hi) - (float)mid);
      __bf16* dst = bA + (size_t)e * 16;
      dst[0] = hi;
      dst[1] = mid;
      dst[2] = lo;
      for (int q = 3; q < 16; ++q) dst[q] = (__bf16)0.0f;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Forward of one 32-sample pass for the calling wave. xt: this lane's normalised point (the
// sample of column n = lane & 31; both lane halves hold the same point); Bm: the encoding matrix.
// ipe: xt[3] holds the sample's variance in the object frame; each feature is its expectation
// under the isotropic Gaussian (integrated positional encoding). Fills the activations
// and, with WITH_HEAD, returns the four output pre-activations z of sample n (valid in both lane
// halves).

template <int H, bool BF, bool WITH_HEAD>
__device__ __forceinline__ void forward_pass(const float xt[4], const unsigned char* smem,
                                             const float* Bm, Acts<H, BF>& A, float z[4],
                                             bool ipe = false) {
  constexpr int MT = H / 32;
  constexpr LdsLayout L = lds_layout(H, BF, 1);
  // Weights are re-read on every pass instead of being held in registers across passes. `smem`
  // is the weight base: the LDS staging, or a wide object's image in device memory.
  asm volatile("" ::: "memory");
  const int lane = threadIdx.x & 63, n = lane & 31, hf = lane >> 5;
  // Gaussian Fourier features: register r of block 0 holds feature rowof(r, hf):
  // r = 0..3 sin(phi[4hf + r]), 4..7 sin(phi[8 + 4hf + r - 4]), 8..15 the cosines.
#pragma unroll
  for (int g = 0; g < 2; ++g) {
#pragma unroll
    for (int i = 0; i < 4; i += 2) {  // two features at a time: one packed pair per half
      float s[2], c[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int f = 8 * g + 4 * hf + i + u;
        const float phi = xt[0] * Bm[f] + xt[1] * Bm[kFeatures + f] + xt[2] * Bm[2 * kFeatures + f];
        vmap_sincosf(phi, &s[u], &c[u]);
        if (ipe) {  // expectation under N(x, v I): attenuation exp(-v |b_f|^2 / 2)
          const float nb = Bm[f] * Bm[f] + Bm[kFeatures + f] * Bm[kFeatures + f] +
                           Bm[2 * kFeatures + f] * Bm[2 * kFeatures + f];
          const float att = expf(-0.5f * xt[3] * nb);
          s[u] *= att;
          c[u] *= att;
        }
      }
      A.set2(0, 0, 4 * g + i, s[0], s[1]);
      A.set2(0, 0, 8 + 4 * g + i, c[0], c[1]);
    }
  }
  if constexpr (weights_global(H)) {
    static_assert(BF, "weights in device memory: BF16 only");
    const __amdgpu_buffer_rsrc_t rs = image_rsrc(smem, image_bytes(H, BF));
#pragma unroll
    for (int l = 0; l < kLayers; ++l) {
      const int KB = (l == 0) ? 1 : MT;
      const int ws = L.w_stride[l];
      const int lw = (n * ws + 16 * hf) * 2;
#pragma unroll
      for (int mo = 0; mo < MT; ++mo) {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            const bf16x8 wa = img_b128(rs, lw, L.w_off[l] + (mo * 32 * ws + kb * 32 + 8 * jj) * 2);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, A.v[l][kb][jj], acc, 0, 0, 0);
          }
#pragma unroll
        for (int g = 0; g < 4; ++g) {  // rows 8g + 4hf + i
          const f32x4 b4 = img_f4(rs, 16 * hf, L.b_off + (l * H + mo * 32 + 8 * g) * 4);
#pragma unroll
          for (int i = 0; i < 4; ++i) A.set(l + 1, mo, 4 * g + i, fmaxf(acc[4 * g + i] + b4[i], 0.0f));
        }
      }
    }
    if constexpr (!WITH_HEAD) return;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const int lw = (min(n, kOut - 1) * (H + 8) + 16 * hf) * 2;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        bf16x8 wa = img_b128(rs, lw, L.whb_off + (mt * 32 + 8 * jj) * 2);
        if (n >= kOut) wa = bf16x8{};
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, A.v[kLayers][mt][jj], acc, 0, 0, 0);
      }
#pragma unroll
    for (int c = 0; c < kOut; ++c) z[c] = __shfl(acc[c], n) + img_f1(rs, 0, L.bh_off + 4 * c);
    return;
  } else {
  const float* bias = reinterpret_cast<const float*>(smem + L.b_off);
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    const int KB = (l == 0) ? 1 : MT;
    const int ws = L.w_stride[l];
#pragma unroll
    for (int mo = 0; mo < MT; ++mo) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
      if constexpr (BF) {  // accumulator starts at the bias (one MFMA, exact)
        const bf16x8 ba = *reinterpret_cast<const bf16x8*>(
            reinterpret_cast<const __bf16*>(smem + L.bA_off) + (l * H + mo * 32 + n) * 16 + 8 * hf);
        const bf16x8 ones3 = {(__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f, (__bf16)0.0f,
                              (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f};
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ba, ones3, acc, 0, 0, 0);
      }
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        if constexpr (BF) {
          const __bf16* wrow = reinterpret_cast<const __bf16*>(smem + L.w_off[l]) +
                               (mo * 32 + n) * ws + kb * 32 + 16 * hf;
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            const bf16x8 wa = *reinterpret_cast<const bf16x8*>(wrow + 8 * jj);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, A.v[l][kb][jj], acc, 0, 0, 0);
          }
        } else {
          const float* wrow = reinterpret_cast<const float*>(smem + L.w_off[l]) +
                              (mo * 32 + n) * ws + kb * 32 + 16 * hf;
#pragma unroll
          for (int q = 0; q < 16; ++q)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wrow[q], A.v[l][kb][q], acc, 0, 0, 0);
        }
      }
      if constexpr (BF) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) A.v[l + 1][mo][jj] = relu_round8(acc, 8 * jj);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          A.set(l + 1, mo, r, fmaxf(acc[r] + bias[l * H + mo * 32 + rowof(r, hf)], 0.0f));
      }
    }
  }
  if constexpr (!WITH_HEAD) return;
  const float* bh = reinterpret_cast<const float*>(smem + L.bh_off);
  if constexpr (BF) {
    // output layer on MFMA: A = W_out with its four rows padded to 32 (zero rows held in
    // registers, not in LDS); sample n's outputs land in rows 0..3 of lane n (half 0)
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const __bf16* wh = reinterpret_cast<const __bf16*>(smem + L.whb_off);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        bf16x8 wa = {};
        if (n < kOut) wa = *reinterpret_cast<const bf16x8*>(wh + n * (H + 8) + mt * 32 + 16 * hf + 8 * jj);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, A.v[kLayers][mt][jj], acc, 0, 0, 0);
      }
#pragma unroll
    for (int c = 0; c < kOut; ++c) z[c] = __shfl(acc[c], n) + bh[c];
  } else {
    // output layer on the VALU: each half sums its 16 features per block, then the halves are
    // added (the same two addends in both halves, so both hold the same value)
    const float* Wh = reinterpret_cast<const float*>(smem + L.wh_off);
#pragma unroll
    for (int c = 0; c < kOut; ++c) {
      float s = 0.f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += Wh[c * (H + 4) + mt * 32 + 16 * hf + r] * A.get(kLayers, mt, r);
      s += __shfl_xor(s, 32);
      z[c] = s + bh[c];
    }
  }
  }  // weights in LDS
}

// Cross-lane moves of the ray scans, by DPP (a VALU operand modifier, no LDS round trip). DPP
// controls: row_shr:n (lane l takes lane l - n of its row of 16), row_shl:n (lane l + n),
// row_ror:n (rotation by n lanes within a row),
// wave_shr:1 / wave_shl:1 (lane l - 1 / l + 1 across the wave), row_bcast:15 (lane 15 of each row
// into the next row, rows 1 and 3 written), row_bcast:31 (lane 31 into rows 2 and 3). Lanes whose
// source does not exist keep 0; the scans below never use those lanes' results. A move reads its
// source lane's register only if that lane is active, so every move runs with the whole wave
// active (computed before any select that uses it, never in a conditional arm).
constexpr int kDppRowShr = 0x110, kDppRowShl = 0x100, kDppRowRor = 0x120, kDppWaveShl1 = 0x130, kDppWaveShr1 = 0x138,
              kDppBcast15 = 0x142, kDppBcast31 = 0x143;

template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               ROW_MASK, 0xf, false));
}

// Values of a wave's lower half (lanes 0..31, in lo) and upper half (in hi), on the lanes of both
// halves, by one v_permlane32_swap_b32.
__device__ __forceinline__ void half_split(float x, float& lo, float& hi) {
  const unsigned int u = __builtin_bit_cast(unsigned int, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  lo = __builtin_bit_cast(float, (unsigned int)r[0]);
  hi = __builtin_bit_cast(float, (unsigned int)r[1]);
}
// a's lower half and b's lower half as one wave (lo), and both upper halves (hi).
__device__ __forceinline__ void half_join(float a, float b, float& lo, float& hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned int, a),
                                                  __builtin_bit_cast(unsigned int, b), false, false);
  lo = __builtin_bit_cast(float, (unsigned int)r[0]);
  hi = __builtin_bit_cast(float, (unsigned int)r[1]);
}
// Sum of x over lanes l and l ^ 32, on both.
__device__ __forceinline__ float half_sum(float x) {
  float lo, hi;
  half_split(x, lo, hi);
  return lo + hi;
}
// Sum over the wave's lanes, on every lane, by lane swaps and rotations within rows of 16: the
// additions of a butterfly over lane distances 32, 16, 8, 4, 2, 1 (the rotations meet values that
// are already equal at that distance), without its LDS round trips.
__device__ __forceinline__ float wave_sum(float x) {
  x = half_sum(x);
  const unsigned int u = __builtin_bit_cast(unsigned int, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = __builtin_bit_cast(float, (unsigned int)r[0]) + __builtin_bit_cast(float, (unsigned int)r[1]);
  x += dpp_mov<kDppRowRor + 8>(x);
  x += dpp_mov<kDppRowRor + 4>(x);
  x += dpp_mov<kDppRowRor + 2>(x);
  x += dpp_mov<kDppRowRor + 1>(x);
  return x;
}

// Gaussian Fourier features of both passes' samples into layer 0 (register r of a lane of half hf
// holds feature rowof(r, hf): sines of 4hf + 0..3 and 8 + 4hf + 0..3, then the cosines). IPE: each
// is its expectation under N(x, v I), attenuated by exp(-v |b_f|^2 / 2), v = xt[p][3]. One branch
// for the whole encoding, so that the features' chains interleave.
template <bool BF, bool IPE>
__device__ __forceinline__ void encode_pair(const float xt[2][4], const float* Bm, int hf, Acts<32, BF> (&A)[2]) {
#pragma unroll
  for (int g = 0; g < 2; ++g) {
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
      float b[3][2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int c = 0; c < 3; ++c) b[c][u] = Bm[c * kFeatures + 8 * g + 4 * hf + i + u];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        float s[2], c[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float phi = xt[p][0] * b[0][u] + xt[p][1] * b[1][u] + xt[p][2] * b[2][u];
          vmap_sincosf(phi, &s[u], &c[u]);
          if constexpr (IPE) {
            const float nb = b[0][u] * b[0][u] + b[1][u] * b[1][u] + b[2][u] * b[2][u];
            const float att = expf(-0.5f * xt[p][3] * nb);
            s[u] *= att;
            c[u] *= att;
          }
        }
        A[p].set2(0, 0, 4 * g + i, s[0], s[1]);
        A[p].set2(0, 0, 8 + 4 * g + i, c[0], c[1]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Forward of both 32-sample passes of a sub-tile at width 32, layer by layer together: each weight
// operand is read from LDS once for the two passes, and their MFMA chains run side by side (one
// pass after the other took 7.2 thousand cycles per 64-sample sub-tile in BF16, of a 16.8 thousand
// cycle sub-tile; the chain of dependent products and conversions bounds it, not the MFMA rate).
// xt[p]: the point of sample n = lane & 31 of pass p. Each pass's arithmetic is forward_pass's, in
// the same order. zs: the output pre-activations of the lane's own slot (slot = lane).
template <bool BF>
__device__ __forceinline__ void forward_pair(const float xt[2][4], const unsigned char* smem, const float* Bm,
                                             int lane, Acts<32, BF> (&A)[2], float zs[kOut], bool ipe) {
  constexpr LdsLayout L = lds_layout(32, BF, 1);
  asm volatile("" ::: "memory");  // weights are re-read for every sub-tile, not held in registers
  const int n = lane & 31, hf = lane >> 5;
  if (ipe) encode_pair<BF, true>(xt, Bm, hf, A);
  else encode_pair<BF, false>(xt, Bm, hf, A);
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
  const float* bias = reinterpret_cast<const float*>(smem + L.b_off);
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    const int ws = L.w_stride[l];
    f32x16 acc[2];
    if constexpr (BF) {
      // both accumulators start at the bias (one MFMA, exact)
      const bf16x8 ba = *reinterpret_cast<const bf16x8*>(
          reinterpret_cast<const __bf16*>(smem + L.bA_off) + (l * 32 + n) * 16 + 8 * hf);
      const bf16x8 ones3 = {(__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f, (__bf16)0.0f,
                            (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f};
      const __bf16* wrow = reinterpret_cast<const __bf16*>(smem + L.w_off[l]) + n * ws + 16 * hf;
      const bf16x8 w0 = *reinterpret_cast<const bf16x8*>(wrow), w1 = *reinterpret_cast<const bf16x8*>(wrow + 8);
      const f32x16 b16 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ba, ones3, zero, 0, 0, 0);
#pragma unroll
      for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0, A[p].v[l][0][0], b16, 0, 0, 0);
#pragma unroll
      for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1, A[p].v[l][0][1], acc[p], 0, 0, 0);
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) A[p].v[l + 1][0][jj] = relu_round8(acc[p], 8 * jj);
    } else {
      const float* wrow = reinterpret_cast<const float*>(smem + L.w_off[l]) + n * ws + 16 * hf;
      acc[0] = acc[1] = zero;
#pragma unroll
      for (int q = 0; q < 16; ++q)
#pragma unroll
        for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(wrow[q], A[p].v[l][0][q], acc[p], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float b = bias[l * 32 + rowof(r, hf)];
#pragma unroll
        for (int p = 0; p < 2; ++p) A[p].set(l + 1, 0, r, fmaxf(acc[p][r] + b, 0.0f));
      }
    }
  }
  const float* bh = reinterpret_cast<const float*>(smem + L.bh_off);
  if constexpr (BF) {
    // output layer on MFMA: A = W_out with its four rows padded to 32 (zero rows held in
    // registers); sample n's outputs land in rows 0..3 of lane n (half 0) of each pass
    const __bf16* wh = reinterpret_cast<const __bf16*>(smem + L.whb_off) + n * 40 + 16 * hf;
    f32x16 acc[2] = {zero, zero};
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      bf16x8 wa = {};
      if (n < kOut) wa = *reinterpret_cast<const bf16x8*>(wh + 8 * jj);
#pragma unroll
      for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, A[p].v[kLayers][0][jj], acc[p], 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < kOut; ++c) {
      float unused;
      half_join(acc[0][c] + bh[c], acc[1][c] + bh[c], zs[c], unused);
    }
  } else {
    // output layer on the VALU: each half sums its 16 features, then the halves are added
    const float* Wh = reinterpret_cast<const float*>(smem + L.wh_off);
#pragma unroll
    for (int c = 0; c < kOut; ++c) {
      float s[2] = {0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float w = Wh[c * 36 + 16 * hf + r];
#pragma unroll
        for (int p = 0; p < 2; ++p) s[p] += w * A[p].v[kLayers][0][r];
      }
      float lo, hi;
      half_join(s[0], s[1], lo, hi);
      zs[c] = (lo + hi) + bh[c];
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The step's tile kernel.

__device__ __forceinline__ void read_batch(StepArgs& a) {
  if (const BatchDev* b = a.bd) {
    a.n_objects = b->n_objects;
    a.n_rays = b->n_rays;
    a.S = b->S;
    a.object_ids = b->object_ids;
    a.ray_offsets = b->ray_offsets;
    a.rays_o = b->rays_o;
    a.rays_d = b->rays_d;
    a.t = b->t;
    a.depth = b->depth;
    a.rgb = b->rgb;
    a.mask = b->mask;
    a.var = b->var;
  }
}

__device__ __forceinline__ void read_batch(OptArgs& a) {
  if (const BatchDev* b = a.bd) {
    a.n_objects = b->n_objects;
    a.ids = b->object_ids;
    a.offs = b->ray_offsets;
    a.loss_out = b->loss_out;
  }
}

// Rendering (Eq. 3), the masked L1 losses (Eqs. 4-7) and, in training, their adjoint for one
// sub-tile of the calling wave: lane = sample slot, zs = the slot's head pre-activations (r, g, b,
// occupancy). Adds the sub-tile's loss to `loss`; forward mode writes the rendered outputs;
// training returns dL/dz of the slot in dzs (zero on slots at or past nslots).
// The rendering's per-sample inputs of a sub-tile (sample depth; the ray's depth, mask and colour
// targets), loaded before the forward pass so that their latency hides behind it.
struct RenderIn {
  float tt, D, M, rgb[3];
};

template <bool TRAIN>
__device__ __forceinline__ RenderIn render_inputs(const StepArgs& a, int r0, int nslots) {
  const int lane = threadIdx.x & 63;
  RenderIn in{0.f, 0.f, 0.f, {0.f, 0.f, 0.f}};
  if (lane < nslots) {
    const int ray = r0 + lane / a.S;
    in.tt = a.t[(size_t)r0 * a.S + lane];
    // rendering without targets (forward mode, NULL target buffers) evaluates the loss terms
    // against zero targets; that loss is not reported
    if (TRAIN || a.depth != nullptr) {
      in.D = a.depth[ray];
      in.M = a.mask[ray];
#pragma unroll
      for (int c = 0; c < 3; ++c) in.rgb[c] = a.rgb[3 * ray + c];
    }
  }
  return in;
}

// Everything a lane loads for its slot of sub-tile `sub` of a tile of the width-32 kernel (rays
// [ray_lo, ray_hi), rpw rays a sub-tile; a sub-tile past the tile's last has no slots).
struct SubTileIn {
  RenderIn r;
  float o[3], d[3], var;
};

template <bool TRAIN>
__device__ __forceinline__ SubTileIn subtile_inputs(const StepArgs& a, int ray_lo, int ray_hi, int sub, int rpw) {
  const int lane = threadIdx.x & 63;
  const int r0 = ray_lo + sub * rpw;
  const int nslots = max(0, min(rpw, ray_hi - r0)) * a.S;
  SubTileIn in{};
  in.r = render_inputs<TRAIN>(a, r0, nslots);
  if (lane < nslots) {
    const int ray = r0 + lane / a.S;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      in.o[c] = a.rays_o[3 * (size_t)ray + c];
      in.d[c] = a.rays_d[3 * (size_t)ray + c];
    }
    if (a.var) in.var = a.var[(size_t)r0 * a.S + lane];
  }
  return in;
}

// Inclusive scans within the rays of a sub-tile. A ray is a segment of S consecutive lanes from
// lane 0 (lanes past the last ray are segments of one lane); si = the lane's position in its
// segment, de = its distance to the segment's last lane. Forward: lane l combines lanes
// [segment start, l], by shifts of 1, 2, 4 and 8 within rows of 16 lanes (a step combines where
// the source lies in both the row and the segment), then lane 15 of each row into the next row
// and lane 31 into rows 2 and 3 (where no segment starts between the row's first lane and l).
// Reverse: lane l combines lanes [l, segment end], by shifts within rows, then the first lane of
// rows 3, 2 and 1 into the row before, in that order.
struct RayScan {
  bool f[6];  // forward steps
  bool r[4];  // reverse steps within rows
  int de, lr, row;

  __device__ __forceinline__ RayScan(int lane, int si, int de_) : de(de_) {
    lr = lane & 15;
    row = lane >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[i] = si >= (1 << i) && lr >= (1 << i);
      r[i] = de >= (1 << i) && lr + (1 << i) <= 15;
    }
    f[4] = (row & 1) && si > lr;
    f[5] = lane >= 32 && si > lane - 32;
  }

  template <int N, class Op>
  __device__ __forceinline__ void forward(float (&v)[N], Op op) const {
    float u[N];
#define VMAP_SCAN_STEP(I, CTRL, RM)                                        \
  {                                                                        \
    _Pragma("unroll") for (int q = 0; q < N; ++q) u[q] = dpp_mov<CTRL, RM>(v[q]); \
    _Pragma("unroll") for (int q = 0; q < N; ++q) v[q] = f[I] ? op(v[q], u[q]) : v[q]; \
  }
    VMAP_SCAN_STEP(0, kDppRowShr + 1, 0xf)
    VMAP_SCAN_STEP(1, kDppRowShr + 2, 0xf)
    VMAP_SCAN_STEP(2, kDppRowShr + 4, 0xf)
    VMAP_SCAN_STEP(3, kDppRowShr + 8, 0xf)
    VMAP_SCAN_STEP(4, kDppBcast15, 0xa)
    VMAP_SCAN_STEP(5, kDppBcast31, 0xc)
#undef VMAP_SCAN_STEP
  }

  __device__ __forceinline__ float reverse_sum(float v) const {
    float u;
    u = dpp_mov<kDppRowShl + 1>(v); v = r[0] ? v + u : v;
    u = dpp_mov<kDppRowShl + 2>(v); v = r[1] ? v + u : v;
    u = dpp_mov<kDppRowShl + 4>(v); v = r[2] ? v + u : v;
    u = dpp_mov<kDppRowShl + 8>(v); v = r[3] ? v + u : v;
#pragma unroll
    for (int rr = 2; rr >= 0; --rr) {
      const float s = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16 * (rr + 1)));
      v = (row == rr && de > 15 - lr) ? v + s : v;
    }
    return v;
  }
};

template <bool TRAIN>
__device__ __forceinline__ void render_subtile(const StepArgs& a, int r0, int nslots, float wseed,
                                               const RenderIn& in, const float zs[kOut], float dzs[kOut],
                                               float& loss) {
  const int lane = threadIdx.x & 63;
  const int S = a.S;
  const float lc = a.lambda_c, lo = a.lambda_o;
  const bool valid = lane < nslots;
  const int jr = valid ? lane / S : 0;
  const int si = valid ? lane - jr * S : 0;
  const int de = valid ? S - 1 - si : 0;
  const int ray = r0 + jr;
  const RayScan sc(lane, si, de);
  float o = 0.f, q = 1.f, c3[3] = {0.f, 0.f, 0.f}, cq[3] = {0.f, 0.f, 0.f};
  const float tt = in.tt;
  if (valid) {
    sigm_pair(zs[3], o, q);  // q = 1 - o, without cancellation
#pragma unroll
    for (int c = 0; c < 3; ++c) sigm_pair(zs[c], c3[c], cq[c]);
  }
  // P_i = prod_{j<i} (1 - o_j): inclusive product scan within the ray, then shift by one lane
  float pin[1] = {q};
  sc.forward(pin, [](float x, float y) { return x * y; });
  const float Pin = pin[0];
  const float Pprev = dpp_mov<kDppWaveShr1>(Pin);  // outside the select: every lane must take part
  const float Pex = (si == 0) ? 1.f : Pprev;
  const float Tw = o * Pex;  // termination probability T_i
  // the ray's sums end up in its last lane
  float sums[5] = {Tw, Tw * tt, Tw * c3[0], Tw * c3[1], Tw * c3[2]};
  sc.forward(sums, [](float x, float y) { return x + y; });

  // the ray's outputs, loss and residual signs, in its last lane; the signs (each -1, 0 or 1)
  // travel packed to the other lanes of the ray
  int code = 0;
  if (valid && de == 0) {
    const float Oh = sums[0], Dh = sums[1];
    const float Ch[3] = {sums[2], sums[3], sums[4]};
    const float D = in.D, M = in.M;
    const float rD = Dh - D;
    float rC[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) rC[c] = Ch[c] - in.rgb[c];
    const float rho = (M == 1.0f) ? -Pin : (Oh - M);
    loss += M * fabsf(rD) + lc * M * (fabsf(rC[0]) + fabsf(rC[1]) + fabsf(rC[2])) + lo * fabsf(rho);
    if constexpr (!TRAIN) {
      if (a.out_depth) a.out_depth[ray] = Dh;
      if (a.out_occ) a.out_occ[ray] = Oh;
      if (a.out_rgb) { a.out_rgb[3 * ray] = Ch[0]; a.out_rgb[3 * ray + 1] = Ch[1]; a.out_rgb[3 * ray + 2] = Ch[2]; }
    }
    auto sgn2 = [](float x) { return (x > 0.f) ? 2 : ((x < 0.f) ? 0 : 1); };
    code = sgn2(rD) | (sgn2(rho) << 2) | (sgn2(rC[0]) << 4) | (sgn2(rC[1]) << 6) | (sgn2(rC[2]) << 8);
  }
  if constexpr (!TRAIN) return;
  code = __shfl(code, jr * S + S - 1);
  auto sgn_of = [&](int i) { return (float)(((code >> (2 * i)) & 3) - 1); };

  float g = 0.f, aC[3] = {0.f, 0.f, 0.f};
  if (valid) {
    const float M = in.M;
    const float aD = wseed * M * sgn_of(0);
    const float aO = wseed * lo * sgn_of(1);
#pragma unroll
    for (int c = 0; c < 3; ++c) aC[c] = wseed * lc * M * sgn_of(2 + c);
    g = aD * tt + aC[0] * c3[0] + aC[1] * c3[1] + aC[2] * c3[2] + aO;
  }
  // adjoint of rendering: dL/dz_occ,i = o_i (q_i g_i P_i - R_i), R_i = sum over the later samples j
  // of the ray of g_j T_j (the exclusive suffix sum, a reverse scan shifted by one lane)
  const float Rin = sc.reverse_sum(g * Tw);
  const float Rnext = dpp_mov<kDppWaveShl1>(Rin);
  const float R = (de == 0) ? 0.f : Rnext;
  dzs[3] = valid ? o * (q * g * Pex - R) : 0.f;
#pragma unroll
  for (int c = 0; c < 3; ++c) dzs[c] = valid ? Tw * aC[c] * c3[c] * cq[c] : 0.f;
}

// ---------------------------------------------------------------------------------------------
// Per-object gradient and optimiser. Tile partials are already unscaled by the tile kernel, which
// also flagged objects with a non-finite partial. Three kernels share the pieces below:
//   k_reduce      — loss and gradient per object (forward/backward split),
//   k_adam        — Adam from the stored gradient (after k_reduce),
//   k_reduce_adam — both in one pass (the training step when it is split into launches).
// The optimiser kernels take each object's next step count from the work-list kernel; block
// (0, j) writes it back; block (0, 0) of k_reduce and k_adam, and the extra last row of
// k_reduce_adam, update the loss scaler from the flags. No block reads what
// another block of the same launch writes, so no device-scope fence is needed. After a MODE_STEP
// tile launch (below) the table, step counts and cleared flags come from the tile kernel and the
// non-finite reports from its tiles.

// Sum of an object's tile partials at parameter p; up to 32 loads are issued before the first add.
// At most kSplitTiles tiles: in tile order. More: the tiles' four consecutive quarters (tile_quarter),
// each in tile order, then the quarters in order, so that a workgroup's waves can take a quarter
// each (k_reduce_adam_wide). The order depends on the object's tile count alone.
constexpr int kSplitTiles = 32;
static_assert(kSpreadTiles >= kSplitTiles, "spread objects are summed in quarters");
// Units of k_reduce_adam_wide of an object (at least one, for its loss).
__device__ __forceinline__ int opt_units(int n_params, int tiles) {
  const int unit = tiles > kSplitTiles ? 256 : 1024;
  return max(1, (n_params + unit - 1) / unit);
}
__device__ __forceinline__ TileRange tile_quarter(int t0, int t1, int q) {
  const int len = (t1 - t0 + 3) >> 2, a = t0 + q * len;
  return TileRange{min(a, t1), min(a + len, t1)};
}
__device__ __forceinline__ float tile_sum(const float* __restrict__ partial, int p_stride, int t0,
                                          int t1, int p) {
  if (t1 - t0 <= kSplitTiles) {
    float g = 0.f, x[kSplitTiles];
#pragma unroll
    for (int u = 0; u < kSplitTiles; ++u) x[u] = (t0 + u < t1) ? partial[(size_t)(t0 + u) * p_stride + p] : 0.f;
#pragma unroll
    for (int u = 0; u < kSplitTiles; ++u)
      if (t0 + u < t1) g += x[u];
    return g;
  }
  TileRange q[4];
  float g[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = tile_quarter(t0, t1, i);
  for (int b = 0; b < q[0].t1 - q[0].t0; b += 8) {  // (the first quarter is the longest)
    float x[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        x[i][u] = (q[i].t0 + b + u < q[i].t1) ? partial[(size_t)(q[i].t0 + b + u) * p_stride + p] : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (q[i].t0 + b + u < q[i].t1) g[i] += x[i][u];
  }
  return ((g[0] + g[1]) + g[2]) + g[3];
}

// Sum of an object's tile losses in tile_sum's order, by a whole wave: 64 tiles (of many: of each
// quarter) are read at once, one per lane, and added one after another from lane registers, the
// quarters side by side (past a quarter's end zeros are added, which change no sum).
__device__ __forceinline__ float loss_sum(const float* __restrict__ tile_loss, int t0, int t1) {
  const int lane = threadIdx.x & 63;
  auto from = [](float v, int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l)); };
  float g[4] = {0.f, 0.f, 0.f, 0.f};
  if (t1 - t0 <= kSplitTiles) {
    const float x = t0 + lane < t1 ? tile_loss[t0 + lane] : 0.f;
    for (int u = 0; u < t1 - t0; ++u) g[0] += from(x, u);
    return g[0];
  }
  const int len = (t1 - t0 + 3) >> 2;
  for (int b = 0; b < len; b += kWave) {
    float x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const TileRange q = tile_quarter(t0, t1, i);
      x[i] = q.t0 + b + lane < q.t1 ? tile_loss[q.t0 + b + lane] : 0.f;
    }
    const int n = min(kWave, len - b);
    for (int u = 0; u < n; ++u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) g[i] += from(x[i], u);
    }
  }
  return ((g[0] + g[1]) + g[2]) + g[3];
}

// Objects of many tiles (more than kSpreadTiles), in a kernel of a row of workgroups per object and a
// thread per parameter: the CUs that a row runs on read its partials at some 6 bytes per cycle each,
// however many loads are in flight, so the rows of such objects are spread over four times as many
// workgroups. A workgroup of 256 parameters keeps the first 64 of them and three extra rows take the
// others (OptArgs::spread of them, the host's bound on such objects), every wave a quarter of the tiles,
// in tile_sum's order. The step of one object of 12,000 rays x 10 samples (BF16, 500 tiles): 56 us with
// its row alone, 38 of them here; 34 spread. One of 5,000 rays x 20 beside fifty of 20: 44 and 34.
// The s-th object of many tiles, or -1 (called by whole waves; four loads per lane at most).
__device__ __forceinline__ int spread_object(const OptArgs& a, int s) {
  const int lane = threadIdx.x & 63;
  for (int base = 0; base < a.n_objects; base += kWave) {
    const int j = base + lane;
    bool many = false;
    if (j < a.n_objects) {
      const TileRange tr = clamp_tile_range(a.tile_start[j], a.tile_start[j + 1], a.max_tiles);
      many = tr.t1 - tr.t0 > kSpreadTiles;
    }
    unsigned long long m = __ballot(many);
    const int c = __popcll(m);
    if (s < c) {
      for (; s > 0; --s) m &= m - 1ull;
      return base + __ffsll((long long)m) - 1;
    }
    s -= c;
  }
  return -1;
}
// Sum of an object's tile partials at 64 parameters, p the lane's (below p_stride), by a workgroup of
// four waves; valid in wave 0.
__device__ __forceinline__ float spread_sum(const float* __restrict__ partial, int p_stride, int t0, int t1, int p) {
  __shared__ float part[4][kWave];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const TileRange q = tile_quarter(t0, t1, wave);
  float g = 0.f;
  for (int t = q.t0; t < q.t1; t += 32) {
    float x[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) x[u] = t + u < q.t1 ? partial[(size_t)(t + u) * p_stride + p] : 0.f;
#pragma unroll
    for (int u = 0; u < 32; ++u)
      if (t + u < q.t1) g += x[u];
  }
  part[wave][lane] = g;
  __syncthreads();
  return ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
}

__device__ __forceinline__ bool obj_valid(const OptArgs& a, int k) {
  return k >= 0 && k < a.max_objects && a.desc[k].registered;
}

// Whether batch object j (id k) had a non-finite tile partial: bit 0 of its flag (set by the tiles;
// k_reduce_adam marks its own overflows in bit 1, which this test leaves out, so every workgroup
// of an object decides alike), or with per-tile reports the OR of its tiles' entries. Called by
// every thread of the workgroup.
__device__ __forceinline__ bool object_bad(const OptArgs& a, int j, int k) {
  if (!a.tile_bad) return __syncthreads_or((a.flags[k] & 1) != 0) != 0;
  int bad = 0;
  const TileRange tr = clamp_tile_range(a.tile_start[j], a.tile_start[j + 1], a.max_tiles);
  for (int t = tr.t0 + (int)threadIdx.x; t < tr.t1; t += blockDim.x) bad |= a.tile_bad[t];
  return __syncthreads_or(bad) != 0;
}

// OR of the non-finite reports of tiles [t0, t1); up to 32 loads are issued before the first use.
__device__ __forceinline__ int tile_or(const int32_t* __restrict__ bad, int t0, int t1) {
  int r = 0;
  for (int t = t0; t < t1; t += 32) {
    int x[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) x[u] = (t + u < t1) ? bad[t + u] : 0;
#pragma unroll
    for (int u = 0; u < 32; ++u) r |= x[u];
  }
  return r;
}

// One workgroup (any size): count the batch objects with rays whose gradient was not finite;
// BF16 loss scaler. (On the split path an overflow that k_reduce_adam finds while summing finite
// partials is flagged during this same launch, so it is counted only if its flag is already
// visible; the per-tile reports of the training step are complete before the launch.) Each thread loads its object's id, rays, tiles and descriptor at once (an id
// out of range reads object 0's descriptor and is then discarded), then its tiles' reports.
__device__ void scaler_update(const OptArgs& a) {
  __shared__ int count;
  if (!a.scaler->batch_ok) return;  // the batch did not run: the scaler stays as it is
  if (threadIdx.x == 0) count = 0;
  __syncthreads();
  int skipped = 0;
  for (int base = 0; base < a.n_objects; base += blockDim.x) {
    const int jj = base + (int)threadIdx.x;
    int kk = -1, r0 = 0, r1 = 0, t0 = 0, t1 = 0;
    if (jj < a.n_objects) {
      kk = a.ids[jj];
      r0 = a.offs[jj];
      r1 = a.offs[jj + 1];
      const TileRange tr = clamp_tile_range(a.tile_start[jj], a.tile_start[jj + 1], a.max_tiles);
      t0 = tr.t0;
      t1 = tr.t1;
    }
    const bool in_range = kk >= 0 && kk < a.max_objects;
    const int kc = in_range ? kk : 0;
    const bool registered = a.desc[kc].registered != 0;
    // from the tiles: the objects' flags are being written by this launch
    int bad = 0;
    if (a.tile_bad) {
      const bool many = t1 - t0 > kSpreadTiles;
      if (!many) bad = tile_or(a.tile_bad, t0, t1);
      for (unsigned long long m = __ballot(many); m; m &= m - 1ull) {  // by the whole wave, in turn
        const int l = __ffsll((long long)m) - 1, s1 = __builtin_amdgcn_readlane(t1, l);
        int any = 0;
        for (int t = __builtin_amdgcn_readlane(t0, l) + (int)(threadIdx.x & 63); t < s1; t += kWave) any |= a.tile_bad[t];
        if (__ballot(any != 0) && (int)(threadIdx.x & 63) == l) bad = 1;
      }
    } else {
      bad = a.flags[kc];
    }
    if (in_range && registered && r1 > r0 && bad != 0) ++skipped;
  }
  if (skipped) atomicAdd(&count, skipped);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int total = count;
    a.scaler->skipped = total;
    if (a.bf16) {
      // the scale stays a power of two in [2^-125, 2^126], so that it and its inverse are normal
      const float sc = a.scaler->scale;
      if (total > 0) {
        if (sc >= 0x1p-124f) a.scaler->scale = sc * 0.5f;
        a.scaler->good_steps = 0;
      } else if (++a.scaler->good_steps >= a.growth) {
        if (sc <= 0x1p125f) a.scaler->scale = sc * 2.0f;
        a.scaler->good_steps = 0;
      }
    }
  }
}

struct AdamCoef {
  float step, rs, b1, c1, b2, c2, eps;
};

// b^t for a step count t >= 0, by squaring: one thread works it out while a workgroup's loads are
// in flight, and the chain of the general pow was longer than theirs.
__device__ __forceinline__ double pow_step(double b, int t) {
  double r = 1.0;
  for (unsigned int e = (unsigned int)max(t, 0); e; e >>= 1, b *= b)
    if (e & 1u) r *= b;
  return r;
}

// Bias-corrected step size and 1/sqrt(bias correction of v) in FP64, then rounded once.
__device__ __forceinline__ void adam_coef_store(const OptArgs& a, int t, float* sh) {
  const double bc1 = 1.0 - pow_step(a.beta1, t), bc2 = 1.0 - pow_step(a.beta2, t);
  sh[0] = (float)(a.lr / bc1);
  sh[1] = (float)(1.0 / sqrt(bc2));
}

__device__ __forceinline__ AdamCoef adam_coef_load(const OptArgs& a, const float* sh) {
  return AdamCoef{sh[0], sh[1], (float)a.beta1, (float)(1.0 - a.beta1), (float)a.beta2,
                  (float)(1.0 - a.beta2), (float)a.eps};
}

__device__ AdamCoef adam_coef(const OptArgs& a, int t) {
  __shared__ float sh[2];
  if (threadIdx.x == 0) adam_coef_store(a, t, sh);
  __syncthreads();
  return adam_coef_load(a, sh);
}

// Parameter p of object k changed to th: its entry in the object's weight image (width 32, also
// for hidden 16, whose image is the zero-padded width-32 one; the BF16 image of hidden 128), or
// in its BF16 parameter copy (layered path, hidden 256 and up). WIDE = false leaves out the
// hidden-128 image, for k_reduce_adam: a stack that can hold hidden-128 objects has at least
// kReduceWide parameter slots per object and takes k_reduce_adam_wide (its launcher checks).
template <bool WIDE = true>
__device__ __forceinline__ void update_image(const OptArgs& a, int k, int hidden, int p, float th) {
  if (a.gimg && keeps_gimg(hidden)) {
    a.gimg[(size_t)k * a.p_stride + p] = (uint16_t)(pack2(th, 0.f) & 0xffffu);
    return;
  }
  if constexpr (WIDE) {
    if (hidden == 128) {
      if (a.wimage && a.bf16) place_param<128, true>(a.wimage + (size_t)k * a.wimage_stride, p, th);
      return;
    }
  }
  if (!a.img32 || kernel_width(hidden) != 32) return;
  const int q = padded_index(hidden, p);
  if (a.bf16) place_param<32, true>(a.img32 + (size_t)k * img32_bytes(true), q, th);
  else place_param<32, false>(a.img32 + (size_t)k * img32_bytes(false), q, th);
}

// One Adam update; the contractions are spelled out so that the rounding does not depend on how
// the compiler schedules the surrounding code.
__device__ __forceinline__ void adam_elem(const AdamCoef& c, float g, float& th, float& m, float& v) {
  m = fmaf(c.b1, m, c.c1 * g);
  v = fmaf(c.b2, v, c.c2 * (g * g));
  th = fmaf(-c.step, m / fmaf(sqrtf(v), c.rs, c.eps), th);
}

// ---------------------------------------------------------------------------------------------
// Training step without a work-list launch (MODE_STEP). Every workgroup of the tile kernel scans
// the batch's ray offsets into a tile table in LDS (what k_worklist writes to device memory);
// workgroup 0 also leaves in device memory what k_worklist leaves for the optimiser: the table,
// the next Adam step counts and cleared flags. Tiles then report a non-finite partial in their
// own tile_bad entry instead of the object's flag (which workgroup 0 may clear concurrently), and
// k_reduce_adam reads those entries.

// Inclusive scan over the wave by DPP: shifts within rows of 16, then lane 15 of each row into the
// next row and lane 31 into rows 2 and 3 (every move with the whole wave active).
__device__ __forceinline__ int wave_scan(int x) {
  const int lane = threadIdx.x & 63, lr = lane & 15;
  int y = __builtin_amdgcn_update_dpp(0, x, kDppRowShr + 1, 0xf, 0xf, false);
  x += (lr >= 1) ? y : 0;
  y = __builtin_amdgcn_update_dpp(0, x, kDppRowShr + 2, 0xf, 0xf, false);
  x += (lr >= 2) ? y : 0;
  y = __builtin_amdgcn_update_dpp(0, x, kDppRowShr + 4, 0xf, 0xf, false);
  x += (lr >= 4) ? y : 0;
  y = __builtin_amdgcn_update_dpp(0, x, kDppRowShr + 8, 0xf, 0xf, false);
  x += (lr >= 8) ? y : 0;
  y = __builtin_amdgcn_update_dpp(0, x, kDppBcast15, 0xa, 0xf, false);
  x += ((lane >> 4) & 1) ? y : 0;
  y = __builtin_amdgcn_update_dpp(0, x, kDppBcast31, 0xc, 0xf, false);
  x += (lane >= 32) ? y : 0;
  return x;
}

// Batch object j of a wave's lane j (at most 64 objects): first tile, tiles, ray segment and id.
struct LaneTable {
  int first, count, o0, o1, k;
};

// The tile table of a batch of at most 64 objects in registers: every wave of the workgroup scans
// it by itself, without LDS or barriers. Returns the tile count or -1 as step_table does.
__device__ __forceinline__ int step_table_small(const StepArgs& a, LaneTable& t) {
  const int j = threadIdx.x & 63;
  t = LaneTable{0, 0, 0, 0, -1};
  bool ok = true;
  if (j < a.n_objects) {
    t.o0 = a.ray_offsets[j];
    t.o1 = a.ray_offsets[j + 1];
    t.k = a.object_ids[j];
    ok = batch_segment_ok(j, a.n_objects, t.o0, t.o1, a.n_rays);
    t.count = ok ? tiles_of(t.o1 - t.o0, a.rays_per_tile) : 0;
  }
  const int x = wave_scan(t.count);
  t.first = x - t.count;
  return __ballot(!ok) ? -1 : __builtin_amdgcn_readlane(x, 63);
}

// tbl[j] = first tile of batch object j, tbl[n_objects] = tiles: the exclusive scan of
// ceil(rays_j / rays_per_tile) over the batch (the launch's objects share one width, so one tile
// size); tray[j] = the batch's ray offsets (n_objects + 1 of them) and tk[j] = object ids, so that
// a tile finds its object and rays in LDS (without a.lds_rays they are read from the batch, and only
// tbl is kept: the launcher's choice for many objects). Returns the tile count, or -1 when the offsets fail
// the check of segment_ok (ray_offsets[0] = 0, every segment inside [0, n_rays] and in order,
// ray_offsets[n] = n_rays); then no tile runs. Called by every thread of the workgroup.
__device__ int step_table(const StepArgs& a, int32_t* tbl, int32_t* tray, int32_t* tk) {
  __shared__ int wtot[8];  // up to eight waves
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  const int rpt = a.rays_per_tile;
  int carry = 0, bad = 0;
  for (int base = 0; base < a.n_objects; base += nt) {
    const int j = base + tid;
    int cnt = 0;
    if (j < a.n_objects) {
      const int o0 = a.ray_offsets[j], o1 = a.ray_offsets[j + 1];
      if (a.lds_rays) {
        tray[j] = o0;
        tk[j] = a.object_ids[j];
        if (j == a.n_objects - 1) tray[j + 1] = o1;
      }
      const bool ok = batch_segment_ok(j, a.n_objects, o0, o1, a.n_rays);
      bad |= !ok;
      cnt = ok ? tiles_of(o1 - o0, rpt) : 0;
    }
    const int x = wave_scan(cnt);
    if (lane == kWave - 1) wtot[wave] = x;
    __syncthreads();
    int before = carry, total = 0;
    for (int w = 0; w < nw; ++w) {
      const int v = wtot[w];
      if (w < wave) before += v;
      total += v;
    }
    if (j < a.n_objects) tbl[j] = before + x - cnt;
    carry += total;
    __syncthreads();
  }
  if (tid == 0) tbl[a.n_objects] = carry;
  return __syncthreads_or(bad) ? -1 : carry;
}

template <int H, bool BF, int MODE>
// BF16 at width 32: up to eight waves per workgroup, 256 registers (two waves per SIMD).
__global__ void __launch_bounds__((BF && H == 32) ? 512 : 256, 1) k_step_tiles(const StepArgs a_in) {
  StepArgs a = a_in;
  read_batch(a);
  if constexpr (MODE == MODE_FWD) {
    if (a.bd && a.bd->rays_per_tile > 0) a.rays_per_tile = a.bd->rays_per_tile;  // (a scene's)
  }
  constexpr int MT = H / 32;
  constexpr bool TABLE = (MODE == MODE_STEP);  // tile table built here, not by k_worklist
  constexpr bool TRAIN = (MODE == MODE_TRAIN) || TABLE;
  constexpr int kTile = pair_tile_bytes(BF);  // staging tiles (vmap_internal.h)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr LdsLayout L = lds_layout(H, BF, 1);
  const int tid = threadIdx.x, lane = tid & 63, lane_ = lane, wave = tid >> 6, nw = blockDim.x >> 6;
  const int S = a.S;
  const int rpw = kSlots / S;

  // first tile of every batch object: from the LDS table or from k_worklist
  // (and, with the LDS table, its ray offsets and object ids)
  const int tbl_pitch = table_layout(0, a.n_objects).pitch;
  int32_t* tbl = reinterpret_cast<int32_t*>(smem + a.lds_table);
  int32_t* tray = tbl + tbl_pitch;
  int32_t* tk = tray + tbl_pitch;
  auto first_tile = [&](int j) { return TABLE ? tbl[j] : a.width_start[j]; };  // among this width's tiles
  int n_tiles;
  LaneTable lt{};
  const bool small = TABLE && a.n_objects <= kWave;
  if constexpr (TABLE) {
    if (small) {
      n_tiles = step_table_small(a, lt);
      if (wave == 0 && lane < a.n_objects) {  // for a workgroup's later tiles
        tbl[lane] = lt.first;
        tray[lane] = lt.o0;
        tk[lane] = lt.k;
        if (lane == a.n_objects - 1) {
          tbl[lane + 1] = lt.first + lt.count;
          tray[lane + 1] = lt.o1;
        }
      }
    } else {
      n_tiles = step_table(a, tbl, tray, tk);
    }
    if (blockIdx.x == 0) {  // what k_worklist leaves for the optimiser
      if (tid == 0) {
        a.scaler->batch_ok = n_tiles >= 0;
        if (n_tiles < 0) atomicOr(&a.scaler->device_error, DERR_OFFSETS);
      }
      if (small) __syncthreads();
      for (int j = tid; j <= a.n_objects; j += blockDim.x) a.tile_start_out[j] = n_tiles >= 0 ? tbl[j] : 0;
      for (int j = tid; j < a.n_objects; j += blockDim.x) {
        const int k = a.lds_rays ? tk[j] : a.object_ids[j];
        const bool valid = k >= 0 && k < a.max_objects;
        if (valid) a.flags[k] = 0;
        a.t_next[j] = (valid && a.desc[k].registered) ? a.desc[k].step + 1 : 0;
      }
      return;  // the other workgroups run the tiles
    }
  } else {
    n_tiles = a.width_start[a.n_objects];
  }
  n_tiles = clamp_tiles(n_tiles, a.max_tiles);

  float* Bl = reinterpret_cast<float*>(smem + L.B_off);
  if (tid < 3 * kFeatures) Bl[tid] = a.B[tid];
  int staged = -1;

  // (with the table, workgroup 0 has published it and returned: the tiles' workgroups follow)
  const int wg = TABLE ? (int)blockIdx.x - 1 : (int)blockIdx.x, wgs = TABLE ? (int)gridDim.x - 1 : (int)gridDim.x;
  int tile = first_tile_of_block(wg, wgs, n_tiles);  // (every tile belongs to this launch)
  // object of a tile: the j with first_tile(j) <= tile < first_tile(j + 1) (objects without rays
  // have an empty range), 64 candidates per wave at a time; a workgroup's first tile of a small
  // batch from the lanes' own entries
  int j = 0, k = -1, o0 = 0, o1 = 0, ft = 0;
  bool known = false;
  if (small && tile < n_tiles) {
    j = __ffsll((long long)__ballot(lt.first <= tile && tile < lt.first + lt.count)) - 1;
    k = __builtin_amdgcn_readlane(lt.k, j);
    o0 = __builtin_amdgcn_readlane(lt.o0, j);
    o1 = __builtin_amdgcn_readlane(lt.o1, j);
    ft = __builtin_amdgcn_readlane(lt.first, j);
    known = true;
  }
  for (; tile < n_tiles; tile += wgs, known = false) {
    if (!known) {
      j = 0;
      for (int base = 0; base < a.n_objects; base += kWave) {
        const int jj = base + lane;
        const bool hit = jj < a.n_objects && first_tile(jj) <= tile && tile < first_tile(jj + 1);
        const unsigned long long m = __ballot(hit);
        if (m) {
          j = base + __ffsll((long long)m) - 1;
          break;
        }
      }
      const bool lds = TABLE && a.lds_rays;
      k = lds ? tk[j] : a.object_ids[j];
      o0 = lds ? tray[j] : a.ray_offsets[j];
      o1 = lds ? tray[j + 1] : a.ray_offsets[j + 1];
      ft = first_tile(j);
    }
    const int rpt = tile_rays(H, a.rays_per_tile, a.rays_per_tile_wide);
    const RayRange rr = tile_ray_range(o0, o1, tile - ft, rpt, a.n_rays);
    const int ray_lo = rr.lo, ray_hi = rr.hi;
    const int nrays = ray_hi - ray_lo;
    const int nsub = (nrays + rpw - 1) / rpw;
    // the tile's index in the batch's work list (its partial, loss and report)
    const int slot = TABLE ? tile : a.tile_start[j] + tile - ft;
    if (slot < 0 || slot >= a.max_tiles) continue;  // (not for a consistent work list)
    // The object's weight image goes to LDS before its descriptor is checked, so that the two are
    // fetched together (an id out of range fetches object 0's image, which is then discarded).
    const bool k_ok = k >= 0 && k < a.max_objects;
    const int kc = k_ok ? k : 0;
    static_assert(H == 32 && L.B_off % 16 == 0, "weight images are kept for width 32");
    const unsigned char* img = a.img32 + (size_t)kc * img32_bytes(BF);
    const bool restage = (k != staged);
    if (restage) {  // the object's weight image, as it is, straight into LDS
      if (staged >= 0) __syncthreads();  // the previous object's weights are no longer read
      fetch_image_lds(img, smem, L.B_off, lane, wave, nw);
      staged = -1;
    }
    const ObjDesc& od = a.desc[kc];
    const int registered = od.registered, hidden = od.hidden;
    const double cx = od.centre[0], cy = od.centre[1], cz = od.centre[2];
    const double inv_s = od.inv_scale;
    float wseed = 1.0f, inv = 1.0f;
    if constexpr (TRAIN) {
      if (a.dloss) wseed = a.dloss[j];
      if (a.use_scale) {
        const float scale = a.scaler->scale;
        wseed *= scale;
        inv = 1.0f / scale;
      }
    }
    // the wave's first sub-tile's inputs are touched while the image is on its way (kept in
    // registers across the loop they would spill)
    const SubTileIn warm = subtile_inputs<TRAIN>(a, ray_lo, ray_hi, wave, rpw);
    if (!k_ok || !registered) {
      if (tid == 0) atomicOr(&a.scaler->device_error, 1);
      if (TABLE) __syncthreads();  // (the table in LDS is complete before a later tile reads it)
      continue;
    }
    if (kernel_width(hidden) != H) {  // handled by the launch for that width
      if (TABLE) __syncthreads();
      continue;
    }
    if (restage) {
      asm volatile("" ::"v"(warm.r.tt), "v"(warm.r.D), "v"(warm.r.M), "v"(warm.r.rgb[0]), "v"(warm.o[0]), "v"(warm.d[0]));
      __builtin_amdgcn_s_waitcnt(0);  // this thread's part of the image is in LDS
      staged = k;
    }
    __syncthreads();

    f32x16 accW[kLayers][MT][MT];
    f32x4 accWh[H / 16];  // BF16: output-layer weight gradient, 16x16 blocks (rows 0..3 used)
    float accH[kOut][MT];
    float accDb[kLayers][MT];
    float accDbH[kOut];
    if constexpr (TRAIN) {
#pragma unroll
      for (int l = 0; l < kLayers; ++l)
#pragma unroll
        for (int mo = 0; mo < MT; ++mo) {
          accDb[l][mo] = 0.f;
#pragma unroll
          for (int ki = 0; ki < MT; ++ki)
#pragma unroll
            for (int r = 0; r < 16; ++r) accW[l][mo][ki][r] = 0.f;
        }
#pragma unroll
      for (int c = 0; c < kOut; ++c) {
        accDbH[c] = 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) accH[c][mt] = 0.f;
      }
#pragma unroll
      for (int b = 0; b < H / 16; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) accWh[b][i] = 0.f;
    }
    float wave_loss = 0.f;

    unsigned char* const dzt = smem + L.scratch_off + wave * L.scratch_wave;
    unsigned char* const dtile = dzt + pair_dz_bytes(BF);
    unsigned char* const htile = dtile + kTile;                // BF16: one per pass
    unsigned char* const etile = htile + 2 * kTile;            // BF16: the encodings, one per pass

    for (int sub = wave; sub < nsub; sub += nw) {
      asm volatile("" ::: "memory");
      // the lane's index through an empty asm statement: lane-dependent LDS addresses are computed
      // where they are used, not hoisted out of the loop and spilled
      int ln = lane_;
      asm volatile("" : "+v"(ln));
      const int lane = ln, n = ln & 31, hf = ln >> 5;
      const int r0 = ray_lo + sub * rpw;
      const int nr = min(rpw, ray_hi - r0);
      const int nslots = nr * S;
      SubTileIn in = subtile_inputs<TRAIN>(a, ray_lo, ray_hi, sub, rpw);
      const RenderIn rin = in.r;
      // the lane's own sample: normalised point and (integrated encoding) normalised variance,
      // then handed to the two lanes that hold its pass's column
      float x[4] = {0.f, 0.f, 0.f, 0.f}, xt[2][4];
      if (lane < nslots) {
        const double tt = (double)rin.tt;
        x[0] = (float)(((double)in.o[0] + tt * (double)in.d[0] - cx) * inv_s);
        x[1] = (float)(((double)in.o[1] + tt * (double)in.d[1] - cy) * inv_s);
        x[2] = (float)(((double)in.o[2] + tt * (double)in.d[2] - cz) * inv_s);
        if (a.var) x[3] = (float)((double)in.var * inv_s * inv_s);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) half_split(x[c], xt[0][c], xt[1][c]);

      Acts<H, BF> act[2];  // kept for the backward
      float zs[kOut];
      forward_pair<BF>(xt, smem, Bl, lane, act, zs, a.var != nullptr);
      if constexpr (TRAIN && BF) {  // the first layer's weight gradient reads them from LDS
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj)
            write_runs(reinterpret_cast<__bf16*>(etile + p * kTile) + n * kTrStride + 16 * jj + 4 * hf, act[p].v[0][0][jj]);
      }

      float dzs[kOut];
      render_subtile<TRAIN>(a, r0, nslots, wseed, rin, zs, dzs, wave_loss);
      if constexpr (!TRAIN) {
        continue;
      }
#pragma unroll
      for (int c = 0; c < kOut; ++c) accDbH[c] += dzs[c];

      // ---------------- MLP backward of both passes, layer by layer together. The wave's LDS
      // accesses execute in order, so its staged tiles need no wait between writes and reads.
      float dz[2][kOut];  // FP32: each pass's dL/dz on both halves
      if constexpr (BF) {
        bf16x4 d4;
#pragma unroll
        for (int c = 0; c < kOut; ++c) {
          d4[c] = (__bf16)dzs[c];
          reinterpret_cast<__bf16*>(dzt)[c * kDzPitch + lane] = d4[c];
        }
        *reinterpret_cast<bf16x4*>(dzt + kOut * kDzPitch * 2 + 8 * lane) = d4;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj)
            write_runs(reinterpret_cast<__bf16*>(htile + p * kTile) + n * kTrStride + 16 * jj + 4 * hf, act[p].v[kLayers][0][jj]);
      } else {
#pragma unroll
        for (int c = 0; c < kOut; ++c) half_split(dzs[c], dz[0][c], dz[1][c]);
        *reinterpret_cast<f32x4*>(dzt + 16 * lane) = f32x4{dzs[0], dzs[1], dzs[2], dzs[3]};
      }
      wave_lds_order();
      Deltas<H, BF> dl[2];
      if constexpr (BF) {
        // output-layer weight gradient on MFMA 16x16x32: rows = the four outputs (padded to 16),
        // columns = 16 features, K = a pass's 32 samples
        const int m16 = lane & 15, kg = lane >> 4;
#pragma unroll
        for (int p = 1; p >= 0; --p) {
          bf16x8 da = {};
          if (m16 < kOut)
            da = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const __bf16*>(dzt) + m16 * kDzPitch + 32 * p + 8 * kg);
          // B operand (feature 16b + m16, samples 8kg..8kg+7): lane x of group kg addresses row
          // 8kg + x/4 at feature 16b + 4(x mod 4)
          const __bf16* hq = reinterpret_cast<const __bf16*>(htile + p * kTile) + (8 * kg + (m16 >> 2)) * kTrStride + 4 * (m16 & 3);
#pragma unroll
          for (int b = 0; b < H / 16; ++b) {
            const bf16x8 hb = tr_read8(hq + 16 * b);
            accWh[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(da, hb, accWh[b], 0, 0, 0);
          }
        }
        // delta of the last hidden layer: W_out^T dz on MFMA (K = 4 outputs padded to 16)
        bf16x8 wa = {};
        if (hf == 0) {
          const bf16x4 w4 = *reinterpret_cast<const bf16x4*>(smem + L.whtb_off + n * kOut * 2);
#pragma unroll
          for (int c = 0; c < kOut; ++c) wa[c] = w4[c];
        }
        f32x16 zero;
#pragma unroll
        for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          bf16x8 dzb = {};
          if (hf == 0) {
            const bf16x4 d4 = *reinterpret_cast<const bf16x4*>(dzt + kOut * kDzPitch * 2 + 8 * (32 * p + n));
#pragma unroll
            for (int c = 0; c < kOut; ++c) dzb[c] = d4[c];
          }
          const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, dzb, zero, 0, 0, 0);
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) dl[p].v[0][jj] = relu_mask(round8(acc, 8 * jj), act[p].v[kLayers][0][jj]);
        }
      } else {
        // output-layer weight gradient: lane owns feature n, half hf takes 16 samples of a pass
        const float* Wh = reinterpret_cast<const float*>(smem + L.wh_off);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            reinterpret_cast<float*>(htile)[n * (H + 4) + rowof(r, hf)] = act[p].v[kLayers][0][r];
          wave_lds_order();
#pragma unroll
          for (int s2 = 0; s2 < 16; ++s2) {
            const int s = 16 * hf + s2;
            const float hv = reinterpret_cast<const float*>(htile)[s * (H + 4) + n];
            const f32x4 d4 = *reinterpret_cast<const f32x4*>(dzt + 16 * (32 * p + s));
#pragma unroll
            for (int c = 0; c < kOut; ++c) accH[c][0] += d4[c] * hv;
          }
          wave_lds_order();
        }
        // delta of the last hidden layer: (W_out^T dz) masked by ReLU'
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float w[kOut];
#pragma unroll
          for (int c = 0; c < kOut; ++c) w[c] = Wh[c * (H + 4) + 16 * hf + r];
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < kOut; ++c) s += w[c] * dz[p][c];
            dl[p].set(0, r, (act[p].v[kLayers][0][r] > 0.f) ? s : 0.f);
          }
        }
      }
#pragma unroll
      for (int l = kLayers - 1; l >= 0; --l) {
        // delta_{l-1} = (W_l^T delta_l) masked by ReLU' of layer l-1: its products first, so that
        // they run while this layer's operands are staged and its weight gradient accumulates
        f32x16 nacc[2];
        if (l > 0) {
#pragma unroll
          for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int r = 0; r < 16; ++r) nacc[p][r] = 0.f;
          if constexpr (BF) {
            // A = W_l^T from its transposed copy: 8 consecutive BF16 per lane
            const __bf16* Wt = reinterpret_cast<const __bf16*>(smem + L.wt_off[l]) + n * (H + 8) + 16 * hf;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
              const bf16x8 wa = *reinterpret_cast<const bf16x8*>(Wt + 8 * jj);
#pragma unroll
              for (int p = 0; p < 2; ++p)
                nacc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, dl[p].v[0][jj], nacc[p], 0, 0, 0);
            }
          } else {
            const float* W = reinterpret_cast<const float*>(smem + L.w_off[l]) + colpos(n);
#pragma unroll
            for (int qq = 0; qq < 16; ++qq) {
              const float w = W[rowof(qq, hf) * L.w_stride[l]];
#pragma unroll
              for (int p = 0; p < 2; ++p)
                nacc[p] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, dl[p].v[0][qq], nacc[p], 0, 0, 0);
            }
          }
        }
        // stage delta_l (out features) and h_{l-1} (in features), sample-major, and accumulate the
        // weight gradient dW_l += delta_l h_{l-1}^T over each pass's 32 samples
        if constexpr (BF) {
          if (l > 0) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
              for (int jj = 0; jj < 2; ++jj)
                write_runs(reinterpret_cast<__bf16*>(htile + p * kTile) + n * kTrStride + 16 * jj + 4 * hf, act[p].v[l][0][jj]);
          }
          const unsigned char* const ht = l > 0 ? htile : etile;
#pragma unroll
          for (int p = 1; p >= 0; --p) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
              write_runs(reinterpret_cast<__bf16*>(dtile) + n * kTrStride + 16 * jj + 4 * hf, dl[p].v[0][jj]);
            wave_lds_order();
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
              // A and B operands (feature row lane & 31, samples 16jj + 8hf + 0..7): lane x of
              // group G = lane / 16 addresses row 16jj + 8(G / 2) + x/4 at feature
              // 16(G mod 2) + 4(x mod 4)
              const int lo = (16 * jj + 8 * hf + ((lane & 15) >> 2)) * kTrStride + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
              const bf16x8 da = tr_read8(reinterpret_cast<const __bf16*>(dtile) + lo);
              const bf16x8 hb = tr_read8(reinterpret_cast<const __bf16*>(ht + p * kTile) + lo);
              accW[l][0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(da, hb, accW[l][0][0], 0, 0, 0);
              // bias gradient: the 8 deltas' sum, two at a time (v_dot2)
              typedef unsigned int u4 __attribute__((ext_vector_type(4)));
              typedef __bf16 b2 __attribute__((ext_vector_type(2)));
              const u4 dw = __builtin_bit_cast(u4, da);
              const b2 ones = {(__bf16)1.0f, (__bf16)1.0f};
              float s = 0.f;
#pragma unroll
              for (int e = 0; e < 4; ++e)
                s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2, (unsigned int)dw[e]), ones, s, false);
              accDb[l][0] += s;
            }
            wave_lds_order();
          }
        } else {
#pragma unroll
          for (int p = 0; p < 2; ++p) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              reinterpret_cast<float*>(dtile)[n * (H + 4) + rowof(r, hf)] = dl[p].v[0][r];
              reinterpret_cast<float*>(htile)[n * (H + 4) + rowof(r, hf)] = act[p].v[l][0][r];
            }
            wave_lds_order();
#pragma unroll
            for (int qq = 0; qq < 16; ++qq) {
              const int s = 2 * qq + hf;
              const float da = reinterpret_cast<const float*>(dtile)[s * (H + 4) + n];
              const float hb = reinterpret_cast<const float*>(htile)[s * (H + 4) + n];
              accW[l][0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(da, hb, accW[l][0][0], 0, 0, 0);
              accDb[l][0] += da;
            }
            wave_lds_order();
          }
        }
        if (l == 0) break;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          if constexpr (BF) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) dl[p].v[0][jj] = relu_mask(round8(nacc[p], 8 * jj), act[p].v[l][0][jj]);
          } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) dl[p].set(0, r, (act[p].v[l][0][r] > 0.f) ? nacc[p][r] : 0.f);
          }
        }
      }
    }  // sub-tiles

    // ---------------- combine the waves of the workgroup in a fixed order
    // per-wave reductions in registers first
    wave_loss = wave_sum(wave_loss);
    if constexpr (TRAIN) {
#pragma unroll
      for (int c = 0; c < kOut; ++c) {
        accDbH[c] = wave_sum(accDbH[c]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) accH[c][mt] = half_sum(accH[c][mt]);
      }
#pragma unroll
      for (int l = 0; l < kLayers; ++l)
#pragma unroll
        for (int mo = 0; mo < MT; ++mo) accDb[l][mo] = half_sum(accDb[l][mo]);
    }
    __syncthreads();  // staging buffers and weights are free: reuse them for the tile's gradient
    // nc copies of the tile's gradient and loss. Four waves write a copy each (the fourth over the
    // weights, which the next tile stages again) and the partial is (0 + 2) + (1 + 3): one barrier,
    // no read-modify-write (two copies, to which waves 2 and 3 added theirs after a barrier, took
    // 7.9 thousand cycles to the sum, a fifth of a tile of two sub-tiles per wave). Other wave
    // counts keep red_copies(nw) copies (two for two to seven waves, four for eight): the first nc
    // waves write them, the others then add theirs in turn (copy c = waves c, c + nc, ..., in that
    // order), and the partial is the sum of the copies in order: the same sum for four waves.
    constexpr int kRedWords = kRedCopyBytes / 4;
    static_assert(kRedCopyBytes <= L.B_off, "the fourth copy ends before the encoding matrix, which is loaded once");
    const bool four = (nw == 4);
    const int nc = four ? 4 : red_copies(nw);
    float* red0 = reinterpret_cast<float*>(smem + L.scratch_off);
    float* red3 = four ? reinterpret_cast<float*>(smem) : red0 + 3 * kRedWords;  // the fourth copy
    float* red = (wave % nc == 3) ? red3 : red0 + (wave % nc) * kRedWords;
    float* lsum = reinterpret_cast<float*>(smem + L.loss_off);
    int* any_bad = reinterpret_cast<int*>(smem + L.loss_off + 16);
    if (tid == 0) *any_bad = 0;  // read after the barriers below
    // lane, n and hf again, through an empty asm statement: the addresses below are then computed
    // here, not hoisted to the kernel's start and kept (spilled) across the sub-tiles
    int rl = lane;
    asm volatile("" : "+v"(rl));
    const int rn = rl & 31, rh = rl >> 5, et = 64 * wave + rl;
    for (int ph = 0; ph < (nw + nc - 1) / nc; ++ph) {
      if (wave / nc == ph) {
        const bool first = (ph == 0);
        if (rl == 0) lsum[wave % nc] = (first ? 0.f : lsum[wave % nc]) + wave_loss;
        if constexpr (TRAIN) {
          int off = 0;
#pragma unroll
          for (int l = 0; l < kLayers; ++l) {
            const int K = (l == 0) ? kEnc : H;
            const int KB = K / 32;
#pragma unroll
            for (int mo = 0; mo < MT; ++mo)
#pragma unroll
              for (int ki = 0; ki < KB; ++ki)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  const int idx = off + (mo * 32 + rowof(r, rh)) * K + ki * 32 + rn;
                  red[idx] = (first ? 0.f : red[idx]) + accW[l][mo][ki][r];
                }
            off += H * K;
            if (rh == 0) {
#pragma unroll
              for (int mo = 0; mo < MT; ++mo) {
                const int idx = off + mo * 32 + rn;
                red[idx] = (first ? 0.f : red[idx]) + accDb[l][mo];
              }
            }
            off += H;
          }
          if constexpr (BF) {
            if (rl < 16) {
#pragma unroll
              for (int c = 0; c < kOut; ++c)
#pragma unroll
                for (int b = 0; b < H / 16; ++b) {
                  const int idx = off + c * H + b * 16 + rl;
                  red[idx] = (first ? 0.f : red[idx]) + accWh[b][c];
                }
            }
          } else if (rh == 0) {
#pragma unroll
            for (int c = 0; c < kOut; ++c)
#pragma unroll
              for (int mt = 0; mt < MT; ++mt) {
                const int idx = off + c * H + mt * 32 + rn;
                red[idx] = (first ? 0.f : red[idx]) + accH[c][mt];
              }
          }
          off += kOut * H;
          if (rl == 0) {
#pragma unroll
            for (int c = 0; c < kOut; ++c) red[off + c] = (first ? 0.f : red[off + c]) + accDbH[c];
          }
        }
      }
      __syncthreads();
    }
    if constexpr (TRAIN) {
      // unscale (exact: the scale is a power of two) and report a partial that is not finite or
      // too large to be summed safely (partial_bad)
      static_assert(n_params_of(H) % 4 == 0, "the partial is written four elements at a time");
      float* dst = a.partial + (size_t)slot * a.p_stride;  // (p_stride is a multiple of 64)
      int bad = 0;
      for (int e = 4 * et; e < n_params_of(H); e += 4 * blockDim.x) {
        f32x4 g = *reinterpret_cast<const f32x4*>(red0 + e);
        if (four) {
          g = (g + *reinterpret_cast<const f32x4*>(red0 + 2 * kRedWords + e)) +
              (*reinterpret_cast<const f32x4*>(red0 + kRedWords + e) + *reinterpret_cast<const f32x4*>(red3 + e));
        } else {
          for (int c = 1; c < nc; ++c) g += *reinterpret_cast<const f32x4*>((c == 3 ? red3 : red0 + c * kRedWords) + e);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          g[i] *= inv;
          bad |= partial_bad(g[i]);
        }
        __builtin_nontemporal_store(g, reinterpret_cast<f32x4*>(dst + e));  // read once, by the next kernel
      }
      if (four) staged = -1;  // the fourth copy lies over the weights
      if (bad) *any_bad = 1;  // every writer stores the same value
      __syncthreads();
      if (tid == 0) {
        if constexpr (TABLE) a.tile_bad[slot] = *any_bad;
        else if (*any_bad) atomicOr(&a.flags[k], 1);
      }
    }
    if (tid == 0) {
      float l = lsum[0];
      if (four) l = (l + lsum[2]) + (lsum[1] + lsum[3]);
      else for (int c = 1; c < nc; ++c) l += lsum[c];
      a.tile_loss[slot] = l;
    }
    __syncthreads();
  }
}

// Batch object of element t (a row tile, row block or work tile) of a chain given by its exclusive
// scan: the largest j below n_objects with scan[j] <= t (objects without elements have an empty
// range and are passed over; scan[0] = 0 <= t). Searched by the whole wave, 64 ways at a time: the
// lanes read 64 evenly spaced entries of the remaining range together and a ballot keeps the last
// one at or below t, so a lookup waits on ceil(log64 n) loads rather than log2 n dependent ones.
// Every lane of the wave must be active and pass the same t.
__device__ __forceinline__ int gen_object(const int32_t* __restrict__ scan, int n_objects, int t) {
  const int lane = (int)(threadIdx.x & 63);
  int lo = 0, len = n_objects;  // the answer lies in [lo, lo + len), scan[lo] <= t
  while (len > 1) {
    const int step = (len + 63) >> 6;
    const int i = lane * step;
    const bool le = i < len && scan[lo + i] <= t;  // a prefix of the lanes (scan is nondecreasing)
    const int c = __popcll(__ballot(le)) - 1;      // lane 0 always counts
    lo += c * step;
    len = min(step, len - c * step);
  }
  return lo;
}

// Sum of the eight BF16 of an MFMA operand, two at a time (v_dot2 against ones), added to s.
__device__ __forceinline__ float operand_sum(bf16x8 v, float s) {
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  const u4 w = __builtin_bit_cast(u4, v);
  const b2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2, (unsigned int)w[e]), ones, s, false);
  return s;
}

// ---------------------------------------------------------------------------------------------
// Tile kernel for hidden 64 in BF16: the four waves of a workgroup take a sub-tile each and split
// every weight gradient by rows, over the 128 samples of the four waves' current pass, as
// k_step_coop does (below). Two workgroups fit on a CU (256 registers, 77 KB of LDS), so that one
// runs while the other waits at a barrier or for its chain of products:
//   - the forward takes a sub-tile's two passes together (each weight operand read once for both);
//     each pass's activations are recomputed for its backward, from its encoding (kept through the
//     rendering they spill);
//   - the input-gradient products read W transposed (ds_read_b64_tr_b16) from the forward's copy;
//   - deltas and activations are staged sample-major in 8-byte runs and read transposed, where
//     k_step_coop stores single BF16 values.
// The LDS reads bound it: per round of four sub-tiles about 1.3 MB a CU, 10 thousand cycles.
// 256 objects, 558,935 rays of 32 samples: 7.05 ms for k_step_coop (one wave per SIMD, 412
// registers), 2.81 ms here.

struct Lds64 {
  int w_off[kLayers];  // W_l, BF16, permuted columns, row stride 40 (l = 0) or 72
  int bA_off;          // biases as (hi, mid, lo, 0 ...): 16 bytes per row
  int whb_off;         // output weights [4][72], permuted columns
  int whtb_off;        // output weights transposed [64][4]
  int bh_off, B_off, loss_off;
  int scratch_off, scratch_wave, total;
};
constexpr int kS64 = 68;                                          // BF16 elements per staged sample
constexpr int kDz64 = kDzRowsBytes + 32 * kOut * 2;               // seeds of a pass (both layouts)
constexpr int kTile64 = 32 * kS64 * 2;
__host__ __device__ constexpr int w_stride64(int l) { return l == 0 ? kEnc + 8 : 72; }
__host__ __device__ constexpr Lds64 lds64() {
  Lds64 L{};
  int off = 0;
  for (int l = 0; l < kLayers; ++l) {
    L.w_off[l] = off;
    off += 64 * w_stride64(l) * 2;
  }
  L.bA_off = off; off += kLayers * 64 * 16;
  L.whb_off = off; off += kOut * 72 * 2;
  L.whtb_off = off; off += 64 * kOut * 2;
  L.bh_off = off; off += 16;
  L.B_off = off; off += 3 * kFeatures * 4;
  L.loss_off = off; off += 32;
  L.scratch_off = round_up(off, 16);
  L.scratch_wave = kDz64 + 2 * kTile64;
  L.total = L.scratch_off + 4 * L.scratch_wave;
  return L;
}
static_assert(2 * lds64().total <= 160 * 1024, "two workgroups of the hidden-64 kernel on a CU");

// Eight BF16 of a transposing read: rows r..r+3 at p, rows further down at p + second.
__device__ __forceinline__ bf16x8 tr_read_pair(const __bf16* p, int second) {
  typedef __attribute__((address_space(3))) v4i16 lds_v4;
  const v4i16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p));
  const v4i16 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p + second));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Object's parameters into LDS by 256 threads, 16-byte loads all in flight together.
__device__ __forceinline__ void stage64(const float* __restrict__ th, unsigned char* smem, int tid) {
  asm volatile("" : "+v"(tid));  // (addresses are computed here, not kept from the kernel's start)
  constexpr Lds64 L = lds64();
  constexpr int H = 64;
  f32x4 x[14];
  int q = 0;
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    const float* W = th + layer_param_off(H, l);
#pragma unroll
    for (int i = 0; i < (l == 0 ? 2 : 4); ++i) x[q++] = *reinterpret_cast<const f32x4*>(W + 4 * (tid + 256 * i));
  }
  const int bl = tid >> 6, br = tid & 63;
  const float b = th[layer_param_off(H, bl) + H * (bl == 0 ? kEnc : H) + br];
  const float wh = th[layer_param_off(H, kLayers) + tid];
  const float bh = tid < kOut ? th[layer_param_off(H, kLayers) + kOut * H + tid] : 0.f;
  typedef unsigned int u2w __attribute__((ext_vector_type(2)));
  q = 0;
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    const int K = (l == 0) ? kEnc : H;
#pragma unroll
    for (int i = 0; i < (l == 0 ? 2 : 4); ++i, ++q) {
      const int e = 4 * (tid + 256 * i), row = e / K, col = e % K;
      *reinterpret_cast<u2w*>(smem + L.w_off[l] + (row * w_stride64(l) + (col & ~31) + colpos(col & 31)) * 2) =
          u2w{pack2(x[q][0], x[q][1]), pack2(x[q][2], x[q][3])};
    }
  }
  const __bf16 hi = (__bf16)b;
  const __bf16 mid = (__bf16)(b - (float)hi);
  const __bf16 lo = (__bf16)((b - (float)hi) - (float)mid);
  bf16x8 pieces = {};
  pieces[0] = hi;
  pieces[1] = mid;
  pieces[2] = lo;
  *reinterpret_cast<bf16x8*>(smem + L.bA_off + 16 * tid) = pieces;
  reinterpret_cast<__bf16*>(smem + L.whb_off)[bl * 72 + (br & ~31) + colpos(br & 31)] = (__bf16)wh;
  reinterpret_cast<__bf16*>(smem + L.whtb_off)[br * kOut + bl] = (__bf16)wh;
  if (tid < kOut) reinterpret_cast<float*>(smem + L.bh_off)[tid] = bh;
}

// One layer of NP passes: out = ReLU(W_l in + b), rounded to BF16 in the accumulator layout.
template <int NP>
__device__ __forceinline__ void layer64(const unsigned char* smem, int l, int lane, const bf16x8 (&in)[NP][2][2],
                                        bf16x8 (&out)[NP][2][2]) {
  constexpr Lds64 L = lds64();
  const int n = lane & 31, hf = lane >> 5, ws = w_stride64(l), KB = (l == 0) ? 1 : 2;
  asm volatile("" ::: "memory");  // weight reads stay in their layer
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
  for (int mo = 0; mo < 2; ++mo) {
    bf16x8 ba = {};
    if (hf == 0) ba = *reinterpret_cast<const bf16x8*>(smem + L.bA_off + 16 * (l * 64 + mo * 32 + n));
    const bf16x8 ones3 = {(__bf16)1.0f, (__bf16)1.0f, (__bf16)1.0f, (__bf16)0.0f,
                          (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f};
    const f32x16 b16 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ba, ones3, zero, 0, 0, 0);
    f32x16 acc[NP];
    const __bf16* wrow = reinterpret_cast<const __bf16*>(smem + L.w_off[l]) + (mo * 32 + n) * ws + 16 * hf;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const bf16x8 wa = *reinterpret_cast<const bf16x8*>(wrow + kb * 32 + 8 * jj);
#pragma unroll
        for (int p = 0; p < NP; ++p)
          acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, in[p][kb][jj], (kb == 0 && jj == 0) ? b16 : acc[p], 0, 0, 0);
      }
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) out[p][mo][jj] = relu_round8(acc[p], 8 * jj);
  }
}

template <int MODE>
__global__ void __launch_bounds__(256, 2) k_step_64(const StepArgs a_in) {
  constexpr int H = 64;
  constexpr bool TRAIN = (MODE == MODE_TRAIN);
  constexpr Lds64 L = lds64();
  constexpr int RW = H / 4;         // weight-gradient rows of one wave
  StepArgs a = a_in;
  read_batch(a);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane_ = tid & 63, wave = tid >> 6;
  const int S = a.S;
  const int rpw = kSlots / S;
  const int n_tiles = clamp_tiles(a.width_start[a.n_objects], a.max_tiles);  // of this width
  float* Bl = reinterpret_cast<float*>(smem + L.B_off);
  if (tid < 3 * kFeatures) Bl[tid] = a.B[tid];
  int staged = -1;

  for (int t = first_tile_of_block(blockIdx.x, gridDim.x, n_tiles); t < n_tiles; t += gridDim.x) {
    const int j = gen_object(a.width_start, a.n_objects, t);
    const int ti = t - a.width_start[j], tile = a.tile_start[j] + ti;  // of the object; of the work list
    if (tile < 0 || tile >= a.max_tiles) continue;  // (not for a consistent work list)
    const int k = __builtin_amdgcn_readfirstlane(a.object_ids[j]);
    if (k < 0 || k >= a.max_objects || !a.desc[k].registered) {
      if (tid == 0) atomicOr(&a.scaler->device_error, 1);
      continue;
    }
    if (kernel_width(a.desc[k].hidden) != H) continue;
    const int rpt = tile_rays(H, a.rays_per_tile, a.rays_per_tile_wide);
    const RayRange rr = tile_ray_range(a.ray_offsets[j], a.ray_offsets[j + 1], ti, rpt, a.n_rays);
    const int ray_lo = rr.lo, ray_hi = rr.hi;
    if (k != staged) {
      __syncthreads();
      stage64(a.theta + (size_t)k * a.p_stride, smem, tid);
      staged = k;
    }
    __syncthreads();
    const double cx = a.desc[k].centre[0], cy = a.desc[k].centre[1], cz = a.desc[k].centre[2];
    const double inv_s = a.desc[k].inv_scale;
    float wseed = 1.0f, inv = 1.0f;
    if constexpr (TRAIN) {
      if (a.dloss) wseed = a.dloss[j];
      if (a.use_scale) {
        const float scale = a.scaler->scale;
        wseed *= scale;
        inv = 1.0f / scale;
      }
    }

    f32x4 accW[kLayers][4];  // this wave's 16 rows of dW_l, 16-column blocks (layer 0: two)
    float accDb[kLayers];    // lane sums of this wave's rows of db_l
    f32x4 accWh;             // this wave's 16 columns of the output layer's dW
    float accDbH[kOut];
    if constexpr (TRAIN) {
#pragma unroll
      for (int l = 0; l < kLayers; ++l) {
        accDb[l] = 0.f;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) accW[l][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      accWh = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < kOut; ++c) accDbH[c] = 0.f;
    }
    float wave_loss = 0.f;
    unsigned char* const scr0 = smem + L.scratch_off;
    unsigned char* const dzt = scr0 + wave * L.scratch_wave;
    unsigned char* const dtile = dzt + kDz64;
    unsigned char* const htile = dtile + kTile64;
    const int nsub = (ray_hi - ray_lo + rpw - 1) / rpw;
    const int rounds = (nsub + 3) / 4;

    // Every wave runs every round (a wave without a sub-tile carries zero seeds), since the
    // weight-gradient products of a round read all four waves' staging tiles.
    for (int rd = 0; rd < rounds; ++rd) {
      // (lane-dependent LDS addresses are computed where they are used, not hoisted and spilled)
      int ln = lane_;
      asm volatile("" : "+v"(ln)::"memory");
      const int lane = ln, n = ln & 31, hf = ln >> 5;
      const int sub = rd * 4 + wave;
      const int r0 = ray_lo + sub * rpw;
      const int nslots = max(0, min(rpw, ray_hi - r0)) * S;
      const SubTileIn in = subtile_inputs<TRAIN>(a, ray_lo, ray_hi, sub, rpw);
      float x[4] = {0.f, 0.f, 0.f, 0.f}, xt[2][4];
      if (lane < nslots) {
        const double tt = (double)in.r.tt;
        x[0] = (float)(((double)in.o[0] + tt * (double)in.d[0] - cx) * inv_s);
        x[1] = (float)(((double)in.o[1] + tt * (double)in.d[1] - cy) * inv_s);
        x[2] = (float)(((double)in.o[2] + tt * (double)in.d[2] - cz) * inv_s);
        if (a.var) x[3] = (float)((double)in.var * inv_s * inv_s);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) half_split(x[c], xt[0][c], xt[1][c]);
      Acts<32, true> E[2];  // layer 0 only: the encodings
      if (a.var) encode_pair<true, true>(xt, Bl, hf, E);
      else encode_pair<true, false>(xt, Bl, hf, E);

      // forward of both passes, for the outputs alone
      bf16x8 h[2][2][2];
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) h[p][0][jj] = E[p].v[0][0][jj];
#pragma unroll
      for (int l = 0; l < kLayers; ++l) {
        bf16x8 o[2][2][2];
        layer64<2>(smem, l, lane, h, o);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) h[p][mt][jj] = o[p][mt][jj];
      }
      f32x16 zero;
#pragma unroll
      for (int r = 0; r < 16; ++r) zero[r] = 0.f;
      float zs[kOut];
      {
        const __bf16* wh = reinterpret_cast<const __bf16*>(smem + L.whb_off) + n * 72 + 16 * hf;
        f32x16 acc[2] = {zero, zero};
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            bf16x8 wa = {};
            if (n < kOut) wa = *reinterpret_cast<const bf16x8*>(wh + mt * 32 + 8 * jj);
#pragma unroll
            for (int p = 0; p < 2; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, h[p][mt][jj], acc[p], 0, 0, 0);
          }
        const float* bh = reinterpret_cast<const float*>(smem + L.bh_off);
#pragma unroll
        for (int c = 0; c < kOut; ++c) {
          float unused;
          half_join(acc[0][c] + bh[c], acc[1][c] + bh[c], zs[c], unused);
        }
      }
      float dzs[kOut];
      render_subtile<TRAIN>(a, r0, nslots, wseed, in.r, zs, dzs, wave_loss);
      if constexpr (!TRAIN) continue;
#pragma unroll
      for (int c = 0; c < kOut; ++c) accDbH[c] += dzs[c];

      const int m16 = lane & 15, kg = lane >> 4;
      // this lane's place in a transposing read of a staged tile: K = samples 8 kg + 0..7 (rows),
      // the operand's row or column = feature base + m16
      const int tr0 = (8 * kg + (m16 >> 2)) * kS64 + 4 * (m16 & 3);
      // ... and of W_l^T: in-feature n of block mi, the outputs of K slot (hf, e) of block ko
      const int wc = 4 * (m16 & 3) + 16 * (kg & 1);
      const int wt0 = (4 * hf + (m16 >> 2)) * 72 + colpos(wc);
#pragma unroll 1
      for (int p = 0; p < 2; ++p) {
        // the pass's activations again, from its encoding
        bf16x8 act[kLayers + 1][2][2];
        {
          bf16x8 c[1][2][2];
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) act[0][0][jj] = c[0][0][jj] = (p == 0) ? E[0].v[0][0][jj] : E[1].v[0][0][jj];
#pragma unroll
          for (int l = 0; l < kLayers; ++l) {
            bf16x8 o[1][2][2];
            layer64<1>(smem, l, lane, c, o);
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
              for (int jj = 0; jj < 2; ++jj) act[l + 1][mt][jj] = c[0][mt][jj] = o[0][mt][jj];
          }
        }
        __syncthreads();  // every wave is done reading the staging tiles
        if (hf == p) {    // the pass's seeds, by the lanes that hold them
          bf16x4 d4;
#pragma unroll
          for (int c = 0; c < kOut; ++c) {
            d4[c] = (__bf16)dzs[c];
            reinterpret_cast<__bf16*>(dzt)[c * 40 + n] = d4[c];
          }
          *reinterpret_cast<bf16x4*>(dzt + kDzRowsBytes + 8 * n) = d4;
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj)
            write_runs(reinterpret_cast<__bf16*>(htile) + n * kS64 + mt * 32 + 16 * jj + 4 * hf, act[kLayers][mt][jj]);
        __syncthreads();
        // output layer: this wave's 16 columns of dW over the four waves' samples
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
          const unsigned char* dz2 = scr0 + w2 * L.scratch_wave;
          bf16x8 da = {};
          if (m16 < kOut)
            da = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const __bf16*>(dz2) + m16 * 40 + 8 * kg);
          const bf16x8 hb = tr_read_pair(reinterpret_cast<const __bf16*>(dz2 + kDz64 + kTile64) + tr0 + 16 * wave, 4 * kS64);
          accWh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(da, hb, accWh, 0, 0, 0);
        }
        // delta of the last hidden layer, own samples: (W_out^T dz) masked by ReLU'
        bf16x8 dl[2][2];
        {
          bf16x8 dzb = {};
          if (hf == 0) {
            const bf16x4 d4 = *reinterpret_cast<const bf16x4*>(dzt + kDzRowsBytes + 8 * n);
#pragma unroll
            for (int c = 0; c < kOut; ++c) dzb[c] = d4[c];
          }
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) {
            bf16x8 wa = {};
            if (hf == 0) {
              const bf16x4 w4 = *reinterpret_cast<const bf16x4*>(smem + L.whtb_off + (mt * 32 + n) * kOut * 2);
#pragma unroll
              for (int c = 0; c < kOut; ++c) wa[c] = w4[c];
            }
            const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, dzb, zero, 0, 0, 0);
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) dl[mt][jj] = relu_mask(round8(acc, 8 * jj), act[kLayers][mt][jj]);
          }
        }
#pragma unroll
        for (int l = kLayers - 1; l >= 0; --l) {
          const int KB = (l == 0) ? 1 : 2;
          // delta_{l-1} = W_l^T delta_l, own samples, before this layer's operands are staged
          f32x16 nacc[2];
          if (l > 0) {
            const __bf16* W = reinterpret_cast<const __bf16*>(smem + L.w_off[l]) + wt0;
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
              nacc[mi] = zero;
#pragma unroll
              for (int ko = 0; ko < 2; ++ko)
#pragma unroll
                for (int jj = 0; jj < 2; ++jj) {
                  const bf16x8 wa = tr_read_pair(W + (ko * 32 + 16 * jj) * 72 + mi * 32, 8 * 72);
                  nacc[mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, dl[ko][jj], nacc[mi], 0, 0, 0);
                }
            }
          }
          __syncthreads();  // every wave is done reading the staging tiles
#pragma unroll
          for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
              write_runs(reinterpret_cast<__bf16*>(dtile) + n * kS64 + mt * 32 + 16 * jj + 4 * hf, dl[mt][jj]);
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
              write_runs(reinterpret_cast<__bf16*>(htile) + n * kS64 + kb * 32 + 16 * jj + 4 * hf, act[l][kb][jj]);
          __syncthreads();  // every wave's tiles are staged
          // this wave's rows of dW_l: D lane holds row 4 kg + i, column 16 cb + m16
#pragma unroll
          for (int w2 = 0; w2 < 4; ++w2) {
            const __bf16* d2 = reinterpret_cast<const __bf16*>(scr0 + w2 * L.scratch_wave + kDz64) + tr0;
            const __bf16* h2 = d2 + kTile64 / 2;
            const bf16x8 da = tr_read_pair(d2 + wave * RW, 4 * kS64);
            accDb[l] += operand_sum(da, 0.f);
#pragma unroll
            for (int cb = 0; cb < 2 * KB; ++cb) {
              const bf16x8 hb = tr_read_pair(h2 + 16 * cb, 4 * kS64);
              accW[l][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(da, hb, accW[l][cb], 0, 0, 0);
            }
          }
          if (l == 0) break;
#pragma unroll
          for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) dl[mi][jj] = relu_mask(round8(nacc[mi], 8 * jj), act[l][mi][jj]);
        }
      }
    }  // rounds

    // ---------------- tile result: loss and output-layer bias combined in wave order, every
    // wave writes its own gradient slices
    int le = lane_;
    asm volatile("" : "+v"(le));
    const int lane = le, m16 = lane & 15, kg = lane >> 4;
    int bad = 0;
    float* dst = a.partial + (size_t)tile * a.p_stride;
    wave_loss = wave_sum(wave_loss);
    if constexpr (TRAIN) {
#pragma unroll
      for (int c = 0; c < kOut; ++c) accDbH[c] = wave_sum(accDbH[c]);
#pragma unroll
      for (int l = 0; l < kLayers; ++l) {
        accDb[l] += __shfl_xor(accDb[l], 16);
        accDb[l] += __shfl_xor(accDb[l], 32);
      }
    }
    float* lsum = reinterpret_cast<float*>(smem + L.loss_off);
    int* any_bad = reinterpret_cast<int*>(smem + L.loss_off + 20);
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
      if (wave == w && lane == 0) {
        lsum[0] = (w == 0 ? 0.f : lsum[0]) + wave_loss;
        if constexpr (TRAIN) {
#pragma unroll
          for (int c = 0; c < kOut; ++c) lsum[1 + c] = (w == 0 ? 0.f : lsum[1 + c]) + accDbH[c];
          if (w == 0) *any_bad = 0;
        }
      }
      __syncthreads();
    }
    if constexpr (TRAIN) {
      auto put = [&](int idx, float g) {
        g *= inv;
        bad |= partial_bad(g);
        dst[idx] = g;
      };
#pragma unroll
      for (int l = 0; l < kLayers; ++l) {
        const int K = (l == 0) ? kEnc : H;
        const int off = layer_param_off(H, l);
#pragma unroll
        for (int cb = 0; cb < K / 16; ++cb)
#pragma unroll
          for (int i = 0; i < 4; ++i) put(off + (wave * RW + 4 * kg + i) * K + cb * 16 + m16, accW[l][cb][i]);
        if (kg == 0) put(off + H * K + wave * RW + m16, accDb[l]);
      }
      const int offh = layer_param_off(H, kLayers);
      if (lane < 16) {
#pragma unroll
        for (int c = 0; c < kOut; ++c) put(offh + c * H + wave * 16 + lane, accWh[c]);
      }
      if (wave == 0 && lane < kOut) put(offh + kOut * H + lane, lsum[1 + lane]);
      if (bad) *any_bad = 1;  // every writer stores the same value
      __syncthreads();
      if (tid == 0 && *any_bad) atomicOr(&a.flags[k], 1);
    }
    if (tid == 0) a.tile_loss[tile] = lsum[0];
    __syncthreads();
  }
}

// Lane `lane`'s MFMA operand from a row-major BF16 tile T (pitch P elements, a multiple of 4): the
// operand's K index runs down the rows kb + 8 (lane / 32) + 0..7 and its row or column index is
// column cb + (lane mod 32). Lanes x, x + 4, x + 8 and x + 12 of each 16-lane group address four
// consecutive rows at the same four-column run, so each ds_read_b64_tr_b16 hands every lane four
// consecutive rows of its own column (the lane mapping the fused kernels' weight gradients use);
// the second read, four rows further down, gives the other four of its eight.
template <int P>
__device__ __forceinline__ bf16x8 tr_operand(const uint16_t* T, int kb, int cb, int lane) {
  typedef __attribute__((address_space(3))) v4i16 lds_v4;
  const uint16_t* p = T + (kb + 8 * (lane >> 5) + ((lane & 15) >> 2)) * P + cb + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const v4i16 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p));
  const v4i16 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p + 4 * P));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
}

// ---------------------------------------------------------------------------------------------
// Training tile kernel for hidden 128 (BF16): eight waves work on one sub-tile together. Wave w
// computes the 32 x 32 block (features 32 (w mod 4).., samples of pass w / 4) of every layer, so
// the chain of a sub-tile is four blocks' length, not four times four; activations and deltas pass
// between layers through LDS, beside the object's weights (112 KB of the image; the input gradient
// reads them transposed). Each weight gradient's sixteen 32 x 32 blocks are split two to a wave and
// accumulate in registers over the tile's sub-tiles (112 of them), so the partial is written once.
//
// k_step_coop ran a sub-tile per wave, one wave per SIMD, spilling, with weights read from device
// memory for every product and the gradient read and written there for every layer and pass: 179
// us for a background of 1,200 rays of 20 samples (100 tiles, 24,000 samples); 46 us here. The
// LDS bounds it: a sub-tile's products read 1.1 MB of operands (about 9 thousand cycles).
//
// Columns of staged tiles (activations, deltas) and of the weights are in the permuted order of
// colpos: a wave's accumulator registers are sixteen consecutive columns, written as two 16-byte
// stores and read back as the next layer's operands.

struct Lds128 {
  int B_off, loss_off, lane_loss_off, dz_off, enc_off, buf_off, total;
};
constexpr int kS128 = 136;  // BF16 elements per staged sample of 128 features
constexpr int kE128 = 40;   // ... of 32 encodings
__host__ __device__ constexpr Lds128 lds128() {
  Lds128 L{};
  int off = lds_layout(128, true, 1).B_off;  // the weight image's bytes
  L.B_off = off; off += 3 * kFeatures * 4;
  L.loss_off = off; off += 32;
  L.lane_loss_off = off; off += 4 * kWave * 4;
  L.dz_off = off; off += pair_dz_bytes(true);
  L.enc_off = off; off += 64 * kE128 * 2;
  L.buf_off = off; off += 2 * 64 * kS128 * 2;
  L.total = off;
  return L;
}
static_assert(lds128().total <= 160 * 1024, "the hidden-128 kernel's LDS");
// Feature at permuted column `pos` (0..31) of a block: the inverse of colpos.
__host__ __device__ constexpr int colfeat(int pos) { return (((pos >> 2) & 3) << 3) + ((pos >> 4) << 2) + (pos & 3); }

__global__ void __launch_bounds__(512, 2) k_step_128(const StepArgs a_in) {
  constexpr int H = 128;
  constexpr LdsLayout W = lds_layout(H, true, 1);
  constexpr Lds128 L = lds128();
  StepArgs a = a_in;
  read_batch(a);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane_ = tid & 63, wave = tid >> 6;
  const int fb = wave & 3, pass = wave >> 2;    // this wave's feature block and pass
  const int ob = wave >> 1, ib = (wave & 1) * 2;  // its weight-gradient blocks: outputs ob, inputs ib and ib + 1
  const int S = a.S;
  const int rpw = kSlots / S;
  const int n_tiles = clamp_tiles(a.width_start[a.n_objects], a.max_tiles);  // of this width
  float* Bl = reinterpret_cast<float*>(smem + L.B_off);
  if (tid < 3 * kFeatures) Bl[tid] = a.B[tid];
  int staged = -1;
  uint16_t* const enc = reinterpret_cast<uint16_t*>(smem + L.enc_off);
  uint16_t* const buf0 = reinterpret_cast<uint16_t*>(smem + L.buf_off);
  uint16_t* const buf1 = buf0 + 64 * kS128;
  unsigned char* const dzt = smem + L.dz_off;
  // wave 0's losses: lane l's of sub-tiles c, c + 4, ... at [c][l]
  float* const lane_loss = reinterpret_cast<float*>(smem + L.lane_loss_off);

  for (int t = first_tile_of_block(blockIdx.x, gridDim.x, n_tiles); t < n_tiles; t += gridDim.x) {
    const int j = gen_object(a.width_start, a.n_objects, t);
    const int ti = t - a.width_start[j], tile = a.tile_start[j] + ti;  // of the object; of the work list
    if (tile < 0 || tile >= a.max_tiles) continue;  // (not for a consistent work list)
    const int k = __builtin_amdgcn_readfirstlane(a.object_ids[j]);
    if (k < 0 || k >= a.max_objects || !a.desc[k].registered) {
      if (tid == 0) atomicOr(&a.scaler->device_error, 1);
      continue;
    }
    if (kernel_width(a.desc[k].hidden) != H) continue;
    const int rpt = tile_rays(H, a.rays_per_tile, a.rays_per_tile_wide);
    const RayRange rr = tile_ray_range(a.ray_offsets[j], a.ray_offsets[j + 1], ti, rpt, a.n_rays);
    const int ray_lo = rr.lo, ray_hi = rr.hi;
    if (tid < kWave) {
#pragma unroll
      for (int c = 0; c < 4; ++c) lane_loss[c * kWave + tid] = 0.f;
    }
    if (k != staged) {
      __syncthreads();
      fetch_image_lds(a.wimage + (size_t)k * a.wimage_stride, smem, W.B_off, lane_, wave, 8);
      staged = k;
    }
    const double cx = a.desc[k].centre[0], cy = a.desc[k].centre[1], cz = a.desc[k].centre[2];
    const double inv_s = a.desc[k].inv_scale;
    float wseed = 1.0f, inv = 1.0f;
    if (a.dloss) wseed = a.dloss[j];
    if (a.use_scale) {
      const float scale = a.scaler->scale;
      wseed *= scale;
      inv = 1.0f / scale;
    }
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
    f32x16 accW[kLayers - 1][2], accW0;  // dW_1..3: blocks (ob, ib), (ob, ib + 1); dW_0: (ob, 0), even waves
    float accDb[kLayers];                // lane sums of db_l's rows ob, even waves
    f32x4 accWh = {0.f, 0.f, 0.f, 0.f};  // this wave's 16 columns of the output layer's dW
    float accDbH[kOut];
    accW0 = zero;
#pragma unroll
    for (int l = 0; l < kLayers - 1; ++l) accW[l][0] = accW[l][1] = zero;
#pragma unroll
    for (int l = 0; l < kLayers; ++l) accDb[l] = 0.f;
#pragma unroll
    for (int c = 0; c < kOut; ++c) accDbH[c] = 0.f;
    __builtin_amdgcn_s_waitcnt(0);  // this thread's part of the image is in LDS
    __syncthreads();

    const int nsub = (ray_hi - ray_lo + rpw - 1) / rpw;
    for (int sub = 0; sub < nsub; ++sub) {
      // (lane-dependent LDS addresses are computed where they are used, not hoisted and spilled)
      int ln = lane_;
      asm volatile("" : "+v"(ln)::"memory");
      const int lane = ln, n = ln & 31, hf = ln >> 5;
      const int r0 = ray_lo + sub * rpw;
      const int nslots = max(0, min(rpw, ray_hi - r0)) * S;
      const SubTileIn in = subtile_inputs<true>(a, ray_lo, ray_hi, sub, rpw);
      // encoding: every lane its own slot's point, every wave two of the sixteen frequencies
      {
        float x[4] = {0.f, 0.f, 0.f, 0.f};
        if (lane < nslots) {
          const double tt = (double)in.r.tt;
          x[0] = (float)(((double)in.o[0] + tt * (double)in.d[0] - cx) * inv_s);
          x[1] = (float)(((double)in.o[1] + tt * (double)in.d[1] - cy) * inv_s);
          x[2] = (float)(((double)in.o[2] + tt * (double)in.d[2] - cz) * inv_s);
          if (a.var) x[3] = (float)((double)in.var * inv_s * inv_s);
        }
        float sv[2], cv[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int f = 2 * wave + u;
          const float b0 = Bl[f], b1 = Bl[kFeatures + f], b2 = Bl[2 * kFeatures + f];
          const float phi = x[0] * b0 + x[1] * b1 + x[2] * b2;
          vmap_sincosf(phi, &sv[u], &cv[u]);
          if (a.var) {  // expectation under N(x, v I): attenuation exp(-v |b_f|^2 / 2)
            const float nb = b0 * b0 + b1 * b1 + b2 * b2;
            const float att = expf(-0.5f * x[3] * nb);
            sv[u] *= att;
            cv[u] *= att;
          }
        }
        *reinterpret_cast<unsigned int*>(enc + lane * kE128 + colpos(2 * wave)) = pack2(sv[0], sv[1]);
        *reinterpret_cast<unsigned int*>(enc + lane * kE128 + colpos(kFeatures + 2 * wave)) = pack2(cv[0], cv[1]);
      }
      __syncthreads();

      // forward: this wave's block of each layer, kept for the ReLU masks and the restaging
      const int row = 32 * pass + n;                       // this lane's sample
      const int col = fb * 32 + 16 * hf;                   // its sixteen columns in a staged row
      bf16x8 act[kLayers + 1][2];                          // [1..4]
#pragma unroll
      for (int l = 0; l < kLayers; ++l) {
        const int ws = W.w_stride[l], KB = (l == 0) ? 1 : 4;
        const uint16_t* src = (l == 0) ? enc + row * kE128 + 16 * hf : ((l & 1) ? buf0 : buf1) + row * kS128 + 16 * hf;
        const uint16_t* wrow = reinterpret_cast<const uint16_t*>(smem + W.w_off[l]) + (fb * 32 + n) * ws + 16 * hf;
        f32x16 acc = zero;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(wrow + kb * 32 + 8 * jj),
                                                         *reinterpret_cast<const bf16x8*>(src + kb * 32 + 8 * jj), acc, 0, 0, 0);
        const float* bias = reinterpret_cast<const float*>(smem + W.b_off) + l * H + fb * 32 + 4 * hf;
        typedef unsigned int u4 __attribute__((ext_vector_type(4)));
        typedef short s2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          u4 w;
#pragma unroll
          for (int q = 0; q < 2; ++q) {  // rows 16 jj + 8 q + 4 hf + i
            const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + 16 * jj + 8 * q);
            float y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = fmaxf(acc[8 * jj + 4 * q + i] + b4[i], 0.0f);
#pragma unroll
            for (int i = 0; i < 2; ++i)  // (a -0 becomes +0: the masks test the bits)
              w[2 * q + i] = __builtin_bit_cast(unsigned int, __builtin_elementwise_max(
                                 __builtin_bit_cast(s2, pack2(y[2 * i], y[2 * i + 1])), (s2){0, 0}));
          }
          act[l + 1][jj] = __builtin_bit_cast(bf16x8, w);
        }
        uint16_t* dst = ((l & 1) ? buf1 : buf0) + row * kS128 + col;
        *reinterpret_cast<bf16x8*>(dst) = act[l + 1][0];
        *reinterpret_cast<bf16x8*>(dst + 8) = act[l + 1][1];
        __syncthreads();
      }
      // output layer, rendering and its adjoint: wave 0, both passes (h_4 in buf1)
      if (wave == 0) {
        const uint16_t* wh = reinterpret_cast<const uint16_t*>(smem + W.whb_off) + n * (H + 8) + 16 * hf;
        const uint16_t* h4 = buf1 + n * kS128 + 16 * hf;
        f32x16 acc[2] = {zero, zero};
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            bf16x8 wa = {};
            if (n < kOut) wa = *reinterpret_cast<const bf16x8*>(wh + mt * 32 + 8 * jj);
#pragma unroll
            for (int p = 0; p < 2; ++p)
              acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  wa, *reinterpret_cast<const bf16x8*>(h4 + p * 32 * kS128 + mt * 32 + 8 * jj), acc[p], 0, 0, 0);
          }
        const float* bh = reinterpret_cast<const float*>(smem + W.bh_off);
        float zs[kOut], dzs[kOut];
#pragma unroll
        for (int c = 0; c < kOut; ++c) {
          float unused;
          half_join(acc[0][c] + bh[c], acc[1][c] + bh[c], zs[c], unused);
        }
        float loss = 0.f;
        render_subtile<true>(a, r0, nslots, wseed, in.r, zs, dzs, loss);
        lane_loss[(sub & 3) * kWave + lane] += loss;
        bf16x4 d4;
#pragma unroll
        for (int c = 0; c < kOut; ++c) {
          accDbH[c] += dzs[c];
          d4[c] = (__bf16)dzs[c];
          reinterpret_cast<__bf16*>(dzt)[c * kDzPitch + lane] = d4[c];
        }
        *reinterpret_cast<bf16x4*>(dzt + kOut * kDzPitch * 2 + 8 * lane) = d4;
      }
      __syncthreads();
      // output layer's dW: this wave's 16 columns, K = a pass's 32 samples
      const int m16 = lane & 15, kg = lane >> 4;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        bf16x8 da = {};
        if (m16 < kOut)
          da = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const __bf16*>(dzt) + m16 * kDzPitch + 32 * p + 8 * kg);
        const bf16x8 hb = tr_read_pair(reinterpret_cast<const __bf16*>(buf1) + (32 * p + 8 * kg + (m16 >> 2)) * kS128 +
                                           16 * wave + 4 * (m16 & 3), 4 * kS128);
        accWh = __builtin_amdgcn_mfma_f32_16x16x32_bf16(da, hb, accWh, 0, 0, 0);
      }
      // delta of the last hidden layer: this wave's block of W_out^T dz, masked by ReLU'
      bf16x8 dl[2];
      {
        bf16x8 dzb = {}, wa = {};
        if (hf == 0) {
          const bf16x4 d4 = *reinterpret_cast<const bf16x4*>(dzt + kOut * kDzPitch * 2 + 8 * row);
          const bf16x4 w4 = *reinterpret_cast<const bf16x4*>(smem + W.whtb_off + (fb * 32 + n) * kOut * 2);
#pragma unroll
          for (int c = 0; c < kOut; ++c) {
            dzb[c] = d4[c];
            wa[c] = w4[c];
          }
        }
        const f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, dzb, zero, 0, 0, 0);
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) dl[jj] = relu_mask(round8(acc, 8 * jj), act[kLayers][jj]);
      }
      // W_l^T operands: in-feature n of block fb, the outputs of K slot (hf, e) of block ko
      const int wc = 4 * (m16 & 3) + 16 * (kg & 1);
      const int wt0 = (4 * hf + (m16 >> 2)) * kS128 + fb * 32 + colpos(wc);
#pragma unroll
      for (int l = kLayers - 1; l >= 0; --l) {
        // stage delta_l in buf1 and the layer's inputs in buf0 (h_3 lies there already; the first
        // layer's are the encodings)
        __syncthreads();  // buf1 and buf0 have been read
        uint16_t* dst = buf1 + row * kS128 + col;
        *reinterpret_cast<bf16x8*>(dst) = dl[0];
        *reinterpret_cast<bf16x8*>(dst + 8) = dl[1];
        if (l > 0 && l < kLayers - 1) {
          dst = buf0 + row * kS128 + col;
          *reinterpret_cast<bf16x8*>(dst) = act[l][0];
          *reinterpret_cast<bf16x8*>(dst + 8) = act[l][1];
        }
        __syncthreads();
        f32x16 nacc = zero;
        if (l > 0) {
          const uint16_t* src = buf1 + row * kS128 + 16 * hf;
          const __bf16* Wt = reinterpret_cast<const __bf16*>(smem + W.w_off[l]) + wt0;
#pragma unroll
          for (int ko = 0; ko < 4; ++ko)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
              nacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_read_pair(Wt + (ko * 32 + 16 * jj) * kS128, 8 * kS128),
                                                            *reinterpret_cast<const bf16x8*>(src + ko * 32 + 8 * jj), nacc, 0, 0, 0);
        }
        // weight gradient: blocks (ob, ib) and (ob, ib + 1) over the 64 samples
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if (l == 0 && (wave & 1)) break;
          const bf16x8 da = tr_operand<kS128>(buf1, 16 * s, ob * 32, lane);
          if (l > 0) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
              accW[l - 1][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  da, tr_operand<kS128>(buf0, 16 * s, (ib + b) * 32, lane), accW[l - 1][b], 0, 0, 0);
          } else {
            accW0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(da, tr_operand<kE128>(enc, 16 * s, 0, lane), accW0, 0, 0, 0);
          }
          if (!(wave & 1)) accDb[l] = operand_sum(da, accDb[l]);
        }
        if (l == 0) break;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) dl[jj] = relu_mask(round8(nacc, 8 * jj), act[l][jj]);
      }
      __syncthreads();  // the next sub-tile writes the encodings
    }  // sub-tiles

    // ---------------- tile result: each wave writes its own gradient blocks
    int le = lane_;
    asm volatile("" : "+v"(le));
    const int lane = le, n = le & 31, hf = le >> 5;
    int bad = 0;
    float* dst = a.partial + (size_t)tile * a.p_stride;
    auto put = [&](int idx, float g) {
      g *= inv;
      bad |= partial_bad(g);
      dst[idx] = g;
    };
    int* any_bad = reinterpret_cast<int*>(smem + L.loss_off);
    if (tid == 0) *any_bad = 0;
    __syncthreads();
    // register r of a lane of half hf holds the gradient of output ob 32 + colfeat(rowof(r, hf)),
    // input block column colfeat(n)
#pragma unroll
    for (int l = 0; l < kLayers; ++l) {
      const int K = (l == 0) ? kEnc : H;
      const int off = layer_param_off(H, l);
      if (l > 0 || !(wave & 1)) {
#pragma unroll
        for (int b = 0; b < (l == 0 ? 1 : 2); ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            put(off + (ob * 32 + colfeat(rowof(r, hf))) * K + (l == 0 ? 0 : (ib + b) * 32) + colfeat(n),
                l == 0 ? accW0[r] : accW[l == 0 ? 0 : l - 1][b][r]);
      }
      if (!(wave & 1)) {
        const float db = half_sum(accDb[l]);
        if (hf == 0) put(off + H * K + ob * 32 + colfeat(n), db);
      }
    }
    const int offh = layer_param_off(H, kLayers);
    if (lane < 16) {
#pragma unroll
      for (int c = 0; c < kOut; ++c) put(offh + c * H + ob * 32 + colfeat(16 * (wave & 1) + lane), accWh[c]);
    }
    if (wave == 0) {
      // the loss in the order of k_step_coop, whose waves take every fourth sub-tile each, so that
      // forward and step report the same sum
      float loss = 0.f;
#pragma unroll
      for (int c = 0; c < 4; ++c) loss += wave_sum(lane_loss[c * kWave + lane]);
      if (lane == 0) a.tile_loss[tile] = loss;
#pragma unroll
      for (int c = 0; c < kOut; ++c) {
        const float g = wave_sum(accDbH[c]);
        if (lane == c) put(offh + kOut * H + c, g);
      }
    }
    if (bad) *any_bad = 1;  // every writer stores the same value
    __syncthreads();
    if (tid == 0 && *any_bad) atomicOr(&a.flags[k], 1);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Tile kernel for hidden 64 in FP32, and for rendering with hidden 128 in BF16: a sub-tile per wave,
// four waves. Training: each wave runs the forward, rendering, adjoint and delta chain of its own
// sub-tile as k_step_tiles does, stages delta_l and h_{l-1} in LDS, and after a workgroup barrier
// computes its quarter of the rows of dW_l (and db_l) over the 128 samples of all four waves, on
// v_mfma_f32_16x16x4f32. A wave thus holds a quarter of the weight-gradient accumulators, and the
// tile needs no cross-wave reduction: the waves' slices are disjoint. The weights of hidden 128 are
// read from the object's weight image in device memory (the byte layout of the LDS staging, staged
// when the parameters are set and kept current by the optimiser kernels).

template <int H, bool BF, int MODE>
__global__ void __launch_bounds__(256, 1) k_step_coop(const StepArgs a_in) {
  static_assert((H == 64 && !BF) || (H == 128 && BF && MODE == MODE_FWD), "widths and modes of this kernel");
  StepArgs a = a_in;
  read_batch(a);
  constexpr int MT = H / 32;
  constexpr bool TRAIN = (MODE == MODE_TRAIN);
  constexpr bool GW = weights_global(H);
  constexpr LdsLayout L = lds_layout(H, BF, 1);
  constexpr CoopLayout C = coop_layout(H, BF);
  constexpr int RW = H / 4;         // weight-gradient rows of one wave
  constexpr int RB = RW / 16;       // ... in 16-row blocks
  constexpr int NBH = H / 16;       // 16-column blocks of a hidden layer's input
  constexpr int FW = H / 4;         // output layer: features of one wave
  constexpr int TB = kDzTileBytes, TT = tr_tile_bytes(H);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 31, hf = lane >> 5;
  const int m16 = lane & 15, kg = lane >> 4;
  const int S = a.S;
  const int rpw = kSlots / S;
  const int n_tiles = clamp_tiles(a.width_start[a.n_objects], a.max_tiles);  // of this width
  float* Bl = reinterpret_cast<float*>(smem + C.B_off);
  if (tid < 3 * kFeatures) Bl[tid] = a.B[tid];
  unsigned char* const scr0 = smem + C.scratch_off;
  int staged = -1;

  for (int t = first_tile_of_block(blockIdx.x, gridDim.x, n_tiles); t < n_tiles; t += gridDim.x) {
    const int j = gen_object(a.width_start, a.n_objects, t);
    const int ti = t - a.width_start[j], tile = a.tile_start[j] + ti;  // of the object; of the work list
    if (tile < 0 || tile >= a.max_tiles) continue;  // (not for a consistent work list)
    // uniform by construction: the weight-image and partial buffer resources live in SGPRs
    const int k = __builtin_amdgcn_readfirstlane(a.object_ids[j]);
    if (k < 0 || k >= a.max_objects || !a.desc[k].registered) {
      if (tid == 0) atomicOr(&a.scaler->device_error, 1);
      continue;
    }
    if (kernel_width(a.desc[k].hidden) != H) continue;
    const int rpt = tile_rays(H, a.rays_per_tile, a.rays_per_tile_wide);
    const RayRange rr = tile_ray_range(a.ray_offsets[j], a.ray_offsets[j + 1], ti, rpt, a.n_rays);
    const int ray_lo = rr.lo, ray_hi = rr.hi;
    const unsigned char* wb = smem;
    if constexpr (GW) {
      wb = a.wimage + (size_t)k * a.wimage_stride;
    } else if (k != staged) {
      __syncthreads();
      stage_weights<H, BF>(a.theta + (size_t)k * a.p_stride, smem, tid, blockDim.x);
      staged = k;
    }
    __syncthreads();
    const double cx = a.desc[k].centre[0], cy = a.desc[k].centre[1], cz = a.desc[k].centre[2];
    const double inv_s = a.desc[k].inv_scale;
    float wseed = 1.0f;
    if constexpr (TRAIN) {
      if (a.dloss) wseed = a.dloss[j];
      if (a.use_scale) wseed *= a.scaler->scale;
    }
    const float inv = (TRAIN && a.use_scale) ? 1.0f / a.scaler->scale : 1.0f;
    float* dst = a.partial + (size_t)tile * a.p_stride;

    f32x4 accW[kLayers][RB][NBH];  // this wave's rows of dW_l (16x16 blocks)
    float accDb[kLayers][RB];      // lane sums of this wave's rows of db_l
    float accH[kOut];              // output layer's dW, one feature per lane group
    float accDbH[kOut];
    if constexpr (TRAIN) {
#pragma unroll
      for (int l = 0; l < kLayers; ++l)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < NBH; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) accW[l][rb][cb][i] = 0.f;
#pragma unroll
      for (int l = 0; l < kLayers; ++l)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) accDb[l][rb] = 0.f;
#pragma unroll
      for (int c = 0; c < kOut; ++c) { accH[c] = 0.f; accDbH[c] = 0.f; }
    }
    float wave_loss = 0.f;
    int bad = 0;

    unsigned char* dzt = scr0 + wave * C.scratch_wave;
    unsigned char* dtile = dzt + TB;
    unsigned char* htile = dtile + TT;
    const int nrays = ray_hi - ray_lo;
    const int nsub = (nrays + rpw - 1) / rpw;
    const int rounds = (nsub + 3) / 4;

    // Every wave runs every round (a wave without a sub-tile carries zero seeds), since the
    // weight-gradient products of a round read all four waves' staging tiles.
    for (int rd = 0; rd < rounds; ++rd) {
      asm volatile("" ::: "memory");
      const int sub = rd * 4 + wave;
      const int r0 = ray_lo + sub * rpw;
      const int nr = (sub < nsub) ? min(rpw, ray_hi - r0) : 0;
      const int nslots = nr * S;
      const RenderIn rin = render_inputs<TRAIN>(a, r0, nslots);  // in flight during the forward

      // the lane's sample: normalised point and (integrated encoding) normalised variance
      auto point = [&](int p, float xt[4]) {
        const int slot = 32 * p + n;
        xt[0] = xt[1] = xt[2] = xt[3] = 0.f;
        if (slot < nslots) {
          const int ray = r0 + slot / S;
          const double tt = (double)a.t[(size_t)r0 * S + slot];
          const float* o3 = a.rays_o + 3 * (size_t)ray;
          const float* d3 = a.rays_d + 3 * (size_t)ray;
          xt[0] = (float)(((double)o3[0] + tt * (double)d3[0] - cx) * inv_s);
          xt[1] = (float)(((double)o3[1] + tt * (double)d3[1] - cy) * inv_s);
          xt[2] = (float)(((double)o3[2] + tt * (double)d3[2] - cz) * inv_s);
          if (a.var) xt[3] = (float)((double)a.var[(size_t)r0 * S + slot] * inv_s * inv_s);
        }
      };
      float zs[kOut] = {0.f, 0.f, 0.f, 0.f};
      if (nslots > 0) {
#pragma unroll 1
        for (int p = 0; p < 2; ++p) {
          Acts<H, BF> tmp;
          float xt[4], z[kOut];
          point(p, xt);
          forward_pass<H, BF, true>(xt, wb, Bl, tmp, z, a.var != nullptr);
#pragma unroll
          for (int c = 0; c < kOut; ++c) zs[c] = (hf == p) ? z[c] : zs[c];
        }
      }
      float dzs[kOut];
      render_subtile<TRAIN>(a, r0, nslots, wseed, rin, zs, dzs, wave_loss);
      if constexpr (TRAIN) {
#pragma unroll
        for (int c = 0; c < kOut; ++c) accDbH[c] += dzs[c];

#pragma unroll 1
        for (int p = 0; p < 2; ++p) {
          Acts<H, BF> act;
          {
            float xt[4], z[kOut];
            point(p, xt);
            forward_pass<H, BF, false>(xt, wb, Bl, act, z, a.var != nullptr);
          }
          float dz[kOut];
#pragma unroll
          for (int c = 0; c < kOut; ++c) dz[c] = __shfl(dzs[c], 32 * p + n);
          __syncthreads();  // every wave is done reading the staging tiles
          if (hf == 0) {
#pragma unroll
            for (int c = 0; c < kOut; ++c) reinterpret_cast<float*>(dzt)[n * kOut + c] = dz[c];
          }
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              reinterpret_cast<float*>(htile)[n * (H + 4) + mt * 32 + rowof(r, hf)] = act.v[kLayers][mt][r];
          __syncthreads();
          // output layer: this wave's columns of dW over the four waves' samples
#pragma unroll
          for (int w2 = 0; w2 < 4; ++w2) {
            const unsigned char* dz2 = scr0 + w2 * C.scratch_wave;
            const unsigned char* h2 = dz2 + TB + TT;
            constexpr int G = 64 / FW, SG = 32 / G;
            const int f = wave * FW + (lane % FW), g = lane / FW;
#pragma unroll
            for (int s2 = 0; s2 < SG; ++s2) {
              const int s = g * SG + s2;
              const float hv = reinterpret_cast<const float*>(h2)[s * (H + 4) + f];
#pragma unroll
              for (int c = 0; c < kOut; ++c) accH[c] += reinterpret_cast<const float*>(dz2)[s * kOut + c] * hv;
            }
          }
          // delta of the last hidden layer, own samples: (W_out^T dz) masked by ReLU'
          Deltas<H, BF> dl;
          const float* Wh = reinterpret_cast<const float*>(wb + L.wh_off);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              float s = 0.f;
#pragma unroll
              for (int c = 0; c < kOut; ++c) s += Wh[c * (H + 4) + mt * 32 + 16 * hf + r] * dz[c];
              const float hv = reinterpret_cast<const float*>(htile)[n * (H + 4) + mt * 32 + rowof(r, hf)];
              dl.set(mt, r, (hv > 0.f) ? s : 0.f);
            }
#pragma unroll
          for (int l = kLayers - 1; l >= 0; --l) {
            const int K = (l == 0) ? kEnc : H;
            const int KB = K / 32, NB = K / 16;
            const int off = layer_param_off(H, l);
            __syncthreads();  // every wave is done reading the staging tiles
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
              for (int r = 0; r < 16; ++r)
                reinterpret_cast<float*>(dtile)[n * (H + 4) + mt * 32 + rowof(r, hf)] = dl.v[mt][r];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
              for (int r = 0; r < 16; ++r)
                reinterpret_cast<float*>(htile)[n * (H + 4) + kb * 32 + rowof(r, hf)] = act.v[l][kb][r];
            __syncthreads();  // every wave's tiles are staged
            // this wave's rows of dW_l: D lane holds row 16 rb + 4 kg + i, column 16 cb + m16
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) {
              const unsigned char* d2 = scr0 + w2 * C.scratch_wave + TB;
              const unsigned char* h2 = d2 + TT;
#pragma unroll
              for (int kk = 0; kk < 8; ++kk) {
                const int s = 4 * kk + kg;
                float da[RB];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                  da[rb] = reinterpret_cast<const float*>(d2)[s * (H + 4) + wave * RW + rb * 16 + m16];
                  accDb[l][rb] += da[rb];
                }
#pragma unroll
                for (int cb = 0; cb < NBH; ++cb) {
                  if (cb >= NB) continue;
                  const float hb = reinterpret_cast<const float*>(h2)[s * (H + 4) + cb * 16 + m16];
#pragma unroll
                  for (int rb = 0; rb < RB; ++rb)
                    accW[l][rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(da[rb], hb, accW[l][rb][cb], 0, 0, 0);
                }
              }
            }
            if (l == 0) break;
            // delta_{l-1} = (W_l^T delta_l) masked by ReLU' of layer l-1, own samples
            const int ws = L.w_stride[l];
            Deltas<H, BF> nd;
#pragma unroll
            for (int mi = 0; mi < MT; ++mi) {
              f32x16 acc2;
#pragma unroll
              for (int r = 0; r < 16; ++r) acc2[r] = 0.f;
              const int col = mi * 32 + colpos(n);
#pragma unroll
              for (int ko = 0; ko < MT; ++ko) {
                const float* W = reinterpret_cast<const float*>(wb + L.w_off[l]);
#pragma unroll
                for (int qq = 0; qq < 16; ++qq)
                  acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(W[(ko * 32 + rowof(qq, hf)) * ws + col],
                                                              dl.v[ko][qq], acc2, 0, 0, 0);
              }
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                const float hv = reinterpret_cast<const float*>(htile)[n * (H + 4) + mi * 32 + rowof(r, hf)];
                nd.set(mi, r, (hv > 0.f) ? acc2[r] : 0.f);
              }
            }
            dl = nd;
          }
        }
      }
    }  // rounds

    // ---------------- tile result: loss and output-layer bias combined in wave order, every
    // wave writes its own gradient slices
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) wave_loss += __shfl_xor(wave_loss, off);
    if constexpr (TRAIN) {
#pragma unroll
      for (int c = 0; c < kOut; ++c) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) accDbH[c] += __shfl_xor(accDbH[c], off);
#pragma unroll
        for (int off = FW; off < 64; off <<= 1) accH[c] += __shfl_xor(accH[c], off);
      }
#pragma unroll
      for (int l = 0; l < kLayers; ++l)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          accDb[l][rb] += __shfl_xor(accDb[l][rb], 16);
          accDb[l][rb] += __shfl_xor(accDb[l][rb], 32);
        }
    }
    float* lsum = reinterpret_cast<float*>(smem + C.loss_off);
    int* any_bad = reinterpret_cast<int*>(smem + C.loss_off + 20);
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
      if (wave == w && lane == 0) {
        lsum[0] = (w == 0 ? 0.f : lsum[0]) + wave_loss;
        if constexpr (TRAIN) {
#pragma unroll
          for (int c = 0; c < kOut; ++c) lsum[1 + c] = (w == 0 ? 0.f : lsum[1 + c]) + accDbH[c];
          if (w == 0) *any_bad = 0;
        }
      }
      __syncthreads();
    }
    if constexpr (TRAIN) {
      auto put = [&](int idx, float g) {
        g *= inv;
        bad |= partial_bad(g);
        dst[idx] = g;
      };
#pragma unroll
      for (int l = 0; l < kLayers; ++l) {
        const int K = (l == 0) ? kEnc : H;
        const int NB = K / 16;
        const int off = layer_param_off(H, l);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < NBH; ++cb) {
            if (cb >= NB) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              put(off + (wave * RW + rb * 16 + 4 * kg + i) * K + cb * 16 + m16, accW[l][rb][cb][i]);
          }
        if (kg == 0) {
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) put(off + H * K + wave * RW + rb * 16 + m16, accDb[l][rb]);
        }
      }
      const int offh = layer_param_off(H, kLayers);
      if (lane < FW) {
#pragma unroll
        for (int c = 0; c < kOut; ++c) put(offh + c * H + wave * FW + lane, accH[c]);
      }
      if (wave == 0 && lane < kOut) put(offh + kOut * H + lane, lsum[1 + lane]);
      if (bad) *any_bad = 1;  // every writer stores the same value
      __syncthreads();
      if (tid == 0 && *any_bad) atomicOr(&a.flags[k], 1);
    }
    if (tid == 0) a.tile_loss[tile] = lsum[0];
    __syncthreads();
  }
}

// Weight image of object `single` (width 32, or hidden 128 in BF16) from its parameters, when they
// are set (added, or written through vmap_set_state); the optimiser kernels keep it current after
// that. With single < 0, block (x, j) stages a share of batch object j's image.
template <int H, bool BF>
__global__ void __launch_bounds__(256) k_stage_image(const StepArgs a_in, int single) {
  StepArgs a = a_in;
  read_batch(a);
  int k = single;
  if (single < 0) {
    if ((int)blockIdx.y >= a.n_objects) return;
    k = a.object_ids[blockIdx.y];
  }
  if (k < 0 || k >= a.max_objects || !a.desc[k].registered || kernel_width(a.desc[k].hidden) != H) return;
  unsigned char* dst = (H == 32) ? a.img32 + (size_t)k * img32_bytes(BF)
                                 : a.wimage + (size_t)k * a.wimage_stride;
  stage_weights<H, BF>(a.theta + (size_t)k * a.p_stride, dst, blockIdx.x * blockDim.x + threadIdx.x,
                       gridDim.x * blockDim.x, a.desc[k].hidden);
}

// ---------------------------------------------------------------------------------------------
// Shape query of one object: forward only, 64 points per wave iteration.

template <int H, bool BF>
__global__ void __launch_bounds__(256) k_query(const QueryArgs qa) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr bool GW = weights_global(H);
  constexpr int B_off = GW ? coop_layout(H, BF).B_off : lds_layout(H, BF, 1).B_off;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int n = lane & 31, hf = lane >> 5;
  float* Bl = reinterpret_cast<float*>(smem + B_off);
  if (tid < 3 * kFeatures) Bl[tid] = qa.B[tid];
  const unsigned char* wb = smem;
  if constexpr (GW) {
    wb = qa.wimage + (size_t)qa.k * qa.wimage_stride;
  } else if constexpr (H == 32) {  // the object's weight image is current
    fetch_image_lds(qa.img32 + (size_t)qa.k * img32_bytes(BF), smem, B_off, lane, wave, nw);
    __builtin_amdgcn_s_waitcnt(0);
  } else stage_weights<H, BF>(qa.theta + (size_t)qa.k * qa.p_stride, smem, tid, blockDim.x, qa.desc[qa.k].hidden);
  __syncthreads();
  const ObjDesc d = qa.desc[qa.k];
  if constexpr (H == 32) {
    // a lane's own point; both passes together, as in the tile kernel (one pass after the other,
    // points, normalisation and logistic computed by both halves: 61 us for 2.1 M points, 48 now)
    const int64_t step = (int64_t)gridDim.x * nw * kSlots;
    int64_t i = ((int64_t)blockIdx.x * nw + wave) * kSlots + lane;
    float q[3] = {0.f, 0.f, 0.f};
    auto fetch = [&](int64_t at) {
#pragma unroll
      for (int c = 0; c < 3; ++c) q[c] = at < qa.n ? qa.pts[3 * at + c] : 0.f;
    };
    fetch(i);
    for (; i - lane < qa.n; i += step) {
      float xt[2][4];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float x = i < qa.n ? (float)(((double)q[c] - d.centre[c]) * d.inv_scale) : 0.f;
        half_split(x, xt[0][c], xt[1][c]);
      }
      xt[0][3] = xt[1][3] = 0.f;
      fetch(i + step);
      Acts<32, BF> act[2];
      float zs[kOut];
      forward_pair<BF>(xt, smem, Bl, lane, act, zs, false);
      if (i < qa.n) {
        qa.occ[i] = sigm(zs[3]);
        if (qa.rgb) {
#pragma unroll
          for (int c = 0; c < 3; ++c) qa.rgb[3 * i + c] = sigm(zs[c]);
        }
      }
    }
    return;
  }
  for (int64_t chunk = (int64_t)blockIdx.x * nw + wave; chunk * kSlots < qa.n; chunk += (int64_t)gridDim.x * nw) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int64_t i = chunk * kSlots + 32 * p + n;
      float xt[4] = {0.f, 0.f, 0.f, 0.f};
      if (i < qa.n) {
#pragma unroll
        for (int c = 0; c < 3; ++c) xt[c] = (float)(((double)qa.pts[3 * i + c] - d.centre[c]) * d.inv_scale);
      }
      Acts<H, BF> act;
      float z[kOut];
      forward_pass<H, BF, true>(xt, wb, Bl, act, z);
      if (i < qa.n && hf == 0) {
        qa.occ[i] = sigm(z[3]);
        if (qa.rgb) {
#pragma unroll
          for (int c = 0; c < 3; ++c) qa.rgb[3 * i + c] = sigm(z[c]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Tile offsets per batch object (exclusive scan of ceil(rays / rays_per_tile)), and the same over
// the objects of each fused kernel width alone (width_start: scans of n_objects + 1), so that
// a width's launch finds its own tiles: workgroup t of it takes the t-th, and none starts only to
// pass over another width's tile. A fourth scan counts each object's units of k_reduce_adam_wide; in a
// stack that may hold a layered width (GEN), three more its row tiles, product blocks and work tiles
// (a launch of their own took 6 us of a 310 us step).
// Clears the non-finite flags of the batch's objects and records
// each object's next Adam step count, so that the optimiser kernels read it from here while one of
// their blocks advances the count. Checks the ray offsets as step_table does: a batch that fails
// gets no tiles, and the optimiser kernels leave every object unchanged (ScalerState::batch_ok).
// One workgroup, an object per thread, scans by DPP within waves: bound by three dependent loads
// (offsets and ids, descriptor, stores).

template <bool GEN>
__global__ void __launch_bounds__(1024) k_worklist(int n_objects, int n_rays, const int32_t* ids,
                                                   const int32_t* offs, int rpt, int rpt_wide, int rpt_gen,
                                                   int max_objects, const ObjDesc* __restrict__ desc,
                                                   ScalerState* __restrict__ scaler,
                                                   int32_t* __restrict__ tile_start,
                                                   int32_t* __restrict__ width_start, int width_pitch,
                                                   int32_t* __restrict__ flags,
                                                   int32_t* __restrict__ t_next,
                                                   const BatchDev* __restrict__ bd, const GenScan gen) {
  constexpr int N = GEN ? 8 : 5;  // scans
  __shared__ int wtot[16][N];
  if (bd) {
    n_objects = bd->n_objects;
    n_rays = bd->n_rays;
    if (bd->rays_per_tile > 0) rpt = bd->rays_per_tile;
    ids = bd->object_ids;
    offs = bd->ray_offsets;
  }
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  int bad = 0;
  for (int j = tid; j < n_objects; j += nt) bad |= !batch_segment_ok(j, n_objects, offs[j], offs[j + 1], n_rays);
  const bool any_bad = __syncthreads_or(bad) != 0;
  // all tiles, those of widths 32, 64 and 128, optimiser units; of layered objects row tiles, product
  // blocks (block_rows rows, or pairs of row tiles) and work tiles
  int carry[N] = {};
  for (int base = 0; base < n_objects; base += nt) {
    const int j = base + tid;
    int cnt[N] = {};
    if (j < n_objects) {
      const int o0 = offs[j], o1 = offs[j + 1], k = ids[j];
      const bool in_range = k >= 0 && k < max_objects;
      const ObjDesc& d = desc[in_range ? k : 0];  // (an id out of range: discarded)
      const int registered = d.registered, hidden = d.hidden, step = d.step, n_params = d.n_params;
      const bool valid = in_range && registered;
      // rays per tile by the object's width (invalid ids take the narrow size)
      const int per = !valid ? rpt : (generic_width(hidden) ? rpt_gen : tile_rays(hidden, rpt, rpt_wide));
      cnt[0] = any_bad ? 0 : tiles_of(o1 - o0, per);
      // an invalid object's tiles go to every width's launch, which report it and pass on
#pragma unroll
      for (int w = 0; w < 3; ++w) cnt[1 + w] = (!valid || kernel_width(hidden) == (32 << w)) ? cnt[0] : 0;
      cnt[4] = valid ? opt_units(n_params, cnt[0]) : 1;
      if constexpr (GEN) {
        if (valid && !any_bad && generic_width(hidden) && o1 > o0) {
          cnt[5] = tiles_of(o1 - o0, gen.rpw);
          const long long rows = (long long)(o1 - o0) * gen.S;
          cnt[6] = gen.chain && gen_chain(hidden) ? (cnt[5] + 1) / 2
                   : gen.block_rows == kGenBlockRows ? (int)((rows + kGenBlockRows - 1) / kGenBlockRows)
                                                     : (int)((rows + kGenHalfRows - 1) / kGenHalfRows);
          cnt[7] = cnt[0];
        }
      }
      if (in_range) flags[k] = 0;
      // step count after this batch's update, read by the optimiser kernels
      t_next[j] = valid ? step + 1 : 0;
    }
    int x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      x[i] = wave_scan(cnt[i]);
      if (lane == kWave - 1) wtot[wave][i] = x[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int before = carry[i];
      for (int w = 0; w < nw; ++w) {
        const int v = wtot[w][i];
        if (w < wave) before += v;
        carry[i] += v;
      }
      int32_t* dst = i == 0 ? tile_start : i < 5 ? width_start + (i - 1) * width_pitch : gen.start[i < 5 ? 0 : i - 5];
      if (j < n_objects) dst[j] = before + x[i] - cnt[i];
    }
    __syncthreads();
  }
  if (tid == 0) {
    tile_start[n_objects] = carry[0];
#pragma unroll
    for (int w = 0; w < 4; ++w) width_start[w * width_pitch + n_objects] = carry[1 + w];
    if constexpr (GEN) {
#pragma unroll
      for (int i = 0; i < 3; ++i) gen.start[i][n_objects] = carry[5 + i];
    }
    scaler->batch_ok = !any_bad;
    if (any_bad) atomicOr(&scaler->device_error, DERR_OFFSETS);
  }
}

// SPREAD: with the extra rows of objects of many tiles (spread_object).
template <bool SPREAD>
__global__ void __launch_bounds__(256) k_reduce(const OptArgs a_in, int want_grad) {
  OptArgs a = a_in;
  read_batch(a);
  int j = blockIdx.y, part = 0;
  if (SPREAD && j >= a.n_objects) {
    part = 1 + (j - a.n_objects) % 3;
    j = spread_object(a, (j - a.n_objects) / 3);
    if (j < 0) return;
  }
  const int k = a.ids[j];
  const bool valid = obj_valid(a, k) && a.scaler->batch_ok;
  const TileRange tr = clamp_tile_range(a.tile_start[j], a.tile_start[j + 1], a.max_tiles);
  const int t0 = tr.t0, t1 = tr.t1;
  if (a.loss_out && part == 0 && blockIdx.x == gridDim.x - 1 && threadIdx.x < kWave) {  // (the fewest parameters)
    const float loss = loss_sum(a.tile_loss, t0, t1);
    if (threadIdx.x == 0) a.loss_out[j] = valid ? loss : 0.f;
  }
  if (!want_grad || !valid) return;
  const int P = a.desc[k].n_params, hidden = a.desc[k].hidden;
  const bool spread = SPREAD && t1 - t0 > kSpreadTiles;
  bool bad = false;
  const int p = blockIdx.x * blockDim.x + (spread ? part * kWave + ((int)threadIdx.x & 63) : (int)threadIdx.x);
  float sum = 0.f;
  if (spread) {
    sum = spread_sum(a.partial, a.p_stride, t0, t1, p < P ? padded_index(hidden, p) : 0);
    if (threadIdx.x >= kWave) return;
  }
  if (p < a.p_stride) {
    const float g = p >= P ? 0.f : spread ? sum : tile_sum(a.partial, a.p_stride, t0, t1, padded_index(hidden, p));
    bad = !isfinite(g);
    a.grad[(size_t)k * a.p_stride + p] = g;
    if (a.grad_out) a.grad_out[(size_t)j * a.p_stride + p] = g;
  }
  if (bad) atomicOr(&a.flags[k], 1);
}

__global__ void __launch_bounds__(256) k_adam(const OptArgs a_in) {
  OptArgs a = a_in;
  read_batch(a);
  const int j = blockIdx.y;
  if (blockIdx.x == 0 && j == 0) scaler_update(a);
  const int k = a.ids[j];
  if (!a.scaler->batch_ok || !obj_valid(a, k) || a.offs[j + 1] <= a.offs[j] || a.flags[k]) return;
  const int t = a.t_next[j];
  const AdamCoef c = adam_coef(a, t);
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < a.desc[k].n_params) {
    const size_t i = (size_t)k * a.p_stride + p;
    float th = a.theta[i], m = a.m[i], v = a.v[i];
    adam_elem(c, a.grad[i], th, m, v);
    a.theta[i] = th;
    a.m[i] = m;
    a.v[i] = v;
    update_image(a, k, a.desc[k].hidden, p, th);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) a.desc[k].step = t;
}

// Training step: gradient and update in one pass. The tiles report a partial holding an element
// that is not finite or reaches 2^64 in magnitude (partial_bad), so an object none of whose tiles
// reported has a finite summed gradient and its skip is decided, for the whole object, before any
// store; the element test below is a guard that this bound makes unreachable. Every load of a thread depends on at most the batch object's id, ray
// range and tile range, so a workgroup waits for device memory twice (those, then the object's
// data); the validity checks only decide what is stored. Thread 0 works out the Adam
// coefficients while the loads are in flight. The grid has one row of workgroups per batch object,
// one whose first workgroup updates the loss scaler (its own chain of loads), and the extra rows of
// objects of many tiles (spread_object).
template <bool SPREAD>
__global__ void __launch_bounds__(256) k_reduce_adam(const OptArgs a_in) {
  OptArgs a = a_in;
  read_batch(a);
  int j = blockIdx.y, part = 0;
  if (j == a.n_objects) {
    if (blockIdx.x == 0) scaler_update(a);
    return;
  }
  if (SPREAD && j > a.n_objects) {  // an extra row (spread_object)
    part = 1 + (j - a.n_objects - 1) % 3;
    j = spread_object(a, (j - a.n_objects - 1) / 3);
    if (j < 0) return;
  }
  const int k = a.ids[j];
  const TileRange tr = clamp_tile_range(a.tile_start[j], a.tile_start[j + 1], a.max_tiles);
  const int t0 = tr.t0, t1 = tr.t1;
  const int r0 = a.offs[j], r1 = a.offs[j + 1];
  const int t = a.t_next[j];
  const int batch_ok = a.scaler->batch_ok;
  const bool in_range = k >= 0 && k < a.max_objects;
  const int kc = in_range ? k : 0;  // loads of an id out of range are discarded
  const ObjDesc& d = a.desc[kc];
  const int registered = d.registered, n_params = d.n_params, hidden = d.hidden;
  const bool spread = SPREAD && t1 - t0 > kSpreadTiles;
  const int p = blockIdx.x * blockDim.x + (spread ? part * kWave + ((int)threadIdx.x & 63) : (int)threadIdx.x);
  const size_t i = (size_t)kc * a.p_stride + p;
  float th = 0.f, m = 0.f, v = 0.f, g = 0.f;
  // slot of p in the partials, which hold the kernel width's layout (hidden 16: padded to 32)
  const int slot = (hidden == 16 && p < n_params) ? padded_index(16, p) : min(p, a.p_stride - 1);
  const bool mine = p < a.p_stride && (!spread || threadIdx.x < kWave);
  if (mine) {
    th = a.theta[i];
    m = a.m[i];
    v = a.v[i];
    if (!spread) g = tile_sum(a.partial, a.p_stride, t0, t1, slot);
  }
  const bool lead = blockIdx.x == 0 && part == 0 && threadIdx.x == 0;
  // the loss: a wave of the workgroup with the fewest parameters
  const bool lossy = a.loss_out && part == 0 && blockIdx.x == gridDim.x - 1 && threadIdx.x < kWave;
  float loss = 0.f;
  if (lossy) loss = loss_sum(a.tile_loss, t0, t1);
  if (spread) g = spread_sum(a.partial, a.p_stride, t0, t1, slot);
  __shared__ float sh[2];
  if (threadIdx.x == 0) adam_coef_store(a, t, sh);
  const bool valid = in_range && registered != 0 && batch_ok;
  if (lossy && threadIdx.x == 0) a.loss_out[j] = valid ? loss : 0.f;
  if (!valid || r1 <= r0) return;
  // the barrier of object_bad also publishes the coefficients
  if (object_bad(a, j, k)) {
    if (a.tile_bad && lead) a.flags[k] = 1;
    return;
  }
  const AdamCoef c = adam_coef_load(a, sh);
  if (mine && p < n_params) {
    a.grad[i] = g;
    if (isfinite(g)) {
      adam_elem(c, g, th, m, v);
      a.theta[i] = th;
      a.m[i] = m;
      a.v[i] = v;
    } else {
      atomicOr(&a.flags[k], 2);  // for the skip count (bit 1: see object_bad)
    }
    update_image<false>(a, k, hidden, p, th);
  }
  if (lead) a.desc[k].step = t;
}

// k_reduce_adam for stacks with objects of many parameters. The batch's parameters are cut into
// units of one object each (opt_units, their scan left by k_worklist). Without `rows` every
// workgroup takes a run of consecutive units, so that an object's descriptor, tile range, skip test
// and Adam coefficients are settled once per workgroup and object, whatever the objects' widths;
// with it a row of that many workgroups per object walks the object's units in turn. Per
// parameter the same arithmetic in the same order: the tiles' partials summed in tile_sum's order
// from zero, then one Adam update. A unit is 1024 parameters, four to a thread; of an object of more
// than kSplitTiles tiles it is 256, each wave summing a quarter of the tiles for all of them (four
// parameters per lane) and each thread updating one.
//
// Memory bound where objects are large (hidden 1024: 34 B per parameter), by dependent loads where
// they are small or have many tiles. A row of workgroups per object, as wide as the largest object
// needs, took 28 us for a hidden-128 object of 100 tiles beside fifty of hidden 32: some 4,000
// workgroups of which all but a few hundred found nothing to do, three to a CU; 15 us in runs.
// Stacks of a layered width (all large objects) keep rows: neighbouring workgroups stream
// neighbouring memory, 1 % of the hidden-1024 step. The partials are read and the gradients
// written without caching (nothing reads them again soon): 1 % of the hidden-256 step.
__global__ void __launch_bounds__(256, 4) k_reduce_adam_wide(const OptArgs a_in, int rows) {
  OptArgs a = a_in;
  read_batch(a);
  a.tile_bad = nullptr;  // (launches of stacks of width 32 alone have them, which take k_reduce_adam)
  const int blocks = (int)gridDim.x - 1;
  if ((int)blockIdx.x == blocks) {
    scaler_update(a);
    return;
  }
  __shared__ float sh[2];
  __shared__ __attribute__((aligned(16))) float part[4][256];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int u0, u1, du = 1;
  if (rows > 0) {
    const int j = blockIdx.x / rows;
    u0 = a.opt_start[j] + (int)blockIdx.x % rows;
    u1 = a.opt_start[j + 1];
    du = rows;
  } else {
    const int total = a.opt_start[a.n_objects];
    u0 = (int)((long long)total * blockIdx.x / blocks);
    u1 = (int)((long long)total * (blockIdx.x + 1) / blocks);
  }
  int first = 0, end = 0, k = 0, t0 = 0, t1 = 0, n_params = 0, hidden = 0;
  bool live = false;
  AdamCoef c{};
  for (int u = u0; u < u1; u += du) {
    if (u >= end) {  // the next object
      const int j = gen_object(a.opt_start, a.n_objects, u);
      first = a.opt_start[j];
      end = a.opt_start[j + 1];
      k = a.ids[j];
      const TileRange tr = clamp_tile_range(a.tile_start[j], a.tile_start[j + 1], a.max_tiles);
      t0 = tr.t0;
      t1 = tr.t1;
      const int r0 = a.offs[j], r1 = a.offs[j + 1], t = a.t_next[j];
      const bool in_range = k >= 0 && k < a.max_objects;
      const ObjDesc& d = a.desc[in_range ? k : 0];
      n_params = d.n_params;
      hidden = d.hidden;
      const bool valid = in_range && d.registered != 0 && a.scaler->batch_ok;
      const bool lead = u == first && tid == 0;
      __syncthreads();  // the previous object's coefficients have been read
      if (tid == 0) adam_coef_store(a, t, sh);
      if (u == first && wave == 1 && a.loss_out) {  // (wave 0 has the coefficients to work out)
        const float loss = loss_sum(a.tile_loss, t0, t1);
        if (lane == 0) a.loss_out[j] = valid ? loss : 0.f;
      }
      live = valid && r1 > r0;
      // (the barrier of object_bad also publishes the coefficients)
      if (live && object_bad(a, j, k)) {
        if (a.tile_bad && lead) a.flags[k] = 1;
        live = false;
      }
      if (live) {
        c = adam_coef_load(a, sh);
        if (lead) a.desc[k].step = t;
      }
    }
    if (!live) {
      u = end - du;  // (a row's workgroups stay with their object)
      continue;
    }
    const size_t base = (size_t)k * a.p_stride;
    if (t1 - t0 > kSplitTiles) {
      const int p0 = (u - first) * 256, p = p0 + tid;
      const bool mine = p < n_params;
      float th = 0.f, m = 0.f, v = 0.f;
      if (mine) {
        th = a.theta[base + p];
        m = a.m[base + p];
        v = a.v[base + p];
      }
      f32x4 g = {0.f, 0.f, 0.f, 0.f};
      if (p0 + 4 * lane < n_params) {  // (four slots from a multiple of 4: within p_stride)
        const TileRange tq = tile_quarter(t0, t1, wave);
        const float* src = a.partial + padded_index(hidden, p0 + 4 * lane);
        for (int tt = tq.t0; tt < tq.t1; tt += 8) {
          f32x4 x[8];
#pragma unroll
          for (int i = 0; i < 8; ++i)
            x[i] = (tt + i < tq.t1) ? *reinterpret_cast<const f32x4*>(src + (size_t)(tt + i) * a.p_stride) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (tt + i < tq.t1) g += x[i];
        }
      }
      __syncthreads();  // the previous unit's sums have been read
      *reinterpret_cast<f32x4*>(&part[wave][4 * lane]) = g;
      __syncthreads();
      if (!mine) continue;
      const float s = ((part[0][tid] + part[1][tid]) + part[2][tid]) + part[3][tid];
      a.grad[base + p] = s;
      if (isfinite(s)) {
        adam_elem(c, s, th, m, v);
        a.theta[base + p] = th;
        a.m[base + p] = m;
        a.v[base + p] = v;
      } else {
        atomicOr(&a.flags[k], 2);
      }
      update_image(a, k, hidden, p, th);
      continue;
    }
    // p_stride is a multiple of 4, so p + 3 < p_stride for every p taken
    const int p = (u - first) * 1024 + 4 * tid;
    if (p >= n_params) continue;
    const size_t i = base + p;
    const f32x4 x = *reinterpret_cast<const f32x4*>(a.theta + i);
    const f32x4 y = *reinterpret_cast<const f32x4*>(a.m + i);
    const f32x4 z = *reinterpret_cast<const f32x4*>(a.v + i);
    float th[4] = {x[0], x[1], x[2], x[3]}, m[4] = {y[0], y[1], y[2], y[3]}, v[4] = {z[0], z[1], z[2], z[3]};
    f32x4 g = {0.f, 0.f, 0.f, 0.f};
    // slot of p in the partials (hidden 16: the width-32 layout, where four parameters p..p+3
    // with p a multiple of 4 stay four consecutive slots)
    const float* src = a.partial + padded_index(hidden, p);
    for (int tt = t0; tt < t1; tt += 4) {
      f32x4 q[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        q[e] = (tt + e < t1) ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + (size_t)(tt + e) * a.p_stride)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (tt + e < t1) g += q[e];
    }
    if (p + 3 < n_params && isfinite(g[0]) && isfinite(g[1]) && isfinite(g[2]) && isfinite(g[3])) {
#pragma unroll
      for (int e = 0; e < 4; ++e) adam_elem(c, g[e], th[e], m[e], v[e]);
      __builtin_nontemporal_store(g, reinterpret_cast<f32x4*>(a.grad + i));
      *reinterpret_cast<f32x4*>(a.theta + i) = f32x4{th[0], th[1], th[2], th[3]};
      *reinterpret_cast<f32x4*>(a.m + i) = f32x4{m[0], m[1], m[2], m[3]};
      *reinterpret_cast<f32x4*>(a.v + i) = f32x4{v[0], v[1], v[2], v[3]};
      if (a.gimg && keeps_gimg(hidden)) {  // the four BF16 copies in one store (i is a multiple of 4)
        typedef unsigned int u2w __attribute__((ext_vector_type(2)));
        *reinterpret_cast<u2w*>(a.gimg + i) = u2w{pack2(th[0], th[1]), pack2(th[2], th[3])};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) update_image(a, k, hidden, p + e, th[e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (p + e >= n_params) continue;
        a.grad[i + e] = g[e];
        if (isfinite(g[e])) {
          adam_elem(c, g[e], th[e], m[e], v[e]);
          a.theta[i + e] = th[e];
          a.m[i + e] = m[e];
          a.v[i + e] = v[e];
        } else {
          atomicOr(&a.flags[k], 2);
        }
        update_image(a, k, hidden, p + e, th[e]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Object initialisation: Xavier-uniform weights from SplitMix64 in counter mode, zero biases,
// zero Adam moments and gradient; also writes the object's descriptor.

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t index) {
  uint64_t z = seed + (index + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

struct InitBounds {
  double bound[kLayers + 1];
  int w_end[kLayers + 1];
  int b_end[kLayers + 1];
};

__global__ void __launch_bounds__(256) k_init(int k, uint64_t seed, InitBounds ib, ObjDesc d,
                                              ObjDesc* __restrict__ desc, float* __restrict__ theta,
                                              float* __restrict__ mom, float* __restrict__ vel,
                                              float* __restrict__ grad, int p_stride, int P, int use_rng) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p == 0) desc[k] = d;
  if (p >= p_stride) return;
  const size_t i = (size_t)k * p_stride + p;
  if (use_rng) {
    float w = 0.f;
    if (p < P) {
      for (int l = 0; l <= kLayers; ++l) {
        if (p < ib.w_end[l]) {  // weight of layer l
          const uint64_t z = splitmix64_at(seed, (uint64_t)p);
          const double u = (double)(z >> 40) * 0x1p-24;
          w = (float)(ib.bound[l] * (2.0 * u - 1.0));
          break;
        }
        if (p < ib.b_end[l]) break;  // bias of layer l: zero
      }
    }
    theta[i] = w;
  } else if (p >= P) {
    theta[i] = 0.f;
  }
  mom[i] = 0.f;
  vel[i] = 0.f;
  grad[i] = 0.f;
}

// ---------------------------------------------------------------------------------------------
// Depth-guided sampling (Sec. 3.3, Eqs. 1 and 2): sample i of a ray is stratified in [t_n, t_s] for
// i < n_strat, N(t_s, sigma^2) otherwise, in FP64 from counter-based SplitMix64 uniforms, and the
// ray's S values are sorted.
//
// A workgroup holds the rays whose samples fit its threads, a thread per sample: first the normal
// samples (logarithm, cosine and square root: several times a stratified one's work), filled up to
// whole waves, then the stratified ones. A sample's place is the number of the ray's keys below its
// own, the value's bits in order and then its index, read from LDS as broadcasts. VALU issue bounds
// it. A group of P lanes (S rounded up to a power of two) per ray, each lane a sample and then a
// place of a bitonic network, spent the normal samples' time on every wave and most of its time in
// the network: 16,881 rays of 20 samples (half of them normal) took 10.5 us, 6.1 now; 500,000 of 10,
// 82 and 40.
constexpr int kSampleThreads = 512;

// Rays per workgroup: their samples with the normal ones rounded up to whole waves fit the threads.
__host__ __device__ constexpr int sample_block_rays(int S) { return (kSampleThreads - (kWave - 1)) / S; }

// One value per lane of the group of P lanes, sorted by a bitonic network (minima and maxima drop
// NaNs): the order of rays that hold one.
__device__ __noinline__ float sample_network(float v, int P) {
  const int i = threadIdx.x & (P - 1);
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      const float other = __shfl_xor(v, j);
      const bool ascending = (i & k) == 0;
      const bool lower = (i & j) == 0;
      v = (lower == ascending) ? fminf(v, other) : fmaxf(v, other);
    }
  }
  return v;
}

__global__ void __launch_bounds__(kSampleThreads) k_sample(int n_rays, int S, int P, int n_strat,
                                                           const float* __restrict__ t_near,
                                                           const float* __restrict__ t_far,
                                                           const float* __restrict__ depth, float sigma,
                                                           uint64_t seed, float* __restrict__ t_out) {
  typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) unsigned long long keys[2 * kSampleThreads];  // [ray][S, even]
  const int R = sample_block_rays(S), r0 = (int)blockIdx.x * R, nr = min(R, n_rays - r0);
  const int ng = S - n_strat, pitch = (S + 1) & ~1;  // (0 <= n_strat <= S)
  const int tid = threadIdx.x, pad = (R * ng + kWave - 1) & ~(kWave - 1);
  const bool normal = tid < pad;
  const int u = normal ? tid : tid - pad, per = normal ? ng : n_strat;  // sample u of its kind, per of them a ray
  const int q = per > 0 ? u / per : R, i = (normal ? n_strat : 0) + u - q * per, r = r0 + q;
  const bool mine = q < nr;
  float v = 0.f;
  if (mine) {
    const double tf = t_far[r], d = depth[r];
    const double ts = (d > 0.0) ? d : tf;
    const uint64_t idx = ((uint64_t)r * (uint64_t)S + (uint64_t)i) * 2ull;
    const double top0 = (double)(splitmix64_at(seed, idx) >> 40);
    if (normal) {
      const double top1 = (double)(splitmix64_at(seed, idx + 1ull) >> 40);
      const double z = sqrt(-2.0 * log((top0 + 1.0) * 0x1p-24)) * cos(6.283185307179586477 * top1 * 0x1p-24);
      v = (float)(ts + (double)sigma * z);
    } else {
      const double tn = t_near[r];
      v = (float)(tn + ((double)i + top0 * 0x1p-24) / (double)n_strat * (ts - tn));
    }
  }
  const unsigned int b = __builtin_bit_cast(unsigned int, v);
  const unsigned long long key = ((unsigned long long)(b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u)) << 32) | (unsigned int)i;
  if (mine) {
    keys[q * pitch + i] = key;
    if (i == S - 1 && pitch > S) keys[q * pitch + S] = ~0ull;
  }
  if (__syncthreads_or(v != v)) {  // (the same branch for the whole workgroup)
    for (int qb = 0; qb < nr; qb += kSampleThreads / P) {
      const int qq = qb + tid / P, ii = tid & (P - 1);
      const bool has = qq < nr && ii < S;
      const unsigned int x = has ? (unsigned int)(keys[qq * pitch + ii] >> 32) : 0u;
      const float y = __builtin_bit_cast(float, x ^ ((x >> 31) ? 0x80000000u : 0xffffffffu));
      const float z = sample_network(has ? y : INFINITY, P);
      if (has) t_out[(size_t)(r0 + qq) * S + ii] = z;
    }
    return;
  }
  if (!mine) return;
  const u64x2* kp = reinterpret_cast<const u64x2*>(keys + q * pitch);
  int rank = 0;
#pragma unroll 4
  for (int j = 0; j < pitch / 2; ++j) {
    const u64x2 x = kp[j];
    rank += (x[0] < key) ? 1 : 0;
    rank += (x[1] < key) ? 1 : 0;
  }
  t_out[(size_t)r * S + rank] = v;
}

hipError_t launch_sample(int n_rays, int S, int n_strat, const float* t_near, const float* t_far,
                         const float* depth, float sigma, uint64_t seed, float* t_out,
                         hipStream_t s) {
  if (n_rays <= 0) return hipSuccess;
  int P = 1;
  while (P < S) P <<= 1;
  const int R = sample_block_rays(S);
  hipLaunchKernelGGL(k_sample, dim3((n_rays - 1) / R + 1), dim3(kSampleThreads), 0, s, n_rays, S, P, n_strat,
                     t_near, t_far, depth, sigma, seed, t_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Scene rendering from object models (Sec. 3.4): ray-box intersection per (ray, object), the
// object renders of the rays that meet each bound, and a per-ray ranking by rendered depth.
// The pairs are laid out as a batch (object-major, rays in image order), which the forward-mode
// tile kernels render through a device batch descriptor; the host never reads the pair count.

// Entry of ray (o, d) into the box c +- s after t_min, and exit; the ray meets the box iff
// t1 > t0. Slab method in FP64 without contraction (the oracle's arithmetic).
__device__ __forceinline__ void scene_slab(const float* o, const float* d, const ObjDesc& od,
                                           double t_min, double& t0, double& t1) {
  const double s = 1.0 / od.inv_scale;
  t0 = -INFINITY;
  t1 = INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double lo = __dsub_rn(od.centre[a], s), hi = __dadd_rn(od.centre[a], s);
    const double oa = (double)o[a], da = (double)d[a];
    double near, far;
    if (da == 0.0) {
      const bool inside = oa >= lo && oa <= hi;
      near = inside ? -INFINITY : INFINITY;
      far = inside ? INFINITY : -INFINITY;
    } else {
      const double ta = __ddiv_rn(__dsub_rn(lo, oa), da), tb = __ddiv_rn(__dsub_rn(hi, oa), da);
      near = fmin(ta, tb);
      far = fmax(ta, tb);
    }
    t0 = fmax(t0, near);
    t1 = fmin(t1, far);
  }
  t0 = fmax(t0, t_min);
}

__device__ __forceinline__ bool scene_pair_valid(const SceneArgs& a, int j, int& k) {
  k = a.object_ids[j];
  return k >= 0 && k < a.max_objects && a.desc[k].registered;
}

// Whether the ray (o, d; inv = 1 / d) certainly misses the box c +- s after t_min, in FP32: the
// interval widened by more than the rounding of its ends (each is a difference of values up to
// |c| + s + |o| times inv, a few roundings of 2^-24 of that; widened by 2^-19), and in the sum and the
// product by 1e-37, where values so small that FP32 holds them to fewer digits, or not at all, round
// by more. Zero direction components and NaN or infinite values are never certain.
// widen[0], widen[1]: the ray's share of the widening, that of a box a centre and half extent of which
// add up to x is x widen[0] + widen[1].
__device__ __forceinline__ bool scene_certain_miss(const float o[3], const float inv[3], const float (*widen)[2],
                                                   const float4& box, float t_min) {
  const float cc[3] = {box.x, box.y, box.z}, s = box.w;
  float t0 = -INFINITY, t1 = INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float c = cc[a];
    const float ta = (c - s - o[a]) * inv[a], tb = (c + s - o[a]) * inv[a];
    const float e = fmaf(fabsf(c) + s, widen[a][0], widen[a][1]);
    t0 = fmaxf(t0, fminf(ta, tb) - e);
    t1 = fminf(t1, fmaxf(ta, tb) + e);
  }
  return t1 < t0 || t1 <= t_min;
}

// Block (x, y): rays [256 x, 256 x + 256) against batch objects [y per, (y + 1) per), per at most
// kSceneGroup: a bit per (object, ray) that meets (words of 32 rays) and the block's hit count per
// object. A ray is loaded once for all of them, and the FP64 slab test (seven divisions) runs only
// where the FP32 interval does not settle it: 76,800 rays, 50 objects 23.2 us with a workgroup per
// object and FP64 for every pair, 12.8 now.
constexpr int kSceneGroup = 64;
__global__ void __launch_bounds__(256) k_scene_count(const SceneArgs a, int nblk, int per) {
  __shared__ int cnt[kSceneGroup];
  __shared__ float4 box[kSceneGroup];  // centre and half extent in FP32 (negative: no object)
  const int tid = threadIdx.x, lane = tid & 63, r = blockIdx.x * 256 + tid;
  const int j0 = blockIdx.y * per, j1 = min(j0 + per, a.n_objects);
  if (j0 + tid < j1) {
    int k;
    const bool valid = scene_pair_valid(a, j0 + tid, k);
    const ObjDesc& od = a.desc[valid ? k : 0];
    box[tid] = make_float4((float)od.centre[0], (float)od.centre[1], (float)od.centre[2],
                           valid ? (float)(1.0 / od.inv_scale) : -1.0f);
    cnt[tid] = 0;
  }
  float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 0.f}, inv[3], widen[3][2];
  const bool ray = r < a.n_rays;
  if (ray) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      o[c] = a.rays_o[3 * (size_t)r + c];
      d[c] = a.rays_d[3 * (size_t)r + c];
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    inv[c] = 1.0f / d[c];
    widen[c][0] = fabsf(inv[c]) * 0x1p-19f;
    widen[c][1] = fmaf(fabsf(o[c]) + 1e-37f, widen[c][0], 1e-37f);
  }
  const int words = (a.n_rays + 31) >> 5;
  __syncthreads();
  for (int j = j0; j < j1; ++j) {
    bool hit = false;
    const float4 b = box[j - j0];
    if (b.w >= 0.f && ray && !scene_certain_miss(o, inv, widen, b, (float)a.t_min)) {
      double t0, t1;
      scene_slab(o, d, a.desc[a.object_ids[j]], a.t_min, t0, t1);
      hit = t1 > t0;
    }
    const unsigned long long m = __ballot(hit);
    if ((lane & 31) == 0 && (r >> 5) < words) a.pair_mask[(size_t)j * words + (r >> 5)] = (uint32_t)(m >> lane);
    if (lane == 0 && m) atomicAdd(&cnt[j - j0], __popcll(m));
  }
  __syncthreads();
  for (int j = j0 + tid; j < j1; j += 256) a.counts[(size_t)j * nblk + blockIdx.x] = cnt[j - j0];
}

// One block: exclusive scan of the counts (object-major), the batch's CSR offsets (clamped to
// the pair capacity) and its device descriptor. Sixteen consecutive counts per thread, loaded
// together, and a DPP scan over the waves (a thread's serial loop over its share and a scan of
// twenty barriers took 17.6 us for 15,000 counts, 9.5 now).
__global__ void __launch_bounds__(1024) k_scene_scan(const SceneArgs a, int nblk) {
  __shared__ int wtot[16];
  const int n = a.n_objects * nblk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int carry = 0;
  for (int base = 0; base < n; base += 16384) {
    const int i0 = base + 16 * tid;
    int c[16], local = 0;
#pragma unroll
    for (int u = 0; u < 16; u += 4) {  // (the counts' region is 256-byte aligned, its end padded)
      int4 v = make_int4(0, 0, 0, 0);
      if (i0 + u < n) v = *reinterpret_cast<const int4*>(a.counts + i0 + u);
      c[u] = v.x;
      c[u + 1] = v.y;
      c[u + 2] = v.z;
      c[u + 3] = v.w;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) local += (i0 + u < n) ? c[u] : 0;
    const int x = wave_scan(local);
    if (lane == kWave - 1) wtot[wave] = x;
    __syncthreads();
    int run = carry + x - local;
    for (int w = 0; w < 16; ++w) {
      const int v = wtot[w];
      if (w < wave) run += v;
      carry += v;
    }
    int j = i0 / nblk, q = i0 - j * nblk;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (i0 + u < n) {
        a.counts[i0 + u] = run;
        if (q == 0) a.ray_offsets[j] = min(run, a.max_pairs);
        run += c[u];
        if (++q == nblk) {
          q = 0;
          ++j;
        }
      }
    }
    __syncthreads();
  }
  // the tile: forward_tile, a candidate per lane (of equal costs the most rounds)
  const int pairs = min(carry, a.max_pairs), k = lane + 1;
  long long cost = kNoTile;
  if (k <= kSceneRounds && k >= a.tile_low / a.tile_round)
    cost = forward_tile_cost(a.bf16, k, a.tile_round, a.tile_waves, pairs, a.n_objects);
  long long least = cost;
#pragma unroll
  for (int off = 4; off >= 1; off >>= 1) least = min(least, __shfl_xor(least, off));
  const unsigned long long best = __ballot(k <= kSceneRounds && cost == least && cost < kNoTile);
  const int tile = best ? (64 - __clzll((long long)best)) * a.tile_round : a.tile_low;
  if (tid == 0) {
    const int total = carry;
    a.ray_offsets[a.n_objects] = min(total, a.max_pairs);
    if (a.n_pairs_out) *a.n_pairs_out = total;
    if (total > a.max_pairs) atomicOr(&a.scaler->device_error, 2);
    // one store of the whole descriptor: every field is written (the scratch holding it is not
    // cleared, and a field left out would be read as garbage); no targets or losses, point samples
    *a.bd = make_batch_dev(a.n_objects, a.S, min(total, a.max_pairs), a.object_ids, a.ray_offsets,
                           a.pair_o, a.pair_d, a.pair_t, nullptr, nullptr, nullptr, nullptr, nullptr,
                           tile);
  }
}

// Block (x, y): the pairs of its rays with its batch objects, in ray order: ray, and samples at the
// midpoints of S equal parts of [t0, t1] (FP64, rounded once). A wave's pairs with an object are
// consecutive, so its lanes write their samples as one run (a lane writing its own pair's S samples
// one by one: 41.9 us for 76,800 rays, 50 objects, 117,000 pairs; 23 now).
__global__ void __launch_bounds__(256) k_scene_fill(const SceneArgs a, int nblk, int per) {
  __shared__ double frac[kSlots];
  __shared__ double span[4][kWave][2];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = blockIdx.x * 256 + tid;
  const int j0 = blockIdx.y * per, j1 = min(j0 + per, a.n_objects);
  const int S = a.S, words = (a.n_rays + 31) >> 5;
  if (tid < S) frac[tid] = __ddiv_rn((double)tid + 0.5, (double)S);
  __syncthreads();
  const int w0 = (r - lane) >> 5;  // the wave's first word
  if (w0 >= words) return;
  float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 0.f};
  if (r < a.n_rays) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      o[c] = a.rays_o[3 * (size_t)r + c];
      d[c] = a.rays_d[3 * (size_t)r + c];
    }
  }
  for (int j = j0; j < j1; ++j) {
    const uint32_t m0 = a.pair_mask[(size_t)j * words + w0];
    const uint32_t m1 = w0 + 1 < words ? a.pair_mask[(size_t)j * words + w0 + 1] : 0u;
    const unsigned long long m = (unsigned long long)m0 | ((unsigned long long)m1 << 32);
    if (!m) continue;  // uniform over the wave
    // first pair of the wave: the block's first (counts, scanned) and the words before in the block
    int p0 = a.counts[(size_t)j * nblk + blockIdx.x];
    for (int i = w0 & ~7; i < w0; ++i) p0 += __popc(a.pair_mask[(size_t)j * words + i]);
    if (lane == 0 && words > 1) {  // for the composite (one word: the block's first)
      a.pair_base[(size_t)j * words + w0] = p0;
      if (w0 + 1 < words) a.pair_base[(size_t)j * words + w0 + 1] = p0 + __popc(m0);
    }
    const int pairs = min(__popcll(m), a.max_pairs - p0);  // (may be negative)
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    wave_lds_sync();  // the previous object's intervals have been read
    if (((m >> lane) & 1ull) && rank < pairs) {
      const int k = a.object_ids[j];  // (a set bit: a registered object)
      double t0, t1;
      scene_slab(o, d, a.desc[k], a.t_min, t0, t1);
      span[w][rank][0] = t0;
      span[w][rank][1] = __dsub_rn(t1, t0);
      const size_t p = (size_t)p0 + rank;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        a.pair_o[3 * p + c] = o[c];
        a.pair_d[3 * p + c] = d[c];
      }
    }
    wave_lds_sync();
    int q = lane / S, i = lane - q * S;
    const int dq = kWave / S, di = kWave - dq * S;
    for (int e = lane; e < pairs * S; e += kWave) {
      a.pair_t[(size_t)p0 * S + e] = (float)__dadd_rn(span[w][q][0], __dmul_rn(frac[i], span[w][q][1]));
      q += dq;
      i += di;
      if (i >= S) {
        i -= S;
        ++q;
      }
    }
  }
}

// Per ray: the nearest object (rendered depth) whose rendered occupancy reaches the threshold;
// an equal depth keeps the earlier batch object. The hits are a bit per (object, ray): a dense
// (object, ray) map of pair indices was 15 MB to write and read for 76,800 rays and 50 objects
// (22.7 us here; 13 now).
__global__ void __launch_bounds__(64) k_scene_composite(const SceneArgs a) {
  const int r = blockIdx.x * 64 + threadIdx.x;
  if (r >= a.n_rays) return;
  const int words = (a.n_rays + 31) >> 5, w = r >> 5;
  float best = INFINITY, occ = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
  int id = -1;
  for (int jb = 0; jb < a.n_objects; jb += 8) {
    uint32_t m[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) m[u] = jb + u < a.n_objects ? a.pair_mask[(size_t)(jb + u) * words + w] : 0u;
    unsigned int hits = 0;  // bit u: this ray meets object jb + u
#pragma unroll
    for (int u = 0; u < 8; ++u) hits |= ((m[u] >> (r & 31)) & 1u) << u;
    while (hits) {  // in batch order
      const int u = __ffs(hits) - 1, j = jb + u;
      hits &= hits - 1u;
      const uint32_t below = a.pair_mask[(size_t)j * words + w] & ((1u << (r & 31)) - 1u);
      const int p = (words > 1 ? a.pair_base[(size_t)j * words + w] : a.counts[j]) + __popc(below);
      if (p >= a.max_pairs) continue;
      const float O = a.pair_occ[p], D = a.pair_depth[p];
      if (O >= a.occ_threshold && D < best) {
        best = D;
        occ = O;
        c0 = a.pair_rgb[3 * (size_t)p];
        c1 = a.pair_rgb[3 * (size_t)p + 1];
        c2 = a.pair_rgb[3 * (size_t)p + 2];
        id = a.object_ids[j];
      }
    }
  }
  a.depth_out[r] = id >= 0 ? best : 0.f;
  if (a.rgb_out) {
    a.rgb_out[3 * (size_t)r] = c0;
    a.rgb_out[3 * (size_t)r + 1] = c1;
    a.rgb_out[3 * (size_t)r + 2] = c2;
  }
  if (a.occ_out) a.occ_out[r] = occ;
  if (a.id_out) a.id_out[r] = id;
}

hipError_t launch_scene(int phase, const SceneArgs& a, hipStream_t s) {
  if (a.n_rays <= 0 || a.n_objects <= 0) return hipSuccess;
  const int nblk = (a.n_rays + 255) / 256;
  // objects per workgroup: as many as leave about 1024 workgroups (four a CU)
  const long long want = ((long long)nblk * a.n_objects) / 1024;
  const int per = (int)std::max<long long>(1, std::min<long long>({want, (long long)kSceneGroup, (long long)a.n_objects}));
  const dim3 grid(nblk, (a.n_objects + per - 1) / per);
  switch (phase) {
    case 0:
      hipLaunchKernelGGL(k_scene_count, grid, dim3(256), 0, s, a, nblk, per);
      hipLaunchKernelGGL(k_scene_scan, dim3(1), dim3(1024), 0, s, a, nblk);
      hipLaunchKernelGGL(k_scene_fill, grid, dim3(256), 0, s, a, nblk, per);
      break;
    default:
      hipLaunchKernelGGL(k_scene_composite, dim3((a.n_rays + 63) / 64), dim3(64), 0, s, a);
  }
  return hipGetLastError();
}

// Debug validation of a batch (contexts created with VMAP_DEBUG=1), before its step: workgroup 0
// checks that no object id appears twice (an id's mark takes the batch index of each occurrence in
// turn; a mark that was not cleared names a repeat), the others that every ray's sample depths
// ascend. Findings go to the sticky device error bits; the step itself is not changed.
__global__ void __launch_bounds__(256) k_debug_batch(const StepArgs a_in, int32_t* __restrict__ mark) {
  StepArgs a = a_in;
  read_batch(a);
  if (blockIdx.x == 0) {
    for (int j = threadIdx.x; j < a.n_objects; j += blockDim.x) {
      const int k = a.object_ids[j];
      if (k >= 0 && k < a.max_objects) mark[k] = -1;
    }
    __syncthreads();
    int dup = 0;
    for (int j = threadIdx.x; j < a.n_objects; j += blockDim.x) {
      const int k = a.object_ids[j];
      if (k >= 0 && k < a.max_objects) dup |= atomicExch(&mark[k], j) != -1;
    }
    if (__syncthreads_or(dup) && threadIdx.x == 0) atomicOr(&a.scaler->device_error, DERR_DUP_ID);
    return;
  }
  const int S = a.S;
  int bad = 0;
  for (int r = (blockIdx.x - 1) * blockDim.x + threadIdx.x; r < a.n_rays; r += (gridDim.x - 1) * blockDim.x) {
    const float* tr = a.t + (size_t)r * S;
    for (int i = 0; i + 1 < S; ++i) bad |= !(tr[i] <= tr[i + 1]);
  }
  if (__syncthreads_or(bad) && threadIdx.x == 0) atomicOr(&a.scaler->device_error, DERR_T_ORDER);
}

hipError_t launch_debug_batch(const StepArgs& a, int32_t* mark, hipStream_t s) {
  const int blocks = 1 + std::max(1, std::min(1024, (a.n_rays + 255) / 256));
  hipLaunchKernelGGL(k_debug_batch, dim3(blocks), dim3(256), 0, s, a, mark);
  return hipGetLastError();
}

__global__ void k_fill_zero(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

__global__ void k_init_scaler(ScalerState* sc, float scale) {
  if (threadIdx.x == 0) {
    sc->scale = scale;
    sc->good_steps = 0;
    sc->skipped = 0;
    sc->device_error = 0;
  }
}

// ---------------------------------------------------------------------------------------------
// Launchers.

// Raise a kernel's dynamic-LDS limit to what a launch needs (once per size increase). Asking for
// the whole 160 KB fails when the kernel also holds static LDS.
static hipError_t allow_lds(const void* fn, int bytes, int* allowed) {
  if (bytes <= *allowed || bytes <= 64 * 1024) return hipSuccess;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) *allowed = bytes;
  return e;
}

template <int H, bool BF, int MODE>
static hipError_t launch_tiles_t(const StepArgs& a_in, int nwaves, int grid, hipStream_t s) {
  static int allowed = 0;
  StepArgs a = a_in;
  const void* fn;
  int bytes;
  if constexpr (H == 32) {
    fn = reinterpret_cast<const void*>(k_step_tiles<H, BF, MODE>);
    // forward mode stages weights only, so that more workgroups fit on a CU (with the training
    // staging it ran two waves per SIMD instead of the four its registers allow)
    bytes = MODE == MODE_FWD ? lds_layout(H, BF, nwaves).scratch_off : lds_layout(H, BF, nwaves).total;
    if constexpr (MODE == MODE_STEP) {  // the tile table follows the layout
      if (a.n_objects > kTableMaxObjects || !a.tile_bad) return hipErrorInvalidValue;
      const TableLayout T = table_layout(bytes, a.n_objects);
      a.lds_table = bytes;
      a.lds_rays = T.rays;
      bytes = T.total;
    }
  } else if constexpr (H == 128 && BF && MODE == MODE_TRAIN) {
    fn = reinterpret_cast<const void*>(k_step_128);
    bytes = lds128().total;
    nwaves = 8;
  } else if constexpr (H == 64 && BF) {
    fn = reinterpret_cast<const void*>(k_step_64<MODE>);
    bytes = MODE == MODE_FWD ? lds64().scratch_off : lds64().total;
    nwaves = 4;
  } else {
    static_assert(MODE != MODE_STEP, "the in-kernel tile table is built for width 32 only");
    fn = reinterpret_cast<const void*>(k_step_coop<H, BF, MODE>);
    // rendering stages nothing in LDS, so that more workgroups fit on a CU: a 320 x 240 scene of 50
    // hidden-64 FP32 objects 1,556 to 1,327 us, 20 hidden-128 objects of 6,000 rows 83 to 53
    bytes = MODE == MODE_FWD ? coop_layout(H, BF).scratch_off : coop_layout(H, BF).total;
    nwaves = 4;
  }
  hipError_t e = allow_lds(fn, bytes, &allowed);
  if (e != hipSuccess) return e;
  // (with the table, a workgroup more: the first publishes it for the optimiser)
  if constexpr (H == 32)
    hipLaunchKernelGGL((k_step_tiles<H, BF, MODE>), dim3(MODE == MODE_STEP ? grid + 1 : grid), dim3(nwaves * kWave), bytes, s, a);
  else if constexpr (H == 128 && BF && MODE == MODE_TRAIN)
    hipLaunchKernelGGL(k_step_128, dim3(grid), dim3(nwaves * kWave), bytes, s, a);
  else if constexpr (H == 64 && BF)
    hipLaunchKernelGGL((k_step_64<MODE>), dim3(grid), dim3(nwaves * kWave), bytes, s, a);
  else
    hipLaunchKernelGGL((k_step_coop<H, BF, MODE>), dim3(grid), dim3(nwaves * kWave), bytes, s, a);
  return hipGetLastError();
}

int tiles_supported(int H, bool bf16) {
  return H == 16 || H == 32 || H == 64 || (H == 128 && bf16) || (generic_width(H) && bf16);
}

int tile_waves(int H, int requested) { return H == 32 ? requested : 4; }

int tile_lds_bytes(int H, bool bf16, int nwaves) {
  if (generic_width(H)) return kGenLdsBytes;
  if (H == 64 && bf16) return lds64().total;
  if (H == 128) return lds128().total;
  return H == 32 ? lds_layout(H, bf16, nwaves).total : coop_layout(H, bf16).total;
}

hipError_t launch_tiles(int H, bool bf16, int mode, const StepArgs& a, int nwaves, int grid,
                        hipStream_t s) {
  if (grid <= 0) return hipSuccess;
#define VMAP_TILES(HH, BB)                                                                     \
  if (H == HH && bf16 == BB) {                                                                 \
    return mode == MODE_TRAIN ? launch_tiles_t<HH, BB, MODE_TRAIN>(a, nwaves, grid, s)        \
                              : launch_tiles_t<HH, BB, MODE_FWD>(a, nwaves, grid, s);         \
  }
  if (mode == MODE_STEP) {
    if (H != 32) return hipErrorInvalidValue;
    return bf16 ? launch_tiles_t<32, true, MODE_STEP>(a, nwaves, grid, s)
                : launch_tiles_t<32, false, MODE_STEP>(a, nwaves, grid, s);
  }
  VMAP_TILES(32, false)
  VMAP_TILES(32, true)
  VMAP_TILES(64, false)
  VMAP_TILES(64, true)
  VMAP_TILES(128, true)
#undef VMAP_TILES
  return hipErrorInvalidValue;
}

hipError_t launch_stage_images(int H, bool bf16, const StepArgs& a, int single, hipStream_t s) {
  if (!weights_global(H)) return hipSuccess;
  if (H != 128 || !bf16 || !a.wimage) return hipErrorInvalidValue;
  const int ny = single >= 0 ? 1 : a.n_objects;
  if (ny <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_stage_image<128, true>), dim3(16, ny), dim3(256), 0, s, a, single);
  return hipGetLastError();
}

hipError_t launch_stage_image32(bool bf16, const StepArgs& a, int k, hipStream_t s) {
  if (!a.img32 || k < 0) return hipErrorInvalidValue;
  if (bf16) hipLaunchKernelGGL((k_stage_image<32, true>), dim3(8), dim3(256), 0, s, a, k);
  else hipLaunchKernelGGL((k_stage_image<32, false>), dim3(8), dim3(256), 0, s, a, k);
  return hipGetLastError();
}

template <int H, bool BF>
static hipError_t launch_query_t(const QueryArgs& q, hipStream_t s) {
  static int allowed = 0;
  auto fn = k_query<H, BF>;
  const int bytes = weights_global(H) ? coop_layout(H, BF).B_off + 3 * kFeatures * 4
                                      : lds_layout(H, BF, 1).B_off + 3 * kFeatures * 4;
  hipError_t e = allow_lds(reinterpret_cast<const void*>(fn), bytes, &allowed);
  if (e != hipSuccess) return e;
  const int nw = 4;
  int64_t chunks = (q.n + kSlots - 1) / kSlots;
  // width 32: four workgroups on every CU (registers), each with the object's weights once
  int grid = (int)std::min<int64_t>((chunks + nw - 1) / nw, H == 32 ? 1024 : 2048);
  if (grid < 1) return hipSuccess;
  hipLaunchKernelGGL(fn, dim3(grid), dim3(nw * kWave), bytes, s, q);
  return hipGetLastError();
}

hipError_t launch_query(int H, bool bf16, const QueryArgs& q, hipStream_t s) {
  if (H == 32 && !bf16) return launch_query_t<32, false>(q, s);
  if (H == 32 && bf16) return launch_query_t<32, true>(q, s);
  if (H == 64 && !bf16) return launch_query_t<64, false>(q, s);
  if (H == 64 && bf16) return launch_query_t<64, true>(q, s);
  if (H == 128 && bf16) return launch_query_t<128, true>(q, s);
  return hipErrorInvalidValue;
}

hipError_t launch_fill_zero(void* dst, size_t bytes, hipStream_t s) {
  const size_t n = bytes / 4;
  if (n == 0) return hipSuccess;
  int grid = (int)std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_fill_zero, dim3(grid), dim3(256), 0, s, reinterpret_cast<uint32_t*>(dst), n);
  return hipGetLastError();
}

hipError_t launch_worklist(int n_objects, int n_rays, const int32_t* object_ids,
                           const int32_t* ray_offsets, int rays_per_tile, int rays_per_tile_wide,
                           int rays_per_tile_gen,
                           int max_objects, const ObjDesc* desc, ScalerState* scaler,
                           int32_t* tile_start, int32_t* width_start, int32_t* flags, int32_t* t_next,
                           const BatchDev* bd, const GenScan& gen, hipStream_t s) {
  if (rays_per_tile_gen < 1) return hipErrorInvalidValue;
  // (fewer waves meet at the barriers for a small batch)
  const dim3 block(n_objects <= 256 ? 256 : 1024);
  if (gen.start[0])
    hipLaunchKernelGGL(k_worklist<true>, dim3(1), block, 0, s, n_objects, n_rays, object_ids,
                       ray_offsets, rays_per_tile, rays_per_tile_wide, rays_per_tile_gen, max_objects,
                       desc, scaler, tile_start, width_start, max_objects + 1, flags, t_next, bd, gen);
  else
    hipLaunchKernelGGL(k_worklist<false>, dim3(1), block, 0, s, n_objects, n_rays, object_ids,
                       ray_offsets, rays_per_tile, rays_per_tile_wide, rays_per_tile_gen, max_objects,
                       desc, scaler, tile_start, width_start, max_objects + 1, flags, t_next, bd, gen);
  return hipGetLastError();
}

// Parameter slots per object from which the optimiser is k_reduce_adam_wide (stacks that may hold
// objects of hidden 128 and up: whole vectors of theta, m, v and the partials). Below, and in a step
// whose objects all have width 32 (tile_bad: its tile kernel built the work list), k_reduce_adam's
// one parameter per thread keeps more workgroups in flight for the few-thousand-parameter objects
// (four per thread measured 2 % slower at hidden 32).
constexpr int kReduceWide = 32768;

hipError_t launch_optimizer(int kind, const OptArgs& a, hipStream_t s) {
  if (a.n_objects <= 0) return hipSuccess;
  const int narrow = (std::min(a.p_stride, round_up(n_params_of(32), 64)) + 255) / 256;
  const dim3 grid(a.tile_bad ? narrow : (a.p_stride + 255) / 256, a.n_objects);
  // rows that fill the chip (four workgroups on every CU) gain nothing from more of them
  const int spread = (long long)grid.x * a.n_objects <= 1024 ? 3 * a.spread : 0;  // extra rows
  auto reduce = [&](dim3 g, int want_grad) {
    g.y += want_grad ? spread : 0;
    if (spread && want_grad) hipLaunchKernelGGL(k_reduce<true>, g, dim3(256), 0, s, a, want_grad);
    else hipLaunchKernelGGL(k_reduce<false>, g, dim3(256), 0, s, a, want_grad);
  };
  auto reduce_adam = [&]() {
    const dim3 g(grid.x, a.n_objects + 1 + spread);
    if (spread) hipLaunchKernelGGL(k_reduce_adam<true>, g, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_reduce_adam<false>, g, dim3(256), 0, s, a);
  };
  if (kind == OPT_REDUCE) reduce(grid, 1);
  else if (kind == OPT_LOSS) reduce(dim3(1, a.n_objects), 0);
  else if (kind == OPT_ADAM) hipLaunchKernelGGL(k_adam, grid, dim3(256), 0, s, a);
  else if (a.tile_bad) {
    reduce_adam();
  } else if (a.p_stride >= kReduceWide && a.p_stride % 4 == 0) {
    if (!a.opt_start) return hipErrorInvalidValue;
    const int units = (a.p_stride + 1023) / 1024;  // of the widest object
    // layered widths: about 4096 workgroups, rows of at most one per unit; otherwise four workgroups
    // on every CU (registers), each a run of units
    const int rows = a.gimg ? std::max(1, std::min(units, (4096 + a.n_objects - 1) / a.n_objects)) : 0;
    const long long blocks = rows ? (long long)rows * a.n_objects : std::min<long long>((long long)a.n_objects * 4 * units, 1024);
    hipLaunchKernelGGL(k_reduce_adam_wide, dim3((unsigned)blocks + 1), dim3(256), 0, s, a, rows);
  } else {
    if (a.wimage) return hipErrorInvalidValue;  // hidden-128 images are kept by the wide kernel
    reduce_adam();
  }
  return hipGetLastError();
}

hipError_t launch_init_object(int k, int H, uint64_t seed, const double* bounds,
                              const ObjDesc& d, ObjDesc* desc, float* theta, float* m,
                              float* v, float* grad, int p_stride, int use_rng,
                              hipStream_t s) {
  InitBounds ib{};
  int off = 0;
  for (int l = 0; l <= kLayers; ++l) {
    const int K = (l == 0) ? kEnc : H;
    const int O = (l == kLayers) ? kOut : H;
    ib.bound[l] = bounds[l];
    off += O * K;
    ib.w_end[l] = off;
    off += O;
    ib.b_end[l] = off;
  }
  const int P = off;
  hipLaunchKernelGGL(k_init, dim3((p_stride + 255) / 256), dim3(256), 0, s, k, seed, ib, d, desc,
                     theta, m, v, grad, p_stride, P, use_rng);
  return hipGetLastError();
}

hipError_t launch_init_scaler(ScalerState* sc, float scale, hipStream_t s) {
  hipLaunchKernelGGL(k_init_scaler, dim3(1), dim3(64), 0, s, sc, scale);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Layered path (widths without a fused tile kernel: hidden 256, 512, 1024; BF16). The step
// of Sec. 3.2-3.3 as a chain of launches over activations kept in device memory: row tiles,
// encoding, one product launch per layer forward, rendering with its adjoint (the fused kernels'
// own render_subtile), then per layer one launch for the weight gradient and one for the input
// gradient. The arithmetic takes the BF16 tile kernels' rounding points: every operand of every
// product is rounded to BF16 (encoding, activations, weights, deltas, the output layer's seed),
// products accumulate in FP32 on v_mfma_f32_32x32x16_bf16; biases, sigmoids, rendering, losses
// and the output layer's bias gradient stay FP32. An object's weight gradient is summed per work
// tile (about kGenWorkRows of its rows) by one workgroup per block of each weight matrix, in an
// order fixed by the object's rows alone, into one partial per work tile that the optimiser adds
// in tile order: the result does not depend on the grid or on the other objects.
//
// Row-tile product kernel (k_gen_gemm): a workgroup (four waves) computes a 64 x 64 block of
// D = A B over one row tile, each wave a 32 x 32 quarter, over K in chunks of 64 staged in LDS as
// BF16. Accumulator element 4 jj + i of lane l holds D[8 jj + 4 (l / 32) + i][l mod 32].
//   forward  (GEN_FWD): rows = samples, n = outputs, k = inputs;   A = h_l,   B = W_l^T
//   input gradient (GEN_DX): rows = samples, n = inputs, k = outputs;  A = delta, B = W_l
// A is staged as its rows lie (k contiguous) and read as one 16-byte LDS read per lane; B is the
// rows of W from the BF16 parameter copy, staged as they lie, read directly (forward) or
// transposed (input gradient).
// Weight gradients (k_gen_dw, k_gen_dw_small): rows = outputs, n = inputs, k = samples;
// A = delta^T, B = h_l^T, both staged as the sample rows lie and read transposed.

// Buffer of the deltas at layer m's outputs (m = 0..3). Where two buffers are taken in turn, delta and
// delta_elems are those of the launch's own two layers.
__device__ __forceinline__ uint16_t* gen_delta_out(const GenArgs& g, int m) { return g.delta + m * g.delta_elems; }

struct GenTile {
  int j, k, lo, hi;  // batch object, object id, rays [lo, hi)
};

// Row tile t of the chain, if it exists (t below the clamped tile count).
__device__ __forceinline__ bool gen_tile(const GenArgs& g, const StepArgs& a, int t, GenTile& o) {
  const int total = clamp_tiles(g.gts[a.n_objects], g.max_gen_tiles);
  if (t >= total) return false;
  const int j = gen_object(g.gts, a.n_objects, t);
  const RayRange rr = tile_ray_range(a.ray_offsets[j], a.ray_offsets[j + 1], t - g.gts[j], g.rpw,
                                     a.n_rays);
  o = GenTile{j, a.object_ids[j], rr.lo, rr.hi};
  return true;
}

// Encoding of sample `slot` of row tile tl: normalised point in FP64 rounded once, Gaussian Fourier
// features (and the integrated encoding's attenuation) as in forward_pass, rounded to BF16 in
// pairs: w[0..7] the sines of features (0, 1) .. (14, 15), w[8..15] the cosines.
__device__ __forceinline__ void gen_encode_row(const StepArgs& a, const GenTile& tl, int slot, unsigned int w[16]) {
  const ObjDesc& d = a.desc[tl.k];
  const int S = a.S;
  const int64_t row = (int64_t)tl.lo * S + slot;
  const int ray = tl.lo + slot / S;
  const double tt = (double)a.t[row];
  const float* o3 = a.rays_o + 3 * (size_t)ray;
  const float* d3 = a.rays_d + 3 * (size_t)ray;
  const double inv_s = d.inv_scale;
  float xt[4];
  xt[0] = (float)(((double)o3[0] + tt * (double)d3[0] - d.centre[0]) * inv_s);
  xt[1] = (float)(((double)o3[1] + tt * (double)d3[1] - d.centre[1]) * inv_s);
  xt[2] = (float)(((double)o3[2] + tt * (double)d3[2] - d.centre[2]) * inv_s);
  xt[3] = a.var ? (float)((double)a.var[row] * inv_s * inv_s) : 0.f;
  const float* Bm = a.B;
#pragma unroll
  for (int f = 0; f < kFeatures; f += 2) {
    float sv[2], cv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int ff = f + u;
      const float phi = xt[0] * Bm[ff] + xt[1] * Bm[kFeatures + ff] + xt[2] * Bm[2 * kFeatures + ff];
      vmap_sincosf(phi, &sv[u], &cv[u]);
      if (a.var) {
        const float nb = Bm[ff] * Bm[ff] + Bm[kFeatures + ff] * Bm[kFeatures + ff] +
                         Bm[2 * kFeatures + ff] * Bm[2 * kFeatures + ff];
        const float att = expf(-0.5f * xt[3] * nb);
        sv[u] *= att;
        cv[u] *= att;
      }
    }
    w[f / 2] = pack2(sv[0], sv[1]);
    w[(kFeatures + f) / 2] = pack2(cv[0], cv[1]);
  }
}

// Encoding of every sample of a row tile (one wave per tile) into layer 0 of the activations.
__global__ void __launch_bounds__(256) k_gen_encode(const GenArgs g_in) {
  GenArgs g = g_in;
  read_batch(g.a);
  const StepArgs& a = g.a;
  const int lane = threadIdx.x & 63, t = blockIdx.x * 4 + (threadIdx.x >> 6);
  GenTile tl;
  if (!gen_tile(g, a, t, tl)) return;
  const int S = a.S, nslots = (tl.hi - tl.lo) * S;
  if (lane >= nslots) return;
  unsigned int w[16];
  gen_encode_row(a, tl, lane, w);
  unsigned int* out = reinterpret_cast<unsigned int*>(g.act + ((int64_t)tl.lo * S + lane) * g.ld);
#pragma unroll
  for (int i = 0; i < 16; ++i) out[i] = w[i];
}

// Rows of product block b of the layered chain: T = 64, row tile b (at most 64 rows, whole rays);
// T = 256, block b of the block table (an object's rows in order, cut every block_rows rows); T = 128,
// block b, or in a table of 256-row blocks half b mod 2 of block b / 2. False if b is past the chain's
// blocks or holds no row. (As halves the 128-row blocks leave every object whose last block is at most
// half full a workgroup without rows, and with objects of one size always on the same XCDs: rendering
// 50 hidden-512 objects of 320 rows, in halves 130 us, in 128-row blocks 106; the step 607 and 547.)
template <int T>
__device__ __forceinline__ bool gen_rows(const GenArgs& g, const StepArgs& a, int b, int& k, int64_t& r0, int& nrows) {
  if constexpr (T == 64) {
    GenTile tl;
    if (!gen_tile(g, a, b, tl)) return false;
    k = tl.k;
    r0 = (int64_t)tl.lo * a.S;
    nrows = (tl.hi - tl.lo) * a.S;
  } else {
    static_assert(T == kGenBlockRows || 2 * T == kGenBlockRows, "whole or half row blocks");
    const int sh = T == kGenBlockRows || g.block_rows == T ? 0 : 1;  // halves
    const int total = clamp_tiles(g.gbs[a.n_objects], g.max_gen_blocks);
    if ((b >> sh) >= total) return false;
    const int j = gen_object(g.gbs, a.n_objects, b >> sh);
    const RayRange rr = tile_ray_range(a.ray_offsets[j], a.ray_offsets[j + 1], 0, kWholeObject, a.n_rays);
    const int64_t first = (int64_t)(b - (g.gbs[j] << sh)) * T;
    const int64_t rows = (int64_t)(rr.hi - rr.lo) * a.S;
    k = a.object_ids[j];
    r0 = (int64_t)rr.lo * a.S + first;
    nrows = (int)(rows - first < T ? rows - first : T);
  }
  return nrows > 0;  // (the second half of an object's last block may hold none)
}

// Forward and input-gradient products of one row block: a workgroup (four waves, 2 x 2) computes
// a T x T block of D = A B (T = 64 or 128), each wave a T/2 x T/2 quarter as (T/64)^2 32 x 32
// MFMA tiles, over K in chunks of 64. A (h_l, or the deltas at layer l's outputs) is staged as its
// rows lie; B is rows of W from the object's BF16 parameter copy (the optimiser keeps it equal to
// the parameters rounded to nearest even), read directly (forward: W rows are
// the output columns, k contiguous) or transposed (input gradient: W rows are the k index). The
// next chunk's loads are in flight while the current chunk's products run. The 128-row input
// gradient is compiled for three waves per SIMD (164 registers, no spill; it had taken 182 and
// run two), as the forward product already runs.
template <int KIND, int T>
__global__ void __launch_bounds__(256, (KIND == GEN_DX && T == 128) ? 3 : 1) k_gen_gemm(const GenArgs g_in, int l, int ncol_blocks) {
  static_assert(KIND == GEN_FWD || KIND == GEN_DX, "products over one row block");
  static_assert(T == 64 || T == 128, "block sizes");
  GenArgs g = g_in;
  read_batch(g.a);
  const StepArgs& a = g.a;
  constexpr int KC = kGenKChunk, PA = KC + 8;  // K per chunk; pitch of k-contiguous tiles
  constexpr int PT = T + T / 8;                // pitch of the transposed W tile (rows = k)
  constexpr int WT = T / 2, NS = WT / 32;      // wave tile, 32 x 32 MFMA tiles per dimension
  constexpr int NA = T * KC / 8 / 256;         // A pieces (8 BF16) per thread and chunk
  constexpr int NB = T * KC / 8 / 256;         // W pieces (8 BF16) per thread and chunk
  constexpr int PC = T + 8;                    // pitch of the staged result block
  constexpr int kA = T * PA, kB = (KIND == GEN_FWD) ? T * PA : KC * PT;
  static_assert(T * PC <= kA + kB, "the result block fits the operand tiles");
  __shared__ __attribute__((aligned(16))) uint16_t lds[kA + kB];
  uint16_t* As = lds;
  uint16_t* Bs = lds + kA;
  const int H = g.H;
  const bool head = (l == kLayers);
  const int K = (l == 0) ? kEnc : H;  // inputs of layer l
  const int O = head ? kOut : H;      // outputs of layer l
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, m32 = lane & 31, kh = lane >> 5;
  const int64_t ld = g.ld;
  const uint16_t* act_l = g.act + (int64_t)l * g.layer_elems;  // h_l (l = 0: the encoding)
  const uint16_t* dout = head ? nullptr : gen_delta_out(g, l);  // delta at layer l's outputs
  // row block bx, column block by (of ncol_blocks), the row blocks dealt to the XCDs in turn
  int bx, by;
  xcd_unit_block((int)blockIdx.x, ncol_blocks, bx, by);
  int k, nrows;
  int64_t r0;
  if (!gen_rows<T>(g, a, bx, k, r0, nrows)) return;
  const int n0 = by * T;
  const float* W = a.theta + (size_t)k * a.p_stride + layer_param_off(H, l);  // [O][K], then b [O]
  const uint16_t* Wb = a.gimg + (size_t)k * a.p_stride + layer_param_off(H, l);  // W in BF16
  const int ktot = (KIND == GEN_FWD) ? K : O;
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  // A piece p = tid + 256 q: row p / 8, k columns 8 (p mod 8); ktot is a multiple of 8, or the
  // output layer's 4 seeds (FP32 [rows][4], rounded here)
  u4 va[NA], vw[NB];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int p = tid + 256 * q, m = p >> 3, c = (p & 7) * 8;
      va[q] = u4{0u, 0u, 0u, 0u};
      if (m < nrows && k0 + c < ktot) {
        const int64_t row = r0 + m;
        if (KIND == GEN_DX && head) {
          const float4 d4 = *reinterpret_cast<const float4*>(g.dz + row * kOut);
          va[q] = u4{pack2(d4.x, d4.y), pack2(d4.z, d4.w), 0u, 0u};
        } else {
          va[q] = *reinterpret_cast<const u4*>(((KIND == GEN_FWD) ? act_l : dout) + row * ld + k0 + c);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int p = tid + 256 * q;
      vw[q] = u4{0u, 0u, 0u, 0u};
      if constexpr (KIND == GEN_FWD) {  // W rows n0 + n, k0 + c .. + 7 (K is a multiple of 8)
        const int n = p >> 3, c = (p & 7) * 8;
        if (n0 + n < O && k0 + c < K) vw[q] = *reinterpret_cast<const u4*>(Wb + (size_t)(n0 + n) * K + k0 + c);
      } else {  // W rows k0 + o, columns n0 + c .. + 7
        const int o = p / (T / 8), c = (p % (T / 8)) * 8;
        if (k0 + o < O && n0 + c < K) vw[q] = *reinterpret_cast<const u4*>(Wb + (size_t)(k0 + o) * K + n0 + c);
      }
    }
  };
  f32x16 acc[NS][NS];
#pragma unroll
  for (int mi = 0; mi < NS; ++mi)
#pragma unroll
    for (int ni = 0; ni < NS; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;
  fetch(0);
  for (int k0 = 0; k0 < ktot; k0 += KC) {
    __syncthreads();  // the previous chunk's operands have been read
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int p = tid + 256 * q;
      *reinterpret_cast<u4*>(As + (p >> 3) * PA + (p & 7) * 8) = va[q];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int p = tid + 256 * q;
      if constexpr (KIND == GEN_FWD) *reinterpret_cast<u4*>(Bs + (p >> 3) * PA + (p & 7) * 8) = vw[q];
      else *reinterpret_cast<u4*>(Bs + (p / (T / 8)) * PT + (p % (T / 8)) * 8) = vw[q];
    }
    if (k0 + KC < ktot) fetch(k0 + KC);
    __syncthreads();
#pragma unroll
    for (int kc = 0; kc < KC / 16; ++kc) {
      bf16x8 av[NS], bv[NS];
#pragma unroll
      for (int mi = 0; mi < NS; ++mi)
        av[mi] = *reinterpret_cast<const bf16x8*>(As + (wm * WT + mi * 32 + m32) * PA + kc * 16 + kh * 8);
#pragma unroll
      for (int ni = 0; ni < NS; ++ni) {
        if constexpr (KIND == GEN_FWD)
          bv[ni] = *reinterpret_cast<const bf16x8*>(Bs + (wn * WT + ni * 32 + m32) * PA + kc * 16 + kh * 8);
        else
          bv[ni] = tr_operand<PT>(Bs, 16 * kc, wn * WT + ni * 32, lane);
      }
#pragma unroll
      for (int mi = 0; mi < NS; ++mi)
#pragma unroll
        for (int ni = 0; ni < NS; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[mi], bv[ni], acc[mi][ni], 0, 0, 0);
    }
  }

  // epilogue: element 4 jj + i of a tile is D[row 8 jj + 4 kh + i][column m32] of that tile
  if (KIND == GEN_FWD && head) {  // the output layer's pre-activations, FP32 [rows][4]
#pragma unroll
    for (int ni = 0; ni < NS; ++ni) {
      const int col = n0 + wn * WT + ni * 32 + m32;
      if (col >= O) continue;
      const float b = W[(size_t)O * K + col];
#pragma unroll
      for (int mi = 0; mi < NS; ++mi)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int r = wm * WT + mi * 32 + 8 * (i >> 2) + 4 * kh + (i & 3);
          if (r < nrows) g.z[(r0 + r) * kOut + col] = acc[mi][ni][i] + b;
        }
    }
    return;
  }
  // Hidden outputs (forward: ReLU(D + b); input gradient: D) rounded to BF16 into a T x T block in
  // LDS, then written as rows, 16 bytes at a time; the input gradient multiplies by ReLU' of layer
  // l - 1 (its BF16 output h_l is +0 exactly where the unit is inactive), read as rows too.
  __syncthreads();  // every wave is done with the operand tiles
  uint16_t* Cs = lds;
  const int ncols = (KIND == GEN_FWD) ? O : K;
#pragma unroll
  for (int ni = 0; ni < NS; ++ni) {
    const int cl = wn * WT + ni * 32 + m32;
    float b = 0.f;
    if constexpr (KIND == GEN_FWD) b = (n0 + cl < O) ? W[(size_t)O * K + n0 + cl] : 0.f;
#pragma unroll
    for (int mi = 0; mi < NS; ++mi)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int rl = wm * WT + mi * 32 + 8 * (i >> 2) + 4 * kh + (i & 3);
        float y = acc[mi][ni][i];
        if constexpr (KIND == GEN_FWD) {
          y += b;
          y = (y <= 0.f) ? 0.f : y;  // ReLU (a NaN stays NaN)
        }
        Cs[rl * PC + cl] = (uint16_t)(pack2(y, 0.f) & 0xffffu);
      }
  }
  __syncthreads();
  uint16_t* dst = (KIND == GEN_FWD) ? g.act + (int64_t)(l + 1) * g.layer_elems : gen_delta_out(g, l - 1);
  constexpr int CPR = T / 8;  // 16-byte pieces per row
#pragma unroll
  for (int q = 0; q < T * CPR / 256; ++q) {
    const int p = tid + 256 * q, r = p / CPR, c = (p % CPR) * 8;
    if (r >= nrows || n0 + c >= ncols) continue;  // ncols is a multiple of 8
    u4 v = *reinterpret_cast<const u4*>(Cs + r * PC + c);
    const int64_t off = (r0 + r) * ld + n0 + c;
    if constexpr (KIND == GEN_DX) {
      const u4 h = *reinterpret_cast<const u4*>(act_l + off);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned int lo = (h[e] & 0xffffu) ? 0xffffu : 0u, hi = (h[e] >> 16) ? 0xffff0000u : 0u;
        v[e] &= lo | hi;
      }
    }
    *reinterpret_cast<u4*>(dst + off) = v;
  }
}

// Work tile w of the layered chain (counted over the chain's objects alone, gws), whose
// weight-gradient partial a workgroup computes: its object's id, its index in the batch's work
// list (tile_start, shared with the other widths) and its rows (g.work_rays rays of one object),
// if w is a work tile of one of the chain's objects with rows (else false).
struct GenObj {
  int k, ts;
  int64_t r0;  // first row
  int nrows;
};
__device__ __forceinline__ bool gen_work_rows(const GenArgs& g, const StepArgs& a, int w, GenObj& o) {
  if (!a.scaler->batch_ok) return false;
  const int total = clamp_tiles(g.gws[a.n_objects], a.max_tiles);
  if (w >= total) return false;
  const int j = gen_object(g.gws, a.n_objects, w);
  const int k = a.object_ids[j];
  if (k < 0 || k >= a.max_objects || !a.desc[k].registered || a.desc[k].hidden != g.H) return false;
  const int i = w - g.gws[j];  // work tile i of object j
  const TileRange tr = clamp_tile_range(a.tile_start[j], a.tile_start[j + 1], a.max_tiles);
  if (i < 0 || tr.t0 + i >= tr.t1) return false;
  const RayRange rr = tile_ray_range(a.ray_offsets[j], a.ray_offsets[j + 1], i, g.work_rays, a.n_rays);
  o = GenObj{k, tr.t0 + i, (int64_t)rr.lo * a.S, (rr.hi - rr.lo) * a.S};
  return o.nrows > 0;
}

// Weight gradient of a hidden layer of more than 32 outputs: dW_l[o][i] = sum over the object's
// rows r of delta_l[r][o] h_l[r][i], and the bias gradient sum_r delta_l[r][o] (the deltas as the
// products see them, BF16). A workgroup computes the T x T block (outputs m0.., inputs n0..) of
// one object (T = 64 or 128), each wave a T/2 x T/2 quarter, over the object's rows in chunks of
// 64 taken in row order. A chunk's rows are staged as they lie in memory (16-byte loads; the next
// chunk's loads are in flight while the current chunk's products run) and the operands are read
// transposed; rows past the object's end are staged as zeros.
// nlayers > 1: the nblk blocks are those of layers l .. l + nlayers - 1 in turn (of equal shapes).
// b: this workgroup among those of the call; lds: 2 dw_tile<T> elements.
template <int T>
constexpr int dw_tile = 64 * (T + T / 8);
template <int T>
__device__ __forceinline__ void gen_dw_block(const GenArgs& g, int b, int l, int nblk, int nlayers, uint16_t* lds) {
  static_assert(T == 64 || T == 128, "block sizes");
  const StepArgs& a = g.a;
  constexpr int R = 64, P = T + T / 8;      // rows per chunk; LDS pitch (elements)
  constexpr int WT = T / 2, NS = WT / 32;   // wave tile, 32 x 32 MFMA tiles per dimension
  constexpr int CPR = T / 8;                // 16-byte pieces per staged row
  constexpr int NP = R * CPR / 256;         // pieces per thread and operand
  static_assert(R * P == dw_tile<T>, "staged rows");
  uint16_t* const As = lds;
  uint16_t* const Bs = lds + R * P;
  const int H = g.H;
  const int K = (l == 0) ? kEnc : H, O = H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, m32 = lane & 31, kh = lane >> 5;
  // work tile bj, weight block by (of nblk), the work tiles dealt to the XCDs in turn
  int bj, by;
  xcd_unit_block(b, nblk, bj, by);
  const int per_layer = nblk / nlayers;
  l += by / per_layer;
  by %= per_layer;
  GenObj ob;
  if (l >= kLayers || O <= 32 || !gen_work_rows(g, a, bj, ob)) return;
  const int64_t ld = g.ld;
  const int nrows = ob.nrows;
  const int nbi = (K + T - 1) / T;
  const int m0 = (by / nbi) * T, n0 = (by % nbi) * T;
  // this thread's pieces of a chunk: p = tid + 256 q, row p / CPR, columns 8 (p mod CPR) .. + 7,
  // the same columns in every chunk
  const int c8 = (tid % CPR) * 8;
  const uint16_t* dsrc = gen_delta_out(g, l) + ob.r0 * ld + m0 + c8;
  const uint16_t* hsrc = g.act + (int64_t)l * g.layer_elems + ob.r0 * ld + n0 + c8;
  const bool aok = m0 + c8 < O, bok = n0 + c8 < K;  // O and K are multiples of 8
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  u4 va[NP], vb[NP];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int r = k0 + (tid + 256 * q) / CPR;
      va[q] = u4{0u, 0u, 0u, 0u};
      vb[q] = u4{0u, 0u, 0u, 0u};
      if (r < nrows) {
        if (aok) va[q] = *reinterpret_cast<const u4*>(dsrc + (int64_t)r * ld);
        if (bok) vb[q] = *reinterpret_cast<const u4*>(hsrc + (int64_t)r * ld);
      }
    }
  };
  f32x16 acc[NS][NS];
#pragma unroll
  for (int mi = 0; mi < NS; ++mi)
#pragma unroll
    for (int ni = 0; ni < NS; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;
  // bias gradient (first column block, the waves of its first half): this lane's rows of
  // outputs m0 + wm WT + 32 mi + m32
  const bool bias = (n0 == 0 && wn == 0);
  float db[NS];
#pragma unroll
  for (int mi = 0; mi < NS; ++mi) db[mi] = 0.f;
  fetch(0);
  for (int k0 = 0; k0 < nrows; k0 += R) {
    __syncthreads();  // the previous chunk's operands have been read
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int row = (tid + 256 * q) / CPR;
      *reinterpret_cast<u4*>(As + row * P + c8) = va[q];
      *reinterpret_cast<u4*>(Bs + row * P + c8) = vb[q];
    }
    if (k0 + R < nrows) fetch(k0 + R);
    __syncthreads();
#pragma unroll
    for (int kc = 0; kc < R / 16; ++kc) {
      bf16x8 av[NS], bv[NS];
#pragma unroll
      for (int mi = 0; mi < NS; ++mi) av[mi] = tr_operand<P>(As, 16 * kc, wm * WT + 32 * mi, lane);
#pragma unroll
      for (int ni = 0; ni < NS; ++ni) bv[ni] = tr_operand<P>(Bs, 16 * kc, wn * WT + 32 * ni, lane);
#pragma unroll
      for (int mi = 0; mi < NS; ++mi)
#pragma unroll
        for (int ni = 0; ni < NS; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[mi], bv[ni], acc[mi][ni], 0, 0, 0);
      if (bias) {
#pragma unroll
        for (int mi = 0; mi < NS; ++mi) db[mi] = operand_sum(av[mi], db[mi]);
      }
    }
  }
  const float inv = a.use_scale ? 1.0f / a.scaler->scale : 1.0f;
  float* dst = a.partial + (size_t)ob.ts * a.p_stride + layer_param_off(H, l);
  int bad = 0;
#pragma unroll
  for (int ni = 0; ni < NS; ++ni) {
    const int col = n0 + wn * WT + ni * 32 + m32;
    if (col >= K) continue;
#pragma unroll
    for (int mi = 0; mi < NS; ++mi)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int o = m0 + wm * WT + mi * 32 + 8 * (i >> 2) + 4 * kh + (i & 3);
        if (o >= O) continue;
        const float v = acc[mi][ni][i] * inv;
        bad |= partial_bad(v);
        dst[(size_t)o * K + col] = v;
      }
  }
  if (bias) {
#pragma unroll
    for (int mi = 0; mi < NS; ++mi) {
      const float other = __shfl(db[mi], lane + 32);  // the output's other eight rows of each step
      const int o = m0 + wm * WT + mi * 32 + m32;
      if (kh == 0 && o < O) {
        const float v = (db[mi] + other) * inv;
        bad |= partial_bad(v);
        dst[(size_t)O * K + o] = v;
      }
    }
  }
  if (__syncthreads_or(bad) && tid == 0) atomicOr(&a.flags[ob.k], 1);
}

// Loss of each object of the chain: its row tiles' losses in order, into its first work tile (its
// other work tiles hold zero, so the optimiser's sum over them is the object's loss).
__device__ __forceinline__ void gen_loss_block(const GenArgs& g, int b) {
  const StepArgs& a = g.a;
  const int lane = threadIdx.x & 63;
  const int j = b * 4 + (threadIdx.x >> 6);  // a wave per batch object
  if (j >= a.n_objects) return;
  const int total = clamp_tiles(g.gts[a.n_objects], g.max_gen_tiles);
  const TileRange tr = clamp_tile_range(g.gts[j], g.gts[j + 1], total);
  const TileRange wr = clamp_tile_range(a.tile_start[j], a.tile_start[j + 1], a.max_tiles);
  if (tr.t1 <= tr.t0 || wr.t1 <= wr.t0) return;
  // the row tiles' losses are read 64 at a time (one per lane) and added one after another in
  // tile order from lane registers: the same sum as a serial loop, without a load per addition
  float s = 0.f;
  for (int t0 = tr.t0; t0 < tr.t1; t0 += 64) {
    const float v = (t0 + lane < tr.t1) ? g.gen_loss[t0 + lane] : 0.f;
    const int n = min(64, tr.t1 - t0);
    for (int i = 0; i < n; ++i) s += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), i));
  }
  if (lane == 0) a.tile_loss[wr.t0] = s;
  for (int t = wr.t0 + 1 + lane; t < wr.t1; t += 64) a.tile_loss[t] = 0.f;
}

// Weight gradients of the first layer (64 x 64 blocks, too few to fill the chip: 24 us of a launch
// of their own at 50 objects of 1,200 rows, hidden 256), of the square layers in 128 x 128 blocks
// (n1 > 0), and the losses (5 us of a launch): n0 and n1 workgroups, nb0 and nb1 to a work tile, and
// the rest. That step's launches took 98 us apart, 82 in one.
__global__ void __launch_bounds__(256) k_gen_dw(const GenArgs g_in, int n0, int nb0, int n1, int nb1) {
  GenArgs g = g_in;
  read_batch(g.a);
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * dw_tile<128>];
  const int b = (int)blockIdx.x;
  if (b < n0) gen_dw_block<64>(g, b, 0, nb0, 1, lds);
  else if (b < n0 + n1) gen_dw_block<128>(g, b - n0, 1, nb1, kLayers - 1, lds);
  else gen_loss_block(g, b - n0 - n1);
}

// A square layer's alone, nb workgroups to a work tile (deltas in two buffers in turn).
__global__ void __launch_bounds__(256) k_gen_dw_layer(const GenArgs g_in, int l, int nb) {
  GenArgs g = g_in;
  read_batch(g.a);
  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * dw_tile<128>];
  gen_dw_block<128>(g, (int)blockIdx.x, l, nb, 1, lds);
}

// 256 x 256 blocks of the products above, for the square layers of widths that are multiples of
// 256: D[feature][column] over K in chunks of 64, eight waves of 128 features x 64 columns each.
//   GEN_FWD: feature = output, column = sample, k = input;  operands W rows, h_l rows
//   GEN_DX:  feature = input, column = sample, k = output;  operands W (transposed reads), delta rows
//   GEN_DW:  feature = output, column = input, k = sample;  operands delta, h_l (transposed reads)
// Products and sums are those of k_gen_gemm and k_gen_dw, each element's over k in the same order.
//
// k_gen_gemm's and k_gen_dw's 128 x 128 blocks run at 560 to 670 TFLOP/s because the LDS is busy
// for longer than the matrix cores: per chunk 416 cycles of writes and 290 (590 where both operands
// are read transposed) of reads for 512 of products. Here an operand read feeds four or two
// products instead of two, and chunks go from memory to LDS without passing registers, into two
// buffers in turn: one barrier per chunk, a chunk's loads in flight while the other is used. 50 objects
// of 1,200 rows at hidden 1024: forward 187 to 157 us per layer, input gradient 208 to 163, the three
// layers' weight gradients 672 to 488 in one launch. The chunks' loads bound it, 16 to 18 bytes per
// cycle and CU from the L2 (without them a chunk takes 2.3 thousand cycles instead of 3.6, without the
// products 3.5); padded row pitches, operands read a step ahead and lines touched a few chunks ahead
// changed nothing.
//
// LDS holds a chunk as the loads deliver it, 16-byte pieces in order of (row, piece). Operands read
// as rows: 256 rows of 64 k (8 pieces), piece c at c ^ ((row / 2) mod 8), so that sixteen rows of
// one column of pieces cover the banks once; operands read transposed: 64 rows (k) of 256 (32
// pieces), piece c at c ^ (4 (row mod 4)), so that a read's four rows of 64 bytes do.
enum { GEN_DW = GEN_DX + 1 };
constexpr int kWideK = 64;

__device__ __forceinline__ bf16x8 wide_rows_operand(const uint16_t* T, int rb, int kc, int lane) {
  const int n = lane & 31;
  return *reinterpret_cast<const bf16x8*>(T + (rb + n) * kWideK + (((2 * kc + (lane >> 5)) ^ ((n >> 1) & 7)) << 3));
}
__device__ __forceinline__ bf16x8 wide_tr_operand(const uint16_t* T, int kc, int cb, int lane) {
  typedef __attribute__((address_space(3))) v4i16 lds_v4;
  const int r = 8 * (lane >> 5) + ((lane & 15) >> 2);
  const int c = ((cb >> 3) ^ ((r & 3) << 2)) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  const uint16_t* p = T + (16 * kc + r) * 256 + 8 * c + 4 * (lane & 1);
  const v4i16 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p));
  const v4i16 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4*)(p + 4 * 256));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
}
// 16 bytes per lane from device memory to LDS: lane i's to dst + 16 i (dst: the wave's, uniform).
__device__ __forceinline__ void wide_load(const uint16_t* src, uint16_t* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
// Unit (of nblk workgroups each) and block of this workgroup, the units in eight runs, one per XCD:
// neighbouring units share an object's weights or rows, and so one L2. False past the last unit.
__device__ __forceinline__ bool xcd_run_block(int units, int nblk, int& unit, int& blk) {
  const int b = (int)blockIdx.x, x = b & 7, i = (b >> 3) / nblk;
  const int lo = (int)((long long)units * x / 8), hi = (int)((long long)units * (x + 1) / 8);
  unit = lo + i;
  blk = (b >> 3) % nblk;
  return unit < hi;
}

// Barrier for LDS alone: loads from and stores to device memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int KIND>
__global__ void __launch_bounds__(512, 2) k_gen_wide(const GenArgs g_in, int l) {
  GenArgs g = g_in;
  read_batch(g.a);
  const StepArgs& a = g.a;
  constexpr bool XT = KIND != GEN_FWD, YT = KIND == GEN_DW;  // operand read transposed
  __shared__ __attribute__((aligned(1024))) uint16_t X0[256 * kWideK], X1[256 * kWideK];
  __shared__ __attribute__((aligned(1024))) uint16_t Y0[256 * kWideK], Y1[256 * kWideK];
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u2w __attribute__((ext_vector_type(2)));
  const int H = g.H, nb = H / 256;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wf = wave & 1, ws = wave >> 1, n = lane & 31, kh = lane >> 5;
  const int64_t ld = g.ld;
  const uint16_t *xs, *ys;  // first row and column of the operands
  int64_t xld = ld;         // (of the samples' rows: ld)
  int k, nrows, ktot, n0, m0 = 0, ts = 0;
  int64_t r0;
  if constexpr (KIND == GEN_DW) {  // unit: a work tile's layer (1 .. kLayers - 1)
    if (!a.scaler->batch_ok) return;
    int u, by;
    if (!xcd_run_block(clamp_tiles(g.gws[a.n_objects], a.max_tiles) * (kLayers - 1), nb * nb, u, by)) return;
    GenObj ob;
    if (!gen_work_rows(g, a, u / (kLayers - 1), ob)) return;
    l = 1 + u % (kLayers - 1);
    k = ob.k;
    r0 = ob.r0;
    ktot = nrows = ob.nrows;
    ts = ob.ts;
    m0 = (by / nb) * 256;
    n0 = (by % nb) * 256;
    xs = gen_delta_out(g, l) + r0 * ld + m0;
    ys = g.act + l * g.layer_elems + r0 * ld + n0;
  } else {
    int bx, by;
    if (!xcd_run_block(clamp_tiles(g.gbs[a.n_objects], g.max_gen_blocks), nb, bx, by)) return;
    if (!gen_rows<kGenBlockRows>(g, a, bx, k, r0, nrows)) return;
    ktot = H;
    n0 = by * 256;
    const uint16_t* Wb = a.gimg + (size_t)k * a.p_stride + layer_param_off(H, l);
    xs = (KIND == GEN_FWD) ? Wb + (size_t)n0 * H : Wb + n0;
    xld = H;
    ys = ((KIND == GEN_FWD) ? g.act + l * g.layer_elems : gen_delta_out(g, l)) + r0 * ld;
  }
  // this thread's four pieces of an operand's chunk. Rows past the samples' end repeat the last one
  // (their results are not written; as k they are zeroed below).
  auto fetch = [&](int c, uint16_t* xb, uint16_t* yb) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rr = (tid >> 3) + 64 * q, rc = 8 * ((tid & 7) ^ ((tid >> 4) & 7));            // as rows
      const int tr = kWideK * c + (tid >> 5) + 16 * q, tc = 8 * ((tid & 31) ^ (((tid >> 5) & 3) << 2));  // transposed
      const int xr = XT ? (KIND == GEN_DW ? min(tr, nrows - 1) : tr) : rr;
      wide_load(xs + xr * xld + (XT ? tc : rc + kWideK * c), xb + (512 * q + 64 * wave) * 8);
      wide_load(ys + min(YT ? tr : rr, nrows - 1) * ld + (YT ? tc : rc + kWideK * c), yb + (512 * q + 64 * wave) * 8);
    }
  };
  f32x16 acc[4][2];
#pragma unroll
  for (int mi = 0; mi < 4; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;
  const bool bias = (KIND == GEN_DW) && n0 == 0 && ws == 0;
  float db[4] = {0.f, 0.f, 0.f, 0.f};
  const int nchunks = (ktot + kWideK - 1) / kWideK;
  // chunk c from (xb, yb), the next one's loads to (xn, yn)
  auto step = [&](int c, uint16_t* xb, uint16_t* yb, uint16_t* xn, uint16_t* yn) {
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's pieces of chunk c are in LDS
    if constexpr (KIND == GEN_DW) {
      if (kWideK * (c + 1) > ktot) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (kWideK * c + (tid >> 5) + 16 * q >= ktot) {
            *reinterpret_cast<u4*>(xb + (tid + 512 * q) * 8) = u4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u4*>(yb + (tid + 512 * q) * 8) = u4{0u, 0u, 0u, 0u};
          }
      }
    }
    __syncthreads();  // chunk c is complete, chunk c - 1 has been read
    if (c + 1 < nchunks) fetch(c + 1, xn, yn);
#pragma unroll
    for (int kc = 0; kc < kWideK / 16; ++kc) {
      bf16x8 x[4], y[2];
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
        x[mi] = XT ? wide_tr_operand(xb, kc, 128 * wf + 32 * mi, lane) : wide_rows_operand(xb, 128 * wf + 32 * mi, kc, lane);
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        y[ni] = YT ? wide_tr_operand(yb, kc, 64 * ws + 32 * ni, lane) : wide_rows_operand(yb, 64 * ws + 32 * ni, kc, lane);
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[mi], y[ni], acc[mi][ni], 0, 0, 0);
      if (bias) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) db[mi] = operand_sum(x[mi], db[mi]);
      }
    }
  };
  fetch(0, X0, Y0);
  for (int c = 0; c < nchunks; c += 2) {
    step(c, X0, Y0, X1, Y1);
    if (c + 1 < nchunks) step(c + 1, X1, Y1, X0, Y0);
  }
  if constexpr (KIND == GEN_DW) {
    const float inv = a.use_scale ? 1.0f / a.scaler->scale : 1.0f;
    float* dst = a.partial + (size_t)ts * a.p_stride + layer_param_off(H, l);
    // (the check first: nothing waits for the stores)
    int bad = 0;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          acc[mi][ni][i] *= inv;
          bad |= partial_bad(acc[mi][ni][i]);
        }
      db[mi] = (db[mi] + __shfl(db[mi], lane ^ 32)) * inv;  // (the output's other eight rows of each step)
      if (bias) bad |= partial_bad(db[mi]);
    }
    if (__syncthreads_or(bad) && tid == 0) atomicOr(&a.flags[k], 1);
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          dst[(size_t)(m0 + 128 * wf + 32 * mi + 8 * (i >> 2) + 4 * kh + (i & 3)) * H + n0 + 64 * ws + 32 * ni + n] = acc[mi][ni][i];
      if (bias && kh == 0) dst[(size_t)H * H + m0 + 128 * wf + 32 * mi + n] = db[mi];
    }
  } else {
    // Rounded to BF16 into rows of samples in LDS (64 samples, those of two waves, per buffer; piece
    // c of a row at c ^ (row mod 16)), then written as rows: forward ReLU(D + b); input gradient D
    // where layer l - 1's unit is active (its output h_l is +0 exactly where it is not).
    const uint16_t* act_l = g.act + l * g.layer_elems + r0 * ld + n0;
    const float* bp = a.theta + (size_t)k * a.p_stride + layer_param_off(H, l) + (size_t)H * H + n0;
    u4 h[16];  // in flight while the results are rounded: h_l's rows, or the biases
#pragma unroll
    for (int q = 0; q < 16; ++q)
      h[q] = (KIND == GEN_FWD)
                 ? *reinterpret_cast<const u4*>(bp + 128 * wf + 8 * q + 4 * kh)
                 : *reinterpret_cast<const u4*>(act_l + min(16 * q + (tid >> 5), nrows - 1) * ld + 8 * (tid & 31));
    lds_barrier();  // every wave is done with the operands
    uint16_t* out = (ws == 0) ? X0 : (ws == 1) ? X1 : (ws == 2) ? Y0 : Y1;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int f = 128 * wf + 32 * mi + 8 * jj;  // features f + 4 kh .. + 3
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
          float y[4] = {acc[mi][ni][4 * jj], acc[mi][ni][4 * jj + 1], acc[mi][ni][4 * jj + 2], acc[mi][ni][4 * jj + 3]};
          if constexpr (KIND == GEN_FWD) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const unsigned int b = h[4 * mi + jj][e];
              y[e] += __builtin_bit_cast(float, b);
              y[e] = (y[e] <= 0.f) ? 0.f : y[e];  // ReLU (a NaN stays NaN)
            }
          }
          *reinterpret_cast<u2w*>(out + (32 * ni + n) * 256 + (((f >> 3) ^ (n & 15)) << 3) + 4 * kh) =
              u2w{pack2(y[0], y[1]), pack2(y[2], y[3])};
        }
      }
    lds_barrier();
    uint16_t* dst = ((KIND == GEN_FWD) ? g.act + (l + 1) * g.layer_elems : gen_delta_out(g, l - 1)) + r0 * ld + n0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {  // piece tid mod 32 of row 16 q + tid / 32
      const int r = 16 * q + (tid >> 5), c = tid & 31;
      const uint16_t* in = (q < 4) ? X0 : (q < 8) ? X1 : (q < 12) ? Y0 : Y1;
      if (r >= nrows) continue;
      u4 v = *reinterpret_cast<const u4*>(in + (r & 63) * 256 + ((c ^ (r & 15)) << 3));
      const int64_t off = r * ld + 8 * c;
      if constexpr (KIND == GEN_DX) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] &= ((h[q][e] & 0xffffu) ? 0xffffu : 0u) | ((h[q][e] >> 16) ? 0xffff0000u : 0u);
      }
      *reinterpret_cast<u4*>(dst + off) = v;
    }
  }
}

// Weight gradient of the output layer (4 outputs) of the layered path: a workgroup computes
// outputs [0, 4) x inputs [n0, n0 + 32) over one work tile of an object, and its NW waves take the
// tile's rows in 32-row chunks in turn (chunk c to wave c mod NW), each in its own LDS tiles,
// staged as the rows lie in memory (16-byte loads, the wave's next chunk in flight during the
// current chunk's products) and read transposed: A = the FP32 seeds dz rounded to BF16 (the MFMA
// operand; rows 4..31 of the tile stay zero), B = h_4. The waves' sums are added in wave order,
// so the result does not depend on the grid. Bias gradient: the FP32 seeds unrounded, summed per
// lane over its staged rows and then over lanes and waves in a fixed order. The wave count is
// fixed (kGenDwWaves, not chosen by the size of the launch), so an object's sums do not depend on
// the rest of the batch; eight waves leave a wave an eighth of the work tile's rows and fit two
// workgroups on a CU (registers). Reading h_4 bounds it. A block's 32 columns are half a line of a row,
// so a work tile's blocks run on one XCD (xcd_unit_block), one after another: the
// hidden-256 step of 64 objects of 12,000 rows 2,357 to 2,317 us, of 32 of 1,200 228 to 223.
__global__ void __launch_bounds__(kGenDwWaves * 64) k_gen_dw_small(const GenArgs g_in, int nblk) {
  constexpr int NW = kGenDwWaves;
  GenArgs g = g_in;
  read_batch(g.a);
  constexpr int l = kLayers;
  const StepArgs& a = g.a;
  constexpr int P = kGenPitch;                   // 32 columns + 4 (elements)
  constexpr int kWaveTile = 2 * 32 * P;          // one wave's A and B tiles (uint16 elements)
  constexpr int kRed = NW * 16 * 64 + NW * 32;  // floats of the final sums: accumulators, bias sums
  __shared__ __attribute__((aligned(16))) uint16_t lds[(NW * kWaveTile > 2 * kRed) ? NW * kWaveTile : 2 * kRed];
  const int H = g.H;
  const int K = H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  GenObj ob;
  int bj, by;
  xcd_unit_block((int)blockIdx.x, nblk, bj, by);
  if (!gen_work_rows(g, a, bj, ob)) return;
  const int64_t ld = g.ld;
  const int nrows = ob.nrows;
  const int n0 = by * 32;
  const bool bias = (n0 == 0);
  uint16_t* As = lds + wave * kWaveTile;
  uint16_t* Bs = As + 32 * P;
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u2w __attribute__((ext_vector_type(2)));
  // columns that no piece covers (A's past the 4 outputs) stay zero
  for (int i = lane; i < kWaveTile / 8; i += 64) *reinterpret_cast<u4*>(As + 8 * i) = u4{0u, 0u, 0u, 0u};
  // pieces of a 32-row chunk: B (h_4, columns n0..n0+31): p = lane + 64 q, row p / 4, columns
  // 8 (p mod 4); A (the FP32 seed [rows][4]): lane < 32, row lane. A lane's columns are the same
  // in every chunk.
  const uint16_t* hsrc = g.act + (int64_t)l * g.layer_elems + ob.r0 * ld + n0;
  const float* zsrc = g.dz + ob.r0 * kOut;
  u4 vb[2];
  float4 vz;
  auto fetch = [&](int c) {
    const int rb = c * 32;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int p = lane + 64 * q, r = rb + (p >> 2), cc = 8 * (p & 3);
      vb[q] = u4{0u, 0u, 0u, 0u};
      if (r < nrows && n0 + cc < K) vb[q] = *reinterpret_cast<const u4*>(hsrc + (int64_t)r * ld + cc);
    }
    vz = make_float4(0.f, 0.f, 0.f, 0.f);
    if (lane < 32 && rb + lane < nrows) vz = *reinterpret_cast<const float4*>(zsrc + (int64_t)(rb + lane) * kOut);
  };
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  float dbv[kOut] = {0.f, 0.f, 0.f, 0.f};  // this lane's bias parts
  if (wave * 32 < nrows) fetch(wave);
  for (int c = wave; c * 32 < nrows; c += NW) {
    wave_lds_sync();  // this wave's previous chunk has been read
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int p = lane + 64 * q;
      *reinterpret_cast<u4*>(Bs + (p >> 2) * P + 8 * (p & 3)) = vb[q];
    }
    if (lane < 32) {
      *reinterpret_cast<u2w*>(As + lane * P) = u2w{pack2(vz.x, vz.y), pack2(vz.z, vz.w)};
      if (bias) {
        dbv[0] += vz.x;
        dbv[1] += vz.y;
        dbv[2] += vz.z;
        dbv[3] += vz.w;
      }
    }
    if ((c + NW) * 32 < nrows) fetch(c + NW);
    wave_lds_sync();
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const bf16x8 av = tr_operand<P>(As, 16 * kc, 0, lane);
      const bf16x8 bv = tr_operand<P>(Bs, 16 * kc, 0, lane);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
    }
  }
  // bias parts: a butterfly over the wave's lanes (the seeds sit on lanes 0..31, the others hold
  // zeros), leaving the wave's sums on every lane, in a fixed order
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int e = 0; e < kOut; ++e) dbv[e] += __shfl_xor(dbv[e], off);
  }
  __syncthreads();  // every wave is done with its tiles
  float* red = reinterpret_cast<float*>(lds);  // [NW waves][16][64], then [NW waves][32] bias sums
  float* redb = red + NW * 16 * 64;
#pragma unroll
  for (int i = 0; i < 16; ++i) red[(wave * 16 + i) * 64 + lane] = acc[i];
  if (lane == 0) {
#pragma unroll
    for (int e = 0; e < kOut; ++e) redb[wave * 32 + e] = dbv[e];
  }
  __syncthreads();
  // element i of the accumulators (output 8 (i / 4) + 4 (lane / 32) + i mod 4, input n0 + lane mod
  // 32) is summed over the waves in wave order by wave i mod NW; outputs 0..3 are elements 0..3
  // of lanes 0..31
  int bad = 0;
  const float inv = a.use_scale ? 1.0f / a.scaler->scale : 1.0f;
  float* dst = a.partial + (size_t)ob.ts * a.p_stride + layer_param_off(H, l);
  const int col = n0 + (lane & 31);
  for (int i = wave; i < kOut; i += NW) {
    if (lane >= 32 || col >= K) continue;
    float v = red[i * 64 + lane];
    for (int w = 1; w < NW; ++w) v += red[(w * 16 + i) * 64 + lane];
    v *= inv;
    bad |= partial_bad(v);
    dst[(size_t)i * K + col] = v;
  }
  if (bias && wave == 0 && lane < kOut) {
    float v = 0.f;
    for (int w = 0; w < NW; ++w) v += redb[w * 32 + lane];
    v *= inv;
    bad |= partial_bad(v);
    dst[(size_t)kOut * K + lane] = v;
  }
  if (__syncthreads_or(bad) && tid == 0) atomicOr(&a.flags[ob.k], 1);
}

// Rendering, loss and (training) the adjoint of one row tile per wave, by the fused kernels'
// render_subtile; the tile's loss (a fixed-order wave sum) goes to gen_loss, dL/dz to dz.
template <bool TRAIN>
__global__ void __launch_bounds__(256) k_gen_render(const GenArgs g_in) {
  GenArgs g = g_in;
  read_batch(g.a);
  const StepArgs& a = g.a;
  const int lane = threadIdx.x & 63, t = blockIdx.x * 4 + (threadIdx.x >> 6);
  GenTile tl;
  if (!gen_tile(g, a, t, tl)) return;  // uniform over the wave
  const int S = a.S, nslots = (tl.hi - tl.lo) * S;
  const int64_t row0 = (int64_t)tl.lo * S;
  float zs[kOut] = {0.f, 0.f, 0.f, 0.f};
  if (lane < nslots) {
#pragma unroll
    for (int c = 0; c < kOut; ++c) zs[c] = g.z[(row0 + lane) * kOut + c];
  }
  float wseed = 1.0f;
  if constexpr (TRAIN) {
    if (a.dloss) wseed = a.dloss[tl.j];
    if (a.use_scale) wseed *= a.scaler->scale;
  }
  const RenderIn rin = render_inputs<TRAIN>(a, tl.lo, nslots);
  float dzs[kOut] = {0.f, 0.f, 0.f, 0.f};
  float loss = 0.f;
  render_subtile<TRAIN>(a, tl.lo, nslots, wseed, rin, zs, dzs, loss);
  if constexpr (TRAIN) {
    if (lane < nslots) {
#pragma unroll
      for (int c = 0; c < kOut; ++c) g.dz[(row0 + lane) * kOut + c] = dzs[c];
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
  if (lane == 0) g.gen_loss[t] = loss;
}

__global__ void __launch_bounds__(256) k_gen_loss(const GenArgs g_in) {
  GenArgs g = g_in;
  read_batch(g.a);
  gen_loss_block(g, (int)blockIdx.x);
}

// BF16 copy of object k's parameter slots (round to nearest even), eight per thread.
__global__ void __launch_bounds__(256) k_gen_stage_gimg(const float* __restrict__ theta, uint16_t* __restrict__ gimg,
                                                       int k, int p_stride) {
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  const int p = (blockIdx.x * blockDim.x + threadIdx.x) * 8;  // p_stride is a multiple of 8
  if (p >= p_stride) return;
  const size_t i = (size_t)k * p_stride + p;
  const float4 x0 = *reinterpret_cast<const float4*>(theta + i);
  const float4 x1 = *reinterpret_cast<const float4*>(theta + i + 4);
  *reinterpret_cast<u4*>(gimg + i) = u4{pack2(x0.x, x0.y), pack2(x0.z, x0.w), pack2(x1.x, x1.y), pack2(x1.z, x1.w)};
}

hipError_t launch_stage_gimg(const float* theta, uint16_t* gimg, int k, int p_stride, hipStream_t s) {
  if (!theta || !gimg || k < 0 || p_stride <= 0 || p_stride % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gen_stage_gimg, dim3((p_stride / 8 + 255) / 256), dim3(256), 0, s, theta, gimg, k, p_stride);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Hidden 256: the forward products, the rendering with its adjoint and the input gradients of two
// row tiles (at most 128 rows of one object) by one workgroup of eight waves, the activations and
// deltas passing between layers through LDS. Wave w computes features 32 w .. + 31 of every layer
// for all rows (four 32 x 32 tiles); its ReLU masks stay in registers, a bit each. What the weight
// gradients read (encodings, activations, deltas, dz) is written to device memory as rows, while the
// next layer runs. W comes from the object's BF16 copy: the forward's operands straight from
// device memory (a wave's rows are its own; the next layer's are fetched during the current one),
// the input gradient's in chunks of 64 rows staged in LDS and read transposed. Operands, products
// and sums are those of k_gen_encode, k_gen_gemm and k_gen_render, in their order.
//
// One launch per layer and direction, each waiting for its first operands for most of its four
// chunks of K, took 224 us of a 441 us step (50 objects of 120 rays x 10 samples, 60,000 rows); this
// one 134. LDS reads of the rows bound it (about 512 KB per layer and workgroup); 500 workgroups
// on 256 CUs leave it two rounds.

struct LdsChain {
  int buf_off, enc_off, z_off, dz_off, total;
};
constexpr int kChainWidth = 256;
constexpr int kChainRows = 128;
constexpr int kChainPitch = kChainWidth + 8;  // BF16 elements per row
constexpr int kChainEncPitch = kEnc + 8;
constexpr int kChainBuf = kChainRows * kChainPitch * 2;
__host__ __device__ constexpr LdsChain lds_chain() {
  LdsChain L{};
  int off = 0;
  L.buf_off = off; off += 2 * kChainBuf;
  L.enc_off = off; off += kChainRows * kChainEncPitch * 2;
  L.z_off = off; off += kChainRows * kOut * 4;
  L.dz_off = off; off += kChainRows * kOut * 2;
  L.total = off;
  return L;
}
static_assert(lds_chain().total <= 160 * 1024, "the hidden-256 chain's LDS");
static_assert(2 * 64 * kChainPitch * 2 <= kChainBuf, "two staged chunks of W fit a row buffer");

template <bool TRAIN>
__global__ void __launch_bounds__(512, 2) k_gen_chain(const GenArgs g_in) {
  constexpr int H = kChainWidth, P = kChainPitch, KS = H / 16;
  constexpr LdsChain L = lds_chain();
  GenArgs g = g_in;
  read_batch(g.a);
  const StepArgs& a = g.a;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* const buf0 = reinterpret_cast<uint16_t*>(smem + L.buf_off);
  uint16_t* const buf1 = buf0 + kChainBuf / 2;
  uint16_t* const enc = reinterpret_cast<uint16_t*>(smem + L.enc_off);
  float* const zl = reinterpret_cast<float*>(smem + L.z_off);
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  typedef unsigned int u2w __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, hf = lane >> 5;
  // unit: row tiles t0 and t0 + 1 of object j (units dealt to the XCDs in turn); rows 0..63 of the
  // buffers hold the first tile's samples, 64..127 the second's
  int unit, one;
  xcd_unit_block((int)blockIdx.x, 1, unit, one);
  if (unit >= clamp_tiles(g.gbs[a.n_objects], g.max_gen_tiles)) return;
  const int j = gen_object(g.gbs, a.n_objects, unit);
  const int k = a.object_ids[j];
  const int o0 = a.ray_offsets[j], o1 = a.ray_offsets[j + 1], S = a.S;
  const int ti = 2 * (unit - g.gbs[j]);
  const RayRange ra = tile_ray_range(o0, o1, ti, g.rpw, a.n_rays), rb = tile_ray_range(o0, o1, ti + 1, g.rpw, a.n_rays);
  const int na = (ra.hi - ra.lo) * S, nb = (rb.hi - rb.lo) * S;  // rows of each tile
  const int64_t base_a = (int64_t)ra.lo * S, base_b = (int64_t)rb.lo * S;
  // global row of buffer row r, or -1
  auto row_of = [&](int r) -> int64_t {
    return r < 64 ? (r < na ? base_a + r : -1) : (r - 64 < nb ? base_b + (r - 64) : -1);
  };
  const uint16_t* const W = a.gimg + (size_t)k * a.p_stride;
  const float* const theta = a.theta + (size_t)k * a.p_stride;
  const int64_t ld = g.ld;

  // encodings: four threads per row, four frequencies each
  {
    const int r = tid >> 2, f0 = 4 * (tid & 3);
    const int64_t row = row_of(r);
    u2w sw{0u, 0u}, cw{0u, 0u};
    if (row >= 0) {
      const ObjDesc& d = a.desc[k];
      const int ray = (r < 64 ? ra.lo : rb.lo) + (r & 63) / S;
      const double tt = (double)a.t[row];
      const float* o3 = a.rays_o + 3 * (size_t)ray;
      const float* d3 = a.rays_d + 3 * (size_t)ray;
      const double inv_s = d.inv_scale;
      float xt[4];
      xt[0] = (float)(((double)o3[0] + tt * (double)d3[0] - d.centre[0]) * inv_s);
      xt[1] = (float)(((double)o3[1] + tt * (double)d3[1] - d.centre[1]) * inv_s);
      xt[2] = (float)(((double)o3[2] + tt * (double)d3[2] - d.centre[2]) * inv_s);
      xt[3] = a.var ? (float)((double)a.var[row] * inv_s * inv_s) : 0.f;
      const float* Bm = a.B;
      float sv[4], cv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int ff = f0 + u;
        const float phi = xt[0] * Bm[ff] + xt[1] * Bm[kFeatures + ff] + xt[2] * Bm[2 * kFeatures + ff];
        vmap_sincosf(phi, &sv[u], &cv[u]);
        if (a.var) {
          const float nbq = Bm[ff] * Bm[ff] + Bm[kFeatures + ff] * Bm[kFeatures + ff] +
                            Bm[2 * kFeatures + ff] * Bm[2 * kFeatures + ff];
          const float att = expf(-0.5f * xt[3] * nbq);
          sv[u] *= att;
          cv[u] *= att;
        }
      }
      sw = u2w{pack2(sv[0], sv[1]), pack2(sv[2], sv[3])};
      cw = u2w{pack2(cv[0], cv[1]), pack2(cv[2], cv[3])};
      if constexpr (TRAIN) {
        *reinterpret_cast<u2w*>(g.act + row * ld + f0) = sw;
        *reinterpret_cast<u2w*>(g.act + row * ld + kFeatures + f0) = cw;
      }
    }
    *reinterpret_cast<u2w*>(enc + r * kChainEncPitch + f0) = sw;
    *reinterpret_cast<u2w*>(enc + r * kChainEncPitch + kFeatures + f0) = cw;
  }

  // this wave's A operands of a forward layer: rows 32 wave + n of W_l, K step kc: 16 kc + 8 hf ..
  bf16x8 wa[KS];
  auto fetch_w = [&](int l) {
    const int K = l == 0 ? kEnc : H;
    const uint16_t* src = W + layer_param_off(H, l) + (size_t)(32 * wave + n) * K + 8 * hf;
#pragma unroll
    for (int kc = 0; kc < KS; ++kc)
      if (16 * kc < K) wa[kc] = *reinterpret_cast<const bf16x8*>(src + 16 * kc);
  };
  // rows of a buffer to device memory, 16 bytes at a time
  auto store_rows = [&](const uint16_t* src, uint16_t* dst) {
    int t = tid;
    asm volatile("" : "+v"(t));  // (addresses are computed here, not kept across the layers)
#pragma unroll
    for (int q = 0; q < kChainRows * H / 8 / 512; ++q) {
      const int p = t + 512 * q, r = p >> 5, c = (p & 31) * 8;
      const int64_t row = row_of(r);
      if (row >= 0) *reinterpret_cast<u4*>(dst + row * ld + c) = *reinterpret_cast<const u4*>(src + r * P + c);
    }
  };
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
  // ReLU masks: element 2 i + e of row block s is active where bit 16 e + 8 (s mod 2) + i of word
  // s / 2 is set (packed words of two elements, their non-zero flags shifted together)
  unsigned int mask[kLayers][2];
  fetch_w(0);
  __syncthreads();

  // ---------------- forward
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    const uint16_t* src = l == 0 ? enc : ((l & 1) ? buf0 : buf1);
    const int pitch = l == 0 ? kChainEncPitch : P;
    uint16_t* dst = (l & 1) ? buf1 : buf0;
    const float* bias = theta + layer_param_off(H, l) + H * (l == 0 ? kEnc : H) + 32 * wave + 4 * hf;
    f32x4 b4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) b4[q] = *reinterpret_cast<const f32x4*>(bias + 8 * q);
    f32x16 acc[4] = {zero, zero, zero, zero};
#pragma unroll
    for (int kc = 0; kc < (l == 0 ? kEnc / 16 : KS); ++kc)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            wa[kc], *reinterpret_cast<const bf16x8*>(src + (32 * s + n) * pitch + 16 * kc + 8 * hf), acc[s], 0, 0, 0);
    if (l + 1 < kLayers) fetch_w(l + 1);
    mask[l][0] = mask[l][1] = 0u;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {  // features 32 wave + 8 q + 4 hf + 0..3 of row 32 s + n
        float y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          y[i] = acc[s][4 * q + i] + b4[q][i];
          y[i] = (y[i] <= 0.f) ? 0.f : y[i];  // ReLU (a NaN stays NaN)
        }
        const u2w w{pack2(y[0], y[1]), pack2(y[2], y[3])};
        *reinterpret_cast<u2w*>(dst + (32 * s + n) * P + 32 * wave + 8 * q + 4 * hf) = w;
        if constexpr (TRAIN)
          mask[l][s >> 1] |= (nonzero16(w[0]) << (8 * (s & 1) + 2 * q)) | (nonzero16(w[1]) << (8 * (s & 1) + 2 * q + 1));
      }
    __syncthreads();
    if constexpr (TRAIN) store_rows(dst, g.act + (int64_t)(l + 1) * g.layer_elems);
  }
  // output layer: waves 0..3 a row block each (W_out's four rows padded to 32)
  if (wave < 4) {
    const uint16_t* wo = W + layer_param_off(H, kLayers) + (size_t)n * H + 8 * hf;
    const uint16_t* src = buf1 + (32 * wave + n) * P + 8 * hf;
    f32x16 acc = zero;
#pragma unroll
    for (int kc = 0; kc < KS; ++kc) {
      bf16x8 w = {};
      if (n < kOut) w = *reinterpret_cast<const bf16x8*>(wo + 16 * kc);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, *reinterpret_cast<const bf16x8*>(src + 16 * kc), acc, 0, 0, 0);
    }
    const float* bo = theta + layer_param_off(H, kLayers) + kOut * H;
    if (hf == 0)
      *reinterpret_cast<f32x4*>(zl + (32 * wave + n) * kOut) = f32x4{acc[0] + bo[0], acc[1] + bo[1], acc[2] + bo[2], acc[3] + bo[3]};
  }
  __syncthreads();
  // rendering, loss and adjoint: waves 0 and 1 a row tile each
  if (wave < 2) {
    const int lo = wave ? rb.lo : ra.lo, nslots = wave ? nb : na;
    float zs[kOut], dzs[kOut] = {0.f, 0.f, 0.f, 0.f}, loss = 0.f, wseed = 1.0f;
#pragma unroll
    for (int c = 0; c < kOut; ++c) zs[c] = lane < nslots ? zl[(64 * wave + lane) * kOut + c] : 0.f;
    if constexpr (TRAIN) {
      if (a.dloss) wseed = a.dloss[j];
      if (a.use_scale) wseed *= a.scaler->scale;
    }
    const RenderIn rin = render_inputs<TRAIN>(a, lo, nslots);
    render_subtile<TRAIN>(a, lo, nslots, wseed, rin, zs, dzs, loss);
    if constexpr (TRAIN) {
      if (lane < nslots)
        *reinterpret_cast<f32x4*>(g.dz + ((int64_t)lo * S + lane) * kOut) = f32x4{dzs[0], dzs[1], dzs[2], dzs[3]};
      *reinterpret_cast<u2w*>(smem + L.dz_off + (64 * wave + lane) * kOut * 2) = u2w{pack2(dzs[0], dzs[1]), pack2(dzs[2], dzs[3])};
    }
    loss = wave_sum(loss);
    if (lane == 0 && nslots > 0) g.gen_loss[g.gts[j] + ti + wave] = loss;
  }
  if constexpr (!TRAIN) return;
  __syncthreads();

  // ---------------- input gradients (deltas in buf0, W chunks in buf1)
  uint16_t* const D = buf0;
  // a lane's deltas of its four row blocks: rounded, masked by ReLU' of layer m, staged
  auto put_delta = [&](const f32x16 (&acc)[4], int m) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        typedef unsigned short us2 __attribute__((ext_vector_type(2)));
        u2w w{pack2(acc[s][4 * q], acc[s][4 * q + 1]), pack2(acc[s][4 * q + 2], acc[s][4 * q + 3])};
#pragma unroll
        for (int e = 0; e < 2; ++e) {  // each packed delta times its flag (0 or 1)
          const unsigned int f = (mask[m][s >> 1] >> (8 * (s & 1) + 2 * q + e)) & 0x00010001u, we = w[e];
          w[e] = __builtin_bit_cast(unsigned int, (us2)(__builtin_bit_cast(us2, we) * __builtin_bit_cast(us2, f)));
        }
        *reinterpret_cast<u2w*>(D + (32 * s + n) * P + 32 * wave + 8 * q + 4 * hf) = w;
      }
  };
  // chunk i of the input gradients: rows 64 (i mod 4) .. + 63 of W_(3 - i / 4), 64 x 256 elements,
  // four 16-byte pieces per thread. Two chunks ahead are in flight or in registers, one in LDS.
  constexpr int kChunks = 4 * (kLayers - 1);
  u4 wc[2][4];
  auto fetch_chunk = [&](int i) {
    const uint16_t* src = W + layer_param_off(H, kLayers - 1 - i / 4) + (size_t)64 * (i & 3) * H;
#pragma unroll
    for (int q = 0; q < 4; ++q) wc[i & 1][q] = *reinterpret_cast<const u4*>(src + (size_t)(tid + 512 * q) * 8);
  };
  auto put_chunk = [&](int i) {
    uint16_t* dst = buf1 + (i & 1) * 64 * P;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int p = tid + 512 * q;
      *reinterpret_cast<u4*>(dst + (p >> 5) * P + (p & 31) * 8) = wc[i & 1][q];
    }
  };
  fetch_chunk(0);
  fetch_chunk(1);
  {
    // delta of the last hidden layer: W_out^T dz (K = 4 outputs padded to 16)
    bf16x8 w = {};
    if (hf == 0) {
      const uint16_t* wo = W + layer_param_off(H, kLayers) + 32 * wave + n;
#pragma unroll
      for (int c = 0; c < kOut; ++c) w[c] = __builtin_bit_cast(__bf16, wo[(size_t)c * H]);
    }
    f32x16 acc[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      bf16x8 d = {};
      if (hf == 0) {
        const bf16x4 d4 = *reinterpret_cast<const bf16x4*>(smem + L.dz_off + (32 * s + n) * kOut * 2);
#pragma unroll
        for (int c = 0; c < kOut; ++c) d[c] = d4[c];
      }
      acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, d, zero, 0, 0, 0);
    }
    put_delta(acc, kLayers - 1);
  }
  // (buf1, the last activations, has been read: by the output layer and store_rows, before the
  // barriers above)
  put_chunk(0);
  __syncthreads();
#pragma unroll
  for (int l = kLayers - 1; l > 0; --l) {
    f32x16 acc[4] = {zero, zero, zero, zero};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = 4 * (kLayers - 1 - l) + c;
      if (i + 2 < kChunks) fetch_chunk(i + 2);
      const uint16_t* wt = buf1 + (i & 1) * 64 * P;
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) {
        const bf16x8 w = tr_operand<P>(wt, 16 * kc, 32 * wave, lane);
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              w, *reinterpret_cast<const bf16x8*>(D + (32 * s + n) * P + 64 * c + 16 * kc + 8 * hf), acc[s], 0, 0, 0);
      }
      if (c == 0) store_rows(D, gen_delta_out(g, l));  // the layer's own deltas, for its weight gradient
      if (i + 1 < kChunks) put_chunk(i + 1);
      __syncthreads();  // (after the last chunk: the deltas have been read)
    }
    put_delta(acc, l - 1);
    __syncthreads();
  }
  store_rows(D, gen_delta_out(g, 0));
}

hipError_t launch_generic(int mode, const GenArgs& g_in, int tiles_bound, int blocks_bound, int work_bound,
                          hipStream_t s) {
  GenArgs g = g_in;
  g.delta_elems = g.layer_elems;
  if (tiles_bound <= 0 || g.a.n_objects <= 0) return hipSuccess;
  if (!generic_width(g.H) || g.a.S < 1 || g.a.S > kSlots || blocks_bound <= 0 || work_bound <= 0 ||
      g.work_rays < 1)
    return hipErrorInvalidValue;
  // the wide products read W from the BF16 parameter copy
  if (keeps_gimg(g.H) && !g.a.gimg) return hipErrorInvalidValue;
  const bool train = (mode == MODE_TRAIN);
  const int H = g.H;
  const int wave_blocks = (tiles_bound + 3) / 4;
  auto blocks = [](int n, int t) { return (n + t - 1) / t; };
  // a product whose output columns number at least 128 takes 128 x 128 blocks over 128-row blocks;
  // narrower ones 64 x 64 blocks over the row tiles
  // one-dimensional grids of 8 ceil(units / 8) x blocks-per-unit workgroups (xcd_unit_block)
  auto grid1 = [&](int units, int nblk) { return dim3((unsigned)(8 * blocks(units, 8) * nblk)); };
  const int nw = H / 256;
  const bool wide = g.block_rows == kGenBlockRows;
  constexpr int kHalves = kGenBlockRows / kGenHalfRows;
  const int halves_bound = (wide ? kHalves : 1) * blocks_bound;
  // Weight gradients take k_gen_wide from 256 workgroups: hidden 512, objects of 1,200 rows, wide against
  // 128, steps in us: 8 objects (192 workgroups) 262 / 255, 16 (384) 367 / 370; hidden 256, 50 objects 318 /
  // 318, of 4,800 rows 941 / 980, 16 of 1,200 164 / 151. At hidden 1024 always: the 128 x 128 blocks of one
  // object all run on one XCD (1 object 263 / 306, 4 368 / 407, 16 1021 / 1059).
  const bool wide_dw = (nw >= 4 || (long long)work_bound * nw * nw * (kLayers - 1) >= kCUs);
  auto fwd_dx = [&](int kind, int ncols, int l) {
    if (wide && l > 0 && l < kLayers) {
      if (kind == GEN_FWD) hipLaunchKernelGGL(k_gen_wide<GEN_FWD>, grid1(blocks_bound, nw), dim3(512), 0, s, g, l);
      else hipLaunchKernelGGL(k_gen_wide<GEN_DX>, grid1(blocks_bound, nw), dim3(512), 0, s, g, l);
    } else if (ncols >= 128) {
      const int nb = blocks(ncols, 128);
      if (kind == GEN_FWD) hipLaunchKernelGGL((k_gen_gemm<GEN_FWD, 128>), grid1(halves_bound, nb), dim3(256), 0, s, g, l, nb);
      else hipLaunchKernelGGL((k_gen_gemm<GEN_DX, 128>), grid1(halves_bound, nb), dim3(256), 0, s, g, l, nb);
    } else {
      const int nb = blocks(ncols, 64);
      if (kind == GEN_FWD) hipLaunchKernelGGL((k_gen_gemm<GEN_FWD, 64>), grid1(tiles_bound, nb), dim3(256), 0, s, g, l, nb);
      else hipLaunchKernelGGL((k_gen_gemm<GEN_DX, 64>), grid1(tiles_bound, nb), dim3(256), 0, s, g, l, nb);
    }
  };
  const int nloss = blocks(g.a.n_objects, 4);
  const int dw_blocks = blocks(H, 128) * blocks(H, 128);  // 128 x 128 blocks of a square layer
  // every layer's weight gradients, from the deltas of all layers, and the losses; square = false: those
  // of the square layers have been launched
  auto launch_dw = [&](bool square) {
    if (wide_dw && square) hipLaunchKernelGGL(k_gen_wide<GEN_DW>, grid1(work_bound * (kLayers - 1), nw * nw), dim3(512), 0, s, g, 0);
    const int nb0 = blocks(H, 64) * blocks(kEnc, 64), nb1 = wide_dw || !square ? 0 : dw_blocks * (kLayers - 1);
    const int n0 = (int)grid1(work_bound, nb0).x, n1 = (int)grid1(work_bound, nb1).x;
    hipLaunchKernelGGL(k_gen_dw, dim3(n0 + n1 + nloss), dim3(256), 0, s, g, n0, nb0, n1, nb1);
    hipLaunchKernelGGL(k_gen_dw_small, grid1(work_bound, blocks(H, 32)), dim3(kGenDwWaves * 64), 0, s, g, blocks(H, 32));
  };
  if (g.chain) {
    if (!gen_chain(H) || (train && g.deltas != kLayers)) return hipErrorInvalidValue;
    static int allowed[2] = {0, 0};
    const void* fn = train ? reinterpret_cast<const void*>(k_gen_chain<true>) : reinterpret_cast<const void*>(k_gen_chain<false>);
    const hipError_t e = allow_lds(fn, lds_chain().total, &allowed[train]);
    if (e != hipSuccess) return e;
    // pairs of row tiles: at most half of them and one per object
    const dim3 grid = grid1((tiles_bound + g.a.n_objects) / 2 + 1, 1);
    if (train) hipLaunchKernelGGL(k_gen_chain<true>, grid, dim3(512), lds_chain().total, s, g);
    else hipLaunchKernelGGL(k_gen_chain<false>, grid, dim3(512), lds_chain().total, s, g);
    if (train) launch_dw(true);
    else hipLaunchKernelGGL(k_gen_loss, dim3(nloss), dim3(256), 0, s, g);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_gen_encode, dim3(wave_blocks), dim3(256), 0, s, g);
  for (int l = 0; l <= kLayers; ++l) fwd_dx(GEN_FWD, (l == kLayers) ? kOut : H, l);
  if (train) hipLaunchKernelGGL(k_gen_render<true>, dim3(wave_blocks), dim3(256), 0, s, g);
  else hipLaunchKernelGGL(k_gen_render<false>, dim3(wave_blocks), dim3(256), 0, s, g);
  if (!train) hipLaunchKernelGGL(k_gen_loss, dim3(nloss), dim3(256), 0, s, g);
  if (train) {
    // two buffers in turn: the deltas of layer m's outputs lie in buffer m mod 2, so that an input
    // gradient writes those of layer l - 1's over those of l + 1's, whose weight gradient has run
    const bool turns = g.deltas != kLayers;
    for (int l = kLayers; l > 0; --l) {
      if (turns) {  // buffers of m = l and l - 1
        g.delta_elems = (l & 1) || l == kLayers ? g.layer_elems : -g.layer_elems;
        g.delta = g_in.delta + ((l - 1) & 1) * g.layer_elems - (l - 1) * g.delta_elems;
      }
      fwd_dx(GEN_DX, H, l);
      if (turns && l > 1)
        hipLaunchKernelGGL(k_gen_dw_layer, grid1(work_bound, dw_blocks), dim3(256), 0, s, g, l - 1, dw_blocks);
    }
    launch_dw(!turns);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Scratch of the allocation-free scene render: one array per GPU, held until the process ends,
// shared by every call on that GPU. Host code never passes the array's name to a kernel (on the
// host it is only a stand-in for the symbol); it uses the device address that
// hipGetSymbolAddress returned for the GPU, looked up once per GPU with that GPU current.
static __device__ __align__(256) unsigned char scratch[kStaticSceneScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

hipError_t static_scratch_init(int device) {
  if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[device]) return hipSuccess;
  int current = -1;
  hipError_t e = hipGetDevice(&current);
  if (e != hipSuccess) return e;
  if (current != device) return hipErrorInvalidDevice;  // the caller makes `device` current
  void* ptr = nullptr;
  e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!ptr) return hipErrorInvalidSymbol;
  g_scratch_ptr[device] = ptr;
  return hipSuccess;
}

void* static_scratch(int device) {
  if (device < 0 || device >= kMaxScratchDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  return g_scratch_ptr[device];
}

}  // namespace vmapi
