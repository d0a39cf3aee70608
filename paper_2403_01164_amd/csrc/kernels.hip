// gfx950 kernels of the heterogeneous Linear: the GPU-share GEMV and the small
// glue kernels around it.
//
// GEMV (HeteGen Sec. 4.2: the GPU computes its share of the module's output
// once its weight rows are in device memory).  At batch 1..8 a linear reads each
// weight element once and does 2B flops on it, i.e. B flop per byte of fp16/bf16
// weight: far below the ridge point of the vector ALUs, so the kernel is bound by
// HBM bandwidth and uses no matrix cores.  Design of the main kernel:
//  * a workgroup (4 wavefronts) owns a contiguous block of output rows; a
//    wavefront takes R rows at a time and walks them in "tasks" of 64*U 16-byte
//    chunks per row: a lane loads 16 bytes (8 elements) of each row per step, so
//    one load instruction reads 1 KiB of a row, fully coalesced, and U*R loads per
//    lane are in flight;
//  * the loads of the next task are issued before the current task is computed
//    (two register buffers), so a wavefront never waits on an empty memory pipe,
//    and the weights of the first task are requested before the prologue;
//  * weight loads are non-temporal: the weights are read once per step and should
//    not evict x or the outputs from the caches;
//  * x [B, K] is staged once per workgroup in LDS (and normalised there when a
//    LayerNorm is fused) and read with ds_read_b128, reused for the R rows;
//  * products accumulate in binary32 through v_dot2 (fp16 pairs or bf16 pairs);
//  * the 64 lane partials of each (row, batch) pair are summed with DPP row
//    permutations and four readlanes;
//  * bias and residual of the block are staged in LDS in the prologue, outputs are
//    gathered in LDS and stored per block with contiguous stores; the epilogue adds
//    the bias, applies ReLU or a residual sum and rounds to the activation type (or
//    stores binary32), so the decode step needs no elementwise kernels.
// x may use the device's whole LDS per workgroup (160 KiB on gfx950, opted in above the
// default 64 KiB, with the grid capped at the workgroups that fit at once); when it
// does not fit even so (large B*K), a K-tiled variant restages x per tile.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "kernels.h"

namespace hg {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kX1MaxRows = 64;  // rows per wavefront the x-direct GEMV keeps bias/residual for
constexpr float kLnEps = 1e-5f;

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Global-memory view of a pointer.  Pointers read from a device-side table are
// generic to the compiler; generic (flat) loads also count against the LDS
// counter, so every LDS wait would drain the weight stream.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* gmem(const T* p) {
  return (const __attribute__((address_space(1))) T*)p;
}

// Cached 16-byte global load.
__device__ __forceinline__ uint4 load_g16(const uint4* p) {
  u32x4 v = *gmem((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Streaming 16-byte weight load (read once: marked non-temporal).
__device__ __forceinline__ uint4 load_stream(const uint4* p) {
  u32x4 v = __builtin_nontemporal_load(gmem((const u32x4*)p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

struct F16 {
  static constexpr bool kRowsTree = false;  // gemv_rows_kernel
  static __device__ __forceinline__ float dot2(uint32_t w, uint32_t x, float acc) {
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w), __builtin_bit_cast(f16x2, x), acc, false);
  }
  static __device__ __forceinline__ float lo(uint32_t v) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(v & 0xFFFFu));
  }
  static __device__ __forceinline__ float hi(uint32_t v) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(v >> 16));
  }
  static __device__ __forceinline__ float to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
  static __device__ __forceinline__ uint16_t from_f32(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }
};

struct BF16 {
  static constexpr bool kRowsTree = true;
  static __device__ __forceinline__ float dot2(uint32_t w, uint32_t x, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, x), acc,
                                           false);
  }
  static __device__ __forceinline__ float lo(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
  static __device__ __forceinline__ float hi(uint32_t v) { return __builtin_bit_cast(float, v & 0xFFFF0000u); }
  static __device__ __forceinline__ float to_f32(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }
  static __device__ __forceinline__ uint16_t from_f32(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
};

template <class T>
__device__ __forceinline__ float dot8(const uint4& w, const uint4& x, float acc) {
  acc = T::dot2(w.x, x.x, acc);
  acc = T::dot2(w.y, x.y, acc);
  acc = T::dot2(w.z, x.z, acc);
  acc = T::dot2(w.w, x.w, acc);
  return acc;
}

template <class T>
__device__ __forceinline__ void unpack8(const uint4& v, float* f) {
  f[0] = T::lo(v.x); f[1] = T::hi(v.x); f[2] = T::lo(v.y); f[3] = T::hi(v.y);
  f[4] = T::lo(v.z); f[5] = T::hi(v.z); f[6] = T::lo(v.w); f[7] = T::hi(v.w);
}

template <class T>
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return (uint32_t)T::from_f32(a) | ((uint32_t)T::from_f32(b) << 16);
}

// Sum over the 64 lanes of a wavefront; every lane returns the total.
__device__ __forceinline__ float wave_sum(float v) {
  int iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0xB1, 0xF, 0xF, false));  // quad_perm 1,0,3,2
  iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x4E, 0xF, 0xF, false));  // quad_perm 2,3,0,1
  iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x141, 0xF, 0xF, false)); // row_half_mirror
  iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x140, 0xF, 0xF, false)); // row_mirror
  iv = __builtin_bit_cast(int, v);
  // each 16-lane row now holds its row sum in every lane
  float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 0));
  float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 16));
  float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 32));
  float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 48));
  return (r0 + r1) + (r2 + r3);
}

// Sum over each row of 16 lanes (lanes 16 r .. 16 r + 15); every lane of the row returns
// its row's total, formed in a fixed order.
__device__ __forceinline__ float row16_sum(float v) {
  int iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0xB1, 0xF, 0xF, false));  // quad_perm 1,0,3,2
  iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x4E, 0xF, 0xF, false));  // quad_perm 2,3,0,1
  iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x141, 0xF, 0xF, false)); // row_half_mirror
  iv = __builtin_bit_cast(int, v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, iv, 0x140, 0xF, 0xF, false)); // row_mirror
  return v;
}

// LayerNorm statistics of B rows of x (16-byte chunk c of row b read by get(b, c))
// for one 256-thread workgroup, two passes (mean, then the mean of squared
// deviations).  Chunk c is always summed by thread c % 256 in increasing c and the
// partials are combined in a fixed tree, so every workgroup of every kernel that
// calls this gets bit-identical statistics, whether x is read from global memory
// or from LDS.
template <class T, int B, class Get>
__device__ __forceinline__ void ln_stats(Get get, int K, float* mean, float* rstd, float (*red)[8][kWaves]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n8 = K >> 3;
  // the B rows are read side by side (B loads in flight per chunk); each row's
  // partial still adds its chunks in increasing c
  float s[B];
#pragma unroll
  for (int b = 0; b < B; ++b) s[b] = 0.f;
#pragma unroll 2
  for (int c = tid; c < n8; c += kThreads) {
    uint4 v[B];
#pragma unroll
    for (int b = 0; b < B; ++b) v[b] = get(b, c);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      float f[8];
      unpack8<T>(v[b], f);
      s[b] += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
    }
  }
#pragma unroll
  for (int b = 0; b < B; ++b) s[b] = wave_sum(s[b]);
  if (lane == 0)
#pragma unroll
    for (int b = 0; b < B; ++b) red[0][b][wave] = s[b];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < B; ++b) {
    mean[b] = ((red[0][b][0] + red[0][b][1]) + (red[0][b][2] + red[0][b][3])) / (float)K;
    s[b] = 0.f;
  }
#pragma unroll 2
  for (int c = tid; c < n8; c += kThreads) {
    uint4 v[B];
#pragma unroll
    for (int b = 0; b < B; ++b) v[b] = get(b, c);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      float f[8];
      unpack8<T>(v[b], f);
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float d = f[e] - mean[b];
        acc += d * d;
      }
      s[b] += acc;
    }
  }
#pragma unroll
  for (int b = 0; b < B; ++b) s[b] = wave_sum(s[b]);
  if (lane == 0)
#pragma unroll
    for (int b = 0; b < B; ++b) red[1][b][wave] = s[b];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < B; ++b) {
    float var = ((red[1][b][0] + red[1][b][1]) + (red[1][b][2] + red[1][b][3])) / (float)K;
    rstd[b] = 1.0f / sqrtf(var + kLnEps);
  }
}

template <class T>
__device__ __forceinline__ uint4 normalize8(const uint4& v, float mean, float rstd) {
  float f[8];
  unpack8<T>(v, f);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    f[e] = (f[e] - mean) * rstd;
    // the binary32 value is materialised before it is rounded to the activation type:
    // otherwise instruction selection may fold the scaling into a mixed-precision
    // multiply-add that rounds once to 16 bits, and results at ties would depend on
    // the surrounding code (the kernels that fuse this must agree bit for bit)
    asm volatile("" : "+v"(f[e]));
  }
  uint4 o;
  o.x = pack2<T>(f[0], f[1]);
  o.y = pack2<T>(f[2], f[3]);
  o.z = pack2<T>(f[4], f[5]);
  o.w = pack2<T>(f[6], f[7]);
  return o;
}

// ReLU or residual sum on a binary32 value (bias already added).
__device__ __forceinline__ float apply_epi(float v, int epi, float resid) {
  if (epi == EPI_RELU) return fmaxf(v, 0.f);
  if (epi == EPI_RESID) return v + resid;
  return v;
}

// A binary32 result rounded to the activation type.  The value is materialised first
// so that it is rounded once from binary32 in every kernel (instruction selection
// could otherwise fold the last add into a mixed-precision operation that rounds
// straight to 16 bits, which differs at ties).
template <class T>
__device__ __forceinline__ uint16_t round_act(float v) {
  asm volatile("" : "+v"(v));
  return T::from_f32(v);
}

template <class T>
__device__ __forceinline__ void store_y(void* y, long long i, int y_f32, float v) {
  if (y_f32) ((float*)y)[i] = v;
  else ((uint16_t*)y)[i] = round_act<T>(v);
}

// ---------------------------------------------------------------------------
// Coherent accesses for data produced by other workgroups of the same kernel
// (the persistent decode step): buffer loads/stores with sc0 sc1, which bypass
// the non-coherent cache levels, so no L2 writeback/invalidate is needed between
// linears.  Word 3 of the buffer descriptor is the gfx9 raw-buffer format.
// ---------------------------------------------------------------------------
constexpr int kBufWord3 = 0x00020000;
constexpr int kCoherent = 1 | 16;  // sc0 | sc1
constexpr uint32_t kXPast = 0x80000000u;  // a buffer offset past every descriptor the GEMVs build

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, kBufWord3);
}

// The descriptor base must be wave-uniform (it lives in scalar registers): pass
// the row base and a per-lane byte offset; `bytes` bounds the row.
template <bool COH>
__device__ __forceinline__ uint4 load_act16(const uint16_t* row, uint32_t bytes, uint32_t off) {
  if (COH) {
    u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc(row, bytes), (int)off, 0, kCoherent);
    return make_uint4(v.x, v.y, v.z, v.w);
  }
  return *(const uint4*)((const char*)row + off);
}

template <bool COH>
__device__ __forceinline__ uint16_t load_act1(const uint16_t* row, uint32_t bytes, uint32_t off) {
  if (COH) return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsrc(row, bytes), (int)off, 0, kCoherent);
  return *(const uint16_t*)((const char*)row + off);
}

// y row base (wave-uniform) and element index within the row.
template <class T, bool COH>
__device__ __forceinline__ void store_y_c(void* yrow, uint32_t n, uint32_t i, int y_f32, float v) {
  if (COH) {
    if (y_f32)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rsrc(yrow, n * 4), (int)(i * 4), 0,
                                            kCoherent);
    else
      __builtin_amdgcn_raw_buffer_store_b16(round_act<T>(v), rsrc(yrow, n * 2), (int)(i * 2), 0, kCoherent);
    return;
  }
  store_y<T>(yrow, i, y_f32, v);
}

// 16-byte group col of row `row` in the segment-major layout of a [rows, K] weight.
__device__ __forceinline__ const uint4* seg_addr(const uint4* W, int rows, int row, int col) {
  constexpr int G = kSegElems / 8;  // 16-byte groups per segment
  return W + ((long long)(col / G) * rows + row) * G + (col % G);
}

// ---------------------------------------------------------------------------
// Main GEMV, one workgroup's block of rows (x fits in LDS).  Dynamic LDS layout:
//   xs [B][K/8] uint4 | bias [rpw] f32 | resid [B][rpw] f32 | out [B][rpw] f32
// The first task of every wavefront is requested before `wait()` and the
// prologue, so its weights stream in while the block waits for its inputs.
// ---------------------------------------------------------------------------
template <class T, int B, int R, int U, bool COH_LOAD, bool COH_STORE, class Wait>
__device__ __forceinline__ void gemv_block(const GemvParams& p, int blk, uint4* smem, float (*red)[8][kWaves],
                                           Wait wait) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = p.K, k8 = K >> 3, rpw = p.rpw;
  uint4* xs = smem;
  float* sb = (float*)(smem + (size_t)B * k8);
  float* sr = sb + rpw;
  float* sy = sr + B * rpw;
  const int row_begin = blk * rpw;
  const int nrows = max(0, min(rpw, p.rows - row_begin));
  constexpr int SEG = 64 * U;  // 16-byte chunks per task and row
  const int nseg = (k8 + SEG - 1) / SEG;
  const int nrg = (nrows + R - 1) / R;
  const int my_rg = nrg > wave ? (nrg - wave + kWaves - 1) / kWaves : 0;
  const int ntask = my_rg * nseg;
  const uint16_t* W = (const uint16_t*)p.W;

  // task t of this wavefront: row group j = t / nseg (local rows (wave + j*kWaves)*R ..), segment t % nseg
  auto load = [&](int t, uint4 (&w)[U][R]) {
    const int j = t / nseg, seg = t - j * nseg;
    const int lr0 = (wave + j * kWaves) * R;
    const int c0 = seg * SEG + lane;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = row_begin + min(lr0 + r, nrows - 1);
      const uint4* wr = (const uint4*)(W + (long long)row * K);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // unconditional load (clamped address): no branch, so the compiler can keep
        // later tasks' loads in flight; lanes past the row end reread its last
        // chunk (same cache line, no extra traffic) and skip it in compute()
        const int col = min(c0 + 64 * u, k8 - 1);
        w[u][r] = load_stream(p.segmajor ? seg_addr((const uint4*)W, p.rows, row, col) : wr + col);
      }
    }
  };
  auto compute = [&](int t, const uint4 (&w)[U][R], float (&acc)[R][B]) {
    const int j = t / nseg, seg = t - j * nseg;
    const int c0 = seg * SEG + lane;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + 64 * u;
      if (c < k8) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
          const uint4 xv = xs[b * k8 + c];
#pragma unroll
          for (int r = 0; r < R; ++r) acc[r][b] = dot8<T>(w[u][r], xv, acc[r][b]);
        }
      }
    }
    if (seg == nseg - 1) {  // row group complete: reduce and finish into LDS
      const int lr0 = (wave + j * kWaves) * R;
#pragma unroll
      for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
          const float s = wave_sum(acc[r][b]);
          acc[r][b] = 0.f;
          const int lr = lr0 + r;
          if (lane == 0 && lr < nrows) sy[b * rpw + lr] = apply_epi(s + sb[lr], p.epi, sr[b * rpw + lr]);
        }
      }
    }
  };

  uint4 wa[U][R], wb[U][R];
  float acc[R][B];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int b = 0; b < B; ++b) acc[r][b] = 0.f;
  if (ntask > 0) load(0, wa);

  wait();

  // prologue: x, bias and residual of the block into LDS
  {
    const uint16_t* x = (const uint16_t*)p.x;
#pragma unroll 2
    for (int c = tid; c < k8; c += kThreads) {
      uint4 v[B];
#pragma unroll
      for (int b = 0; b < B; ++b) v[b] = load_act16<COH_LOAD>(x + b * p.ldx, (uint32_t)K * 2, (uint32_t)c * 16);
#pragma unroll
      for (int b = 0; b < B; ++b) xs[b * k8 + c] = v[b];
    }
    const uint16_t* bias = (const uint16_t*)p.bias;
    for (int i = tid; i < nrows; i += kThreads) sb[i] = bias ? T::to_f32(gmem(bias)[row_begin + i]) : 0.f;
    if (p.epi == EPI_RESID) {
      const uint16_t* res = (const uint16_t*)p.resid;
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const uint16_t* rrow = res + b * p.ldr + row_begin;
        for (int lr = tid; lr < nrows; lr += kThreads)
          sr[b * rpw + lr] = T::to_f32(load_act1<COH_LOAD>(rrow, (uint32_t)nrows * 2, (uint32_t)lr * 2));
      }
    }
    __syncthreads();
    if (p.ln) {
      float mean[B], rstd[B];
      ln_stats<T, B>([&](int b, int c) { return xs[b * k8 + c]; }, K, mean, rstd, red);
      const bool write_h = p.h_out != nullptr && blk == 0;
      for (int c = tid; c < k8; c += kThreads) {  // each thread rewrites only the chunks it summed
#pragma unroll
        for (int b = 0; b < B; ++b) {
          const uint4 v = normalize8<T>(xs[b * k8 + c], mean[b], rstd[b]);
          xs[b * k8 + c] = v;
          if (write_h) *(uint4*)((uint16_t*)p.h_out + b * p.ldh + (long long)c * 8) = v;
        }
      }
      __syncthreads();
    }
  }

  // main loop, two register buffers: loads of task t+1 are in flight while t is
  // computed.  The loop body issues its loads unconditionally; the last one or two
  // tasks are peeled.
  int t = 0;
  for (; t + 2 < ntask; t += 2) {
    load(t + 1, wb);
    compute(t, wa, acc);
    load(t + 2, wa);
    compute(t + 1, wb, acc);
  }
  if (t + 1 < ntask) {
    load(t + 1, wb);
    compute(t, wa, acc);
    compute(t + 1, wb, acc);
  } else if (t < ntask) {
    compute(t, wa, acc);
  }

  // block outputs: contiguous stores
  __syncthreads();
  const size_t ys = p.y_f32 ? 4 : 2;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    void* yrow = (char*)p.y + ((size_t)b * p.ldy + row_begin) * ys;
    for (int lr = tid; lr < nrows; lr += kThreads)
      store_y_c<T, COH_STORE>(yrow, (uint32_t)nrows, (uint32_t)lr, p.y_f32, sy[b * rpw + lr]);
  }
}

template <class T, int B, int R, int U>
__global__ __launch_bounds__(kThreads) void gemv_kernel(GemvParams p) {
  extern __shared__ uint4 smem[];
  __shared__ float red[2][8][kWaves];
  gemv_block<T, B, R, U, false, false>(p, blockIdx.x, smem, red, [] {});
}

// ---------------------------------------------------------------------------
// GEMV of NB <= 2 batch rows without a fused LayerNorm: x is read straight from
// L1/L2 inside the task loop (it is the same NB*2*K bytes for every wavefront, so
// it stays cached), which removes the LDS prologue and its barrier; the bias and residual
// of a wavefront's rows are loaded once, ahead of its weight stream, into that
// wavefront's slice of LDS, and lane 0 stores each finished row.  Each
// lane accumulates its chunks in the same order as gemv_block, so both kernels
// give bit-identical results.
// ---------------------------------------------------------------------------
template <class T, int U, int NB>
__global__ __launch_bounds__(kThreads) void gemv_x1_kernel(GemvParams p) {
  // per wavefront: bias and residual of its rows (row j of the wave: local row wave + j*kWaves)
  __shared__ float sbias[kWaves][kX1MaxRows], sres[kWaves][NB][kX1MaxRows];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int K = p.K, k8 = K >> 3, rpw = p.rpw;
  const int row_begin = blockIdx.x * rpw;
  const int nrows = min(rpw, p.rows - row_begin);  // >= 1: the grid covers rows exactly
  constexpr int SEG = 64 * U;
  static_assert(SEG * 8 == kSegElems, "a request segment is one segment of the segment-major layout");
  const int nseg = (k8 + SEG - 1) / SEG;
  const int my_rg = nrows > wave ? (nrows - wave + kWaves - 1) / kWaves : 0;  // <= kX1MaxRows (launcher)
  const int ntask = my_rg * nseg;
  const uint16_t* W = (const uint16_t*)p.W;
  const uint16_t* bias = (const uint16_t*)p.bias;
  const uint16_t* res = (const uint16_t*)p.resid;
  // bias and residual first: waiting for them later does not wait for the weights
  float bj = 0.f, rj[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) rj[b] = 0.f;
  if (lane < my_rg) {
    const int row = row_begin + wave + lane * kWaves;
    if (bias) bj = T::to_f32(gmem(bias)[row]);
    if (p.epi == EPI_RESID)
#pragma unroll
      for (int b = 0; b < NB; ++b) rj[b] = T::to_f32(gmem(res)[(long long)b * p.ldr + row]);
  }
  struct Buf {
    uint4 w[U], x[NB][U];
  };
  auto load = [&](int t, Buf& f) {
    const int j = t / nseg, seg = t - j * nseg;
    const int row = row_begin + wave + j * kWaves;
    // segment-major: segment seg of this row at (seg * rows + row) * SEG 16-byte groups
    const uint4* wr = p.segmajor ? (const uint4*)W + ((long long)seg * p.rows + row) * SEG - (long long)seg * SEG
                                 : (const uint4*)(W + (long long)row * K);
    const int c0 = seg * SEG + lane;
#pragma unroll
    for (int u = 0; u < U; ++u) f.w[u] = load_stream(wr + min(c0 + 64 * u, k8 - 1));
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const uint4* xb = (const uint4*)((const uint16_t*)p.x + (long long)b * p.ldx);
#pragma unroll
      for (int u = 0; u < U; ++u) f.x[b][u] = load_g16(xb + min(c0 + 64 * u, k8 - 1));
    }
  };
  Buf fa, fb;
  if (ntask > 0) load(0, fa);
  if (lane < my_rg) {
    sbias[wave][lane] = bj;
#pragma unroll
    for (int b = 0; b < NB; ++b) sres[wave][b][lane] = rj[b];
  }
  float acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = 0.f;
  auto compute = [&](int t, const Buf& f) {
    const int j = t / nseg, seg = t - j * nseg;
    const int c0 = seg * SEG + lane;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c0 + 64 * u < k8)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = dot8<T>(f.w[u], f.x[b][u], acc[b]);
    if (seg == nseg - 1) {
      const int row = row_begin + wave + j * kWaves;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float s = wave_sum(acc[b]);
        acc[b] = 0.f;
        if (lane == 0)
          store_y<T>(p.y, (long long)b * p.ldy + row, p.y_f32, apply_epi(s + sbias[wave][j], p.epi, sres[wave][b][j]));
      }
    }
  };
  int t = 0;
  for (; t + 2 < ntask; t += 2) {
    load(t + 1, fb);
    compute(t, fa);
    load(t + 2, fa);
    compute(t + 1, fb);
  }
  if (t + 1 < ntask) {
    load(t + 1, fb);
    compute(t, fa);
    compute(t + 1, fb);
  } else if (t < ntask) {
    compute(t, fa);
  }
}

// ---------------------------------------------------------------------------
// Batch-1 GEMV with a fused LayerNorm for K <= 512 * NC (NC <= 14): every wavefront
// loads the whole input row into registers (lane l holds the 16-byte chunks
// l + 64u, exactly the chunks it multiplies in every row), normalises it there and
// keeps it for all its rows: no LDS staging and no workgroup barrier.  When K is not a
// multiple of 512 (TAIL) lanes past the row's end in the last chunk reread the row's last chunk of
// the input and of the weights and leave both out of their sums: such widths ran on the
// LDS kernel, whole batch-1 steps (us): H = 520, 12 layers 200.6 -> 167.7; 1544, 8 layers 199.9 ->
// 179.0; 4104, 2 layers 182.5 -> 164.4; 7000, 1 layer 200.9 -> 196.7.  The
// statistics are summed in the order of ln_stats and the products in the order of
// gemv_block, so the result is bit-identical to the workgroup kernels.
// ---------------------------------------------------------------------------
template <class T, int NC, bool TAIL>
__device__ __forceinline__ void ln_stats_wave(const uint4 (&xv)[NC], int K, bool in, float& mean, float& rstd) {
  // "thread" t = 64 w + l of ln_stats sums chunks t + 256 i, i.e. chunks u = w + 4 i of lane l
  float part[kWaves];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    float s = 0.f;
#pragma unroll
    for (int u = w; u < NC; u += kWaves) {
      float f[8];
      unpack8<T>(xv[u], f);
      const float c = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
      s = TAIL && u == NC - 1 && !in ? s : s + c;
    }
    part[w] = wave_sum(s);
  }
  mean = ((part[0] + part[1]) + (part[2] + part[3])) / (float)K;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    float s = 0.f;
#pragma unroll
    for (int u = w; u < NC; u += kWaves) {
      float f[8];
      unpack8<T>(xv[u], f);
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float d = f[e] - mean;
        acc += d * d;
      }
      s = TAIL && u == NC - 1 && !in ? s : s + acc;
    }
    part[w] = wave_sum(s);
  }
  const float var = ((part[0] + part[1]) + (part[2] + part[3])) / (float)K;
  rstd = 1.0f / sqrtf(var + kLnEps);
}

template <class T, int NC, bool TAIL>
__global__ __launch_bounds__(kThreads) void gemv_ln1_kernel(GemvParams p) {
  __shared__ float sbias[kWaves][kX1MaxRows], sres[kWaves][kX1MaxRows];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int K = p.K, rpw = p.rpw;  // 512 (NC - 1) < K <= 512 NC, TAIL: K < 512 NC (launcher)
  const bool in = !TAIL || lane + 64 * (NC - 1) < (K >> 3);  // this lane's last chunk is inside the row
  const int last = TAIL ? min(lane + 64 * (NC - 1), (K >> 3) - 1) : lane + 64 * (NC - 1);
  const int row_begin = blockIdx.x * rpw;
  const int nrows = min(rpw, p.rows - row_begin);  // >= 1: the grid covers rows exactly
  const int my_rg = nrows > wave ? (nrows - wave + kWaves - 1) / kWaves : 0;  // <= kX1MaxRows (launcher)
  const uint16_t* W = (const uint16_t*)p.W;
  const uint16_t* bias = (const uint16_t*)p.bias;
  const uint16_t* res = (const uint16_t*)p.resid;
  float bj = 0.f, rj = 0.f;
  if (lane < my_rg) {
    const int row = row_begin + wave + lane * kWaves;
    if (bias) bj = T::to_f32(gmem(bias)[row]);
    if (p.epi == EPI_RESID) rj = T::to_f32(gmem(res)[row]);
  }
  auto load = [&](int j, uint4 (&w)[NC]) {
    const uint4* wr = (const uint4*)(W + (long long)(row_begin + wave + j * kWaves) * K);
#pragma unroll
    for (int u = 0; u < NC; ++u) w[u] = load_stream(wr + (u == NC - 1 ? last : lane + 64 * u));
  };
  uint4 wa[NC], wb[NC], xn[NC];
  if (my_rg > 0) load(0, wa);
  const uint4* x = (const uint4*)p.x;
#pragma unroll
  for (int u = 0; u < NC; ++u) xn[u] = load_g16(x + (u == NC - 1 ? last : lane + 64 * u));
  if (lane < my_rg) {
    sbias[wave][lane] = bj;
    sres[wave][lane] = rj;
  }
  float mean, rstd;
  ln_stats_wave<T, NC, TAIL>(xn, K, in, mean, rstd);
#pragma unroll
  for (int u = 0; u < NC; ++u) xn[u] = normalize8<T>(xn[u], mean, rstd);
  if (p.h_out && blockIdx.x == 0 && wave == 0)
#pragma unroll
    for (int u = 0; u < NC; ++u)
      if (!TAIL || u < NC - 1 || in) *(uint4*)((uint16_t*)p.h_out + (long long)(lane + 64 * u) * 8) = xn[u];
  auto compute = [&](int j, const uint4 (&w)[NC]) {
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      const float d = dot8<T>(w[u], xn[u], acc);
      acc = TAIL && u == NC - 1 && !in ? acc : d;
    }
    const float s = wave_sum(acc);
    if (lane == 0)
      store_y<T>(p.y, row_begin + wave + j * kWaves, p.y_f32, apply_epi(s + sbias[wave][j], p.epi, sres[wave][j]));
  };
  int j = 0;
  for (; j + 2 < my_rg; j += 2) {
    load(j + 1, wb);
    compute(j, wa);
    load(j + 2, wa);
    compute(j + 1, wb);
  }
  if (j + 1 < my_rg) {
    load(j + 1, wb);
    compute(j, wa);
    compute(j + 1, wb);
  } else if (j < my_rg) {
    compute(j, wa);
  }
}

// ---------------------------------------------------------------------------
// Matrix-core GEMV on tile-ordered weights (batches 1..8).  A linear is a product of
// B <= 8 activation rows with N weight rows; v_mfma_f32_16x16x32 takes one 1 KiB tile
// of 16 weight rows x 32 columns as its 16-row operand (one 16-byte load per lane,
// the whole tile in one coalesced instruction) and the matching 32 columns of x as its
// 16-column operand.  The products and their fp32 sums happen in the matrix core, so no
// lane reduction is needed and the instruction cost per weight byte does not grow with B:
// the kernel stays bound by HBM at every batch size, where the vector GEMV becomes bound by
// its dot products and LDS reads of x.
//
// What it costs beyond the weights is x: B rows of it, read by every workgroup from L2
// through the same load pipeline.  One load fetches the fragments of two k-tiles (see the
// kernel), and a workgroup may hold R row tiles that share them (mfma_rows).  Against one
// fragment load per weight tile (B = 8, us): [4096, 16384] 24.1 -> 22.6, [4096, 4096] 8.8
// -> 7.9, with the LayerNorm [12288, 4096] 19.4 -> 18.3 and [15360, 5120] 30.1 -> 27.0, and
// [9216, 36864] 120 -> 105 (6.5 TB/s).
//
// Workgroup (R row tiles, split g) of 4 wavefronts takes the k-tiles of split g of its
// rows, dealt to the wavefronts in chunks of 4 (so the workgroup walks one window of K: with
// a contiguous quarter per wavefront [4096, 16384] took 24.0 us), U tiles per step with
// the next step's loads in flight.  The four partial tiles are summed in LDS in wavefront
// order.  With G > 1 splits, each workgroup stores its partial (coherent stores to
// memory: the splits run on different XCDs with their own L2) and the last of the G to
// arrive (an arrival counter, no waiting) adds the G partials in split order, so the
// result does not depend on timing.  Column order inside a tile is free (both
// operands use the same one), so every lane's x fragment is 16 contiguous bytes.  Which
// tiles are added in which order depends on K and G only: not on B, U or R.
//
// LayerNorm without a launch of its own (LN = true): the linear that produced x (out or
// fc2, this kernel with ln_out) left per-16-row partials of its output; the consumer
// combines them in its prologue, while its first weight tiles are in flight, and
// normalises each x fragment as it multiplies it (one fused multiply-add per element).
// ---------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

template <class T> struct Mma;
template <> struct Mma<F16> {
  static __device__ __forceinline__ f32x4 run(const uint4& w, const uint4& x, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), c, 0, 0,
                                                  0);
  }
};
template <> struct Mma<BF16> {
  static __device__ __forceinline__ f32x4 run(const uint4& w, const uint4& x, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0,
                                                   0, 0);
  }
};

// (x - mean) * rstd for 8 packed elements as one fused multiply-add x * a + c (a = rstd,
// c = -mean * rstd), rounded to the activation type: for fp16 a mixed-precision fma that
// reads the halves of a register and writes one half (v_fma_mix{lo,hi}_f16, 8
// instructions), for bf16 fp32 fmas and packed conversions (v_cvt_pk_bf16_f32).  A GEMV
// that normalises every x fragment it multiplies does this once per weight tile.
template <class T> struct NormFma;
template <> struct NormFma<F16> {
  static __device__ __forceinline__ uint32_t two(uint32_t w, float a, float c) {
    const f16x2 h = __builtin_bit_cast(f16x2, w);
    const f16x2 r = {(_Float16)__builtin_fmaf((float)h.x, a, c), (_Float16)__builtin_fmaf((float)h.y, a, c)};
    return __builtin_bit_cast(uint32_t, r);
  }
};
template <> struct NormFma<BF16> {
  static __device__ __forceinline__ uint32_t two(uint32_t w, float a, float c) {
    const f32x2 f = {__builtin_fmaf(__builtin_bit_cast(float, w << 16), a, c),
                     __builtin_fmaf(__builtin_bit_cast(float, w & 0xFFFF0000u), a, c)};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
  }
};
template <class T>
__device__ __forceinline__ uint4 normalize8_fma(const uint4& v, float a, float c) {
  return make_uint4(NormFma<T>::two(v.x, a, c), NormFma<T>::two(v.y, a, c), NormFma<T>::two(v.z, a, c),
                    NormFma<T>::two(v.w, a, c));
}

constexpr int kTileRows = 16, kTileK = 32;
constexpr int kChunkTiles = 4;  // k-tiles dealt to a wavefront at a time
constexpr int kShortTiles = 8;  // 2 at a time up to here
// K-split choice of the matrix-core GEMV (even_splits, splits_on)
constexpr double kMaxUneven = 1.15;  // busiest CU's workgroups over the mean, tolerated unsplit
constexpr int kMaxSplits = 8, kMinSplitTiles = 32;
constexpr int kMinTilesToSplit = 128, kLongTiles = 256;  // k-tiles of a row
constexpr double kMaxUnevenShort = 1.3;                   // below kLongTiles
constexpr int kMaxDevices = 64, kDefaultCus = 256;
constexpr int kMaxKmajorPerCu = 3;  // mfma_kmajor
// mfma_rows
constexpr int kLongSplitTiles = 128;
constexpr double kRowTilesEven = 1.05, kRowTilesUneven = 1.1;
constexpr int kSoonTiles = 20, kFullTiles = 32, kFullTilesMany = 40, kShortRowTiles = 64;  // k-tiles of a row
// gemv_rows_wanted, rows_by_8
constexpr int kRowsFew = 1024, kRowsMany = 16384;
constexpr int kRowsMinK8 = 1024, kRowsLongK = 3584;
constexpr double kRowsUneven = 1.2, kRowsLopsided = 1.4;
constexpr long long kLdsPerCu = 160 * 1024;
constexpr int kLongLnK = 4096;        // launch_mfma_t
constexpr int kLnGroup = 16;    // elements per LayerNorm partial
constexpr int kLnSlots = 8;     // batch rows per partial group (the largest batch)

// LayerNorm statistics of B rows from their partials (see ln_partials_floats): the mean
// is the sum of the group sums over K, and the variance combines each group's squared
// deviations with its count times the squared distance of its mean from the row mean
// (the pairwise combination of Chan, Golub and LeVeque), so no large sums of squares
// are subtracted.  Wavefront w owns batch rows 2w and 2w + 1 (one 16-byte load per
// group holds both rows' pairs): lane l takes groups l + 64 i in increasing i, and the
// lanes are combined in a fixed DPP tree, so every workgroup gets the same bits with no
// reduction across wavefronts; one barrier publishes the statistics.
constexpr int kLnRegGroups = 6;  // groups per lane kept in registers: K <= 6144, the widths that use partials by default

// Group i of this lane for wavefront w's rows: a lane past the last group of a round rereads
// it (the reduction drops it); slot 2w + 1 past B holds nothing the launch uses.
__device__ __forceinline__ f32x4 ln_partial(const float* __restrict__ pt, int QG, int i) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = min(lane + 64 * i, QG - 1);
  return *gmem((const f32x4*)(pt + ((size_t)q * kLnSlots + 2 * wave) * 2));
}

__device__ __forceinline__ void ln_partials_load(const float* __restrict__ pt, int K, int B,
                                                 f32x4 (&v)[kLnRegGroups]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int QG = (K + kLnGroup - 1) / kLnGroup, rounds = (QG + 63) / 64;  // the same for the workgroup
  if (2 * wave >= B || rounds > kLnRegGroups) return;
#pragma unroll
  for (int i = 0; i < kLnRegGroups; ++i)
    if (i < rounds) v[i] = ln_partial(pt, QG, i);
}

__device__ __forceinline__ void ln_partials_reduce(const float* __restrict__ pt, const f32x4 (&v)[kLnRegGroups], int K,
                                                   int B, float (*st)[2]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int QG = (K + kLnGroup - 1) / kLnGroup, rounds = (QG + 63) / 64;
  if (2 * wave < B) {
    const float inv_k = 1.0f / (float)K;
    float s0 = 0.f, s1 = 0.f, m0 = 0.f, m1 = 0.f, t0 = 0.f, t1 = 0.f;
    auto add = [&](int i, const f32x4& g) {
      if (lane + 64 * i < QG) {
        s0 += g.x;
        s1 += g.z;
      }
    };
    auto dev = [&](int i, const f32x4& g) {
      const int q = lane + 64 * i;
      if (q < QG) {
        // a group holds 16 elements, or 8 (the last one when K % 16 == 8; K % 8 == 0): its
        // mean is its sum times an exact power-of-two reciprocal
        const bool full = K - kLnGroup * q >= kLnGroup;
        const float n = full ? (float)kLnGroup : 8.f, inv_n = full ? 1.f / kLnGroup : 0.125f;
        const float d0 = g.x * inv_n - m0, d1 = g.z * inv_n - m1;
        t0 += g.y + n * d0 * d0;
        t1 += g.w + n * d1 * d1;
      }
    };
    const bool regs = rounds <= kLnRegGroups;
    if (regs) {
#pragma unroll
      for (int i = 0; i < kLnRegGroups; ++i)
        if (i < rounds) add(i, v[i]);
    } else {  // wider rows: both passes read the partials from the cache
      for (int i = 0; i < rounds; ++i) add(i, ln_partial(pt, QG, i));
    }
    m0 = wave_sum(s0) * inv_k;
    m1 = wave_sum(s1) * inv_k;
    if (regs) {
#pragma unroll
      for (int i = 0; i < kLnRegGroups; ++i)
        if (i < rounds) dev(i, v[i]);
    } else {
      for (int i = 0; i < rounds; ++i) dev(i, ln_partial(pt, QG, i));
    }
    t0 = wave_sum(t0);
    t1 = wave_sum(t1);
    if (lane == 0) {
      st[2 * wave][0] = m0;
      st[2 * wave][1] = 1.0f / sqrtf(t0 * inv_k + kLnEps);
      if (2 * wave + 1 < B) {
        st[2 * wave + 1][0] = m1;
        st[2 * wave + 1][1] = 1.0f / sqrtf(t1 * inv_k + kLnEps);
      }
    }
  }
  __syncthreads();
}

template <class T, int U, int R, bool LN>
__global__ __launch_bounds__(kThreads) void gemv_mfma_kernel(GemvParams p, int B, int G) {
  static_assert(U % kChunkTiles == 0, "a request holds whole chunks");
  constexpr int NQ = (R + 1) / 2;  // outputs per thread: 2 row tiles of 16 rows x 8 batch rows at a time
  __shared__ float part[kWaves][R][4][64];
  __shared__ float lnst[kLnSlots][2];  // LN: mean and 1 / sqrt(var + eps) of each batch row
  __shared__ int last;
  // the wavefront index through a scalar register: every tile bound below is then
  // wave-uniform and the skipped products are skipped by a branch.  A condition the
  // compiler cannot prove uniform becomes an execution mask, which matrix-core
  // instructions do not obey (they would run for every skipped tile).
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K = p.K, KT = (K + kTileK - 1) / kTileK, RT = (p.rows + kTileRows - 1) / kTileRows;
  const int rg = blockIdx.x / G, gi = blockIdx.x - rg * G, rt0 = rg * R;
  const int kg = (KT + G - 1) / G;
  const int kb = min(KT, gi * kg), kn = min(KT, kb + kg);
  // this wavefront's chunks: c = 0, 1, ... at k-tiles k0 + c * kWaves * kChunkTiles; up to
  // kShortTiles k-tiles in all are dealt in twos instead, so that no product continues another's
  // sum (in chunks of 4 the error against 64 bits at K = 128 was 1.05-1.10 of that of one tile per
  // wavefront; in twos it is 0.93-1.00 for K = 72..256, at the same time per launch)
  const bool twos = kn - kb <= kShortTiles;
  const int k0 = kb + wave * (twos ? 2 : kChunkTiles), ke = twos ? min(kn, k0 + 2) : kn;
  constexpr int kStep = kWaves * kChunkTiles;
  const int nst = ke > k0 ? ((ke - k0 + kStep - 1) / kStep * kChunkTiles + U - 1) / U : 0;
  auto ktile = [&](int st, int u) { return k0 + (st * (U / kChunkTiles) + u / kChunkTiles) * kStep + u % kChunkTiles; };
  // k-tile kt of row tile rt: tile rt * KT + kt (row-tile order) or kt * RT + rt (k-major)
  const size_t kstride = p.korder ? (size_t)RT * 64 : 64, rstride = p.korder ? 64 : (size_t)KT * 64;
  const uint4* wp[R];
#pragma unroll
  for (int r = 0; r < R; ++r) wp[r] = (const uint4*)p.W + min(rt0 + r, RT - 1) * rstride + lane;
  // x fragments, two k-tiles per load: the 16 columns of a product are batch rows 0..7 of
  // the even k-tile of the pair and batch rows 0..7 of the odd one, so the lanes of a row of
  // 16 that would hold nothing for B <= 8 fetch the next k-tile's x instead.  The even
  // tile's product is read from columns 0..7 of its accumulator, the odd tile's from columns
  // 8..15 of another one; the other halves multiply the wrong x and are dropped.  x goes
  // through a buffer descriptor over rows [0, B) of x: a lane whose batch row is past B, a
  // group past K and the tiles past the split's end get an offset past the descriptor's
  // size, for which the load returns zeros without a memory access and without a branch
  // (a branch around the loads makes the compiler wait for the weights in flight)
  const int half = (lane >> 3) & 1, grp = lane >> 4, b = min(lane & 7, B - 1);
  const auto xrs = rsrc(p.x, (uint32_t)(((long long)(B - 1) * p.ldx + K) * 2));
  const bool xlane = (lane & 7) < B;
  const uint32_t xrow = (uint32_t)((long long)b * p.ldx * 2);
  const uint32_t xlast = xrow + 2u * (half * kTileK + 8 * grp);
  const uint32_t xfull = xlane ? xlast : kXPast;
  struct Buf {
    uint4 w[R][U], x[U / 2];
  };
  // Step st < nst - 1 holds whole chunks only; the last one (and, with the LayerNorm, the
  // unconditional first one) may run past ke: its tiles past ke reread tile ke - 1 and are
  // not multiplied.
  auto load = [&](int st, Buf& f) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kt = ktile(st, u);
#pragma unroll
      for (int r = 0; r < R; ++r) f.w[r][u] = load_stream(wp[r] + kt * kstride);
      if (u % 2 == 0) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(xrs, xfull, kt * (kTileK * 2), 0);
        f.x[u / 2] = make_uint4(v.x, v.y, v.z, v.w);
      }
    }
  };
  auto load_last = [&](int st, Buf& f) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kt = ktile(st, u), ktc = min(kt, ke - 1);
#pragma unroll
      for (int r = 0; r < R; ++r) f.w[r][u] = load_stream(wp[r] + ktc * kstride);
      if (u % 2 == 0) {
        // K % 8 == 0: a group of 8 columns is wholly inside or past K
        const bool in = xlane & ((kt + half) * kTileK + 8 * grp < K) & (kt + half < ke);  // no short circuit: no branch
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(xrs, in ? xlast + 2u * kt * kTileK : kXPast, 0, 0);
        f.x[u / 2] = make_uint4(v.x, v.y, v.z, v.w);
      }
    }
  };
  // LayerNorm of x on the fly: xn = x * ln_a + ln_c for this lane's batch row
  float ln_a = 0.f, ln_c = 0.f;
  f32x4 acc[R][2];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r][0] = acc[r][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const Buf& f) {
#pragma unroll
    for (int u = 0; u < U; u += 2) {
      const uint4 xv = LN ? normalize8_fma<T>(f.x[u / 2], ln_a, ln_c) : f.x[u / 2];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        acc[r][0] = Mma<T>::run(f.w[r][u], xv, acc[r][0]);
        acc[r][1] = Mma<T>::run(f.w[r][u + 1], xv, acc[r][1]);
      }
    }
  };
  auto compute_last = [&](int st, const Buf& f) {
#pragma unroll
    for (int u = 0; u < U; u += 2) {
      const int kt = ktile(st, u);
      uint4 xv = f.x[u / 2];
      if (LN) {
        xv = normalize8_fma<T>(xv, ln_a, ln_c);
        // columns past K (only in the last k-tile when K % 32 != 0) multiply zeros
        if ((K & (kTileK - 1)) && (kt + half) * kTileK + 8 * grp >= K) xv = make_uint4(0u, 0u, 0u, 0u);
      }
      if (kt < ke) {
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r][0] = Mma<T>::run(f.w[r][u], xv, acc[r][0]);
      }
      if (kt + 1 < ke) {
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r][1] = Mma<T>::run(f.w[r][u + 1], xv, acc[r][1]);
      }
    }
  };
  // thread t finishes row i of row tiles rt0 + r0 + 2 q, q < NQ, for batch row j; its bias and
  // residual are requested ahead of the products (in the epilogue they would cost one more
  // memory round trip)
  const int t = threadIdx.x, i = t & 15, j = (t >> 4) & 7, r0 = t >> 7;
  const int row0 = (rt0 + r0) * kTileRows + i;
  auto mine = [&](int q) { return j < B && r0 + 2 * q < R; };
  auto valid = [&](int q) { return mine(q) && row0 + 2 * kTileRows * q < p.rows; };
  uint16_t bias_v[NQ], resid_v[NQ];
  auto load_epi = [&] {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int row = row0 + 2 * kTileRows * q;
      bias_v[q] = resid_v[q] = 0;
      if (valid(q) && p.bias) bias_v[q] = gmem((const uint16_t*)p.bias)[row];
      if (valid(q) && p.epi == EPI_RESID) resid_v[q] = gmem((const uint16_t*)p.resid)[j * p.ldr + row];
    }
  };
  Buf fa, fb;
  // the LayerNorm partials are requested before the first weights, so that waiting for
  // them leaves the weight loads in flight
  f32x4 lnv[LN ? kLnRegGroups : 1];
  if constexpr (LN) {
    ln_partials_load(p.ln_in, K, B, lnv);
    __builtin_amdgcn_sched_barrier(0);  // keep them ahead of the weight loads
  } else {
    load_epi();
  }
  // (with the LayerNorm the first loads are unconditional, for the same reason; a
  // wavefront without tiles rereads tile ke - 1 >= 0 and computes nothing)
  if (LN || nst > 0) load_last(0, fa);
  if constexpr (LN) {
    load_epi();  // after the first weights: waiting for the partials does not wait for these
    ln_partials_reduce(p.ln_in, lnv, K, B, lnst);
    ln_a = lnst[b][1];
    ln_c = -lnst[b][0] * lnst[b][1];
    if (p.h_out && blockIdx.x == 0) {
      // the normalised input, for a caller that records it
      const int n8 = K >> 3;
      for (int c = threadIdx.x; c < B * n8; c += kThreads) {
        const int r = c / n8, cc = c - r * n8;
        const uint4 xv = load_g16((const uint4*)((const uint16_t*)p.x + (long long)r * p.ldx + 8 * cc));
        *(uint4*)((uint16_t*)p.h_out + (long long)r * p.ldh + 8 * cc) =
            normalize8_fma<T>(xv, lnst[r][1], -lnst[r][0] * lnst[r][1]);
      }
    }
  }
  // a step's loads stay ahead of the products of the step before (the scheduler would move
  // the normalisation of arrived fragments above them and let the memory pipe run dry)
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  int st = 0;
  for (; st + 3 < nst; st += 2) {
    load(st + 1, fb);
    fence();
    compute(fa);
    fence();
    load(st + 2, fa);
    fence();
    compute(fb);
    fence();
  }
  if (st + 2 < nst) {
    load(st + 1, fb);
    fence();
    compute(fa);
    load_last(st + 2, fa);
    fence();
    compute(fb);
    fence();
    compute_last(st + 2, fa);
  } else if (st + 1 < nst) {
    load_last(st + 1, fb);
    fence();
    compute(fa);
    fence();
    compute_last(st + 1, fb);
  } else if (st < nst) {
    compute_last(st, fa);
  }
  // lane l of an accumulator holds rows 4 (l / 16) + v, v < 4, of column l % 16: the even
  // tiles' sum of batch row j is in column j, the odd tiles' in column j + 8 (rotated by 8
  // lanes within its row of 16)
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float odd = acc[r][1][v];
      part[wave][r][v][lane] = acc[r][0][v] + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                                                            0, __builtin_bit_cast(int, odd), 0x128, 0xF,
                                                                            0xF, false));  // row_ror:8
    }
  __syncthreads();
  const int l = j + 16 * (i >> 2), v = i & 3;
  float s[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int r = min(r0 + 2 * q, R - 1);
    s[q] = (part[0][r][v][l] + part[1][r][v][l]) + (part[2][r][v][l] + part[3][r][v][l]);
  }
  if (G > 1) {
    const int nr = min(R, RT - rt0), one = kTileRows * B;  // floats of one row tile's partial
    const auto rs = rsrc(p.ws + (size_t)rt0 * G * one, (uint32_t)(nr * G * one * (int)sizeof(float)));
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (mine(q) && r0 + 2 * q < nr)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, s[q]), rs,
                                              (((r0 + 2 * q) * G + gi) * one + j * kTileRows + i) * 4, 0, kCoherent);
    __builtin_amdgcn_s_waitcnt(0);  // this thread's partial stores have completed
    __syncthreads();
    if (t == 0) {
      const uint32_t prev = __hip_atomic_fetch_add(p.cnt + rg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = prev == (uint32_t)(G - 1);
      if (last) __hip_atomic_store(p.cnt + rg, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next launch
    }
    __syncthreads();
    if (!last) return;
    // the partials are requested together (one round trip) and added in split order; a split
    // past G reads past the descriptor's size and is not added
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      float pv[kMaxSplits];
#pragma unroll
      for (int g = 0; g < kMaxSplits; ++g)
        pv[g] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(
                       rs, mine(q) && g < G ? (uint32_t)(((r0 + 2 * q) * G + g) * one + j * kTileRows + i) * 4u : kXPast,
                       0, kCoherent));
      s[q] = pv[0];
#pragma unroll
      for (int g = 1; g < kMaxSplits; ++g)
        if (g < G) s[q] += pv[g];
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int rt = rt0 + r0 + 2 * q, row = row0 + 2 * kTileRows * q;
    float yv = 0.f;
    if (valid(q)) {
      yv = apply_epi(s[q] + T::to_f32(bias_v[q]), p.epi, T::to_f32(resid_v[q]));
      store_y<T>(p.y, j * p.ldy + row, p.y_f32, yv);
    }
    // LayerNorm partials of this row tile's outputs for the next linear: a row of 16 lanes
    // holds the 16 rows of one batch row
    if (!p.ln_out) continue;
    const float n = (float)min(kTileRows, p.rows - rt * kTileRows);
    const float a = valid(q) ? T::to_f32(round_act<T>(yv)) : 0.f;
    const float s1 = row16_sum(a);
    const float d = valid(q) ? a - s1 / n : 0.f;
    const float m2 = row16_sum(d * d);
    if (valid(q) && i == 0) *(f32x2*)(p.ln_out + ((size_t)rt * kLnSlots + j) * 2) = f32x2{s1, m2};
  }
}

// ---------------------------------------------------------------------------
// Matrix-core GEMV on row-major weights (hetegen_linear's resident rows, see
// gemv_rows_wanted; no LayerNorm).  Read in the operand's order, a row-major weight would cost
// half-line loads (64 bytes of each of 16 rows per load); instead a wavefront loads 512 or
// 1024 contiguous bytes of each of its H = 16 or 8 rows, turns them into operands through
// its own slice of LDS (rows 16 bytes apart modulo the banks; no workgroup barrier) and
// multiplies them as gemv_mfma_kernel does, x fragments of two k-tiles per load.
//  * H = 16: the two k-tiles of a fragment are two products, as in gemv_mfma_kernel.
//  * H = 8: one product takes both: operand rows 0..7 are the 8 rows at the first k-tile,
//    rows 8..15 the same rows at the second, so the first tile's sums are in rows 0..7 of
//    columns 0..7 and the second's in rows 8..15 of columns 8..15.  Twice the workgroups for
//    the same rows, for grids that would not fill the device; x is then read as often as W.
// A workgroup owns H rows; its 4 wavefronts take steps of SC columns in turn and are summed
// in LDS in order, so a row's bits depend on K and H alone.
// Bound by HBM from a few thousand rows on: [16384, 4096] at B = 8 25.0 us (5.4 TB/s) against
// 31.8 us on the vector GEMV, [36864, 9216] 101 (6.7 TB/s) against 159; [4096, 4096] 8.6 / 13.0.
// 8 wavefronts per workgroup, two row tiles per wavefront and wavefronts starting at
// different columns were slower nearly everywhere.
// ---------------------------------------------------------------------------
template <class T, int H>
__global__ __launch_bounds__(kThreads) void gemv_rows_kernel(GemvParams p, int B) {
  constexpr int SC = 4096 / H;           // columns per step: 8 KiB of weights per wavefront
  constexpr int LPR = SC / 8;            // lanes per row of a load
  constexpr int NL = 8, RPL = 64 / LPR;  // loads per step, rows per load
  constexpr int NP = SC / 64;            // x fragments (pairs of k-tiles) per step
  constexpr int PAIR = H == 16 ? 1 : 2;  // k-tiles between the two of a pair (2: other LDS banks)
  constexpr int kRow = SC * 2 + 16;      // bytes of a row in LDS
  __shared__ __align__(16) char tile[kWaves][H * kRow];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int K = p.K, row0 = blockIdx.x * H;
  const int steps = (K + SC - 1) / SC;
  const int nst = steps > wave ? (steps - wave + kWaves - 1) / kWaves : 0;  // this wavefront's steps wave + 4 st
  const int col = (lane % LPR) * 8;
  const uint16_t* wp[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i)
    wp[i] = (const uint16_t*)p.W + (long long)min(row0 + RPL * i + lane / LPR, p.rows - 1) * K + col;
  const int half = (lane >> 3) & 1, grp = lane >> 4;
  const auto xrs = rsrc(p.x, (uint32_t)(((long long)(B - 1) * p.ldx + K) * 2));
  const bool xlane = (lane & 7) < B;
  const int xcol = half * PAIR * kTileK + 8 * grp;
  const uint32_t xoff = (uint32_t)((long long)min(lane & 7, B - 1) * p.ldx * 2) + 2u * xcol;
  // first k-tile of pair u: 2 u, or the pairs (0, 2), (1, 3) of every four
  auto first = [](int u) { return PAIR == 1 ? 2 * u : (u >> 1) * 4 + (u & 1); };
  struct Buf {
    uint4 w[NL], x[NP];
  };
  auto load = [&](int st, Buf& f) {
    const int k0 = (wave + st * kWaves) * SC;
    // past the row's end (K % 8 == 0: a group of 8 columns is wholly inside or past K): the
    // row's last group, zeroed below, for the row may hold infinities there
    const int off = k0 + col < K ? k0 : K - 8 - col;
#pragma unroll
    for (int i = 0; i < NL; ++i) f.w[i] = load_stream((const uint4*)(wp[i] + off));
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int kx = k0 + first(u) * kTileK;
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(
          xrs, (xlane & (kx + xcol < K)) ? xoff + 2u * kx : kXPast, 0, 0);
      f.x[u] = make_uint4(v.x, v.y, v.z, v.w);
    }
  };
  // A wavefront's sum over K is kept within the vector GEMV's error against 64 bits (64 lanes'
  // partials) at every K.  binary16: chains of 4 products, then the sums of two steps (in one chain
  // the error was 1.7 times the vector GEMV's at K = 5128; now 0.37-1.00 of it).  bfloat16, whose
  // exact products are shorter, so that the vector GEMV rounds less: every product starts from
  // zero, a step's are added pairwise and the steps in turn (0.86-1.00; with the chains it was
  // 1.02-1.09 for K = 264..4096).
  constexpr int NH = H == 16 ? 2 : 1;  // the k-tiles of a pair: two products, or one for both
  constexpr int NA = NP / 2;           // accumulators per product
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[NH][NA], sum[NH];
  auto clear = [&] {
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
      for (int n = 0; n < NA; ++n) acc[h][n] = zero;
  };
  auto fold = [&] {  // what compute has left in acc
    if constexpr (!T::kRowsTree) {
#pragma unroll
      for (int h = 0; h < NH; ++h) sum[h] += NA == 4 ? (acc[h][0] + acc[h][1]) + (acc[h][2 % NA] + acc[h][3 % NA])
                                                     : acc[h][0] + acc[h][1];
      clear();
    }
  };
#pragma unroll
  for (int h = 0; h < NH; ++h) sum[h] = zero;
  clear();
  char* my = tile[wave];
  auto compute = [&](int st, const Buf& f) {
    const bool in = (wave + st * kWaves) * SC + col < K;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      uint4 v = f.w[i];
      if (!in) v = make_uint4(0u, 0u, 0u, 0u);
      *(uint4*)(my + (RPL * i + lane / LPR) * kRow + col * 2) = v;
    }
    // the lanes of a wavefront exchange the rows: LDS serves a wavefront in order, so only
    // the compiler has to keep the reads behind the writes (and the next step's writes behind)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const char* op = my + (lane & (H - 1)) * kRow + grp * 16 + (H == 8 ? half * PAIR * 64 : 0);
    auto weights = [&](int u, int h) { return *(const uint4*)(op + (first(u) + h) * 64); };
    if constexpr (T::kRowsTree) {
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        f32x4 pr[NP];
#pragma unroll
        for (int u = 0; u < NP; ++u) pr[u] = Mma<T>::run(weights(u, h), f.x[u], zero);
#pragma unroll
        for (int n = NP / 2; n >= 1; n /= 2)
#pragma unroll
          for (int u = 0; u < n; ++u) pr[u] += pr[u + n];
        sum[h] += pr[0];
      }
    } else {
#pragma unroll
      for (int u = 0; u < NP; ++u)
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[h][u % NA] = Mma<T>::run(weights(u, h), f.x[u], acc[h][u % NA]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // thread t finishes row i of batch row j; its bias and residual are requested first
  const int t = threadIdx.x, i = t % H, j = t / H;
  const bool valid = j < B && row0 + i < p.rows;
  uint16_t bias_v = 0, resid_v = 0;
  if (valid && p.bias) bias_v = gmem((const uint16_t*)p.bias)[row0 + i];
  if (valid && p.epi == EPI_RESID) resid_v = gmem((const uint16_t*)p.resid)[j * p.ldr + row0 + i];
  Buf fa, fb;
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };  // the loads stay ahead of the products
  if (nst > 0) load(0, fa);
  int st = 0;
  for (; st + 2 < nst; st += 2) {
    load(st + 1, fb);
    fence();
    compute(st, fa);
    fence();
    load(st + 2, fa);
    fence();
    compute(st + 1, fb);
    fold();
    fence();
  }
  if (st + 1 < nst) {
    load(st + 1, fb);
    fence();
    compute(st, fa);
    compute(st + 1, fb);
  } else if (st < nst) {
    compute(st, fa);
  }
  fold();
  // the wavefronts' partial tiles through LDS (over the staging rows: a barrier first).  Lane
  // l holds rows 4 (l / 16) + v of column l % 16; the second tiles' sums are 8 columns on
  float(*part)[2][4][64] = (float(*)[2][4][64])tile;
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    part[wave][0][v][lane] = sum[0][v];
    if constexpr (H == 16) part[wave][1][v][lane] = sum[NH - 1][v];
  }
  __syncthreads();
  if (valid) {
    const int l0 = j + 16 * (i >> 2), l1 = H == 16 ? l0 + 8 : j + 8 + 16 * ((i + 8) >> 2), v = i & 3;
    float s[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s[w] = part[w][0][v][l0] + part[w][H == 16 ? 1 : 0][v][l1];
    store_y<T>(p.y, j * p.ldy + row0 + i, p.y_f32,
               apply_epi(((s[0] + s[3]) + (s[1] + s[2])) + T::to_f32(bias_v), p.epi, T::to_f32(resid_v)));
  }
}

// Tile order of W [rows, K]: one 16-byte group per thread (see tiled_bytes in kernels.h).
__global__ __launch_bounds__(kThreads) void tile_kernel(const uint16_t* __restrict__ W, long long ldw, int rows,
                                                        int K, uint4* __restrict__ dst, long long groups, int korder) {
  const int KT = (K + kTileK - 1) / kTileK;
  const long long RT = (rows + kTileRows - 1) / kTileRows;
  for (long long q = (long long)blockIdx.x * kThreads + threadIdx.x; q < groups;
       q += (long long)gridDim.x * kThreads) {
    const int l = (int)(q & 63);
    const long long tile = q >> 6;
    const int kt = korder ? (int)(tile / RT) : (int)(tile % KT);
    const long long rt = korder ? tile % RT : tile / KT;
    const long long row = rt * kTileRows + (l & 15);
    const int k = kt * kTileK + 8 * (l >> 4);
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (row < rows && k < K) v = *(const uint4*)(W + row * ldw + k);
    dst[q] = v;
  }
}

// ---------------------------------------------------------------------------
// Persistent decode step: one cooperative launch runs every linear of the step,
// each workgroup taking the same row block of every linear, with a grid barrier
// between dependent linears.  A workgroup requests the weights of its first
// task of linear i+1 before it waits at the barrier of linear i, so HBM keeps
// streaming through the barrier and the next prologue.
// Barrier: workgroups arrive on one of `ngroups` counters (blockIdx % ngroups);
// the last arrival of a group bumps the top counter, which the waiting
// workgroups poll.  Counters only grow (wrap-safe comparisons); barrier n of the
// model's lifetime completes when the top counter reaches (n + 1) * ngroups.
// The wait gives up after a bounded number of polls, records the failure in
// `err` and lets the kernel run to its end, so the grid always drains.
// ---------------------------------------------------------------------------
constexpr int kCounterStride = 64;  // uint32 words: one 256-byte line per counter

__device__ __forceinline__ bool reached(uint32_t v, uint32_t target) { return (int32_t)(v - target) >= 0; }

__device__ __forceinline__ void grid_arrive(const StepArgs& a, uint32_t n) {
  // every thread's output stores have completed (coherent stores: visible device-wide)
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int g = blockIdx.x % a.ngroups;
    const uint32_t gsize = gridDim.x / a.ngroups + ((uint32_t)g < gridDim.x % a.ngroups ? 1u : 0u);
    const uint32_t old =
        __hip_atomic_fetch_add(a.counters + g * kCounterStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1u == (n + 1u) * gsize)
      __hip_atomic_fetch_add(a.counters + a.ngroups * kCounterStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ void grid_wait(const StepArgs& a, uint32_t n) {
  if (threadIdx.x == 0) {
    const uint32_t target = (n + 1u) * (uint32_t)a.ngroups;
    const uint32_t* top = a.counters + a.ngroups * kCounterStride;
    uint32_t spins = 0;
    while (!reached(__hip_atomic_load(top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), target)) {
      if (++spins > a.spin_limit) {
        __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
  }
  __syncthreads();
}

template <class T, int B, int R, int U>
__global__ __launch_bounds__(kThreads) void step_kernel(StepArgs a) {
  extern __shared__ uint4 smem[];
  __shared__ float red[2][8][kWaves];
  for (int i = 0; i < a.nlin; ++i) {
    const StepLinear& d = a.lin[i];
    GemvParams p{};
    p.x = d.x_in ? a.x_in : d.x;
    p.ldx = d.ldx;
    p.W = d.W;
    p.bias = d.bias;
    p.y = d.y_out ? a.out : d.y;
    p.ldy = d.ldy;
    p.resid = d.resid_in ? a.x_in : d.resid;
    p.ldr = d.ldr;
    p.rows = d.rows;
    p.K = d.K;
    p.epi = d.epi;
    p.ln = d.ln;
    p.rpw = d.rpw;
    p.segmajor = d.segmajor;
    const uint32_t n = a.barrier_base + (uint32_t)i;
    gemv_block<T, B, R, U, true, true>(p, blockIdx.x, smem, red, [&] {
      if (i > 0) grid_wait(a, n - 1u);
    });
    grid_arrive(a, n);
  }
}

// ---------------------------------------------------------------------------
// K-tiled GEMV for x that does not fit in LDS: x is restaged per K tile and row
// group (grid-stride over row groups).  No fused LayerNorm: a LayerNorm input fits in
// LDS at the batches that fuse it (B <= 4, hidden size <= kMaxLnK).
// ---------------------------------------------------------------------------
template <int B>
__device__ __forceinline__ void stage_x_tile(const GemvParams& p, uint4* xs, int k0, int kn) {
  const uint16_t* x = (const uint16_t*)p.x;
  const int n8 = kn >> 3, kt8 = p.ktile >> 3;
  for (int c = threadIdx.x; c < n8; c += kThreads) {
    uint4 v[B];
#pragma unroll
    for (int b = 0; b < B; ++b) v[b] = *(const uint4*)(x + b * p.ldx + k0 + (long long)c * 8);
#pragma unroll
    for (int b = 0; b < B; ++b) xs[b * kt8 + c] = v[b];
  }
}

template <class T, int B, int R, int U>
__global__ __launch_bounds__(kThreads) void gemv_tiled_kernel(GemvParams p) {
  extern __shared__ uint4 xs[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int K = p.K, ktile = p.ktile, kt8 = ktile >> 3;
  const int ntiles = (K + ktile - 1) / ktile;
  const int nrg = (p.rows + R - 1) / R;
  const uint16_t* W = (const uint16_t*)p.W;
  const uint16_t* bias = (const uint16_t*)p.bias;
  for (int rg0 = blockIdx.x * kWaves; rg0 < nrg; rg0 += gridDim.x * kWaves) {
    const int rg = rg0 + wave;
    const bool valid = rg < nrg;  // uniform per wavefront
    const int row0 = rg * R;
    const uint4* wp[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wp[r] = (const uint4*)(W + (long long)min(row0 + r, p.rows - 1) * K);
    float acc[R][B];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int b = 0; b < B; ++b) acc[r][b] = 0.f;
    for (int t = 0; t < ntiles; ++t) {
      const int k0 = t * ktile, kn = min(ktile, K - k0);
      __syncthreads();
      stage_x_tile<B>(p, xs, k0, kn);
      __syncthreads();
      if (valid) {
        const int n8 = kn >> 3, c0 = k0 >> 3;
        int c = lane;
        for (; c + 64 * (U - 1) < n8; c += 64 * U) {
          uint4 w[U][R];
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) w[u][r] = load_stream(wp[r] + c0 + c + 64 * u);
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < B; ++b) {
              const uint4 xv = xs[b * kt8 + c + 64 * u];
#pragma unroll
              for (int r = 0; r < R; ++r) acc[r][b] = dot8<T>(w[u][r], xv, acc[r][b]);
            }
        }
        for (; c < n8; c += 64) {
          uint4 w[R];
#pragma unroll
          for (int r = 0; r < R; ++r) w[r] = load_stream(wp[r] + c0 + c);
#pragma unroll
          for (int b = 0; b < B; ++b) {
            const uint4 xv = xs[b * kt8 + c];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r][b] = dot8<T>(w[r], xv, acc[r][b]);
          }
        }
      }
    }
    if (valid) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
          float s = wave_sum(acc[r][b]);
          const int row = row0 + r;
          if (lane == 0 && row < p.rows) {
            if (bias) s += T::to_f32(bias[row]);
            const float rv = p.epi == EPI_RESID ? T::to_f32(((const uint16_t*)p.resid)[b * p.ldr + row]) : 0.f;
            store_y<T>(p.y, b * p.ldy + row, p.y_f32, apply_epi(s, p.epi, rv));
          }
        }
      }
    }
  }
}

// LayerNorm of a materialised input, one batch row per blockIdx.y (the statistics of a
// row are the same bits whatever the batch), the row held in registers (thread t keeps
// chunks t + 256 i, the chunks ln_stats gives it, for i < NI): every sum is formed in
// ln_stats' order, so the bits are those of the GEMVs that fuse the LayerNorm.
template <class T, int NI>
__global__ __launch_bounds__(kThreads) void layernorm_regs_kernel(const uint16_t* __restrict__ x, long long ldx,
                                                                  int K, uint16_t* __restrict__ h, long long ldh,
                                                                  float* __restrict__ h_host) {
  __shared__ float red[2][kWaves];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint16_t* xr = x + b * ldx;
  const int n8 = K >> 3;  // <= kThreads * NI (launcher)
  uint4 v[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = tid + kThreads * i;
    v[i] = c < n8 ? *(const uint4*)(xr + (long long)c * 8) : make_uint4(0u, 0u, 0u, 0u);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (tid + kThreads * i < n8) {
      float f[8];
      unpack8<T>(v[i], f);
      s += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
    }
  }
  s = wave_sum(s);
  if (lane == 0) red[0][wave] = s;
  __syncthreads();
  const float mean = ((red[0][0] + red[0][1]) + (red[0][2] + red[0][3])) / (float)K;
  s = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (tid + kThreads * i < n8) {
      float f[8];
      unpack8<T>(v[i], f);
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float d = f[e] - mean;
        acc += d * d;
      }
      s += acc;
    }
  }
  s = wave_sum(s);
  if (lane == 0) red[1][wave] = s;
  __syncthreads();
  const float var = ((red[1][0] + red[1][1]) + (red[1][2] + red[1][3])) / (float)K;
  const float rstd = 1.0f / sqrtf(var + kLnEps);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = tid + kThreads * i;
    if (c < n8) {
      const uint4 o = normalize8<T>(v[i], mean, rstd);
      *(uint4*)(h + b * ldh + (long long)c * 8) = o;
      if (h_host) {
        float f[8];
        unpack8<T>(o, f);
        float4* dst = (float4*)(h_host + (long long)b * K + (long long)c * 8);
        dst[0] = make_float4(f[0], f[1], f[2], f[3]);
        dst[1] = make_float4(f[4], f[5], f[6], f[7]);
      }
    }
  }
}

template <class T>
__global__ __launch_bounds__(kThreads) void export_kernel(const uint16_t* __restrict__ x, long long ldx, int B, int K,
                                                          float* __restrict__ dst) {
  const int n8 = K >> 3;
  const long long total = (long long)B * n8;
  for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < total; i += (long long)gridDim.x * kThreads) {
    const int b = (int)(i / n8), c = (int)(i - (long long)b * n8);
    float f[8];
    unpack8<T>(*(const uint4*)(x + b * ldx + (long long)c * 8), f);
    float4* d = (float4*)(dst + (long long)b * K + (long long)c * 8);
    d[0] = make_float4(f[0], f[1], f[2], f[3]);
    d[1] = make_float4(f[4], f[5], f[6], f[7]);
  }
}

template <class T>
__global__ __launch_bounds__(kThreads) void import_kernel(const float* __restrict__ src, int B, int n, int epi,
                                                          void* __restrict__ y, long long ldy, int y_f32,
                                                          const void* __restrict__ resid, long long ldr) {
  const long long total = (long long)B * n;
  for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < total; i += (long long)gridDim.x * kThreads) {
    const int b = (int)(i / n), c = (int)(i - (long long)b * n);
    const float rv = epi == EPI_RESID ? T::to_f32(((const uint16_t*)resid)[b * ldr + c]) : 0.f;
    store_y<T>(y, b * ldy + c, y_f32, apply_epi(src[i], epi, rv));
  }
}

// Per-batch tiling: rows per wavefront R and 16-byte steps per task U (U*R loads in flight).
template <int B> struct Tile;
// (Measured on OPT-6.7B/13B shapes: one row per wavefront up to B = 4, two from B = 5.)
template <> struct Tile<1> { static constexpr int R = 1, U = 8; };
template <> struct Tile<2> { static constexpr int R = 1, U = 8; };
template <> struct Tile<3> { static constexpr int R = 1, U = 4; };
template <> struct Tile<4> { static constexpr int R = 1, U = 4; };
template <> struct Tile<5> { static constexpr int R = 2, U = 2; };
template <> struct Tile<6> { static constexpr int R = 2, U = 2; };
template <> struct Tile<7> { static constexpr int R = 2, U = 2; };
template <> struct Tile<8> { static constexpr int R = 2, U = 2; };

constexpr size_t kLdsMain = 65536 - 1024;  // dynamic LDS of the persistent step (x, bias, residual, outputs)

// LDS a workgroup of the per-linear main GEMV may use on this device (gfx950: 160 KiB
// per CU, all of it addressable by one workgroup), less a margin for the static
// arrays; and the LDS of one CU, which bounds the co-resident workgroups.
struct LdsInfo {
  size_t per_block = 65536, per_cu = 65536;
  int cus = 1;
};
const LdsInfo& lds_info() {
  static const LdsInfo info = [] {
    LdsInfo i;
    int dev = 0, blk = 0, cu = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&blk, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
        hipDeviceGetAttribute(&cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && blk > 0 && cu > 0 &&
        n > 0) {
      i.per_block = (size_t)blk;
      i.per_cu = (size_t)cu;
      i.cus = n;
    }
    (void)hipGetLastError();
    return i;
  }();
  return info;
}
constexpr int kTiledLdsBudget = 32768;  // bytes of x per tile in the K-tiled kernel
constexpr int kDefaultGridCap = 1024;

// Batches up to this size run linears without a fused LayerNorm on gemv_x1_kernel (x
// read per wavefront from L1/L2) rather than staging x in LDS per workgroup (OPT-6.7B
// shapes at B = 2: out 9.3 -> 8.6 us, fc2 25.9 -> 25.3 us; slower from B = 3 on, and
// the register LayerNorm kernel only pays at B = 1).
constexpr int kX1MaxB = 2;
constexpr int kMaxLnRegChunks = 14;  // 512-element chunks of a row gemv_ln1_kernel keeps in registers

// gemv_ln1_kernel for rows of nc chunks of 512.
template <class T, int NC>
hipError_t launch_ln1(const GemvParams& p, int nc, int grid, hipStream_t s) {
  if constexpr (NC <= kMaxLnRegChunks) {
    if (nc != NC) return launch_ln1<T, NC + 1>(p, nc, grid, s);
    if (p.K == 512 * NC) hipLaunchKernelGGL((gemv_ln1_kernel<T, NC, false>), dim3(grid), dim3(kThreads), 0, s, p);
    else hipLaunchKernelGGL((gemv_ln1_kernel<T, NC, true>), dim3(grid), dim3(kThreads), 0, s, p);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <class T, int B>
hipError_t launch_gemv_b(GemvParams p, hipStream_t s, int grid_cap) {
  constexpr int R = Tile<B>::R, U = Tile<B>::U;
  const int cap = grid_cap > 0 ? grid_cap : kDefaultGridCap;
  if constexpr (B <= kX1MaxB) {
    // rows of up to 7168 (NC = 14): at NC = 18 (9216) the row no longer fits the registers well
    // and the LDS kernel is as fast
    const int nc = (p.K + 511) / 512;
    const bool ln_regs = B == 1 && p.ln && nc <= kMaxLnRegChunks;
    // segment-major weights: gemv_x1_kernel and gemv_block (below) read them, the register
    // LayerNorm kernel does not
    if (p.segmajor && ln_regs) return hipErrorInvalidValue;
    if (!p.ln || ln_regs) {
      const long long units = (p.rows + kWaves - 1) / kWaves;
      const long long per = std::min<long long>((units + cap - 1) / cap, kX1MaxRows);
      p.rpw = (int)(per * kWaves);
      const int grid = (int)((p.rows + p.rpw - 1) / p.rpw);
      if (!p.ln) {
        hipLaunchKernelGGL((gemv_x1_kernel<T, 4, B>), dim3(grid), dim3(kThreads), 0, s, p);
        return hipGetLastError();
      }
      return launch_ln1<T, 1>(p, nc, grid, s);
    }
  }
  // contiguous row blocks of a multiple of R*kWaves rows, at most `cap` blocks; a block
  // that needs much LDS also caps the grid at the workgroups that fit at once (more
  // would run in a second round)
  const int unit = R * kWaves;
  const long long units = (p.rows + unit - 1) / unit;
  const LdsInfo& li = lds_info();
  const size_t lds_max = li.per_block - 1024;
  auto block_lds = [&](int c) {
    const long long per = (units + c - 1) / c;
    return (size_t)B * p.K * 2 + (size_t)(1 + 2 * B) * (size_t)(per * unit) * 4;  // gemv_lds_bytes
  };
  int cap_b = cap;
  const size_t lds0 = block_lds(cap_b);
  if (lds0 <= lds_max) {
    const long long fit = (long long)li.cus * (long long)std::max<size_t>(1, li.per_cu / lds0);
    if (fit < cap_b && block_lds((int)std::max<long long>(1, fit)) <= lds_max)
      cap_b = (int)std::max<long long>(1, fit);
    const long long per = (units + cap_b - 1) / cap_b;
    const int rpw = (int)(per * unit);
    const size_t lds = block_lds(cap_b);
    if (lds > 65536) {  // beyond the default dynamic LDS: opt in once per kernel
      static const hipError_t opt = hipFuncSetAttribute((const void*)gemv_kernel<T, B, R, U>,
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
      if (opt != hipSuccess) return opt;
    }
    p.rpw = rpw;
    p.ktile = p.K;
    const int grid = (int)((p.rows + rpw - 1) / rpw);
    hipLaunchKernelGGL((gemv_kernel<T, B, R, U>), dim3(grid), dim3(kThreads), lds, s, p);
    return hipGetLastError();
  }
  if (p.ln) return hipErrorInvalidValue;  // not reached: see gemv_tiled_kernel
  if (p.segmajor) return hipErrorInvalidValue;  // gemv_tiled_kernel reads row-major weights
  int kt = kTiledLdsBudget / (2 * B);
  kt -= kt % 512;
  p.ktile = kt;
  const int nrg = (p.rows + R - 1) / R;
  int grid = (nrg + kWaves - 1) / kWaves;
  if (grid > cap) grid = cap;
  hipLaunchKernelGGL((gemv_tiled_kernel<T, B, R, U>), dim3(grid), dim3(kThreads), (size_t)B * kt * 2, s, p);
  return hipGetLastError();
}

template <class T>
hipError_t launch_gemv_t(const GemvParams& p, int B, hipStream_t s, int cap) {
  switch (B) {
    case 1: return launch_gemv_b<T, 1>(p, s, cap);
    case 2: return launch_gemv_b<T, 2>(p, s, cap);
    case 3: return launch_gemv_b<T, 3>(p, s, cap);
    case 4: return launch_gemv_b<T, 4>(p, s, cap);
    case 5: return launch_gemv_b<T, 5>(p, s, cap);
    case 6: return launch_gemv_b<T, 6>(p, s, cap);
    case 7: return launch_gemv_b<T, 7>(p, s, cap);
    case 8: return launch_gemv_b<T, 8>(p, s, cap);
  }
  return hipErrorInvalidValue;
}

template <class T, int NI>
hipError_t launch_ln_regs(int B, const uint16_t* x, long long ldx, int K, uint16_t* h, long long ldh, float* hh,
                          hipStream_t s) {
  hipLaunchKernelGGL((layernorm_regs_kernel<T, NI>), dim3(1, B), dim3(kThreads), 0, s, x, ldx, K, h, ldh, hh);
  return hipGetLastError();
}

template <class T>
hipError_t launch_ln_t(const void* x, long long ldx, int B, int K, void* h, long long ldh, float* hh, hipStream_t s) {
  if (B < 1 || B > 8) return hipErrorInvalidValue;
  const int n8 = K >> 3;
  // rows of up to 8 * kThreads * 8 elements (hidden sizes up to kMaxLnK) stay in registers
  const int ni = (n8 + kThreads - 1) / kThreads;
  const uint16_t* xx = (const uint16_t*)x;
  uint16_t* hp = (uint16_t*)h;
  switch (ni) {
    case 1: return launch_ln_regs<T, 1>(B, xx, ldx, K, hp, ldh, hh, s);
    case 2: return launch_ln_regs<T, 2>(B, xx, ldx, K, hp, ldh, hh, s);
    case 3: return launch_ln_regs<T, 3>(B, xx, ldx, K, hp, ldh, hh, s);
    case 4: return launch_ln_regs<T, 4>(B, xx, ldx, K, hp, ldh, hh, s);
    case 5: return launch_ln_regs<T, 5>(B, xx, ldx, K, hp, ldh, hh, s);
    case 6:
    case 7:
    case 8: return launch_ln_regs<T, 8>(B, xx, ldx, K, hp, ldh, hh, s);
    default: return hipErrorInvalidValue;  // K > kMaxLnK
  }
}

// The persistent step runs the row-major copy, which only batch 1 uses (models created for
// larger batches run batches from 2 on their matrix-core tiles; the batch-2 instance is
// not launched by the library).
template <class T>
const void* step_fn(int B) {
  switch (B) {
    case 1: return (const void*)step_kernel<T, 1, Tile<1>::R, Tile<1>::U>;
    case 2: return (const void*)step_kernel<T, 2, Tile<2>::R, Tile<2>::U>;
  }
  return nullptr;
}

int small_grid(long long work_items) {
  long long g = (work_items + kThreads - 1) / kThreads;
  if (g < 1) g = 1;
  if (g > 256) g = 256;
  return (int)g;
}

}  // namespace

int gemv_rows_unit(int B) {
  static const int r[9] = {0, Tile<1>::R, Tile<2>::R, Tile<3>::R, Tile<4>::R,
                           Tile<5>::R, Tile<6>::R, Tile<7>::R, Tile<8>::R};
  return (B >= 1 && B <= 8) ? r[B] : 0;
}

size_t gemv_lds_bytes(int B, int K, int rows_per_block) {
  return (size_t)B * K * 2 + (size_t)(1 + 2 * B) * rows_per_block * 4;
}

size_t gemv_lds_limit() { return kLdsMain; }

// Measured on OPT-6.7B shapes: from B = 5 on, normalising x once per workgroup in the
// prologue costs more than a separate LayerNorm launch.
bool gemv_fuses_ln(int B) { return B <= 4; }

int step_blocks_per_cu(int dtype, int B, size_t lds) {
  const void* f = dtype == 1 ? step_fn<BF16>(B) : step_fn<F16>(B);
  if (!f) return 0;
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, kThreads, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return n;
}

hipError_t launch_step(const StepArgs& a, int dtype, int B, int grid, size_t lds, hipStream_t stream) {
  const void* f = dtype == 1 ? step_fn<BF16>(B) : step_fn<F16>(B);
  if (!f) return hipErrorInvalidValue;
  StepArgs args = a;
  void* kargs[] = {(void*)&args};
  return hipLaunchCooperativeKernel(f, dim3(grid), dim3(kThreads), kargs, (unsigned)lds, stream);
}

hipError_t launch_gemv(GemvParams p, int dtype, int B, hipStream_t stream, int grid_cap) {
  if (p.rows <= 0) return hipSuccess;
  if (p.segmajor && (B != 1 || p.K % kSegElems)) return hipErrorInvalidValue;
  return dtype == 1 ? launch_gemv_t<BF16>(p, B, stream, grid_cap) : launch_gemv_t<F16>(p, B, stream, grid_cap);
}

hipError_t launch_layernorm(const void* x, long long ldx, int B, int K, int dtype, void* h, long long ldh,
                            float* h_host_f32, hipStream_t stream) {
  return dtype == 1 ? launch_ln_t<BF16>(x, ldx, B, K, h, ldh, h_host_f32, stream)
                    : launch_ln_t<F16>(x, ldx, B, K, h, ldh, h_host_f32, stream);
}

hipError_t launch_export_f32(const void* x, long long ldx, int B, int K, int dtype, float* dst, hipStream_t stream) {
  const int grid = small_grid((long long)B * (K >> 3));
  if (dtype == 1)
    hipLaunchKernelGGL(export_kernel<BF16>, dim3(grid), dim3(kThreads), 0, stream, (const uint16_t*)x, ldx, B, K, dst);
  else
    hipLaunchKernelGGL(export_kernel<F16>, dim3(grid), dim3(kThreads), 0, stream, (const uint16_t*)x, ldx, B, K, dst);
  return hipGetLastError();
}

hipError_t launch_import_rows(const float* src, int B, int n, int dtype, int epi, void* y, long long ldy, int y_f32,
                              const void* resid, long long ldr, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int grid = small_grid((long long)B * n);
  if (dtype == 1)
    hipLaunchKernelGGL(import_kernel<BF16>, dim3(grid), dim3(kThreads), 0, stream, src, B, n, epi, y, ldy, y_f32,
                       resid, ldr);
  else
    hipLaunchKernelGGL(import_kernel<F16>, dim3(grid), dim3(kThreads), 0, stream, src, B, n, epi, y, ldy, y_f32,
                       resid, ldr);
  return hipGetLastError();
}

size_t tiled_bytes(int rows, int K) {
  if (rows <= 0 || K <= 0) return 0;
  return (size_t)((rows + kTileRows - 1) / kTileRows) * (size_t)((K + kTileK - 1) / kTileK) * 1024;
}

// Segment-major copy (see launch_segmajor): one 16-byte group per thread.
__global__ __launch_bounds__(kThreads) void segmajor_kernel(const uint4* __restrict__ W, int rows, int k8,
                                                            uint4* __restrict__ dst, long long n) {
  constexpr int SEG = kSegElems / 8;
  for (long long q = (long long)blockIdx.x * kThreads + threadIdx.x; q < n; q += (long long)gridDim.x * kThreads) {
    const long long s = q / ((long long)rows * SEG), rem = q - s * rows * SEG, r = rem / SEG, i = rem - r * SEG;
    dst[q] = W[r * k8 + s * SEG + i];
  }
}

hipError_t launch_segmajor(const void* W, int rows, int K, void* dst, hipStream_t stream) {
  if (rows <= 0 || K <= 0 || K % kSegElems) return hipErrorInvalidValue;
  const long long n = (long long)rows * (K / 8);
  long long g = std::min<long long>((n + kThreads - 1) / kThreads, 4096);
  hipLaunchKernelGGL(segmajor_kernel, dim3((unsigned)g), dim3(kThreads), 0, stream, (const uint4*)W, rows, K / 8,
                     (uint4*)dst, n);
  return hipGetLastError();
}

hipError_t launch_tile(const void* W, long long ldw, int rows, int K, void* dst, hipStream_t stream, int korder) {
  const long long groups = (long long)(tiled_bytes(rows, K) / 16);
  if (groups == 0) return hipSuccess;
  long long g = (groups + kThreads - 1) / kThreads;
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(tile_kernel, dim3((unsigned)g), dim3(kThreads), 0, stream, (const uint16_t*)W, ldw, rows, K,
                     (uint4*)dst, groups, korder);
  return hipGetLastError();
}

// Compute units of the current device (read once per device).
static int device_cus() {
  static std::atomic<int> cus[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return kDefaultCus;
  int c = cus[dev].load(std::memory_order_relaxed);
  if (c == 0) {
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c < 1) c = kDefaultCus;
    cus[dev].store(c, std::memory_order_relaxed);
  }
  return c;
}

// How unevenly `wgs` equal workgroups load `cus` compute units: the busiest unit's
// workgroups over the mean (1 when wgs is a multiple of cus).
static double uneven(long long wgs, int cus) {
  const long long per = (wgs + cus - 1) / cus;
  return (double)(per * cus) / (double)wgs;
}

// The most K-splits a linear takes, by evenness alone: one workgroup per row tile unless that
// loads the CUs unevenly (more than 1.15x the mean on the busiest); then the fewest splits
// that do not, each at least 32 k-tiles long, or else the most even split.
static int even_splits(int rows, int K, int cus) {
  if (rows <= 0 || K <= 0) return 1;
  const int KT = (K + kTileK - 1) / kTileK, RT = (rows + kTileRows - 1) / kTileRows;
  double best_u = uneven(RT, cus);
  if (best_u <= kMaxUneven) return 1;
  int best = 1;
  for (int g = 2; g <= kMaxSplits && KT / g >= kMinSplitTiles; g *= 2) {
    const double u = uneven((long long)RT * g, cus);
    if (u <= kMaxUneven) return g;
    if (u < best_u) {
      best = g;
      best_u = u;
    }
  }
  return best;
}

// K-splits of a launch.  Splitting pays for an uneven grid only when K is long enough: the merge
// (partial store, arrival, loads) costs about 1.5 us at the tail.  Rows of fewer than 4096
// columns are not split ([2048, 2048] 4.8 us unsplit against 5.7 in 2, [768, 3072] 4.8 / 5.6,
// [10240, 2560] with the LayerNorm 11.4 / 13.6, all at B = 2 or 4), rows of fewer than 8192
// not in 2 up to 1.3x ([13000, 4360] with the LayerNorm 21.5 us unsplit against 24.8 in 2,
// [10007, 5128] 18.9 / 20.4; [5120, 5120], 1.6x, takes 4).  The two accumulators of an unsplit
// sum keep the error against 64 bits of two splits (0.98-1.00 of it), but not that of four
// ([6400, 4096] unsplit 1.31, [6400, 8160] 1.39 of it, though 10.4 against 12.7 us at B = 2):
// those are split as evenness says.  Long rows by evenness: OPT-13B fc2
// [5120, 20480] (320 row tiles) took 49.4 us unsplit and 39.1 in 4 splits, OPT-6.7B fc2 [4096,
// 16384] (256 row tiles, even) 23.9 unsplit and 26.2 in 4.  The choice does not depend on B, so
// a batch row's bits do not either.
static int splits_on(int rows, int K, int cus) {
  const int KT = (K + kTileK - 1) / kTileK, RT = (rows + kTileRows - 1) / kTileRows;
  if (KT < kMinTilesToSplit) return 1;
  const int G = even_splits(rows, K, cus);
  return KT < kLongTiles && G == 2 && uneven(RT, cus) <= kMaxUnevenShort ? 1 : G;
}

int mfma_splits(int rows, int K) { return rows <= 0 || K <= 0 ? 1 : splits_on(rows, K, device_cus()); }

// k-major tiles when the row tiles and splits put the same number of workgroups, 1 to 3, on
// every CU: all of them then start together and walk K side by side, and in row-tile order
// their loads would fall on the same offsets of blocks a fixed multiple of 16 rows apart,
// crowding a few memory channels (B = 8, row-tile order / k-major: OPT-6.7B fc2 [4096, 16384]
// 24.2 / 22.8 us, out [4096, 4096] 8.6 / 8.0, qkv [12288, 4096] 19.1 / 18.2); k-major, the
// walk reads one contiguous window.  With more workgroups per CU, or uneven ones, they drift
// apart and k-major scatters the loads instead (OPT-6.7B fc1 [16384, 4096], 4 per CU: 22.6 /
// 23.5 us; OPT-30B fc1 [28672, 7168], 7 per CU: 70.5 / 72.8).
int mfma_kmajor(int rows, int K) {
  if (rows <= 0 || K <= 0) return 0;
  const int cus = device_cus();
  const long long wgs = (long long)((rows + kTileRows - 1) / kTileRows) * splits_on(rows, K, cus);
  return wgs % cus == 0 && wgs / cus <= kMaxKmajorPerCu ? 1 : 0;
}

size_t mfma_ws_floats(int rows, int K, int B) {
  const int G = mfma_splits(rows, K);
  if (G == 1) return 0;
  return (size_t)((rows + kTileRows - 1) / kTileRows) * G * kTileRows * B;
}

size_t mfma_cnt_words(int rows, int K) {
  if (mfma_splits(rows, K) == 1) return 0;
  return (size_t)((rows + kTileRows - 1) / kTileRows);
}

// Row tiles per workgroup.  More of them share the x fragments (and the LayerNorm prologue
// and normalisation) of a k-tile, but make the grid coarser: what a CU then reads is
// ceil(workgroups / CUs) * R row tiles, and R is taken only where that is no more than with
// one row tile per workgroup.
//  * Unsplit with the LayerNorm: the largest such R up to 3.  B = 8 (us, R = 1 / 2 / 3 / 5): [15360,
//    5120] 29.0 / 27.0 / 33.6 / 30.1, [16384, 4096] 25.2 / 23.5 / 27.8 / 25.0.
//  * Unsplit without: 2, or 3 on a grid that one row tile per workgroup loads more than 1.1x
//    unevenly (R = 1 / 2 / 3: [5120, 3072] 9.0 / 8.0 / 10.0, [14336, 4096] 21.1 / 20.3 / 26.0, [8300,
//    3072], 1.48x, 12.5 / 13.9 / 11.3, but [12272, 3072], 1.001x, 13.5 / 14.8 / 14.4).  Rows of up to
//    640 columns are over so soon that fewer workgroups win on every grid above one per CU
//    ([16384, 264] 6.0 / 4.2 / 5.0, [20480, 520] 7.5 / 7.0 / 6.7).  Rows of 904 to 1024 are one full
//    request of 8 k-tiles per wavefront, which only R = 1 makes; above 4 row tiles per CU it wins up
//    to 1280 ([40000, 1024] at B = 1 14.2 / 15.7 / 15.9, [24576, 1152] at 8 11.5 / 12.6 / 11.3), and on
//    an even grid of so many from 2056 on too ([24576, 4096] at B = 4 31.0 / 32.5, but 1536 14.4 / 13.4).
//  * Split: 5 on an uneven grid, with the LayerNorm or for long splits (it brings the OPT-66B
//    grids, 1152 workgroups, to 232, all running at once), 3 for short splits of an even grid up
//    to a fifth more per CU (the workgroups of an even grid in row-tile order walk K in step and
//    crowd a few memory channels), else 1.  B = 8, R = 1 / 3 / 5: [9216, 36864] in 2 115 / 120 / 105,
//    [5120, 20480] in 4 39.6 / 38.8 / 38.2, [5120, 5120] in 4 14.0 / 13.2 / 14.5 and [5056, 5120],
//    1.01x, the same, [2560, 10240] in 8 14.5 / 13.5 / 14.6; [8300, 4096] in 4, 1.11x, 16.7 / 18.4 / 20.1.
// R does not change the bits.
static int mfma_rows(int rows, int K, int G, bool ln, int cus) {
  const int KT = (K + kTileK - 1) / kTileK, RT = (rows + kTileRows - 1) / kTileRows;
  auto load = [&](int r) { return ((long long)(RT + r - 1) / r * G + cus - 1) / cus * r; };
  const double u = uneven((long long)RT * G, cus);
  if (G > 1) {
    const bool even = u <= kRowTilesEven;
    if (even && !ln && KT / G < kLongSplitTiles && 5 * load(3) <= 6 * load(1)) return 3;
    return load(5) <= load(1) && (ln || !even || KT / G >= kLongSplitTiles) ? 5 : 1;
  }
  if (!ln && KT <= kSoonTiles) return RT <= cus ? 1 : load(3) <= load(2) ? 3 : 2;
  if (!ln && KT > kFullTiles - kChunkTiles && KT <= (RT > 4 * cus ? kFullTilesMany : kFullTiles)) return 1;
  if (load(3) <= std::min(load(1), load(2)) && (ln || u > kRowTilesUneven)) return 3;
  const bool many_even = !ln && RT > 4 * cus && u <= kRowTilesEven;
  return load(2) <= load(1) && !(many_even && KT > kShortRowTiles) ? 2 : 1;
}

template <class T, int U, int R, bool LN>
hipError_t launch_mfma_k(const GemvParams& p, int B, int G, hipStream_t s) {
  const int RT = (p.rows + kTileRows - 1) / kTileRows;
  hipLaunchKernelGGL((gemv_mfma_kernel<T, U, R, LN>), dim3((RT + R - 1) / R * G), dim3(kThreads), 0, s, p, B, G);
  return hipGetLastError();
}

// k-tiles per request and row tile: 4 when a workgroup holds several row tiles and in split
// launches (more requests in flight gained nothing there), 8 otherwise; with the LayerNorm
// and one row tile 8 only where registers are not short, i.e. at most one workgroup per CU
// ([4096, 1024] 4.55 against 5.05 us with 4: its whole K is one request) or rows long enough
// to pay for it ([20480, 5120] 36.2 against 37.0, but [12288, 4096] 18.7 against 18.4).
template <class T, bool LN>
hipError_t launch_mfma_t(const GemvParams& p, int B, int G, int cus, hipStream_t s) {
  const int RT = (p.rows + kTileRows - 1) / kTileRows;
  switch (mfma_rows(p.rows, p.K, G, LN, cus)) {
    case 5: return launch_mfma_k<T, 4, 5, LN>(p, B, G, s);
    case 3: return launch_mfma_k<T, 4, 3, LN>(p, B, G, s);
    case 2: return launch_mfma_k<T, 4, 2, LN>(p, B, G, s);
  }
  const bool u8 = G == 1 && (!LN || RT <= cus || p.K > kLongLnK);
  return u8 ? launch_mfma_k<T, 8, 1, LN>(p, B, G, s) : launch_mfma_k<T, 4, 1, LN>(p, B, G, s);
}

size_t ln_partials_floats(int n) { return n > 0 ? (size_t)((n + kLnGroup - 1) / kLnGroup) * kLnSlots * 2 : 0; }

hipError_t launch_gemv_mfma(GemvParams p, int dtype, int B, hipStream_t stream) {
  if (p.rows <= 0) return hipSuccess;
  if (p.K < 8 || p.K % 8 || B < 1 || B > kLnSlots) return hipErrorInvalidValue;
  if (p.ln && (!p.ln_in || p.K > kMaxLnK)) return hipErrorInvalidValue;
  if (p.ln_out && p.y_f32) return hipErrorInvalidValue;
  if (p.ldx < p.K || ((long long)(B - 1) * p.ldx + p.K) * 2 >= (long long)kXPast) return hipErrorInvalidValue;
  const int cus = device_cus(), G = splits_on(p.rows, p.K, cus);
  const size_t RT = (size_t)((p.rows + kTileRows - 1) / kTileRows);
  if (G > 1 && (!p.ws || !p.cnt || p.ws_floats < RT * G * kTileRows * B || p.cnt_words < RT))
    return hipErrorInvalidValue;
  if (p.ln) return dtype == 1 ? launch_mfma_t<BF16, true>(p, B, G, cus, stream)
                                : launch_mfma_t<F16, true>(p, B, G, cus, stream);
  return dtype == 1 ? launch_mfma_t<BF16, false>(p, B, G, cus, stream) : launch_mfma_t<F16, false>(p, B, G, cus, stream);
}

template <class T, int H>
hipError_t launch_rows_k(const GemvParams& p, int B, hipStream_t s) {
  hipLaunchKernelGGL((gemv_rows_kernel<T, H>), dim3((p.rows + H - 1) / H), dim3(kThreads), 0, s, p, B);
  return hipGetLastError();
}

// Row strides (2 K bytes) at which the rows of a workgroup crowd a few memory channels: 16 and
// 32 KiB, and (skewed) 64 bytes off a multiple of 16 KiB or 32 bytes off an odd multiple of 8 KiB.
static bool rows_skewed(int K) {
  const int m = K % 8192;
  return K > 4000 && (m == 32 || m == 8192 - 32 || m == 4096 - 16 || m == 4096 + 16);
}
static bool rows_crowded(int K) { return K == 8192 || K == 16384 || rows_skewed(K); }

// Resident row-major rows of a linear [N, K] on the matrix cores (N, not the GPU's share of it, so
// that a GPU row's bits do not depend on alpha).  The vector GEMV is bound by its products and by
// its reads of x from LDS, the more the larger the batch and again where x (2 B K bytes) lets one
// workgroup on a CU or does not fit; the matrix cores by an uneven grid and crowded channels.  The
// lines lie where both are equal in a sweep of 24 row counts (64..40000) by 44 lengths (64..36864);
// speed over it against the vector GEMV, geometric mean and worst: B = 1 1.01 / 0.98, 2 1.18 / 0.93,
// 3 1.09 / 0.92, 4 1.14 / 0.92, 5 1.30 / 0.94, 6 1.36 / 0.95, 8 1.45 / 0.93.  us, vector / matrix cores:
//  * B = 1: only with several rows to a wavefront, [18000, 264] 8.7 / 6.4, [20480, 5128] 36.5 /
//    34.8, [36864, 9216] 111 / 98; not K = 1032..2048 nor strides of 4 to 32 KiB, [20480, 2048]
//    14.6 / 17.2, [20480, 8192] 52.6 / 53.5.
//  * up to 1024 rows CUs are idle that one row per wavefront keeps busy: [1000, 4096] 4.0 / 4.4 at
//    B = 2, 4.8 / 4.6 at 3, 9.0 / 5.4 at 8; [1000, 8208] 6.8 / 7.2 at 3.
//  * crowded channels: [12288, 8160] 39.3 / 43.1 at 4, 56.7 / 47.2 at 8; [4096, 16384] 26.0 / 29.1 at
//    2, 29.4 / 29.6 at 4; [12288, 2048] 10.8 / 12.2 at 3, 12.2 / 11.9 at 4.
//  * B = 3, where the vector GEMV is at its best: [5120, 12288] 23.3 / 24.4, [12288, 12288] 49.0 /
//    46.7, [4200, 5128] 12.4 / 11.8; beyond the LDS [1500, 28672] 27.1 / 18.0.
//  * B = 4, uneven grids: [4200, 8064] 15.7 / 17.1, [4200, 5128] 13.2 / 12.5.
//  * B = 8, x beyond the LDS: [16400, 16000] (uneven) 95.8 / 105.8, [12288, 16000] 72.1 / 63.7.
// An x too large for its buffer descriptor stays on the vector GEMV.
bool gemv_rows_wanted(int N, int K, long long ldx, int B, int dtype) {
  if (B < 1 || B > kLnSlots || ((long long)(B - 1) * ldx + K) * 2 >= (long long)kXPast) return false;
  // bfloat16 rows a little longer than 2 or 3 steps of 256 columns: the last step's wavefront adds
  // one more rounding at the size of the result than the vector GEMV has (error against 64 bits
  // 1.02-1.00 of it for K = 520..584, 1.01-1.00 for 776..832; every other K 0.86-1.00)
  if (dtype == 1 && K > 512 && K < 1024 && K % 256 > 0 && K % 256 < 96) return false;
  if (B == 1) {
    for (int p = 2048; p <= 16384; p *= 2)
      if (abs(K - p) <= p / 64) return false;
    return N > kRowsMany && (K <= 1024 || K > 2048);
  }
  const int n16 = (N + 15) / 16, cus = device_cus();
  const double grid = n16 > cus ? uneven(n16, cus) : 1.0;
  const long long x_bytes = 2LL * B * K;
  if (B <= 4 && rows_skewed(K)) return false;
  if (B <= 4 && N <= kRowsFew) return B >= 3 && (K <= (B == 3 ? 4096 : 6144) || x_bytes > kLdsPerCu);
  if (B == 2) return N > 4096 || abs(K - 16384) > 128;
  if (B == 3) return N <= 4096 || x_bytes > kLdsPerCu || (abs(K - 2048) > 32 && K <= (grid <= kRowsLopsided ? 9216 : 3072));
  if (B == 4) return grid <= kRowsLopsided || K <= 6144 || x_bytes > kLdsPerCu / 2;
  return B <= 6 || grid <= kRowsUneven || x_bytes < kLdsPerCu;
}

// Rows per workgroup: 8 (twice the workgroups, x read as often as W) when 16 would leave more
// than half of the CUs idle or load them unevenly, and on crowded channels (half as many rows at
// a time, twice as much of each); 16 otherwise and on rows too short for that.  us, 8 / 16 rows:
// [1000, 4096] 4.8 / 5.8 at B = 4; [10007, 5128] 19.4 / 20.6 at 2, 23.9 / 23.8 at 8; [6000, 6144] 14.2 /
// 15.7, 17.6 / 18.1; [4096, 16384] 29.1 / 32.5, 31.0 / 32.0; [12288, 8160] 42.4 / 49.4, 47.2 / 53.5; but
// [20480, 5128] 37.8 / 36.2 at 4, [8192, 2048] 9.1 / 8.3, [28672, 264] 13.5 / 8.6.
// bfloat16 rows a little longer than 2 or 3 steps of 512 columns take 16: with 8 the last step's
// wavefront rounds once more at the size of the result (error against 64 bits 1.02 of the vector
// GEMV's at K = 1032, 1.01 at 1088, 1.004 at 1544; with 16 rows 0.99-1.00).
static bool rows_by_8(int N, int K, int dtype) {
  const int n16 = (N + 15) / 16, cus = device_cus();
  if (K < kRowsMinK8) return false;
  if (dtype == 1 && K < 2048 && K % 512 > 0 && K % 512 < 128) return false;
  if (n16 <= cus / 2) return true;
  if (rows_crowded(K) && (n16 > cus || uneven((N + 7) / 8, cus) <= kRowsLopsided)) return true;
  return K >= kRowsLongK && n16 > cus && uneven(n16, cus) > kRowsUneven;
}

hipError_t launch_gemv_rows(GemvParams p, int N, int dtype, int B, hipStream_t stream) {
  if (p.rows <= 0) return hipSuccess;
  if (p.K < 8 || p.K % 8 || B < 1 || B > kLnSlots || p.ln || p.segmajor) return hipErrorInvalidValue;
  if (p.ldx < p.K || ((long long)(B - 1) * p.ldx + p.K) * 2 >= (long long)kXPast) return hipErrorInvalidValue;
  if (rows_by_8(N, p.K, dtype))
    return dtype == 1 ? launch_rows_k<BF16, 8>(p, B, stream) : launch_rows_k<F16, 8>(p, B, stream);
  return dtype == 1 ? launch_rows_k<BF16, 16>(p, B, stream) : launch_rows_k<F16, 16>(p, B, stream);
}

}  // namespace hg
