// gfx950 decode attention over a KV cache (HeteGen Sec. 2.1, Eq. 1: at a decode
// step the new token's key and value are appended to the cached ones and its
// query attends to every cached position).  Batch b, head h, position pos:
//
//   s_j = (q . K_j) / sqrt(D)  for j <= pos,   out = sum_j softmax(s)_j V_j,
//
// with K_pos, V_pos the new token's key and value (taken from the qkv output and
// written into the cache by this kernel).  Everything is read once, so the kernel
// is bound by HBM bandwidth (2 * (pos + 1) * D * 2 bytes per (b, h)), not by
// arithmetic; no matrix cores.
//
// Split over positions: workgroup (c, h, b) takes the positions of chunk c, D / 8 lanes per
// key or value row (a 16-byte slice each, so a load instruction reads whole rows, coalesced),
// and requests all of its rows at once.  Each wavefront scores its own rows (row sums by DPP,
// the largest by readlane), exponentiates against its own maximum and sums its value rows;
// the wavefronts meet once, in LDS.  The workgroup's (max score, sum of exponentials, weighted
// sum of V) goes to memory and the last workgroup of (b, h) to finish (an arrival counter, no
// waiting) merges the chunks in chunk order and writes the output rounded to the
// activation type.  Every reduction has a fixed order, so results are deterministic.
//
// What bounds it: a chain of memory round trips at one sequence (rows, partial and arrival,
// merge), the bandwidth at eight long ones.  Chunks: 64 positions for short caches, 128 from
// 384 positions on (fewer partials to merge), 256 from 2048; the size depends on the position
// alone, so a batch row's bits do not depend on the batch size.  32 heads of 128, us, 64 / 128
// / 256 positions per chunk: 1 sequence, 201 positions 5.3 / 5.7 / -, 513 7.6 / 6.7 / 7.7, 1001
// 10.0 / 8.0 / 8.5, 4096 - / 21.9 / 16.5; 8 sequences, 513 positions 16.1 / 15.9 / 18.0, 1001
// 28.9 / 26.3 / 26.5, 4096 - / 104 / 95.7 (5.6 TB/s); 8 x 40 heads, 2049 positions - / 63.5 / 59.3.
// With the scores exchanged through LDS, one wavefront's softmax for the workgroup and sums by
// ds_bpermute the same cases took, at 64 (128 from 2048) positions per chunk, 6.4, 9.0, 11.6, 24.2;
// 18.0, 31.6, 111; 69.8.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "attention.h"

namespace hg {
namespace {

constexpr int kThreads = 256;    // kv_copy_kernel
constexpr int kChunk = 64;       // positions per workgroup (256 threads), short caches
constexpr int kMidChunk = 128;   // positions per workgroup (512 threads) from kMidFrom positions on
constexpr int kMidFrom = 384;
constexpr int kLongChunk = 256;  // positions per workgroup (512 threads) from kLongFrom positions on
constexpr int kLongFrom = 2048;
constexpr int kMaxChunks = 64;   // chunks the merge holds in LDS
constexpr int kMaxPositions = kMaxChunks * kLongChunk;  // the longest cache
constexpr int kMergeRegs = 16;   // chunks whose partial outputs the merge requests at once

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Query: dot(k) is a lane's 8 products of q with a key row's 16 bytes, finish() the row's
// score (in the log2 domain) from their sum.  fp16 multiplies pairs (exact products, binary32
// sums) and scales the sum; bf16 scales q first, in binary32: products of its largest values
// would overflow before they are scaled.
struct F16 {
  struct Query {
    uint4 q;
    float scale;
    __device__ __forceinline__ Query(const uint4& v, float s) : q(v), scale(s) {}
    __device__ __forceinline__ float dot(const uint4& k) const {
      float d = 0.f;
      const uint32_t a[4] = {q.x, q.y, q.z, q.w}, b[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        d = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a[i]), __builtin_bit_cast(f16x2, b[i]), d, false);
      return d;
    }
    __device__ __forceinline__ float finish(float sum) const { return sum * scale; }
  };
  static __device__ __forceinline__ float to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
  static __device__ __forceinline__ uint16_t from_f32(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }
};

struct BF16 {
  struct Query {
    float q[8];
    __device__ __forceinline__ Query(const uint4& v, float s) {
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        q[2 * i] = __builtin_bit_cast(float, w[i] << 16) * s;
        q[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xFFFF0000u) * s;
      }
    }
    __device__ __forceinline__ float dot(const uint4& k) const {
      float d = 0.f;
      const uint32_t w[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d = fmaf(q[2 * i], __builtin_bit_cast(float, w[i] << 16), d);
        d = fmaf(q[2 * i + 1], __builtin_bit_cast(float, w[i] & 0xFFFF0000u), d);
      }
      return d;
    }
    __device__ __forceinline__ float finish(float sum) const { return sum; }
  };
  static __device__ __forceinline__ float to_f32(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }
  static __device__ __forceinline__ uint16_t from_f32(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ void unpack8(const uint4& v, float* f) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = T::to_f32((uint16_t)(w[i] & 0xFFFFu));
    f[2 * i + 1] = T::to_f32((uint16_t)(w[i] >> 16));
  }
}

// 16-byte load through the global address space (a generic load would also count
// against the LDS counter); `stream`: read once, non-temporal.
template <bool STREAM>
__device__ __forceinline__ uint4 load16(const uint16_t* p) {
  const __attribute__((address_space(1))) u32x4* g = (const __attribute__((address_space(1))) u32x4*)p;
  const u32x4 v = STREAM ? __builtin_nontemporal_load(g) : *g;
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Partials of the chunk merge cross workgroups on different XCDs (separate L2s):
// they are written and read with sc0 sc1 buffer accesses, which go to memory, so
// no cache-wide writeback or invalidate is needed.  The descriptor base is
// wave-uniform; word 3 is the gfx9 raw-buffer format.
constexpr int kCoherent = 1 | 16;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// v + v of the lane the DPP control names (0xB1 lane ^ 1, 0x4E lane ^ 2, 0x141 mirrored half
// row, 0x140 mirrored row of 16).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// Sum over the LP (8 or 16) lanes that hold one row, in every lane of the row.
template <int LP>
__device__ __forceinline__ float row_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  if (LP == 16) v += dpp<0x140>(v);
  return v;
}

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

__device__ __forceinline__ float exp2_hw(float v) { return __builtin_amdgcn_exp2f(v); }

// A workgroup's chunk: scores in the log2 domain (scale includes log2 e), m = their largest,
// p = 2^(s - m), l = sum of p, o = sum of p V.
template <class T, int D, int CH, int NT>
__global__ __launch_bounds__(NT) void attn_kernel(AttnParams a) {
  constexpr int kWaves = NT / 64;
  constexpr int LP = D / 8;          // lanes per key/value row
  constexpr int PPW = 64 / LP;       // rows per wavefront per round
  constexpr int PPR = PPW * kWaves;  // rows per workgroup per round
  constexpr int ROUNDS = CH / PPR;
  __shared__ __align__(16) float sacc[kWaves * PPW][D + 4];
  __shared__ float sl[kWaves * PPW], sm[kWaves];
  __shared__ float s_m[kMaxChunks], s_l[kMaxChunks];
  __shared__ int s_last;

  const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = lane % LP, grp = lane / LP;
  const int H = a.heads * D;
  const uint16_t* qkv = (const uint16_t*)a.qkv + (size_t)b * a.ldq;
  const uint16_t* knew = qkv + H + h * D;
  const uint16_t* vnew = qkv + 2 * H + h * D;
  const size_t head = ((size_t)b * a.heads + h) * a.max_seq;
  uint16_t* Kc = (uint16_t*)a.kc + head * D;
  uint16_t* Vc = (uint16_t*)a.vc + head * D;
  const int j0 = c * CH;

  // q, then every key and value row of the chunk is requested at once, the keys first
  // (positions past pos reread the new token's row and are masked below; position pos
  // comes from qkv)
  const uint4 qv = load16<false>(qkv + h * D + sub * 8);
  uint4 kr[ROUNDS], vr[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int j = j0 + r * PPR + wave * PPW + grp;
    kr[r] = load16<true>((j >= a.pos ? knew : Kc + (size_t)j * D) + sub * 8);
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int j = j0 + r * PPR + wave * PPW + grp;
    vr[r] = load16<true>((j >= a.pos ? vnew : Vc + (size_t)j * D) + sub * 8);
  }

  // scores of this wavefront's positions, every lane of a row holding its row's
  const typename T::Query q(qv, a.scale);
  float s[ROUNDS], m = -INFINITY;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int j = j0 + r * PPR + wave * PPW + grp;
    s[r] = j <= a.pos ? q.finish(row_sum<LP>(q.dot(kr[r]))) : -INFINITY;
    m = fmaxf(m, s[r]);
  }
  if (LP == 8) m = fmaxf(m, dpp<0x140>(m));  // the two rows of a 16-lane row
  m = fmaxf(fmaxf(lane_value(m, 0), lane_value(m, 16)), fmaxf(lane_value(m, 32), lane_value(m, 48)));

  // weighted sum of its value rows (masked positions have weight 0)
  float l = 0.f, acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const float p = s[r] == -INFINITY ? 0.f : exp2_hw(s[r] - m);
    l += p;
    float v[8];
    unpack8<T>(vr[r], v);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = fmaf(p, v[e], acc[e]);
  }
  const int slot = wave * PPW + grp;
  *(float4*)&sacc[slot][sub * 8] = make_float4(acc[0], acc[1], acc[2], acc[3]);
  *(float4*)&sacc[slot][sub * 8 + 4] = make_float4(acc[4], acc[5], acc[6], acc[7]);
  if (sub == 0) sl[slot] = l;
  if (lane == 0) sm[wave] = m;

  // the chunk holding pos appends the new key and value to the cache
  if (c == a.nchunk - 1 && threadIdx.x < 2 * LP) {
    const int e = threadIdx.x % LP * 8;
    if (threadIdx.x < LP) *(uint4*)(Kc + (size_t)a.pos * D + e) = load16<false>(knew + e);
    else *(uint4*)(Vc + (size_t)a.pos * D + e) = load16<false>(vnew + e);
  }
  __syncthreads();

  // the wavefronts' sums, in order (one without a valid position has m = -inf, weight 0)
  const int t = threadIdx.x;
  float M = sm[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) M = fmaxf(M, sm[w]);
  float o = 0.f, L = 0.f;
  if (t < D) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = sm[w] == -INFINITY ? 0.f : exp2_hw(sm[w] - M);
      float so = 0.f, ss = 0.f;
#pragma unroll
      for (int g = 0; g < PPW; ++g) {
        so += sacc[w * PPW + g][t];
        ss += sl[w * PPW + g];
      }
      o = fmaf(f, so, o);
      L = fmaf(f, ss, L);
    }
  }
  uint16_t* out = (uint16_t*)a.out + (size_t)b * a.ldo + h * D;
  if (a.nchunk == 1) {
    if (t < D) out[t] = T::from_f32(o / L);
    return;
  }

  // partial of this chunk, [m, l, o[0..D)], stored to memory
  const float* part = a.part + ((size_t)(b * a.heads + h) * a.max_chunks) * (D + 2);
  const uint32_t pbytes = (uint32_t)(a.max_chunks * (D + 2) * sizeof(float));
  const auto rs = rsrc(part, pbytes);
  const int mine = c * (D + 2);
  if (t < D) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, o), rs, (mine + 2 + t) * 4, 0,
                                                   kCoherent);
  if (t == 0) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, M), rs, mine * 4, 0, kCoherent);
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, L), rs, (mine + 1) * 4, 0, kCoherent);
  }
  __builtin_amdgcn_s_waitcnt(0);  // this thread's partial stores have completed
  __syncthreads();
  if (t == 0) {
    uint32_t* cnt = a.cnt + (size_t)b * a.heads + h;
    const uint32_t prev = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = prev == (uint32_t)(a.nchunk - 1);
    if (s_last) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next call
  }
  __syncthreads();
  if (!s_last) return;
  // merge, in chunk order: the partials are requested kMergeRegs chunks at a time (one
  // memory round trip per kMergeRegs chunks), m and l through LDS
  auto ld = [&](int i) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, i * 4, 0, kCoherent));
  };
  float ov[kMergeRegs];
  if (t < D) {
#pragma unroll
    for (int u = 0; u < kMergeRegs; ++u) ov[u] = u < a.nchunk ? ld(u * (D + 2) + 2 + t) : 0.f;
  }
  for (int k = t; k < a.nchunk; k += NT) {
    s_m[k] = ld(k * (D + 2));
    s_l[k] = ld(k * (D + 2) + 1);
  }
  __syncthreads();
  if (t < D) {
    float Mx = -INFINITY;
    for (int k = 0; k < a.nchunk; ++k) Mx = fmaxf(Mx, s_m[k]);
    float Ls = 0.f, O = 0.f;
    for (int k0 = 0; k0 < a.nchunk; k0 += kMergeRegs) {
      if (k0 > 0) {
#pragma unroll
        for (int u = 0; u < kMergeRegs; ++u) ov[u] = k0 + u < a.nchunk ? ld((k0 + u) * (D + 2) + 2 + t) : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kMergeRegs; ++u) {
        if (k0 + u < a.nchunk) {
          const float w = exp2_hw(s_m[k0 + u] - Mx);
          Ls = fmaf(s_l[k0 + u], w, Ls);
          O = fmaf(ov[u], w, O);
        }
      }
    }
    out[t] = T::from_f32(O / Ls);
  }
}

template <class T, int CH, int NT>
hipError_t launch_t(const AttnParams& a, int B, hipStream_t s) {
  const dim3 grid(a.nchunk, a.heads, B);
  if (a.head_dim == 128) hipLaunchKernelGGL((attn_kernel<T, 128, CH, NT>), grid, dim3(NT), 0, s, a);
  else hipLaunchKernelGGL((attn_kernel<T, 64, CH, NT>), grid, dim3(NT), 0, s, a);
  return hipGetLastError();
}

template <class T>
hipError_t launch_ch(const AttnParams& a, int ch, int B, hipStream_t s) {
  switch (ch) {
    case kChunk: return launch_t<T, kChunk, 256>(a, B, s);
    case kMidChunk: return launch_t<T, kMidChunk, 512>(a, B, s);
  }
  return launch_t<T, kLongChunk, 512>(a, B, s);
}

// Positions [pos0, pos0 + n) of one layer between the cache and token-major buffers of the
// same values (keys: which = 0, values: 1).  A workgroup moves 4 positions of a group of
// heads: a head's rows of 4 positions are contiguous in the cache (1 KiB at head_dim 128),
// a position's rows of the heads are contiguous in the buffer, so both sides move whole
// lines, kCopyIter 16-byte loads per thread in flight.  Bound by memory: 512 positions of 8
// sequences of 32 heads (D = 128) written and read back take 43 us (268 MB moved; part of the
// read comes from the memory-side cache, a plain copy between buffers that do not fit it runs at
// 4.8 TB/s).
constexpr int kCopyTok = 4;
constexpr int kCopyIter = 4;

template <int D, bool TO_CACHE>
__global__ __launch_bounds__(kThreads) void kv_copy_kernel(KvCopyParams a) {
  constexpr int LP = D / 8;                              // lanes per row
  constexpr int HPI = kThreads / LP / kCopyTok;          // heads per iteration
  const int which = blockIdx.z & 1, b = blockIdx.z >> 1;
  const int sub = threadIdx.x % LP, row = threadIdx.x / LP;
  const int tok = blockIdx.x * kCopyTok + row % kCopyTok;
  const int h0 = blockIdx.y * (HPI * kCopyIter) + row / kCopyTok;
  uint16_t* cache = (uint16_t*)(which ? a.vc : a.kc) + ((size_t)b * a.heads * a.max_seq + a.pos0) * D;
  uint16_t* buf = (uint16_t*)(which ? a.v : a.k) + (size_t)b * a.n * a.heads * D;
  if (tok >= a.n) return;
  uint4 r[kCopyIter];
#pragma unroll
  for (int i = 0; i < kCopyIter; ++i) {
    const int h = h0 + i * HPI;
    if (h >= a.heads) continue;
    const uint16_t* src = TO_CACHE ? buf + ((size_t)tok * a.heads + h) * D : cache + ((size_t)h * a.max_seq + tok) * D;
    r[i] = load16<true>(src + sub * 8);
  }
#pragma unroll
  for (int i = 0; i < kCopyIter; ++i) {
    const int h = h0 + i * HPI;
    if (h >= a.heads) continue;
    uint16_t* dst = TO_CACHE ? cache + ((size_t)h * a.max_seq + tok) * D : buf + ((size_t)tok * a.heads + h) * D;
    *(uint4*)(dst + sub * 8) = r[i];
  }
}

template <int D>
hipError_t launch_kv_copy_d(const KvCopyParams& a, int B, bool to_cache, hipStream_t s) {
  constexpr int HPB = kThreads / (D / 8) / kCopyTok * kCopyIter;  // heads per workgroup
  const dim3 grid((a.n + kCopyTok - 1) / kCopyTok, (a.heads + HPB - 1) / HPB, 2 * B);
  if (to_cache) hipLaunchKernelGGL((kv_copy_kernel<D, true>), grid, dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL((kv_copy_kernel<D, false>), grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace

static int chunk_of(int positions) {
  return positions >= kLongFrom ? kLongChunk : positions >= kMidFrom ? kMidChunk : kChunk;
}
static int chunks_of(int positions) {
  const int ch = chunk_of(positions);
  return (positions + ch - 1) / ch;
}

int attn_max_positions() { return kMaxPositions; }

// the most chunks lie at the end of the cache or just before a larger chunk is taken
int attn_max_chunks(int positions) {
  return std::max({chunks_of(positions), chunks_of(std::min(positions, kMidFrom - 1)),
                   chunks_of(std::min(positions, kLongFrom - 1))});
}

hipError_t launch_attention(AttnParams a, int dtype, int B, hipStream_t stream) {
  if (B < 1 || a.pos < 0 || a.pos >= a.max_seq || (a.head_dim != 64 && a.head_dim != 128) || a.heads < 1)
    return hipErrorInvalidValue;
  const int ch = chunk_of(a.pos + 1);
  a.nchunk = chunks_of(a.pos + 1);
  if (a.nchunk > a.max_chunks || a.nchunk > kMaxChunks) return hipErrorInvalidValue;
  a.scale = 1.4426950408889634f / sqrtf((float)a.head_dim);  // log2 e / sqrt(D)
  return dtype == 1 ? launch_ch<BF16>(a, ch, B, stream) : launch_ch<F16>(a, ch, B, stream);
}

hipError_t launch_kv_copy(const KvCopyParams& a, int B, bool to_cache, hipStream_t stream) {
  if (B < 1 || a.n < 1 || a.pos0 < 0 || a.pos0 + a.n > a.max_seq || (a.head_dim != 64 && a.head_dim != 128) ||
      a.heads < 1)
    return hipErrorInvalidValue;
  return a.head_dim == 128 ? launch_kv_copy_d<128>(a, B, to_cache, stream) : launch_kv_copy_d<64>(a, B, to_cache, stream);
}

}  // namespace hg
