// Bandwidth-bound kernels of the layer: RMSNorm (with the RoPE inputs of the
// QKV epilogue), the KV append copy, and the profiling fills.
#include <algorithm>

#include "hb_device.h"
#include "hb_kernels.h"

namespace hb {

// ---------------------------------------------------------------------------
// RMSNorm: one 256-thread workgroup per token row; each thread holds up to
// MAXV vectors of 8 elements in registers between the reduction and the scale.
// ROPE: the workgroup also writes the token's RoPE cos/sin row and pool slot
// for the QKV epilogue (angles formed and reduced mod 2 pi in fp64, evaluated
// in fp32).
// ---------------------------------------------------------------------------
template <bool F32IN, int MAXV, bool ROPE>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const void* __restrict__ x, const uint16_t* __restrict__ g,
                                                      uint16_t* __restrict__ out, int H, float eps, RopePrep rp) {
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  const int nvec = H >> 3;
  // the row's loads are issued first; the RoPE work below runs while they
  // are in flight
  u32x4 raw[MAXV][F32IN ? 2 : 1];
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int vi = tid + 256 * i;
    if (vi < nvec) {
      if (F32IN) {
        const float* xr = reinterpret_cast<const float*>(x) + (size_t)row * H + 8 * vi;
        raw[i][0] = ld16(xr);
        raw[i][F32IN ? 1 : 0] = ld16(xr + 4);
      } else {
        raw[i][0] = ld16(reinterpret_cast<const uint16_t*>(x) + (size_t)row * H + 8 * vi);
      }
    }
  }
  if (ROPE) {
    const int p = rp.tok_pos[row];
    const int half = rp.hd >> 1;
    if (tid < half) {
      const double ang = (double)p * rp.inv_freq[tid];
      const double r = ang - 6.283185307179586 * rint(ang * 0.15915494309189535);
      float sv, cv;
      sincosf((float)r, &sv, &cv);
      rp.cs[(size_t)row * rp.hd + tid] = cv;
      rp.cs[(size_t)row * rp.hd + half + tid] = sv;
    } else if (tid == half) {
      const int blk = rp.bt[rp.req_bt[rp.tok_req[row]] + (p >> 4)];
      rp.slot[row] = blk * 16 + (p & 15);
    }
  }
  float v[MAXV][8];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int vi = tid + 256 * i;
    if (vi < nvec) {
      if (F32IN) {
        for (int j = 0; j < 4; ++j) {
          v[i][j] = __uint_as_float(raw[i][0][j]);
          v[i][4 + j] = __uint_as_float(raw[i][F32IN ? 1 : 0][j]);
        }
      } else {
        for (int j = 0; j < 4; ++j) { v[i][2 * j] = bf16_lo(raw[i][0][j]); v[i][2 * j + 1] = bf16_hi(raw[i][0][j]); }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) ss += v[i][j] * v[i][j];
    }
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  const float tot = red[0] + red[1] + red[2] + red[3];
  const float r = 1.0f / sqrtf(tot / (float)H + eps);
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int vi = tid + 256 * i;
    if (vi < nvec) {
      u32x4 gw = ld16(g + 8 * vi), o;
      for (int j = 0; j < 4; ++j)
        o[j] = pack_bf16x2(v[i][2 * j] * r * bf16_lo(gw[j]), v[i][2 * j + 1] * r * bf16_hi(gw[j]));
      st16(out + (size_t)row * H + 8 * vi, o);
    }
  }
}

template <int MAXV>
static void launch_rmsnorm_v(hipStream_t s, const void* x, bool x_f32, const uint16_t* g, uint16_t* out, int T, int H,
                             float eps, const RopePrep* rope) {
  const RopePrep rp = rope ? *rope : RopePrep{};
  if (rope) rmsnorm_kernel<false, MAXV, true><<<T, 256, 0, s>>>(x, g, out, H, eps, rp);
  else if (x_f32) rmsnorm_kernel<true, MAXV, false><<<T, 256, 0, s>>>(x, g, out, H, eps, rp);
  else rmsnorm_kernel<false, MAXV, false><<<T, 256, 0, s>>>(x, g, out, H, eps, rp);
}

void launch_rmsnorm(hipStream_t s, const void* x, bool x_f32, const uint16_t* g, uint16_t* out, int T, int H,
                    float eps, const RopePrep* rope) {
  if (T <= 0) return;
  const int nvec = H / 8;
  if (nvec <= 256) launch_rmsnorm_v<1>(s, x, x_f32, g, out, T, H, eps, rope);
  else if (nvec <= 1024) launch_rmsnorm_v<4>(s, x, x_f32, g, out, T, H, eps, rope);
  else launch_rmsnorm_v<8>(s, x, x_f32, g, out, T, H, eps, rope);
}

// ---------------------------------------------------------------------------
// Metadata upload: a 16-byte load per thread from pinned host memory, all in
// flight together, so a batch's metadata takes one round trip over PCIe. In
// place of hipMemcpyAsync on the same stream: 8 decodes of a 70B TP8 shard
// (allocation-free entry) 91.5 -> 78.5 us per call.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void copy_words_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

void launch_copy_words(hipStream_t s, const int32_t* host, int32_t* dev, size_t n) {
  const int nv = (int)((n + 3) / 4);
  if (nv == 0) return;
  copy_words_kernel<<<(nv + 255) / 256, 256, 0, s>>>(reinterpret_cast<const u32x4*>(host), reinterpret_cast<u32x4*>(dev), nv);
}

// The same for a stream under graph capture: the words travel in the kernels'
// arguments, kWordsPerLaunch at a time, so that a replay at any later time
// writes the words of the captured call whatever the staging holds by then.
namespace {
constexpr int kWordsPerLaunch = 960;  // of the 4 KB a launch's arguments may take
struct InlineWords {
  int32_t w[kWordsPerLaunch];
};

__global__ __launch_bounds__(256) void store_words_kernel(InlineWords src, int32_t* __restrict__ dst, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src.w[i];
}
}  // namespace

void launch_store_words(hipStream_t s, const int32_t* host, int32_t* dev, size_t n) {
  for (size_t i = 0; i < n; i += kWordsPerLaunch) {
    InlineWords w{};
    const int m = (int)std::min<size_t>(kWordsPerLaunch, n - i);
    std::copy(host + i, host + i + m, w.w);
    store_words_kernel<<<(m + 255) / 256, 256, 0, s>>>(w, dev + i, m);
  }
}

// ---------------------------------------------------------------------------
// KV append: a copy into the pool's layouts.
// ---------------------------------------------------------------------------
namespace {
// Where an append's block ids come from: by value with the launch, or a device
// copy of them. Entry i is the block of positions 16 (first + i) ..
struct InlineIds {
  int32_t id[kAppendInlineBlocks];
  __device__ int32_t operator[](int i) const { return id[i]; }
};
struct DeviceIds {
  const int32_t* id;
  __device__ int32_t operator[](int i) const { return id[i]; }
};

// 16-byte path. A thread moves the 8 slots of one half block, 8 dimensions of
// one kv head, of K or of V: 8 loads, all in flight together, and 8 stores --
// K as it is (a slot's 8 dimensions are 16 bytes of the pool), V transposed in
// registers (a dimension's 8 slots are). Bound by one memory round trip and
// the copy rate: 3001 tokens of 8 heads x 128 (24.6 MB) 17.8 -> 10.3 us against
// a thread per element with 2-byte stores (which remains for operands that are
// not 16-byte aligned). Half blocks that reach past the appended range write
// single slots.
constexpr int kAppendThreads = 128;

template <int HD, typename Ids>
__global__ __launch_bounds__(kAppendThreads) void append_kv_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                        int ctx, int n, int blocks, Ids ids, int nkv,
                                                        uint16_t* __restrict__ k_pool, uint16_t* __restrict__ v_pool) {
  constexpr int CH = HD / 8;
  const int64_t item = (int64_t)blockIdx.x * kAppendThreads + threadIdx.x;
  const int c = (int)(item % CH), half = (int)(item / CH) & 1;
  const int64_t bh = item / (2 * CH);
  const int bi = (int)(bh / nkv), g = (int)(bh - (int64_t)bi * nkv);
  if (bi >= blocks) return;
  const int t0 = 16 * ((ctx >> 4) + bi) + 8 * half - ctx;  // token of the half's first slot (may lie outside [0, n))
  if (t0 + 8 <= 0 || t0 >= n) return;
  const bool whole = t0 >= 0 && t0 + 8 <= n;
  const size_t base = ((size_t)ids[bi] * nkv + g) * 16 * HD;
  const uint16_t* src = blockIdx.y ? v : k;
  u32x4 r[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) r[t] = ld16(src + ((size_t)min(max(t0 + t, 0), n - 1) * nkv + g) * HD + 8 * c);
  if (blockIdx.y == 0) {
    uint16_t* kb = k_pool + base;
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (whole || (t0 + t >= 0 && t0 + t < n)) st16(kb + k_block_offset(8 * half + t, 8 * c, HD), r[t]);
    return;
  }
  uint16_t* vb = v_pool + base + (size_t)(half * HD + 8 * c) * 8;
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    u32x4 o;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t a = r[2 * w][d >> 1], b = r[2 * w + 1][d >> 1];
      o[w] = (d & 1) ? (a >> 16) | (b & 0xFFFF0000u) : (a & 0xFFFFu) | (b << 16);
    }
    if (whole) {
      st16(vb + 8 * d, o);
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t)
        if (t0 + t >= 0 && t0 + t < n) vb[8 * d + t] = (uint16_t)(o[t >> 1] >> (16 * (t & 1)));
    }
  }
}

// One workgroup per token, a thread per element: operands of any alignment.
template <typename Ids>
__global__ __launch_bounds__(256) void append_kv_bytes_kernel(const uint16_t* __restrict__ k,
                                                              const uint16_t* __restrict__ v, int ctx, Ids ids, int nkv,
                                                              int hd, uint16_t* __restrict__ k_pool,
                                                              uint16_t* __restrict__ v_pool) {
  const int t = blockIdx.x;
  const int p = ctx + t;
  const int blk = ids[(p >> 4) - (ctx >> 4)], slot = p & 15;
  const int n = nkv * hd;
  for (int idx = threadIdx.x; idx < n; idx += 256) {
    const int g = idx / hd, d = idx - g * hd;
    k_pool[((size_t)blk * nkv + g) * 16 * hd + k_block_offset(slot, d, hd)] = k[(size_t)t * n + idx];
    v_pool[((size_t)blk * nkv + g) * 16 * hd + ((slot >> 3) * hd + d) * 8 + (slot & 7)] = v[(size_t)t * n + idx];
  }
}

template <typename Ids>
void launch_append_ids(hipStream_t s, const uint16_t* k, const uint16_t* v, int n_tokens, int ctx, const Ids& ids,
                       int nkv, int hd, uint16_t* k_pool, uint16_t* v_pool) {
  const uintptr_t align = (uintptr_t)k | (uintptr_t)v | (uintptr_t)k_pool | (uintptr_t)v_pool;
  if (align & 15) {
    append_kv_bytes_kernel<<<n_tokens, 256, 0, s>>>(k, v, ctx, ids, nkv, hd, k_pool, v_pool);
    return;
  }
  const int blocks = ((ctx & 15) + n_tokens + 15) / 16;
  const dim3 wgs((unsigned)(((int64_t)blocks * nkv * 2 * (hd / 8) + kAppendThreads - 1) / kAppendThreads), 2);  // K, V
  if (hd == 128) append_kv_kernel<128><<<wgs, kAppendThreads, 0, s>>>(k, v, ctx, n_tokens, blocks, ids, nkv, k_pool, v_pool);
  else append_kv_kernel<64><<<wgs, kAppendThreads, 0, s>>>(k, v, ctx, n_tokens, blocks, ids, nkv, k_pool, v_pool);
}
}  // namespace

void launch_append_kv(hipStream_t s, const uint16_t* k, const uint16_t* v, int n_tokens, int ctx, const int32_t* bt,
                      int nkv, int hd, uint16_t* k_pool, uint16_t* v_pool) {
  if (n_tokens <= 0) return;
  launch_append_ids(s, k, v, n_tokens, ctx, DeviceIds{bt}, nkv, hd, k_pool, v_pool);
}

void launch_append_kv_inline(hipStream_t s, const uint16_t* k, const uint16_t* v, int n_tokens, int ctx,
                             const int32_t* bt, int nkv, int hd, uint16_t* k_pool, uint16_t* v_pool) {
  if (n_tokens <= 0) return;
  InlineIds ids;
  const int n = ((ctx & 15) + n_tokens + 15) / 16;
  for (int i = 0; i < kAppendInlineBlocks; ++i) ids.id[i] = i < n ? bt[i] : 0;
  launch_append_ids(s, k, v, n_tokens, ctx, ids, nkv, hd, k_pool, v_pool);
}

// ---------------------------------------------------------------------------
// Profiling fills: counter-based hash (splitmix64 finaliser) -> uniform in
// [-scale, scale) -> bf16.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ uint16_t rand_bf16(uint64_t seed, uint64_t i, float scale) {
  const uint64_t h = mix64(seed * 0x9E3779B97F4A7C15ull + i);
  const float u = (float)(h >> 40) * (1.0f / 16777216.0f);  // [0,1)
  return (uint16_t)f32_to_bf16((2.f * u - 1.f) * scale);
}

__global__ void fill_random_kernel(uint16_t* p, int64_t n, uint64_t seed, float scale) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = rand_bf16(seed, (uint64_t)i, scale);
}

void launch_fill_random_bf16(hipStream_t s, uint16_t* p, int64_t n, uint64_t seed, float scale) {
  if (n <= 0) return;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  fill_random_kernel<<<(int)blocks, 256, 0, s>>>(p, n, seed, scale);
}

__global__ void fill_blocks_kernel(const int32_t* blocks, int nkv, int hd, uint16_t* k_pool, uint16_t* v_pool,
                                   uint64_t seed) {
  const int64_t per = (int64_t)nkv * 16 * hd;
  const int64_t b = blocks[blockIdx.x];
  for (int64_t i = threadIdx.x; i < per; i += blockDim.x) {
    k_pool[b * per + i] = rand_bf16(seed, (uint64_t)(b * per + i) * 2, 1.7f);
    v_pool[b * per + i] = rand_bf16(seed, (uint64_t)(b * per + i) * 2 + 1, 1.7f);
  }
}

void launch_fill_blocks(hipStream_t s, const int32_t* blocks, int n, int nkv, int hd, uint16_t* k_pool,
                        uint16_t* v_pool, uint64_t seed) {
  if (n <= 0) return;
  fill_blocks_kernel<<<n, 256, 0, s>>>(blocks, nkv, hd, k_pool, v_pool, seed);
}

__global__ void flush_kernel(u32x4* p, int64_t n, uint32_t value) {
  const u32x4 v = {value, value, value, value};
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Grid-stride read of p[0, n); the XOR of the data is stored to *sink only in
// the (never expected) case that it equals a marker, which keeps the loads.
__global__ void flush_read_kernel(const u32x4* __restrict__ p, int64_t n, uint32_t* sink) {
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    acc ^= p[i];
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x5EED5EEDu) *sink = acc[0];
}

void launch_flush(hipStream_t s, void* buf, int64_t bytes, uint32_t value) {
  const int64_t n = bytes / 32;  // 16-byte elements per half
  if (n <= 0) return;
  u32x4* p = reinterpret_cast<u32x4*>(buf);
  flush_kernel<<<4096, 256, 0, s>>>(p, n, value);
  flush_read_kernel<<<4096, 256, 0, s>>>(p + n, n, reinterpret_cast<uint32_t*>(buf));
}

// out[r] = src[rows[r]] for r < n_rows, H bf16 each (H % 8 == 0): token
// embedding lookup and the selection of each request's last row. One
// workgroup per row.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint16_t* __restrict__ src, int64_t n_src,
                                                          const int32_t* __restrict__ rows, int H,
                                                          uint16_t* __restrict__ out) {
  const int r = blockIdx.x;
  const int64_t row = min<int64_t>(max(rows[r], 0), n_src - 1);  // ids outside [0, n_src) read the nearest row
  const u32x4* s4 = reinterpret_cast<const u32x4*>(src + row * H);
  u32x4* d4 = reinterpret_cast<u32x4*>(out + (int64_t)r * H);
  for (int v = threadIdx.x; v < H / 8; v += 256) d4[v] = s4[v];
}

void launch_gather_rows(hipStream_t s, const uint16_t* src, int64_t n_src, const int32_t* rows, int n_rows, int H,
                        uint16_t* out) {
  if (n_rows <= 0) return;
  gather_rows_kernel<<<n_rows, 256, 0, s>>>(src, n_src, rows, H, out);
}

// Index of the largest of V fp32 values per row (the lowest index among
// equal maxima; NaN never wins), V % 8 == 0. One workgroup per row, bound by
// memory latency: each of 1024 threads has eight 16-byte loads in flight, so a
// 128256-wide row takes four round trips (49 rows: 200 -> 15.6 us; 256 threads
// of one 4-byte load each took 501).
constexpr int kArgmaxThreads = 1024, kArgmaxLoads = 8;

__device__ __forceinline__ void argmax_take(float& best, int& bi, float v, int i) {
  if (v > best || (v == best && i < bi)) { best = v; bi = i; }
}

__global__ __launch_bounds__(kArgmaxThreads) void argmax_kernel(const float* __restrict__ x, int V,
                                                                int32_t* __restrict__ out) {
  __shared__ float sv[kArgmaxThreads / 64];
  __shared__ int si[kArgmaxThreads / 64];
  const u32x4* row = reinterpret_cast<const u32x4*>(x + (int64_t)blockIdx.x * V);
  const int nv = V >> 2;
  float best = -INFINITY;
  int bi = 0x7FFFFFFF;
  for (int v0 = threadIdx.x; v0 < nv; v0 += kArgmaxThreads * kArgmaxLoads) {
    u32x4 r[kArgmaxLoads];
#pragma unroll
    for (int k = 0; k < kArgmaxLoads; ++k) r[k] = row[min(v0 + k * kArgmaxThreads, nv - 1)];  // repeats change nothing
#pragma unroll
    for (int k = 0; k < kArgmaxLoads; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        argmax_take(best, bi, __uint_as_float(r[k][j]), 4 * min(v0 + k * kArgmaxThreads, nv - 1) + j);
  }
  // wave: pairwise (value, index) maxima through lane swaps of distance 32..1
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const float ov = __shfl_xor(best, d);
    const int oi = __shfl_xor(bi, d);
    argmax_take(best, bi, ov, oi);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sv[w] = best; si[w] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kArgmaxThreads / 64; ++k) argmax_take(best, bi, sv[k], si[k]);
    out[blockIdx.x] = bi == 0x7FFFFFFF ? 0 : bi;  // a row of NaNs gives 0
  }
}

void launch_argmax(hipStream_t s, const float* x, int n_rows, int V, int32_t* out) {
  if (n_rows <= 0) return;
  argmax_kernel<<<n_rows, kArgmaxThreads, 0, s>>>(x, V, out);
}

}  // namespace hb
