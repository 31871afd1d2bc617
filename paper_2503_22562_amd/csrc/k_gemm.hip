// bf16 MFMA GEMMs of the layer (QKV, O + residual, gate/up + SwiGLU,
// down + residual): C[M][N] = A[M][K] B[N][K]^T, both operands K-contiguous
// (activations row-major, weights row-major [out][in]), fp32 accumulation.
//
// Tiling: 256 threads = 4 wavefronts in a 2 x 2 arrangement over a
// 128 x 128 output tile; each wave owns 64 x 64 = 4 x 4 MFMA 16x16 tiles.
// K advances in steps of 64 through LDS (rows padded by 16 bytes so the
// 16-byte fragment reads of eight consecutive rows hit distinct banks); the
// next K step is fetched into registers while the current one is multiplied.
// Each MFMA computes a transposed 16x16 block (weights as the A operand), so a
// lane ends up with four consecutive output columns of one row and the
// epilogue stores 8- or 16-byte vectors.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "hb_device.h"
#include "hb_kernels.h"

namespace hb {

namespace {
constexpr int BM = 128, BN = 128, BK = 64, LDSW = BK + 8;  // LDS row width in bf16

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }

template <int EPI>
__global__ __launch_bounds__(256) void gemm_kernel(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t As[BM * LDSW];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * LDSW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * BM;
  const int nb = blockIdx.x;
  const int M = a.M, N = a.N, K = a.K;

  // global -> register staging: 4 x 16 B of A and of B per thread
  u32x4 ra[4], rb[4];
  const u32x4 zero = {0u, 0u, 0u, 0u};
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = tid + 256 * i, row = v >> 3, kk = k0 + ((v & 7) << 3);
      const int gm = m0 + row;
      ra[i] = (gm < M && kk < K) ? ld16(a.A + (size_t)gm * a.lda + kk) : zero;
      int brow;
      bool ok;
      if (EPI == GEMM_SWIGLU) {
        const int c = nb * 64 + (row & 63);
        ok = c < N;
        brow = (row < 64) ? c : N + c;
      } else {
        brow = nb * BN + row;
        ok = brow < N;
      }
      rb[i] = (ok && kk < K) ? ld16(a.B + (size_t)brow * a.ldb + kk) : zero;
    }
  };
  auto sstore = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = tid + 256 * i, row = v >> 3, kk = (v & 7) << 3;
      *reinterpret_cast<u32x4*>(&As[row * LDSW + kk]) = ra[i];
      *reinterpret_cast<u32x4*>(&Bs[row * LDSW + kk]) = rb[i];
    }
  };
  // LDS row of the wave's B fragment ni
  auto brow_lds = [&](int ni) -> int {
    if (EPI == GEMM_SWIGLU) return (ni >> 1) * 64 + wn * 32 + 16 * (ni & 1);
    return wn * 64 + 16 * ni;
  };

  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = (K + BK - 1) / BK;
  gload(0);
  sstore();
  __syncthreads();
  const int fr = lane & 15, fk = (lane >> 4) << 3;
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + 1 < nk) gload((kt + 1) * BK);
#pragma unroll
    for (int kc = 0; kc < BK; kc += 32) {
      bf16x8 af[4], bfr[4];
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
        af[mi] = as_bf16x8(*reinterpret_cast<const u32x4*>(&As[(wm * 64 + 16 * mi + fr) * LDSW + kc + fk]));
#pragma unroll
      for (int ni = 0; ni < 4; ++ni)
        bfr[ni] = as_bf16x8(*reinterpret_cast<const u32x4*>(&Bs[(brow_lds(ni) + fr) * LDSW + kc + fk]));
#pragma unroll
      for (int mi = 0; mi < 4; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) acc[mi][ni] = mfma16x16x32(bfr[ni], af[mi], acc[mi][ni]);
    }
    __syncthreads();
    if (kt + 1 < nk) {
      sstore();
      __syncthreads();
    }
  }

  // epilogue: acc[mi][ni][r] = C[m][n + r], m = row of lane, n = 4 consecutive columns
  const int cq = (lane >> 4) << 2;
#pragma unroll
  for (int mi = 0; mi < 4; ++mi) {
    const int m = m0 + wm * 64 + 16 * mi + fr;
    if (m >= M) continue;
    if (EPI == GEMM_SWIGLU) {
#pragma unroll
      for (int ni = 0; ni < 2; ++ni) {
        const int n = nb * 64 + wn * 32 + 16 * ni + cq;
        if (n >= N) continue;
        const f32x4 gt = acc[mi][ni], up = acc[mi][ni + 2];
        u32x2 o;
        o[0] = pack_bf16x2(silu_f(gt[0]) * up[0], silu_f(gt[1]) * up[1]);
        o[1] = pack_bf16x2(silu_f(gt[2]) * up[2], silu_f(gt[3]) * up[3]);
        st8(reinterpret_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + n, o);
      }
    } else {
#pragma unroll
      for (int ni = 0; ni < 4; ++ni) {
        const int n = nb * BN + wn * 64 + 16 * ni + cq;
        if (n >= N) continue;
        f32x4 c = acc[mi][ni];
        if (EPI == GEMM_RESIDUAL && a.R) {
          if (a.r_f32) {
            const u32x4 r = ld16(reinterpret_cast<const float*>(a.R) + (size_t)m * a.ldr + n);
            for (int j = 0; j < 4; ++j) c[j] += __uint_as_float(r[j]);
          } else {
            const u32x2 r = ld8(reinterpret_cast<const uint16_t*>(a.R) + (size_t)m * a.ldr + n);
            c[0] += bf16_lo(r[0]); c[1] += bf16_hi(r[0]);
            c[2] += bf16_lo(r[1]); c[3] += bf16_hi(r[1]);
          }
        }
        if (EPI == GEMM_RESIDUAL && a.c_f32) {
          u32x4 o = {__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])};
          st16(reinterpret_cast<float*>(a.C) + (size_t)m * a.ldc + n, o);
        } else {
          u32x2 o = {pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])};
          st8(reinterpret_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + n, o);
        }
      }
    }
  }
}
}  // namespace

static void launch_gemm_regstaged(hipStream_t s, const GemmArgs& a) {
  const int ncols = (a.epi == GEMM_SWIGLU) ? 64 : BN;
  dim3 grid((a.N + ncols - 1) / ncols, (a.M + BM - 1) / BM);
  switch (a.epi) {
    case GEMM_RESIDUAL: gemm_kernel<GEMM_RESIDUAL><<<grid, 256, 0, s>>>(a); break;
    default: gemm_kernel<GEMM_SWIGLU><<<grid, 256, 0, s>>>(a); break;
  }
}


// ---------------------------------------------------------------------------
// LDS-pipelined GEMM for K % 64 == 0.
//
// Tile BM x BN = 16 TM WR x 16 TN WC: WR x WC waves (2 x 2, 2 x 4 or 4 x 2)
// each own TM x TN 16x16 MFMA blocks (accumulators in VGPRs: the kernels are
// built with the MFMA VGPR form, so no copies between register files). K advances
// in stages of 64 through a ring of S LDS buffers that global memory fills
// directly (16-byte global-to-LDS loads, no register staging). A 1-KB load
// instruction of a wave fills eight 128-byte rows; inside a row the eight
// 16-byte chunks are XOR-swizzled with the row index, so the fragment reads
// of eight consecutive rows fall into eight different chunk positions.
//
// Software pipeline: a stage is consumed in two K halves of 32 whose MFMA
// operands live in two register sets. While the MFMAs of one half run, the
// fragment reads of the next half are issued between them (the scheduler is
// told the interleave), so LDS latency and bandwidth hide under the matrix
// cores. One barrier per stage, between the halves: after it, the buffer just
// read is refilled with the stage S ahead and the next stage's first half is
// read. Workgroups are numbered so that those sharing a weight tile run on the
// same XCD (one L2); K can be split over workgroups whose fp32 partials a
// second kernel sums in a fixed order.
// ---------------------------------------------------------------------------
namespace gemm_detail {

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lgkm0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// One K stage (64 columns) of the A and B tiles: LA (LB) 1-KB loads fill the
// A (B) tile, 8 rows each; wave w issues loads w, w + NW, w + 2 NW, ...
// (NA / NB slots, the last possibly empty); lane L of a load lands at byte
// 16 L. The loads are buffer loads straight into LDS: the wave-uniform byte
// offset of each slot's 8-row group (ao / bo, plus the stage's K offset) is a
// scalar operand, and the lane's offset inside the group (la / lb) the only
// vector one, so no per-load address registers are needed.
template <int NW, int LA, int LB, int NA, int NB>
__device__ __forceinline__ void issue_stage(uint8_t* base, int a_bytes, __amdgpu_buffer_rsrc_t ra,
                                            __amdgpu_buffer_rsrc_t rb, const uint32_t (&ao)[NA],
                                            const uint32_t (&bo)[NB], uint32_t la, uint32_t lb, int wave,
                                            uint32_t kbytes) {
  typedef __attribute__((address_space(3))) void* lds_ptr;
#pragma unroll
  for (int j = 0; j < NA; ++j)
    if (LA % NW == 0 || j * NW + wave < LA) {
      uint8_t* p = base + (j * NW + wave) * 1024;
      const uint32_t so = ao[j] + kbytes;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr)p, 16, la, so, 0, 0);
    }
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (LB % NW == 0 || j * NW + wave < LB) {
      uint8_t* p = base + a_bytes + (j * NW + wave) * 1024;
      const uint32_t so = bo[j] + kbytes;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_ptr)p, 16, lb, so, 0, 0);
    }
}

// Buffer resource over [p, p + bytes) for raw (unstrided) loads.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Fragment reads of one K half: TM A fragments (16-row blocks 2 KB apart)
// and TN B fragments at the given per-fragment row offsets.
template <int TM, int TN>
__device__ __forceinline__ void read_frags(bf16x8 (&fa)[TM], bf16x8 (&fb)[TN], const uint8_t* ap, const uint8_t* bp,
                                           const int (&broff)[TN]) {
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) fa[mi] = as_bf16x8(*reinterpret_cast<const u32x4*>(ap + mi * 2048));
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) fb[ni] = as_bf16x8(*reinterpret_cast<const u32x4*>(bp + broff[ni]));
}

template <int TM, int TN>
__device__ __forceinline__ void mfma_block(f32x4 (&acc)[TM][TN], const bf16x8 (&fa)[TM], const bf16x8 (&fb)[TN]) {
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = mfma16x16x32(fb[ni], fa[mi], acc[mi][ni]);
}

// Scheduling directive for the region just emitted: NMFMA MFMAs with NREAD
// LDS reads spread evenly between them, an MFMA first (its operands were read
// one K half earlier, so the new reads never delay it).
template <int NREAD, int NMFMA>
__device__ __forceinline__ void interleave_reads() {
  constexpr int per = NMFMA / NREAD > 0 ? NMFMA / NREAD : 1;
  constexpr int groups = NMFMA / per < NREAD ? NMFMA / per : NREAD;
  constexpr int extra = NMFMA - per * groups;
#pragma unroll
  for (int i = 0; i + 1 < groups; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, per, 0);  // `per` MFMAs
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    // then one LDS read
  }
  __builtin_amdgcn_sched_group_barrier(0x008, per, 0);
  __builtin_amdgcn_sched_group_barrier(0x100, NREAD - groups + 1, 0);
  if (extra > 0) __builtin_amdgcn_sched_group_barrier(0x008, extra, 0);
}

// Scheduling directive for the second K half: after the barrier, NLOAD
// global-to-LDS loads (the stage S ahead) and NREAD LDS reads (the next
// stage's first half) each follow an MFMA of this half, loads first, so the
// MFMA pipe keeps running while they issue.
template <int NLOAD, int NREAD, int NMFMA>
__device__ __forceinline__ void interleave_loads_reads() {
  constexpr int ops = NLOAD + NREAD;
  constexpr int per_op = (ops + NMFMA - 1) / NMFMA;  // ops after each MFMA
  constexpr int slots = (ops + per_op - 1) / per_op;
  int loads = NLOAD, reads = NREAD;
#pragma unroll
  for (int i = 0; i < slots; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
    for (int j = 0; j < per_op; ++j) {
      if (loads > 0) {
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        --loads;
      } else if (reads > 0) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        --reads;
      }
    }
  }
  if (NMFMA > slots) __builtin_amdgcn_sched_group_barrier(0x008, NMFMA > slots ? NMFMA - slots : 1, 0);
}

// Whether a tile (TM x TN blocks per wave, NW waves) applies RoPE in its own
// epilogue for head size hd: each wave row must span whole heads (rotation
// partners in one lane), and 8-wave tiles (256 VGPRs per wave) must keep
// their accumulators within 128 VGPRs to leave room for the rotation.
constexpr bool rope_in_tile(int tm, int tn, int nw, int hd) {
  return (16 * tn) % hd == 0 && (nw == 4 || tm * tn <= 32);
}

// Rotation pair (columns j .. j + 3 and j + hd/2 .. of head h) of row m of the
// QKV product: q and k rotated with the row's cos/sin (c4, s4: its columns j ..
// j + 3), q to C, k to the token's pool slot.
__device__ __forceinline__ void store_rotated_pair(const GemmArgs& a, int m, int h, int j, const f32x4& lo,
                                                   const f32x4& hi, const u32x4& c4, const u32x4& s4) {
  const int hd = a.hd, half = hd >> 1;
  float rl[4], rh[4];
  for (int e = 0; e < 4; ++e) {
    const float c = __uint_as_float(c4[e]), sn = __uint_as_float(s4[e]);
    rl[e] = lo[e] * c - hi[e] * sn;
    rh[e] = hi[e] * c + lo[e] * sn;
  }
  const u32x2 wl = {pack_bf16x2(rl[0], rl[1]), pack_bf16x2(rl[2], rl[3])};
  const u32x2 wh = {pack_bf16x2(rh[0], rh[1]), pack_bf16x2(rh[2], rh[3])};
  if (h < a.nq) {
    uint16_t* dst = reinterpret_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + h * hd;
    st8(dst + j, wl);
    st8(dst + half + j, wh);
  } else {
    const int slotm = a.tok_slot[m], slot = slotm & 15;
    uint16_t* kb = a.k_pool + ((size_t)(slotm >> 4) * a.nkv + (h - a.nq)) * 16 * hd;
    st8(kb + k_block_offset(slot, j, hd), wl);
    st8(kb + k_block_offset(slot, half + j, hd), wh);
  }
}

// The same for any head: v goes to the token's pool slot as it is.
__device__ __forceinline__ void store_qkv_pair(const GemmArgs& a, int m, int h, int j, const f32x4& lo,
                                               const f32x4& hi) {
  const int hd = a.hd, half = hd >> 1;
  if (h < a.nq + a.nkv) {
    const float* csr = a.rope_cs + (size_t)m * hd;
    store_rotated_pair(a, m, h, j, lo, hi, ld16(csr + j), ld16(csr + half + j));
    return;
  }
  const int slotm = a.tok_slot[m], slot = slotm & 15, g = h - a.nq - a.nkv;
  uint16_t* vp = a.v_pool + ((size_t)(slotm >> 4) * a.nkv + g) * 16 * hd + ((slot >> 3) * hd + j) * 8 + (slot & 7);
  for (int e = 0; e < 4; ++e) {
    vp[8 * e] = (uint16_t)f32_to_bf16(lo[e]);
    vp[8 * (half + e)] = (uint16_t)f32_to_bf16(hi[e]);
  }
}

// ---------------------------------------------------------------------------
// Epilogues. An accumulator fragment has neighbouring lanes in different rows
// (lane % 16), and a memory instruction whose lanes jump between rows takes a
// cycle per lane instead of one per 64 bytes. Each wave therefore turns its
// 16-row blocks around in LDS (a strip of its own, no barrier:
// wave_lds_order) and stores them row by row, neighbouring lanes
// along a row: 256-512 contiguous bytes per row, with the residual or cos/sin
// loads of the next blocks in flight. 8B, us: QKV with RoPE at M = 2048 108 ->
// 102, with a K split at M = 576 38 -> 36.5 and at M = 822 (TP2 shard) 35.5 ->
// 32; O with its fp32 residual stream at M = 2048 74 -> 71.
// ---------------------------------------------------------------------------
// Floats per row of a staged block of 16 TN columns: 16 bytes of padding keep
// the 16 rows of a column on different banks.
template <int TN>
constexpr int kEpiPitch = 16 * TN + 4;

// Stage one block: lane (row fr, columns 16 ni + 4 fg ..), after the other
// lanes' reads of the block before it and before their reads of this one.
template <int TN>
__device__ __forceinline__ void epi_stage(float* buf, const f32x4 (&acc)[TN], int fr, int fg) {
  wave_lds_order();
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) *reinterpret_cast<f32x4*>(buf + fr * kEpiPitch<TN> + 16 * ni + 4 * fg) = acc[ni];
  wave_lds_order();
}

// Residual operand of one block, four columns per lane and slot j (element
// lane + 64 j of the block's 16 x 4 TN vectors). RK: none (0), bf16 (1) or
// fp32 (2). base is the wave's first row and column; rows past last_row and
// columns past last_col are clamped. Addresses are a wave-uniform base and
// 32-bit byte offsets (the 16 rows of a block span less than 4 GiB).
template <int TN, int RK>
struct EpiResidual {
  std::conditional_t<RK == 1, u32x2, u32x4> v[RK == 0 ? 1 : TN];
  __device__ __forceinline__ void load(const uint8_t* base, uint32_t ld, int row0, int last_row, int last_col, int lane) {
    if constexpr (RK > 0) {
      constexpr uint32_t EB = RK == 2 ? 4 : 2;
      if (row0 > last_row) return;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int e = lane + 64 * j;
        const uint32_t off = (uint32_t)min(e / (4 * TN), last_row - row0) * (ld * EB) +
                             (uint32_t)min(4 * (e % (4 * TN)), last_col) * EB;
        const uint8_t* block = base + (size_t)row0 * (ld * EB);
        if constexpr (RK == 2) v[j] = ld16(block + off);
        else v[j] = ld8(block + off);
      }
    }
  }
  __device__ __forceinline__ f32x4 add(f32x4 c, int j) const {
    if constexpr (RK == 2)
      return c + f32x4{__uint_as_float(v[j][0]), __uint_as_float(v[j][1]), __uint_as_float(v[j][2]), __uint_as_float(v[j][3])};
    else if constexpr (RK == 1)
      return c + f32x4{bf16_lo(v[j][0]), bf16_hi(v[j][0]), bf16_lo(v[j][1]), bf16_hi(v[j][1])};
    else
      return c;
  }
};

// Rows of fp32 (CF) or bf16, plus a residual: out has row stride ld, its rows
// m < M and columns n < N are written. The wave's blocks start at row mw,
// column nw.
template <int TM, int TN, int RK, bool CF>
__device__ __forceinline__ void epi_rows(const GemmArgs& a, float* buf, const f32x4 (&acc)[TM][TN], void* out, uint32_t ld,
                                         int mw, int nw, int lane) {
  if (mw >= a.M || nw >= a.N) return;
  const int fr = lane & 15, fg = lane >> 4;
  constexpr uint32_t EB = CF ? 4 : 2;
  const int last_row = a.M - 1 - mw, last_col = a.N - 4 - nw;
  const uint8_t* rbase = static_cast<const uint8_t*>(a.R) + ((size_t)mw * a.ldr + nw) * (RK == 2 ? 4 : 2);
  uint8_t* obase = static_cast<uint8_t*>(out) + ((size_t)mw * ld + nw) * EB;
  // residual blocks in flight ahead of the one being stored: as many as the
  // registers hold beside the accumulators (a staged block's are free)
  constexpr int AHEAD = TM * TN <= 32 && TN <= 4 ? 2 : 1;
  EpiResidual<TN, RK> r[AHEAD + 1];
#pragma unroll
  for (int p = 0; p < AHEAD; ++p)
    if (p < TM) r[p].load(rbase, a.ldr, 16 * p, last_row, last_col, lane);
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) {
    if (16 * mi > last_row) return;
    epi_stage<TN>(buf, acc[mi], fr, fg);
    if (mi + AHEAD < TM) r[(mi + AHEAD) % (AHEAD + 1)].load(rbase, a.ldr, 16 * (mi + AHEAD), last_row, last_col, lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int e = lane + 64 * j, row = e / (4 * TN), col = 4 * (e % (4 * TN));
      const f32x4 c = r[mi % (AHEAD + 1)].add(*reinterpret_cast<const f32x4*>(buf + row * kEpiPitch<TN> + col), j);
      if (16 * mi + row > last_row || col > last_col) continue;
      uint8_t* o = obase + (size_t)(16 * mi) * (ld * EB) + ((uint32_t)row * (ld * EB) + (uint32_t)col * EB);
      if (CF) st16(o, u32x4{__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])});
      else st8(o, u32x2{pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])});
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Split-K partial sums of gate/up: the wave's first TN / 2 fragments are gate
// columns (at nw), the others up columns (at N + nw), in rows of 2 N.
template <int TM, int TN>
__device__ __forceinline__ void epi_partial_pairs(const GemmArgs& a, float* buf, const f32x4 (&acc)[TM][TN], float* out,
                                                  int mw, int nw, int lane) {
  const int fr = lane & 15, fg = lane >> 4;
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) {
    const int mb = mw + 16 * mi;
    if (mb >= a.M) return;
    epi_stage<TN>(buf, acc[mi], fr, fg);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int e = lane + 64 * j, row = e / (4 * TN), col = 4 * (e % (4 * TN));
      const f32x4 c = *reinterpret_cast<const f32x4*>(buf + row * kEpiPitch<TN> + col);
      const bool up = col >= 8 * TN;
      const int m = mb + row, n = nw + col - (up ? 8 * TN : 0);
      if (m >= a.M || n >= a.N) continue;
      st16(out + (size_t)m * 2 * a.N + (up ? a.N : 0) + n,
           u32x4{__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])});
    }
  }
}

// SwiGLU: silu(gate) * up of fragment pairs (ni, ni + TN / 2), stored from the
// accumulators: half the bytes of the other epilogues and no operand to wait
// for, so turning the blocks around in LDS gains nothing (8B gate/up at M =
// 2048 400 us, 403 us with it).
template <int TM, int TN>
__device__ __forceinline__ void epi_swiglu(const GemmArgs& a, const f32x4 (&acc)[TM][TN], int mw, int nw, int lane) {
  const int fr = lane & 15, fg = lane >> 4;
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) {
    const int m = mw + 16 * mi + fr;
    if (m >= a.M) continue;
#pragma unroll
    for (int ni = 0; ni < TN / 2; ++ni) {
      const int n = nw + 16 * ni + 4 * fg;
      if (n >= a.N) continue;
      const f32x4 gt = acc[mi][ni], up = acc[mi][ni + TN / 2];
      st8(static_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + n,
          u32x2{pack_bf16x2(silu_f(gt[0]) * up[0], silu_f(gt[1]) * up[1]),
                pack_bf16x2(silu_f(gt[2]) * up[2], silu_f(gt[3]) * up[3])});
    }
  }
}

// QKV: the wave's 16 TN columns from nw are whole heads of HD. q and k are
// rotated from the staged block, a lane taking 4 columns of a row and their
// partners HD / 2 further on; v goes to its pool slots from the accumulators
// (neighbouring lanes are neighbouring slots of a dimension).
template <int TM, int TN, int HD>
__device__ __forceinline__ void epi_qkv(const GemmArgs& a, float* buf, const f32x4 (&acc)[TM][TN], int mw, int nw,
                                        int lane) {
  constexpr int HALF = HD / 2, PAIRS = 4 * TN / 2;  // 4-column pairs per row
  const int fr = lane & 15, fg = lane >> 4;
  if (mw >= a.M || nw >= a.N) return;
  const int v_col = (a.nq + a.nkv) * HD;  // first v column
  // cos/sin of a block's pairs, loaded one block ahead
  u32x4 cs[2][TN / 2], sn[2][TN / 2];
  auto load_cs = [&](int mi) {
#pragma unroll
    for (int j = 0; j < TN / 2; ++j) {
      const int e = lane + 64 * j, cj = 4 * ((e % PAIRS) % (HALF / 4));
      const float* csr = a.rope_cs + (size_t)min(mw + 16 * mi + e / PAIRS, a.M - 1) * HD + cj;
      cs[mi & 1][j] = ld16(csr);
      sn[mi & 1][j] = ld16(csr + HALF);
    }
  };
  if (nw < v_col) load_cs(0);
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) {
    const int mb = mw + 16 * mi;
    if (mb >= a.M) return;
    if (nw < v_col) {
      epi_stage<TN>(buf, acc[mi], fr, fg);
      if (mi + 1 < TM) load_cs(mi + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TN / 2; ++j) {
        const int e = lane + 64 * j, row = e / PAIRS, p = e % PAIRS;
        const int hl = p / (HALF / 4), cj = 4 * (p % (HALF / 4));  // head of the wave's, column inside it
        const int m = mb + row, h = nw / HD + hl;
        if (m >= a.M || h >= a.nq + a.nkv) continue;
        const float* b = buf + row * kEpiPitch<TN> + hl * HD + cj;
        store_rotated_pair(a, m, h, cj, *reinterpret_cast<const f32x4*>(b), *reinterpret_cast<const f32x4*>(b + HALF),
                           cs[mi & 1][j], sn[mi & 1][j]);
      }
    }
    if (nw + 16 * TN <= v_col) continue;
    const int m = mb + fr;
    if (m >= a.M) continue;
    const int slotm = a.tok_slot[m], slot = slotm & 15;
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
      const int n = nw + 16 * ni + 4 * fg;
      if (n < v_col || n >= a.N) continue;
      const int g = (n - v_col) / HD, d = n % HD;
      uint16_t* vp = a.v_pool + ((size_t)(slotm >> 4) * a.nkv + g) * 16 * HD + ((slot >> 3) * HD + d) * 8 + (slot & 7);
#pragma unroll
      for (int e = 0; e < 4; ++e) vp[8 * e] = (uint16_t)f32_to_bf16(acc[mi][ni][e]);
    }
  }
}

template <int TM, int TN, int WR, int WC, int S, int EPI>
__global__ __launch_bounds__(64 * WR * WC) void gemm_pipe_kernel(GemmArgs a, int tiles_m, int tiles_n, int ksplit,
                                                                  int kchunk, float* __restrict__ partial) {
  constexpr int NW = WR * WC;
  constexpr int WM = 16 * TM, WN = 16 * TN, BM = WM * WR, BN = WN * WC;
  constexpr int A_BYTES = BM * 128, STAGE_BYTES = (BM + BN) * 128;
  constexpr int LA = BM / 8, LB = BN / 8;                      // 1-KB loads per stage
  constexpr int NA = (LA + NW - 1) / NW, NB = (LB + NW - 1) / NW;  // load slots per wave
  constexpr int LOADS = LA / NW + LB / NW;                     // fewest loads any wave issues
  static_assert(S >= 2 && (S - 2) * LOADS < 64, "stage count");
  static_assert(EPI != GEMM_SWIGLU || (TN % 2 == 0), "gate/up pairs");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

  const int lane = threadIdx.x & 63, wave = wave_id();
  const int wm = wave / WC, wn = wave % WC;
  // XCD-aware tile order: workgroup g runs on XCD g % 8; give each XCD a
  // contiguous run of tiles, M fastest, so tiles sharing weights share an L2.
  const int total = tiles_m * tiles_n * ksplit;
  const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3, q = total >> 3, r = total & 7;
  const int t = (xcd < r) ? xcd * (q + 1) + loc : r * (q + 1) + (xcd - r) * q + loc;
  const int mt = t % tiles_m;
  const int ks = (t / tiles_m) % ksplit;
  const int nt = t / (tiles_m * ksplit);
  const int m0 = mt * BM;
  const int M = a.M, N = a.N;
  const int k_begin = ks * kchunk;
  const int k_end = min(a.K, k_begin + kchunk);
  const int nk = (k_end - k_begin) >> 6;

  // Load offsets (bytes): the first row of each of this wave's 8-row groups
  // is wave-uniform; a lane adds row lrow and its swizzled 16-byte chunk.
  // A rows past M read the caller's padding rows (they only feed outputs that
  // are never stored); B row groups past N are clamped whole (N % 8 == 0).
  const int lrow = lane >> 3;
  const int lchunk = (lane & 7) ^ lrow;
  const uint32_t la = 2u * (uint32_t)(lrow * a.lda + 8 * lchunk), lb = 2u * (uint32_t)(lrow * a.ldb + 8 * lchunk);
  uint32_t ao[NA], bo[NB];
#pragma unroll
  for (int j = 0; j < NA; ++j) ao[j] = 2u * (uint32_t)(m0 + min(8 * (j * NW + wave), BM - 8)) * (uint32_t)a.lda;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int r8 = min(8 * (j * NW + wave), BN - 8);
    int brow;
    if (EPI == GEMM_SWIGLU) {
      const int c = min(nt * (BN / 2) + (r8 % (BN / 2)), N - 8);
      brow = (r8 < BN / 2) ? c : N + c;
    } else {
      brow = min(nt * BN + r8, N - 8);
    }
    bo[j] = 2u * (uint32_t)brow * (uint32_t)a.ldb;
  }
  const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(a.A + k_begin, (uint32_t)kOperandWindow);
  const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(a.B + k_begin, (uint32_t)kOperandWindow);

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Fragment rows of a wave differ by multiples of 8, so the chunk swizzle
  // (row & 7) is that of the lane's own row: every fragment address is one
  // per-lane base plus a compile-time offset. K half kc flips chunk bit 2.
  const int fr = lane & 15, fg = lane >> 4;
  const int swz = ((fg ^ (fr & 7)) << 4);
  const int a_lane = (wm * WM + fr) * 128 + swz;
  const int b_lane = A_BYTES + (EPI == GEMM_SWIGLU ? wn * (WN / 2) : wn * WN) * 128 + fr * 128 + swz;
  int broff[TN];
#pragma unroll
  for (int ni = 0; ni < TN; ++ni)
    broff[ni] = 128 * ((EPI == GEMM_SWIGLU) ? ((ni < TN / 2) ? 16 * ni : BN / 2 + 16 * (ni - TN / 2)) : 16 * ni);

  bf16x8 fa0[TM], fb0[TN], fa1[TM], fb1[TN];

#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s < nk) issue_stage<NW, LA, LB, NA, NB>(smem + s * STAGE_BYTES, A_BYTES, ra, rb, ao, bo, la, lb, wave, s * 128);
  // stage 0 complete: the later prologue stages may stay in flight
  {
    const int pend = min(S, nk) - 1;
    if (S >= 4 && pend >= 3) wait_vmcnt<(S >= 4 ? 3 * LOADS : 0)>();
    else if (S >= 3 && pend >= 2) wait_vmcnt<(S >= 3 ? 2 * LOADS : 0)>();
    else if (pend >= 1) wait_vmcnt<LOADS>();
    else wait_vmcnt<0>();
  }
  __builtin_amdgcn_s_barrier();
  read_frags<TM, TN>(fa0, fb0, smem + a_lane, smem + b_lane, broff);
  __builtin_amdgcn_sched_barrier(0);

  // (the last stage is peeled so that every loop body is one straight block
  // in which reads and MFMAs can be interleaved)
  const int pend = min(S, nk) - 2;
  for (int kt = 0; kt < nk - 1; ++kt) {
    const int buf = kt % S;
    const uint8_t* st = smem + buf * STAGE_BYTES;
    // first K half: read the second half's fragments under the MFMAs
    read_frags<TM, TN>(fa1, fb1, st + (a_lane ^ 64), st + (b_lane ^ 64), broff);
    mfma_block<TM, TN>(acc, fa0, fb0);
    interleave_reads<TM + TN, TM * TN>();
    __builtin_amdgcn_sched_barrier(0);
    // this buffer is fully read (second-half fragments are in registers);
    // the next stage must be complete, the later ones may stay in flight
    wait_lgkm0();
    // the prologue issued min(S, nk) stages and every iteration one more
    // (past the end: the last stage again, into a buffer no later stage
    // reads), so min(S, nk) - 2 stages may stay in flight
    if (pend >= S - 2) wait_vmcnt<(S - 2) * LOADS>();
    else if (S >= 4 && pend >= 2) wait_vmcnt<(S >= 4 ? 2 * LOADS : 0)>();
    else if (S >= 3 && pend >= 1) wait_vmcnt<(S >= 3 ? LOADS : 0)>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    // second K half: refill this buffer with the stage S ahead and read the
    // next stage's first half, both under this half's MFMAs
    issue_stage<NW, LA, LB, NA, NB>(smem + buf * STAGE_BYTES, A_BYTES, ra, rb, ao, bo, la, lb, wave,
                                    min(kt + S, nk - 1) * 128);
    const uint8_t* nx = smem + ((kt + 1) % S) * STAGE_BYTES;
    read_frags<TM, TN>(fa0, fb0, nx + a_lane, nx + b_lane, broff);
    mfma_block<TM, TN>(acc, fa1, fb1);
    interleave_loads_reads<NA + NB, TM + TN, TM * TN>();
    __builtin_amdgcn_sched_barrier(0);
  }
  if (nk > 0) {
    const uint8_t* st = smem + ((nk - 1) % S) * STAGE_BYTES;
    read_frags<TM, TN>(fa1, fb1, st + (a_lane ^ 64), st + (b_lane ^ 64), broff);
    mfma_block<TM, TN>(acc, fa0, fb0);
    interleave_reads<TM + TN, TM * TN>();
    __builtin_amdgcn_sched_barrier(0);
    mfma_block<TM, TN>(acc, fa1, fb1);
  }
  // the loads issued past the end land in LDS before the workgroup ends
  wait_vmcnt<0>();
  const int mw = m0 + wm * WM;
  if (EPI == GEMM_SWIGLU && ksplit == 1) {
    epi_swiglu<TM, TN>(a, acc, mw, nt * (BN / 2) + wn * (WN / 2), lane);
    return;
  }
  // every wave is done with the ring before the epilogue reuses it
  wait_lgkm0();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);

  static_assert(NW * 16 * kEpiPitch<TN> * 4 <= S * STAGE_BYTES, "staging strips fit the ring");
  float* strip = reinterpret_cast<float*>(smem) + wave * 16 * kEpiPitch<TN>;
  if (ksplit > 1) {
    // fp32 partial sums, rows of partial_width(N) columns: the reduce kernel
    // applies the epilogue (SwiGLU: gate at n, up at N + n)
    float* out = partial + (size_t)ks * M * (EPI == GEMM_SWIGLU ? 2 * N : N);
    if (EPI == GEMM_SWIGLU) epi_partial_pairs<TM, TN>(a, strip, acc, out, mw, nt * (BN / 2) + wn * (WN / 2), lane);
    else epi_rows<TM, TN, 0, true>(a, strip, acc, out, N, mw, nt * BN + wn * WN, lane);
    return;
  }
  if (EPI == GEMM_QKV_ROPE) {
    // the planner sends tiles that cannot rotate in-tile (rope_in_tile)
    // through a K split, so their epilogues are not built
    const int nw = nt * BN + wn * WN;
    if constexpr (rope_in_tile(TM, TN, NW, 128)) {
      if (a.hd == 128) epi_qkv<TM, TN, 128>(a, strip, acc, mw, nw, lane);
      else epi_qkv<TM, TN, 64>(a, strip, acc, mw, nw, lane);
    } else if constexpr (rope_in_tile(TM, TN, NW, 64)) {
      if (a.hd == 64) epi_qkv<TM, TN, 64>(a, strip, acc, mw, nw, lane);
    }
  } else if (EPI != GEMM_SWIGLU) {
    const int nw = nt * BN + wn * WN;
    const uint32_t ld = a.ldc;
    if (!a.R) {
      if (a.c_f32) epi_rows<TM, TN, 0, true>(a, strip, acc, a.C, ld, mw, nw, lane);
      else epi_rows<TM, TN, 0, false>(a, strip, acc, a.C, ld, mw, nw, lane);
    } else if (a.r_f32) {
      if (a.c_f32) epi_rows<TM, TN, 2, true>(a, strip, acc, a.C, ld, mw, nw, lane);
      else epi_rows<TM, TN, 2, false>(a, strip, acc, a.C, ld, mw, nw, lane);
    } else {
      if (a.c_f32) epi_rows<TM, TN, 1, true>(a, strip, acc, a.C, ld, mw, nw, lane);
      else epi_rows<TM, TN, 1, false>(a, strip, acc, a.C, ld, mw, nw, lane);
    }
  }
}

// Sum of the split-K partials in split order, then the GEMM's epilogue: for
// the QKV GEMM the RoPE rotation of q and k and the pool scatter of k and v
// (a work item is 4 columns of a row and their rotation partners), for
// gate/up the SwiGLU product, else the residual add and the store.
// Largest K split the planner chooses; the reduce kernels are instantiated
// per split count so that all of a work item's partial loads are in flight
// together.
constexpr int kMaxKSplit = 8;

// Four consecutive fp32 partials summed over the KS splits, in split order.
template <int KS>
__device__ __forceinline__ f32x4 sum_splits(const float* p, size_t stride) {
  u32x4 v[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) v[s] = ld16(p + s * stride);
  f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] += __uint_as_float(v[s][j]);
  return c;
}

template <int EPI, int KS>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a, const float* __restrict__ partial) {
  const int W = (EPI == GEMM_SWIGLU) ? 2 * a.N : a.N;
  const size_t split_stride = (size_t)a.M * W;
  auto sum4 = [&](int m, int n) { return sum_splits<KS>(partial + (size_t)m * W + n, split_stride); };
  const int64_t step = (int64_t)gridDim.x * 256;
  if (EPI == GEMM_QKV_ROPE) {
    // Workgroups [0, M * qk_wgs): one row each, a thread one (q or k head,
    // 4 columns and their rotation partners). The rest: V, one wave item of
    // (kv head, 32 dimensions, 8 consecutive rows) per wave, lane = (row
    // lane % 8, 4 dimensions lane / 8), so the 8 lanes of a dimension write
    // the 8 slots of one 16-byte V group together: a chunk's V lines are
    // written whole by one wave instead of 2 bytes at a time.
    const int hd = a.hd, half = hd / 2, qk_heads = a.nq + a.nkv;
    const int qs = half / 4;  // work items per q/k head (a power of two)
    const int qs_log = __builtin_ctz(qs);
    const int qk_units = qk_heads * qs, qk_wgs = (qk_units + 255) / 256;
    const int b = blockIdx.x;
    if (b < a.M * qk_wgs) {
      const int m = b / qk_wgs, r = (b - m * qk_wgs) * 256 + threadIdx.x;
      if (r >= qk_units) return;
      const int h = r >> qs_log, j = (r & (qs - 1)) * 4;
      store_qkv_pair(a, m, h, j, sum4(m, h * hd + j), sum4(m, h * hd + half + j));
      return;
    }
    const int dblocks = hd / 32;
    const int item = (b - a.M * qk_wgs) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rb = item / (a.nkv * dblocks), rem = item - rb * (a.nkv * dblocks);
    const int g = rem / dblocks, d = 32 * (rem - g * dblocks) + 4 * (lane >> 3);
    const int m = 8 * rb + (lane & 7);
    if (m >= a.M) return;
    const f32x4 c = sum4(m, (qk_heads + g) * hd + d);
    const int slotm = a.tok_slot[m], slot = slotm & 15;
    uint16_t* vp = a.v_pool + ((size_t)(slotm >> 4) * a.nkv + g) * 16 * hd + ((slot >> 3) * hd + d) * 8 + (slot & 7);
    for (int e = 0; e < 4; ++e) vp[8 * e] = (uint16_t)f32_to_bf16(c[e]);
    return;
  }
  const int64_t nvec = (int64_t)a.M * a.N / 4;
  for (int64_t v = blockIdx.x * 256ll + threadIdx.x; v < nvec; v += step) {
    const int64_t e = v * 4;
    const int m = (int)(e / a.N), n = (int)(e - (int64_t)m * a.N);
    f32x4 c = sum4(m, n);
    if (EPI == GEMM_SWIGLU) {
      const f32x4 up = sum4(m, a.N + n);
      const u32x2 o = {pack_bf16x2(silu_f(c[0]) * up[0], silu_f(c[1]) * up[1]),
                       pack_bf16x2(silu_f(c[2]) * up[2], silu_f(c[3]) * up[3])};
      st8(reinterpret_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + n, o);
      continue;
    }
    if (EPI == GEMM_RESIDUAL && a.R) {
      if (a.r_f32) {
        const u32x4 rr = ld16(reinterpret_cast<const float*>(a.R) + (size_t)m * a.ldr + n);
        for (int j = 0; j < 4; ++j) c[j] += __uint_as_float(rr[j]);
      } else {
        const u32x2 rr = ld8(reinterpret_cast<const uint16_t*>(a.R) + (size_t)m * a.ldr + n);
        c[0] += bf16_lo(rr[0]); c[1] += bf16_hi(rr[0]);
        c[2] += bf16_lo(rr[1]); c[3] += bf16_hi(rr[1]);
      }
    }
    if (EPI == GEMM_RESIDUAL && a.c_f32) {
      u32x4 o = {__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])};
      st16(reinterpret_cast<float*>(a.C) + (size_t)m * a.ldc + n, o);
    } else {
      u32x2 o = {pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])};
      st8(reinterpret_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + n, o);
    }
  }
}

// Split-K reduce of the fp32 residual GEMM fused with the RMSNorm that
// follows it: one workgroup per row sums the partials in split order, adds the
// residual, stores the row (fp32) and normalises it into norm_out (bf16), with
// the same element-to-thread mapping and reduction order as the RMSNorm kernel.
template <int MAXV, int KS>
__global__ __launch_bounds__(256) void splitk_reduce_rmsnorm_kernel(GemmArgs a, const float* __restrict__ partial) {
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x, N = a.N;
  const int nvec = N >> 3;
  const size_t split_stride = (size_t)a.M * N;
  float v[MAXV][8];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int vi = tid + 256 * i;
    if (vi < nvec) {
      const float* p = partial + (size_t)row * N + 8 * vi;
      const f32x4 c0 = sum_splits<KS>(p, split_stride), c1 = sum_splits<KS>(p + 4, split_stride);
      float c[8] = {c0[0], c0[1], c0[2], c0[3], c1[0], c1[1], c1[2], c1[3]};
      if (!a.R) {
      } else if (a.r_f32) {
        const float* rr = reinterpret_cast<const float*>(a.R) + (size_t)row * a.ldr + 8 * vi;
        const u32x4 r0 = ld16(rr), r1 = ld16(rr + 4);
        for (int j = 0; j < 4; ++j) { c[j] += __uint_as_float(r0[j]); c[4 + j] += __uint_as_float(r1[j]); }
      } else {
        const u32x4 rr = ld16(reinterpret_cast<const uint16_t*>(a.R) + (size_t)row * a.ldr + 8 * vi);
        for (int j = 0; j < 4; ++j) { c[2 * j] += bf16_lo(rr[j]); c[2 * j + 1] += bf16_hi(rr[j]); }
      }
      float* cr = reinterpret_cast<float*>(a.C) + (size_t)row * a.ldc + 8 * vi;
      st16(cr, u32x4{__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])});
      st16(cr + 4, u32x4{__float_as_uint(c[4]), __float_as_uint(c[5]), __float_as_uint(c[6]), __float_as_uint(c[7])});
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[i][j] = c[j];
        ss += c[j] * c[j];
      }
    }
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  const float tot = red[0] + red[1] + red[2] + red[3];
  const float r = 1.0f / sqrtf(tot / (float)N + a.norm_eps);
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int vi = tid + 256 * i;
    if (vi < nvec) {
      u32x4 gw = ld16(a.norm_g + 8 * vi), o;
      for (int j = 0; j < 4; ++j)
        o[j] = pack_bf16x2(v[i][2 * j] * r * bf16_lo(gw[j]), v[i][2 * j + 1] * r * bf16_hi(gw[j]));
      st16(a.norm_out + (size_t)row * N + 8 * vi, o);
    }
  }
}

}  // namespace gemm_detail

// ---------------------------------------------------------------------------
// Small-batch GEMM (M <= 64): HBM-bound, the weights are streamed once.
//
// A workgroup owns 16 RT weight rows over the whole K, so no partial sums
// leave the chip and the epilogue (RoPE + scatter, SwiGLU, residual) needs no
// second kernel. Its NW waves take the 64-wide K steps round-robin and sum
// their results in LDS at the end, in wave order. Each wave fills a ring of S
// steps of its own (its weight rows and the M activation rows, 8 rows of 128
// bytes per 1-KB global-to-LDS load), so the K loop has no barrier. Short rings
// (two steps from 17 rows on) let several workgroups share a CU, whose loads
// stay in flight while one of them starts or ends. Loading MFMA operands
// straight into registers instead (16 rows of 64 bytes, neighbouring lanes in
// different rows) is not coalesced: gate/up of the 8B layer at M = 16 took
// 61 us that way, against 44.5 us here.
//
// What bounds it: at M <= 16 the HBM stream (8B gate/up at M = 1: 40 us, 5.85
// of the 6.1 TB/s a plain read reaches); above that the activation rows every
// workgroup re-reads from L2, XL KB beside 2 RT KB of weights per step, hence
// the larger row counts of stream_rows. Layer GEMMs at 8B, us, pipelined tiles
// with K split and their reduce -> this kernel (QKV, gate/up, down):
// M = 1 16.1 -> 13.5, 53.2 -> 40.2, 35.7 -> 24.8; M = 32 19.4 -> 15.7,
// 56.6 -> 47.3, 41.4 -> 34.1; M = 64 22.8 -> 18.5, 69.7 -> 55.8, 42.2 -> 42.6.
// ---------------------------------------------------------------------------
namespace gemm_detail {

// LDS bytes of one K step: 2 RT KB of weight rows and the activation rows in
// whole 16-row MFMA tiles (rows past 8 XL are not loaded; they only reach
// outputs that are never stored).
__host__ __device__ constexpr int stream_stage_bytes(int xl, int rt) { return (2 * rt + 2 * ((xl + 1) / 2)) * 1024; }

// Workgroups of 16 rt weight rows (gate/up: N gate and N up rows).
inline int stream_units(const GemmArgs& a, int rt) {
  const int rows = a.epi == GEMM_SWIGLU ? 2 * a.N : a.N;
  return (rows + 16 * rt - 1) / (16 * rt);
}

// First weight row of 8-row group j (0 .. 2 RT - 1) of a unit. Units pair the
// rows whose results meet in the epilogue: gate with up, and the two halves
// of a head's rotation pairs; the first half of a unit's 16 RT rows comes
// from the first region, the second half from the other.
template <int EPI, int RT>
__device__ __forceinline__ int stream_group_row(const GemmArgs& a, int unit, int j) {
  if (EPI == GEMM_SWIGLU || EPI == GEMM_QKV_ROPE) {
    constexpr int HR = 8 * RT;  // rows per region
    const int second = j >= RT, l = 8 * (second ? j - RT : j);
    if (EPI == GEMM_SWIGLU) return (second ? a.N : 0) + unit * HR + l;
    const int half = a.hd >> 1, per = half / HR;  // units per head
    const int h = unit / per, j0 = (unit - h * per) * HR;
    return h * a.hd + j0 + l + (second ? half : 0);
  }
  return min(unit * 16 * RT + 8 * j, a.N - 8);
}

// One 64-wide K step into a wave's ring: 2 RT loads of 8 weight rows, XL of 8
// activation rows (row groups x_rows bytes apart), XOR-swizzled as in the
// pipelined kernel.
template <int XL, int RT>
__device__ __forceinline__ void stream_issue(uint8_t* p, __amdgpu_buffer_rsrc_t rx, __amdgpu_buffer_rsrc_t rw,
                                             const uint32_t (&wo)[2 * RT], uint32_t la, uint32_t lb, uint32_t x_rows,
                                             uint32_t kbytes) {
  typedef __attribute__((address_space(3))) void* lds_ptr;
#pragma unroll
  for (int j = 0; j < 2 * RT; ++j) {
    uint8_t* d = p + j * 1024;
    const uint32_t so = wo[j] + kbytes;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)d, 16, lb, so, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < XL; ++j) {
    uint8_t* d = p + (2 * RT + j) * 1024;
    const uint32_t so = j * x_rows + kbytes;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr)d, 16, la, so, 0, 0);
  }
}

template <int EPI, int XL, int RT, int NW, int S>
__global__ __launch_bounds__(64 * NW) void gemm_stream_kernel(GemmArgs a) {
  constexpr bool PAIR = EPI == GEMM_SWIGLU || EPI == GEMM_QKV_ROPE;
  constexpr int MT = (XL + 1) / 2, LOADS = 2 * RT + XL;
  constexpr int STAGE = stream_stage_bytes(XL, RT), RING = S * STAGE;
  static_assert(RING >= RT * MT * 1024 && (S - 1) * LOADS < 64, "ring");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const int lane = threadIdx.x & 63, wave = wave_id(), unit = blockIdx.x;
  const __amdgpu_buffer_rsrc_t rx = buffer_rsrc(a.A, (uint32_t)kOperandWindow);
  const __amdgpu_buffer_rsrc_t rw = buffer_rsrc(a.B, (uint32_t)kOperandWindow);
  uint8_t* ring = smem + wave * RING;
  const int lrow = lane >> 3, lchunk = (lane & 7) ^ lrow;
  const uint32_t la = 2u * (uint32_t)(lrow * a.lda + 8 * lchunk), lb = 2u * (uint32_t)(lrow * a.ldb + 8 * lchunk);
  uint32_t wo[2 * RT];
#pragma unroll
  for (int j = 0; j < 2 * RT; ++j) wo[j] = 2u * (uint32_t)stream_group_row<EPI, RT>(a, unit, j) * (uint32_t)a.ldb;

  const int nsteps = a.K >> 6, n = (nsteps - wave + NW - 1) / NW;  // this wave's steps: wave, wave + NW, ...
  const uint32_t x_rows = 16u * (uint32_t)a.lda;
  f32x4 acc[RT][MT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[rt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, fg = lane >> 4;
  const int frag = fr * 128 + ((fg ^ (fr & 7)) << 4);
  auto step = [&](int i) {
    const uint8_t* p = ring + (i % S) * STAGE;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 w[RT], x[MT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) w[rt] = as_bf16x8(*reinterpret_cast<const u32x4*>(p + rt * 2048 + (frag ^ (64 * h))));
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        x[mt] = as_bf16x8(*reinterpret_cast<const u32x4*>(p + (RT + mt) * 2048 + (frag ^ (64 * h))));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[rt][mt] = mfma16x16x32(w[rt], x[mt], acc[rt][mt]);
    }
  };
#pragma unroll
  for (int i = 0; i < S; ++i)
    if (i < n) stream_issue<XL, RT>(ring + i * STAGE, rx, rw, wo, la, lb, x_rows, 128u * (uint32_t)(wave + NW * i));
  int i = 0;
  for (; i + S < n; ++i) {
    wait_vmcnt<(S - 1) * LOADS>();
    __builtin_amdgcn_sched_barrier(0);
    step(i);
    wait_lgkm0();
    __builtin_amdgcn_sched_barrier(0);
    stream_issue<XL, RT>(ring + (i % S) * STAGE, rx, rw, wo, la, lb, x_rows, 128u * (uint32_t)(wave + NW * (i + S)));
  }
  wait_vmcnt<0>();
  __builtin_amdgcn_sched_barrier(0);
  for (; i < n; ++i) step(i);
  wait_lgkm0();
  __builtin_amdgcn_sched_barrier(0);
  f32x4* own = reinterpret_cast<f32x4*>(ring);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) own[(rt * MT + mt) * 64 + lane] = acc[rt][mt];
  __syncthreads();
  auto sum = [&](int t, int l) {
    f32x4 c = reinterpret_cast<const f32x4*>(smem)[t * 64 + l];
#pragma unroll
    for (int w = 1; w < NW; ++w) c += reinterpret_cast<const f32x4*>(smem + w * RING)[t * 64 + l];
    return c;
  };
  // an output vector: 4 consecutive weight rows (n .. n + 3) of activation row m
  constexpr int ITEMS = (PAIR ? 32 : 64) * RT * MT;
  for (int it = threadIdx.x; it < ITEMS; it += 64 * NW) {
    if constexpr (PAIR) {
      // first-region vector and its partner in the second region: 8 rows
      // apart in one row tile (RT 1), or RT / 2 row tiles apart
      const int q = RT == 1 ? it & 31 : it & 63, t = RT == 1 ? it >> 5 : it >> 6;
      const int rt = t / MT, mt = t - rt * MT;
      const int m = 16 * mt + (q & 15), l4 = 16 * rt + ((q >> 4) << 2);  // row inside the region
      if (m >= a.M) continue;
      const f32x4 lo = sum(t, q), hi = RT == 1 ? sum(t, q + 32) : sum(t + RT / 2 * MT, q);
      if (EPI == GEMM_SWIGLU) {
        const int n0 = unit * 8 * RT + l4;
        const u32x2 o = {pack_bf16x2(silu_f(lo[0]) * hi[0], silu_f(lo[1]) * hi[1]),
                         pack_bf16x2(silu_f(lo[2]) * hi[2], silu_f(lo[3]) * hi[3])};
        st8(reinterpret_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + n0, o);
      } else {
        const int hd = a.hd, half = hd >> 1, per = half / (8 * RT);
        const int h = unit / per, j = (unit - h * per) * 8 * RT + l4;
        store_qkv_pair(a, m, h, j, lo, hi);
      }
    } else {
      const int t = it >> 6, l = it & 63, rt = t / MT, mt = t - rt * MT;
      const int m = 16 * mt + (l & 15), n0 = unit * 16 * RT + 16 * rt + ((l >> 4) << 2);
      if (m >= a.M || n0 >= a.N) continue;
      f32x4 c = sum(t, l);
      if (EPI == GEMM_RESIDUAL && a.R) {
        if (a.r_f32) {
          const u32x4 rr = ld16(reinterpret_cast<const float*>(a.R) + (size_t)m * a.ldr + n0);
          for (int j = 0; j < 4; ++j) c[j] += __uint_as_float(rr[j]);
        } else {
          const u32x2 rr = ld8(reinterpret_cast<const uint16_t*>(a.R) + (size_t)m * a.ldr + n0);
          c[0] += bf16_lo(rr[0]); c[1] += bf16_hi(rr[0]);
          c[2] += bf16_lo(rr[1]); c[3] += bf16_hi(rr[1]);
        }
      }
      if (EPI == GEMM_RESIDUAL && a.c_f32) {
        const u32x4 o = {__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])};
        st16(reinterpret_cast<float*>(a.C) + (size_t)m * a.ldc + n0, o);
      } else {
        const u32x2 o = {pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])};
        st8(reinterpret_cast<uint16_t*>(a.C) + (size_t)m * a.ldc + n0, o);
      }
    }
  }
}

}  // namespace gemm_detail

namespace {
using namespace gemm_detail;

struct TileCfg {
  int tm, tn, wr, wc, stages;  // per-wave MFMA blocks, wave grid, LDS stages
  // fitted cost (us): one 64-wide K stage of a workgroup that waits for nothing
  // but itself, and a round's start and end
  float stage_us, round_us;
};
// Accumulators and both fragment sets stay within the 256 VGPRs of a wave.
// 8-wave workgroups put two waves on each SIMD; 4-wave ones with LDS rings
// of at most 80 KB run two workgroups per CU. The shapes are the fourteen that
// lose least against the best of 50 (and against the planner before them) over
// the four GEMMs of the 8B and 70B layers and their shards at 15-21 row counts
// from 80 to 2563, 312 cases in all. Small and middle row counts gain from
// rings of three and four stages under 128-column tiles, where the earlier
// shapes had two stages or 256 columns: 8B, us, before -> now: gate/up at M =
// 112 72 -> 53, at M = 160 75 -> 58, down at M = 160 47.6 -> 41.2, O at M = 240
// 26 -> 21; over the 312 cases 7.2 % (geometric mean).
constexpr TileCfg kTiles[] = {
    {4, 4, 2, 2, 4, 0.436f, 0.848f}, {0, 0, 0, 0, 0, 0.f, 0.f},
    {2, 4, 2, 2, 3, 0.281f, 0.004f}, {5, 4, 2, 2, 3, 0.563f, 0.835f},
    {7, 4, 2, 2, 3, 0.689f, 1.627f}, {3, 4, 2, 2, 4, 0.377f, 0.511f},
    {4, 4, 4, 2, 3, 0.709f, 1.276f}, {9, 4, 2, 2, 3, 0.808f, 1.800f},
    {3, 4, 4, 2, 4, 0.533f, 1.639f}, {5, 4, 2, 4, 3, 0.888f, 1.273f},
    {4, 8, 4, 2, 2, 1.393f, 0.622f}, {3, 8, 4, 2, 2, 1.255f, 0.010f},
    {2, 8, 4, 2, 3, 0.756f, 0.942f}, {6, 6, 2, 4, 2, 1.584f, 0.635f},
    {9, 4, 2, 4, 2, 1.556f, 1.374f},
};
constexpr int kNumTiles = (int)(sizeof(kTiles) / sizeof(kTiles[0]));
constexpr int kStreamTile = 1;  // the small-batch kernel's place in the tile numbering (not a pipelined tile)
static_assert(kTiles[kStreamTile].tm == 0, "no pipelined tile");

template <int TM, int TN, int WR, int WC, int ST, int EPI>
void launch_tile(hipStream_t s, const GemmArgs& a, int tiles_m, int tiles_n, int ksplit, int kchunk, float* partial) {
  constexpr int lds = ST * 16 * (TM * WR + TN * WC) * 128;
  static_assert(lds <= 160 * 1024, "LDS");
  static std::atomic<uint64_t> lds_raised{0};
  raise_dynamic_lds(reinterpret_cast<const void*>(&gemm_pipe_kernel<TM, TN, WR, WC, ST, EPI>), lds, lds_raised);
  gemm_pipe_kernel<TM, TN, WR, WC, ST, EPI>
      <<<tiles_m * tiles_n * ksplit, 64 * WR * WC, lds, s>>>(a, tiles_m, tiles_n, ksplit, kchunk, partial);
}

template <int EPI>
void launch_cfg(int idx, hipStream_t s, const GemmArgs& a, int tm, int tn, int ks, int kchunk, float* part) {
  switch (idx) {
    case 0: launch_tile<4, 4, 2, 2, 4, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 2: launch_tile<2, 4, 2, 2, 3, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 3: launch_tile<5, 4, 2, 2, 3, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 4: launch_tile<7, 4, 2, 2, 3, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 5: launch_tile<3, 4, 2, 2, 4, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 6: launch_tile<4, 4, 4, 2, 3, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 7: launch_tile<9, 4, 2, 2, 3, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 8: launch_tile<3, 4, 4, 2, 4, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 9: launch_tile<5, 4, 2, 4, 3, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 10: launch_tile<4, 8, 4, 2, 2, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 11: launch_tile<3, 8, 4, 2, 2, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 12: launch_tile<2, 8, 4, 2, 3, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    case 13: launch_tile<6, 6, 2, 4, 2, EPI>(s, a, tm, tn, ks, kchunk, part); break;
    default: launch_tile<9, 4, 2, 4, 2, EPI>(s, a, tm, tn, ks, kchunk, part); break;
  }
}

// 16-row weight tiles per workgroup (RT) of the small-batch kernel, 0 where the
// pipelined tiles are the better choice.
//
// Above 32 rows the re-read activations outweigh the weights, and long K
// loops amortise what a K split costs the pipelined tiles: 70B gate/up (940
// MB) at M = 32 175 us here against 205 us, at M = 64 209 against 178 us;
// 70B down (470 MB) 103 against 101 and 129 against 103 us; 8B gate/up
// (235 MB) at M = 64 54 against 62-70 us. The line lies between, at 128 MiB
// of weights (gate/up, whose partial sums are twice as wide: 256 MiB). Above
// 16 rows so do weights whose 256-row tiles fill the CUs one and a half times
// without a K split: a 128256-row head at M = 24 204 us here against 191 us
// (at M = 1 160 against 193 us, at M = 16 194 against 193 us).
//
// Forced, the best tile and split would win on this side of the lines too: O, whose
// split does the RMSNorm that here is a launch of its own, at M = 17-64 (8B 19-22
// us here, 17-18 on 64 x 128 tiles with splits of 6 to 8; 70B 44-49, 38-42), 8B down
// at M = 40-64 (40-43, 31-33), a 28K x 5K gate/up at M = 17-32 (59-64, 54), a 96000
// x 8192 head at M = 17-32 (418-433; on tiles 380 at M = 40). The cost model does
// not find those splits: it takes 70B QKV at M = 64 with a split of 2, 50 us, where
// 3 takes 41. Nor is this kernel ahead of the two-stage 64 x 256 tiles it replaced
// everywhere: 70B QKV at M = 17-32 47-49 us, 41-42 with those, O 44-45, 40-41.
//
// RT: the least bytes through the fullest CU, ceil(units / CUs) workgroups of
// 2 RT KB of weights and g KB of activations per step. 8B down at M = 32: RT
// 1 (256 workgroups) 34.1 us, RT 2 (128) 41.1 us; gate/up at M = 48: RT 2
// 54.2 us, RT 4 51.8 us. Up to 16 rows RT 1 is the best or ties (8B gate/up at
// M = 16: 44.5 us, RT 2 45.6 us).
constexpr int kStreamMaxM = 64;
int stream_rows(const GemmArgs& a, int cu_count) {
  const int g = (a.M + 7) / 8;  // 8-row activation groups
  const int64_t rows = (int64_t)(a.epi == GEMM_SWIGLU ? 2 : 1) * a.N, cus = std::max(1, cu_count);
  if (a.M > kStreamMaxM || (a.M > 32 && (int64_t)a.N * a.K * 2 > ((int64_t)128 << 20))) return 0;
  if (a.M > 16 && rows >= 384 * cus) return 0;
  int best = 1;
  int64_t best_kb = INT64_MAX;
  for (int rt = 1; rt <= (g <= 2 ? 1 : g <= 4 ? 2 : 4); rt *= 2) {
    if (rt > 1 && rows % (16 * rt)) break;
    const int64_t kb = ((rows / (16 * rt) + cus - 1) / cus) * (2 * rt + g);
    if (kb < best_kb) best = rt, best_kb = kb;
  }
  return best;
}

template <int EPI, int XL, int RT>
void launch_stream_rt(hipStream_t s, const GemmArgs& a) {
  constexpr int NW = 4, S = XL <= 2 ? 4 : 2, lds = NW * S * stream_stage_bytes(XL, RT);
  static_assert(lds <= 160 * 1024, "LDS");
  static std::atomic<uint64_t> lds_raised{0};
  raise_dynamic_lds(reinterpret_cast<const void*>(&gemm_stream_kernel<EPI, XL, RT, NW, S>), lds, lds_raised);
  gemm_stream_kernel<EPI, XL, RT, NW, S><<<stream_units(a, RT), 64 * NW, lds, s>>>(a);
}

// Activation rows are loaded in groups of 8: up to 8, 16, 24, 32, 48 or 64.
template <int EPI>
void launch_stream(hipStream_t s, const GemmArgs& a, int rt) {
  const int g = (a.M + 7) / 8;
  if (g <= 1) launch_stream_rt<EPI, 1, 1>(s, a);
  else if (g <= 2) launch_stream_rt<EPI, 2, 1>(s, a);
  else if (g <= 3) rt == 1 ? launch_stream_rt<EPI, 3, 1>(s, a) : launch_stream_rt<EPI, 3, 2>(s, a);
  else if (g <= 4) rt == 1 ? launch_stream_rt<EPI, 4, 1>(s, a) : launch_stream_rt<EPI, 4, 2>(s, a);
  else if (g <= 6) rt == 1 ? launch_stream_rt<EPI, 6, 1>(s, a)
                           : rt == 2 ? launch_stream_rt<EPI, 6, 2>(s, a) : launch_stream_rt<EPI, 6, 4>(s, a);
  else rt == 1 ? launch_stream_rt<EPI, 8, 1>(s, a)
               : rt == 2 ? launch_stream_rt<EPI, 8, 2>(s, a) : launch_stream_rt<EPI, 8, 4>(s, a);
}

// The reduce grids fit one wave of workgroups over the chip (about four per
// CU), each thread looping over an equal share of the work items: short
// workgroups in a second, mostly empty round cost more than the loop.
constexpr int kReduceWgs = 1024;

template <int EPI, int KS>
void launch_reduce_ks(hipStream_t s, const GemmArgs& a, const float* partial) {
  if (EPI == GEMM_QKV_ROPE) {
    // q/k rows, then V wave items (kv head, 32 dimensions, 8 rows), 4 per workgroup
    const int qk_units = (a.nq + a.nkv) * (a.hd / 8);
    const int v_items = a.nkv * (a.hd / 32) * ((a.M + 7) / 8);
    splitk_reduce_kernel<EPI, KS><<<a.M * ((qk_units + 255) / 256) + (v_items + 3) / 4, 256, 0, s>>>(a, partial);
  } else {
    const int64_t wgs = ((int64_t)a.M * a.N / 4 + 255) / 256;
    const int64_t per = (wgs + kReduceWgs - 1) / kReduceWgs;
    splitk_reduce_kernel<EPI, KS><<<(int)((wgs + per - 1) / per), 256, 0, s>>>(a, partial);
  }
}

template <int EPI>
void launch_reduce(hipStream_t s, const GemmArgs& a, int ks, const float* partial) {
  static_assert(kMaxKSplit == 8, "one case per split count");
  switch (ks) {
    case 2: launch_reduce_ks<EPI, 2>(s, a, partial); break;
    case 3: launch_reduce_ks<EPI, 3>(s, a, partial); break;
    case 4: launch_reduce_ks<EPI, 4>(s, a, partial); break;
    case 5: launch_reduce_ks<EPI, 5>(s, a, partial); break;
    case 6: launch_reduce_ks<EPI, 6>(s, a, partial); break;
    case 7: launch_reduce_ks<EPI, 7>(s, a, partial); break;
    default: launch_reduce_ks<EPI, 8>(s, a, partial); break;
  }
}

template <int MAXV>
void launch_reduce_rmsnorm(hipStream_t s, const GemmArgs& a, int ks, const float* partial) {
  switch (ks) {
    case 2: splitk_reduce_rmsnorm_kernel<MAXV, 2><<<a.M, 256, 0, s>>>(a, partial); break;
    case 3: splitk_reduce_rmsnorm_kernel<MAXV, 3><<<a.M, 256, 0, s>>>(a, partial); break;
    case 4: splitk_reduce_rmsnorm_kernel<MAXV, 4><<<a.M, 256, 0, s>>>(a, partial); break;
    case 5: splitk_reduce_rmsnorm_kernel<MAXV, 5><<<a.M, 256, 0, s>>>(a, partial); break;
    case 6: splitk_reduce_rmsnorm_kernel<MAXV, 6><<<a.M, 256, 0, s>>>(a, partial); break;
    case 7: splitk_reduce_rmsnorm_kernel<MAXV, 7><<<a.M, 256, 0, s>>>(a, partial); break;
    default: splitk_reduce_rmsnorm_kernel<MAXV, 8><<<a.M, 256, 0, s>>>(a, partial); break;
  }
}
}  // namespace

int gemm_tile_count() { return kNumTiles; }

int partial_width(const GemmArgs& a) { return a.epi == GEMM_SWIGLU ? 2 * a.N : a.N; }

static int tiles_per_cu(const TileCfg& c) {
  const int lds = c.stages * 16 * (c.tm * c.wr + c.tn * c.wc) * 128;
  return (c.wr * c.wc == 4 && 2 * lds <= 160 * 1024) ? 2 : 1;
}

// Cost model (us): workgroups run in rounds of one (two, for small LDS rings)
// per CU. A K stage of a round takes the 4-norm (a smooth maximum) of three
// times: the tile's own (the same with two workgroups on a CU), its
// distinct weight rows at the HBM rate, and all rows its workgroups load at
// the rate the caches fill LDS. A K split adds its reduce (a launch and the
// partials' traffic), a whole K the epilogue's own traffic and, behind the O
// projection, the RMSNorm launch that the reduce would have done. Constants
// fitted to MI355X timings of every shape and split up to 8, each launch with
// its reduce or RMSNorm and the gaps: tiles, QKV and gate/up on those 312 cases;
// O's row and down's last price on the 8B and 70B layers and their TP2 and TP8
// shards at 36 row counts from 66 to 2374 (one layer over and over and four in
// turn), with the layers of hidden 5120 and 3072 left out of the fit. Loss of the
// picks against the best measured choice, mean and worst, fitted / left out: O
// 1.6 % and 19 % / 1.5 % and 9 % (6.5 % and 48 % / 7.6 % and 47 % while an unsplit
// O was not charged its RMSNorm launch: 8B at M = 384 32.0 + 4.9 us on 64 x 128
// tiles where a K split takes less than 29), down 3.0 % and 16 % / 1.4 % and 10 %
// (3.9 % and 33 % / 1.4 % and 10 % while an unsplit down's residual and output
// counted 33 TB/s: TP2 at M = 822 75 us unsplit, 64 with a split of 2), QKV 2.4 %,
// gate/up 0.5 %.
struct EpilogueCost {
  float split_us, split_bytes_us;  // per reduce; per MB of reduce traffic
  float whole_us, whole_bytes_us;  // per whole-K launch; per MB of fp32 output
};
constexpr double kHbmBytesUs = 5.589e6, kFillBytesUs = 16.197e6, kLaterRounds = 1.003, kGemmLaunchUs = 2.684;
constexpr EpilogueCost kEpilogueCost[] = {{1.32, 1 / 5.828, 0, 0},     // QKV + RoPE
                                          {4, 1 / 8.0, 6, 1 / 5.0},    // O, with the RMSNorm behind it
                                          {2.474, 1 / 7.487, 0, 0},    // gate/up
                                          {0, 1 / 5.271, 0, 1 / 5.0},  // down
                                          // LM head: down's without the residual read (a 128256 x 4096 head at
                                          // 17-256 rows within 2 % of the best of 56 choices)
                                          {0, 1 / 5.271, 0, 1 / 10.0}};

static const EpilogueCost& epilogue_cost(const GemmArgs& a) {
  return kEpilogueCost[a.epi == GEMM_QKV_ROPE ? 0 : a.epi == GEMM_SWIGLU ? 2 : a.r_f32 ? 3 : a.ldr ? 1 : 4];
}

static double plan_cost(const GemmArgs& a, const TileCfg& c, int tiles_m, int tiles_n, int ks, int kst, int cus) {
  const int bm = 16 * c.tm * c.wr, bn = 16 * c.tn * c.wc;
  const int slots = cus * tiles_per_cu(c), nwg = tiles_m * tiles_n * ks;
  const int rounds = (nwg + slots - 1) / slots, last = nwg - (rounds - 1) * slots;
  auto stage = [&](int n, double later) {  // one K stage with n workgroups in flight
    const double own = c.stage_us * later;
    const double hbm = (double)((n + tiles_m - 1) / tiles_m) * bn * 128.0 / kHbmBytesUs * later;
    const double fill = (double)n * (bm + bn) * 128.0 / kFillBytesUs;
    auto p4 = [](double x) { return x * x * x * x; };
    return std::sqrt(std::sqrt(p4(own) + p4(hbm) + p4(fill)));
  };
  double us = kGemmLaunchUs + rounds * c.round_us;
  us += kst * (rounds == 1 ? stage(last, 1.0)
                           : stage(slots, 1.0) + (rounds - 2) * stage(slots, kLaterRounds) + stage(last, kLaterRounds));
  const EpilogueCost& e = epilogue_cost(a);
  const double mb = (double)a.M * partial_width(a) * 4.0e-6;
  return us + (ks > 1 ? e.split_us + mb * (2 * ks + 1) * e.split_bytes_us : e.whole_us + mb * e.whole_bytes_us);
}

// The small-batch kernel where it applies and nothing else is forced; else
// the cheapest tile and split by the cost model whose partial sums are at most
// max_partial floats.
static GemmPlan search_plan(const GemmArgs& a, int cu_count, int force_cfg, int force_ksplit, double max_partial) {
  if ((force_cfg < 0 || force_cfg == kStreamTile) && force_ksplit <= 1) {
    const int rt = stream_rows(a, cu_count);
    if (rt > 0) return GemmPlan{kStreamTile, 1, rt, 1, a.K};
  }
  GemmPlan best{-1, 0, 0, 1, 0};
  double best_cost = 1e300;
  const int ksteps = a.K / 64;
  // tiles that cannot rotate in their epilogue take QKV with a K split, whose
  // reduce kernel rotates
  auto fits = [&](const TileCfg& c, int ks) {
    return a.epi != GEMM_QKV_ROPE || ks > 1 || rope_in_tile(c.tm, c.tn, c.wr * c.wc, a.hd);
  };
  const int W = partial_width(a);
  for (int i = 0; i < kNumTiles; ++i) {
    if (i == kStreamTile || (force_cfg >= 0 && i != force_cfg)) continue;
    const TileCfg& c = kTiles[i];
    const int bm = 16 * c.tm * c.wr, bn = 16 * c.tn * c.wc;
    const int ncols = (a.epi == GEMM_SWIGLU) ? bn / 2 : bn;
    const int tm = (a.M + bm - 1) / bm, tn = (a.N + ncols - 1) / ncols;
    for (int ks = 1; ks <= kMaxKSplit; ++ks) {
      if (ks > 1 && ksteps < 4 * ks) break;
      // 7 only when forced: the model has it ahead of 8 where 8 is the faster
      // (8B down, M = 112: 41.2 against 38.6 us; M = 160: 43.9 against 41.2)
      if (force_ksplit > 0 ? ks != force_ksplit : ks == 7) continue;
      if (!fits(c, ks)) continue;
      const int kst = (ksteps + ks - 1) / ks;
      if ((ks - 1) * kst >= ksteps) continue;  // every split gets at least one stage
      if (ks > 1 && (double)ks * a.M * W > max_partial) continue;
      const double cost = plan_cost(a, c, tm, tn, ks, kst, std::max(1, cu_count));
      if (cost < best_cost * 0.999) {
        best_cost = cost;
        best = GemmPlan{i, tm, tn, ks, kst * 64};
      }
    }
  }
  return best;
}

GemmPlan plan_gemm(const GemmArgs& a, int cu_count, int force_cfg, int force_ksplit, double max_partial) {
  if (a.K % 64 != 0 || a.N % 8 != 0) return GemmPlan{-1, 0, 0, 1, 0};
  if (force_cfg >= kNumTiles) force_cfg = -1;
  // a forced shape or split that cannot run this GEMM is relaxed: first the
  // split, then the shape
  GemmPlan p = search_plan(a, cu_count, force_cfg, force_ksplit, max_partial);
  if (p.cfg < 0) p = search_plan(a, cu_count, force_cfg, 0, max_partial);
  if (p.cfg < 0) p = search_plan(a, cu_count, -1, 0, max_partial);
  return p;
}

bool launch_gemm(hipStream_t s, const GemmArgs& a, const GemmPlan& p, float* partial) {
  if (a.M <= 0 || a.N <= 0) return false;
  if (p.cfg < 0) {
    launch_gemm_regstaged(s, a);
    return false;
  }
  if (p.cfg == kStreamTile) {
    switch (a.epi) {
      case GEMM_QKV_ROPE: launch_stream<GEMM_QKV_ROPE>(s, a, p.tiles_n); break;
      case GEMM_RESIDUAL: launch_stream<GEMM_RESIDUAL>(s, a, p.tiles_n); break;
      default: launch_stream<GEMM_SWIGLU>(s, a, p.tiles_n); break;
    }
    return false;
  }
  switch (a.epi) {
    case GEMM_QKV_ROPE: launch_cfg<GEMM_QKV_ROPE>(p.cfg, s, a, p.tiles_m, p.tiles_n, p.ksplit, p.kchunk, partial); break;
    case GEMM_RESIDUAL: launch_cfg<GEMM_RESIDUAL>(p.cfg, s, a, p.tiles_m, p.tiles_n, p.ksplit, p.kchunk, partial); break;
    default: launch_cfg<GEMM_SWIGLU>(p.cfg, s, a, p.tiles_m, p.tiles_n, p.ksplit, p.kchunk, partial); break;
  }
  if (p.ksplit > 1 && a.epi == GEMM_RESIDUAL && a.c_f32 && a.norm_out && a.N % 8 == 0 && a.ldc == a.N &&
      a.N <= 8 * 256 * 8) {
    const int nvec = a.N / 8;
    if (nvec <= 256) launch_reduce_rmsnorm<1>(s, a, p.ksplit, partial);
    else if (nvec <= 1024) launch_reduce_rmsnorm<4>(s, a, p.ksplit, partial);
    else launch_reduce_rmsnorm<8>(s, a, p.ksplit, partial);
    return true;
  }
  if (p.ksplit > 1) {
    switch (a.epi) {
      case GEMM_QKV_ROPE: launch_reduce<GEMM_QKV_ROPE>(s, a, p.ksplit, partial); break;
      case GEMM_SWIGLU: launch_reduce<GEMM_SWIGLU>(s, a, p.ksplit, partial); break;
      default: launch_reduce<GEMM_RESIDUAL>(s, a, p.ksplit, partial); break;
    }
  }
  return false;
}

}  // namespace hb
