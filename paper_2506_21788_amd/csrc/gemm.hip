// Matrix-core kernels for gfx950 (wave64, MFMA):
//   k_pack    fp32 [in,out] weight slices -> blocks in B-operand order (bf16 or fp32)
//   k_gemm    row tile x (H x H) blocks, A staged through padded LDS, B streamed from L2 in operand
//             order, epilogue (bias / SiLU' / residual adds) applied on the accumulator registers
//   k_wgrad   sum over rows of outer products with split-K partials reduced in a fixed order
//   k_colsum  column sums with the same deterministic two-stage reduction
//
// Operand layouts used below (v_mfma_f32_32x32x16_bf16 and v_mfma_f32_32x32x2_f32):
//   A: lane l holds row (l & 31); bf16: 8 consecutive k at 8*(l>>5); fp32: the single k = (l>>5)
//   B: lane l holds column (l & 31), same k as A
//   D: register v of lane l is element (row 8*(v>>2) + 4*(l>>5) + (v&3), column (l & 31))
// For fp32 the k index inside a block of 8 is permuted (lane half g takes k = 4g..4g+3 over four
// consecutive instructions) so that both operands are fetched as one float4; the permutation is the
// same for A and B and therefore cancels.
#include <type_traits>

#include "devmath.h"
#include "gemm.h"

namespace hgnn {

// ---------------------------------------------------------------------------------------------
// pack
// ---------------------------------------------------------------------------------------------
// c_e of edges first, first + step, ...
__device__ __forceinline__ void pack_cvec(const PackArgs& a, int64_t first, int64_t step) {
  for (int64_t e = first; e < a.E; e += step) {
    const size_t i = (size_t)a.dst_e[e];
    a.cvec[e] = a.alpha * (a.g_v[3 * i] * a.rvec[3 * e] + a.g_v[3 * i + 1] * a.rvec[3 * e + 1] + a.g_v[3 * i + 2] * a.rvec[3 * e + 2]);
  }
}
// element idx < H * H of block b of a group (b == nblocks: the extra block as three bf16 planes)
template <bool BF16>
__device__ __forceinline__ void pack_element(const PackArgs& a, int H, int b, int idx, int grp, long src_grp_stride,
                                             long dst_grp_stride) {
  if (b == a.nblocks) {   // (see split_bf16x3; each plane in the bf16 operand order)
    const PackDesc d = a.d[a.x3_desc];
    const int t = idx & 7, lane = (idx >> 3) & 63, kb = (idx >> 9) % (H / 16), nb = (idx >> 9) / (H / 16);
    const int n = nb * 32 + (lane & 31);
    const int k = kb * 16 + (lane >> 5) * 8 + t;
    const float v = a.src[d.src_off + (long)k * d.sk + (long)n * d.sn];
    const unsigned h = f2bf_bits(v);
    const float r = v - __uint_as_float(h << 16);
    const unsigned m = f2bf_bits(r);
    const float q = r - __uint_as_float(m << 16);
    unsigned short* dst = static_cast<unsigned short*>(a.x3_dst);
    dst[idx] = (unsigned short)h;
    dst[(long)H * H + idx] = (unsigned short)m;
    dst[2L * H * H + idx] = (unsigned short)f2bf_bits(q);
    return;
  }
  const PackDesc d = a.d[b];
  const float* src = a.src + grp * src_grp_stride + d.src_off;
  int n, k;
  if (BF16) {
    const int t = idx & 7, lane = (idx >> 3) & 63, kb = (idx >> 9) % (H / 16), nb = (idx >> 9) / (H / 16);
    n = nb * 32 + (lane & 31);
    k = kb * 16 + (lane >> 5) * 8 + t;
  } else {
    const int t = idx & 3, lane = (idx >> 2) & 63, kb = (idx >> 8) % (H / 8), nb = (idx >> 8) / (H / 8);
    n = nb * 32 + (lane & 31);
    k = kb * 8 + (lane >> 5) * 4 + t;
  }
  const float v = src[(long)k * d.sk + (long)n * d.sn];
  const long o = grp * dst_grp_stride + (long)b * H * H + idx;
  if (BF16) {
    reinterpret_cast<unsigned short*>(a.dst)[o] = (unsigned short)f2bf_bits(v);
  } else {
    reinterpret_cast<float*>(a.dst)[o] = v;
  }
}

template <bool BF16>
__global__ void k_pack(PackArgs a, int H, long src_grp_stride, long dst_grp_stride) {
  const int b = blockIdx.y;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int planes = a.nblocks + (a.x3_dst ? 1 : 0);
  if (b >= planes) {
    const int64_t plane = (int64_t)gridDim.x * blockDim.x;
    pack_cvec(a, (b - planes) * plane + idx, (gridDim.y - planes) * plane);
    return;
  }
  if (idx >= H * H) return;
  pack_element<BF16>(a, H, b, idx, blockIdx.z, src_grp_stride, dst_grp_stride);
}

int32_t launch_pack(hipStream_t st, int H, bool bf16, const PackArgs& a, int groups, long src_grp_stride,
                    long dst_grp_stride_elems) {
  if (a.nblocks <= 0 || groups <= 0) return HGNN_OK;
  HGNN_REQUIRE(groups == 1 || (!a.x3_dst && !a.cvec), HGNN_ERR_BAD_SHAPE, "pack: one group with the extra jobs");
  HGNN_REQUIRE(!bf16 || !a.x3_dst, HGNN_ERR_BAD_SHAPE, "pack: bf16 planes go with fp32 operands");
  ProfScope ps(PT_PACK, st);
  const int xb = (H * H + 255) / 256;
  int64_t eplanes = a.cvec ? (a.E + (int64_t)xb * 256 - 1) / ((int64_t)xb * 256) : 0;
  if (eplanes > 8192) eplanes = 8192;   // (the y dimension ends at 65,535; the rest in a loop)
  dim3 grid(xb, (unsigned)(a.nblocks + (a.x3_dst ? 1 : 0) + eplanes), groups);
  if (bf16) k_pack<true><<<grid, 256, 0, st>>>(a, H, src_grp_stride, dst_grp_stride_elems);
  else k_pack<false><<<grid, 256, 0, st>>>(a, H, src_grp_stride, dst_grp_stride_elems);
  HGNN_LAUNCH_CHECK("k_pack");
  return HGNN_OK;
}

// ---------------------------------------------------------------------------------------------
// row-tile GEMM
// ---------------------------------------------------------------------------------------------
// 32-bit byte offsets from a uniform base (row * pitch fits 24 x 24 -> 32 bits for every node tensor here):
// one full-rate multiply per row instead of 64-bit index arithmetic per element
__device__ __forceinline__ float ld_f32(const float* base, unsigned byte_off) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + byte_off);
}
__device__ __forceinline__ float4 ld_f32x4(const float* base, unsigned byte_off) {
  return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(base) + byte_off);
}
__device__ __forceinline__ void st_f32(float* base, unsigned byte_off, float v) {
  *reinterpret_cast<float*>(reinterpret_cast<char*>(base) + byte_off) = v;
}

// TM_ rows per workgroup tile
template <int H, bool BF16, int TM_ = 64>
struct GemmCfg {
  static constexpr int TM = TM_;
  static constexpr int WC = (H / 32 < 4) ? H / 32 : 4;   // wavefronts side by side over columns
  static constexpr int WR = 4 / WC;                      // and over rows
  static constexpr int WROWS = TM / WR;
  static constexpr int WCOLS = H / WC;
  static constexpr int RB = WROWS / 32;
  static constexpr int CB = WCOLS / 32;
  static constexpr int STRIDE = BF16 ? H + 8 : H + 4;    // LDS row pitch in elements (bank spread)
  static constexpr int CSTR = H + 4;                      // epilogue staging row pitch (floats)
  static constexpr size_t A_BYTES = (size_t)TM * STRIDE * (BF16 ? 2 : 4);
  static constexpr size_t C_BYTES = (size_t)WR * 32 * CSTR * 4;
  static constexpr size_t LDS_BYTES = A_BYTES > C_BYTES ? A_BYTES : C_BYTES;
  static_assert(WROWS % 32 == 0 && (TM * (H / 4)) % 256 == 0, "tile height does not fit the wavefront grid");
};

__device__ __forceinline__ bool tile_of_group(const int32_t* grp_ptr, int S, int TM, int tile, int& grp, int& rbeg,
                                              int& rend) {
  for (int s = 0; s < S; ++s) {
    const int b = grp_ptr[s], e = grp_ptr[s + 1];
    const int nt = (e - b + TM - 1) / TM;
    if (tile < nt) {
      grp = s;
      rbeg = b + tile * TM;
      rend = e;
      return true;
    }
    tile -= nt;
  }
  return false;
}

// The three parts of a row-tile product. They share the workgroup's LDS: the A tile of one k chunk, then (after a
// barrier) the accumulators on their way to row-major stores.
template <int H, bool BF16, int TM>
__device__ __forceinline__ void gemm_stage_a(const GemmArgs& p, int kc, int rbeg, int rend, unsigned char* smem) {
  using C = GemmCfg<H, BF16, TM>;
  const int tid = threadIdx.x;
  {
    // ---- stage the A tile (rows rbeg.., all H columns of chunk kc) into LDS
    const float* __restrict__ A = p.A[kc];
    const int lda = p.lda[kc];
    constexpr int CH = H / 4;
    constexpr int ITER = C::TM * CH / 256;
    constexpr int UN = ITER % 8 == 0 ? 8 : (ITER % 6 == 0 ? 6 : (ITER % 4 == 0 ? 4 : (ITER % 2 == 0 ? 2 : 1)));
    static_assert(ITER % UN == 0, "staging loop must divide evenly");
    for (int it0 = 0; it0 < ITER; it0 += UN) {
      float4 v[UN];
      long gr[UN];
      // all loads of the batch are issued before any of them is used (rows past the end are clamped, then zeroed).
      // The row indices come first, under one uniform branch: with the test inside the loop every load waited
      // for the one before it.
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int r = (tid + (it0 + u) * 256) / CH;
        const int pos = rbeg + r;
        gr[u] = pos < rend ? pos : rend - 1;
      }
      if (p.row_idx) {
#pragma unroll
        for (int u = 0; u < UN; ++u) gr[u] = p.row_idx[gr[u]];
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int c = tid + (it0 + u) * 256;
        const int q = c % CH;
        v[u] = *reinterpret_cast<const float4*>(A + gr[u] * lda + q * 4);
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int c = tid + (it0 + u) * 256;
        const int r = c / CH, q = c - r * CH;
        float4 w = v[u];
        if (p.a_silu) {
          w.x = silu_f(w.x); w.y = silu_f(w.y); w.z = silu_f(w.z); w.w = silu_f(w.w);
        }
        if (rbeg + r >= rend) w = make_float4(0.f, 0.f, 0.f, 0.f);
        if (BF16) {
          uint2 o;
          o.x = pack_bf16x2(w.x, w.y);
          o.y = pack_bf16x2(w.z, w.w);
          *reinterpret_cast<uint2*>(smem + ((size_t)r * C::STRIDE + q * 4) * 2) = o;
        } else {
          *reinterpret_cast<float4*>(smem + ((size_t)r * C::STRIDE + q * 4) * 4) = w;
        }
      }
    }
  }
}

template <int H, bool BF16, int TM>
__device__ __forceinline__ void gemm_multiply(const GemmArgs& p, int kc, int cb, int grp, const unsigned char* smem,
                                              f32x16_t (&acc)[GemmCfg<H, BF16, TM>::RB][GemmCfg<H, BF16, TM>::CB]) {
  using C = GemmCfg<H, BF16, TM>;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: fragment offsets stay in scalar registers
  const int wr = wave / C::WC, wc = wave % C::WC;
  {
    // ---- multiply. All workgroups run this loop at about the same time over the same packed block: each starts at
    // a different k step so that they do not all ask the same L2 lines at once.
    const int krot = blockIdx.x * 5;
    const long bblk0 = grp * p.grp_blk_stride + p.blk[kc][cb];
    if (BF16) {
      // B fragments D steps ahead in a register ring, through buffer loads (resource and fragment offset in scalar
      // registers, one per-lane offset register); A fragments one step ahead. With each load next to its use the
      // loop was a chain of L2 round trips, one per step. The scheduling barrier keeps the refills where they are.
      constexpr int NKB = H / 16;
      constexpr int D = NKB < 4 ? NKB : 4;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<char*>(reinterpret_cast<const char*>(p.B)) + bblk0 * (long)(H * H * 2), 0, H * H * 2, 0x00020000);
      unsigned lo = lane * 16u;
      unsigned ao = (unsigned)(((wr * C::WROWS + (lane & 31)) * C::STRIDE + (lane >> 5) * 8) * 2);
      asm volatile("" : "+v"(lo), "+v"(ao));   // kept as one register each: not folded into per-step addresses
      bf16x8_t b[D][C::CB], a[2][C::RB];
      auto load_b = [&](int kk, bf16x8_t (&o)[C::CB]) {
        const int kb = (kk + krot) & (NKB - 1);
#pragma unroll
        for (int j = 0; j < C::CB; ++j)
          o[j] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rs, lo, ((wc * C::CB + j) * NKB + kb) * 1024, 0));
      };
      auto load_a = [&](int kk, bf16x8_t (&o)[C::RB]) {
        const int kb = (kk + krot) & (NKB - 1);
#pragma unroll
        for (int i = 0; i < C::RB; ++i)
          o[i] = *reinterpret_cast<const bf16x8_t*>(smem + ao + (i * 32 * C::STRIDE + kb * 16) * 2);
      };
#pragma unroll
      for (int d = 0; d < D; ++d) load_b(d, b[d]);
      load_a(0, a[0]);
#pragma unroll
      for (int kk = 0; kk < NKB; ++kk) {
        if (kk + 1 < NKB) load_a(kk + 1, a[(kk + 1) & 1]);
#pragma unroll
        for (int j = 0; j < C::CB; ++j)
#pragma unroll
          for (int i = 0; i < C::RB; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk & 1][i], b[kk % D][j], acc[i][j], 0, 0, 0);
        if (kk + D < NKB) load_b(kk + D, b[kk % D]);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      // the same ring for fp32 operands (four steps of 8 k ahead; A fragments one step ahead)
      constexpr int NKB = H / 8;
      constexpr int D = 4;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<char*>(reinterpret_cast<const char*>(p.B)) + bblk0 * (long)(H * H * 4), 0, H * H * 4, 0x00020000);
      unsigned lo = lane * 16u;
      unsigned ao = (unsigned)(((wr * C::WROWS + (lane & 31)) * C::STRIDE + (lane >> 5) * 4) * 4);
      asm volatile("" : "+v"(lo), "+v"(ao));
      typedef float f32x4v_t __attribute__((ext_vector_type(4)));
      f32x4v_t b[D][C::CB], a[2][C::RB];
      auto load_b = [&](int kk, f32x4v_t (&o)[C::CB]) {
        const int kb = (kk + krot) & (NKB - 1);
#pragma unroll
        for (int j = 0; j < C::CB; ++j)
          o[j] = __builtin_bit_cast(f32x4v_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rs, lo, ((wc * C::CB + j) * NKB + kb) * 1024, 0));
      };
      auto load_a = [&](int kk, f32x4v_t (&o)[C::RB]) {
        const int kb = (kk + krot) & (NKB - 1);
#pragma unroll
        for (int i = 0; i < C::RB; ++i)
          o[i] = *reinterpret_cast<const f32x4v_t*>(smem + ao + (i * 32 * C::STRIDE + kb * 8) * 4);
      };
#pragma unroll
      for (int d = 0; d < D; ++d) load_b(d, b[d]);
      load_a(0, a[0]);
#pragma unroll
      for (int kk = 0; kk < NKB; ++kk) {
        if (kk + 1 < NKB) load_a(kk + 1, a[(kk + 1) & 1]);
#pragma unroll
        for (int j = 0; j < C::CB; ++j)
#pragma unroll
          for (int i = 0; i < C::RB; ++i) {
            const f32x4v_t av = a[kk & 1][i], bv = b[kk % D][j];
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, bv.x, acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, bv.y, acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, bv.z, acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, bv.w, acc[i][j], 0, 0, 0);
          }
        if (kk + D < NKB) load_b(kk + D, b[kk % D]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// KEEP: the finished values (through silu when keep_silu is set; zeros in rows past the end) also go, in the layout
// of an A tile, to `keep`, which must not overlap `smem`: the next product of a chain takes them from there.
template <int H, bool BF16, int TM, bool KEEP>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& p, int cb, int grp, int rbeg, int rend,
                                              f32x16_t (&acc)[GemmCfg<H, BF16, TM>::RB][GemmCfg<H, BF16, TM>::CB],
                                              unsigned char* smem, unsigned char* keep, int keep_silu) {
  using C = GemmCfg<H, BF16, TM>;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave / C::WC, wc = wave % C::WC;
  // ---- epilogue: the accumulators go through LDS, one 32-row block per wavefront row at a time, so that the
  // auxiliary operands and C are accessed row-major with 16-byte loads and stores (few, wide, whole cache lines)
  const bool use_bias = p.bias && ((p.bias_cb_mask >> cb) & 1);
  const bool pair_out = C::CB == 2 && ((p.pair_cb_mask >> cb) & 1);
  const bool use_add = p.add1 && ((p.add1_cb_mask >> cb) & 1);
  constexpr int CH = H / 4;                 // 4-column chunks per row
  constexpr int PROWS = C::WR * 32;         // rows per pass
  constexpr int RSTEP = 256 / CH;           // rows swept by the 256 threads at once
  constexpr int NCH = PROWS / RSTEP;        // chunks per thread and pass
  float* cst = reinterpret_cast<float*>(smem);
  const int q = tid % CH, r0 = tid / CH;
  float4 bv = make_float4(0.f, 0.f, 0.f, 0.f);
  if (use_bias && !pair_out) bv = *reinterpret_cast<const float4*>(p.bias + grp * p.grp_bias_stride + q * 4);
#pragma unroll
  for (int i = 0; i < C::RB; ++i) {
    __syncthreads();   // nobody reads the A tile (or the previous pass) any more
#pragma unroll
    for (int j = 0; j < C::CB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        cst[(wr * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * C::CSTR + wc * C::WCOLS + j * 32 + (lane & 31)] = acc[i][j][v];
    __syncthreads();
    if (pair_out) {
      if constexpr (C::CB == 2) {
        // bf16 pairs: word w = wc'*32 + x' of a row holds columns wc'*64 + x' and wc'*64 + 32 + x'
        constexpr int WCH = H / 8;          // 4-word chunks per row
        constexpr int WSTEP = 256 / WCH;
        const int qw = tid % WCH, rw0 = tid / WCH;
        const int c_lo = (qw * 4 / 32) * 64 + (qw * 4) % 32;
        float4 b_lo = make_float4(0.f, 0.f, 0.f, 0.f), b_hi = b_lo;
        if (use_bias) {
          b_lo = *reinterpret_cast<const float4*>(p.bias + grp * p.grp_bias_stride + c_lo);
          b_hi = *reinterpret_cast<const float4*>(p.bias + grp * p.grp_bias_stride + c_lo + 32);
        }
#pragma unroll
        for (int k = 0; k < PROWS / WSTEP; ++k) {
          const int sr = rw0 + k * WSTEP;
          const int pos = rbeg + (sr / 32) * C::WROWS + i * 32 + (sr % 32);
          if (pos < rend) {
            const long gr = p.row_idx ? p.row_idx[pos] : pos;
            const float4 lo = *reinterpret_cast<const float4*>(cst + sr * C::CSTR + c_lo);
            const float4 hi = *reinterpret_cast<const float4*>(cst + sr * C::CSTR + c_lo + 32);
            uint4 o;
            o.x = pack_bf16x2((lo.x + b_lo.x) * p.pair_scale, (hi.x + b_hi.x) * p.pair_scale);
            o.y = pack_bf16x2((lo.y + b_lo.y) * p.pair_scale, (hi.y + b_hi.y) * p.pair_scale);
            o.z = pack_bf16x2((lo.z + b_lo.z) * p.pair_scale, (hi.z + b_hi.z) * p.pair_scale);
            o.w = pack_bf16x2((lo.w + b_lo.w) * p.pair_scale, (hi.w + b_hi.w) * p.pair_scale);
            *reinterpret_cast<uint4*>(p.Cpair + gr * p.ldpair + p.pair_off[cb] + qw * 4) = o;
          }
        }
      }
    } else {
      const int gcol = cb * H + q * 4;
      long grow[NCH];
      bool ok[NCH];
      float4 mv[NCH], a1[NCH], a2[NCH];
      // every auxiliary load of the pass is issued before any result is stored (rows past the end are clamped)
      // (each kind of operand under one uniform branch around its loads, not one branch per load)
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int sr = r0 + k * RSTEP;
        const int pos = rbeg + (sr / 32) * C::WROWS + i * 32 + (sr % 32);
        ok[k] = pos < rend;
        grow[k] = ok[k] ? pos : rend - 1;
      }
      if (p.row_idx) {
#pragma unroll
        for (int k = 0; k < NCH; ++k) grow[k] = p.row_idx[grow[k]];
      }
      if (p.mul) {
#pragma unroll
        for (int k = 0; k < NCH; ++k) mv[k] = *reinterpret_cast<const float4*>(p.mul + grow[k] * p.ldmul + gcol);
      }
      if (use_add) {
#pragma unroll
        for (int k = 0; k < NCH; ++k) a1[k] = *reinterpret_cast<const float4*>(p.add1 + grow[k] * p.ldadd1 + gcol);
      }
      if (p.add2) {
#pragma unroll
        for (int k = 0; k < NCH; ++k) a2[k] = *reinterpret_cast<const float4*>(p.add2 + grow[k] * p.ldadd2 + gcol);
      }
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int sr = r0 + k * RSTEP;
        float4 x = *reinterpret_cast<const float4*>(cst + sr * C::CSTR + q * 4);
        x.x += bv.x; x.y += bv.y; x.z += bv.z; x.w += bv.w;
        if (p.mul) {
          if (p.mul_is_z) {
            x.x *= dsilu_f(mv[k].x); x.y *= dsilu_f(mv[k].y); x.z *= dsilu_f(mv[k].z); x.w *= dsilu_f(mv[k].w);
          } else {
            x.x *= mv[k].x; x.y *= mv[k].y; x.z *= mv[k].z; x.w *= mv[k].w;
          }
        }
        if (use_add) { x.x += a1[k].x; x.y += a1[k].y; x.z += a1[k].z; x.w += a1[k].w; }
        if (p.add2) { x.x += a2[k].x; x.y += a2[k].y; x.z += a2[k].z; x.w += a2[k].w; }
        if (ok[k]) *reinterpret_cast<float4*>(p.C + grow[k] * p.ldc + gcol) = x;
        if constexpr (KEEP) {
          float4 y = x;
          if (keep_silu) { y.x = silu_f(y.x); y.y = silu_f(y.y); y.z = silu_f(y.z); y.w = silu_f(y.w); }
          if (!ok[k]) y = make_float4(0.f, 0.f, 0.f, 0.f);
          const int trow = (sr / 32) * C::WROWS + i * 32 + (sr % 32);   // row of the tile
          if (BF16) {
            uint2 o;
            o.x = pack_bf16x2(y.x, y.y);
            o.y = pack_bf16x2(y.z, y.w);
            *reinterpret_cast<uint2*>(keep + ((size_t)trow * C::STRIDE + q * 4) * 2) = o;
          } else {
            *reinterpret_cast<float4*>(keep + ((size_t)trow * C::STRIDE + q * 4) * 4) = y;
          }
        }
      }
    }
  }
}

template <int H, bool BF16, int TM>
__global__ void __launch_bounds__(256, TM <= 32 ? 4 : 2) k_gemm(GemmArgs p) {
  using C = GemmCfg<H, BF16, TM>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int cb = blockIdx.y;
  int grp = 0, rbeg, rend;
  if (p.grp_ptr) {
    if (!tile_of_group(p.grp_ptr, p.S, C::TM, blockIdx.x, grp, rbeg, rend)) return;
  } else {
    rbeg = blockIdx.x * C::TM;
    rend = p.M;
    if (rbeg >= rend) return;
  }
  f32x16_t acc[C::RB][C::CB];
#pragma unroll
  for (int i = 0; i < C::RB; ++i)
#pragma unroll
    for (int j = 0; j < C::CB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  for (int kc = 0; kc < p.nkc; ++kc) {
    if (kc) __syncthreads();
    gemm_stage_a<H, BF16, TM>(p, kc, rbeg, rend, smem);
    __syncthreads();
    gemm_multiply<H, BF16, TM>(p, kc, cb, grp, smem, acc);
  }
  gemm_epilogue<H, BF16, TM, false>(p, cb, grp, rbeg, rend, acc, smem, nullptr, 0);
}

// Two products in a row on one row tile, the second one taking the first one's finished tile from LDS as its A
// operand (has_first), or only the second one with its A tile staged once for all of its column blocks: the rows
// are read once and what lies between the two products never leaves the compute unit. LDS: [staging / epilogue |
// the kept A tile]. No groups and no row indirection here.
template <int H, bool BF16, int TM>
__global__ void __launch_bounds__(256, 3) k_gemm_chain(GemmArgs p1, GemmArgs p2, int has_first, int keep_silu) {
  using C = GemmCfg<H, BF16, TM>;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* keep = smem + C::LDS_BYTES;
  const int rbeg = blockIdx.x * C::TM, rend = p2.M;
  if (rbeg >= rend) return;
  f32x16_t acc[C::RB][C::CB];
  if (has_first) {
#pragma unroll
    for (int i = 0; i < C::RB; ++i)
#pragma unroll
      for (int j = 0; j < C::CB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    for (int kc = 0; kc < p1.nkc; ++kc) {
      if (kc) __syncthreads();
      gemm_stage_a<H, BF16, TM>(p1, kc, rbeg, rend, smem);
      __syncthreads();
      gemm_multiply<H, BF16, TM>(p1, kc, 0, 0, smem, acc);
    }
    gemm_epilogue<H, BF16, TM, true>(p1, 0, 0, rbeg, rend, acc, smem, keep, keep_silu);
  } else {
    gemm_stage_a<H, BF16, TM>(p2, 0, rbeg, rend, keep);
  }
  __syncthreads();
  for (int cb = 0; cb < p2.ncb; ++cb) {
#pragma unroll
    for (int i = 0; i < C::RB; ++i)
#pragma unroll
      for (int j = 0; j < C::CB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    gemm_multiply<H, BF16, TM>(p2, 0, cb, 0, keep, acc);
    gemm_epilogue<H, BF16, TM, false>(p2, cb, 0, rbeg, rend, acc, smem, nullptr, 0);
  }
}

// ---------------------------------------------------------------------------------------------
// The same products where the batch has few atoms: 16-row tiles
// ---------------------------------------------------------------------------------------------
// With fewer tiles than compute units such a launch takes as long as ONE tile takes, and a tile is a chain: load A, a
// row of dependent matrix instructions per wavefront, an epilogue that loads its operands, and the same again for the
// second product. This variant shortens the chain: 16-row tiles on the 16 x 16 matrix instructions, one 16-column block
// per wavefront (two at H = 256), so a wavefront's product is a quarter of the instructions (half the instruction time)
// of the 32-row form; both k chunks of A, the weights of the first chunk and all operands of the epilogues are asked for
// at the start; weights are kept one whole chunk ahead in registers; results go from the accumulators straight to memory.
template <int H, bool BF16>
struct SmallCfg {
  static constexpr int TM = 16;
  static constexpr int WAVES = H == 64 ? 4 : 8;
  static constexpr int THREADS = WAVES * 64;
  static constexpr int CB = H / 16 / WAVES;              // 16-column blocks per wavefront
  static constexpr int NKB = H / (BF16 ? 32 : 16);       // 16-byte operand loads per chunk of H
  static constexpr int STRIDE = BF16 ? H + 8 : H + 4;    // LDS row pitch in elements
  static constexpr int ESZ = BF16 ? 2 : 4;
  static constexpr size_t A_BYTES = (size_t)TM * STRIDE * ESZ;
  static constexpr size_t LDS_BYTES = 3 * A_BYTES;       // two k chunks of A | the first product's finished tile
  // first column of block j: at H = 256 the two blocks are 32 columns apart, so that a lane owns both halves of a
  // bf16 pair word (see edge_pairs())
  __device__ static __forceinline__ int col0(int wave, int j) {
    return H == 256 ? (wave >> 1) * 64 + (wave & 1) * 16 + 32 * j : wave * 16;
  }
};
typedef unsigned u32x4s_t __attribute__((ext_vector_type(4)));
template <int H, bool BF16>
struct SmallAux {   // operands of an epilogue, in the accumulator mapping: row 4 (lane >> 4) + v, column lane & 15
  static constexpr int CB = SmallCfg<H, BF16>::CB;
  float bias[CB], mul[CB][4], a1[CB][4], a2[CB][4];
  __device__ __forceinline__ void load(const GemmArgs& p, int cb, int grp, const long (&gr)[4], int wave, int c) {
    const bool ub = p.bias && ((p.bias_cb_mask >> cb) & 1), ua = p.add1 && ((p.add1_cb_mask >> cb) & 1);
#pragma unroll
    for (int j = 0; j < CB; ++j) bias[j] = ub ? p.bias[grp * p.grp_bias_stride + SmallCfg<H, BF16>::col0(wave, j) + c] : 0.f;
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const int gc = cb * H + SmallCfg<H, BF16>::col0(wave, j) + c;
      if (p.mul) {
#pragma unroll
        for (int v = 0; v < 4; ++v) mul[j][v] = p.mul[gr[v] * p.ldmul + gc];
      }
      if (ua) {
#pragma unroll
        for (int v = 0; v < 4; ++v) a1[j][v] = p.add1[gr[v] * p.ldadd1 + gc];
      }
      if (p.add2) {
#pragma unroll
        for (int v = 0; v < 4; ++v) a2[j][v] = p.add2[gr[v] * p.ldadd2 + gc];
      }
    }
  }
};

// RAW: the weights of these products are among the blocks that `pk` describes, and are not packed yet: workgroups beyond the
// `tiles` of the products pack all of them for the kernels that follow, while the products read their own straight from the
// fp32 source (rounded as the packing does), so that they need not wait for a packing launch. Source order: [in, out] for
// a lone product, transposed for a chain (16-byte aligned), see launch_pack_gemm_chain().
// m: the two products of a chain, or lone products of one launch (blockIdx.z)
struct GemmJobs {
  GemmArgs job[2];
};
// SEG: the second chunk of A is rows.M, whose last steps (and v') are taken here, see SegRows
template <int H, bool BF16, bool CHAIN, bool RAW, bool SEG = false>
__device__ __forceinline__ void gemm_small(const GemmJobs& m, int keep_silu, const PackArgs& pk, int tiles, unsigned char* smem,
                                           const SegRows& rows) {
  using C = SmallCfg<H, BF16>;
  const GemmArgs& p1 = m.job[0];
  const GemmArgs& p2 = m.job[CHAIN ? 1 : RAW ? 0 : blockIdx.z];
  unsigned char* keep = smem + 2 * C::A_BYTES;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, hq = lane >> 4;
  const int cb0 = blockIdx.y;   // a lone product takes one column block per workgroup, a chain all of them in turn
  if constexpr (RAW) {
    if ((int)blockIdx.x >= tiles) {   // uniform over the workgroup, before any barrier
      const int pb = ((int)blockIdx.x - tiles) * gridDim.y + blockIdx.y;
      constexpr int XB = H * H / C::THREADS;   // workgroups per block
      static_assert(H * H % C::THREADS == 0, "whole workgroups per block");
      const int planes = pk.nblocks + (pk.x3_dst ? 1 : 0), eb = pb - planes * XB;
      if (eb >= 0) pack_cvec(pk, (int64_t)eb * C::THREADS + tid, (int64_t)((gridDim.x - tiles) * gridDim.y - planes * XB) * C::THREADS);
      else pack_element<BF16>(pk, H, pb / XB, (pb % XB) * C::THREADS + tid, 0, 0, 0);
      return;
    }
  }
  int grp = 0, rbeg, rend;
  if (p2.grp_ptr) {
    if (!tile_of_group(p2.grp_ptr, p2.S, C::TM, blockIdx.x, grp, rbeg, rend)) return;
  } else {
    rbeg = blockIdx.x * C::TM;
    rend = p2.M;
    if (rbeg >= rend) return;
  }
  constexpr int NKC = RAW ? 1 : 2;   // most k chunks of the product that reads A from memory
  const GemmArgs& pa = CHAIN ? p1 : p2;   // the product that reads A from memory
  // ---- weights: lane (column c, quarter hq) of step kb takes k = kb * KS + hq * KS / 4 .. of its column, one 16-byte
  // piece of the packed 32-column operand order (its own 32-column block, k step 2 kb + hq / 2, half hq & 1)
  constexpr int KT = BF16 ? 8 : 4;   // k per lane and step
  u32x4s_t b[RAW ? 1 : C::NKB][C::CB];
  float braw[RAW ? C::NKB : 1][C::CB][KT];
  struct BSrc {
    __amdgpu_buffer_rsrc_t rs;
    const float* src;
  };
  auto b_src = [&](const GemmArgs& p, int kc, int cb) {
    BSrc o;
    if constexpr (RAW) {
      o.src = pk.src + pk.d[p.blk[kc][cb]].src_off;
    } else {
      o.rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<char*>(reinterpret_cast<const char*>(p.B)) + (grp * p.grp_blk_stride + p.blk[kc][cb]) * (long)(H * H * C::ESZ), 0,
          H * H * C::ESZ, 0x00020000);
    }
    return o;
  };
  unsigned bo[C::CB];
#pragma unroll
  for (int j = 0; j < C::CB; ++j) {
    const int n0 = C::col0(wave, j);
    if constexpr (RAW) bo[j] = CHAIN ? (n0 + c) * H + hq * KT : hq * KT * H + n0 + c;
    else bo[j] = (unsigned)((((n0 >> 5) * (2 * C::NKB) + (hq >> 1)) * 64 + (hq & 1) * 32 + (n0 & 16) + c) * 16);
  }
  auto load_b = [&](const BSrc& o, int kb) {
#pragma unroll
    for (int j = 0; j < C::CB; ++j) {
      if constexpr (RAW && CHAIN) {
#pragma unroll
        for (int t = 0; t < KT; t += 4) {
          const float4 w = *reinterpret_cast<const float4*>(o.src + bo[j] + kb * 4 * KT + t);
          braw[kb][j][t] = w.x; braw[kb][j][t + 1] = w.y; braw[kb][j][t + 2] = w.z; braw[kb][j][t + 3] = w.w;
        }
      } else if constexpr (RAW) {
#pragma unroll
        for (int t = 0; t < KT; ++t) braw[kb][j][t] = o.src[bo[j] + (kb * 4 * KT + t) * H];
      } else {
        b[kb][j] = __builtin_amdgcn_raw_buffer_load_b128(o.rs, bo[j], kb * 2048, 0);
      }
    }
  };
  // the operand of step kb, block j
  auto b_frag = [&](int kb, int j) {
    if constexpr (RAW && BF16) {
      const float(&w)[KT] = braw[kb][j];
      return u32x4s_t{pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]), pack_bf16x2(w[4 % KT], w[5 % KT]), pack_bf16x2(w[6 % KT], w[7 % KT])};
    } else if constexpr (RAW) {
      return u32x4s_t{__float_as_uint(braw[kb][j][0]), __float_as_uint(braw[kb][j][1]), __float_as_uint(braw[kb][j][2]), __float_as_uint(braw[kb][j][3])};
    } else {
      return b[kb][j];
    }
  };
  {
    const BSrc rs = b_src(pa, 0, CHAIN ? 0 : cb0);
#pragma unroll
    for (int kb = 0; kb < C::NKB; ++kb) load_b(rs, kb);
  }
  // ---- A: every k chunk at once
  constexpr int CH = H / 4, NA = C::TM * CH / C::THREADS;   // 4-column pieces per thread and chunk
  static_assert(C::TM * CH % C::THREADS == 0, "whole pieces per thread");
  float4 av[NKC][NA];
  long arow[NA];
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int pos = rbeg + (tid + u * C::THREADS) / CH;
    arow[u] = pos < rend ? pos : rend - 1;
    if (pa.row_idx) arow[u] = pa.row_idx[arow[u]];
  }
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc)
    if (kc < pa.nkc && !(SEG && kc == 1)) {
#pragma unroll
      for (int u = 0; u < NA; ++u)
        av[kc][u] = *reinterpret_cast<const float4*>(pa.A[kc] + arow[u] * pa.lda[kc] + ((tid + u * C::THREADS) % CH) * 4);
    }
  if constexpr (SEG) {
    constexpr int UNIT = SegRows::unit(H);
    int ra[NA], rb[NA];
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      ra[u] = rows.row_ptr[arow[u]];
      rb[u] = rows.row_ptr[arow[u] + 1];
    }
    float4 p[NA][2];   // M, or the partials of the first two strips
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int q = ((tid + u * C::THREADS) % CH) * 4, s0 = ra[u] / UNIT;
      const bool over = rb[u] > ra[u] && (rb[u] - 1) / UNIT != s0;
      p[u][0] = p[u][1] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (rb[u] > ra[u]) p[u][0] = *reinterpret_cast<const float4*>(over ? rows.mpart + ((size_t)s0 * 2 + 1) * H + q : rows.M + arow[u] * H + q);
      if (over) p[u][1] = *reinterpret_cast<const float4*>(rows.mpart + (size_t)(s0 + 1) * 2 * H + q);
    }
    // v': sixteen lanes per row
    if (tid < 16 * C::TM) {
      const int pos = rbeg + (tid >> 4);
      const long i = pos < rend ? pos : rend - 1;
      const int e1 = rows.row_ptr[i + 1];
      float sv[3] = {0.f, 0.f, 0.f};
      for (int e0 = rows.row_ptr[i] + (tid & 15); e0 < e1; e0 += 32) {   // two edges per trip
        float t[2], r[2][3];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int e = e0 + 16 * h < e1 ? e0 + 16 * h : e0;
          t[h] = rows.xe_part[e];
#pragma unroll
          for (int k = 1; k < SegRows::parts(H); ++k) t[h] += rows.xe_part[k * rows.xe_stride + e];
#pragma unroll
          for (int k = 0; k < 3; ++k) r[h][k] = rows.rvec[3 * (size_t)e + k];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (e0 + 16 * h < e1) {
            if (rows.xe_out && pos < rend) rows.xe_out[e0 + 16 * h] = t[h];
#pragma unroll
            for (int k = 0; k < 3; ++k) sv[k] = fmaf(t[h], r[h][k], sv[k]);
          }
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        sv[k] += dpp_f<0x140>(sv[k]);
        sv[k] += dpp_f<0x141>(sv[k]);
        sv[k] += dpp_f<0x1b>(sv[k]);
        sv[k] += dpp_f<0xb1>(sv[k]);
      }
      const int k = tid & 15;
      if (k < 3 && pos < rend) rows.v_out[3 * i + k] = rows.v_in[3 * i + k] + rows.alpha * (k == 0 ? sv[0] : k == 1 ? sv[1] : sv[2]);
    }
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int q = ((tid + u * C::THREADS) % CH) * 4, s0 = ra[u] / UNIT, s1 = (rb[u] - 1) / UNIT;
      float4 w = p[u][0];
      if (rb[u] == ra[u] || s1 != s0) {
        auto add = [&](const float4& t) { w.x += t.x; w.y += t.y; w.z += t.z; w.w += t.w; };
        add(p[u][1]);
        if (rb[u] > ra[u])
          for (int s = s0 + 2; s <= s1; ++s) add(*reinterpret_cast<const float4*>(rows.mpart + (size_t)s * 2 * H + q));
        w.x *= rows.alpha; w.y *= rows.alpha; w.z *= rows.alpha; w.w *= rows.alpha;
        if (rbeg + (tid + u * C::THREADS) / CH < rend) *reinterpret_cast<float4*>(rows.M + arow[u] * H + q) = w;
      }
      av[NKC - 1][u] = w;
    }
  }
  // ---- rows of this lane's accumulators and the epilogues' operands
  long gr[4];
  bool ok[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int pos = rbeg + 4 * hq + v;
    ok[v] = pos < rend;
    gr[v] = ok[v] ? pos : rend - 1;
    if (p2.row_idx) gr[v] = p2.row_idx[gr[v]];
  }
  SmallAux<H, BF16> x1, x2;
  if constexpr (CHAIN) x1.load(p1, 0, grp, gr, wave, c);
  x2.load(p2, cb0, grp, gr, wave, c);
  // ---- A to LDS
  auto put_a = [&](unsigned char* dst, int r, int q, float4 w) {
    if constexpr (BF16) *reinterpret_cast<uint2*>(dst + ((size_t)r * C::STRIDE + q * 4) * 2) = make_uint2(pack_bf16x2(w.x, w.y), pack_bf16x2(w.z, w.w));
    else *reinterpret_cast<float4*>(dst + ((size_t)r * C::STRIDE + q * 4) * 4) = w;
  };
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc)
    if (kc < pa.nkc) {
#pragma unroll
      for (int u = 0; u < NA; ++u) {
        const int r = (tid + u * C::THREADS) / CH;
        float4 w = av[kc][u];
        if (pa.a_silu) { w.x = silu_f(w.x); w.y = silu_f(w.y); w.z = silu_f(w.z); w.w = silu_f(w.w); }
        if (rbeg + r >= rend) w = make_float4(0.f, 0.f, 0.f, 0.f);
        put_a(smem + kc * C::A_BYTES, r, (tid + u * C::THREADS) % CH, w);
      }
    }
  __syncthreads();
  f32x4_t acc[C::CB];
  auto clear = [&]() {
#pragma unroll
    for (int j = 0; j < C::CB; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  // one chunk; the weights of the next one take each register as it is used up
  const unsigned ao = (unsigned)((c * C::STRIDE + hq * (16 / C::ESZ)) * C::ESZ);
  auto multiply = [&](const unsigned char* a_lds, bool next, const BSrc& rs) {
    u32x4s_t a[C::NKB];
#pragma unroll
    for (int kb = 0; kb < C::NKB; ++kb) a[kb] = *reinterpret_cast<const u32x4s_t*>(a_lds + ao + kb * 64);
#pragma unroll
    for (int kb = 0; kb < C::NKB; ++kb) {
#pragma unroll
      for (int j = 0; j < C::CB; ++j) {
        if constexpr (BF16) {
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[kb]), __builtin_bit_cast(bf16x8_t, b_frag(kb, j)), acc[j], 0, 0, 0);
        } else {
          const f32x4_t af = __builtin_bit_cast(f32x4_t, a[kb]), bf = __builtin_bit_cast(f32x4_t, b_frag(kb, j));
#pragma unroll
          for (int t = 0; t < 4; ++t) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[t], bf[t], acc[j], 0, 0, 0);
        }
      }
      if (next) load_b(rs, kb);
    }
  };
  // values of block j, row v of the accumulators through the epilogue
  auto finish = [&](const GemmArgs& p, const SmallAux<H, BF16>& x, bool ua, int j, int v) {
    float y = acc[j][v] + x.bias[j];
    if (p.mul) y *= p.mul_is_z ? dsilu_f(x.mul[j][v]) : x.mul[j][v];
    if (ua) y += x.a1[j][v];
    if (p.add2) y += x.a2[j][v];
    return y;
  };
  const unsigned char* a2 = smem;   // A of the second product
  if constexpr (CHAIN) {
    clear();
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc)
      if (kc < p1.nkc) multiply(smem + kc * C::A_BYTES, true, kc + 1 < p1.nkc ? b_src(p1, kc + 1, 0) : b_src(p2, 0, 0));
    const bool ua = p1.add1 && (p1.add1_cb_mask & 1);
#pragma unroll
    for (int j = 0; j < C::CB; ++j) {
      const int n = C::col0(wave, j) + c;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float y = finish(p1, x1, ua, j, v);
        if (ok[v]) p1.C[gr[v] * p1.ldc + n] = y;
        if (keep_silu) y = silu_f(y);
        if (!ok[v]) y = 0.f;
        if constexpr (BF16) *reinterpret_cast<unsigned short*>(keep + ((4 * hq + v) * C::STRIDE + n) * 2) = (unsigned short)f2bf_bits(y);
        else *reinterpret_cast<float*>(keep + ((4 * hq + v) * C::STRIDE + n) * 4) = y;
      }
    }
    a2 = keep;
    __syncthreads();
  }
  const int cbe = CHAIN ? p2.ncb : cb0 + 1;
  for (int cb = cb0; cb < cbe; ++cb) {
    clear();
    if constexpr (CHAIN) {
      multiply(a2, cb + 1 < cbe, b_src(p2, 0, cb + 1 < cbe ? cb + 1 : cb));
    } else {
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc)
        if (kc < p2.nkc) multiply(a2 + kc * C::A_BYTES, kc + 1 < p2.nkc, b_src(p2, kc + 1 < p2.nkc ? kc + 1 : kc, cb));
    }
    const bool ua = p2.add1 && ((p2.add1_cb_mask >> cb) & 1);
    if constexpr (H == 256) {
      if ((p2.pair_cb_mask >> cb) & 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (ok[v])
            p2.Cpair[gr[v] * p2.ldpair + p2.pair_off[cb] + (wave >> 1) * 32 + (wave & 1) * 16 + c] =
                pack_bf16x2((acc[0][v] + x2.bias[0]) * p2.pair_scale, (acc[1][v] + x2.bias[1]) * p2.pair_scale);
        if (cb + 1 < cbe) x2.load(p2, cb + 1, grp, gr, wave, c);
        continue;
      }
    }
#pragma unroll
    for (int j = 0; j < C::CB; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float y = finish(p2, x2, ua, j, v);
        if (ok[v]) p2.C[gr[v] * p2.ldc + cb * H + C::col0(wave, j) + c] = y;
      }
    if (cb + 1 < cbe) x2.load(p2, cb + 1, grp, gr, wave, c);
  }
}

template <int H, bool BF16, bool CHAIN, bool RAW>
__global__ void __launch_bounds__((SmallCfg<H, BF16>::THREADS)) k_gemm_small(GemmJobs m, int keep_silu, PackArgs pk, int tiles) {
  extern __shared__ __align__(16) unsigned char smem[];
  gemm_small<H, BF16, CHAIN, RAW>(m, keep_silu, pk, tiles, smem, SegRows{});
}
template <int H, bool BF16>
__global__ void __launch_bounds__((SmallCfg<H, BF16>::THREADS)) k_gemm_small_rows(GemmJobs m, int keep_silu, SegRows rows) {
  extern __shared__ __align__(16) unsigned char smem[];
  gemm_small<H, BF16, true, false, true>(m, keep_silu, PackArgs{}, 0, smem, rows);
}

// (rule: see small_gemm())
template <int H, bool BF16>
static int32_t launch_gemm_small_t(hipStream_t st, const GemmArgs* first, const GemmArgs& a, int keep_silu, const SegRows* rows = nullptr) {
  using C = SmallCfg<H, BF16>;
  const int tiles = (a.M + C::TM - 1) / C::TM + (a.grp_ptr ? a.S : 0);
  ProfScope ps(rows ? (int)PT_GEMM_ROWS : a.tag, st);
  if (rows) k_gemm_small_rows<H, BF16><<<dim3(tiles), C::THREADS, C::LDS_BYTES, st>>>(GemmJobs{{*first, a}}, keep_silu, *rows);
  else if (first) k_gemm_small<H, BF16, true, false><<<dim3(tiles), C::THREADS, C::LDS_BYTES, st>>>(GemmJobs{{*first, a}}, keep_silu, PackArgs{}, tiles);
  else k_gemm_small<H, BF16, false, false><<<dim3(tiles, a.ncb), C::THREADS, C::LDS_BYTES, st>>>(GemmJobs{{a, a}}, 0, PackArgs{}, tiles);
  HGNN_LAUNCH_CHECK("k_gemm_small");
  return HGNN_OK;
}
template <int H, bool BF16>
static int32_t launch_pack_gemm_small_t(hipStream_t st, const PackArgs& pk, const GemmArgs* first, const GemmArgs& a, int keep_silu) {
  using C = SmallCfg<H, BF16>;
  const int tiles = (a.M + C::TM - 1) / C::TM, gy = first ? 1 : a.ncb;
  int64_t eb = pk.cvec ? (pk.E + C::THREADS - 1) / C::THREADS : 0;
  if (eb > 8192) eb = 8192;   // (the rest in a loop)
  const int pack = (pk.nblocks + (pk.x3_dst ? 1 : 0)) * (H * H / C::THREADS) + (int)eb;
  const dim3 grid(tiles + (pack + gy - 1) / gy, gy);
  ProfScope ps(a.tag, st);
  if (first) k_gemm_small<H, BF16, true, true><<<grid, C::THREADS, C::LDS_BYTES, st>>>(GemmJobs{{*first, a}}, keep_silu, pk, tiles);
  else k_gemm_small<H, BF16, false, true><<<grid, C::THREADS, C::LDS_BYTES, st>>>(GemmJobs{{a, a}}, 0, pk, tiles);
  HGNN_LAUNCH_CHECK("k_gemm_small (packing)");
  return HGNN_OK;
}
// The short chains win while the taller tiles would not give every compute unit one of them; beyond that twice the
// tiles mean twice the weight traffic. Steps, 32 / 64-row tiles against 16-row tiles: 32 molecules (7 tiles) 485 -> 461 us,
// a crystal's conservative forces (6) 944 -> 863, 16 crystals (32) 1175 -> 1083, 64 crystals (127) 1881 -> 1806,
// 128 molecules (140) 973 -> 946, 203 molecules, energies and forces only (222) 315 -> 302; past the line 160 mixed
// structures (338) 2980 -> 3028, 300 (600) 4885 -> 5094. fp32 operands at H = 256 keep the taller tiles: a chunk of
// their weights is 128 registers.
// Groups count as a tile each: rows are rarely whole tiles of a group, every workgroup walks the groups to find its own, and
// the shorter the tiles, the more workgroups walk. Heads, forward, taller tiles -> 16-row tiles: 400 rows, 200 groups,
// H = 128, 70 -> 61 us; 4,600 rows, 64 groups 38 -> 37; past the line 8,000 rows, 64 groups 40 -> 44, 500 groups 169 -> 357.
constexpr int tall_rows(int H) { return H >= 128 ? 32 : 64; }   // rows of the taller tiles
static bool small_gemm(int H, bool bf16, const GemmArgs& a, int tile_rows) {
  return (bf16 || H < 256) && a.M > 0 && (a.M + tile_rows - 1) / tile_rows + (a.grp_ptr ? a.S : 0) <= num_cus();
}
static bool small_gemm(int H, bool bf16, const GemmArgs& a) { return small_gemm(H, bf16, a, tall_rows(H)); }
// Chains at H = 256 only while every compute unit has one 16-row tile at most: 512 threads hold two blocks of both weights each
// (layer forward, 64- / 32-row tiles -> 16-row tiles, 4,000 atoms 44 -> 37 us, 5,000 44 -> 47, 8,000 49 -> 53).
static bool small_chain(int H, bool bf16, const GemmArgs& a) { return small_gemm(H, bf16, a, H == 256 ? 16 : tall_rows(H)); }

// workgroups of this variant that one CU holds at a time (asked once; also raises the LDS limit of the kernel)
template <int H, bool BF16, int TM>
static int gemm_resident_wgs() {
  using C = GemmCfg<H, BF16, TM>;
  static int n = 0;
  if (n == 0) {
    const void* fn = reinterpret_cast<const void*>(&k_gemm<H, BF16, TM>);
    int occ = 0;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS_BYTES) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, 256, C::LDS_BYTES) != hipSuccess || occ < 1)
      occ = 1;
    n = occ;
  }
  return n;
}

template <int H, bool BF16, int TM>
static int32_t launch_gemm_tm(hipStream_t st, const GemmArgs& a) {
  using C = GemmCfg<H, BF16, TM>;
  const int tiles = (a.M + C::TM - 1) / C::TM + (a.grp_ptr ? a.S : 0);
  gemm_resident_wgs<H, BF16, TM>();
  ProfScope ps(a.tag, st);
  k_gemm<H, BF16, TM><<<dim3(tiles, a.ncb), 256, C::LDS_BYTES, st>>>(a);
  HGNN_LAUNCH_CHECK("k_gemm");
  return HGNN_OK;
}

// Tile height: a workgroup runs load -> product -> epilogue as one dependent chain whose length grows with the tile
// height, so the shortest tile the wavefront grid allows (32 rows where the four wavefronts sit side by side over
// the columns, i.e. H >= 128; four workgroups per compute unit) gives the most chains in flight. Measured per step
// against 64 / 96-row tiles: config 3 0.64 -> 0.37 ms, config 4 1.69 -> 1.50 ms, config 5 1.28 -> 1.22 ms.
template <int H, bool BF16>
static int32_t launch_gemm_t(hipStream_t st, const GemmArgs& a) {
  if (a.M <= 0) return HGNN_OK;
  if constexpr (BF16 || H < 256) {
    if (small_gemm(H, BF16, a)) return launch_gemm_small_t<H, BF16>(st, nullptr, a, 0);
  }
  return launch_gemm_tm<H, BF16, tall_rows(H)>(st, a);
}

template <int H, bool BF16>
static int32_t launch_gemm_chain_t(hipStream_t st, const GemmArgs* first, const GemmArgs& second, int keep_silu, const SegRows* rows) {
  constexpr int TM = tall_rows(H);
  using C = GemmCfg<H, BF16, TM>;
  if (second.M <= 0) return HGNN_OK;
  if constexpr (BF16 || H < 256) {
    if (small_chain(H, BF16, second)) return launch_gemm_small_t<H, BF16>(st, first, second, keep_silu, rows);
  }
  HGNN_REQUIRE(!rows, HGNN_ERR_BAD_SHAPE, "gemm chain: the forward sums are finished by 16-row tiles only");
  constexpr size_t LDS = C::LDS_BYTES + C::A_BYTES;
  static bool raised = false;   // the kernel's LDS limit is raised once per variant
  if (!raised) {
    HGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_chain<H, BF16, TM>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS));
    raised = true;
  }
  const int tiles = (second.M + TM - 1) / TM;
  ProfScope ps(second.tag, st);
  k_gemm_chain<H, BF16, TM><<<dim3(tiles), 256, LDS, st>>>(first ? *first : second, second, first ? 1 : 0, keep_silu);
  HGNN_LAUNCH_CHECK("k_gemm_chain");
  return HGNN_OK;
}

// `first` (optional): one column block, its finished tile (through silu when keep_silu) is the A operand of `second`,
// whose own A fields are then ignored; without `first`, `second` runs alone with its A tile (one k chunk) staged
// once for all its column blocks.
static int32_t check_gemm_chain(int H, const GemmArgs* first, const GemmArgs& second) {
  for (const GemmArgs* g : {first, &second}) {
    if (!g) continue;
    HGNN_REQUIRE(!g->row_idx && !g->grp_ptr, HGNN_ERR_BAD_SHAPE, "gemm chain: no groups, no row indirection");
    HGNN_REQUIRE(g->B && (g->C || g->Cpair), HGNN_ERR_NULLPTR, "gemm chain: null operand");
    HGNN_REQUIRE(g->pair_cb_mask == 0 || (H == 256 && g->Cpair), HGNN_ERR_BAD_SHAPE, "gemm chain: pair output needs H = 256");
  }
  HGNN_REQUIRE(second.ncb >= 1 && second.ncb <= 2, HGNN_ERR_BAD_SHAPE, "gemm chain: bad chunk counts");
  if (first) {
    HGNN_REQUIRE(first->nkc >= 1 && first->nkc <= 2 && first->ncb == 1 && first->A[0] && first->pair_cb_mask == 0 &&
                     first->M == second.M,
                 HGNN_ERR_BAD_SHAPE, "gemm chain: bad first product");
  } else {
    HGNN_REQUIRE(second.nkc == 1 && second.A[0], HGNN_ERR_BAD_SHAPE, "gemm chain: the lone product takes one k chunk");
  }
  return HGNN_OK;
}
// Chains of 16-row tiles finish the forward sums of their rows themselves: a launch fewer per layer, whose loads travel with the
// chain's own. Steps, launch of its own -> in the chain: one molecule, forward 131 -> 126 us, 203 molecules, forward 272 -> 265, 32 small molecules 259 -> 254, 128 molecules 766 -> 762, one crystal of 60 atoms, forward 197 -> 191;
// a crystal's conservative forces (12 tiles, rows of 57 edges) 473 -> 472.
bool gemm_chain_takes_rows(int H, bool bf16, int M) {
  GemmArgs a;
  a.M = M;
  return small_chain(H, bf16, a);
}
int32_t launch_gemm_chain(hipStream_t st, int H, bool bf16, const GemmArgs* first, const GemmArgs& second, int keep_silu,
                          const SegRows* rows) {
  HGNN_TRY(check_gemm_chain(H, first, second));
  HGNN_REQUIRE(!rows || (first && first->nkc == 2 && first->A[1] == rows->M && first->lda[1] == H), HGNN_ERR_BAD_SHAPE,
               "gemm chain: the forward sums are finished by the product that reads them");
  switch (H) {
    case 64: return bf16 ? launch_gemm_chain_t<64, true>(st, first, second, keep_silu, rows) : launch_gemm_chain_t<64, false>(st, first, second, keep_silu, rows);
    case 128: return bf16 ? launch_gemm_chain_t<128, true>(st, first, second, keep_silu, rows) : launch_gemm_chain_t<128, false>(st, first, second, keep_silu, rows);
    case 256: return bf16 ? launch_gemm_chain_t<256, true>(st, first, second, keep_silu, rows) : launch_gemm_chain_t<256, false>(st, first, second, keep_silu, rows);
  }
  return set_error(HGNN_ERR_BAD_SHAPE, "H must be 64, 128 or 256 (got %d)", H);
}

// One launch while the products read at most RAW_BYTES of unpacked weights (every 16-row tile reads its blocks whole, twice the
// bytes of packed ones with bf16 operands). Per step, two launches against one: one molecule, forward 215 -> 208 us, 32 small
// molecules 395 -> 377, a crystal's conservative forces 605 -> 598, 16 molecules at H = 128 497 -> 482; past the line nothing changes.
constexpr long RAW_BYTES = 16l << 20;
static bool pack_along(int H, bool bf16, const PackArgs& pk, const GemmArgs* first, const GemmArgs& second) {
  if (H > 128 || !small_gemm(H, bf16, second)) return false;
  if (first && first->nkc != 1) return false;
  const int nblk = (first ? 1 : 0) + second.ncb;
  if (((second.M + 15) / 16) * (long)nblk * H * H * 4 > RAW_BYTES) return false;
  if (first && reinterpret_cast<uintptr_t>(pk.src) % 16 != 0) return false;
  for (const GemmArgs* g : {first, &second}) {   // blocks of this packing, in the order of the source that the kernel reads
    if (!g) continue;
    if (g->B != pk.dst) return false;
    for (int cb = 0; cb < g->ncb; ++cb) {
      const long b = g->blk[0][cb];
      if (b < 0 || b >= pk.nblocks || pk.d[b].sk != (first ? 1 : H) || pk.d[b].sn != (first ? H : 1)) return false;
      if (first && pk.d[b].src_off % 4 != 0) return false;
    }
  }
  return true;
}
int32_t launch_pack_gemm_chain(hipStream_t st, int H, bool bf16, const PackArgs& pk, const GemmArgs* first,
                               const GemmArgs& second, int keep_silu) {
  if (!pack_along(H, bf16, pk, first, second)) {
    HGNN_TRY(launch_pack(st, H, bf16, pk));
    return launch_gemm_chain(st, H, bf16, first, second, keep_silu);
  }
  HGNN_TRY(check_gemm_chain(H, first, second));
  if (H == 64) return bf16 ? launch_pack_gemm_small_t<64, true>(st, pk, first, second, keep_silu)
                           : launch_pack_gemm_small_t<64, false>(st, pk, first, second, keep_silu);
  return bf16 ? launch_pack_gemm_small_t<128, true>(st, pk, first, second, keep_silu)
              : launch_pack_gemm_small_t<128, false>(st, pk, first, second, keep_silu);
}

static int32_t check_gemm(int H, const GemmArgs& a) {
  HGNN_REQUIRE(a.nkc >= 1 && a.nkc <= 2 && a.ncb >= 1 && a.ncb <= 2, HGNN_ERR_BAD_SHAPE, "gemm: bad chunk counts");
  HGNN_REQUIRE(a.A[0] && a.B && (a.C || a.Cpair), HGNN_ERR_NULLPTR, "gemm: null operand");
  HGNN_REQUIRE(a.pair_cb_mask == 0 || (H == 256 && a.Cpair), HGNN_ERR_BAD_SHAPE, "gemm: pair output needs H = 256");
  return HGNN_OK;
}
int32_t launch_gemm(hipStream_t st, int H, bool bf16, const GemmArgs& a) {
  HGNN_TRY(check_gemm(H, a));
  switch (H) {
    case 64: return bf16 ? launch_gemm_t<64, true>(st, a) : launch_gemm_t<64, false>(st, a);
    case 128: return bf16 ? launch_gemm_t<128, true>(st, a) : launch_gemm_t<128, false>(st, a);
    case 256: return bf16 ? launch_gemm_t<256, true>(st, a) : launch_gemm_t<256, false>(st, a);
  }
  return set_error(HGNN_ERR_BAD_SHAPE, "H must be 64, 128 or 256 (got %d)", H);
}

template <int H, bool BF16>
static int32_t launch_gemm_small_pair_t(hipStream_t st, const GemmArgs& a, const GemmArgs& b) {
  using C = SmallCfg<H, BF16>;
  const auto tiles = [](const GemmArgs& g) { return (g.M + C::TM - 1) / C::TM + (g.grp_ptr ? g.S : 0); };
  const int ta = tiles(a), tb = tiles(b), t = ta > tb ? ta : tb;
  ProfScope ps(a.tag, st);
  k_gemm_small<H, BF16, false, false><<<dim3(t, a.ncb, 2), C::THREADS, C::LDS_BYTES, st>>>(GemmJobs{{a, b}}, 0, PackArgs{}, t);
  HGNN_LAUNCH_CHECK("k_gemm_small (two products)");
  return HGNN_OK;
}
int32_t launch_gemm_pair(hipStream_t st, int H, bool bf16, const GemmArgs& a, const GemmArgs& b) {
  const bool one = a.ncb == b.ncb && small_gemm(H, bf16, a) && small_gemm(H, bf16, b);
  if (!one) {
    HGNN_TRY(launch_gemm(st, H, bf16, a));
    return launch_gemm(st, H, bf16, b);
  }
  HGNN_TRY(check_gemm(H, a));
  HGNN_TRY(check_gemm(H, b));
  switch (H) {
    case 64: return bf16 ? launch_gemm_small_pair_t<64, true>(st, a, b) : launch_gemm_small_pair_t<64, false>(st, a, b);
    case 128: return bf16 ? launch_gemm_small_pair_t<128, true>(st, a, b) : launch_gemm_small_pair_t<128, false>(st, a, b);
  }
  return launch_gemm_small_pair_t<256, true>(st, a, b);
}

// ---------------------------------------------------------------------------------------------
// deterministic reduction of split partials:  dest[blk][i] = sum_s partial[grp][s][blk][i]
// ---------------------------------------------------------------------------------------------
struct ReduceArgs {
  const float* partial;
  int nsplit;
  int nblk;
  long blk_elems;
  float* dest[8];
  long grp_dest_stride;
};

// partials k0 .. k1 - 1 in ascending order, sixteen loads in flight at a time (the last batch clamped, then left out)
__device__ __forceinline__ float reduce_range(const float* p, long step, int k0, int k1) {
  float s = 0.f;
  int k = k0;
  for (; k + 16 <= k1; k += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(long)(k + u) * step];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += v[u];
  }
  for (; k < k1; k += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(long)(k + u < k1 ? k + u : k1 - 1) * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += k + u < k1 ? v[u] : 0.f;
  }
  return s;
}

// (T: threads per workgroup)
// wide blocks: one thread per element
template <int T>
__device__ __forceinline__ void reduce_wide(const ReduceArgs& a, int bx, int blk, int grp) {
  const long i = (long)bx * T + threadIdx.x;
  if (i >= a.blk_elems || !a.dest[blk]) return;
  const float* p = a.partial + ((long)grp * a.nsplit * a.nblk + blk) * a.blk_elems + i;
  const long step = (long)a.nblk * a.blk_elems;
  if (a.nsplit == 1) {   // a plain copy (also of negative zeros)
    a.dest[blk][grp * a.grp_dest_stride + i] = p[0];
    return;
  }
  a.dest[blk][grp * a.grp_dest_stride + i] = reduce_range(p, step, 0, a.nsplit);
}

// Many partials: T / EPB threads per element take a contiguous share of the partials each (in order), then the shares are
// added in order. sh: T floats of LDS. Every thread of the workgroup calls it.
template <int EPB, int T>
__device__ __forceinline__ void reduce_tall(const ReduceArgs& a, int bx, int blk, int grp, float* sh) {
  constexpr int PH = T / EPB;
  const int e = threadIdx.x % EPB, ph = threadIdx.x / EPB;
  const long i = (long)bx * EPB + e;
  const int per = (a.nsplit + PH - 1) / PH;
  const int k0 = ph * per;
  const int k1 = k0 + per < a.nsplit ? k0 + per : a.nsplit;
  float s = 0.f;
  if (!a.dest[blk]) return;   // uniform over the block
  if (i < a.blk_elems) {
    const float* p = a.partial + ((long)grp * a.nsplit * a.nblk + blk) * a.blk_elems + i;
    const long step = (long)a.nblk * a.blk_elems;
    s = reduce_range(p, step, k0, k1);
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  if (ph == 0 && i < a.blk_elems) {
    float t = sh[e];
#pragma unroll
    for (int q = 1; q < PH; ++q) t += sh[q * EPB + e];
    a.dest[blk][grp * a.grp_dest_stride + i] = t;
  }
}
// Elements per workgroup: a sum of partials is a chain of batches of 16 loads, and one thread per element leaves most of the
// chip idle besides (16,384 elements are 64 workgroups). From 32 partials on, eight threads share an element (128-byte rows of
// a partial), sixteen where there are few elements (bias-type sums); below, a chain is at most two batches long.
// Steps: 128 molecules 883 -> 853 us, 32 small molecules 359 -> 343, a crystal's conservative forces 572 -> 559, 160 mixed structures
// with moving atoms 2962 -> 2918; 643 mixed structures the same within 0.5 %.
static int reduce_epb(long blk_elems, int nsplit) { return nsplit < 32 ? 256 : blk_elems <= 1024 ? 16 : 32; }
static unsigned reduce_xblocks(long blk_elems, int nsplit) {
  const int epb = reduce_epb(blk_elems, nsplit);
  return (unsigned)((blk_elems + epb - 1) / epb);
}
// (epb: elements per 256 threads; the threads that share an element stay as many in a larger workgroup)
template <int T>
__device__ __forceinline__ void reduce_any(const ReduceArgs& a, int epb, int bx, int blk, int grp, float* sh) {
  if (epb == 16) reduce_tall<16 * T / 256, T>(a, bx, blk, grp, sh);
  else if (epb == 32) reduce_tall<32 * T / 256, T>(a, bx, blk, grp, sh);
  else reduce_wide<T>(a, bx, blk, grp);
}

__global__ void __launch_bounds__(256) k_reduce_partials(ReduceArgs a, int epb) {
  __shared__ float sh[256];
  reduce_any<256>(a, epb, blockIdx.x, blockIdx.y, blockIdx.z, sh);
}

// several reductions in one launch: the workgroups of all jobs one after the other, in a job element blocks first, then the
// blocks of the partials, then the groups (a three-dimensional grid over the largest job would be mostly empty workgroups)
constexpr int REDUCE_QUEUE_MAX = 8;
// A launch holds fewer than 2^32 threads in x. Two weight gradients at H = 256 pass that from about 32,400 sources on: what
// does not fit runs as a launch of its own, with the groups in z.
constexpr long REDUCE_QUEUE_WGS = (1L << 32) / 256 - 1;
// Most that share a launch with a product (small batches only, by the rule of the products). Long reductions run into the few
// workgroups that the product's registers leave room for. Two launches -> one: 32 small molecules (2.7 MB of partials) 338 -> 318 us
// per step, a crystal's conservative forces (12 MB) 523 -> 504, 16 molecules at H = 128 (13 MB) 485 -> 467, 128 molecules (51 MB)
// 850 -> 834, 8 crystals (79 MB) 688 -> 677; past the line 64 crystals (101 MB) 1599 -> 1620.
constexpr long REDUCE_WITH_BYTES = 80L << 20, REDUCE_WITH_WGS = 1L << 20;
struct ReduceQueueArgs {
  ReduceArgs job[REDUCE_QUEUE_MAX];
  int njobs;
  long off[REDUCE_QUEUE_MAX + 1];
  int xblocks[REDUCE_QUEUE_MAX];
  int epb[REDUCE_QUEUE_MAX];
  long bytes() const {   // of the partials
    long b = 0;
    for (int j = 0; j < njobs; ++j) b += (off[j + 1] - off[j]) / xblocks[j] * job[j].blk_elems * job[j].nsplit * 4;
    return b;
  }
};
template <int T>
__device__ __forceinline__ void reduce_queue(const ReduceQueueArgs& q, long wg, float* sh) {
  int j = 0;   // uniform over the workgroup
  while (j + 1 < q.njobs && wg >= q.off[j + 1]) ++j;
  const int r = (int)(wg - q.off[j]);
  const int bx = r % q.xblocks[j], y = r / q.xblocks[j];
  reduce_any<T>(q.job[j], q.epb[j], bx, y % q.job[j].nblk, y / q.job[j].nblk, sh);
}
__global__ void __launch_bounds__(256) k_reduce_queue(ReduceQueueArgs q) {
  __shared__ float sh[256];
  reduce_queue<256>(q, blockIdx.x, sh);
}
// One or two lone products of a small batch (blockIdx.z) and the reductions that wait for the end of a reverse pass: neither reads
// what the other writes, and both are launches of 4-10 us that leave most of the chip idle. Workgroups behind the `tiles` of
// the products take the reductions.
template <int H, bool BF16>
__global__ void __launch_bounds__((SmallCfg<H, BF16>::THREADS)) k_gemm_small_reduce(GemmJobs m, ReduceQueueArgs q, int tiles) {
  extern __shared__ __align__(16) unsigned char smem[];
  static_assert(SmallCfg<H, BF16>::LDS_BYTES >= SmallCfg<H, BF16>::THREADS * sizeof(float), "a float per thread");
  if ((int)blockIdx.x < tiles) {
    gemm_small<H, BF16, false, false>(m, 0, PackArgs{}, tiles, smem, SegRows{});
  } else {
    const long wg = (long)((int)blockIdx.x - tiles) * gridDim.z + blockIdx.z;
    if (wg < q.off[q.njobs]) reduce_queue<SmallCfg<H, BF16>::THREADS>(q, wg, reinterpret_cast<float*>(smem));
  }
}

struct ReduceQueue {
  hipStream_t st;
  ReduceQueueArgs q;
};
static thread_local ReduceQueue* tl_reduce_queue = nullptr;

ReduceQueueScope::ReduceQueueScope(hipStream_t st, bool enable) : active_(enable && tl_reduce_queue == nullptr) {
  if (active_) {
    tl_reduce_queue = new ReduceQueue;
    tl_reduce_queue->st = st;
    tl_reduce_queue->q.njobs = 0;
    tl_reduce_queue->q.off[0] = 0;
  }
}
ReduceQueueScope::~ReduceQueueScope() {
  if (active_) {
    delete tl_reduce_queue;
    tl_reduce_queue = nullptr;
  }
}
int32_t ReduceQueueScope::flush() {
  if (!active_ || tl_reduce_queue->q.njobs == 0) return HGNN_OK;
  ReduceQueueArgs& q = tl_reduce_queue->q;
  k_reduce_queue<<<dim3((unsigned)q.off[q.njobs]), 256, 0, tl_reduce_queue->st>>>(q);
  q.njobs = 0;
  HGNN_LAUNCH_CHECK("k_reduce_queue");
  return HGNN_OK;
}

template <int H, bool BF16>
static int32_t launch_gemm_small_reduce_t(hipStream_t st, const GemmArgs& a, const GemmArgs* b, ReduceQueueArgs q) {
  using C = SmallCfg<H, BF16>;
  long begin = q.off[0], end = q.off[1];
  for (int j = 0; j < q.njobs; ++j) {   // the same jobs in workgroups of this size
    const int epb = q.epb[j] * (C::THREADS / 256);
    const long rows = (end - begin) / q.xblocks[j];   // partial blocks x groups
    begin = end;
    if (j + 2 <= q.njobs) end = q.off[j + 2];
    q.xblocks[j] = (int)((q.job[j].blk_elems + epb - 1) / epb);
    q.off[j + 1] = q.off[j] + rows * q.xblocks[j];
  }
  const auto tiles_of = [](const GemmArgs& g) { return (g.M + C::TM - 1) / C::TM + (g.grp_ptr ? g.S : 0); };
  const int ta = tiles_of(a), tb = b ? tiles_of(*b) : 0, tiles = ta > tb ? ta : tb, gz = b ? 2 : 1;
  ProfScope ps(PT_GEMM_REDUCE, st);
  k_gemm_small_reduce<H, BF16><<<dim3((unsigned)(tiles + (q.off[q.njobs] + gz - 1) / gz), 1, gz), C::THREADS, C::LDS_BYTES, st>>>(
      GemmJobs{{a, b ? *b : a}}, q, tiles);
  HGNN_LAUNCH_CHECK("k_gemm_small_reduce");
  return HGNN_OK;
}
int32_t ReduceQueueScope::flush_with(hipStream_t st, int H, bool bf16, int tag, const GemmArgs& a, const GemmArgs* b) {
  const bool one = active_ && tl_reduce_queue->q.njobs > 0 && tl_reduce_queue->st == st && a.ncb == 1 && small_gemm(H, bf16, a) &&
                   (!b || (b->ncb == 1 && small_gemm(H, bf16, *b))) &&
                   tl_reduce_queue->q.off[tl_reduce_queue->q.njobs] <= REDUCE_WITH_WGS && tl_reduce_queue->q.bytes() <= REDUCE_WITH_BYTES;
  if (!one) {
    if (b) HGNN_TRY(launch_gemm_pair(st, H, bf16, a, *b));
    else HGNN_TRY(launch_gemm(st, H, bf16, a));
    ProfScope ps(tag, st);
    return flush();
  }
  HGNN_TRY(check_gemm(H, a));
  if (b) HGNN_TRY(check_gemm(H, *b));
  const ReduceQueueArgs q = tl_reduce_queue->q;
  tl_reduce_queue->q.njobs = 0;   // (off[0] stays 0)
  switch (H) {
    case 64: return bf16 ? launch_gemm_small_reduce_t<64, true>(st, a, b, q) : launch_gemm_small_reduce_t<64, false>(st, a, b, q);
    case 128: return bf16 ? launch_gemm_small_reduce_t<128, true>(st, a, b, q) : launch_gemm_small_reduce_t<128, false>(st, a, b, q);
  }
  return launch_gemm_small_reduce_t<256, true>(st, a, b, q);
}

static int32_t launch_reduce_partials_n(hipStream_t st, const float* partial, int nsplit, int nblk, long blk_elems,
                                         float* const* dest, int ndest, int groups, long grp_dest_stride);
int32_t launch_reduce_partials(hipStream_t st, const float* partial, int nsplit, int nblk, long blk_elems,
                               float* const dest[4], int groups, long grp_dest_stride) {
  return launch_reduce_partials_n(st, partial, nsplit, nblk, blk_elems, dest, 4, groups, grp_dest_stride);
}
static int32_t launch_reduce_partials_n(hipStream_t st, const float* partial, int nsplit, int nblk, long blk_elems,
                                         float* const* dest, int ndest, int groups, long grp_dest_stride) {
  ReduceArgs r;
  r.partial = partial;
  r.nsplit = nsplit;
  r.nblk = nblk;
  r.blk_elems = blk_elems;
  for (int i = 0; i < 8; ++i) r.dest[i] = i < ndest ? dest[i] : nullptr;
  r.grp_dest_stride = grp_dest_stride;
  const int epb = reduce_epb(blk_elems, nsplit);
  const unsigned xb = reduce_xblocks(blk_elems, nsplit);
  const long wgs = (long)xb * nblk * groups;
  if (tl_reduce_queue && wgs > 0 && tl_reduce_queue->q.njobs < REDUCE_QUEUE_MAX &&
      tl_reduce_queue->q.off[tl_reduce_queue->q.njobs] + wgs <= REDUCE_QUEUE_WGS) {
    // collected: runs with the others when the scope is flushed
    ReduceQueueArgs& q = tl_reduce_queue->q;
    const int j = q.njobs++;
    q.job[j] = r;
    q.epb[j] = epb;
    q.xblocks[j] = (int)xb;
    q.off[j + 1] = q.off[j] + wgs;
    return HGNN_OK;
  }
  k_reduce_partials<<<dim3(xb, nblk, groups), 256, 0, st>>>(r, epb);
  HGNN_LAUNCH_CHECK("k_reduce_partials");
  return HGNN_OK;
}

// ---------------------------------------------------------------------------------------------
// transposed GEMM
// ---------------------------------------------------------------------------------------------
constexpr int WG_RC = 32;  // rows staged per step

template <int H>
struct WgradCfg {
  static constexpr int OT = H < 128 ? H : 128;  // output tile edge
  static constexpr int WT = OT / 2;             // per-wave edge (2 x 2 wavefronts)
  static constexpr int NB = WT / 32;
  static constexpr int STRIDE = OT + 4;         // LDS row pitch, fp32 operands
  static constexpr int BSTRIDE = OT + 16;       // bf16 operands (elements): four rows in four different groups of 8 banks
  static constexpr int TILES = H / OT;
};

// the jobs of one launch: their output tiles are numbered one job after the other (ny_off), and so are the B operands
// in the column-sum partials (cs_off). Jobs over the same rows share a partial buffer, blocks one job after the other;
// jobs over rows of their own have splits and a buffer of their own.
struct WgradJobs {
  WgradArgs job[3];
  int njobs;
  int ny_off[4], cs_off[4];
  int nsplit[3], rows_per_split[3];
  int nblk[3];            // blocks per split in the job's partial buffer
  float* partial[3];      // the job's first block of split 0
  float* colsum_partial;
};

// two transposing LDS reads: the eight rows of one lane's column (bf16)
typedef short s16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8_t lds_read_tr(const unsigned short* lo, const unsigned short* hi) {
  const s16x4_t l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(lo));
  const s16x4_t h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(hi));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int H, bool BF16>
__global__ void __launch_bounds__(256, 2) k_wgrad(WgradJobs m, int ny) {
  using C = WgradCfg<H>;
  // bf16 operands are rounded when they are staged and read back with the transposing LDS reads (two per operand of 16
  // rows, see wgrad_group() of the edge kernels). Kept as fp32 an operand was eight 4-byte reads and four conversions, done
  // by each of the two wavefronts that share it. Steps at H = 256: mixed batch of 643 structures 9.45 -> 9.38 ms, 64 crystals
  // 1651 -> 1636 us.
  using ST = typename std::conditional<BF16, unsigned short, float>::type;
  constexpr int SP = BF16 ? C::BSTRIDE : C::STRIDE;
  __shared__ __align__(16) ST sA[WG_RC * SP];
  __shared__ __align__(16) ST sB[WG_RC * SP];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wa = wave >> 1, wb = wave & 1;
  // Workgroups are dealt to the 8 XCDs round-robin. The ny workgroups that read the same rows (one per output tile)
  // take consecutive places on one XCD, so that they run at the same time behind the same L2 and the rows come
  // from memory once: split s lives on XCD s % 8.
  const int xcd = blockIdx.x & 7, place = blockIdx.x >> 3;
  const int split = (place / ny) * 8 + xcd, grp = blockIdx.z;
  int y = place % ny;
  int jb = 0;   // uniform over the workgroup
  if (m.njobs > 1 && y >= m.ny_off[1]) jb = 1;
  if (m.njobs > 2 && y >= m.ny_off[2]) jb = 2;
  y -= m.ny_off[jb];
  const int nsplit = m.nsplit[jb], rows_per_split = m.rows_per_split[jb];
  if (split >= nsplit || (grp > 0 && (!m.job[jb].grp_ptr || grp >= m.job[jb].S))) return;   // uniform over the workgroup (the grid covers whole groups of 8 splits of the largest job)
  const WgradArgs& p = m.job[jb];
  const int tb = y % C::TILES; y /= C::TILES;
  const int ta = y % C::TILES; y /= C::TILES;
  const int ib = y % p.nB;
  const int ia = y / p.nB;
  const int blkid = ia * p.nB + ib;
  long gbeg = 0, gend = p.M;
  if (p.grp_ptr) { gbeg = p.grp_ptr[grp]; gend = p.grp_ptr[grp + 1]; }
  long rbeg = gbeg + (long)split * rows_per_split;
  long rend = rbeg + rows_per_split;
  if (rend > gend) rend = gend;

  f32x16_t acc[C::NB][C::NB];
#pragma unroll
  for (int i = 0; i < C::NB; ++i)
#pragma unroll
    for (int j = 0; j < C::NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const float* __restrict__ A = p.A[ia];
  const float* __restrict__ B = p.B[ib];
  const int lda = p.lda[ia], ldb = p.ldb[ib];
  constexpr int CH = C::OT / 4;
  constexpr int ITER = WG_RC * CH / 256;   // 1, 2 or 4
  // the rows of step r0 (clamped to the last valid row; rows past the end are zeroed when they are staged). The
  // row indices are read first, under one uniform branch: with the test inside the loop every load waited for the
  // one before it.
  auto fetch = [&](long r0, float4 (&va)[ITER], float4 (&vb)[ITER]) {
    long gr[ITER];
#pragma unroll
    for (int u = 0; u < ITER; ++u) {
      const long pos = r0 + (tid + u * 256) / CH;
      gr[u] = pos < rend ? pos : rend - 1;
    }
    if (p.row_idx) {
#pragma unroll
      for (int u = 0; u < ITER; ++u) gr[u] = p.row_idx[gr[u]];
    }
#pragma unroll
    for (int u = 0; u < ITER; ++u) {
      const int q = (tid + u * 256) % CH;
      va[u] = *reinterpret_cast<const float4*>(A + gr[u] * lda + ta * C::OT + q * 4);
      vb[u] = *reinterpret_cast<const float4*>(B + gr[u] * ldb + tb * C::OT + q * 4);
    }
  };
  // column sums of this workgroup's B tile ride along where they are asked for (one workgroup per B tile: the
  // one of the first A block and the first A tile); a thread's chunk column is the same at every step
  const bool do_cs = m.colsum_partial != nullptr && (p.colsum_dest[0] || p.colsum_dest[1]) && ia == 0 && ta == 0;
  static_assert(256 % CH == 0, "a thread keeps its chunk column over the steps");
  float4 cs = make_float4(0.f, 0.f, 0.f, 0.f);
  // one step: the rows held in va / vb go to LDS, the registers are refilled with the rows two steps on (they travel
  // while this step and the next are multiplied), then the product
  auto step = [&](long r0, float4 (&va)[ITER], float4 (&vb)[ITER]) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ITER; ++u) {
      const int c = tid + u * 256;
      const int r = c / CH, q = c - r * CH;
      float4 a = va[u], b = vb[u];
      if (p.a_silu) { a.x = silu_f(a.x); a.y = silu_f(a.y); a.z = silu_f(a.z); a.w = silu_f(a.w); }
      if (r0 + r >= rend) { a = make_float4(0.f, 0.f, 0.f, 0.f); b = a; }
      cs.x += b.x; cs.y += b.y; cs.z += b.z; cs.w += b.w;
      if constexpr (BF16) {
        *reinterpret_cast<uint2*>(&sA[r * SP + q * 4]) = make_uint2(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w));
        *reinterpret_cast<uint2*>(&sB[r * SP + q * 4]) = make_uint2(pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w));
      } else {
        *reinterpret_cast<float4*>(&sA[r * SP + q * 4]) = a;
        *reinterpret_cast<float4*>(&sB[r * SP + q * 4]) = b;
      }
    }
    if (r0 + 2 * WG_RC < rend) fetch(r0 + 2 * WG_RC, va, vb);
    __syncthreads();
    if constexpr (BF16) {
#pragma unroll
      for (int ks = 0; ks < WG_RC / 16; ++ks) {
        // lane group g: rows 16 ks + 4 g + 0..3 and + 8 of its column, the same for both operands
        const int lo = (ks * 16 + 4 * (lane >> 5) + ((lane & 15) >> 2)) * SP + (lane & 16) + (lane & 3) * 4;
        bf16x8_t a[C::NB], b[C::NB];
#pragma unroll
        for (int i = 0; i < C::NB; ++i) {
          a[i] = lds_read_tr(&sA[lo + wa * C::WT + i * 32], &sA[lo + wa * C::WT + i * 32 + 8 * SP]);
          b[i] = lds_read_tr(&sB[lo + wb * C::WT + i * 32], &sB[lo + wb * C::WT + i * 32 + 8 * SP]);
        }
#pragma unroll
        for (int i = 0; i < C::NB; ++i)
#pragma unroll
          for (int j = 0; j < C::NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < WG_RC / 2; ++ks) {
        const int rr = ks * 2 + (lane >> 5);
        float a[C::NB], b[C::NB];
#pragma unroll
        for (int i = 0; i < C::NB; ++i) {
          a[i] = sA[rr * C::STRIDE + wa * C::WT + i * 32 + (lane & 31)];
          b[i] = sB[rr * C::STRIDE + wb * C::WT + i * 32 + (lane & 31)];
        }
#pragma unroll
        for (int i = 0; i < C::NB; ++i)
#pragma unroll
          for (int j = 0; j < C::NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    }
  };
  float4 va0[ITER], vb0[ITER], va1[ITER], vb1[ITER];
  if (rbeg < rend) fetch(rbeg, va0, vb0);
  if (rbeg + WG_RC < rend) fetch(rbeg + WG_RC, va1, vb1);
  for (long r0 = rbeg; r0 < rend; r0 += 2 * WG_RC) {
    step(r0, va0, vb0);
    if (r0 + WG_RC < rend) step(r0 + WG_RC, va1, vb1);
  }
  if (do_cs) {   // uniform over the workgroup: row phases are added in order through LDS
    __syncthreads();
    float4* sh = reinterpret_cast<float4*>(sA);
    sh[tid] = cs;
    __syncthreads();
    if (tid < CH) {
      float4 s = sh[tid];
      for (int k = 1; k < 256 / CH; ++k) {
        const float4 t = sh[k * CH + tid];
        s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
      }
      *reinterpret_cast<float4*>(m.colsum_partial + (((long)grp * nsplit + split) * m.cs_off[m.njobs] + m.cs_off[jb] + ib) * H + tb * C::OT + tid * 4) = s;
    }
  }
  float* out = m.partial[jb] + (((long)grp * nsplit + split) * m.nblk[jb] + blkid) * (long)(H * H);
#pragma unroll
  for (int i = 0; i < C::NB; ++i)
#pragma unroll
    for (int j = 0; j < C::NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int k1 = ta * C::OT + wa * C::WT + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        const int k2 = tb * C::OT + wb * C::WT + j * 32 + (lane & 31);
        out[k1 * H + k2] = acc[i][j][v];
      }
}

int wgrad_splits(int64_t M) {
  int64_t s = (M + 63) / 64;   // about 64 rows per split (two steps): short chains when there are few atoms
  if (s < 1) s = 1;
  if (s > 160) s = 160;
  return (int)s;
}

size_t wgrad_colsum_partial_floats(int H, int64_t M) { return (size_t)wgrad_splits(M) * 4 * H; }

size_t wgrad_partial_floats(int H, int64_t M, int nblocks, int S) {
  return (size_t)wgrad_splits(M) * nblocks * S * H * H;
}

// workgroups of k_wgrad that one CU holds at a time (asked once per variant)
template <int H, bool BF16>
static int wgrad_resident_wgs() {
  static int n = 0;
  if (n == 0) {
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, reinterpret_cast<const void*>(&k_wgrad<H, BF16>), 256, 0) !=
            hipSuccess || occ < 1)
      occ = 1;
    n = occ;
  }
  return n;
}

// splits of M rows for `ny` output tiles per split and group, and their rows
template <int H, bool BF16>
static int wgrad_plan(int64_t M, int ny, int groups, int& rows_per_split) {
  // Splits: never more than the workspace was sized for, and at most one round of resident workgroups (a second,
  // partly filled round costs a whole one). Split s runs on XCD s % 8, so the round is counted per XCD: a whole
  // number of splits on each of them (25 splits of 20 workgroups put 80 workgroups on the first XCD's 64 places
  // and doubled the kernel's time). Below one round: a whole number of workgroups per CU, so that no CU carries two
  // while its neighbour carries one. Fewer splits also mean fewer partials to write and add up.
  int nsplit = wgrad_splits(M);
  const long per_split = (long)ny * groups;
  const long xcd_places = (long)wgrad_resident_wgs<H, BF16>() * (num_cus() / 8);
  const long one_round = xcd_places / per_split >= 1 ? 8 * (xcd_places / per_split)
                                                     : (long)wgrad_resident_wgs<H, BF16>() * num_cus() / per_split;
  if (nsplit > one_round) {
    nsplit = one_round < 1 ? 1 : (int)one_round;
  } else {
    const long whole = nsplit * per_split / num_cus();
    if (whole >= 1) nsplit = (int)(whole * num_cus() / per_split);
  }
  if (nsplit < 1) nsplit = 1;   // many groups with few rows each: per_split alone can exceed the CU count
  int64_t rps = (M + nsplit - 1) / nsplit;
  rps = (rps + WG_RC - 1) / WG_RC * WG_RC;
  if (rps < WG_RC) rps = WG_RC;
  rows_per_split = (int)rps;
  return nsplit;
}

// own_rows: every job has its own rows, groups and partial buffer (as many launches in one); otherwise they share job 0's
template <int H, bool BF16>
static int32_t launch_wgrad_t(hipStream_t st, const WgradArgs* jobs, int njobs, bool own_rows) {
  using C = WgradCfg<H>;
  const WgradArgs& a = jobs[0];
  WgradJobs m;
  m.njobs = njobs;
  m.colsum_partial = nullptr;
  int blk_off[4] = {0, 0, 0, 0};
  m.ny_off[0] = m.cs_off[0] = 0;
  for (int j = 0; j < njobs; ++j) {
    m.job[j] = jobs[j];
    m.ny_off[j + 1] = m.ny_off[j] + jobs[j].nA * jobs[j].nB * C::TILES * C::TILES;
    blk_off[j + 1] = blk_off[j] + jobs[j].nA * jobs[j].nB;
    m.cs_off[j + 1] = m.cs_off[j] + jobs[j].nB;
    if (jobs[j].colsum_dest[0] || jobs[j].colsum_dest[1]) m.colsum_partial = a.colsum_partial;
  }
  const int nblk = blk_off[njobs];
  const int ny = m.ny_off[njobs];
  int most = 1, groups = 1;
  for (int j = 0; j < njobs; ++j) {
    const int gj = jobs[j].grp_ptr ? jobs[j].S : 1;
    if (gj > groups) groups = gj;
    if (own_rows) {
      m.nsplit[j] = wgrad_plan<H, BF16>(jobs[j].M, m.ny_off[j + 1] - m.ny_off[j], gj, m.rows_per_split[j]);
      m.nblk[j] = blk_off[j + 1] - blk_off[j];
      m.partial[j] = jobs[j].partial;
    } else {
      m.nsplit[j] = wgrad_plan<H, BF16>(a.M, ny, gj, m.rows_per_split[j]);
      m.nblk[j] = nblk;
      m.partial[j] = a.partial + (long)blk_off[j] * H * H;
    }
    if (m.nsplit[j] > most) most = m.nsplit[j];
  }
  for (int j = njobs; j < 3; ++j) m.ny_off[j + 1] = m.cs_off[j + 1] = 0;
  ProfScope ps(a.tag, st);
  k_wgrad<H, BF16><<<dim3((unsigned)((most + 7) / 8 * 8 * ny), 1, groups), 256, 0, st>>>(m, ny);
  HGNN_LAUNCH_CHECK("k_wgrad");
  if (own_rows) {
    for (int j = 0; j < njobs; ++j)
      HGNN_TRY(launch_reduce_partials_n(st, m.partial[j], m.nsplit[j], m.nblk[j], (long)H * H, jobs[j].dest, 4,
                                        jobs[j].grp_ptr ? jobs[j].S : 1, jobs[j].grp_dest_stride));
    return HGNN_OK;
  }
  float* dest[8] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  float* cd[4] = {nullptr, nullptr, nullptr, nullptr};
  for (int j = 0; j < njobs; ++j) {
    for (int b = 0; b < jobs[j].nA * jobs[j].nB; ++b) dest[blk_off[j] + b] = jobs[j].dest[b];
    for (int b = 0; b < jobs[j].nB; ++b) cd[m.cs_off[j] + b] = jobs[j].colsum_dest[b];
  }
  HGNN_TRY(launch_reduce_partials_n(st, a.partial, m.nsplit[0], nblk, (long)H * H, dest, 8, groups, a.grp_dest_stride));
  if (m.colsum_partial) HGNN_TRY(launch_reduce_partials_n(st, m.colsum_partial, m.nsplit[0], m.cs_off[njobs], H, cd, 4, 1, 0));
  return HGNN_OK;
}

template <bool BF16>
static int32_t launch_wgrad_h(hipStream_t st, int H, const WgradArgs* jobs, int njobs, bool own_rows) {
  switch (H) {
    case 64: return launch_wgrad_t<64, BF16>(st, jobs, njobs, own_rows);
    case 128: return launch_wgrad_t<128, BF16>(st, jobs, njobs, own_rows);
    case 256: return launch_wgrad_t<256, BF16>(st, jobs, njobs, own_rows);
  }
  return set_error(HGNN_ERR_BAD_SHAPE, "H must be 64, 128 or 256 (got %d)", H);
}

int32_t launch_wgrad_multi(hipStream_t st, int H, bool bf16, const WgradArgs* jobs, int njobs) {
  HGNN_REQUIRE(jobs && njobs >= 1 && njobs <= 3, HGNN_ERR_BAD_SHAPE, "wgrad: one to three jobs");
  int blocks = 0, nb = 0;
  for (int j = 0; j < njobs; ++j) {
    const WgradArgs& a = jobs[j];
    HGNN_REQUIRE(a.nA >= 1 && a.nB >= 1 && a.nA * a.nB <= 4, HGNN_ERR_BAD_SHAPE, "wgrad: bad block counts");
    HGNN_REQUIRE(a.A[0] && a.B[0] && a.dest[0], HGNN_ERR_NULLPTR, "wgrad: null operand");
    HGNN_REQUIRE(!(a.colsum_dest[0] || a.colsum_dest[1]) || jobs[0].colsum_partial, HGNN_ERR_NULLPTR, "wgrad: no room for the column sums");
    HGNN_REQUIRE(njobs == 1 || (!a.grp_ptr && !a.row_idx && a.M == jobs[0].M), HGNN_ERR_BAD_SHAPE,
                 "wgrad: several jobs share their rows (no groups, no row indirection)");
    blocks += a.nA * a.nB;
    nb += a.nB;
  }
  HGNN_REQUIRE(jobs[0].partial, HGNN_ERR_NULLPTR, "wgrad: null partial buffer");
  HGNN_REQUIRE(blocks <= 8 && nb <= 4, HGNN_ERR_BAD_SHAPE, "wgrad: too many blocks in one launch");
  HGNN_REQUIRE(!(jobs[0].colsum_partial && (jobs[0].colsum_dest[0] || jobs[0].colsum_dest[1])) || !jobs[0].grp_ptr,
               HGNN_ERR_BAD_SHAPE, "wgrad: column sums are not available per group");
  return bf16 ? launch_wgrad_h<true>(st, H, jobs, njobs, false) : launch_wgrad_h<false>(st, H, jobs, njobs, false);
}

int32_t launch_wgrad_own_rows(hipStream_t st, int H, bool bf16, const WgradArgs* jobs, int njobs) {
  HGNN_REQUIRE(jobs && njobs >= 1 && njobs <= 3, HGNN_ERR_BAD_SHAPE, "wgrad: one to three jobs");
  for (int j = 0; j < njobs; ++j) {
    const WgradArgs& a = jobs[j];
    HGNN_REQUIRE(a.nA >= 1 && a.nB >= 1 && a.nA * a.nB <= 4, HGNN_ERR_BAD_SHAPE, "wgrad: bad block counts");
    HGNN_REQUIRE(a.A[0] && a.B[0] && a.dest[0] && a.partial, HGNN_ERR_NULLPTR, "wgrad: null operand");
    HGNN_REQUIRE(!a.colsum_dest[0] && !a.colsum_dest[1], HGNN_ERR_BAD_SHAPE, "wgrad: no column sums here");
  }
  // One launch saves a launch, which counts where both are short or of few groups; beyond that a few long workgroups among
  // many short ones end up sharing compute units. Reverse pass of the heads, apart -> in one launch, H = 128 fp32: 16,000 atoms
  // and 8,000 graphs of one group 69 -> 60 us, 40,000 atoms of 5 groups 115 -> 132, 18,000 atoms of 32 groups 184 -> 267.
  bool one = true;
  for (int j = 0; j < njobs; ++j) {
    const int groups = jobs[j].grp_ptr ? jobs[j].S : 1;
    one = one && (groups <= 4 || (jobs[j].M + 31) / 32 + groups <= num_cus());
  }
  if (!one) {
    for (int j = 0; j < njobs; ++j)
      HGNN_TRY(bf16 ? launch_wgrad_h<true>(st, H, jobs + j, 1, true) : launch_wgrad_h<false>(st, H, jobs + j, 1, true));
    return HGNN_OK;
  }
  return bf16 ? launch_wgrad_h<true>(st, H, jobs, njobs, true) : launch_wgrad_h<false>(st, H, jobs, njobs, true);
}

// ---------------------------------------------------------------------------------------------
// column sums
// ---------------------------------------------------------------------------------------------
// up to four column sums in one launch, each over its own rows: the splits of all jobs one after the other (blockIdx.x; with
// the jobs in z, 500 groups of two rows beside 500 of 40,000 were 625,000 workgroups without work, 120 us)
struct ColsumJobs {
  ColsumArgs job[4];
  int nsplit[4], rows_per_split[4], off[4];   // off: first split of the job (past the last one for jobs that are not there)
};
__global__ void __launch_bounds__(256) k_colsum(ColsumJobs m, int H) {
  const int jb = ((int)blockIdx.x >= m.off[1]) + ((int)blockIdx.x >= m.off[2]) + ((int)blockIdx.x >= m.off[3]);   // uniform
  const ColsumArgs& p = m.job[jb];
  const int nsplit = m.nsplit[jb], rows_per_split = m.rows_per_split[jb];
  // thread = (4-column chunk q, row phase ph); every phase walks its rows with four loads in flight
  __shared__ float4 sh[256];
  __shared__ float shw[16];   // sum of the weights of every phase
  const int tid = threadIdx.x;
  const int CH = H >> 2;
  const int q = tid % CH, ph = tid / CH, nph = 256 / CH;
  const int split = (int)blockIdx.x - m.off[jb], grp = blockIdx.y;
  if (grp > 0 && (!p.grp_ptr || grp >= p.S)) return;   // uniform over the workgroup
  long gbeg = 0, gend = p.M;
  if (p.grp_ptr) { gbeg = p.grp_ptr[grp]; gend = p.grp_ptr[grp + 1]; }
  float ws = 0.f;   // this phase's sum of the weights
  long rbeg = gbeg + (long)split * rows_per_split;
  long rend = rbeg + rows_per_split;
  if (rend > gend) rend = gend;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (rbeg >= rend) {   // uniform: most splits of most groups where there are many groups
    if (ph == 0) *reinterpret_cast<float4*>(p.partial + ((long)grp * nsplit + split) * H + q * 4) = s;
    if (p.w_dest && tid == 64) p.w_partial[(long)grp * nsplit + split] = 0.f;
    return;
  }
  for (long r0 = rbeg + ph; r0 < rend; r0 += 4 * nph) {
    float4 xv[4];
    float wv[4];
    long gr[4];
    // (indices, rows and weights each under one uniform branch: with the tests inside the loop the loads wait for
    // one another)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long r = r0 + (long)u * nph;
      gr[u] = r < rend ? r : rend - 1;
      wv[u] = 1.f;
    }
    if (p.row_idx) {
#pragma unroll
      for (int u = 0; u < 4; ++u) gr[u] = p.row_idx[gr[u]];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) xv[u] = *reinterpret_cast<const float4*>(p.X + gr[u] * p.ldx + q * 4);
    if (p.w) {
#pragma unroll
      for (int u = 0; u < 4; ++u) wv[u] = p.w[gr[u]];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (r0 + (long)u * nph >= rend) wv[u] = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float4 x = xv[u];
      if (p.f_silu) { x.x = silu_f(x.x); x.y = silu_f(x.y); x.z = silu_f(x.z); x.w = silu_f(x.w); }
      s.x += wv[u] * x.x; s.y += wv[u] * x.y; s.z += wv[u] * x.z; s.w += wv[u] * x.w;
      ws += wv[u];
    }
  }
  sh[tid] = s;
  if (q == 0) shw[ph] = ws;
  __syncthreads();
  if (ph == 0) {
    for (int k = 1; k < nph; ++k) {
      const float4 t = sh[k * CH + q];
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    *reinterpret_cast<float4*>(p.partial + ((long)grp * nsplit + split) * H + q * 4) = s;
  }
  if (p.w_dest && tid == 64) {   // (another wavefront than the columns': CH <= 64)
    ws = shw[0];
    for (int k = 1; k < nph; ++k) ws += shw[k];
    p.w_partial[(long)grp * nsplit + split] = ws;
  }
}

static int colsum_splits(int64_t M) {
  int64_t s = (M + 63) / 64;   // 64 rows per workgroup: four trips of loads each (at 256 rows a workgroup's chain of trips set the kernel's time)
  if (s < 1) s = 1;
  if (s > 1024) s = 1024;
  return (int)s;
}

size_t colsum_partial_floats(int H, int64_t M, int S) { return (size_t)colsum_splits(M) * S * H; }

int32_t launch_colsum_multi(hipStream_t st, int H, const ColsumArgs* jobs, int njobs) {
  HGNN_REQUIRE(jobs && njobs >= 1 && njobs <= 4, HGNN_ERR_BAD_SHAPE, "colsum: one to four jobs");
  HGNN_REQUIRE(valid_H(H), HGNN_ERR_BAD_SHAPE, "H must be 64, 128 or 256 (got %d)", H);
  ColsumJobs m;
  int splits = 0, groups = 1;
  for (int j = 0; j < njobs; ++j) {
    const ColsumArgs& a = jobs[j];
    HGNN_REQUIRE(a.X && a.dest && a.partial, HGNN_ERR_NULLPTR, "colsum: null operand");
    HGNN_REQUIRE(!a.w_dest || (a.w && a.w_partial), HGNN_ERR_NULLPTR, "colsum: null weights");
    m.job[j] = a;
    m.nsplit[j] = colsum_splits(a.M);
    const int64_t rps = (a.M + m.nsplit[j] - 1) / m.nsplit[j];
    m.rows_per_split[j] = rps < 1 ? 1 : (int)rps;
    m.off[j] = splits;
    splits += m.nsplit[j];
    if (a.grp_ptr && a.S > groups) groups = a.S;
  }
  for (int j = njobs; j < 4; ++j) m.off[j] = splits;
  ProfScope ps(PT_COLSUM, st);
  k_colsum<<<dim3(splits, groups), 256, 0, st>>>(m, H);
  HGNN_LAUNCH_CHECK("k_colsum");
  for (int j = 0; j < njobs; ++j) {
    const ColsumArgs& a = jobs[j];
    const int g = a.grp_ptr ? a.S : 1;
    float* dest[4] = {a.dest, nullptr, nullptr, nullptr};
    HGNN_TRY(launch_reduce_partials(st, a.partial, m.nsplit[j], 1, H, dest, g, a.grp_dest_stride));
    if (a.w_dest) {
      float* wd[4] = {a.w_dest, nullptr, nullptr, nullptr};
      HGNN_TRY(launch_reduce_partials(st, a.w_partial, m.nsplit[j], 1, 1, wd, g, a.grp_dest_stride));
    }
  }
  return HGNN_OK;
}

}  // namespace hgnn
