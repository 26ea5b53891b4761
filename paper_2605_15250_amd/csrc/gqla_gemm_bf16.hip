// The two dense contractions around the decode kernels, bf16 MFMA with fp32 accumulation:
//   query absorption  q_hat = W_UK[j] q_C              (paper Sec. 3.1, MQA-absorb equation, line 1)
//   cache expansion   K_C = W_UK^T c,  V = W_UV^T c    (Sec. 3.1, "Two equivalent decoding paths": one-shot expand)
#include <algorithm>

#include "gqla_device.h"
#include "gqla_lds.h"

namespace gqla {

namespace {

// ---- query absorption ------------------------------------------------------------------------------------
// One wave per (group j, 32 query rows of the group, 128 latent dims):
//   Qhat^T[r][row] = W_UK[j][r][d] * Q_C^T[d][row]   A = weight rows straight from global (d contiguous),
//                                                    B = query rows straight from global.
template <int DH, int RKV>
__global__ void __launch_bounds__(256) absorb_query_bf16_kernel(AbsorbQueryArgs a, int rows_per_group) {
  constexpr int KS = DH / 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 31, h = lane >> 5;
  const int j = blockIdx.z;
  const int rblk = blockIdx.y * 4 + wave;  // 128 latent dims each
  if (rblk * 128 >= RKV) return;
  const int x = blockIdx.x * 32 + n;       // x = row * G + head-in-group, row = b * s_q + t
  const bool row_ok = x < rows_per_group;
  const int64_t qrow = row_ok ? (int64_t)(x / a.G) * a.h_q + j * a.G + x % a.G : 0;
  bf16x8 qf[KS];
  const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = row_ok ? *(const bf16x8*)((const __bf16*)a.q_c + qrow * DH + ks * 16 + h * 8) : zero;
  const __bf16* w = (const __bf16*)a.w_uk + ((int64_t)j * RKV + rblk * 128 + n) * DH + h * 8;
  f32x16 acc[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[mt][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc[mt] = mfma32(*(const bf16x8*)(w + (int64_t)mt * 32 * DH + ks * 16), qf[ks], acc[mt]);
  }
  if (!row_ok) return;
  __bf16* out = (__bf16*)a.q_hat + qrow * RKV + rblk * 128;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u32x2 v = {pack_bf16(acc[mt][4 * q], acc[mt][4 * q + 1]), pack_bf16(acc[mt][4 * q + 2], acc[mt][4 * q + 3])};
      *(u32x2*)(out + mt * 32 + 8 * q + 4 * h) = v;
    }
}

// The same product for d_h = 128 with both sides of the kernel coalesced (the call is a short kernel in front of every
// absorb decode, and what it costs is how many memory lines its instructions touch): one workgroup per group j and share of
// RKV / SHARES latent dims, for one or more blocks of 32 query rows of the group; a wave takes a quarter of the share.  The
// share's rows of W_UK[j] (256 bytes each, contiguous) are staged in LDS once, with LDS-DMA, 1 KB of consecutive memory per
// instruction, and read back as conflict-free A fragments; the results go back through LDS so that a store instruction writes
// whole lines of rows instead of 8-byte pieces of 32 rows.  Same MFMAs in the same order as the kernel above.
// SHARES: with few row blocks the staging of 128 KB by one compute unit is most of the call, so it is shared out; with more
// than a round of workgroups they keep their weights and walk over the row blocks, the next block's queries in flight.
// Measured: one sequence, 128 heads in 8 groups 5.2 -> 3.5 us (8 -> 32 workgroups); 128 sequences x 2 tokens, 1024 blocks
// 24.3 -> 17.9 us (256 workgroups of four blocks; q_c read and q_hat written once are 42 MB, 6 us).
template <int RKV, int SHARES>
__global__ void __launch_bounds__(256) absorb_query_staged_bf16_kernel(AbsorbQueryArgs a, int rows_per_group) {
  constexpr int DH = 128, KS = DH / 16;
  constexpr int ROWS = RKV / SHARES;              // latent dims of the workgroup
  constexpr int MT = ROWS / 128;                  // 32-dim tiles of a wave
  constexpr int MP = MT < 2 ? MT : 2;             // ... that leave through LDS together
  constexpr int PITCH = MP * 64 + 16;             // bytes per row of the output tile in LDS
  constexpr int LPR = MP * 4;                     // lanes per row of a store
  static_assert(RKV == 512 && (SHARES == 1 || SHARES == 2 || SHARES == 4), "four waves x 32 to 128 latent dims");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int j = blockIdx.z, dim0 = blockIdx.y * ROWS;
  stage_panels_full<ROWS, DH / 64, 4, DH * 2>(smem, (const char*)a.w_uk + ((int64_t)j * RKV + dim0) * DH * 2, wave, lane);
  char* tile = smem + ROWS * DH * 2 + wave * (32 * PITCH);  // read by this wave only
  auto query_row = [&](int x) -> int64_t { return (int64_t)(x / a.G) * a.h_q + j * a.G + x % a.G; };  // x = row * G + head-in-group
  bf16x8 qf[KS];
  auto load_queries = [&](int blk) {              // rows beyond the last: that one (not stored)
    const __bf16* q = (const __bf16*)a.q_c + query_row(min(blk * 32 + n, rows_per_group - 1)) * DH + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(q + ks * 16);
  };
  const int n_blocks = (rows_per_group + 31) / 32;
  load_queries(blockIdx.x);
  wait_all_memory();
  __syncthreads();  // the weights are staged
  for (int blk = blockIdx.x; blk < n_blocks; blk += gridDim.x) {
    f32x16 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mt][i] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) acc[mt] = mfma32(row_frag<ROWS>(smem, (MT * wave + mt) * 32 + n, 2 * ks + h), qf[ks], acc[mt]);
    }
    if (blk + (int)gridDim.x < n_blocks) load_queries(blk + gridDim.x);
#pragma unroll
    for (int m0 = 0; m0 < MT; m0 += MP) {
#pragma unroll
      for (int mt = 0; mt < MP; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16 x = acc[m0 + mt];
          *(u32x2*)(tile + n * PITCH + (mt * 32 + 8 * q + 4 * h) * 2) = u32x2{pack_bf16(x[4 * q], x[4 * q + 1]), pack_bf16(x[4 * q + 2], x[4 * q + 3])};
        }
      // (the compiler's wait for the LDS writes is all the ordering needed)
#pragma unroll
      for (int p = 0; p < 32 * LPR / 64; ++p) {
        const int r = (64 / LPR) * p + lane / LPR, c = lane % LPR;
        const u32x4 v = *(const u32x4*)(tile + r * PITCH + c * 16);
        if (blk * 32 + r < rows_per_group)
          *(u32x4*)((__bf16*)a.q_hat + query_row(blk * 32 + r) * RKV + dim0 + (MT * wave + m0) * 32 + c * 8) = v;
      }
    }
  }
}

// MFMAs written out so that the latent fragments can live in the accumulation registers (the compiler's own selection
// keeps A and B operands in ordinary registers only): c (+)= A * B with one operand in an AGPR quad.  The *_first forms
// start a sum from zero.  Dependent MFMAs on one accumulator interlock in hardware; before any other instruction reads
// the results, mfma_results_ready() covers the 16-pass latency of the last one.
__device__ __forceinline__ void mfma_va(f32x16& c, bf16x8 a_vgpr, bf16x8 b_agpr) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a_vgpr), "a"(b_agpr));
}
__device__ __forceinline__ void mfma_va_first(f32x16& c, bf16x8 a_vgpr, bf16x8 b_agpr) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a_vgpr), "a"(b_agpr));
}
__device__ __forceinline__ void mfma_av(f32x16& c, bf16x8 a_agpr, bf16x8 b_vgpr) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "a"(a_agpr), "v"(b_vgpr));
}
__device__ __forceinline__ void mfma_av_first(f32x16& c, bf16x8 a_agpr, bf16x8 b_vgpr) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "a"(a_agpr), "v"(b_vgpr));
}
__device__ __forceinline__ void mfma_results_ready(f32x16& c0, f32x16& c1, f32x16& c2, f32x16& c3) {
  asm volatile("s_nop 15\n\ts_nop 7" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
}

// ---- cache expansion -----------------------------------------------------------------------------------------
// Step 1 (tiny): the weights of the expanded groups are repacked once per call into MFMA fragment order.  A "stage"
// is one 64-column block of one group's W_UK or W_UV; a group has DH/64 key stages followed by DV/64 value stages
// (DH = DV = 128: two and two; the shape of Sec. 3.2.2, DH = 192 and DV = 256: three and four):
//   packed[jj * (DH + DV)/64 + sub][ks][e][lane][8]  with  lane (m = l % 32, h = l / 32), element i  =
//   W_kind[group_begin + jj][r = 16*ks + 8*h + i][d = 64*mtp + 32*e + m],   (kind, mtp) = stage_kind<DH>(sub)
// i.e. each 1 KB block is one A fragment of W^T (or, with the same register contents, one B fragment of W), and each
// stage is one contiguous 64 KB.
// One workgroup per (stage, 4 k-steps): a [64 latent dims][64 columns] tile of W goes through LDS, read with whole
// 16-byte vectors along the rows and written as whole fragments.
template <int DH, int DV, int RKV>
__global__ void __launch_bounds__(256) pack_weights_bf16_kernel(ExpandArgs a, __bf16* packed) {
  constexpr int KS = RKV / 16;
  constexpr int NSK = DH / 64, NSUB = (DH + DV) / 64;
  __shared__ __attribute__((aligned(16))) __bf16 tile[64][64 + 8];  // rows padded by one vector: column reads spread over the banks
  const int stage = blockIdx.x;  // jj * NSUB + sub
  const int kq = blockIdx.y;     // k-steps 4*kq .. 4*kq + 3
  const int jj = stage / NSUB, sub = stage % NSUB;
  const int kind = sub >= NSK, mtp = kind ? sub - NSK : sub;
  const int dim = kind ? DV : DH;  // columns of this kind's weight
  const __bf16* w = (const __bf16*)(kind ? a.w_uv : a.w_uk) + ((int64_t)(a.group_begin + jj) * RKV + 64 * kq) * dim + 64 * mtp;
  for (int v = threadIdx.x; v < 512; v += 256) {
    const int r = v >> 3, c = (v & 7) * 8;
    *(u32x4*)&tile[r][c] = *(const u32x4*)(w + (int64_t)r * dim + c);
  }
  __syncthreads();
  __bf16* out = packed + (int64_t)stage * KS * 2 * 512 + (int64_t)(4 * kq) * 2 * 512;
  for (int v = threadIdx.x; v < 512; v += 256) {
    const int lane = v & 63, e = (v >> 6) & 1, ksl = v >> 7;
    const int m = lane & 31, h = lane >> 5;
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = tile[16 * ksl + 8 * h + i][32 * e + m];
    *(bf16x8*)(out + (ksl * 2 + e) * 512 + lane * 8) = o;
  }
}

// Step 2: one workgroup of 4 waves per 256-token block of a sequence; wave w owns 64 tokens (two 32-token tiles) and,
// alone on its SIMD, the whole 512-entry register file.  Each wave keeps its tokens' latent rows as 2 x 32 register
// fragments (lane = token, 8 consecutive latent dims per k-step) and reuses them for every group and for both K and V,
// so the latent is read from HBM once.  The packed weights stream through LDS one 64 KB stage at a time (LDS-DMA,
// double buffered, the next stage in flight while the current one is multiplied); every weight fragment read from LDS
// feeds two MFMAs (one per token tile):
//   K^T[d][tok] = W_UK^T[d][r] * C^T[r][tok]     A = weight fragment, B = latent fragment
//   V[tok][d]   = C[tok][r]    * W_UV[r][d]      A = latent fragment, B = weight fragment (same register contents)
// The two output orientations put 4 consecutive dims (K plane) or 4 consecutive tokens (V plane) of the expanded
// page's 8-element vectors in one lane.  A stage's results are stored while the next stage is being multiplied, so
// that the end-of-stage wait (which also covers stores on this hardware) finds them long gone.
// With an odd number of stages per group (DH = 192, DV = 256: seven) the two result sets would meet at the group
// boundary, so there the group's last stage stores its results at once instead of in the next stage's shadow.
__host__ __device__ __forceinline__ int expand_parts(int rest, int groups) {  // shares of the groups for `rest` blocks of a round
  int p = 256 / rest;
  if (p > groups) p = groups;
  const int per = (groups + p - 1) / p;
  return (groups + per - 1) / per;   // no more shares than that size of share needs
}

// One block of 256 tokens (block `blk` of sequence b, which has L) and groups jj_begin .. jj_begin + jj_count - 1 of the slice.
// DIRECT: the weights come as the caller holds them, without step 1 (a launch of 5 us, as much as a short call's second): a stage
// is staged as a panel of [512 latent dims][128 bytes] (gqla_lds.h) and its fragments are read transposed, two reads each.
template <int DH, int DV, int RKV, int DR, bool FP8, bool DIRECT>
__device__ __forceinline__ void expand_block(const ExpandArgs& a, const __bf16* packed, char* smem, int b, int blk, int L, int jj_begin, int jj_count) {
  constexpr int W = RKV + DR;
  constexpr int KS = RKV / 16;
  constexpr int STAGE_BYTES = KS * 2 * 1024;  // 64 KB
  constexpr int DEPTH = 2;                    // weight fragments are fetched this many k-steps ahead
  constexpr int NSK = DH / 64, NSUB = (DH + DV) / 64;  // key stages, all stages of a group
  constexpr bool ODD = (NSUB & 1) != 0;
  static_assert(DH % 64 == 0 && DV % 64 == 0, "64-column stages");
  static_assert(!FP8 || (DH == 128 && DV == 128), "the 8-bit page format is written for equal dims of 128");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int P = a.latent.page_size;
  const int gc = a.group_count;
  const int tok0 = blk * 256;
  const int tokw = tok0 + wave * 64;  // first token of this wave (a wave never straddles a page: P % 64 == 0)
  int32_t pg_in = -1, pg_out = -1;
  if (tokw < L) {
    pg_in = page_of_uniform(a.latent, b, tokw / P);
    pg_out = page_of_uniform(a.expanded, b, tokw / P);
  }
  const bool wave_ok = pg_in >= 0 && pg_out >= 0;  // wave-uniform
  const int slot0 = tokw % P;

  // latent rows of this wave's 64 tokens as fragments, loaded straight into aligned AGPR quads.  Rows past L_b read a
  // clamped (valid) address instead: a token is one MFMA column (K) or row (V), so whatever such a lane computes
  // stays in that token's outputs, and those are never stored.
  bf16x8 xf[2][KS];
  const __bf16* in_page = (const __bf16*)a.latent.pool + (int64_t)(wave_ok ? pg_in : 0) * P * W;
  // FP8: `expanded` is an 8-bit cache (E4M3 code planes and a 16-bit k_R plane, see the header): 2 gc DH + 2 DR bytes per token
  constexpr int EB = FP8 ? 1 : 2;  // bytes per K_C / V element
  char* const page_bytes = (char*)a.expanded.pool + (int64_t)(wave_ok ? pg_out : 0) * P * (gc * (DH + DV) * EB + 2 * DR);
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const bool tok_ok = wave_ok && (tokw + 32 * nt + n < L);
    const __bf16* in_row = in_page + (int64_t)(slot0 + (tok_ok ? 32 * nt + n : 0)) * W;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      asm volatile("global_load_dwordx4 %0, %1, off" : "=a"(xf[nt][ks]) : "v"(in_row + ks * 16 + h * 8));
  }

  // LDS-DMA of one stage: 64 instructions of 1 KB, 16 per wave, linear (the packed layout is already fragment order).  DIRECT: 8
  // rows x 128 bytes of column block `mtp` of a weight matrix; the swizzle of a lane's row alternates with u.
  uint32_t w_off[2][2];  // [kind][u & 1]
#pragma unroll
  for (int i = 0; i < 4; ++i) w_off[i >> 1][i & 1] = (lane >> 3) * ((i >> 1 ? DV : DH) * 2) + (((lane & 7) ^ lds_swz(8 * (i & 1) + (lane >> 3))) << 4);
  const TrNatural tr = make_tr_natural(lane);
  auto stage_in_step = [&](int stage, auto SUBT, char* buf, int u) {  // u = 0..15; SUBT: stage % NSUB
    const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)(buf + wave * (16 * 1024)));
    if constexpr (DIRECT) {
      constexpr int sub = decltype(SUBT)::value, kind = sub >= NSK, mtp = kind ? sub - NSK : sub, dim = kind ? DV : DH;
      const int jj = stage / NSUB;
      const char* src = (const char*)(kind ? a.w_uv : a.w_uk) + (((int64_t)(a.group_begin + jj_begin + jj) * RKV + 8 * (16 * wave + u)) * dim + 64 * mtp) * 2;
      const uint32_t off = w_off[kind][u & 1];
      asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off), "s"(src), "n"(u * 1024) : "memory", "scc");
    } else {
      const char* src = (const char*)packed + (int64_t)stage * STAGE_BYTES + wave * (16 * 1024) + u * 1024;
      const uint32_t off = lane * 16;
      asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst), "v"(off), "s"(src), "n"(u * 1024) : "memory", "scc");  // the add writes SCC
    }
  };
  auto stage_in = [&](int stage, auto SUBT, char* buf) {
    static_for<16>([&](auto U) { stage_in_step(stage, SUBT, buf, decltype(U)::value); });
  };
  // results of the previous stage ([token tile][32-column half]), kept until the next stage's arithmetic is under way
  f32x16 accs[2][2][2];  // [stage parity][token tile][32-column half]: one set accumulates while the other is stored
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int k = 0; k < 16; ++k) accs[i >> 2][(i >> 1) & 1][i & 1][k] = 0.f;
  // stores address the page through one uniform base and 32-bit offsets (a page is at most a few MB)
  const uint32_t plane_k = (uint32_t)DH * P, plane_v = (uint32_t)DV * P;          // elements of one group's K and V plane
  // from here on groups are counted from the share's first: its offset is in these and in `packed`
  if (!DIRECT) packed += (int64_t)jj_begin * NSUB * (STAGE_BYTES / 2);
  const uint32_t k_lane = (uint32_t)jj_begin * plane_k + (uint32_t)(slot0 + n) * 8 + (uint32_t)h * P * 8;   // K plane: token slot0 + n, 8-dim block + h
  const uint32_t v_lane = (uint32_t)jj_begin * plane_v + (uint32_t)((slot0 >> 3) + h) * DV * 8 + n * 8;     // V plane: dim n, 8-token block slot0/8 + h
  const bool wave_full = tokw + 64 <= L;                                          // no token of this wave lies beyond L_b
  // One 16-byte store per lane: piece (nt, e, qp) of the previous stage's results; kind, mtp and the piece are compile-time.
  // A lane holds rows 4h..4h+3 of each 8-row block of its column; the two half-waves trade so that lane (n, h) ends up
  // with all 8 rows of block 2*qp + h, i.e. one complete vector of the page layout.
  // 8-bit destination: one 16-byte store per lane and (nt, e): the 32 results of the lane's column as the two code
  // vectors of the page layout (a vector holds 8-row blocks h' and 2 + h' of the 32 rows, each block 4 rows from either
  // half-wave); every result is rounded to bf16 first, so that the codes are those of expanding and then converting.
  auto store_prev8 = [&](int par, int kind, int mtp, int jj, int nt, int e) {
    if (jj < 0 || !wave_ok) return;
    const f32x16& acc = accs[par][nt][e];
    const float inv = kind == 0 ? a.k_inv_scale : a.v_inv_scale;
    uint32_t code[4];  // code[q] = rows 8q + 4h + 0..3
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float x0 = acc[4 * q], x1 = acc[4 * q + 1], x2 = acc[4 * q + 2], x3 = acc[4 * q + 3];
      round_to_bf16x2(x0, x1);
      round_to_bf16x2(x2, x3);
      code[q] = quantize_e4m3x4(x0, x1, x2, x3, inv);
    }
    uint32_t r0, r1, r2, r3;
    half_swap(code[0], code[1], r0, r1);  // lower half: block 0 own, block 0 of the upper half; upper: block 1 of the lower half, block 1 own
    half_swap(code[2], code[3], r2, r3);
    const u32x4 v = {r0, r1, r2, r3};
    if (kind == 0) {
      // lane = token; vector h of pair kp = 2 mtp + e of the K8 plane
      if (wave_full || tokw + 32 * nt + n < L) {
        const uint32_t off = ((uint32_t)(jj * (DH / 16) + 2 * (2 * mtp + e) + h) * P + slot0 + 32 * nt + n) * 16 + jj_begin * plane_k;
        __builtin_nontemporal_store(v, (u32x4*)(page_bytes + off));
      }
    } else {
      // lane = dim 64 mtp + 32 e + n; vector h of 32-token tile (slot0 + 32 nt) / 32 of the V8 plane: tokens 8h + 0..7, 16 + 8h + 0..7
      const uint32_t off = (uint32_t)(gc + jj_begin) * plane_k +
                           (((uint32_t)(jj * (P / 32) + (slot0 >> 5) + nt) * DH + 64 * mtp + 32 * e + n) * 2 + h) * 16;
      char* dst = page_bytes + off;
      const int tk = tokw + 32 * nt + 8 * h;  // first token of the vector's first half; the second half starts 16 later
      if (wave_full || tk + 23 < L) {
        __builtin_nontemporal_store(v, (u32x4*)dst);
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (tk + 16 * (i >> 3) + (i & 7) < L) dst[i] = (char)((v[i >> 2] >> (8 * (i & 3))) & 0xffu);
      }
    }
  };
  // The two halves of a store are separate so that each fits in the shadow of one matrix instruction: pack_prev rounds
  // and trades (6 vector instructions), emit_prev forms the address and stores.
  auto pack_prev = [&](int par, int nt, int e, int qp) -> u32x4 {
    const f32x16& acc = accs[par][nt][e];
    const int q0 = 2 * qp;
    const uint32_t x0 = pack_bf16(acc[4 * q0], acc[4 * q0 + 1]), x1 = pack_bf16(acc[4 * q0 + 2], acc[4 * q0 + 3]);
    const uint32_t y0 = pack_bf16(acc[4 * q0 + 4], acc[4 * q0 + 5]), y1 = pack_bf16(acc[4 * q0 + 6], acc[4 * q0 + 7]);
    uint32_t r0, r1, r2, r3;
    half_swap(x0, y0, r0, r2);
    half_swap(x1, y1, r1, r3);
    return u32x4{r0, r1, r2, r3};
  };
  auto emit_prev = [&](const u32x4 v, int kind, int mtp, int jj, int nt, int e, int qp) {
    if (jj < 0 || !wave_ok) return;
    const int q0 = 2 * qp;
    if (kind == 0) {
      // lane = token; the vector is dims 64*mtp + 32*e + 8*(2*qp + h) + 0..7 of the K plane
      if (wave_full || tokw + 32 * nt + n < L) {
        const uint32_t off = (uint32_t)jj * plane_k + (uint32_t)(8 * mtp + 4 * e + q0) * P * 8 + 32 * nt * 8 + k_lane;
        __builtin_nontemporal_store(v, (u32x4*)(page_bytes + (size_t)off * 2));
      }
    } else {
      // lane = dim 64*mtp + 32*e + n; the vector is tokens 32*nt + 8*(2*qp + h) + 0..7 of the V plane
      const uint32_t off = (uint32_t)gc * plane_k + (uint32_t)jj * plane_v + (uint32_t)(4 * nt + q0) * DV * 8 + (2 * mtp + e) * 32 * 8 + v_lane;
      __bf16* dst = (__bf16*)(page_bytes + (size_t)off * 2);
      const int tk = tokw + 32 * nt + 8 * (q0 + h);  // first of 8 tokens
      if (wave_full || tk + 7 < L) {
        __builtin_nontemporal_store(v, (u32x4*)dst);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (tk + i < L) ((uint16_t*)dst)[i] = (uint16_t)(v[i >> 1] >> (16 * (i & 1)));
      }
    }
  };
  auto store_prev = [&](int par, int kind, int mtp, int jj, int nt, int e, int qp) {
    if (jj < 0 || !wave_ok) return;
    emit_prev(pack_prev(par, nt, e, qp), kind, mtp, jj, nt, e, qp);
  };

  stage_in(0, std::integral_constant<int, 0>{}, smem);
  wait_all_memory();
  __syncthreads();
  for (int jj = 0; jj < jj_count; ++jj) {
    static_for<NSUB>([&](auto SUB) __attribute__((always_inline)) {  // compile time: fixes the kind (MFMA operand order) and the result set
      constexpr int sub = decltype(SUB)::value;
      const int stage = jj * NSUB + sub;
      const int odd = stage & 1;                       // LDS buffer of this stage
      const char* buf = smem + odd * STAGE_BYTES + (DIRECT ? 0 : lane * 16);
      auto weight = [&](int ks, int e) __attribute__((always_inline)) -> bf16x8 {
        if constexpr (DIRECT) return tr_natural_frag<RKV>(buf, tr, ks, e);
        else return *(const bf16x8*)(buf + (2 * ks + e) * 1024);
      };
      // the stage after this one (behind the last: the last group's first, into the buffer nobody reads any more: no branch)
      const bool last_group = jj + 1 == jj_count;
      using Next = std::integral_constant<int, (sub + 1) % NSUB>;
      const int next = sub + 1 < NSUB ? stage + 1 : (last_group ? jj * NSUB : stage + 1);
      f32x16 (&acc)[2][2] = accs[sub & 1];
      // the stage before this one, whose results leave in this stage's shadow (none at the start of a group when the
      // group's last stage has stored its own)
      constexpr int kPrevNone = -1;
      constexpr int psub = sub > 0 ? sub - 1 : (ODD ? kPrevNone : NSUB - 1);
      constexpr int pkind = psub >= NSK, pmtp = pkind ? psub - NSK : psub, ppar = psub & 1;
      const int pjj = psub == kPrevNone ? -1 : (sub == 0 ? jj - 1 : jj);
      if (wave_ok) {
        bf16x8 w[DEPTH + 1][2];
#pragma unroll
        for (int ks = 0; ks < DEPTH; ++ks) {
          w[ks][0] = weight(ks, 0);
          w[ks][1] = weight(ks, 1);
        }
        // A wave issues in order and is alone on its SIMD: whatever stands between two matrix instructions delays the
        // second one unless it fits into the 32 cycles the first one occupies the pipe.  The other work of a k-step is
        // therefore dealt out one small piece per gap: the two fragment reads for two k-steps ahead, the k-step's share
        // of the next stage's staging, and half of a store of the previous stage's results (pack in the odd k-steps,
        // address and store in the even ones that follow).
        u32x4 packed_piece = {0u, 0u, 0u, 0u};
        auto mm = [&](int ks, int nt, int e) __attribute__((always_inline)) {
          const bf16x8 wf = w[ks % (DEPTH + 1)][e];
          if (sub < NSK) {
            if (ks == 0) mfma_va_first(acc[nt][e], wf, xf[nt][ks]);
            else mfma_va(acc[nt][e], wf, xf[nt][ks]);
          } else {
            if (ks == 0) mfma_av_first(acc[nt][e], xf[nt][ks], wf);
            else mfma_av(acc[nt][e], xf[nt][ks], wf);
          }
          __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          __builtin_amdgcn_sched_barrier(0);
          mm(ks, 0, 0);
          if (ks + DEPTH < KS) w[(ks + DEPTH) % (DEPTH + 1)][0] = weight(ks + DEPTH, 0);
          __builtin_amdgcn_sched_barrier(0);
          mm(ks, 0, 1);
          if (ks + DEPTH < KS) w[(ks + DEPTH) % (DEPTH + 1)][1] = weight(ks + DEPTH, 1);
          __builtin_amdgcn_sched_barrier(0);
          mm(ks, 1, 0);
          if (ks < 16) stage_in_step(next, Next{}, smem + (odd ^ 1) * STAGE_BYTES, ks);
          __builtin_amdgcn_sched_barrier(0);
          mm(ks, 1, 1);
          // the previous stage's results leave in the shadow of this stage's MFMAs
          if constexpr (FP8) {
            if ((ks & 3) == 3 && ks <= 15)  // four pieces (nt, e)
              store_prev8(ppar, pkind, pmtp, pjj, (ks >> 2) >> 1, (ks >> 2) & 1);
          } else if (psub != kPrevNone && ks >= 1 && ks <= 16) {
            const int piece = (ks - 1) >> 1;  // packed at k-step 2 piece + 1, stored at 2 piece + 2
            if (ks & 1) {
              packed_piece = pack_prev(ppar, piece >> 2, (piece >> 1) & 1, piece & 1);  // (before the first stage: zeros, never stored)
            } else {
              emit_prev(packed_piece, pkind, pmtp, pjj, piece >> 2, (piece >> 1) & 1, piece & 1);
            }
          }
        }
        mfma_results_ready(acc[0][0], acc[0][1], acc[1][0], acc[1][1]);
        if constexpr (ODD && !FP8) {
          if (sub == NSUB - 1) {
#pragma unroll
            for (int piece = 0; piece < 8; ++piece) store_prev(sub & 1, 1, sub - NSK, jj, piece >> 2, (piece >> 1) & 1, piece & 1);
          }
        }
      } else {
        stage_in(next, Next{}, smem + (odd ^ 1) * STAGE_BYTES);  // a wave without tokens still stages its share
      }
      wait_all_memory();
      __syncthreads();  // next stage has landed; everyone is done with this stage's buffer
    });
  }
  // k_R plane: a straight copy, 8 dims (16 bytes) per lane and vector, fetched behind the last stage's results: there its
  // latency is covered by their stores, and the start of the block has one wait for all of its loads
  u32x4 kr[2][DR / 16];
  auto rope_row = [&](int nt) { return in_page + (int64_t)(slot0 + (wave_ok && tokw + 32 * nt + n < L ? 32 * nt + n : 0)) * W + RKV + h * 8; };
  if (jj_begin == 0) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int i = 0; i < DR / 16; ++i) kr[nt][i] = *(const u32x4*)(rope_row(nt) + 16 * i);
  }
  if constexpr (FP8) {
#pragma unroll
    for (int piece = 0; piece < 4; ++piece) store_prev8((NSUB - 1) & 1, 1, NSUB - 1 - NSK, jj_count - 1, piece >> 1, piece & 1);
  } else if constexpr (!ODD) {
#pragma unroll
    for (int piece = 0; piece < 8; ++piece) store_prev((NSUB - 1) & 1, 1, NSUB - 1 - NSK, jj_count - 1, piece >> 2, (piece >> 1) & 1, piece & 1);
  }
  if (jj_begin == 0) {
    char* const rp = page_bytes + (int64_t)gc * (DH + DV) * P * EB + ((int64_t)h * P + slot0 + n) * 16;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
      if (wave_ok && tokw + 32 * nt + n < L) {
#pragma unroll
        for (int i = 0; i < DR / 16; ++i) __builtin_nontemporal_store(kr[nt][i], (u32x4*)(rp + ((int64_t)2 * i * P + 32 * nt) * 16));
      }
  }
}

// Workgroup -> (256-token block, share of the groups).  A compute unit holds one workgroup: blocks run in rounds of 256.
// Blocks of whole rounds keep all groups; if the last round has at most 128, its blocks share their groups out over `parts`
// workgroups, as far as one round takes it (each reads the latent rows again).  With more blocks in it than 128, but at least two
// groups' time to win, its (block, group) pairs are dealt out evenly in order, and a workgroup may go from one block into the
// next (8 groups, 146 ragged blocks into the 8-bit cache 102.1 -> 83.4 us, 144 blocks 88.7 -> 81.0, 400 216 -> 198, 184 the same to
// 1.5 %; one block a workgroup leaves the other units idle).
// The lengths live on the device and the host knows only what a page-table row could hold, so the grid is bounded and a
// workgroup takes block blockIdx.x, then the one a grid further, and so on.
template <int DH, int DV, int RKV, int DR, bool FP8, bool DIRECT>
__global__ void __launch_bounds__(256) expand_bf16_kernel(ExpandArgs a, const __bf16* packed) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int gc = a.group_count;
  BlockScan<256> blocks;
  const int total = blocks.count(a.seq_lens, a.B, a.max_tokens);
  const int whole = total & ~255, rest = total & 255;
  const int parts = rest > 0 && rest <= 128 && gc > 1 ? expand_parts(rest, gc) : 1;
  const bool even = rest > 128 && rest * gc <= 256 * (gc - 2);
  for (int wg = blockIdx.x; wg < whole + (even ? 256 : rest * parts); wg += gridDim.x) {
    int id = wg, jj = 0, left = gc;  // `left` groups from group jj of block id on, over the end of the block into the next
    if (wg >= whole && even) {
      const int u0 = (wg - whole) * (rest * gc) / 256, u1 = (wg - whole + 1) * (rest * gc) / 256;
      id = whole + u0 / gc;
      jj = u0 % gc;
      left = u1 - u0;
    } else if (wg >= whole && parts > 1) {
      const int part = (wg - whole) % parts;
      id = whole + (wg - whole) / parts;
      jj = gc * part / parts;
      left = gc * (part + 1) / parts - jj;
    }
    for (; left > 0; ++id) {
      int b, blk, L;
      if (!blocks.find(id, b, blk, L)) return;  // whole workgroup
      const int n = min(gc - jj, left);
      // (the last stage's barrier has freed both LDS buffers for the next block)
      expand_block<DH, DV, RKV, DR, FP8, DIRECT>(a, packed, smem, b, blk, L, jj, n);
      left -= n;
      jj = 0;
    }
  }
}

// ---- cache expansion of the last a.tail positions of every sequence (the step's new tokens) ------------------------
// The B * tail tokens form one list (index = b * tail + t) cut into 32-token tiles; a wave takes half of a packed weight
// stage (32 output columns of one group's W_UK or W_UV, see pack_weights_bf16_kernel) times a tile.  A workgroup is one wave
// or the two halves of a stage on one tile (see the launcher):
//   K^T[d][tok] = W_UK^T[d][r] * C^T[r][tok]   and   V^T[d][tok] = W_UV^T[d][r] * C^T[r][tok]
//   A = packed weight fragment straight from global memory (1 KB, contiguous), B = the tokens' latent rows, gathered
//   (lane = token, 8 consecutive latent dims per k-step).
// Tokens of a tile belong to different sequences and pages, so results go out as 8-byte (K plane: 4 consecutive dims
// of one token) and 2-byte (V plane: one token's element of an 8-token vector) stores; with a few hundred tokens per
// step that is a few hundred KB.  The first stage's workgroups also copy the tokens' k_R.
// FP8 = true: `expanded` is an 8-bit cache (E4M3 code planes, see the header); every result is first rounded to bf16,
// the value the 16-bit cache would hold, and then quantised, so that the codes equal those of expanding into a 16-bit
// cache and converting it.
// DIRECT (WAVES = 1): the weights come as the caller holds them, without a launch that repacks them: the wave's 32 columns of all
// RKV rows go to LDS by LDS-DMA (64 bytes a row, back to back: 16 lanes of a transposed read meet every bank once) and are
// read as the same fragments, transposed.
template <int DH, int DV, int RKV, int DR, bool FP8, int WAVES, bool DIRECT>
__global__ void __launch_bounds__(64 * WAVES) expand_tail_bf16_kernel(ExpandArgs a, const __bf16* packed) {
  constexpr int W = RKV + DR;
  constexpr int KS = RKV / 16;
  constexpr int NSK = DH / 64, NSUB = (DH + DV) / 64;
  static_assert(!FP8 || (DH == 128 && DV == 128), "the 8-bit page format is written for equal dims of 128");
  static_assert(WAVES == 1 || (WAVES == 2 && !DIRECT), "one half of a stage, or both halves");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int stage = WAVES == 1 ? blockIdx.x >> 1 : blockIdx.x;  // jj * NSUB + sub
  const int jj = stage / NSUB, sub = stage % NSUB;
  const int kind = sub >= NSK, mtp = kind ? sub - NSK : sub;
  const int e = WAVES == 1 ? blockIdx.x & 1 : wave & 1;
  __shared__ __attribute__((aligned(16))) char w_lds[DIRECT ? RKV * 64 : 16];
  if constexpr (DIRECT) {  // (ahead of the chain length -> page -> latent row)
    const int dim = kind ? DV : DH;
    const char* w = (const char*)(kind ? a.w_uv : a.w_uk) + ((int64_t)(a.group_begin + jj) * RKV * dim + 64 * mtp + 32 * e) * 2;
    const uint32_t off = (lane >> 2) * (dim * 2) + (lane & 3) * 16;  // 16 rows an instruction
    const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)w_lds);
#pragma unroll
    for (int u = 0; u < RKV / 16; ++u)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(dst + u * 1024), "v"(off), "s"(w + (int64_t)(16 * u) * (dim * 2)) : "memory");
  }
  const int idx = blockIdx.y * 32 + n;  // this lane's token in the list
  const int P = a.latent.page_size;
  const int gc = a.group_count;
  bool ok = idx < a.B * a.tail;
  int b = 0, pos = 0;
  if (ok) {
    b = idx / a.tail;
    pos = a.seq_lens[b] - a.tail + idx % a.tail;
    ok = pos >= 0;
  }
  int32_t pg_in = -1, pg_out = -1;
  if (ok) {
    pg_in = page_of(a.latent, b, pos / P);
    pg_out = page_of(a.expanded, b, pos / P);
    ok = pg_in >= 0 && pg_out >= 0;
  }
  const int slot = ok ? pos % P : 0;
  // a lane without a token reads row 0 of page 0 (valid memory); its MFMA column is never stored
  const __bf16* row = (const __bf16*)a.latent.pool + ((int64_t)(ok ? pg_in : 0) * P + slot) * W;
  const __bf16* wf = packed + (int64_t)stage * KS * 2 * 512 + e * 512 + lane * 8;
  // Every load of the contraction is in flight before the first MFMA (the call is a chain of short kernels: what it costs
  // is memory latency, paid once this way): the latent fragments go straight into accumulation registers, as in the
  // one-shot kernel, which leaves the ordinary registers to the 32 weight fragments.  One accumulation chain in k order,
  // the one-shot kernel's order: the two produce the same bits.
  bf16x8 xf[KS], wv[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("global_load_dwordx4 %0, %1, off" : "=a"(xf[ks]) : "v"(row + ks * 16 + h * 8));
  if constexpr (!DIRECT) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) wv[ks] = *(const bf16x8*)(wf + (int64_t)ks * 1024);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if constexpr (DIRECT) {
    const int i16 = lane & 15;  // addresses row 8 h + i16 / 4 (+ 4) of the k-step, columns 16 ((lane / 16) % 2) + 4 (i16 % 4) ..
    const char* base = w_lds + (8 * h + (i16 >> 2)) * 64 + ((lane >> 4) & 1) * 32 + (i16 & 3) * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const i16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(base + ks * 1024));
      const i16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(base + ks * 1024 + 256));
      const i16x8 r = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
      wv[ks] = __builtin_bit_cast(bf16x8, r);
    }
  }
  f32x16 acc;
  mfma_va_first(acc, wv[0], xf[0]);
#pragma unroll
  for (int ks = 1; ks < KS; ++ks) mfma_va(acc, wv[ks], xf[ks]);
  asm volatile("s_nop 15\n\ts_nop 7" : "+v"(acc));  // the last MFMA's passes, before anything else reads the results
  if (!ok) return;
  const int d0 = 64 * mtp + 32 * e;  // register i holds dim d0 + 8*(i/4) + 4*h + i%4 of this lane's token
  if constexpr (FP8) {
    char* out8 = (char*)a.expanded.pool + (int64_t)pg_out * P * (2 * gc * DH + 2 * DR);
    const float inv = kind == 0 ? a.k_inv_scale : a.v_inv_scale;
    uint32_t code[4];  // code[q] = dims d0 + 8q + 4h + 0..3
#pragma unroll
    for (int q = 0; q < 4; ++q)
      code[q] = quantize_e4m3x4(round_to_bf16(acc[4 * q]), round_to_bf16(acc[4 * q + 1]), round_to_bf16(acc[4 * q + 2]),
                                round_to_bf16(acc[4 * q + 3]), inv);
    if (kind == 0) {  // dim 32 kp + 16 u + 8 h' + i: here kp = d0/32, u = q/2, h' = q%2, i = 4h + 0..3 -> four consecutive bytes
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(uint32_t*)(out8 + ((int64_t)(jj * (DH / 16) + 2 * (d0 / 32) + (q & 1)) * P + slot) * 16 + 8 * (q >> 1) + 4 * h) = code[q];
    } else {          // slot 32 T + 16 u + 8 h' + i: one byte per dim
      char* vp = out8 + (int64_t)gc * P * DH + ((int64_t)(jj * (P / 32) + slot / 32) * DH * 2 + ((slot >> 3) & 1)) * 16 +
                 8 * ((slot >> 4) & 1) + (slot & 7);
#pragma unroll
      for (int i = 0; i < 16; ++i)
        vp[(int64_t)(d0 + 8 * (i >> 2) + 4 * h + (i & 3)) * 32] = (char)((code[i >> 2] >> (8 * (i & 3))) & 0xffu);
    }
    if (stage == 0 && e == 0) {
      char* rp = out8 + (int64_t)2 * gc * P * DH;
#pragma unroll
      for (int c = h; c < DR / 8; c += 2) *(u32x4*)(rp + ((int64_t)c * P + slot) * 16) = *(const u32x4*)(row + RKV + c * 8);
    }
    return;
  }
  __bf16* out_page = (__bf16*)a.expanded.pool + (int64_t)pg_out * P * (gc * (DH + DV) + DR);
  if (kind == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u32x2 v = {pack_bf16(acc[4 * q], acc[4 * q + 1]), pack_bf16(acc[4 * q + 2], acc[4 * q + 3])};
      *(u32x2*)(out_page + ((int64_t)(jj * (DH / 8) + d0 / 8 + q) * P + slot) * 8 + 4 * h) = v;
    }
  } else {
    __bf16* vp = out_page + (int64_t)gc * P * DH + ((int64_t)(jj * (P / 8) + slot / 8) * DV) * 8 + slot % 8;
#pragma unroll
    for (int i = 0; i < 16; ++i) vp[(int64_t)(d0 + 8 * (i >> 2) + 4 * h + (i & 3)) * 8] = (__bf16)acc[i];
  }
  if (stage == 0 && e == 0) {  // k_R of this token: dims 8*c .. 8*c + 7 for c = h, h + 2, ...
    __bf16* rp = out_page + (int64_t)gc * P * (DH + DV);
#pragma unroll
    for (int c = h; c < DR / 8; c += 2) *(u32x4*)(rp + ((int64_t)c * P + slot) * 8) = *(const u32x4*)(row + RKV + c * 8);
  }
}

// ---- cache compression: latent from the expanded keys (Sec. 3.1: the reverse cache switch) --------------------------
// c_s = A^+ k^C_s with the caller's left inverse A^+ ([r_kv][g*d_h], k^C ordered group-major, dim-minor); k_R copied.
// One workgroup of 4 waves per 128 tokens of a sequence computes all r_kv latent dims of its tokens; wave w owns latent dims
// [128 w, 128 w + 128) of all 128 tokens (16 accumulator tiles: half of the SIMD's register file, the wave is alone on it):
//   C^T[r][tok] = A^+[r][k] * K^T[k][tok]
// Stages of 64 k (whole 128-byte lines of A^+).  A wave holds the stage's 16 key fragments in registers and takes its rows of
// A^+ in four units of 32: a unit is four fragments and 16 MFMAs, so that a fragment read from LDS serves four MFMAs.
// Both operands travel by LDS-DMA:
//   A^+   a private ring of seven 4 KB units per wave (it reads what it requested itself: no barrier), up to seven units, or
//         3.6 k cycles of MFMAs, ahead; rows of 128 bytes, 16-byte chunks XORed with (row >> 1) & 7: conflict-free reads
//   keys  a ring of three stages shared by the waves, [8 vector planes][128 tokens][16 bytes]: the cache page's own order,
//         1 KB of consecutive memory per request; one barrier per stage
// A unit's slot takes the request for the unit seven ahead as soon as its fragments are in registers, one unit before its
// MFMAs end; the next stage's key fragments replace the current ones one by one behind the MFMAs that use them last.
// What bounds it is the L2 that serves A^+ (every workgroup reads all of it, 1 MB at g d_h = 1024): 64-byte pieces of lines
// (stages of 32 k) cost as many L2 requests as whole ones, and workgroups of a die that walk k in step ask one of its 16
// channels for all their rows (they lie a multiple of 2 KB apart), so each starts at a different stage and wraps.
// The results leave through LDS as whole rows (c_kv | k_R, 64 of them contiguous in the latent page).
// Measured, 122 680 tokens in 32 ragged sequences, g d_h = 1024 (129 GFLOP, 409 MB): 246 us with registers -> LDS staging two
// stages of 32 k ahead; 183 us with LDS-DMA and a ring of four such stages; 171 us with rotated starts; 138 us in this form
// (whole lines, private rings, dense numbering of the tiles): 0.93 PFLOP/s, 3.0 TB/s.  The MFMA pipes are busy 46 % of the time;
// the rest is waiting for A^+ and keys (20 % of the wave cycles), the start and end of a tile, and a clock below the nominal.
constexpr int kCompressK = 64;                        // contraction elements per stage
constexpr int kCompressTok = 128;                     // tokens per workgroup
constexpr int kCompressUnits = 7;                     // ring of A^+ units per wave
constexpr int kCompressKeySlots = 3;                  // ring of key stages
constexpr int kCompressUnit = 32 * kCompressK * 2;    // bytes of a unit: 32 rows x 128 bytes
constexpr int kCompressKeys = kCompressTok * kCompressK * 2;
constexpr int kCompressLds = 4 * kCompressUnits * kCompressUnit + kCompressKeySlots * kCompressKeys;  // all 160 KB

// The two 64-token halves of a tile: page and slot (P is a multiple of 64, so a half lies in one page).  A half
// without tokens or behind a page id outside the pool reads page 0 instead: a token is one MFMA column, and the
// columns of such a half are never stored.
// The four table entries (two halves, two caches) come with one load, a lane each.
struct CompressHalves {
  const char* src[2];
  int32_t pg_out[2];
};
template <int DH, int DV, int DR>
__device__ __forceinline__ CompressHalves compress_halves(const CompressArgs& a, int b, int tok0, int L) {
  const int lane = threadIdx.x & 63, P = a.expanded.page_size;
  const int64_t in_page_bytes = (int64_t)P * (a.g * (DH + DV) + DR) * 2;
  const int my_tok = tok0 + 64 * (lane & 1);
  // (selected field by field: through a reference to either view a lane would load the fields from memory first)
  const bool out = lane & 2;
  const int p = my_tok / P, max_pages = out ? a.latent.max_pages : a.expanded.max_pages, num_pages = out ? a.latent.num_pages : a.expanded.num_pages;
  const int32_t* const table = out ? a.latent.page_table : a.expanded.page_table;
  int32_t pg = -1;
  if (my_tok < L && p < max_pages) pg = table ? table[(int64_t)b * max_pages + p] : b * max_pages + p;
  if ((uint32_t)pg >= (uint32_t)num_pages) pg = -1;
  CompressHalves r;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int tk = tok0 + 64 * e;
    const int32_t pin = __builtin_amdgcn_readlane(pg, e);
    r.pg_out[e] = pin >= 0 ? __builtin_amdgcn_readlane(pg, 2 + e) : -1;
    r.src[e] = (const char*)a.expanded.pool + (pin >= 0 ? pin : 0) * in_page_bytes + (pin >= 0 ? tk % P : 0) * 16;
  }
  return r;
}

// Tile `id` of the numbering: 128-token tile `blk` of sequence b, which has L tokens.
template <int DH, int DV, int RKV, int DR>
__device__ __forceinline__ void compress_tile(const CompressArgs& a, char* smem, int id, int b, int blk, int L) {
  static_assert(RKV == 512 && DH % kCompressK == 0 && DH / kCompressK >= 2, "four waves x 128 latent dims, at least two stages");
  constexpr int W = RKV + DR;
  constexpr int PITCH = W * 2 + 16;                   // bytes per token of the output tile in LDS
  static_assert(kCompressTok * PITCH <= kCompressLds, "the output tile reuses the rings");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int P = a.expanded.page_size;
  const int tok0 = blk * kCompressTok;
  const int K = a.g * DH;

  const CompressHalves hv = compress_halves<DH, DV, DR>(a, b, tok0, L);
  const char* const* half_src = hv.src;
  // k_R of the tile, kept for the end: vector plane (tid >> 7) + 2 i of token tid % 128
  u32x4 kr[DR / 16];
  {
    const int tk = tid & (kCompressTok - 1);
    const char* src = (tk & 64 ? half_src[1] : half_src[0]) + (int64_t)a.g * P * (DH + DV) * 2 + (tk & 63) * 16;
#pragma unroll
    for (int i = 0; i < DR / 16; ++i) kr[i] = *(const u32x4*)(src + (int64_t)((tid >> 7) + 2 * i) * P * 16);
  }

  // requests.  A^+ unit (u = 4 stage + rt): four of 8 rows; this lane's row and chunk (the swizzle term of rows 8 i .. 8 i + 7
  // alternates with i).  Key stage: planes 2 wave, 2 wave + 1 of both token halves.
  const uint32_t a_off0 = (uint32_t)((lane >> 3) * K * 2 + (((lane & 7) ^ (lane >> 4)) << 4));
  const uint32_t a_off1 = (uint32_t)((lane >> 3) * K * 2 + (((lane & 7) ^ (4 + (lane >> 4))) << 4));
  const uint32_t k_off = lane * 16;
  const int stages = K / kCompressK;
  const int rot = (id >> 3) % stages;                 // workgroups go to the eight dies in turn: id / 8 counts a die's own
  const char* const a_rows = (const char*)a.w_inv + (int64_t)(128 * wave) * K * 2;
  const int64_t rows8 = (int64_t)8 * K * 2;           // bytes from one request's rows to the next one's
  const int64_t plane = (int64_t)P * 16;              // bytes of one vector plane of the page
  char* const a_ring = smem + wave * (kCompressUnits * kCompressUnit);
  char* const k_ring = smem + 4 * kCompressUnits * kCompressUnit;
  const uint32_t a_lds = (uint32_t)(uintptr_t)(lds_ptr_t)a_ring;
  const uint32_t k_lds = (uint32_t)(uintptr_t)(lds_ptr_t)k_ring + (2 * wave) * (kCompressTok * 16);
  int a_stage = rot, k_stage = rot;                   // stage (in the rotated walk) of the next A^+ unit / key request
  int a_fill = 0, k_fill = 0;                         // ring slots they go to
  auto dma = [&](uint32_t dst, uint32_t off, const char* src) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(__builtin_amdgcn_readfirstlane(dst)), "v"(off), "s"(src) : "memory");
  };
  auto request_a = [&](int rt, int i) __attribute__((always_inline)) {   // request i = 0..3 of the next unit, rows 32 rt ..
    dma(a_lds + a_fill * kCompressUnit + i * 1024, i & 1 ? a_off1 : a_off0, a_rows + (4 * rt + i) * rows8 + a_stage * (kCompressK * 2));
    if (i == 3) {
      a_fill = a_fill + 1 == kCompressUnits ? 0 : a_fill + 1;
      if (rt == 3) a_stage = a_stage + 1 == stages ? 0 : a_stage + 1;
    }
  };
  auto request_k = [&](int i) __attribute__((always_inline)) {           // i = 0..3: plane 2 wave + i / 2, half i % 2
    dma(k_lds + k_fill * kCompressKeys + (i >> 1) * (kCompressTok * 16) + (i & 1) * 1024, k_off,
        half_src[i & 1] + (int64_t)(8 * k_stage + 2 * wave + (i >> 1)) * plane);
    if (i == 3) {
      k_fill = k_fill + 1 == kCompressKeySlots ? 0 : k_fill + 1;
      k_stage = k_stage + 1 == stages ? 0 : k_stage + 1;
    }
  };

  f32x16 acc[4][4];                                   // [latent tile][token tile]
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rt][tt][i] = 0.f;

  bf16x8 af[2][4], kf[4][4];                          // A^+ fragments [unit parity][k-step], key fragments [k-step][token tile]
  uint32_t a_read[4], k_read = h * (kCompressTok * 16) + n * 16;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) a_read[ks] = n * 128 + (((2 * ks + h) ^ ((n >> 1) & 7)) << 4);
  int a_slot = 0, k_slot = 0;                         // ring slots of the next unit / key stage to be read
  auto load_a = [&](int par, int ks) __attribute__((always_inline)) { af[par][ks] = *(const bf16x8*)(a_ring + a_slot * kCompressUnit + a_read[ks]); };
  auto load_k = [&](int ks, int tt) __attribute__((always_inline)) {
    kf[ks][tt] = *(const bf16x8*)(k_ring + k_slot * kCompressKeys + k_read + 2 * ks * (kCompressTok * 16) + 32 * tt * 16);
  };

  // Order of the requests: key stage s + 3 goes out right before A^+ unit 4 s + 10.  Requests complete in order, so a
  // unit that has landed vouches for the key stage requested before it.
  auto request_unit = [&](int rt) __attribute__((always_inline)) {
    static_for<4>([&](auto I) __attribute__((always_inline)) { request_a(rt, decltype(I)::value); });
  };
  auto request_keys = [&]() __attribute__((always_inline)) {
    static_for<4>([&](auto I) __attribute__((always_inline)) { request_k(decltype(I)::value); });
  };
  request_keys();
  request_unit(0);
  request_unit(1);
  request_keys();
  request_unit(2);
  request_unit(3);
  request_unit(0);
  request_unit(1);
  if (stages > 2) request_keys();
  request_unit(2);
  asm volatile("s_waitcnt vmcnt(28)" ::: "memory");   // at most units 1 .. 6 and the second key stage outstanding
  __syncthreads();                                    // key stage 0 has landed for every wave
  static_for<4>([&](auto KS) __attribute__((always_inline)) {
    load_a(0, decltype(KS)::value);
    static_for<4>([&](auto TT) __attribute__((always_inline)) { load_k(decltype(KS)::value, decltype(TT)::value); });
  });
  a_slot = 1;
  k_slot = 1;

  // One unit: its 16 MFMAs, and behind them the fragments of the next unit, the request for the unit seven ahead and, in
  // the stage's last unit, the next stage's key fragments.  KIND: 0 steady, 3 the third last
  // (no key stage left to request), 1 the stage before the last, 2 the last (nothing left to request): compile-time, so
  // that nothing branches between the MFMAs.
  auto stage_step = [&](auto KIND_T) __attribute__((always_inline)) {
    constexpr int KIND = decltype(KIND_T)::value;
    static_for<4>([&](auto RT_T) __attribute__((always_inline)) {
      constexpr int rt = decltype(RT_T)::value;
      constexpr bool next_unit = KIND != 2 || rt < 3;             // a unit follows
      constexpr bool req = KIND == 0 || KIND == 3 || (KIND == 1 && rt == 0);   // the unit seven ahead exists
      constexpr bool next_keys = KIND != 2 && rt == 3;
      // requests made after those of the next unit (see the order above): what may still be outstanding
      constexpr int behind = KIND == 0 || KIND == 3 ? (rt == 0 ? 28 : 24) : (KIND == 1 ? (rt == 0 ? 24 : (rt == 1 ? 20 : (rt == 2 ? 16 : 12)))
                                                                          : (rt == 0 ? 8 : (rt == 1 ? 4 : 0)));
      if constexpr (next_unit) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(behind) : "memory");
      if constexpr (next_keys) __syncthreads();       // the next key stage has landed for every wave; all hold this one in registers
      __builtin_amdgcn_sched_barrier(0);
      static_for<16>([&](auto X) __attribute__((always_inline)) {
        constexpr int x = decltype(X)::value, ks = x >> 2, tt = x & 3;
        acc[rt][tt] = mfma32(af[rt & 1][ks], kf[ks][tt], acc[rt][tt]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (next_unit && x < 4) load_a((rt + 1) & 1, x);
        if constexpr (next_keys) load_k(ks, tt);      // (the fragment's last use was the MFMA above)
        if constexpr (KIND == 0 && rt == 3 && x >= 4 && x < 8) request_k(x - 4);
        // (the unit's last fragments were operands of MFMA 12: its ring slot is free)
        if constexpr (req && x >= 12) request_a((rt + 3) & 3, x - 12);
        __builtin_amdgcn_sched_barrier(0);
      });
      a_slot = a_slot + 1 == kCompressUnits ? 0 : a_slot + 1;
      if constexpr (next_keys) k_slot = k_slot + 1 == kCompressKeySlots ? 0 : k_slot + 1;
    });
  };
  int st = 0;
#pragma unroll 1
  for (; st + 3 < stages; ++st) stage_step(std::integral_constant<int, 0>{});
#pragma unroll 1
  for (; st + 2 < stages; ++st) stage_step(std::integral_constant<int, 3>{});
  stage_step(std::integral_constant<int, 1>{});
  stage_step(std::integral_constant<int, 2>{});

  __syncthreads();                                    // (every fragment has been read: the last barrier was before that)
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const u32x2 v = {pack_bf16(acc[rt][tt][4 * q], acc[rt][tt][4 * q + 1]), pack_bf16(acc[rt][tt][4 * q + 2], acc[rt][tt][4 * q + 3])};
        *(u32x2*)(smem + (32 * tt + n) * PITCH + (128 * wave + 32 * rt + 8 * q + 4 * h) * 2) = v;
      }
#pragma unroll
  for (int i = 0; i < DR / 16; ++i)
    *(u32x4*)(smem + (tid & (kCompressTok - 1)) * PITCH + RKV * 2 + ((tid >> 7) + 2 * i) * 16) = kr[i];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    if (hv.pg_out[e] < 0) continue;
    const int tk = tok0 + 64 * e;
    constexpr int VPR = W / 8;                        // 16-byte vectors per row
    const int total = min(64, L - tk) * VPR;
    u32x4* dst = (u32x4*)((char*)a.latent.pool + ((int64_t)hv.pg_out[e] * P + tk % P) * (W * 2));
    for (int v = tid; v < total; v += 256) {
      const int r = v / VPR, c = v % VPR;
      __builtin_nontemporal_store(*(const u32x4*)(smem + (64 * e + r) * PITCH + c * 16), dst + v);
    }
  }
}

// A share of the latent dims of a tile (a quarter or a half: 128 RT dims from 128 RT part on), for calls with few tiles: a tile
// alone is 1024 MFMAs per wave and 1 MB of A^+ through one unit, 14 us, while most of the chip idles.  Wave w owns 32 RT latent
// dims of all 128 tokens.  Stages of 64 k hold 128 RT rows of A^+ (panel layout of gqla_lds.h) and the keys of the tile (as
// above), 16 RT and 16 KB, in a ring of five or three; one barrier per stage: stage p is awaited (counted: requests complete in
// order), and the buffer that stage p - 1 has just left takes the requests of stage p + NS - 1.  What bounds it is the unit's
// memory path (64 bytes a clock) and the start and end of a tile.  Whole tiles -> shares, g d_h = 1024: one sequence of 2400
// tokens 24.1 -> 15.0 us, 76 tiles of four 24.8 -> 22.2.
constexpr int kCompressQuarterTiles = 64, kCompressHalfTiles = 96;   // at most: see the kernel below
template <int DH, int DV, int RKV, int DR, int RT>
__device__ __forceinline__ void compress_part(const CompressArgs& a, char* smem, int id, int b, int blk, int L, int part) {
  constexpr int W = RKV + DR, DIMS = 128 * RT, NS = RT == 1 ? 5 : 3;
  constexpr int ABYTES = DIMS * kCompressK * 2, STAGE = ABYTES + kCompressKeys;
  constexpr int PITCH = DIMS * 2 + 16;                 // bytes per token of the output tile in LDS
  static_assert(NS * STAGE <= kCompressLds && kCompressTok * PITCH <= kCompressLds, "the rings, and the output tile over them");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int P = a.expanded.page_size;
  const int tok0 = blk * kCompressTok;
  const int K = a.g * DH;
  const CompressHalves hv = compress_halves<DH, DV, DR>(a, b, tok0, L);
  const int64_t plane = (int64_t)P * 16;              // bytes of one vector plane of the page
  // k_R of the tile (first share only), kept for the end: vector plane (tid >> 7) + 2 i of token tid % 128
  u32x4 kr[DR / 16];
  if (part == 0) {
    const int tk = tid & (kCompressTok - 1);
    const char* src = (tk & 64 ? hv.src[1] : hv.src[0]) + (int64_t)a.g * P * (DH + DV) * 2 + (tk & 63) * 16;
#pragma unroll
    for (int i = 0; i < DR / 16; ++i) kr[i] = *(const u32x4*)(src + (int64_t)((tid >> 7) + 2 * i) * P * 16);
  }
  const int stages = K / kCompressK;
  int at = (id >> 3) % stages;                        // rotated walk, as above
  int fill = 0;
  const uint32_t a_off = (uint32_t)((lane >> 3) * K * 2 + (((lane & 7) ^ lds_swz(8 * wave + (lane >> 3))) << 4));  // rows 8 (wave + 4 j) ..
  const char* const a_rows = (const char*)a.w_inv + (int64_t)(DIMS * part) * K * 2;
  auto request = [&]() __attribute__((always_inline)) {  // this wave's share of the next stage
    char* const buf = smem + fill * STAGE;
    fill = fill + 1 == NS ? 0 : fill + 1;
    auto dma = [&](char* dst, uint32_t off, const char* src) __attribute__((always_inline)) {
      const uint32_t d = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)dst);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(d), "v"(off), "s"(src) : "memory");
    };
#pragma unroll
    for (int j = 0; j < 4 * RT; ++j) dma(buf + (wave + 4 * j) * 1024, a_off, a_rows + (int64_t)(8 * (wave + 4 * j)) * K * 2 + at * (kCompressK * 2));
#pragma unroll
    for (int i = 0; i < 4; ++i)                       // planes 2 wave, 2 wave + 1 of both token halves
      dma(buf + ABYTES + (2 * wave + (i >> 1)) * (kCompressTok * 16) + (i & 1) * 1024, lane * 16, hv.src[i & 1] + (int64_t)(8 * at + 2 * wave + (i >> 1)) * plane);
    at = at + 1 == stages ? 0 : at + 1;
  };
  f32x16 acc[RT][4];                                  // [latent tile][token tile]
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[rt][tt][i] = 0.f;
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < stages) request();
  int slot = 0;
  for (int st = 0; st < stages; ++st) {
    const int behind = min(stages - 1 - st, NS - 2);  // stages requested behind this one
    static_for<NS - 1>([&](auto q) {
      if (behind == decltype(q)::value) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(decltype(q)::value * (4 * RT + 4)) : "memory");
    });
    __syncthreads();
    if (st + NS - 1 < stages) request();
    const char* const buf = smem + slot * STAGE;
    slot = slot + 1 == NS ? 0 : slot + 1;
    bf16x8 af[4][RT], kf[4][4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) af[ks][rt] = row_frag<DIMS>(buf, 32 * (RT * wave + rt) + n, 2 * ks + h);
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) kf[ks][tt] = *(const bf16x8*)(buf + ABYTES + (2 * ks + h) * (kCompressTok * 16) + (32 * tt + n) * 16);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) acc[rt][tt] = mfma32(af[ks][rt], kf[ks][tt], acc[rt][tt]);
  }
  __syncthreads();                                    // every wave has read the last stage
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(u32x2*)(smem + (32 * tt + n) * PITCH + (32 * (RT * wave + rt) + 8 * q + 4 * h) * 2) =
            u32x2{pack_bf16(acc[rt][tt][4 * q], acc[rt][tt][4 * q + 1]), pack_bf16(acc[rt][tt][4 * q + 2], acc[rt][tt][4 * q + 3])};
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    if (hv.pg_out[e] < 0) continue;
    const int tk = tok0 + 64 * e, rows = min(64, L - tk);
    char* const dst = (char*)a.latent.pool + ((int64_t)hv.pg_out[e] * P + tk % P) * (W * 2);
    constexpr int VPR = DIMS / 8;                     // 16-byte vectors of a row's share
    for (int v = tid; v < rows * VPR; v += 256)
      __builtin_nontemporal_store(*(const u32x4*)(smem + (64 * e + v / VPR) * PITCH + v % VPR * 16), (u32x4*)(dst + (int64_t)(v / VPR) * (W * 2) + part * (DIMS * 2) + v % VPR * 16));
    if (part == 0 && (tid & 64) == 64 * e && (tid & 63) < rows) {
#pragma unroll
      for (int i = 0; i < DR / 16; ++i) __builtin_nontemporal_store(kr[i], (u32x4*)(dst + (int64_t)(tid & 63) * (W * 2) + RKV * 2 + ((tid >> 7) + 2 * i) * 16));
    }
  }
}

// Grid as in the expansion: bounded, a workgroup takes tile blockIdx.x, then the one a grid further, and so on.  With few tiles
// (the lengths live on the device: counted here) a workgroup takes a quarter or half of a tile's latent dims, as long as all
// of them run at once (quarters in two rounds: 76 tiles 24.9 -> 29.4 us) and do not crowd the L2 that serves A^+ and the keys,
// which each share reads again (halves: 65 tiles 24.2 -> 21.5 us, 96 tiles 24.6 -> 22.9, but 126 tiles 25.7 -> 26.7; the same with
// g d_h = 768 to 4096: 96 tiles 7 to 13 % faster).
template <int DH, int DV, int RKV, int DR>
__global__ void __launch_bounds__(256) compress_bf16_kernel(CompressArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  BlockScan<kCompressTok> blocks;
  const int total = blocks.count(a.seq_lens, a.B, a.max_tokens);
  if (__builtin_expect(total > kCompressHalfTiles, 1)) {
    for (int id = blockIdx.x; id < total; id += gridDim.x) {
      int b, blk, L;
      if (!blocks.find(id, b, blk, L)) return;  // whole workgroup
      compress_tile<DH, DV, RKV, DR>(a, smem, id, b, blk, L);
      __syncthreads();  // the next tile's requests go where this one's rows leave from
    }
    return;
  }
  const int shares = total <= kCompressQuarterTiles ? 4 : 2, id = blockIdx.x;
  int b, blk, L;
  if (id >= shares * total || !blocks.find(id / shares, b, blk, L)) return;  // whole workgroup (the grid holds every share)
  if (shares == 4) compress_part<DH, DV, RKV, DR, 1>(a, smem, id, b, blk, L, id & 3);
  else compress_part<DH, DV, RKV, DR, 2>(a, smem, id, b, blk, L, id & 1);
}

// Workgroups of a launch over blocks of ragged sequences: eight rounds of 256.  Up to that number (half a million tokens of
// the expansion) the blocks are dealt out as workgroups come free; beyond it the workgroups loop.  A workgroup without a
// block only scans the lengths, but holds a compute unit's LDS meanwhile, 1.4 to 2.1 ns each over the chip.  Measured with rows of
// 2^20 tokens, one workgroup per block that the rows could hold -> this: expansion of 32 ragged sequences 448 -> 251 us, of
// 128 short ones 1358 -> 101 us; compression 442 -> 157 and 2076 -> 57 us (all as with rows of the sequences' own size).
constexpr int kMaxWorkgroups = 8 * 256;

}  // namespace

template <int DH, int DV>
static hipError_t launch_compress_dims(const CompressArgs& a, hipStream_t s) {
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)compress_bf16_kernel<DH, DV, 512, 64>, hipFuncAttributeMaxDynamicSharedMemorySize, kCompressLds);
  if (attr != hipSuccess) return attr;
  // as many workgroups as tiles that the rows of the page table could hold, and enough for the shares of a few
  const int64_t blocks = ((int64_t)a.max_tokens + kCompressTok - 1) / kCompressTok * a.B;
  const int64_t grid = std::max(std::min<int64_t>(blocks, kMaxWorkgroups), std::min<int64_t>(4 * blocks, 256));
  compress_bf16_kernel<DH, DV, 512, 64><<<(unsigned)grid, 256, kCompressLds, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_compress_bf16(const CompressArgs& a, hipStream_t s) {
  return a.d_h == 192 ? launch_compress_dims<192, 256>(a, s) : launch_compress_dims<128, 128>(a, s);
}

template <int SHARES>
static hipError_t launch_absorb_query_staged(const AbsorbQueryArgs& a, int rows_per_group, int grid_x, hipStream_t s) {
  constexpr int kRows = 512 / SHARES, kLds = kRows * 128 * 2 + 4 * 32 * ((kRows >= 256 ? 128 : 64) + 16);  // the share of W_UK[j], output tiles
  static const hipError_t attr = hipFuncSetAttribute((const void*)absorb_query_staged_bf16_kernel<512, SHARES>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return attr;
  absorb_query_staged_bf16_kernel<512, SHARES><<<dim3(grid_x, SHARES, a.g), 256, kLds, s>>>(a, rows_per_group);
  return hipGetLastError();
}

hipError_t launch_absorb_query_bf16(const AbsorbQueryArgs& a, hipStream_t s) {
  const int rows_per_group = a.rows * a.G;
  dim3 grid((rows_per_group + 31) / 32, (512 / 128 + 3) / 4, a.g);
  if (a.d_h == 192) {
    absorb_query_bf16_kernel<192, 512><<<grid, 256, 0, s>>>(a, rows_per_group);
    return hipGetLastError();
  }
  // one workgroup per compute unit: the latent dims in 4 or 2 shares while that leaves units idle, several row blocks each
  // where there are more
  const int blocks = (int)grid.x * a.g;
  if (blocks * 4 <= 256) return launch_absorb_query_staged<4>(a, rows_per_group, grid.x, s);
  if (blocks * 2 <= 256) return launch_absorb_query_staged<2>(a, rows_per_group, grid.x, s);
  const int per_group = a.g < 256 ? 256 / a.g : 1;
  return launch_absorb_query_staged<1>(a, rows_per_group, (int)grid.x < per_group ? (int)grid.x : per_group, s);
}

template <int DH, int DV, bool FP8>
static hipError_t launch_expand_tail_dims(const ExpandArgs& a, void* ws, hipStream_t s) {
  constexpr int NSUB = (DH + DV) / 64;
  const int tokens = a.B * a.tail;
  const int stages = a.group_count * NSUB, tiles = (tokens + 31) / 32;
  // Weights that are not repacked yet and few tokens: taken as they are (4 tokens, 8 groups, 8-bit step 27.8 -> 23.0 us, 64 tokens
  // 201.3 -> 198.6: a launch of 5 us less, 2 us more for the transposed reads).  Each tile of 32 tokens reads all weights that way,
  // 64 KB a stage and slower than repacked ones once they are far beyond the L2s, so the more stages, the fewer tiles.  Call,
  // repacked over direct, 16-bit / 8-bit cache of (128, 128): 192 stages (48 groups), 8 tiles 1.25 / 1.09; 256 stages, 6 tiles 1.15 /
  // 1.02, 8 1.07 / 0.96; 320 stages, 3 tiles 1.07 / 1.01, 4 1.08 / 0.97, 5 0.94 / 0.89; 384 stages, 2 tiles 1.17 / 1.12, 3 1.02 / 0.92;
  // 448 stages, 2 tiles 1.04 / 0.98; 512 stages, 1 tile 1.47 / 1.43, 2 1.02 / 0.96, 8 0.75 / 0.69; of (192, 256): 224 stages (32
  // groups), 6 tiles 1.05, 8 0.98; 448 stages, 1 tile 1.53, 2 1.11, 4 0.85.
  const int most = stages <= 192 ? 8 : stages <= 256 ? 6 : stages <= 320 ? 3 : stages <= 384 ? 2 : 1;
  if (a.weights == 0 && tiles <= most) {
    expand_tail_bf16_kernel<DH, DV, 512, 64, FP8, 1, true><<<dim3(stages * 2, tiles), 64, 0, s>>>(a, nullptr);
    return hipGetLastError();
  }
  if (a.weights != 2) {
    pack_weights_bf16_kernel<DH, DV, 512><<<dim3(a.group_count * NSUB, 512 / 64), 256, 0, s>>>(a, (__bf16*)ws);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.weights == 1) return e;
  }
  // The call is latency and what one compute unit can fetch, 64 KB a wave, so the waves are spread over as many units as there
  // are: 128 tokens, 8 groups, 256 waves: 9.2 us as 64 workgroups of four waves, 5.1 us as 256 of one; one group 8.8 -> 4.9 us.
  // Workgroups go to the eight dies in turn: with at most four stages no die has two halves, every die reads all the latent
  // rows by itself, and from a few hundred waves on that costs more than the spread gives.  Two waves on the same rows then:
  // one group, 1024 waves 9.6 -> 8.8 us, 4096 waves 33.8 -> 29.5 us; 512 waves 5.9 us either way, 256 waves 4.9 against 5.5.
  // (8 groups, 8192 tokens: 104 us in pairs, 92 us as single waves; 4 groups the same to 3 %.)
  if (stages <= 4 && (int64_t)tiles * stages * 2 >= 512)
    expand_tail_bf16_kernel<DH, DV, 512, 64, FP8, 2, false><<<dim3(stages, tiles), 128, 0, s>>>(a, (const __bf16*)ws);
  else
    expand_tail_bf16_kernel<DH, DV, 512, 64, FP8, 1, false><<<dim3(stages * 2, tiles), 64, 0, s>>>(a, (const __bf16*)ws);
  return hipGetLastError();
}

hipError_t launch_expand_tail_bf16(const ExpandArgs& a, void* ws, hipStream_t s) {
  return a.d_h == 192 ? launch_expand_tail_dims<192, 256, false>(a, ws, s) : launch_expand_tail_dims<128, 128, false>(a, ws, s);
}

hipError_t launch_expand_tail_fp8(const ExpandArgs& a, void* ws, hipStream_t s) { return launch_expand_tail_dims<128, 128, true>(a, ws, s); }

template <int DH, int DV, bool FP8, bool DIRECT>
static hipError_t launch_expand_kernel(const ExpandArgs& a, const void* ws, unsigned grid, hipStream_t s) {
  constexpr int kLds = 2 * (512 / 16) * 2 * 1024;
  // once per process (function-local statics are initialised under a lock); an error is reported by every call
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)expand_bf16_kernel<DH, DV, 512, 64, FP8, DIRECT>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return attr;
  expand_bf16_kernel<DH, DV, 512, 64, FP8, DIRECT><<<grid, 256, kLds, s>>>(a, (const __bf16*)ws);
  return hipGetLastError();
}
template <int DH, int DV, bool FP8>
static hipError_t launch_expand_one_shot(const ExpandArgs& a, void* ws, hipStream_t s) {
  constexpr int NSUB = (DH + DV) / 64;
  // The lengths live on the device, so the kernel decides how the last round is shared out; whole rounds of 256, so that
  // those shares find workgroups as well.  Measured against a grid over (blocks of the longest sequence, sequences), whose holes
  // gave some dies a third round of blocks: one sequence of 8192 tokens, 8 groups 80 -> 31 us; 20 ragged sequences of 3000 to 6000
  // tokens into the 8-bit cache 216 -> 190 us; 122 680 ragged tokens in 32 sequences 286 -> 240 us.
  const int64_t blocks = ((int64_t)a.max_tokens + 255) / 256 * a.B;
  const unsigned grid = (unsigned)std::min<int64_t>((blocks + 255) & ~(int64_t)255, kMaxWorkgroups);
  // Few blocks (what the rows of the page table could hold) and few groups a workgroup: the weights as they are, without the launch
  // that repacks them.  The transposed reads cost a block 3 % (10 blocks, 8 groups 24.6 -> 21.8 us, 80 blocks the same either way,
  // 128 blocks 64.1 -> 66.0), and a wave whose 64 tokens are not all there about 1 us a group, which stores at half the speed for
  // want of scalar registers (sequences of 20 to 250 tokens: 20 blocks, 32 groups, 3 a workgroup 1.05 times as fast; 44 blocks, 7 a
  // workgroup 1.00; 60 blocks, 48 groups, 12 a workgroup 0.96; 72 blocks, 64 groups, 22 a workgroup 0.91).  With seven stages a group,
  // (192, 256), that outweighs the launch at once (200 tokens, 1 group 30.4 us repacked, 32.5 direct; 64 ragged sequences, 8 groups
  // 51.7 and 56.0; full waves 2 to 10 % faster): always repacked.
  if constexpr (NSUB % 2 == 0) {
    if (blocks <= 72) {
      const int parts = expand_parts((int)blocks, a.group_count);
      if ((a.group_count + parts - 1) / parts <= 6) return launch_expand_kernel<DH, DV, FP8, true>(a, nullptr, grid, s);
    }
  }
  pack_weights_bf16_kernel<DH, DV, 512><<<dim3(a.group_count * NSUB, 512 / 64), 256, 0, s>>>(a, (__bf16*)ws);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_expand_kernel<DH, DV, FP8, false>(a, ws, grid, s);
}
hipError_t launch_expand_bf16(const ExpandArgs& a, void* ws, hipStream_t s) {
  return a.d_h == 192 ? launch_expand_one_shot<192, 256, false>(a, ws, s) : launch_expand_one_shot<128, 128, false>(a, ws, s);
}
hipError_t launch_expand_fp8(const ExpandArgs& a, void* ws, hipStream_t s) { return launch_expand_one_shot<128, 128, true>(a, ws, s); }

}  // namespace gqla
