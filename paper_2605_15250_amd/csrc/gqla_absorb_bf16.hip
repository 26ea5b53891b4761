// MQA-absorb split-L decode over the 16-bit or 8-bit latent cache, bf16 MFMA (paper Sec. 3.1, MQA-absorb equation, lines 2-5).
//
// One workgroup of 4 waves per (chunk, block of 128 query rows); wave w owns rows 32w..32w+31 of the block.
// A 32-token latent tile [32][r_kv + d_r] is staged once into LDS (global_load_lds into a ring of four tile
// buffers, three tiles ahead of its use) and serves every row of the block twice: row-wise as the key operand
// [c | k_R] and transposed (ds_read_b64_tr_b16) as the value operand c:
//   S^T[token][row]  = Kt[token][576] * Qhat^T[576][row]      A = LDS row fragments,   B = queries in registers
//   O^T[r][row]     += C^T[r][token]  * P^T[token][row]       A = LDS transposed frags, B = probabilities
// O^T (512 x 32 fp32 per wave) lives in the 256 accumulation registers, addressed by name (see acc_* below); the
// softmax reference maximum is only moved (and O^T rescaled) when a row's maximum grows by more than 2^8, so that
// rescaling is rare.
// Each chunk's normalised latent-space output is written as bf16 with its log-sum-exp; the combine kernel merges
// chunks and applies W_UV.  Intensity h_q s_q (2 r_kv + d_r) / (r_kv + d_r) (Sec. 4.2.1): 242 FLOP/byte for 128 rows,
// 484 for 256 (s_q = 2), against a ridge of about 310 on this chip.
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "gqla_device.h"
#include "gqla_lds.h"

#ifdef GQLA_PHASE_TIMING
__device__ unsigned long long gqla_phase_cycles[16];
extern "C" int gqla_debug_read_phases(unsigned long long* host16, int reset) {
  if (hipMemcpyFromSymbol(host16, HIP_SYMBOL(gqla_phase_cycles), 16 * 8) != hipSuccess) return 1;
  if (reset) {
    unsigned long long z[16] = {};
    if (hipMemcpyToSymbol(HIP_SYMBOL(gqla_phase_cycles), z, 16 * 8) != hipSuccess) return 1;
  }
  return 0;
}
#if GQLA_PHASE_TIMING >= 2
#define GQLA_STAMP(k) do { const long long now_ = __builtin_readcyclecounter(); ph_[k] += now_ - last_; last_ = now_; } while (0)
#else
#define GQLA_STAMP(k) do { (void)ph_; (void)last_; } while (0)   // level 1: kernel entry and exit only
#endif
#else
#define GQLA_STAMP(k) do { } while (0)
#endif

namespace gqla {

namespace {

__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

constexpr int kTile = 32;                 // tokens per LDS tile
constexpr int kSlots = 4;                 // tile buffers in the LDS ring
constexpr int kRowsPerBlock = 128;        // query rows per workgroup
constexpr float kRescaleThreshold = 8.f;  // log2 units

// ---- O^T accumulators, managed by hand ----
// O^T (512 x 32 fp32 per wave) fills all 256 accumulation registers: tile dt (32 latent dims x 32 rows) is a[16*dt : 16*dt+15].
// They are addressed by NAME in inline assembly and never appear as C++ values: the compiler then has nothing to
// allocate, copy or spill there, and the rest of the kernel gets the 256 ordinary registers to itself.  Every statement
// below is `asm volatile`, so they keep their program order; the callers keep the hardware's timing rules
// (results of an MFMA are read by non-MFMA instructions only after its last pass has long retired).
#define GQLA_ACC(D) "a[" #D "*16:" #D "*16+15]"
#define GQLA_ACC_CLOBBER(D) GQLA_ACC_CLOBBER_##D
#define GQLA_ACC_CLOBBER_0 "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15"
#define GQLA_ACC_CLOBBER_1 "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31"
#define GQLA_ACC_CLOBBER_2 "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47"
#define GQLA_ACC_CLOBBER_3 "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63"
#define GQLA_ACC_CLOBBER_4 "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79"
#define GQLA_ACC_CLOBBER_5 "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95"
#define GQLA_ACC_CLOBBER_6 "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111"
#define GQLA_ACC_CLOBBER_7 "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127"
#define GQLA_ACC_CLOBBER_8 "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143"
#define GQLA_ACC_CLOBBER_9 "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159"
#define GQLA_ACC_CLOBBER_10 "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175"
#define GQLA_ACC_CLOBBER_11 "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191"
#define GQLA_ACC_CLOBBER_12 "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207"
#define GQLA_ACC_CLOBBER_13 "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223"
#define GQLA_ACC_CLOBBER_14 "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239"
#define GQLA_ACC_CLOBBER_15 "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"
#define GQLA_FOR_DT(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)

__device__ __forceinline__ void acc_zero() {
  asm volatile(".set gqla_i, 0\n.rept 256\n\tv_accvgpr_write_b32 a[gqla_i], 0\n.set gqla_i, gqla_i+1\n.endr" : : : GQLA_ALL_AGPRS);
}
// O^T tile dt += A * B (dt is a compile-time value at every call site: the switch folds away)
__device__ __forceinline__ void acc_mfma(int dt, bf16x8 a, bf16x8 b) {
  switch (dt) {
    // (the tile's registers are named as clobbered: the compiler must not keep values of its own in them across this
    // statement -- it would otherwise use "free" accumulation registers as parking space when ordinary ones run short)
#define X(D) case D: asm volatile("v_mfma_f32_32x32x16_bf16 " GQLA_ACC(D) ", %0, %1, " GQLA_ACC(D) : : "v"(a), "v"(b) : GQLA_ACC_CLOBBER(D)); break;
    GQLA_FOR_DT(X)
#undef X
  }
}
// every accumulator of this lane times alpha (one query row per lane, so alpha is per lane)
__device__ __forceinline__ void acc_scale(float alpha) {
  float t0, t1;
  asm volatile(
      ".set gqla_i, 0\n.rept 128\n"
      "\tv_accvgpr_read_b32 %0, a[gqla_i]\n\tv_accvgpr_read_b32 %1, a[gqla_i+1]\n"
      "\tv_mul_f32 %0, %0, %2\n\tv_mul_f32 %1, %1, %2\n\ts_nop 0\n"
      "\tv_accvgpr_write_b32 a[gqla_i], %0\n\tv_accvgpr_write_b32 a[gqla_i+1], %1\n"
      ".set gqla_i, gqla_i+2\n.endr"
      : "=&v"(t0), "=&v"(t1)
      : "v"(alpha));
}
// tile dt into 16 ordinary registers (first call after the last MFMA: pass wait = true)
__device__ __forceinline__ void acc_read(int dt, bool wait, float (&x)[16]) {
  if (wait) asm volatile("s_nop 15\n\ts_nop 7");
  switch (dt) {
#define X(D)                                                                                                            \
  case D:                                                                                                               \
    asm volatile(".set gqla_i, 0\n.irp r, %0, %1, %2, %3, %4, %5, %6, %7, %8, %9, %10, %11, %12, %13, %14, %15\n"        \
                 "\tv_accvgpr_read_b32 \\r, a[" #D "*16+gqla_i]\n.set gqla_i, gqla_i+1\n.endr"                           \
                 : "=v"(x[0]), "=v"(x[1]), "=v"(x[2]), "=v"(x[3]), "=v"(x[4]), "=v"(x[5]), "=v"(x[6]), "=v"(x[7]),      \
                   "=v"(x[8]), "=v"(x[9]), "=v"(x[10]), "=v"(x[11]), "=v"(x[12]), "=v"(x[13]), "=v"(x[14]), "=v"(x[15])); \
    break;
    GQLA_FOR_DT(X)
#undef X
  }
}

// The layout above; any row count (whole blocks of 128 rows and at most 32 rows per workgroup have kernels of their own below).
template <int RKV, int DR>
__global__ void __launch_bounds__(256) decode_absorb_bf16_kernel(DecodeArgs a, int row_blocks) {
  constexpr int W = RKV + DR;        // elements per latent row
  constexpr int ROWB = W * 2;        // bytes per latent row
  constexpr int NP = W / 64;         // 128-byte panels per latent row
  constexpr int PANEL = kTile * 128; // bytes per panel
  constexpr int KS = W / 16;         // k-steps of the key contraction
  constexpr int DT = RKV / 32;       // 32-wide tiles of the latent output
  constexpr int TILE_BYTES = kTile * ROWB;
  static_assert(W % 64 == 0 && RKV % 64 == 0, "latent row must be a whole number of 128-byte panels");
  static_assert((16 + 8 + 4) * 128 + 128 + PANEL * (RKV / 64 - 1) < 65536, "value-fragment offsets must fit the 16-bit LDS immediate");
  extern __shared__ __attribute__((aligned(16))) char smem[];

  // blockIdx -> (chunk, row block): the row blocks of one chunk get ids that are equal modulo 8 so that they run on
  // the same XCD (ids are dealt round-robin over the 8 XCDs) and share the chunk's cache lines in that XCD's L2.
  int chunk, rbk;
  {
    const int id = blockIdx.x;
    const int grp = id / (8 * row_blocks), rem = id % (8 * row_blocks);
    rbk = rem / 8;
    chunk = grp * 8 + rem % 8;
  }
  if (chunk >= a.n_chunks) return;  // whole workgroup leaves together
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform by construction: keep it scalar
  const int n = lane & 31, h = lane >> 5;
  const ChunkEntry ce = a.chunks[chunk];

  const int rho = rbk * kRowsPerBlock + wave * 32 + n;  // row = t * h_q + i
  const bool row_ok = rho < a.M;
  const int t = row_ok ? rho / a.h_q : 0;
  const int vis_end = row_ok ? min(ce.tok_end, ce.L - a.s_q + t + 1) : 0;
  const int unmasked_end = min(ce.tok_end, ce.L - a.s_q + 1);
  const bool wave_active = rbk * kRowsPerBlock + wave * 32 < a.M;

  const int P = a.cache.page_size;
  const char* pool = (const char*)a.cache.pool;
  // Tiles are always staged whole: rows past the chunk end still come from the page (allocated memory), an
  // out-of-pool page id falls back to page 0; such rows are zeroed in LDS before use (see the loop).
  const int32_t* table_row = a.cache.page_table ? a.cache.page_table + (int64_t)ce.b * a.cache.max_pages : nullptr;
  auto checked = [&](int32_t pg) -> int32_t { return ((uint32_t)pg < (uint32_t)a.cache.num_pages) ? pg : -1; };
  auto tile_src = [&](int32_t pg, int slot) -> const char* {  // first row of a tile: page pg (or page 0), slot `slot`
    return pool + ((int64_t)(pg >= 0 ? pg : 0) * P + slot) * ROWB;
  };

  // Per-lane LDS byte offsets inside a tile (panel layout of gqla_lds.h; everything else is a compile-time offset):
  //  key fragments     row n, chunk 2*ks + h with ks = 4*a4 + b: panel a4, in-panel chunk 2*b + h
  //                    -> four bases (b = 0..3), plus a4*PANEL.
  //  value fragments   (transposed reads) this lane addresses row R0 + 4*h + e (and 8 rows further for the second read),
  //                    4 columns at 32*dt + 16*g1 + 4*q: panel dt/2, in-panel chunk 4*(dt & 1) + cl, cl = 2*g1 + q/2.
  //                    With R0 a multiple of 16 the chunk lands at (4*(dt & 1) + cl) ^ lds_swz(4*h + e); 8 rows further the
  //                    swizzle differs in bit 0, so dt & 1 flips bit 2 of the chunk (64 bytes) and the second read bit 0 (16 bytes): one
  //                    base per lane.
  uint32_t kbase[4], vbase;
  {
#pragma unroll
    for (int b = 0; b < 4; ++b) kbase[b] = n * 128 + (((2 * b + h) ^ lds_swz(n)) << 4);
    const int i16 = lane & 15, e = i16 >> 2, q = i16 & 3, g1 = (lane >> 4) & 1;
    vbase = (4 * h + e) * 128 + (((2 * g1 + (q >> 1)) ^ lds_swz(4 * h + e)) << 4) + (q & 1) * 8;
  }

  static_assert(DT == 16, "O^T fills the 256 accumulation registers exactly");
  acc_zero();
  float m_ref = GQLA_NEG_INF, l_run = 0.f;

  // Ring of kSlots tile buffers.  Tile it + kAhead is staged (9 LDS-DMA instructions per wave, after the S phase)
  // while tile `it` is worked on, so every load has about three tile times to land and only a few KB per wave are
  // ever requested at once.  Loads complete in issue order, so "tile `it` has landed" is a count:
  // at most the instructions of the tiles staged after it may still be outstanding.  No other vector-memory
  // instruction is issued inside the loop: page ids come through the scalar cache, one tile ahead of their use.
  constexpr int kAhead = kSlots - 1;
  constexpr int kStageSteps = NP * (kTile / 8 / 4);  // LDS-DMA instructions per wave and tile
  static_assert(kStageSteps == 9, "the wait counts below assume 9 instructions per wave and tile");
  const int n_tiles = (ce.tok_end - ce.tok_begin + kTile - 1) / kTile;
  // page ids of tiles it, it+1, it+2 (staged) and it+3 (staged during tile it); the four first lookups go out together
  // (indices clamped to the chunk's last page, results of tiles that do not exist discarded)
  int32_t pg0, pg1, pg2, pg3;
  {
    const int p_last = (ce.tok_end - 1) / P;
    int32_t raw[4];
    if (table_row) {  // four scalar loads in flight together, one wait
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int p = __builtin_amdgcn_readfirstlane(min(ce.tok_begin / P + (k * kTile) / P, p_last));
        asm volatile("s_load_dword %0, %1, 0x0" : "=s"(raw[k]) : "s"(table_row + p) : "memory");
      }
      asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(raw[0]), "+s"(raw[1]), "+s"(raw[2]), "+s"(raw[3]) : : "memory");
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) raw[k] = ce.b * a.cache.max_pages + min(ce.tok_begin / P + (k * kTile) / P, p_last);
    }
    pg0 = checked(raw[0]);
    pg1 = n_tiles > 1 ? checked(raw[1]) : -1;
    pg2 = n_tiles > 2 ? checked(raw[2]) : -1;
    pg3 = n_tiles > 3 ? checked(raw[3]) : -1;
  }
  int32_t pg_raw = 0;  // table entry of tile it + 4, in flight through the scalar cache
  // Chunks start on a page boundary and pages hold a whole number of tiles: (page index, slot) of the tiles ahead are
  // advanced by addition, and the table is consulted once per page.
  const int p_first = ce.tok_begin / P;
  int st_slot = (kAhead * kTile) % P;                                       // slot of tile it + 3 in its page
  int lk_slot = ((kAhead + 1) * kTile) % P, lk_p = p_first + ((kAhead + 1) * kTile) / P;  // tile it + 4
  static_assert(kAhead == 3, "the page-id shift register holds four tiles");
  stage_panels_full<kTile, NP, 4, ROWB, true>(smem, tile_src(pg0, 0), wave, lane);
  if (n_tiles > 1) stage_panels_full<kTile, NP, 4, ROWB, true>(smem + TILE_BYTES, tile_src(pg1, kTile % P), wave, lane);
  if (n_tiles > 2) stage_panels_full<kTile, NP, 4, ROWB, true>(smem + 2 * TILE_BYTES, tile_src(pg2, (2 * kTile) % P), wave, lane);

  // queries of this lane's row, as B fragments: [q_hat (RKV) | q_R (DR)], 8 consecutive dims per k-step
  bf16x8 qf[KS];
  {
    const int64_t qrow = (int64_t)ce.b * a.M + min(rho, a.M - 1);
    const __bf16* ph = (const __bf16*)a.q_a + qrow * RKV + h * 8;
    const __bf16* pr = (const __bf16*)a.q_r + qrow * DR + h * 8;
#pragma unroll
    for (int a4 = 0; a4 < KS / 4; ++a4)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        qf[a4 * 4 + b] = *(const bf16x8*)((a4 < RKV / 64 ? ph + a4 * 64 : pr + (a4 - RKV / 64) * 64) + b * 16);
  }

  // The query loads go out behind the first tile requests (one memory latency for both) and are made to complete
  // here, before the loop.  Otherwise the compiler, which counts only the loads it issued itself, keeps "wait for
  // the query loads" counts in front of the loop's first MFMAs; on the hardware counter those waits would also
  // cover the tile requests in flight and drain the ring on every tile.  (The wait that the compiler places here
  // covers the three tiles requested above as well; the loop's own counted waits then pass at once for them.)
#pragma unroll
  for (int k = 0; k < KS; k += 9)
    asm volatile("" : "+v"(qf[k]), "+v"(qf[k + 1]), "+v"(qf[k + 2]), "+v"(qf[k + 3]), "+v"(qf[k + 4]), "+v"(qf[k + 5]),
                      "+v"(qf[k + 6]), "+v"(qf[k + 7]), "+v"(qf[k + 8]));
  static_assert(KS % 9 == 0, "query fragments are touched nine at a time");

#pragma unroll 1
  for (int it = 0; it < n_tiles; ++it) {
    const int tok = ce.tok_begin + it * kTile;
    const char* buf = smem + (it & (kSlots - 1)) * TILE_BYTES;
    // everything that does not need the tile goes before the wait for it
    const bool stage_next = it + kAhead < n_tiles;
    const char* next_g = tile_src(stage_next ? pg3 : 0, st_slot);
    char* next_buf = smem + ((it + kAhead) & (kSlots - 1)) * TILE_BYTES;
    const bool lookup = it + kAhead + 1 < n_tiles;
    const bool new_page = lookup && lk_slot == 0;
    if (new_page && table_row)  // scalar load, consumed at the end of the tile (its wait is written out there)
      asm volatile("s_load_dword %0, %1, 0x0" : "=s"(pg_raw) : "s"(table_row + lk_p) : "memory");
    {
      const int behind = min(kAhead - 1, n_tiles - 1 - it);  // tiles staged after this one
      if (behind >= 2) asm volatile("s_waitcnt vmcnt(18)" ::: "memory");
      else if (behind == 1) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();  // tile `it` has landed for every wave; every wave is done reading tile it-1
    const bool tile_ok = pg0 >= 0;
    const int valid = tile_ok ? min(kTile, ce.tok_end - tok) : 0;
    if (valid < kTile) {
      // rows past the chunk end hold whatever the page holds (NaN bits included): zero them so that 0 * v stays 0
      for (int idx = threadIdx.x; idx < (kTile - valid) * (W / 8); idx += 256) {
        const int r = valid + idx / (W / 8), c = idx % (W / 8);
        *(u32x4*)(smem + (it & (kSlots - 1)) * TILE_BYTES + (c >> 3) * PANEL + r * 128 + (c & 7) * 16) = u32x4{0u, 0u, 0u, 0u};
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      __syncthreads();
    }

    auto shift_pages = [&]() {  // tile it+1 becomes current; the page of tile it + 4 joins the window
      if (new_page && table_row) asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(pg_raw) : : "memory");
      pg0 = pg1;
      pg1 = pg2;
      pg2 = pg3;
      if (new_page) pg3 = checked(table_row ? pg_raw : ce.b * a.cache.max_pages + lk_p);
      if (!lookup) pg3 = -1;
      st_slot = lk_slot;
      lk_slot += kTile;
      if (lk_slot == P) {
        lk_slot = 0;
        ++lk_p;
      }
    };
    if (!wave_active) {  // waves without query rows only help staging (uniform per wave): their share, in one burst
      if (stage_next) stage_panels_full<kTile, NP, 4, ROWB, true>(next_buf, next_g, wave, lane);
      shift_pages();
      continue;
    }
    {
      const bool need_mask = (tok + kTile > unmasked_end) || !row_ok || !tile_ok;
      const int lim = tile_ok ? vis_end : 0;

      // ---- S^T[token][row] = Kt * Qhat^T ----
      // These MFMAs accumulate in ordinary VGPRs (written as inline assembly) because all 256 accumulation
      // registers hold O^T; the compiler's own MFMA selection would put S^T there as well and spill.
      f32x16 s;
      {
        bf16x8 f[3][4];  // ring of fragment batches: loads run two batches (8 MFMAs) ahead of their use
#pragma unroll
        for (int b = 0; b < 4; ++b) f[0][b] = *(const bf16x8*)(buf + kbase[b]);
#pragma unroll
        for (int b = 0; b < 4; ++b) f[1][b] = *(const bf16x8*)(buf + kbase[b] + PANEL);
#pragma unroll
        for (int a4 = 0; a4 < KS / 4; ++a4) {
          if (a4 + 2 < KS / 4) {
#pragma unroll
            for (int b = 0; b < 4; ++b) f[(a4 + 2) % 3][b] = *(const bf16x8*)(buf + kbase[b] + ((a4 + 2) * PANEL));
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            if (a4 == 0 && b == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(f[0][0]), "v"(qf[0]));  // result registers must not overlap the operands
            else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(f[a4 % 3][b]), "v"(qf[4 * a4 + b]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // Tile it + kAhead is requested here, in one burst: at this point no LDS read of this wave is outstanding.
      // (An LDS-DMA instruction issued while reads are in flight holds the wave, and with it the MFMA stream, until
      // they have returned.)
      if (stage_next) stage_panels_full<kTile, NP, 4, ROWB, true>(next_buf, next_g, wave, lane);
      // first batches of value fragments: issued now, consumed after the softmax
      i16x4 r[3][4][2];
      auto load_v = [&](int slot, int u, int p4) {  // output tiles dt = 4*p4 .. 4*p4 + 3 of k-step u
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int dt = 4 * p4 + d;
          const int off = (dt >> 1) * PANEL + (16 * u) * 128;
          r[slot][d][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(buf + (vbase ^ (64 * (dt & 1))) + off));
          r[slot][d][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(buf + (vbase ^ (64 * (dt & 1) + 16)) + (off + 8 * 128)));
        }
      };
      constexpr int NBT = 2 * (DT / 4);  // batches of four value fragments: k-step bt / (DT/4), tiles 4*(bt % (DT/4)) ..
      load_v(0, 0, 0);
      load_v(1, 1 / (DT / 4), 1 % (DT / 4));
      // the matrix pipeline's result is not interlocked against vector-ALU reads: wait out its 8 passes
      asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s));

      // ---- online softmax (base 2); register i is token tok + 8*(i/4) + 4*h + i%4 ----
      // The maximum is taken on the raw logits (the scale is positive) and the scale rides in the exponent's FMA.
      if (__builtin_amdgcn_ballot_w64(need_mask) != 0) {  // wave-uniform: only tiles at the chunk end, or padding rows
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (need_mask && tok + 8 * (i >> 2) + 4 * h + (i & 3) >= lim) s[i] = GQLA_NEG_INF;
      }
      float tmax = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, s[i]);
      tmax = pair_max(tmax) * a.scale_log2e;
      if (__builtin_amdgcn_ballot_w64(tmax > m_ref + kRescaleThreshold) != 0) {
        const float m_new = fmaxf(m_ref, tmax);
        const float alpha = fast_exp2(m_ref - ((m_new == GQLA_NEG_INF) ? 0.f : m_new));
        m_ref = m_new;
        l_run *= alpha;
        if (it > 0) acc_scale(alpha);
      }
      const float m_use = (m_ref == GQLA_NEG_INF) ? 0.f : m_ref;
      // P^T fragments, k-step u: tokens 16*u + {4h..4h+3, 8+4h..8+4h+3}.  Only the first is finished before the
      // O^T update starts; the exponentials of the second ride in the shadow of the first k-step's MFMAs (one
      // exponential, its FMA and its add fit behind one MFMA of the same wave).
      bf16x8 pf[2];
      float p1[8];
      u32x4 w1;
      {
        float p[8], psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          p[e] = fast_exp2(__builtin_fmaf(s[e], a.scale_log2e, -m_use));
          psum += p[e];
        }
        u32x4 w = {pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])};
        pf[0] = __builtin_bit_cast(bf16x8, w);
        l_run += psum;
      }
      // An MFMA may read a register as an operand no sooner than two wait states after a vector-ALU instruction wrote
      // it.  The compiler keeps that distance for its own MFMAs but does not look inside inline assembly, so the
      // distance between the last pack of the probabilities and the first O^T update is made here.
      asm volatile("s_nop 1" : "+v"(pf[0]));
      __builtin_amdgcn_sched_barrier(0);

      // ---- O^T[r][row] += C^T * P^T, value fragments one batch of four tiles ahead ----
#pragma unroll
      for (int bt = 0; bt < NBT; ++bt) {
        const int u = bt / (DT / 4), p4 = bt % (DT / 4);
        if (bt + 2 < NBT) load_v((bt + 2) % 3, (bt + 2) / (DT / 4), (bt + 2) % (DT / 4));
        if (bt == DT / 4) pf[1] = __builtin_bit_cast(bf16x8, w1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const i16x4 lo = r[bt % 3][d][0], hi = r[bt % 3][d][1];
          const i16x8 fr = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          acc_mfma(4 * p4 + d, __builtin_bit_cast(bf16x8, fr), pf[u]);
          if (u == 0) {  // second k-step's probabilities, one piece per MFMA
            const int idx = 4 * bt + d;
            if (idx < 8) {
              p1[idx] = fast_exp2(__builtin_fmaf(s[8 + idx], a.scale_log2e, -m_use));
              l_run += p1[idx];
            } else if (idx < 12) {
              w1[idx - 8] = pack_bf16(p1[2 * (idx - 8)], p1[2 * (idx - 8) + 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    shift_pages();
  }

  const float l_tot = pair_sum(l_run);
  if (!row_ok) return;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const int64_t prow = (int64_t)chunk * a.M + rho;
  // this lane holds dims 4 h .. 4 h + 3 of vector 4 dt + q of its row: with consecutive rows in consecutive
  // lanes a store instruction writes 512 contiguous bytes
  __bf16* po = (__bf16*)a.part_o + part_vec_index(chunk, rho, a.M, RKV / 8, 0) * 8 + 4 * h;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    float x[16];
    acc_read(dt, dt == 0, x);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      u32x2 v = {pack_bf16(x[4 * q] * inv, x[4 * q + 1] * inv), pack_bf16(x[4 * q + 2] * inv, x[4 * q + 3] * inv)};
      *(u32x2*)(po + (dt * 4 + q) * (32 * 8)) = v;
    }
  }
  if (h == 0) a.part_lse[prow] = l_tot > 0.f ? (m_ref + fast_log2(l_tot)) * kLn2 : GQLA_NEG_INF;
}

// eight E4M3 codes as bf16 (exact)
__device__ __forceinline__ bf16x8 widen_e4m3x8(uint32_t w0, uint32_t w1) {
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2v;
  const bf16x2v p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, false), p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, true);
  const bf16x2v p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, false), p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, true);
  const u32x4 r = {__builtin_bit_cast(uint32_t, p0), __builtin_bit_cast(uint32_t, p1), __builtin_bit_cast(uint32_t, p2), __builtin_bit_cast(uint32_t, p3)};
  return __builtin_bit_cast(bf16x8, r);
}

// At most 32 query rows per workgroup (at most 32 rows per sequence, or so few chunks that one workgroup per 32 rows still
// fits the chip in one round).  With so few rows a tile is little work and what costs is the chain of a tile -- S^T, softmax,
// probabilities to everyone, O^T -- on which one wave per SIMD issues at best an instruction every four cycles.  So eight
// waves, two per SIMD, take pairs of tiles (64 tokens) with one barrier per pair:
//   S^T: wave w owns 16 tokens (16 (w & 3) ..) against 16 rows (16 (w >> 2) ..) over the whole key dimension: 18 MFMAs of
//        16 x 16 x 32, no partial sums to trade, four logits per lane.
//   P^T: published in LDS, already in operand order.
//   O^T: wave w owns latent dims 64 w .. 64 w + 63 of all 32 rows, one pair late: iteration j is
//        barrier (pair j has landed, probabilities of j - 1 published) | requests for pair j + 1, into the buffers of j - 1,
//        whose value fragments are in registers | S^T(j) and O^T(j - 1) | value fragments of j requested, softmax, P^T(j) out
// The queries come through the ring (same layout and fragment addresses as keys) with the first tiles.
// The reference maximum of a row is common to the eight waves and moves rarely (threshold 2^8): a wave that wants to move it
// says so in the sign bit of a probability, which every wave reads with its operands; all then trade their maxima, rescale,
// and publish the probabilities of that pair again.
// Measured: one sequence of 8192 tokens x 128 rows (88 workgroups of 6 pairs) 23.0 -> 15.5 us, against four waves that split
// the key dimension and traded fp32 partial sums (2.9 k cycles a tile; the same four waves with O^T one tile late: 22.0 us);
// one of 32768 tokens x 16 rows 81 -> 46 us for the whole step; 32 ragged sequences of 4096 tokens x 32 rows (151 MB, all
// compute units) 34.9 -> 29.5 us, 5.1 TB/s: there the loop runs at the memory's rate and the rest is its start.
// FP8: the cache holds E4M3 codes of c_kv (one scale) and k_R in 16 bits (page format: see the next kernel).  Codes are staged
// as they are -- a pair takes 40 KB, so three pairs fit and two are under way -- and widened in registers (exact): the keys
// by each wave for its 16 tokens, 64 conversions a pair, the values out of transposed 8-bit reads, 32.  Against four waves
// that split the key dimension, widened each tile through registers into a bf16 buffer and traded fp32 partial sums with two
// barriers a tile (step without W^O): one sequence of 8192 tokens x 128 rows 42.2 -> 31.0 us, 64 x 8192 x 16 rows
// 144 -> 76 us, 128 ragged sequences x 20 rows 80 -> 56 us.
template <int RKV, int DR, bool FP8>
__global__ void __launch_bounds__(512) decode_absorb_rows32_bf16_kernel(DecodeArgs a, int row_blocks, float c_scale) {
  constexpr int W = RKV + DR;
  constexpr int CB = FP8 ? 1 : 2;             // bytes per element of c_kv
  constexpr int ROWB = FP8 ? RKV : 2 * W;     // bytes from one row of a page to the next
  constexpr int NPC = RKV * CB / 128;         // panels of c_kv; k_R is one more
  constexpr int NP = NPC + 1;
  constexpr int QP = W / 64;                  // panels of the queries
  constexpr int PANEL = kTile * 128;
  constexpr int KS = W / 32;                  // k-steps of 32
  constexpr int KS_C = RKV / 32;
  constexpr int TILE_BYTES = NP * PANEL;
  constexpr int PAIRS = FP8 ? 3 : 2;          // ring: pairs of tiles
  constexpr int QBUF = FP8 ? 4 : 3;           // tile buffer where the queries start out
  constexpr int kQPanels = (QP + 1) / 2;      // panels of the queries that waves 0..3 request; the others take the rest
  static_assert(RKV == 512 && DR == 64, "eight waves of 64 latent dims");
  static_assert(QBUF * TILE_BYTES + QP * PANEL <= 2 * PAIRS * TILE_BYTES, "the queries lie in the ring");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // Probabilities, [parity of the pair][16 tokens][lane] 16 bytes: with one barrier per pair a wave may publish those of pair
  // j while another still reads those of j - 1.
  char* const pex = smem + 2 * PAIRS * TILE_BYTES;
  float* const mex = (float*)(pex + 2 * 4096);   // row maxima, and at the end the denominators: [16 tokens][row]

  int chunk, rbk;
  {
    const int id = blockIdx.x;
    const int grp = id / (8 * row_blocks), rem = id % (8 * row_blocks);
    rbk = rem / 8;
    chunk = grp * 8 + rem % 8;
  }
  if (chunk >= a.n_chunks) return;  // whole workgroup leaves together
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;        // O^T: row n
  const int n16 = lane & 15, g4 = lane >> 4;     // S^T: row 16 rh + n16, tokens 16 tb + 4 g4 + 0..3
  const int tb = wave & 3, rh = wave >> 2;       // (staging: wave tb of the four that request tile rh of a pair)
  const ChunkEntry ce = a.chunks[chunk];
  const int rho0 = rbk * 32;
  const int rho = rho0 + 16 * rh + n16;
  const bool row_ok = rho < a.M;
  const int vis_end = row_ok ? min(ce.tok_end, ce.L - a.s_q + rho / a.h_q + 1) : 0;
  const int unmasked_end = rho0 + 16 * rh + 16 <= a.M ? min(ce.tok_end, ce.L - a.s_q + 1) : 0;  // wave-uniform
  const int P = a.cache.page_size;
  const char* pool = (const char*)a.cache.pool;
  const int32_t* table_row = a.cache.page_table ? a.cache.page_table + (int64_t)ce.b * a.cache.max_pages : nullptr;
  auto checked = [&](int32_t pg) -> int32_t { return ((uint32_t)pg < (uint32_t)a.cache.num_pages) ? pg : -1; };
  // tiles are always staged whole: rows past the chunk end come from the page, an out-of-pool page id falls back to page 0;
  // such rows are zeroed in LDS before use
  const int64_t page_bytes = (int64_t)P * (RKV * CB + DR * 2);
  auto tile_src = [&](int32_t pg, int slot) -> const char* { return pool + (int64_t)(pg >= 0 ? pg : 0) * page_bytes + (int64_t)slot * ROWB; };

  {  // queries into buffer QBUF; rows beyond the last read that one instead (their results are not stored)
    const int srow = 8 * tb + (lane >> 3), c = (lane & 7) ^ lds_swz(srow);
    const int64_t qrow = (int64_t)ce.b * a.M + min(rho0 + srow, a.M - 1);
    const char* gh = (const char*)a.q_a + qrow * (RKV * 2) + c * 16;
    const char* gr = (const char*)a.q_r + qrow * (DR * 2) + c * 16;
#pragma unroll
    for (int u = 0; u < QP; ++u) {
      if ((u < kQPanels) != (rh == 0)) continue;
      const uint32_t dst = (uint32_t)(uintptr_t)(lds_ptr_t)(smem + QBUF * TILE_BYTES + u * PANEL + tb * 1024);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dst), "v"(u < RKV / 64 ? gh + u * 128 : gr + (u - RKV / 64) * 128) : "memory");
    }
  }
  const int n_tiles = (ce.tok_end - ce.tok_begin + kTile - 1) / kTile;
  const int n_pairs = (n_tiles + 1) / 2;
  // A pair of tiles lies in one page (pages hold a multiple of 64 tokens, chunks start on one).  Pages of pairs j (pg[0]) to
  // j + PAIRS - 1, whose first tokens are in slots slot[..]; the table entry of pair j + PAIRS is looked up during iteration j
  // through the scalar cache.  (lk_p, lk_slot): page index and slot of the next pair to look up.
  constexpr int kPair = 2 * kTile;
  int lk_p = ce.tok_begin / P, lk_slot = 0;
  auto advance = [&]() {
    lk_slot += kPair;
    if (lk_slot == P) {
      lk_slot = 0;
      ++lk_p;
    }
  };
  int32_t pg[PAIRS], raw = 0;
  int slot[PAIRS];
  {
    int p[PAIRS];
    int32_t r[PAIRS];
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) {
      p[u] = __builtin_amdgcn_readfirstlane(u < n_pairs ? lk_p : p[0]);
      slot[u] = lk_slot;
      advance();
    }
    if (table_row) {  // the scalar loads in flight together, one wait
#pragma unroll
      for (int u = 0; u < PAIRS; ++u) asm volatile("s_load_dword %0, %1, 0x0" : "=s"(r[u]) : "s"(table_row + p[u]) : "memory");
      if constexpr (PAIRS == 3) asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(r[0]), "+s"(r[1]), "+s"(r[PAIRS - 1]) : : "memory");
      else asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(r[0]), "+s"(r[1]) : : "memory");
    } else {
#pragma unroll
      for (int u = 0; u < PAIRS; ++u) r[u] = ce.b * a.cache.max_pages + p[u];
    }
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) pg[u] = checked(r[u]);
  }
  auto stage_tile = [&](int buffer, int32_t page, int row) {
    char* dst = smem + buffer * TILE_BYTES;
    if constexpr (FP8) {  // codes, and k_R out of its plane behind the codes of the page
      stage_panels_full<kTile, NPC, 4, RKV, true>(dst, tile_src(page, row), tb, lane);
      stage_panels_full<kTile, 1, 4, DR * 2, true>(dst + NPC * PANEL, tile_src(page, 0) + (int64_t)P * RKV + (int64_t)row * (DR * 2), tb, lane);
    } else {
      stage_panels_full<kTile, NP, 4, ROWB, true>(dst, tile_src(page, row), tb, lane);
    }
  };
  // Tiles 0 and 1, and behind them what lies clear of the queries: tile 2 (16 bits), tiles 2 and 3 (8 bits).  Wave group rh
  // requests tile rh of a pair.
  const bool ahead = 2 + rh < n_tiles && (FP8 || rh == 0);  // this wave has requests of pair 1 out
  if (rh < n_tiles) stage_tile(rh, pg[0], rh * kTile);
  if (ahead) stage_tile(2 + rh, pg[1], slot[1] + rh * kTile);

  // per-lane LDS offsets.  Operand fragments of S^T, k-step ks: panel ks / 2, in-panel chunk 2 (ks & 1) + place(g4) with
  // place = 0, 4, 1, 5: lanes 16 apart then read chunks 4 apart, which keeps the 16 lanes that the LDS serves together (16
  // rows, half of them on each of the two chunks) on different banks.  8 bits: a 16-byte vector of codes is a lane's share of
  // two k-steps, dims 128 (ks / 4) + 16 (2 (ks / 2 % 2) + place(g4)) + 8 (ks % 2) + 0..7 (qcode[ks % 4]: the queries of those
  // dims).
  uint32_t kbase[2], qbase[2], qcode[4], vbase;
  {
    const int krow = 16 * (tb & 1) + n16, qrow = 16 * rh + n16, place = 4 * (g4 & 1) + (g4 >> 1);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      kbase[b] = (tb >> 1) * TILE_BYTES + krow * 128 + (((2 * b + place) ^ lds_swz(krow)) << 4);
      qbase[b] = QBUF * TILE_BYTES + qrow * 128 + (((2 * b + place) ^ lds_swz(qrow)) << 4);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
      qcode[b] = QBUF * TILE_BYTES + (g4 & 1) * PANEL + qrow * 128 + (((2 * ((g4 >> 1) + 2 * (b >> 1)) + (b & 1)) ^ lds_swz(qrow)) << 4);
    // value fragments (transposed reads): as in the kernel above, panel `wave`
    const int i16 = lane & 15, e = i16 >> 2, q = i16 & 3, g1 = (lane >> 4) & 1;
    if constexpr (FP8) {  // 8-bit transposed reads: see the next kernel; dim tile d is chunks d, d + 2 of half a panel
      const int t = i16 >> 1, row = 8 * (t >> 2) + 4 * h + (t & 3);
      vbase = row * 128 + (((4 * (wave & 1) + 2 * g1) ^ lds_swz(row)) << 4) + (i16 & 1) * 8 + (wave >> 1) * PANEL;
    } else {
      vbase = (4 * h + e) * 128 + (((2 * g1 + (q >> 1)) ^ lds_swz(4 * h + e)) << 4) + (q & 1) * 8 + wave * PANEL;
    }
  }
  f32x16 o[2];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[d][i] = 0.f;
  float m_s = GQLA_NEG_INF, m_o = GQLA_NEG_INF, l_run = 0.f;  // reference of this lane's row in S^T, in O^T

  // queries and tiles 0, 1 (pair 1, where this wave has a part in it, was requested last)
  if (ahead) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NP) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  bf16x8 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(FP8 && ks < KS_C ? smem + qcode[ks & 3] + 2 * (ks >> 2) * PANEL : smem + qbase[ks & 1] + (ks >> 1) * PANEL);

  float z[4], z_max = GQLA_NEG_INF, psum_last = 0.f;  // of the last pair: raw logits, scaled maximum, sum of probabilities
  typedef typename std::conditional<FP8, u32x2, i16x4>::type value_t;
  value_t r[4][2][FP8 ? 1 : 2] = {};                  // value fragments of the last pair (8 bits: codes)
  char* const p_dst = pex + tb * 1024 + ((g4 & 1) * 32 + 16 * rh + n16) * 16 + (g4 >> 1) * 8;
  auto publish = [&](int pair, float m_use, bool flag) {
    float p[4], sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = fast_exp2(__builtin_fmaf(z[i], a.scale_log2e, -m_use));
      sum += p[i];
    }
    *(u32x2*)(p_dst + (pair & 1) * 4096) = u32x2{pack_bf16(p[0], p[1]) | (flag ? 0x8000u : 0u), pack_bf16(p[2], p[3])};
    return sum;
  };

  int ring = 0;  // j % PAIRS
#pragma unroll 1
  for (int j = 0;; ++j) {
    const int tok = ce.tok_begin + j * kPair;
    char* const buf = smem + ring * 2 * TILE_BYTES;
    const bool more = j < n_pairs;
    const bool lookup = j + PAIRS < n_pairs;
    const int look_slot = lk_slot;
    if (lookup) {
      const int p = __builtin_amdgcn_readfirstlane(lk_p);
      if (table_row) asm volatile("s_load_dword %0, %1, 0x0" : "=s"(raw) : "s"(table_row + p) : "memory");  // consumed at the end of the iteration (the wait is written out there)
      else raw = ce.b * a.cache.max_pages + p;
      advance();
    }
    if (j > 0) {  // pair j has landed; 8 bits: pair j + 1 may be under way
      if (FP8 && 2 * j + 2 + rh < n_tiles) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NP) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    const int last = ring == 0 ? PAIRS - 1 : ring - 1;  // buffers of pair j - 1, for pair j + PAIRS - 1
    if (2 * (j + PAIRS - 1) + rh < n_tiles && !(j == 0 && ahead && !FP8)) stage_tile(2 * last + rh, pg[PAIRS - 1], slot[PAIRS - 1] + rh * kTile);
    const bool whole = pg[0] >= 0 && tok + kPair <= ce.tok_end;
    if (more && !whole) {
      // rows past the chunk end hold whatever the page holds (NaN bits included): zero them so that 0 * v stays 0
      const int valid = pg[0] >= 0 ? max(ce.tok_end - tok, 0) : 0;
      for (int idx = threadIdx.x; idx < (kPair - valid) * (NP * 8); idx += 512) {
        const int rr = valid + idx / (NP * 8), c = idx % (NP * 8);
        *(u32x4*)(buf + rr / kTile * TILE_BYTES + (c >> 3) * PANEL + rr % kTile * 128 + (c & 7) * 16) = u32x4{0u, 0u, 0u, 0u};
      }
      __syncthreads();
    }
    // operands of the iteration: probabilities of the last pair (0 ahead of the first: O^T is updated without a branch), key
    // fragments of this one (behind the last, whatever is there: not used)
    u32x4 pw[4];
    auto read_p = [&]() {
#pragma unroll
      for (int u = 0; u < 4; ++u) pw[u] = *(const u32x4*)(pex + ((j - 1) & 1) * 4096 + u * 1024 + lane * 16);
    };
    if (j > 0) {
      read_p();
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) pw[u] = u32x4{0u, 0u, 0u, 0u};
    }
    auto key_frag = [&](int ks) { return *(const bf16x8*)(buf + kbase[ks & 1] + (ks >> 1) * PANEL); };
    constexpr int KF = FP8 ? KS_C / 2 + KS - KS_C : KS / 2;  // fragments requested ahead (8 bits: all, codes of two k-steps each, then k_R)
    bf16x8 f[KF];
    static_for<KF>([&](auto k) {
      constexpr int u = decltype(k)::value;
      // (8 bits: vectors 0 .. KS_C / 2 - 1 of codes, then k-steps KS_C, KS_C + 1 of the last panel, k_R)
      f[u] = FP8 && u >= KS_C / 2 ? *(const bf16x8*)(buf + kbase[u & 1] + NPC * PANEL) : key_frag(u);
    });
    if (j > 0) {
      const uint32_t flags = pw[0][0] | pw[0][2] | pw[1][0] | pw[1][2] | pw[2][0] | pw[2][2] | pw[3][0] | pw[3][2];
      if (__builtin_amdgcn_ballot_w64((flags & 0x8000u) != 0) != 0) {  // the same bits in every wave: all come here or none
        if (g4 == 0) mex[tb * 32 + 16 * rh + n16] = z_max;
        __syncthreads();  // (also: every wave has read the probabilities that are about to be replaced)
        auto moved = [&](float m, int row) {
#pragma unroll
          for (int k = 0; k < 4; ++k) m = fmaxf(m, mex[k * 32 + row]);
          return m;
        };
        auto factor = [&](float m_old, float m_new) { return fast_exp2(m_old - ((m_new == GQLA_NEG_INF) ? 0.f : m_new)); };
        const float ms_new = moved(m_s, 16 * rh + n16), mo_new = moved(m_o, n);
        l_run *= factor(m_s, ms_new);
        if (j > 1) {
          const float alpha = factor(m_o, mo_new);
#pragma unroll
          for (int d = 0; d < 2; ++d) o[d] *= alpha;
        }
        m_s = ms_new;
        m_o = mo_new;
        psum_last = publish(j - 1, (m_s == GQLA_NEG_INF) ? 0.f : m_s, false);
        __syncthreads();
        read_p();
      }
      l_run += psum_last;
    }
    auto output_step = [&](auto uc) {  // O^T of the last pair, 16 tokens
      constexpr int u = decltype(uc)::value;
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        bf16x8 fr;
        if constexpr (FP8) {
          fr = widen_e4m3x8(r[u][d][0][0], r[u][d][0][1]);
        } else {
          const i16x4 lo = r[u][d][0], hi = r[u][d][1];
          const i16x8 x = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          fr = __builtin_bit_cast(bf16x8, x);
        }
        o[d] = mfma32(fr, __builtin_bit_cast(bf16x8, pw[u]), o[d]);
      }
    };
    f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    [[maybe_unused]] f32x4 s_r = {0.f, 0.f, 0.f, 0.f};  // 8 bits: the RoPE part (the cache's scale enters the rest alone)
    static_for<KS>([&](auto kc) {
      constexpr int ks = decltype(kc)::value;
      if constexpr (!FP8) {
        s[ks & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[ks % KF], qf[ks], s[ks & 1], 0, 0, 0);
        if constexpr (ks + KF < KS) f[ks] = key_frag(ks + KF);
      } else if constexpr (ks < KS_C) {
        const u32x4 c = __builtin_bit_cast(u32x4, f[ks / 2]);
        s[ks & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16((ks & 1) ? widen_e4m3x8(c[2], c[3]) : widen_e4m3x8(c[0], c[1]), qf[ks], s[ks & 1], 0, 0, 0);
      } else {
        s_r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[KS_C / 2 + ks - KS_C], qf[ks], s_r, 0, 0, 0);
      }
      if constexpr (ks % 4 == 3) output_step(std::integral_constant<int, ks / 4>{});
    });
    if (!more) break;
    // value fragments of this pair, consumed in the next iteration
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const int off = (u >> 1) * TILE_BYTES + 16 * (u & 1) * 128;
        if constexpr (FP8) {
          typedef __attribute__((ext_vector_type(2))) int i32x2;
          r[u][d][0] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2*)(buf + (vbase ^ (d << 4)) + off)));
          continue;
        } else {
        r[u][d][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(buf + (vbase ^ (64 * d)) + off));
        r[u][d][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(buf + (vbase ^ (64 * d + 16)) + (off + 8 * 128)));
        }
      }
    // ---- softmax of this wave's 16 tokens x 16 rows ----
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = FP8 ? __builtin_fmaf(s[0][i] + s[1][i], c_scale, s_r[i]) : s[0][i] + s[1][i];
    if (!whole || tok + kPair > unmasked_end) {
      const int lim = pg[0] >= 0 ? vis_end : 0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (tok + 16 * tb + 4 * g4 + i >= lim) z[i] = GQLA_NEG_INF;
    }
    z_max = pair_max(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
    {
      const uint32_t u = __builtin_bit_cast(uint32_t, z_max);
      const auto x = __builtin_amdgcn_permlane16_swap(u, u, false, false);  // the other row of 16 lanes
      z_max = fmaxf(__builtin_bit_cast(float, (uint32_t)x[0]), __builtin_bit_cast(float, (uint32_t)x[1])) * a.scale_log2e;
    }
    const bool move = __builtin_amdgcn_ballot_w64(z_max > m_s + kRescaleThreshold) != 0;
    psum_last = publish(j, (m_s == GQLA_NEG_INF) ? 0.f : m_s, move);

    ring = ring + 1 == PAIRS ? 0 : ring + 1;
#pragma unroll
    for (int u = 0; u + 1 < PAIRS; ++u) {
      pg[u] = pg[u + 1];
      slot[u] = slot[u + 1];
    }
    pg[PAIRS - 1] = -1;
    slot[PAIRS - 1] = look_slot;
    if (lookup) {
      if (table_row) asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(raw) : : "memory");
      pg[PAIRS - 1] = checked(raw);
    }
  }

  // denominators: the four lanes of a row, then its four waves, in the same order for all
  l_run = pair_sum(l_run);
  {
    const uint32_t u = __builtin_bit_cast(uint32_t, l_run);
    const auto x = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    l_run = __builtin_bit_cast(float, (uint32_t)x[0]) + __builtin_bit_cast(float, (uint32_t)x[1]);
  }
  __syncthreads();  // (the maxima of a move in the last iteration have been read)
  if (g4 == 0) mex[tb * 32 + 16 * rh + n16] = l_run;
  __syncthreads();
  const float l_tot = mex[n] + mex[32 + n] + mex[64 + n] + mex[96 + n];
  const int row = rho0 + n;
  if (row >= a.M) return;
  const float inv = (l_tot > 0.f ? 1.f / l_tot : 0.f) * (FP8 ? c_scale : 1.f);
  // dims 4 h .. 4 h + 3 of vector 4 (2 wave + d) + q of the row: consecutive rows in consecutive lanes
  __bf16* po = (__bf16*)a.part_o + part_vec_index(chunk, row, a.M, RKV / 8, 0) * 8 + 4 * h;
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(u32x2*)(po + (FP8 ? 8 * wave + 2 * (d + 2 * (q >> 1)) + (q & 1) : (wave * 2 + d) * 4 + q) * (32 * 8)) =
          u32x2{pack_bf16(o[d][4 * q] * inv, o[d][4 * q + 1] * inv), pack_bf16(o[d][4 * q + 2] * inv, o[d][4 * q + 3] * inv)};
  if (h == 0 && wave == 0)
    a.part_lse[(int64_t)chunk * a.M + row] = l_tot > 0.f ? (m_o + fast_log2(l_tot)) * kLn2 : GQLA_NEG_INF;
}

// every accumulator of row block rb (tiles 4*dtl + rb, dtl = 0..3) of this lane times alpha
__device__ __forceinline__ void acc_scale_rb(int rb, float alpha) {
  float t0, t1;
  switch (rb) {
#define X(R)                                                                                                             \
  case R:                                                                                                                \
    asm volatile(".irp gqla_t, " #R ", 4+" #R ", 8+" #R ", 12+" #R "\n.set gqla_i, 0\n.rept 8\n"                          \
                 "\tv_accvgpr_read_b32 %0, a[(\\gqla_t)*16+gqla_i]\n\tv_accvgpr_read_b32 %1, a[(\\gqla_t)*16+gqla_i+1]\n"  \
                 "\tv_mul_f32 %0, %0, %2\n\tv_mul_f32 %1, %1, %2\n\ts_nop 0\n"                                              \
                 "\tv_accvgpr_write_b32 a[(\\gqla_t)*16+gqla_i], %0\n\tv_accvgpr_write_b32 a[(\\gqla_t)*16+gqla_i+1], %1\n" \
                 ".set gqla_i, gqla_i+2\n.endr\n.endr"                                                                     \
                 : "=&v"(t0), "=&v"(t1)                                                                                    \
                 : "v"(alpha));                                                                                            \
    break;
    X(0) X(1) X(2) X(3)
#undef X
  }
}

// More than 32 query rows per sequence and enough chunks to fill the chip: one workgroup of 4 waves per (chunk, block of
// 128 rows), and the two contractions are dealt over the waves in two different ways.
//   S^T: wave w owns row block w (rows 32w..32w+31) against the whole tile, queries in registers.
//   O^T: wave w owns latent dims 128w..128w+127 of ALL four row blocks: accumulator tile 4*d + rb holds dims
//        128w + 32d.. of row block rb.  Each transposed value fragment read from LDS then feeds four MFMAs (one per row
//        block) instead of one, which cuts the transposed reads per tile by four; the price is that the waves trade
//        their probabilities: wave rb writes its two P^T operand fragments (1 KB each, already in B-operand order) into a
//        double-buffered 8 KB exchange behind the tile ring, and every wave reads all eight.
// The loop is software-pipelined so that nothing but MFMAs (and what fits in their shadows) is on a wave's critical path
// (measured on this chip: behind each 32-cycle MFMA a wave issues four simple vector-ALU instructions or two
// exponentials for free, an LDS read costs about 5 cycles, an LDS-DMA instruction 10-20):
//   iteration i:   S^T(i)          36 MFMAs; in their gaps: the key-fragment reads (a ring of 8 fragments, 8 MFMAs ahead),
//                                  the 9 LDS-DMA instructions that stage tile i+2, and the first operands of the next phase
//                  O^T += (i-1)    32 MFMAs; in their gaps: the softmax of tile i (maximum, exponentials, packing) and the
//                                  write of its probabilities
//                  one workgroup barrier, then the first key fragments of tile i+1 are requested
// The barrier is the only one of the tile: each wave waits for its share of tile i+1's staging before it arrives, so
// passing it means "tile i+1 has landed for everyone", "the probabilities of tile i are visible" and "everyone is done
// with tile i-1", whose buffer the staging of tile i+3 (issued in the next iteration's gaps) overwrites.  What must not stand
// between the barrier and the next tile's first MFMA is pinned in front of it (the sum of the probabilities, 16 dependent
// additions, and the addresses of the next staging: the compiler had moved both behind the barrier; kernel 134 -> 130 us at
// 64 sequences x 8192 tokens x 128 rows).
// The softmax state (reference maximum, denominator) of a row lives in the wave that owns its row block.  A move of the
// reference maximum of rows that already have output (rare: the maximum must grow by more than 2^8) has to rescale
// accumulators in all four waves: the owning wave announces it in the sign bit of its first probability (probabilities
// are never negative), all waves see the same bits, and together they take a slow path that passes the factors through
// the idle half of the exchange.
// FP8: the cache holds E4M3 codes of c_kv with one scale, and k_R in 16 bits.  The paper names quantised caches as complementary
// and fixes no format (Sec. 2; Sec. 5.1, item (i)); the page format is this library's (gqla.h): code rows [P][r_kv] back to
// back, then k_R [P][d_r] -- r_kv + 2 d_r bytes per token; the decode is the MQA-absorb equation on value(code) * scale.  The same MFMAs on
// the same bf16 operands: codes and k_R are staged as they are (20 KB a tile instead of 36) and widened in registers
// (v_cvt_scalef32_pk_bf16_fp8, exact) -- the keys by every wave for itself, 128 conversions a tile, in the gaps of S^T; the
// values once, by the wave that owns their dims, out of transposed 8-bit reads.  The scale enters the content part of the
// logits (the RoPE part has accumulators of its own and is added in the softmax) and the chunk's output.  8-bit MFMAs on the
// codes, with queries and probabilities split in two, would save the widening and take as long; they add 64 products in
// about 15 bits below the largest (measured: 1.6e-5 of the logits' norm, 2.6e-8 with these), so they are not used.
// Against one wave per 32 rows that widened a quarter of each tile on its way into a bf16 buffer (two buffers, softmax in the
// open): 64 ragged sequences of 3000 to 12000 tokens x 128 rows 172 -> 146 us; 64 x 4096 x 64 rows 89 -> 84 us a step.
// 16 bits: whole blocks of 128 rows (the launcher sends other row counts to the kernel above).  8 bits: any row count above
// 32; rows beyond the last read that one's queries, see no token and store nothing.  There is no branch per row block, and
// the register budget is exact -- the compiler must never run out of ordinary
// registers here, or it would park values in accumulation registers, which hold O^T behind its back (the MFMA
// statements name their accumulators as clobbered, and the build checks the generated code for both).
template <int RKV, int DR, bool FP8>
__global__ void __launch_bounds__(256) decode_absorb_shared_bf16_kernel(DecodeArgs a, int row_blocks, float c_scale) {
  constexpr int W = RKV + DR;
  constexpr int CB = FP8 ? 1 : 2;              // bytes per element of c_kv
  constexpr int NPC = RKV * CB / 128;          // panels of c_kv; k_R is one more
  constexpr int NP = NPC + 1;
  constexpr int PANEL = kTile * 128;
  constexpr int KS = W / 16;
  constexpr int KS_R = DR / 16;                // k-steps over the RoPE key
  constexpr int DT = RKV / 32;
  constexpr int TILE_BYTES = NP * PANEL;
  constexpr int EX = kSlots * TILE_BYTES;  // exchange: [2 buffers][4 row blocks][2 k-steps][64 lanes][16 bytes]
  constexpr int KR = 4;                    // key fragments in flight (more do not fit the 256 ordinary registers)
  static_assert(DT == 16, "O^T fills the 256 accumulation registers exactly: 4 dim tiles x 4 row blocks per wave");
  static_assert(DR == 64 && RKV % 128 == 0, "latent row must be a whole number of 128-byte panels, one or two per wave and one of k_R");
  static_assert(KS == 36 && NP <= 9, "the gap schedule below is written for 36 key k-steps and up to 9 staging instructions");
  extern __shared__ __attribute__((aligned(16))) char smem[];

  int chunk, rbk;
  {
    const int id = blockIdx.x;
    const int grp = id / (8 * row_blocks), rem = id % (8 * row_blocks);
    rbk = rem / 8;
    chunk = grp * 8 + rem % 8;
  }
  if (chunk >= a.n_chunks) return;  // whole workgroup leaves together
#ifdef GQLA_PHASE_TIMING
  const long long t_entry_ = __builtin_readcyclecounter();
  long long ph_[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  long long last_ = t_entry_;
#endif
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;
  const ChunkEntry ce = a.chunks[chunk];

  const int row0 = rbk * kRowsPerBlock;
  const int rho = row0 + wave * 32 + n;  // row = t * h_q + i
  const bool row_ok = !FP8 || rho < a.M;  // (16 bits: always a real row)
  const int t = rho / a.h_q;
  const int vis_end = row_ok ? min(ce.tok_end, ce.L - a.s_q + t + 1) : 0;
  const int unmasked_end = min(ce.tok_end, ce.L - a.s_q + 1);

  const int P = a.cache.page_size;
  const char* pool = (const char*)a.cache.pool;
  const int32_t* table_row = a.cache.page_table ? a.cache.page_table + (int64_t)ce.b * a.cache.max_pages : nullptr;
  auto checked = [&](int32_t pg) -> int32_t { return ((uint32_t)pg < (uint32_t)a.cache.num_pages) ? pg : -1; };
  // first row of a tile, and (8 bits, where k_R has a plane of its own behind the codes of the page) its first k_R row; an
  // id outside the pool falls back to page 0
  constexpr int ROWB = FP8 ? RKV : 2 * W;
  const int64_t page_bytes = (int64_t)P * (RKV * CB + DR * 2);
  auto tile_src = [&](int32_t pg, int slot) -> const char* { return pool + (int64_t)(pg >= 0 ? pg : 0) * page_bytes + (int64_t)slot * ROWB; };
  auto kr_src = [&](int32_t pg, int slot) -> const char* {
    return FP8 ? pool + (int64_t)(pg >= 0 ? pg : 0) * page_bytes + (int64_t)P * RKV + (int64_t)slot * (DR * 2) : nullptr;
  };

  // per-lane LDS offsets inside a tile (panel layout of gqla_lds.h): key fragment of k-step ks = 4*a4 + b at
  // kbase[b] + a4*PANEL; transposed value reads at vbase + compile-time offsets (this wave's dims: panels 2w, 2w+1)
  uint32_t kbase[4], vbase;
  {
#pragma unroll
    for (int b = 0; b < 4; ++b) kbase[b] = n * 128 + (((2 * b + h) ^ lds_swz(n)) << 4);
    const int i16 = lane & 15, e = i16 >> 2, q = i16 & 3, g1 = (lane >> 4) & 1;
    if constexpr (FP8) {
      // Transposed 8-bit reads: 16 lanes address 8 tokens x 16 dims (lane 2 k + p: 8 bytes of token k) and each receives
      // the 8 tokens of one dim.  Token k of k-step u is row 16 u + 8 (k / 4) + 4 h + k % 4, the order in which a lane of
      // S^T holds them.  The second group of 16 lanes takes the dims two chunks further on (not one), so that a half-wave
      // meets every bank once; dim tile d of this wave is chunks vchunk(d), vchunk(d) + 2 of panel `wave`.
      const int k = i16 >> 1, row = 8 * (k >> 2) + 4 * h + (k & 3);
      vbase = row * 128 + (((2 * g1) ^ lds_swz(row)) << 4) + (i16 & 1) * 8 + wave * PANEL;
    } else {
      vbase = (4 * h + e) * 128 + (((2 * g1 + (q >> 1)) ^ lds_swz(4 * h + e)) << 4) + (q & 1) * 8;
      vbase += wave * 2 * PANEL;
    }
  }
  const uint32_t stage_off = stage_lane_offset<kTile, NP, 4, ROWB>(wave, lane);
  const uint32_t kr_off = FP8 ? stage_lane_offset<kTile, 1, 4, DR * 2>(wave, lane) : 0;
  // request u (0 .. NP - 1) of this wave's share of a tile
  auto stage_step = [&](char* dst, const char* src, const char* kr, int u) __attribute__((always_inline)) {
    if (FP8 && u == NPC) stage_panels_step<kTile, 1, 4, DR * 2, true>(dst + NPC * PANEL, kr, wave, kr_off, 0);
    else stage_panels_step<kTile, NP, 4, ROWB, true>(dst, src, wave, stage_off, u);
  };
  auto stage_tile = [&](int slot, int32_t pg, int row) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NP; ++u) stage_step(smem + slot * TILE_BYTES, tile_src(pg, row), kr_src(pg, row), u);
  };

  GQLA_STAMP(4);
  float m_ref = GQLA_NEG_INF, l_run = 0.f;

  // the queries are requested first: their addresses need only the chunk entry, and they are the bulk of what a
  // workgroup waits for before its first MFMA; the page ids (a dependent scalar load) arrive in their shadow
  bf16x8 qf[KS];
  {
    const int64_t qrow = (int64_t)ce.b * a.M + (FP8 ? min(rho, a.M - 1) : rho);
    const __bf16* ph = (const __bf16*)a.q_a + qrow * RKV + h * 8 * (FP8 ? 2 : 1);
    const __bf16* pr = (const __bf16*)a.q_r + qrow * DR + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      // 8 bits: a 16-byte vector of codes is a lane's share of two k-steps, dims 32 (ks / 2) + 16 h + 8 (ks % 2) + 0..7
      const int dim = FP8 ? 32 * (ks >> 1) + 8 * (ks & 1) : 16 * ks;
      qf[ks] = *(const bf16x8*)(ks < RKV / 16 ? ph + dim : pr + (ks - RKV / 16) * 16);
    }
  }

  const int n_tiles = (ce.tok_end - ce.tok_begin + kTile - 1) / kTile;
  // page ids of tiles it .. it+3; iteration `it` stages tile it+2 (the first three are staged up front), the table entry
  // of tile it+4 travels through the scalar cache meanwhile
  int32_t pg0, pg1, pg2, pg3;
  {
    const int p_last = (ce.tok_end - 1) / P;
    int32_t raw[4];
    if (table_row) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int p = __builtin_amdgcn_readfirstlane(min(ce.tok_begin / P + (k * kTile) / P, p_last));
        asm volatile("s_load_dword %0, %1, 0x0" : "=s"(raw[k]) : "s"(table_row + p) : "memory");
      }
      asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(raw[0]), "+s"(raw[1]), "+s"(raw[2]), "+s"(raw[3]) : : "memory");
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) raw[k] = ce.b * a.cache.max_pages + min(ce.tok_begin / P + (k * kTile) / P, p_last);
    }
    pg0 = checked(raw[0]);
    pg1 = n_tiles > 1 ? checked(raw[1]) : -1;
    pg2 = n_tiles > 2 ? checked(raw[2]) : -1;
    pg3 = n_tiles > 3 ? checked(raw[3]) : -1;
  }
  GQLA_STAMP(5);
  int32_t pg_raw = 0;
  const char *next_g = pool, *next_kr = pool;  // first rows of the tile the next iteration stages (set when the window moves)
  const int p_first = ce.tok_begin / P;
  int st_slot = (3 * kTile) % P;                                     // slot of tile it+3 in its page
  int lk_slot = (4 * kTile) % P, lk_p = p_first + (4 * kTile) / P;   // tile it+4

  // Start-up: all workgroups begin at once, on cold address translations, and each walks a chain of dependent first
  // touches (chunk entry, page table, queries and tile 0): about 15 k cycles pass before the first MFMA, 7 % of the
  // kernel at the canonical shape, the same whether the queries (147 KB per workgroup, 38 MB over the chip) are loaded
  // as fragments or staged through LDS in whole lines, and the same with the chunks of a sequence on one die -- it is
  // neither the shape of the loads nor their volume.  The queries go first (above), then tile 0; tiles 1 and 2 are
  // requested once those have landed, while tile 0 is being multiplied.
  stage_tile(0, pg0, 0);
  acc_zero();  // 256 register writes, in the shadow of the requests above
  // The query loads complete here, before the loop (the compiler's wait for them also covers the request for tile 0
  // above); inside the loop only hand-counted waits remain.
#pragma unroll
  for (int k = 0; k < KS; k += 4) asm volatile("" : "+v"(qf[k]), "+v"(qf[k + 1]), "+v"(qf[k + 2]), "+v"(qf[k + 3]));

  // rows of a tile past the chunk end (or a whole tile behind an out-of-pool page id) hold whatever the page holds:
  // zeroed in LDS by the whole workgroup before anyone reads them, so that 0 * v stays 0
  auto zero_rows = [&](int slot, int valid) {
    constexpr int kChunks = NP * 8;
    int tid = threadIdx.x, zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero), "+v"(tid));  // formed here: nothing of this rare path is kept in registers across the loop
    const u32x4 zeros = {(uint32_t)zero, (uint32_t)zero, (uint32_t)zero, (uint32_t)zero};
    for (int idx = tid; idx < (kTile - valid) * kChunks; idx += 256) {
      const int r = valid + idx / kChunks, c = idx % kChunks;
      *(u32x4*)(smem + slot * TILE_BYTES + (c >> 3) * PANEL + r * 128 + (c & 7) * 16) = zeros;
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __syncthreads();
  };
  GQLA_STAMP(6);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();  // the first tiles have landed for every wave
  GQLA_STAMP(7);
  if (n_tiles > 1) stage_tile(1, pg1, kTile % P);
  if (n_tiles > 2) stage_tile(2, pg2, (2 * kTile) % P);
  {
    const int valid0 = pg0 >= 0 ? min(kTile, ce.tok_end - ce.tok_begin) : 0;
    if (valid0 < kTile) zero_rows(0, valid0);
  }

  // operands that live across the phases of the pipeline
  bf16x8 kf[KR];        // key fragments, requested KR MFMAs ahead of their use (8 bits: of k_R)
  [[maybe_unused]] u32x4 kraw[3];        // 8 bits: codes of the keys, two k-steps each, and ...
  [[maybe_unused]] bf16x8 kw[3];         // ... widened fragments, ready two MFMAs ahead (first k_R as it is, with kf[0])
  bf16x8 pfr[4][2];     // probabilities of the tile whose O^T update is running: [row block][k-step]
  i16x4 vr[2][4][2];    // its value fragments [k-step][dim tile][read]
  [[maybe_unused]] u32x2 vraw[2][4];     // 8 bits: codes of its values, and ...
  [[maybe_unused]] u32x4 vw[2];          // ... widened fragments of this dim tile and the next
  f32x16 s;             // raw logits of the tile whose softmax is running
  [[maybe_unused]] f32x16 s_r;           // 8 bits: their RoPE part (the cache's scale enters s alone)
  float alpha_prev = 1.f;   // factor of this wave's rows announced with the probabilities of the previous tile
  bool announce_prev = false;

  auto load_k = [&](const char* tb, int ks) __attribute__((always_inline)) {  // key fragment of k-step ks of the tile at tb
    kf[ks % KR] = *(const bf16x8*)(tb + kbase[ks & 3] + (FP8 ? NPC : ks >> 2) * PANEL);
  };
  auto load_codes = [&](const char* tb, int i) __attribute__((always_inline)) {  // of k-steps 2 i, 2 i + 1
    kraw[i % 3] = *(const u32x4*)(tb + kbase[i & 3] + (i >> 2) * PANEL);
  };
  auto load_kr = [&](const char* tb, int ks) __attribute__((always_inline)) { (ks < 3 ? kw[ks] : kf[0]) = *(const bf16x8*)(tb + kbase[ks] + NPC * PANEL); };
  auto first_keys = [&](const char* tb) __attribute__((always_inline)) {
    if constexpr (FP8) {  // the first two; the rest follow at the start of the tile
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) load_kr(tb, ks);
    } else {
#pragma unroll
      for (int ks = 0; ks < KR; ++ks) load_k(tb, ks);
    }
  };
  auto widen_half = [&](u32x4& w, const u32x2& c, int half) __attribute__((always_inline)) {  // codes 4 half .. 4 half + 3
    w[2 * half] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[half], 1.0f, false));
    w[2 * half + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c[half], 1.0f, true));
  };
  constexpr auto vchunk = [](int d) constexpr { return (d & 1) + 4 * (d >> 1); };
  auto load_v = [&](const char* tb, int u, int d) __attribute__((always_inline)) {
    if constexpr (FP8) {
      typedef __attribute__((ext_vector_type(2))) int i32x2;
      const char* p = tb + (vbase ^ (vchunk(d) << 4)) + 16 * u * 128;
      vraw[u][d] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2*)p));
      return;
    }
    const int off = (d >> 1) * PANEL + (16 * u) * 128;
    vr[u][d][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(tb + (vbase ^ (64 * (d & 1))) + off));
    vr[u][d][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(tb + (vbase ^ (64 * (d & 1) + 16)) + (off + 8 * 128)));
  };
  auto load_p = [&](const char* exr, int rb, int u) __attribute__((always_inline)) { pfr[rb][u] = *(const bf16x8*)(exr + (rb * 2 + u) * 1024); };

  first_keys(smem);

  // Iterations 0 .. n_tiles: iteration it computes S^T of tile it (HAS_S: it < n_tiles) and updates O^T with tile it-1
  // (HAS_PV: it > 0); STAGE: tile it+2 exists and is staged in this iteration (tiles 0..2 were staged up front).  The
  // three flags are compile-time so that the steady-state body has no branch per gap.
  auto iteration = [&](int it, auto HAS_S_T, auto HAS_PV_T, auto STAGE_T) __attribute__((always_inline)) {
    constexpr bool HAS_S = decltype(HAS_S_T)::value, HAS_PV = decltype(HAS_PV_T)::value, STAGE = decltype(STAGE_T)::value;
    const int tok = ce.tok_begin + it * kTile;
    const char* buf = smem + (it & (kSlots - 1)) * TILE_BYTES;                 // tile it
    const char* pbuf = smem + ((it + kSlots - 1) & (kSlots - 1)) * TILE_BYTES;  // tile it-1
    const char* exr = smem + EX + ((it + 1) & 1) * 8192 + lane * 16;           // probabilities of tile it-1
    char* exw = smem + EX + (it & 1) * 8192;                                   // probabilities of tile it
    char* next_buf = smem + ((it + 2) & (kSlots - 1)) * TILE_BYTES;
    const bool lookup = it + 4 < n_tiles;
    const bool new_page = lookup && lk_slot == 0;
    if (new_page && table_row)  // scalar load, consumed at the end of the iteration (its wait is written out there)
      asm volatile("s_load_dword %0, %1, 0x0" : "=s"(pg_raw) : "s"(table_row + lk_p) : "memory");
    const bool tile_ok = pg0 >= 0;
    const int lk_p_prev = lk_p;
    // Tile it+1 becomes current: the window of page ids moves, and the source of the tile that the next iteration
    // stages (tile it+3) is formed.  Scalar work; it runs in the shadow of the first MFMA of phase 2.
    auto move_window = [&]() __attribute__((always_inline)) {
      pg0 = pg1;
      pg1 = pg2;
      pg2 = pg3;  // pg3 (tile it+4) is the same page unless a new one was looked up; set behind the barrier
      next_g = tile_src(pg2, st_slot);
      if (FP8) next_kr = kr_src(pg2, st_slot);
      st_slot = lk_slot;
      lk_slot += kTile;
      if (lk_slot == P) {
        lk_slot = 0;
        ++lk_p;
      }
      // (here and not behind the tile's barrier, where the compiler would move it all, in front of the next tile's first MFMA)
      asm volatile("" : "+s"(next_g), "+s"(st_slot), "+s"(lk_slot), "+s"(lk_p));
      if (FP8) asm volatile("" : "+s"(next_kr));
    };

    // ---------------- phase 1: S^T(it), staging of tile it+2, first operands of phase 2 ----------------
    if constexpr (HAS_S) {
      if constexpr (FP8) {  // (not ahead of the end of the last iteration: more would be kept across it than there are registers)
        load_codes(buf, 0);
        load_kr(buf, 2);
        load_kr(buf, 3);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (FP8)
      static_for<KS>([&](auto GI) __attribute__((always_inline)) {
        constexpr int g = decltype(GI)::value, ks = g - KS_R;  // the RoPE k-steps first: the first codes are widened behind them
        if (g == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s_r) : "v"(kw[0]), "v"(qf[KS - KS_R]));
        else if (g < 3) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s_r) : "v"(kw[g % 3]), "v"(qf[KS - KS_R + g % 3]));
        else if (g == 3) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s_r) : "v"(kf[0]), "v"(qf[KS - 1]));
        else if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(kw[0]), "v"(qf[0]));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(kw[ks < 0 ? 0 : ks % 3]), "v"(qf[ks < 0 ? 0 : ks]));
        __builtin_amdgcn_sched_barrier(0);
        if (g < 2) load_codes(buf, g + 1);
        // Widened two MFMAs ahead of their use (the matrix pipeline does not wait for a vector-ALU result by itself), 3, 3 and 6
        // conversions in turn: up to three cost nothing behind an MFMA, four to six cost the same six cycles.
        constexpr int c0 = g < 2 ? 0 : 4 * (g - 2) + (g % 3 == 0 ? 2 : g % 3 == 1 ? 1 : 0), c1 = g < 2 ? 0 : 4 * (g - 1) + (g % 3 == 2 ? 2 : g % 3 == 0 ? 1 : 0);
        static_for<6>([&](auto CI) __attribute__((always_inline)) {
          constexpr int c = c0 + decltype(CI)::value;  // conversion: codes 2 (c % 4), .. + 1 of k-step c / 4
          if constexpr (c < c1 && c < RKV / 4) {
            const uint32_t w = kraw[(c >> 3) % 3][(c >> 1) & 3];
            const uint32_t r = __builtin_bit_cast(uint32_t, (c & 1) ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true)
                                                                    : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false));
            u32x4 x = __builtin_bit_cast(u32x4, kw[(c >> 2) % 3]);
            x[c & 3] = r;
            kw[(c >> 2) % 3] = __builtin_bit_cast(bf16x8, x);
            if constexpr (c % 8 == 7 && (c >> 3) + 3 < RKV / 32) load_codes(buf, (c >> 3) + 3);
          }
        });
        if (STAGE && g % 6 == 4 && g / 6 < NP) stage_step(next_buf, next_g, next_kr, g / 6);
        if (HAS_PV) {  // operands of the first k-step of the O^T update, in the last gaps
          if (g >= 26 && g < 30) load_v(pbuf, 0, g - 26);
          if (g >= 30 && g < 34) load_p(exr, g - 30, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      else
      static_for<KS>([&](auto KSI) __attribute__((always_inline)) {
        constexpr int ks = decltype(KSI)::value;
        if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(kf[0]), "v"(qf[0]));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(kf[ks % KR]), "v"(qf[ks]));
        __builtin_amdgcn_sched_barrier(0);
        if (ks + KR < KS) load_k(buf, ks + KR);
        if (STAGE && ks % 3 == 1 && ks / 3 < NP) stage_step(next_buf, next_g, next_kr, ks / 3);
        if (HAS_PV) {  // operands of the first k-step of the O^T update, in the last gaps
          if (ks >= 28 && ks < 32) load_p(exr, ks - 28, 0);
          if (ks >= 32) load_v(pbuf, 0, ks - 32);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {  // the last iteration: only the O^T update of the last tile is left
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) load_p(exr, rb, 0);
#pragma unroll
      for (int d = 0; d < 4; ++d) load_v(pbuf, 0, d);
    }
    GQLA_STAMP(0);

    // ---------------- phase 2: O^T += tile it-1, softmax of tile it in the gaps ----------------
    if (HAS_PV) {
      // announced moves of the reference maximum (uniform over the workgroup: every wave sees the same bits)
      uint32_t flags = 0;
#pragma unroll
      for (int rb = 0; rb < 4; ++rb)
        flags |= __builtin_bit_cast(u32x4, pfr[rb][0])[0];
      if (__builtin_amdgcn_readfirstlane(flags & 0x8000u) != 0) {
        // the factors travel through the idle half of the exchange (no probabilities of tile it are written before the
        // second barrier below)
        float* al = (float*)exw;
        int n = lane;  // (formed here, as in zero_rows)
        asm volatile("v_and_b32 %0, 31, %0" : "+v"(n));
        if (announce_prev) al[wave * 32 + n] = alpha_prev;  // both half-waves hold the row's factor and write the same value
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
          u32x4 w = __builtin_bit_cast(u32x4, pfr[rb][0]);
          if (__builtin_amdgcn_readfirstlane(w[0] & 0x8000u) != 0) {
            acc_scale_rb(rb, al[rb * 32 + n]);
            w[0] &= ~0x8000u;
            pfr[rb][0] = __builtin_bit_cast(bf16x8, w);
          }
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __syncthreads();
      }
    }
    // softmax state of this iteration (pieces run in the gaps below)
    constexpr bool sm = HAS_S;
    const bool need_mask = (tok + kTile > unmasked_end) || !tile_ok || !row_ok;
    const int lim = tile_ok ? vis_end : 0;
    float tmax = 0.f, m_use = 0.f, psum = 0.f, alpha = 1.f;
    bool announce = false;
    u32x4 w0 = {0u, 0u, 0u, 0u}, w1 = {0u, 0u, 0u, 0u};
    float whole[16];
    auto add_rope = [&](int q) __attribute__((always_inline)) {  // logits 4 q .. 4 q + 3 complete
#pragma unroll
      for (int i = 4 * q; i < 4 * q + 4; ++i) whole[i] = __builtin_fmaf(s[i], c_scale, s_r[i]);
    };
    auto& x = [&]() -> auto& {  // the logits, and later the probabilities
      if constexpr (FP8) return whole;
      else return s;
    }();
    auto softmax_piece = [&](auto GI) __attribute__((always_inline)) {  // g = 0..31: position in the phase
      constexpr int g = decltype(GI)::value;
      if (g == 2) {
        // S^T is read here for the first time: three MFMAs of the O^T update have been issued since its last MFMA, which
        // has therefore retired (the matrix pipeline's result is not interlocked against vector-ALU reads)
        if (__builtin_amdgcn_ballot_w64(need_mask) != 0) {  // wave-uniform: only tiles at the chunk end, or padding rows
          // register i is token tok + 4h + 8*(i/4) + i%4: compared as a constant against one per-lane distance (formed
          // here, so that no per-register offsets are kept alive across the loop)
          int dist = lim - tok - 4 * h;
          asm volatile("" : "+v"(dist));
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (FP8) {
              s[i] = 8 * (i >> 2) + (i & 3) >= dist ? GQLA_NEG_INF : s[i];
              s_r[i] = 8 * (i >> 2) + (i & 3) >= dist ? 0.f : s_r[i];
            } else if (need_mask && 8 * (i >> 2) + (i & 3) >= dist) {
              s[i] = GQLA_NEG_INF;
            }
        }
        if (FP8) add_rope(0);
        // the row maximum of the tile: eight three-way maxima (written as instructions: the logits come out of inline
        // assembly, and the compiler would first canonicalise every one of them)
        tmax = max3(x[0], x[1], x[2]);
        tmax = max3(tmax, x[3], FP8 ? x[3] : x[4]);
      } else if (g == 3) {
        if (FP8) add_rope(1);
        tmax = FP8 ? max3(tmax, x[4], x[5]) : max3(tmax, x[5], x[6]);
        tmax = FP8 ? max3(tmax, x[6], x[7]) : max3(tmax, x[7], x[8]);
      } else if (g == 4) {
        if (FP8) add_rope(2);
        tmax = FP8 ? max3(tmax, x[8], x[9]) : max3(tmax, x[9], x[10]);
        tmax = FP8 ? max3(tmax, x[10], x[11]) : max3(tmax, x[11], x[12]);
      } else if (g == 5) {
        if (FP8) add_rope(3);
        tmax = FP8 ? max3(tmax, x[12], x[13]) : max3(tmax, x[13], x[14]);
        tmax = FP8 ? max3(tmax, x[14], x[15]) : max3(tmax, x[15], x[15]);
      } else if (g == 6) {
        tmax = pair_max(tmax) * a.scale_log2e;
        if (__builtin_amdgcn_ballot_w64(tmax > m_ref + kRescaleThreshold) != 0) {
          const float m_new = fmaxf(m_ref, tmax);
          alpha = fast_exp2(m_ref - ((m_new == GQLA_NEG_INF) ? 0.f : m_new));
          // a row whose maximum was -inf has seen no token yet: its accumulators are zero and need no factor
          announce = __builtin_amdgcn_ballot_w64(m_new != m_ref && m_ref != GQLA_NEG_INF) != 0;
          m_ref = m_new;
          l_run *= alpha;
        }
        m_use = (m_ref == GQLA_NEG_INF) ? 0.f : m_ref;
      } else if (g >= 7 && g < 23) {
        constexpr int e = g >= 7 && g < 23 ? g - 7 : 0;
        x[e] = fast_exp2(__builtin_fmaf(x[e], a.scale_log2e, -m_use));  // the probability replaces the logit
        psum += x[e];
      } else if (g >= 23 && g < 27) {
        constexpr int q = g >= 23 && g < 27 ? g - 23 : 0;
        w0[q] = pack_bf16(x[2 * q], x[2 * q + 1]);
        w1[q] = pack_bf16(x[8 + 2 * q], x[8 + 2 * q + 1]);
      } else if (g == 27) {
        l_run += psum;
        asm volatile("" : "+v"(l_run));  // (added up here, not behind the barrier)
        if (announce) w0[0] |= 0x8000u;  // sign bit of the first probability
        *(u32x4*)(exw + (wave * 2 + 0) * 1024 + lane * 16) = w0;
      } else if (g == 28) {
        *(u32x4*)(exw + (wave * 2 + 1) * 1024 + lane * 16) = w1;
      }
    };
    if (HAS_PV) {
      if constexpr (FP8) {
        widen_half(vw[0], vraw[0][0], 0);
        widen_half(vw[0], vraw[0][0], 1);
        asm volatile("s_nop 1" : "+v"(vw[0]));  // two wait states between a vector-ALU write and an MFMA that reads it
      }
      static_for<32>([&](auto GI) __attribute__((always_inline)) {
        constexpr int g = decltype(GI)::value;
        constexpr int u = g >> 4, d = (g >> 2) & 3, rb = g & 3;
        if constexpr (FP8) {
          acc_mfma(4 * d + rb, __builtin_bit_cast(bf16x8, vw[d & 1]), pfr[rb][u]);
        } else {
          const i16x4 lo = vr[u][d][0], hi = vr[u][d][1];
          const i16x8 fr = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          acc_mfma(4 * d + rb, __builtin_bit_cast(bf16x8, fr), pfr[rb][u]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (g == 0 && HAS_S) move_window();
        if (g >= 8 && g < 12) load_p(exr, g - 8, 1);  // second k-step's operands, as the first k-step's registers free up
        if constexpr (FP8) {
          if (g >= 4 && g < 8) load_v(pbuf, 1, g - 4);
          if constexpr (rb < 2 && g < 28) widen_half(vw[(d + 1) & 1], vraw[(g + 4) >> 4][(d + 1) & 3], rb);  // two MFMAs and more ahead of its use
        } else {
          if (g >= 12 && g < 16) load_v(pbuf, 1, g - 12);
        }
        if (sm) softmax_piece(GI);
        __builtin_amdgcn_sched_barrier(0);
      });
    } else {  // the first iteration: there is no O^T update yet to hide the softmax behind
      move_window();
      asm volatile("s_nop 15\n\ts_nop 7" : "+v"(s));  // the matrix pipeline's result is not interlocked against vector-ALU reads
      static_for<32>([&](auto GI) __attribute__((always_inline)) { softmax_piece(GI); });
    }
    alpha_prev = alpha;
    announce_prev = announce;
    GQLA_STAMP(1);

    // ---------------- the tile's barrier ----------------
    if (HAS_S) {
      if (FP8 ? STAGE || it + 2 < n_tiles : it + 2 < n_tiles) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NP) : "memory");  // this wave's share of tile it+1 has landed
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the probabilities are written
      __syncthreads();
      GQLA_STAMP(2);
      if (it + 1 < n_tiles) {
        const int valid1 = pg0 >= 0 ? min(kTile, ce.tok_end - (tok + kTile)) : 0;  // (the window has moved: pg0 is tile it+1)
        if (valid1 < kTile) zero_rows((it + 1) & (kSlots - 1), valid1);  // only the chunk's last tile can have invalid rows
        first_keys(smem + ((it + 1) & (kSlots - 1)) * TILE_BYTES);
      }
      // the page of tile it+4 joins the window (the scalar load was requested at the top of the iteration; no LDS
      // operation is outstanding here, so its wait costs nothing extra)
      if (new_page && table_row) asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(pg_raw) : : "memory");
      if (new_page) pg3 = checked(table_row ? pg_raw : ce.b * a.cache.max_pages + lk_p_prev);
      if (!lookup) pg3 = -1;
    }
    GQLA_STAMP(3);
  };
  using T_ = std::true_type;
  using F_ = std::false_type;
  iteration(0, T_{}, F_{}, F_{});
  {
    int it = 1;
    if constexpr (FP8) {
      // one loop: behind the last tile the staging goes on, from page 0 into buffers that nobody reads any more (a second
      // loop without it did not fit the registers)
#pragma unroll 1
      for (; it < n_tiles; ++it) iteration(it, T_{}, T_{}, T_{});
    } else {
#pragma unroll 1
      for (; it + 2 < n_tiles; ++it) iteration(it, T_{}, T_{}, T_{});
#pragma unroll 1
      for (; it < n_tiles; ++it) iteration(it, T_{}, T_{}, F_{});
    }
  }
  iteration(n_tiles, F_{}, T_{}, F_{});
  if (FP8) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no request may outlive the workgroup's LDS

#ifdef GQLA_PHASE_TIMING
  if (threadIdx.x == 0) {
    for (int k = 0; k < 8; ++k) atomicAdd(&gqla_phase_cycles[k], (unsigned long long)ph_[k]);
    atomicAdd(&gqla_phase_cycles[15], (unsigned long long)n_tiles);
    atomicAdd(&gqla_phase_cycles[14], (unsigned long long)(__builtin_readcyclecounter() - t_entry_));
    atomicAdd(&gqla_phase_cycles[13], 1ull);
  }
#endif
  // ---- chunk partial: O^T / l as bf16 in latent space, log-sum-exp per row ----
  const float l_tot = pair_sum(l_run);
  __syncthreads();  // every wave is done with the exchange
  float* inv_l = (float*)(smem + EX);
  if (h == 0) inv_l[wave * 32 + n] = (l_tot > 0.f ? 1.f / l_tot : 0.f) * (FP8 ? c_scale : 1.f);
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __syncthreads();
  if (h == 0 && row_ok)
    a.part_lse[(int64_t)chunk * a.M + rho] = l_tot > 0.f ? (m_ref + fast_log2(l_tot)) * kLn2 : GQLA_NEG_INF;
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    const int row = row0 + rb * 32 + n;
    if (FP8 && row >= a.M) continue;
    const float inv = inv_l[rb * 32 + n];
    // dims 4 h .. 4 h + 3 of vector 16 wave + 4 d + q (8 bits: of the chunks of dim tile d) of the lane's row: 512 contiguous
    // bytes per store instruction
    __bf16* po = (__bf16*)a.part_o + part_vec_index(chunk, row, a.M, RKV / 8, 16 * wave) * 8 + 4 * h;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      float x[16];
      acc_read(4 * d + rb, rb == 0 && d == 0, x);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        u32x2 v = {pack_bf16(x[4 * q] * inv, x[4 * q + 1] * inv), pack_bf16(x[4 * q + 2] * inv, x[4 * q + 3] * inv)};
        *(u32x2*)(po + (FP8 ? 2 * (vchunk(d) + 2 * (q >> 1)) + (q & 1) : 4 * d + q) * (32 * 8)) = v;
      }
    }
  }
}

// ---- combine + latent-output projection: out = W_UV[j]^T (sum_k w_k o_hat_k)   (MQA-absorb equation, line 6) ----
// A workgroup of 8 waves takes blocks of query rows of one group j.  W_UV[j] ([r_kv][PD = 128 or 64 of the value dims], 128 or
// 64 KB) is staged in LDS once and stays there for all of them.  Per block:
//   merge     wave w merges the chunk partials of latent dims [64 w, 64 w + 64) by their log-sum-exps (online, kNB chunks in
//             flight) and writes the merged latent as four MFMA operand fragments (bf16) into a 32 KB exchange
//   project   O^T[d][row] = W^T[d][r] * Ohat^T[r][row]: wave w < PD / 32 owns value dims [32 w, 32 w + 32) over all r; the first
//             partials of everyone's next block are already requested
// A block has 32 columns: 32 rows, or rows_per_block = 8 or 4 rows times 4 or 8 slices of the chunks (column = row +
// rows_per_block * slice), so that a single sequence's long chain of partials (20 to 130 chunks) is merged by all lanes at
// once.  The projection is linear: the slices' columns, each scaled by its share of the softmax weight, are projected as
// they are and summed afterwards, when a row has 16 values per lane left instead of 64.
// What it costs is the chain first_slot -> partials -> exchange -> MFMAs and the bytes of partials and W_UV a CU pulls in; the
// staging of W_UV goes out behind the first partials, because loads complete in order and the partials are needed first.
// Measured (kernel): one sequence, 22 chunks, 128 rows: 18.2 -> 7.9 us; 64 sequences, 4 chunks each: 13.1 -> 12.0 us; 128
// ragged sequences of 256 rows, 201 MB of partials: 50.7 -> 35.5 us.  (Before: a block per workgroup, W_UV staged by each and
// ahead of the partials, the K range split over the waves and 64 KB of fp32 results summed through LDS.)
// DV: value dims per head (columns of W_UV[j], elements of an output row); a workgroup projects onto PD of them (the merge is
// repeated per slice).  PD = 64 where that still is one workgroup per unit: a unit stages half of
// W_UV (4 sequences x 8192 tokens x 128 rows 8.8 -> 8.2 us, 32 ragged x 32 rows 7.8 -> 7.2, 16 rows of a group 8.6 -> 7.8).
// The slices of a block go to ids that are equal modulo 8, i.e. to one die: read through two L2s, a block's partials also cost the
// next call's decode, which writes those lines again (4 sequences of 2000 to 4000 tokens, 3 groups x 36 rows: 27.7 -> 25.0 us a call;
// with all 128 dims in one workgroup 25.7).
// wgs: workgroups per group and slice.
template <int RKV, int DV, int PD>
__global__ void __launch_bounds__(512) combine_project_bf16_kernel(CombineArgs a, int rows_per_group, int log2_rows, int n_blocks, int wgs) {
  constexpr int KSW = RKV / 16 / 8;  // k-steps of the contraction that one wave merges
  constexpr int kNB = 4;             // chunks in flight
  static_assert(KSW == 4, "eight waves x 4 k-steps");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  char* const exch = smem + RKV * PD * 2;  // [k-step][lane][16 bytes]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, h = lane >> 5;
  constexpr int kSlices = DV / PD;
  const int wg = kSlices == 1 ? blockIdx.x : blockIdx.x / (8 * kSlices) * 8 + blockIdx.x % 8;
  if (wg >= wgs * a.g) return;  // whole workgroup (the grid is filled up to eights)
  const int j = wg / wgs, first = wg % wgs;
  const int col0 = kSlices == 1 ? 0 : blockIdx.x / 8 % kSlices * PD;  // first value dim of this workgroup
  const int rows = 1 << log2_rows, slice = n >> log2_rows, slices = 32 >> log2_rows;
  const int64_t chunk_stride = (int64_t)((a.M + 31) / 32) * 32 * RKV;  // elements from one chunk's partials to the next

  // this lane's row (index rho within its sequence b) and its chunks: s0 + slice, s0 + slice + slices, ... below s1
  struct Row {
    int b, rho, s0, s1, ok;
  };
  auto row_of = [&](int blk) __attribute__((always_inline)) {
    Row r;
    const int x = blk * rows + (n & (rows - 1));  // row of group j: (b * s_q + t) * G + head-in-group
    r.ok = x < rows_per_group;
    const int xc = r.ok ? x : 0;                  // a lane without a row computes on row 0 and stores nothing
    r.b = xc / (a.s_q * a.G);
    r.rho = (xc / a.G) % a.s_q * a.h_q + j * a.G + xc % a.G;
    r.s0 = a.first_slot[r.b];
    r.s1 = a.first_slot[r.b + 1];
    return r;
  };
  float l[kNB];
  u32x4 v[kNB][KSW];
  auto fetch = [&](const Row& r, int k, int chunk) __attribute__((always_inline)) {
    const int sc = min(chunk, r.s1 - 1);          // a chunk beyond the range is loaded again and given weight 0
    l[k] = a.part_lse[(int64_t)sc * a.M + r.rho];
    const __bf16* po = (const __bf16*)a.part_o + part_vec_index(0, r.rho, a.M, RKV / 8, 2 * KSW * wave + h) * 8 + sc * chunk_stride;
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks) v[k][ks] = *(const u32x4*)(po + ks * (2 * 32 * 8));
  };

  Row row = row_of(first);
#pragma unroll
  for (int k = 0; k < kNB; ++k) fetch(row, k, row.s0 + slice + k * slices);
  {
    // (the builtin, not the assembly of gqla_lds.h: the compiler then counts these requests and waits for the partials
    // without them)
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t off = stage_lane_offset<RKV, PD / 64, 8, DV * 2>(wave, lane);
    const char* w = (const char*)a.w_uv + ((int64_t)j * RKV * DV + col0) * 2;
#pragma unroll
    for (int u = 0; u < PD / 8; ++u)  // panel u / 8, rows 64 (u % 8) + 8 wave + 0..7
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)(w + off + (64 * (u & 7)) * (DV * 2) + (u >> 3) * 128),
                                       (lds_ptr_t)(smem + (u >> 3) * (RKV * 128) + (wave + 8 * (u & 7)) * 1024), 16, 0, 0);
  }
  // transposed fragments of W_UV (tr_natural_frag of gqla_lds.h for tile `wave`: its parity picks the lane offsets)
  const TrNatural tr = make_tr_natural(lane);
  const char* const tr0 = smem + (wave >> 1) * (RKV * 128) + (wave & 1 ? tr.base[0][1] : tr.base[0][0]);
  const char* const tr1 = smem + (wave >> 1) * (RKV * 128) + (wave & 1 ? tr.base[1][1] : tr.base[1][0]);
  auto w_frag = [&](int ks) __attribute__((always_inline)) -> bf16x8 {
    const i16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(tr0 + ks * 2048));
    const i16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(tr1 + ks * 2048));
    const i16x8 r = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
    return __builtin_bit_cast(bf16x8, r);
  };
  bool staged = false;

  for (int blk = first; blk < n_blocks; blk += wgs) {
    Row next = row;
    if (blk + wgs < n_blocks) next = row_of(blk + wgs);  // (its chunk range arrives behind the merge)
    float m = GQLA_NEG_INF, den = 0.f;
    float acc[KSW][8];  // merged latent of this lane's column, dims 16 * (KSW * wave + ks) + 8 * h + 0..7
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[ks][e] = 0.f;
    auto add_batch = [&](int sb) __attribute__((always_inline)) {  // chunks sb, sb + slices, ... in the registers
      float w[kNB], m_new = m;
#pragma unroll
      for (int k = 0; k < kNB; ++k) {
        w[k] = sb + k * slices < row.s1 ? l[k] : GQLA_NEG_INF;
        m_new = fmaxf(m_new, w[k]);
      }
      const float m_use = (m_new == GQLA_NEG_INF) ? 0.f : m_new;
      const float rescale = __expf(m - m_use);  // 0 on the first batch (m = -inf), where den and acc are 0 anyway
      den *= rescale;
#pragma unroll
      for (int ks = 0; ks < KSW; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[ks][e] *= rescale;
      m = m_new;
#pragma unroll
      for (int k = 0; k < kNB; ++k) {
        const float wk = __expf(w[k] - m_use);
        den += wk;
#pragma unroll
        for (int ks = 0; ks < KSW; ++ks)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[ks][2 * e] += wk * bf16_bits_to_float(v[k][ks][e] & 0xffffu);
            acc[ks][2 * e + 1] += wk * bf16_bits_to_float(v[k][ks][e] >> 16);
          }
      }
    };
    int sb = row.s0 + slice;
    add_batch(sb);
    sb += kNB * slices;
    // (every lane walks as many batches as the longest of its wave needs)
    for (; __builtin_amdgcn_ballot_w64(sb < row.s1) != 0; sb += kNB * slices) {
#pragma unroll
      for (int k = 0; k < kNB; ++k) fetch(row, k, sb + k * slices);
      add_batch(sb);
    }
    // the slices of a row: common reference and denominator
    float m_row = m;
    for (int o = rows; o < 32; o <<= 1) m_row = fmaxf(m_row, __shfl_xor(m_row, o));
    const float scale_own = __expf(m - ((m_row == GQLA_NEG_INF) ? 0.f : m_row));
    float den_row = den * scale_own;
    for (int o = rows; o < 32; o <<= 1) den_row += __shfl_xor(den_row, o);
    const float norm = (row.ok && den_row > 0.f) ? scale_own / den_row : 0.f;
    if (blk != first) __syncthreads();  // every wave has read the previous block's exchange
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks)
      *(u32x4*)(exch + (KSW * wave + ks) * 1024 + lane * 16) =
          u32x4{pack_bf16(acc[ks][0] * norm, acc[ks][1] * norm), pack_bf16(acc[ks][2] * norm, acc[ks][3] * norm),
                pack_bf16(acc[ks][4] * norm, acc[ks][5] * norm), pack_bf16(acc[ks][6] * norm, acc[ks][7] * norm)};
    if (!staged) {
      wait_all_memory();                           // W_UV[j]: this wave's share
      staged = true;
    }
    if (blk + wgs < n_blocks) {
#pragma unroll
      for (int k = 0; k < kNB; ++k) fetch(next, k, next.s0 + slice + k * slices);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);            // lgkmcnt(0)
    __syncthreads();                               // the exchange (and, the first time, W_UV[j]) is complete
    if (wave < PD / 32) {
      f32x16 o;
#pragma unroll
      for (int i = 0; i < 16; ++i) o[i] = 0.f;
#pragma unroll
      for (int ks = 0; ks < RKV / 16; ++ks)
        o = mfma32(w_frag(ks), *(const bf16x8*)(exch + ks * 1024 + lane * 16), o);
      for (int sh = rows; sh < 32; sh <<= 1)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] += __shfl_xor(o[i], sh);
      if (row.ok && slice == 0) {
        __bf16* out = (__bf16*)a.out + ((int64_t)row.b * a.M + row.rho) * DV + col0 + wave * 32;  // this wave's dims
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *(u32x2*)(out + 8 * q + 4 * h) = u32x2{pack_bf16(o[4 * q], o[4 * q + 1]), pack_bf16(o[4 * q + 2], o[4 * q + 3])};
        if (a.lse && h == 0 && wave == 0 && col0 == 0) a.lse[(int64_t)row.b * a.M + row.rho] = m_row + __logf(den_row);
      }
    }
    row = next;
  }
}

}  // namespace

static hipError_t launch_decode_absorb_general(const DecodeArgs& a, hipStream_t s) {
  constexpr int kLds = kSlots * kTile * (512 + 64) * 2;  // tile ring
  // once per process (function-local statics are initialised under a lock); an error is reported by every call
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)decode_absorb_bf16_kernel<512, 64>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return attr;
  const int row_blocks = (a.M + kRowsPerBlock - 1) / kRowsPerBlock;
  const int chunks_padded = (a.n_chunks + 7) / 8 * 8;
  decode_absorb_bf16_kernel<512, 64><<<chunks_padded * row_blocks, 256, kLds, s>>>(a, row_blocks);
  return hipGetLastError();
}

template <bool FP8>
static hipError_t launch_decode_absorb_rows32(const DecodeArgs& a, float c_scale, hipStream_t s) {
  constexpr int kLds = (FP8 ? 6 * kTile * (512 + 64 * 2) : 4 * kTile * (512 + 64) * 2) + 2 * 4096 + 512;  // tile ring, probabilities, row maxima
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)decode_absorb_rows32_bf16_kernel<512, 64, FP8>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return attr;
  const int row_blocks = (a.M + 31) / 32;
  const int chunks_padded = (a.n_chunks + 7) / 8 * 8;
  decode_absorb_rows32_bf16_kernel<512, 64, FP8><<<chunks_padded * row_blocks, 512, kLds, s>>>(a, row_blocks, c_scale);
  return hipGetLastError();
}

template <bool FP8>
static hipError_t launch_decode_absorb_shared(const DecodeArgs& a, float c_scale, hipStream_t s) {
  constexpr int kLds = kSlots * kTile * (512 * (FP8 ? 1 : 2) + 64 * 2) + 2 * 8192;  // tile ring + the double-buffered exchange (16 bits: all 160 KB)
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)decode_absorb_shared_bf16_kernel<512, 64, FP8>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return attr;
  const int row_blocks = (a.M + kRowsPerBlock - 1) / kRowsPerBlock;
  const int chunks_padded = (a.n_chunks + 7) / 8 * 8;
  decode_absorb_shared_bf16_kernel<512, 64, FP8><<<chunks_padded * row_blocks, 256, kLds, s>>>(a, row_blocks, c_scale);
  return hipGetLastError();
}

hipError_t launch_decode_absorb_bf16(const DecodeArgs& a, hipStream_t s) {
  // At most 32 query rows, or more but few chunks (small batches): one workgroup per (chunk, 32 rows) as long as all of them
  // still run at once -- more workgroups, each with a shorter chain per tile (the tiles' re-reads hit the L2, and with so few
  // chunks the chip is nowhere near its memory rate).  Beyond one round the re-reads cost more than they give: 64 sequences
  // x 4096 tokens x 64 rows take 104 us a step that way and 92 us with the general kernel, 96 rows 139 and 97 us.
  const int chunks_padded = (a.n_chunks + 7) / 8 * 8;
  if (a.M <= 32 || chunks_padded * ((a.M + 31) / 32) <= a.num_cus) return launch_decode_absorb_rows32<false>(a, 1.f, s);
  // whole blocks of 128 rows (h_q s_q a multiple of 128): the pipelined kernel with shared probabilities; other row
  // counts above 32: one wave per 32 rows, each with its own probabilities
  return a.M % kRowsPerBlock == 0 ? launch_decode_absorb_shared<false>(a, 1.f, s) : launch_decode_absorb_general(a, s);
}

hipError_t launch_decode_absorb_fp8(const DecodeArgs& a, float c_scale, hipStream_t s) {
  // the same choice of row mapping as for the 16-bit cache; more rows: blocks of 128, the last one padded (64 rows: see the
  // kernel; padding most of a second block still wins over one wave per 32 rows: 64 ragged sequences of 3000 to 12000 tokens x 130
  // rows 343 -> 289 us, x 160 rows 342 -> 290, 128 of 300 to 900 x 144 rows 85 -> 69)
  const int chunks_padded = (a.n_chunks + 7) / 8 * 8;
  if (a.M <= 32 || chunks_padded * ((a.M + 31) / 32) <= a.num_cus) return launch_decode_absorb_rows32<true>(a, c_scale, s);
  return launch_decode_absorb_shared<true>(a, c_scale, s);
}

template <int DV, int PD>
static hipError_t launch_combine_project_dims(const CombineArgs& a, int log2_rows, int n_blocks, hipStream_t s) {
  constexpr int kLds = 512 * PD * 2 + 32 * 1024;  // W_UV[j] and the exchange (128 dims: all 160 KB)
  // once per process (function-local statics are initialised under a lock); an error is reported by every call
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)combine_project_bf16_kernel<512, DV, PD>, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  if (attr != hipSuccess) return attr;
  const int per_group = 256 / (a.g * (DV / PD));  // workgroups per group: one per compute unit, each with its share of the blocks
  const int wgs = n_blocks < per_group || per_group < 1 ? n_blocks : per_group;
  const int grid = DV == PD ? wgs * a.g : (wgs * a.g + 7) / 8 * 8 * (DV / PD);
  combine_project_bf16_kernel<512, DV, PD><<<grid, 512, kLds, s>>>(a, a.B * a.s_q * a.G, log2_rows, n_blocks, wgs);
  return hipGetLastError();
}

template <int DV>
static hipError_t launch_combine_project_dv(const CombineArgs& a, hipStream_t s) {
  const int rows_per_group = a.B * a.s_q * a.G;
  // 32 rows per block fill the MFMA tile; with fewer than half a chip's worth of such blocks, 8 or 4 rows each
  const int log2_rows = ((rows_per_group + 31) / 32) * a.g >= 128 ? 5 : (((rows_per_group + 7) / 8) * a.g >= 128 ? 3 : 2);
  const int n_blocks = (rows_per_group + (1 << log2_rows) - 1) >> log2_rows;
  // half of the value dims per workgroup where twice as many workgroups still run at once
  if (n_blocks * a.g * (DV / 64) <= 256) return launch_combine_project_dims<DV, 64>(a, log2_rows, n_blocks, s);
  return launch_combine_project_dims<DV, 128>(a, log2_rows, n_blocks, s);
}

hipError_t launch_combine_project_bf16(const CombineArgs& a, hipStream_t s) {
  return a.d_h == 256 ? launch_combine_project_dv<256>(a, s) : launch_combine_project_dv<128>(a, s);  // a.d_h: value dims here
}

}  // namespace gqla
