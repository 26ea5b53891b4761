// fp32 kernels of the GQLA library (vector ALU only, any dims that are multiples of 8).
// They serve the small fp32 configuration; the bf16 MFMA kernels live in their own files.
// The calls are small (a few thousand tokens at most), so what bounds them is the chain of dependent memory accesses of
// one workgroup, not bandwidth or arithmetic: every kernel shares its sums out over 256 threads and joins them through
// lane exchanges or LDS, and reads 16-byte vectors.
#include "gqla_device.h"

namespace gqla {

namespace {

__device__ __forceinline__ float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ float dot4(f32x4 x, f32x4 y, float acc) {
  for (int k = 0; k < 4; ++k) acc = fmaf(x[k], y[k], acc);
  return acc;
}

constexpr int kThreads = 256;
constexpr int kTile = 64;          // cached tokens per pass of the decode
constexpr int kRed = 4 * kThreads; // floats through which 256 threads join up to four sums each

// q_hat[row, i, r] = sum_d W_UK[j(i)][r][d] * q_c[row, i, d]      (MQA-absorb equation, line 1)
// Four neighbouring lanes share a row of W_UK, so that they ask for 64 consecutive bytes of it.
__global__ void __launch_bounds__(kThreads) absorb_query_f32_kernel(AbsorbQueryArgs a) {
  const int head = blockIdx.x, row = blockIdx.y;
  const int j = head / a.G, quarter = threadIdx.x & 3, nv = a.d_h / 4;
  const f32x4* q = (const f32x4*)((const float*)a.q_c + ((int64_t)row * a.h_q + head) * a.d_h);
  const f32x4* w = (const f32x4*)((const float*)a.w_uk + (int64_t)j * a.r_kv * a.d_h);
  float* out = (float*)a.q_hat + ((int64_t)row * a.h_q + head) * a.r_kv;
  for (int r = threadIdx.x >> 2; r < a.r_kv; r += kThreads / 4) {
    float acc = 0.f;
    for (int v = quarter; v < nv; v += 4) acc = dot4(w[(int64_t)r * nv + v], q[v], acc);
    acc += __shfl_xor(acc, 1);
    acc += __shfl_xor(acc, 2);
    if (quarter == 0) out[r] = acc;
  }
}

// o = W_UV[j]^T o_hat (MQA-absorb equation, line 6) by a whole workgroup: four columns and a share of the latent dims per
// thread, joined through `red`.  `o_hat` and `red` are LDS; the caller has put a barrier behind the writes of o_hat.
__device__ __forceinline__ void project_latent_f32(const float* o_hat, const float* w_uv, int r_kv, int d_v, float* red, float* out) {
  const int nv = d_v / 4, shares = kThreads / nv;
  const int share = threadIdx.x / nv, v = threadIdx.x % nv;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (share < shares) {
    const f32x4* w = (const f32x4*)w_uv + v;
#pragma unroll 4
    for (int r = share; r < r_kv; r += shares) {
      const f32x4 x = w[(int64_t)r * nv];
      for (int k = 0; k < 4; ++k) acc[k] = fmaf(x[k], o_hat[r], acc[k]);
    }
    *(f32x4*)(red + (share * nv + v) * 4) = acc;
  }
  __syncthreads();
  for (int d = threadIdx.x; d < d_v; d += kThreads) {
    float sum = 0.f;
    for (int s = 0; s < shares; ++s) sum += red[s * d_v + d];
    out[d] = sum;
  }
}

// Shared body of the two fp32 decode kernels, one workgroup per (chunk, query row).  kAbsorb: keys = [c | k_R] rows of the
// latent page, values = c.  Otherwise: keys = [K_C[j] | k_R], values = V[j] of the expanded page.  Logits: four lanes per
// token; weighted sum: as many shares of the tile's tokens as 256 threads allow, joined through LDS behind the last tile.
// (One wave per row, whose lanes fetched one token's row each and then walked the 64 tokens in turn, took 13.4 us over 64
// tokens at r_kv = 32 where this takes 5.0; both paths over 4 x 1000 tokens, 64 rows, r_kv = 128: 741 -> 92 us.)
// kFinal: every sequence is one chunk, so that there is nothing to combine and the rows of the output (projected, on the
// absorb path) are written here, with the values that a combine of one partial gives.
template <bool kAbsorb, bool kFinal>
__global__ void __launch_bounds__(kThreads) decode_f32_kernel(DecodeArgs a, CombineArgs c) {
  __shared__ float z_s[2][kTile], p_s[kThreads / 64][kTile], red[kRed], o_hat[kFinal && kAbsorb ? 512 : 1];
  __shared__ int64_t page_s[2][kTile];  // first element of the token's page, -1: the token is not seen
  const int chunk = blockIdx.x, rho = blockIdx.y;  // rho = t * h_q + i
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const ChunkEntry ce = a.chunks[chunk];
  const int t = rho / a.h_q, i = rho % a.h_q, j = i / a.G;
  const int P = a.cache.page_size;
  const int dk = kAbsorb ? a.r_kv : a.d_h;  // content part of the key
  const int dv = kAbsorb ? a.r_kv : a.d_v;  // value dims
  const f32x4* qa = (const f32x4*)((const float*)a.q_a + ((int64_t)(ce.b * a.s_q + t) * a.h_q + i) * dk);
  const f32x4* qr = (const f32x4*)((const float*)a.q_r + ((int64_t)(ce.b * a.s_q + t) * a.h_q + i) * a.d_r);
  const float* pool = (const float*)a.cache.pool;
  const int gc = a.cache.groups, W = a.r_kv + a.d_r;
  const int64_t page_elems = kAbsorb ? (int64_t)P * W : (int64_t)P * (gc * (a.d_h + a.d_v) + a.d_r);
  const int vis_end = min(ce.tok_end, ce.L - a.s_q + t + 1);

  // units of the weighted sum: four dims of a token (absorb), four tokens of a dim (GQA)
  const int units = kAbsorb ? dv / 4 : 2 * dv;
  const int shares = max(1, kThreads / units), share = units <= kThreads ? threadIdx.x / units : 0;
  const int unit = units <= kThreads ? threadIdx.x % units : threadIdx.x;

  float m_run = GQLA_NEG_INF, l_run = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};  // absorb: the unit's four dims;  GQA: units unit, unit + 256, ...

  for (int tok0 = ce.tok_begin, buf = 0; tok0 < ce.tok_end; tok0 += kTile, buf ^= 1) {
    const int x = threadIdx.x >> 2, quarter = threadIdx.x & 3, tok = tok0 + x;
    int64_t page = -1;
    float z = GQLA_NEG_INF;
    if (tok < vis_end) {
      const int32_t pg = page_of(a.cache, ce.b, tok / P);
      if (pg >= 0) page = pg * page_elems;
    }
    if (page >= 0) {
      const int slot = tok % P;
      float acc = 0.f;
      if (kAbsorb) {
        const f32x4* row = (const f32x4*)(pool + page + (int64_t)slot * W);
#pragma unroll 4
        for (int v = quarter; v < dk / 4; v += 4) acc = dot4(qa[v], row[v], acc);
        for (int v = quarter; v < a.d_r / 4; v += 4) acc = dot4(qr[v], row[dk / 4 + v], acc);
      } else {
        const f32x4* kc = (const f32x4*)(pool + page + ((int64_t)j * (dk / 8) * P + slot) * 8);
        const f32x4* kr = (const f32x4*)(pool + page + ((int64_t)gc * P * (a.d_h + a.d_v) + slot * 8));
#pragma unroll 4
        for (int v = quarter; v < dk / 4; v += 4) acc = dot4(qa[v], kc[(int64_t)(v >> 1) * P * 2 + (v & 1)], acc);
        for (int v = quarter; v < a.d_r / 4; v += 4) acc = dot4(qr[v], kr[(int64_t)(v >> 1) * P * 2 + (v & 1)], acc);
      }
      z = acc;
    }
    // every lane of the quad takes part, seen or not: the four have the same token
    z += __shfl_xor(z, 1);
    z += __shfl_xor(z, 2);
    if (quarter == 0) {
      z_s[buf][x] = page >= 0 ? z * a.scale_log2e : GQLA_NEG_INF;
      page_s[buf][x] = page;
    }
    __syncthreads();  // the other buffer is free again: everyone has left the pass before
    const float zt = z_s[buf][lane];
    const float m_new = fmaxf(m_run, wave_max(zt));
    const float m_use = (m_new == GQLA_NEG_INF) ? 0.f : m_new;
    const float alpha = fast_exp2(m_run - m_use);
    const float p = (zt == GQLA_NEG_INF) ? 0.f : fast_exp2(zt - m_use);
    l_run = l_run * alpha + wave_sum(p);
    m_run = m_new;
    o *= alpha;
    p_s[wave][lane] = p;  // read by this wave only
    __builtin_amdgcn_wave_barrier();
    if (share < shares) {
      if (kAbsorb) {
#pragma unroll 4
        for (int src = share; src < kTile; src += shares) {
          const float ps = p_s[wave][src];
          const int64_t pgs = page_s[buf][src];
          if (ps != 0.f && pgs >= 0) {
            const f32x4 v = *(const f32x4*)(pool + pgs + (int64_t)((tok0 + src) % P) * W + unit * 4);
            for (int k = 0; k < 4; ++k) o[k] = fmaf(ps, v[k], o[k]);
          }
        }
      } else {
        for (int u = 0; u < 4; ++u) {
          const int un = unit + u * kThreads;
          if (un >= units) break;
          for (int oct = share; oct < kTile / 8; oct += shares) {
            const int64_t pgs = page_s[buf][oct * 8];  // an octet lies in one page, and its first token is seen if any is
            if (pgs < 0) continue;
            const f32x4 v = *(const f32x4*)(pool + pgs + (int64_t)gc * P * a.d_h +
                                            ((int64_t)(j * (P / 8) + (tok0 + oct * 8) % P / 8) * dv) * 8 + un * 4);
            for (int k = 0; k < 4; ++k) {
              const float ps = p_s[wave][oct * 8 + (un & 1) * 4 + k];
              o[u] = ps != 0.f ? fmaf(ps, v[k], o[u]) : o[u];  // a slot that is not seen may hold anything
            }
          }
        }
      }
    }
  }
  // a row without a visible token: 0 and -inf as a partial; with nothing to combine, what a combine makes of that
  const bool any = l_run > 0.f;
  const float inv = any ? 1.f / l_run : (kFinal ? __builtin_nanf("") : 0.f);
  if (share < shares) {
    if (kAbsorb) *(f32x4*)(red + (share * units + unit) * 4) = o * inv;
    else
      for (int u = 0; u < 4; ++u) {
        const int un = unit + u * kThreads;
        if (un < units) red[(share * 2 + (un & 1)) * dv + (un >> 1)] = o[u] * inv;
      }
  }
  __syncthreads();
  const int parts = kAbsorb ? shares : 2 * shares;
  const int64_t row = kFinal ? (int64_t)ce.b * a.M + rho : (int64_t)chunk * a.M + rho;
  float* dst = kFinal ? (kAbsorb ? o_hat : (float*)c.out + row * dv) : (float*)a.part_o + row * dv;
  for (int d = threadIdx.x; d < dv; d += kThreads) {
    float sum = 0.f;
    for (int s = 0; s < parts; ++s) sum += red[s * dv + d];
    dst[d] = sum;
  }
  if (threadIdx.x == 0) {
    const float lse = any ? (m_run + fast_log2(l_run)) * kLn2 : (kFinal && kAbsorb ? __builtin_nanf("") : GQLA_NEG_INF);
    if (!kFinal) a.part_lse[row] = lse;
    else if (c.lse) c.lse[row] = lse;
  }
  if (kFinal && kAbsorb) {
    __syncthreads();
    project_latent_f32(o_hat, (const float*)c.w_uv + (int64_t)j * a.r_kv * c.d_h, a.r_kv, c.d_h, red, (float*)c.out + row * c.d_h);
  }
}

// Log-sum-exp combine of chunk partials that are already in d_h space.  32 lanes per (b, row), 4 dims per lane and
// step.  One pass over the chunks, kNB at a time so that their loads are in flight together; the running maximum
// moves as in an online softmax (three passes with one dependent load per chunk each would cost three memory
// latencies per chunk).
__global__ void __launch_bounds__(256) combine_kernel(CombineArgs a) {
  constexpr int kNB = 4;
  const int64_t row = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);  // row = b * M + rho
  if (row >= (int64_t)a.B * a.M) return;
  const int b = (int)(row / a.M), rho = (int)(row % a.M);
  const int s0 = a.first_slot[b], s1 = a.first_slot[b + 1];
  const float* po = (const float*)a.part_o + (int64_t)rho * a.d_h;
  float m = GQLA_NEG_INF, den = 0.f;
  for (int d = (threadIdx.x & 31) * 4; d < a.d_h; d += 128) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    m = GQLA_NEG_INF;
    den = 0.f;
    for (int sb = s0; sb < s1; sb += kNB) {
      float l[kNB];
      f32x4 v[kNB];
#pragma unroll
      for (int k = 0; k < kNB; ++k) {
        const int sc = min(sb + k, s1 - 1);  // clamped: a chunk beyond the range is loaded again and given weight 0
        l[k] = a.part_lse[(int64_t)sc * a.M + rho];
        v[k] = *(const f32x4*)(po + (int64_t)sc * a.M * a.d_h + d);
      }
      float m_new = m;
#pragma unroll
      for (int k = 0; k < kNB; ++k) {
        if (sb + k >= s1) l[k] = GQLA_NEG_INF;
        m_new = fmaxf(m_new, l[k]);
      }
      const float m_use = (m_new == GQLA_NEG_INF) ? 0.f : m_new;
      const float rescale = __expf(m - m_use);  // 0 on the first batch (m = -inf), where den and acc are 0 anyway
      den *= rescale;
      acc *= rescale;
      m = m_new;
#pragma unroll
      for (int k = 0; k < kNB; ++k) {
        const float w = __expf(l[k] - m_use);
        den += w;
        if (w > 0.f) acc += w * v[k];  // a chunk without visible tokens may hold anything
      }
    }
    acc *= 1.f / den;
    *(f32x4*)((float*)a.out + row * a.d_h + d) = acc;
  }
  if (a.lse && (threadIdx.x & 31) == 0) a.lse[row] = m + __logf(den);
}

// fp32 absorb path: combine latent-space partials, then o = W_UV[j]^T o_hat  (MQA-absorb equation, line 6).
// One workgroup per (row, sequence); the chunks are shared out over the threads, four dims each.
__global__ void __launch_bounds__(kThreads) combine_project_f32_kernel(CombineArgs a) {
  __shared__ float o_hat[512], red[kRed];
  const int rho = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63;
  const int i = rho % a.h_q, j = i / a.G;
  const int s0 = a.first_slot[b], s1 = a.first_slot[b + 1];
  // every wave by itself: largest lse, then the sum of the weights
  float m = GQLA_NEG_INF, den = 0.f;
  for (int s = s0 + lane; s < s1; s += 64) m = fmaxf(m, a.part_lse[(int64_t)s * a.M + rho]);
  m = wave_max(m);
  for (int s = s0 + lane; s < s1; s += 64) den += __expf(a.part_lse[(int64_t)s * a.M + rho] - m);
  den = wave_sum(den);
  const int nv = a.r_kv / 4, shares = kThreads / nv;
  const int share = threadIdx.x / nv, v = threadIdx.x % nv;
  if (share < shares) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int s = s0 + share; s < s1; s += shares) {
      const float w = __expf(a.part_lse[(int64_t)s * a.M + rho] - m);
      const f32x4 x = *(const f32x4*)((const float*)a.part_o + ((int64_t)s * a.M + rho) * a.r_kv + v * 4);
      if (w > 0.f) acc += w * x;
    }
    *(f32x4*)(red + (share * nv + v) * 4) = acc;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < a.r_kv; r += kThreads) {
    float sum = 0.f;
    for (int s = 0; s < shares; ++s) sum += red[s * a.r_kv + r];
    o_hat[r] = sum / den;
  }
  __syncthreads();
  project_latent_f32(o_hat, (const float*)a.w_uv + (int64_t)j * a.r_kv * a.d_h, a.r_kv, a.d_h, red,
                     (float*)a.out + ((int64_t)b * a.M + rho) * a.d_h);
  if (a.lse && threadIdx.x == 0) a.lse[(int64_t)b * a.M + rho] = m + __logf(den);
}

// Cache switch, fp32: one workgroup per (8 tokens of a page, sequence, 256 of the weights' columns).  A thread has four
// columns (a 16-byte vector of a weight row) times the eight tokens, so every weight that is read serves eight tokens, and
// the four waves share out r_kv and join their sums through LDS, whence results leave as 16-byte vectors.
// kTail: only the last a.tail positions of every sequence, from the same sums (the two calls give the same bits).
// (Each element by itself, two loads a product and one workgroup a page: 14 us where this takes 4.9, over 64 tokens, r_kv = 32.)
// kLoop: the grid may be smaller than the row, a workgroup takes every gridDim.x-th eight.  An instance of its own, since the
// loop holds its state across the barriers: over those 64 tokens 5.1 us with it, 5.0 without, and 0.4 us of
// the 24.6 that both decode paths and the switch take at that size.
template <bool kTail, bool kLoop>
__global__ void __launch_bounds__(kThreads) expand_f32_kernel(ExpandArgs a) {
  constexpr int kTok = 8, kRow = 72;  // kRow: 64 column vectors; padded so that the writes below spread over the banks
  __shared__ f32x4 c_s[512 * kTok / 4];             // [r][token]
  __shared__ float red[kThreads / 64][4 * kTok][kRow];
  const int P = a.latent.page_size, b = blockIdx.y;
  const int L = a.seq_lens[b], from = kTail ? max(L - a.tail, 0) : 0, end = kTail ? L : min(L, a.max_tokens);
  for (int64_t at = from / kTok * kTok + (int64_t)blockIdx.x * kTok; at < end; at += (int64_t)gridDim.x * kTok) {
    const int tok0 = (int)at;
    const int32_t pg_in = page_of(a.latent, b, tok0 / P);
    const int32_t pg_out = page_of(a.expanded, b, tok0 / P);
    if (pg_in < 0 || pg_out < 0) {  // whole workgroup
      if (kLoop) continue;
      return;
    }
    const int slot0 = tok0 % P, first = max(from - tok0, 0), valid = min(kTok, L - tok0);  // tokens first .. valid - 1 are written
    const int W = a.r_kv + a.d_r, gc = a.group_count;
    const float* in = (const float*)a.latent.pool + ((int64_t)pg_in * P + slot0) * W;
    float* out = (float*)a.expanded.pool + (int64_t)pg_out * P * (gc * (a.d_h + a.d_v) + a.d_r);
    for (int idx = threadIdx.x; idx < kTok * a.r_kv; idx += kThreads) {
      const int tok = idx / a.r_kv, r = idx % a.r_kv;
      ((float*)c_s)[r * kTok + tok] = tok < valid ? in[(int64_t)tok * W + r] : 0.f;
    }
    if (blockIdx.z == 0)
      for (int idx = first * a.d_r + threadIdx.x; idx < valid * a.d_r; idx += kThreads) {
        const int tok = idx / a.d_r, d = idx % a.d_r;
        out[(int64_t)gc * P * (a.d_h + a.d_v) + ((int64_t)(d / 8) * P + slot0 + tok) * 8 + d % 8] = in[(int64_t)tok * W + a.r_kv + d];
      }
    __syncthreads();
    const int nk = gc * a.d_h / 4, n_all = nk + gc * a.d_v / 4;  // column vectors: keys, all
    const int cv0 = blockIdx.z * 64, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cv = cv0 + lane;
    if (cv < n_all) {
      const bool is_v = cv >= nk;
      const int per = (is_v ? a.d_v : a.d_h) / 4, x = is_v ? cv - nk : cv;
      const f32x4* w = (const f32x4*)(is_v ? a.w_uv : a.w_uk) + (int64_t)(a.group_begin + x / per) * a.r_kv * per + x % per;
      f32x4 lo[4] = {}, hi[4] = {};  // [column]: tokens 0..3, 4..7
#pragma unroll 4
      for (int r = wave; r < a.r_kv; r += kThreads / 64) {
        const f32x4 wv = w[(int64_t)r * per], c0 = c_s[r * 2], c1 = c_s[r * 2 + 1];
        for (int k = 0; k < 4; ++k)
          for (int y = 0; y < 4; ++y) {
            lo[k][y] = fmaf(wv[k], c0[y], lo[k][y]);
            hi[k][y] = fmaf(wv[k], c1[y], hi[k][y]);
          }
      }
      for (int k = 0; k < 4; ++k)
        for (int y = 0; y < 4; ++y) {
          red[wave][y * 4 + k][lane] = lo[k][y];
          red[wave][(y + 4) * 4 + k][lane] = hi[k][y];
        }
    }
    __syncthreads();
    // 512 vectors: of a key, four columns of one token; of a value, four tokens of one column
    for (int u = threadIdx.x; u < 8 * 64; u += kThreads) {
      const int l = u >> 3, vec = cv0 + l;
      if (vec >= n_all) break;
      const bool is_v = vec >= nk;
      const int dim = is_v ? a.d_v : a.d_h, e = (is_v ? vec - nk : vec) * 4, jj = e / dim, d = e % dim;
      const int tok = is_v ? (u & 1) * 4 : u & 7, col = is_v ? (u >> 1) & 3 : 0;
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < kThreads / 64; ++s)
        for (int k = 0; k < 4; ++k) sum[k] += is_v ? red[s][(tok + k) * 4 + col][l] : red[s][tok * 4 + k][l];
      if (is_v) {
        float* dst = out + (int64_t)gc * P * a.d_h + ((int64_t)(jj * (P / 8) + slot0 / 8) * a.d_v + d + col) * 8 + tok;
        if (tok >= first && tok + 4 <= valid) *(f32x4*)dst = sum;
        else
          for (int k = 0; k < 4; ++k)
            if (tok + k >= first && tok + k < valid) dst[k] = sum[k];  // slots that no token owns are not written
      } else if (tok >= first && tok < valid) {
        *(f32x4*)(out + ((int64_t)(jj * (a.d_h / 8) + d / 8) * P + slot0 + tok) * 8 + d % 8) = sum;
      }
    }
    if (!kLoop) return;
  }
}

// Cache compression, fp32: one workgroup per (logical page, sequence); c = A^+ k^C per token, k_R copied.
__global__ void compress_f32_kernel(CompressArgs a) {
  const int p = blockIdx.x, b = blockIdx.y;
  const int L = a.seq_lens[b];
  const int P = a.expanded.page_size;
  if ((int64_t)p * P >= L) return;
  const int32_t pg_in = page_of(a.expanded, b, p), pg_out = page_of(a.latent, b, p);
  if (pg_in < 0 || pg_out < 0) return;
  const int valid = min(P, L - p * P);
  const int g = a.g, W = a.r_kv + a.d_r, K = g * a.d_h;
  const float* in = (const float*)a.expanded.pool + (int64_t)pg_in * P * (g * (a.d_h + a.d_v) + a.d_r);
  float* out = (float*)a.latent.pool + (int64_t)pg_out * P * W;
  for (int idx = threadIdx.x; idx < valid * W; idx += blockDim.x) {
    const int slot = idx / W, e = idx % W;
    float v;
    if (e < a.r_kv) {
      const float* w = (const float*)a.w_inv + (int64_t)e * K;
      float acc = 0.f;
      for (int k = 0; k < K; ++k) {
        const int j = k / a.d_h, d = k % a.d_h;
        acc += w[k] * in[((int64_t)(j * (a.d_h / 8) + d / 8) * P + slot) * 8 + d % 8];
      }
      v = acc;
    } else {
      const int d = e - a.r_kv;
      v = in[(int64_t)g * P * (a.d_h + a.d_v) + ((int64_t)(d / 8) * P + slot) * 8 + d % 8];
    }
    out[(int64_t)slot * W + e] = v;
  }
}

// The step's latent rows into their cache slots (any element type: rows are copied as 16-byte vectors).
// One workgroup per (step token, sequence).  A chain of memory latencies, length -> page id -> slot; the row itself depends on
// neither and is requested first (with the rotary step, a step of one sequence x 128 heads 34.0 -> 32.3 us, of 32 x 32 heads
// 56.6 -> 55.8).
__global__ void append_latent_kernel(AppendArgs a) {
  const int t = blockIdx.x, b = blockIdx.y;
  const int vecs = a.row_bytes / 16;
  const u32x4* src = (const u32x4*)((const char*)a.rows + ((int64_t)b * a.s_q + t) * a.row_bytes);
  u32x4 v = {0, 0, 0, 0};
  if ((int)threadIdx.x < vecs) v = src[threadIdx.x];
  asm volatile("" ::: "memory");   // (the request stays ahead of the branches below)
  const int pos = a.seq_lens[b] - a.s_q + t;
  if (pos < 0) return;
  const int P = a.latent.page_size;
  const int32_t pg = page_of(a.latent, b, pos / P);
  if (pg < 0) return;
  u32x4* dst = (u32x4*)((char*)a.latent.pool + ((int64_t)pg * P + pos % P) * a.row_bytes);
  if ((int)threadIdx.x < vecs) dst[threadIdx.x] = v;
  for (int i = threadIdx.x + blockDim.x; i < vecs; i += blockDim.x) dst[i] = src[i];
}

}  // namespace

hipError_t launch_compress_f32(const CompressArgs& a, hipStream_t s) {
  compress_f32_kernel<<<dim3(a.expanded.max_pages, a.B), 256, 0, s>>>(a);
  return hipGetLastError();
}
hipError_t launch_expand_tail_f32(const ExpandArgs& a, hipStream_t s) {
  const int col_blocks = (a.group_count * (a.d_h + a.d_v) + 255) / 256;
  expand_f32_kernel<true, false><<<dim3((a.tail + 6) / 8 + 1, a.B, col_blocks), kThreads, 0, s>>>(a);
  return hipGetLastError();
}
hipError_t launch_append_latent(const AppendArgs& a, hipStream_t s) {
  append_latent_kernel<<<dim3(a.s_q, a.B), 128, 0, s>>>(a);
  return hipGetLastError();
}
hipError_t launch_absorb_query_f32(const AbsorbQueryArgs& a, hipStream_t s) {
  absorb_query_f32_kernel<<<dim3(a.h_q, a.rows), kThreads, 0, s>>>(a);
  return hipGetLastError();
}
// One chunk per sequence: the decode writes the output itself, the combine of one partial (2 to 5 us) falls away.  Not where
// the caller has laid the output over the queries: other workgroups still read those then.
static bool f32_decode_is_final(const DecodeArgs& a, const CombineArgs& c, int dk) {
  auto apart = [](const void* x, size_t nx, const void* y, size_t ny) { return (const char*)x + nx <= (const char*)y || (const char*)y + ny <= (const char*)x; };
  const size_t rows = (size_t)a.B * a.M, out = rows * c.d_h * sizeof(float), lse = rows * sizeof(float);
  const size_t q_a = rows * dk * sizeof(float), q_r = rows * a.d_r * sizeof(float);
  return a.n_chunks == a.B && apart(c.out, out, a.q_a, q_a) && apart(c.out, out, a.q_r, q_r) &&
         (!c.lse || (apart(c.lse, lse, a.q_a, q_a) && apart(c.lse, lse, a.q_r, q_r)));
}
hipError_t launch_decode_gqa_f32(const DecodeArgs& a, const CombineArgs& c, hipStream_t s) {
  if (f32_decode_is_final(a, c, a.d_h)) decode_f32_kernel<false, true><<<dim3(a.n_chunks, a.M), kThreads, 0, s>>>(a, c);
  else decode_f32_kernel<false, false><<<dim3(a.n_chunks, a.M), kThreads, 0, s>>>(a, c);
  return hipGetLastError();
}
hipError_t launch_decode_absorb_f32(const DecodeArgs& a, const CombineArgs& c, hipStream_t s) {
  if (f32_decode_is_final(a, c, a.r_kv)) decode_f32_kernel<true, true><<<dim3(a.n_chunks, a.M), kThreads, 0, s>>>(a, c);
  else decode_f32_kernel<true, false><<<dim3(a.n_chunks, a.M), kThreads, 0, s>>>(a, c);
  return hipGetLastError();
}
hipError_t launch_combine_f32(const DecodeArgs& d, const CombineArgs& a, hipStream_t s) {
  if (f32_decode_is_final(d, a, d.d_h)) return hipSuccess;  // the decode has written the output
  const unsigned blocks = (unsigned)(((int64_t)a.B * a.M + 7) / 8);
  combine_kernel<<<blocks, 256, 0, s>>>(a);
  return hipGetLastError();
}
hipError_t launch_combine_project_f32(const DecodeArgs& d, const CombineArgs& a, hipStream_t s) {
  if (f32_decode_is_final(d, a, d.r_kv)) return hipSuccess;  // the decode has written the output
  combine_project_f32_kernel<<<dim3(a.M, a.B), kThreads, 0, s>>>(a);
  return hipGetLastError();
}
hipError_t launch_expand_f32(const ExpandArgs& a, hipStream_t s) {
  const int col_blocks = (a.group_count * (a.d_h + a.d_v) + 255) / 256;
  // What a row of the page table could hold bounds the tokens; beyond 8192 of them a workgroup takes every 1024th eight.  (With a
  // workgroup for each, rows of 131 072 tokens made 16 sequences x 4000 tokens, four column blocks take 231 us instead of 190.)
  const int eights = a.max_tokens / 8;
  if (eights <= 1024) expand_f32_kernel<false, false><<<dim3(eights, a.B, col_blocks), kThreads, 0, s>>>(a);
  else expand_f32_kernel<false, true><<<dim3(1024, a.B, col_blocks), kThreads, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace gqla
