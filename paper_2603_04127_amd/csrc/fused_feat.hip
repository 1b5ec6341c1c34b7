// Fused MFMA feature-map kernel of the DARK attention library (gfx950): bf16 in, bf16 out.
//
// phi_j(x) = exp(w_j^T (M x') - 1/2 |M x'|^2 - c) / sqrt(m),  x' = sqrt(scale) x   (Section 4.1, the
// feature map before Eq. (3); omega~_j = M^T w_j as in Appendix B), computed in the log2 domain
// from the fp16 operands A' = alpha log2(e) W M and M' = alpha sqrt(log2(e)/2) M that the attention
// kernels use as well.  The pre-exponential logits never leave registers.
//
// k_featurize: workgroup = m / 64 waves; a wave keeps its 64 rows of A' in registers and the workgroup walks a run of
// 32-token tiles of one (b,h), the tokens as MFMA columns (U^T[feat][tok] = A' X^T): every logit is formed
// once and stays in its accumulator until the token's shift is known.  The waves' row maxima and their parts
// of |M' x|^2 (32 rows of M' at a time) meet in LDS, one barrier a tile.  The tiles come in batches of one per wave,
// fetched a batch ahead and converted to fp16 on their way into LDS: a tile at a time, fetched by every wave for
// itself, left the memory idle (the keys' maxima alone took 14 us).  Queries: one launch.  Keys: the
// shift is the maximum over the whole (b,h) slice, so a first launch leaves one partial maximum per workgroup
// and the second launch reduces those.  The feature tile is turned through a per-wave LDS stage so that the
// stores are 128-byte rows.
// Measured, queries and keys of 98,304 rows, d = 64, m = 256 with the operand preparation: 60 us with waves of 64 tokens that swept
// all features twice with A' in LDS, 51 with A' in registers, 46 with A' read as fragments (a copy of the bytes takes 25 us); the
// launches are bound by the stores and by the chain projection, exchange, exponential, stage of a tile.
#include <cmath>

#include "fused_common.h"

namespace dark {
using namespace fz;
namespace {

template <int D>
struct FtSmem {
  static constexpr int MS = D + 8;                        // halves per row of M'
  static constexpr size_t m_bytes = (size_t)D * MS * 2;
  static constexpr size_t stage_bytes = 32 * 128;         // per wave: 32 tokens x 64 features, 16-byte chunk c of row r at c ^ (r % 8)
  static constexpr size_t ex_bytes = 2 * 2 * 32 * 4;      // per wave: maxima and partial norms of two tiles
  static constexpr size_t x_bytes = (size_t)32 * MS * 2;  // per wave: a tile of the batch
  __host__ __device__ static size_t total(int nw) { return m_bytes + nw * (stage_bytes + ex_bytes + x_bytes); }
};

enum { FT_QUERY = 0, FT_KEY_MAX = 1, FT_KEY = 2 };   // row shifts; partial maxima only; features with the slice shift
// Registers for four waves a SIMD (D = 64; up to fourteen waves a workgroup) or two (D = 128; up to six).
template <int D, int MODE>
__global__ __launch_bounds__(D == 64 ? 1024 : 512, D == 64 ? 4 : 2) void k_featurize(
    const unsigned short* __restrict__ Xg, const _Float16* __restrict__ Ah, const _Float16* __restrict__ Mh,
    unsigned short* __restrict__ phi, float* __restrict__ stab, float* __restrict__ pmax, int H, int L, int m,
    int wgs_per_bh, int tiles_per_wg) {
  using SM = FtSmem<D>;
  constexpr int NS = D / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  _Float16* Ms = reinterpret_cast<_Float16*>(smem);
  const int nw = m / 64;
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hf = lane / 32;
  float* ex = reinterpret_cast<float*>(smem + SM::m_bytes);   // [parity][max | norm][wave][32]
  _Float16* Xs = reinterpret_cast<_Float16*>(smem + SM::m_bytes + nw * SM::ex_bytes);   // [tile of the batch][32][MS]
  unsigned char* stage = smem + SM::m_bytes + nw * (SM::ex_bytes + SM::x_bytes) + wv * SM::stage_bytes;
  const int bh = blockIdx.x / wgs_per_bh, run = blockIdx.x % wgs_per_bh, h = bh % H;
  const int ntile = (L + 31) / 32, t_begin = run * tiles_per_wg, t_end = min(ntile, t_begin + tiles_per_wg);
  const unsigned short* Xb = Xg + (size_t)bh * L * D;

  // a wave's tile of a batch: 16-byte pieces, whole rows; rows past the end repeat the last row
  constexpr int NP = 32 * D / 8 / 64, CPR = D / 8;
  u32x4 raw[NP];
  auto fetch = [&](int t) {
    if (t < t_end) {   // wave-uniform
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int i = 64 * u + lane;
        raw[u] = *reinterpret_cast<const u32x4*>(Xb + (size_t)min(32 * t + i / CPR, L - 1) * D + 8 * (i % CPR));
      }
    }
  };
  auto put = [&](int t) {
    if (t < t_end) {
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int i = 64 * u + lane;
        *reinterpret_cast<u32x4*>(Xs + (32 * wv + i / CPR) * SM::MS + 8 * (i % CPR)) = bf16x8_to_f16x8(raw[u]);
      }
    }
  };
  fetch(t_begin + wv);
  half8 af[2][NS];
#pragma unroll
  for (int fs = 0; fs < 2; ++fs)
#pragma unroll
    for (int s = 0; s < NS; ++s)
      af[fs][s] = *reinterpret_cast<const half8*>(a_frag16<D>(Ah, h, m, 64 * wv + 32 * fs, s, lane));
  for (int ci = tid; ci < D * D / 8; ci += 64 * nw)
    *reinterpret_cast<u32x4*>(Ms + (ci / (D / 8)) * SM::MS + 8 * (ci % (D / 8))) =
        *reinterpret_cast<const u32x4*>(Mh + (size_t)h * D * D + 8 * (size_t)ci);
  float cslice = 0.f;   // keys: the shift of the (b,h) slice (log2 domain)
  if (MODE == FT_KEY) {
    cslice = -INFINITY;
    for (int i = lane; i < wgs_per_bh; i += 64) cslice = fmaxf(cslice, pmax[(size_t)bh * wgs_per_bh + i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cslice = fmaxf(cslice, __shfl_xor(cslice, o, 64));
    if (run == 0 && tid == 0 && stab != nullptr) stab[bh] = cslice / kLog2e;
  }
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float half_log2_m = 0.5f * log2f((float)m);
  float wmax = -INFINITY;
  put(t_begin + wv);
  __syncthreads();
  fetch(t_begin + nw + wv);

  for (int t = t_begin, q = 0; t < t_end; ++t, ++q) {
    if (q == nw) {   // the next batch takes the place of this one
      q = 0;
      lds_barrier();
      put(t + wv);
      fetch(t + nw + wv);
      lds_barrier();
    }
    // X fragments (B operand): token 32 t + l32, k = 16 s + 8 hf + [0,8)
    half8 xf[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) xf[s] = *reinterpret_cast<const half8*>(Xs + (32 * q + l32) * SM::MS + 16 * s + 8 * hf);
    // n'(token) = |M' x|^2: 32 rows of M' per wave, squares summed over the register rows and the halves
    float nrm = 0.f;
    for (int rb = wv; rb < D / 32; rb += nw) {
      f32x16 xt;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        xt = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const half8*>(Ms + (32 * rb + l32) * SM::MS + 16 * s + 8 * hf),
                                                    xf[s], s == 0 ? zero16 : xt, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 16; ++v) nrm = fmaf(xt[v], xt[v], nrm);
    }
    nrm += xor32(nrm);
    f32x16 U[2];
#pragma unroll
    for (int fs = 0; fs < 2; ++fs)
#pragma unroll
      for (int s = 0; s < NS; ++s) U[fs] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[fs][s], xf[s], s == 0 ? zero16 : U[fs], 0, 0, 0);
    float* e = ex + (t & 1) * 2 * 32 * nw + l32;
    if (MODE != FT_KEY) {
      float mx = -INFINITY;
#pragma unroll
      for (int fs = 0; fs < 2; ++fs)
#pragma unroll
        for (int v = 0; v < 16; v += 2) mx = max3(mx, U[fs][v], U[fs][v + 1]);
      mx = fmaxf(mx, xor32(mx));
      if (hf == 0) e[32 * wv] = mx;
    }
    if (hf == 0) e[32 * (nw + wv)] = nrm;
    lds_barrier();
    const bool in = 32 * t + l32 < L;
    const int nb = min(nw, D / 32);   // waves with rows of M'
    float part[D / 32];
#pragma unroll
    for (int w = 0; w < D / 32; ++w) part[w] = e[32 * (nw + min(w, nb - 1))];
    float sh = cslice;
    if (MODE != FT_KEY) {
      sh = -INFINITY;
      for (int w = 0; w < nw; w += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u) sh = fmaxf(sh, e[32 * min(w + u, nw - 1)]);
    }
    nrm = part[0];
#pragma unroll
    for (int w = 1; w < D / 32; ++w) nrm += w < nb ? part[w] : 0.f;
    if (MODE != FT_KEY) sh -= nrm;   // the row's largest logit
    if (MODE == FT_QUERY && wv == 0 && hf == 0 && in && stab != nullptr) stab[(size_t)bh * L + 32 * t + l32] = sh / kLog2e;
    if (MODE == FT_KEY_MAX) {
      if (in) wmax = fmaxf(wmax, sh);
      continue;
    }
    const float off = -nrm - sh - half_log2_m;
#pragma unroll
    for (int fs = 0; fs < 2; ++fs)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const u32x2 w = {pack_bf16(fast_exp2(U[fs][4 * a] + off), fast_exp2(U[fs][4 * a + 1] + off)),
                         pack_bf16(fast_exp2(U[fs][4 * a + 2] + off), fast_exp2(U[fs][4 * a + 3] + off))};
        *reinterpret_cast<u32x2*>(stage + l32 * 128 + 16 * ((4 * fs + a) ^ (l32 % 8)) + 8 * hf) = w;
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int row = lane / 8, ch = lane % 8;
#pragma unroll
    for (int ps = 0; ps < 4; ++ps) {
      const u32x4 w = *reinterpret_cast<const u32x4*>(stage + (8 * ps + row) * 128 + 16 * (ch ^ row));
      const int tok = 32 * t + 8 * ps + row;
      if (tok < L) *reinterpret_cast<u32x4*>(phi + ((size_t)bh * L + tok) * m + 64 * wv + 8 * ch) = w;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  if (MODE == FT_KEY_MAX && wv == 0) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wmax = fmaxf(wmax, __shfl_xor(wmax, o, 64));
    if (lane == 0) pmax[blockIdx.x] = wmax;
  }
}

// Few features of wide rows (feat_rows): four waves of 64 tokens each sweep all features twice (once for the row maxima, once
// for the features) with A' and M' in LDS, so that a fragment of M' serves 64 tokens where the kernel above reads it for 32; work
// items of 256 tokens, dealt to at most 512 workgroups.  Queries + keys, us, k_featurize / this one, d = 128: m = 64 at 384 x 4000
// rows 201 + 339 / 137 + 233, at 96 x 1000 27 + 46 / 19 + 28, at 96 x 64 16 + 25 / 14 + 18; m = 128 at 384 x 4000 298 + 474 /
// 228 + 347, at 384 x 1000 83 + 133 / 72 + 114, at 96 x 4000 70 + 112 / 70 + 109, at 384 x 256 31 + 50 / 35 + 51, at 384 x 64
// 16 + 25 / 28 + 39; m = 192 at 384 x 1000 80 + 130 / 96 + 140.  d = 64, m = 64 at 384 x 4000 88 + 125 / 89 + 120, at
// 384 x 1000 25 + 42 / 27 + 39: the kernel above.
template <int D>
struct FrSmem {
  static constexpr int AS = D + 8;
  static constexpr int stage_row = 128 + 8;              // bytes: 64 bf16 plus pad
  static constexpr size_t stage_bytes = 32 * stage_row;  // per wave: 32 tokens x 64 features
  __host__ __device__ static size_t a_bytes(int m) { return (size_t)m * AS * 2; }
  static constexpr size_t m_bytes = (size_t)D * AS * 2;
  __host__ __device__ static size_t total(int m) { return a_bytes(m) + m_bytes + 4 * stage_bytes + 64; }
};

template <int D, int MODE>
__global__ __launch_bounds__(256, 2) void k_featurize_rows(
    const unsigned short* __restrict__ Xg, const _Float16* __restrict__ Ah, const _Float16* __restrict__ Mh,
    unsigned short* __restrict__ phi, float* __restrict__ stab, float* __restrict__ pmax,
    int H, int L, int m, int chunks_per_bh, int n_items, int items_per_wg) {
  using SM = FrSmem<D>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  _Float16* Asl = reinterpret_cast<_Float16*>(smem);
  _Float16* Ms = reinterpret_cast<_Float16*>(smem + SM::a_bytes(m));
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  unsigned char* stage = smem + SM::a_bytes(m) + SM::m_bytes + wv * SM::stage_bytes;
  float* red = reinterpret_cast<float*>(smem + SM::a_bytes(m) + SM::m_bytes + 4 * SM::stage_bytes);
  const int l32 = lane % 32, hf = lane / 32;
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float half_log2_m = 0.5f * log2f((float)m);

  const int item_begin = blockIdx.x * items_per_wg;
  const int item_end = min(n_items, item_begin + items_per_wg);
  int cur_bh = -1, cur_h = -1;
  float cslice = 0.f;  // keys: the shift of the current (b,h) slice (log2 domain)
  for (int item = item_begin; item < item_end; ++item) {
    const int bh = item / chunks_per_bh, chunk = item % chunks_per_bh;
    if (bh != cur_bh) {
      const int h = bh % H;
      if (cur_bh >= 0) __syncthreads();
      if (h != cur_h) {
        for (int ci = tid; ci < m * D / 8; ci += 256) {
          const int row = ci / (D / 8), kc = ci % (D / 8);
          *reinterpret_cast<u32x4*>(Asl + row * SM::AS + 8 * kc) =
              *reinterpret_cast<const u32x4*>(Ah + ((size_t)h * m + row) * D + 8 * kc);
        }
        for (int ci = tid; ci < D * D / 8; ci += 256) {
          const int row = ci / (D / 8), kc = ci % (D / 8);
          *reinterpret_cast<u32x4*>(Ms + row * SM::AS + 8 * kc) =
              *reinterpret_cast<const u32x4*>(Mh + ((size_t)h * D + row) * D + 8 * kc);
        }
        cur_h = h;
      }
      if (MODE == FT_KEY) {  // slice shift = maximum of the partial maxima of the first launch
        float v = -INFINITY;
        for (int i = tid; i < chunks_per_bh; i += 256) v = fmaxf(v, pmax[(size_t)bh * chunks_per_bh + i]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
        if (lane == 0) red[wv] = v;
        __syncthreads();
        cslice = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
      }
      __syncthreads();
      cur_bh = bh;
    }
    const int t0 = chunk * 256 + 64 * wv;
    const bool active = t0 < L;  // wave-uniform; inactive waves still take part in the barriers below
    float wmax = -INFINITY;
    if (active) {
      const unsigned short* Xb = Xg + (size_t)bh * L * D;
      // X fragments (B operand): token = t0 + 32 tt + l32, k = 16 s + 8 hf + [0,8)
      // (all loads are issued before the first is converted: one wait for memory, not one per load)
      half8 xf[2][D / 16];
      u32x4 raw[2][D / 16];
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const int tok = min(t0 + 32 * tt + l32, L - 1);  // rows past the end repeat the last row; never stored
#pragma unroll
        for (int s = 0; s < D / 16; ++s) raw[tt][s] = *reinterpret_cast<const u32x4*>(Xb + (size_t)tok * D + 16 * s + 8 * hf);
      }
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
          u32x4 cv = bf16x8_to_f16x8(raw[tt][s]);
          xf[tt][s] = *reinterpret_cast<half8*>(&cv);
        }
      // n'(token) = |M' x|^2: x~^T[r][tok] by MFMA, squares summed over the register rows and the halves
      float nrm[2] = {0.f, 0.f};
#pragma unroll
      for (int rt = 0; rt < D / 32; ++rt) {
        f32x16 xt[2] = {zero16, zero16};
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
          half8 a = *reinterpret_cast<const half8*>(Ms + (32 * rt + l32) * SM::AS + 16 * s + 8 * hf);
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) xt[tt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, xf[tt][s], xt[tt], 0, 0, 0);
        }
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
          for (int v = 0; v < 16; ++v) nrm[tt] = fmaf(xt[tt][v], xt[tt][v], nrm[tt]);
      }
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) nrm[tt] += __shfl_xor(nrm[tt], 32, 64);

      auto project = [&](int g, f32x16 (&U)[2]) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
          half8 a = *reinterpret_cast<const half8*>(Asl + (32 * g + l32) * SM::AS + 16 * s + 8 * hf);
#pragma unroll
          for (int tt = 0; tt < 2; ++tt)
            U[tt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, xf[tt][s], s == 0 ? zero16 : U[tt], 0, 0, 0);
        }
      };
      // shift per token (log2 domain): queries and the keys' first launch need the row maxima
      float sh[2];
      if (MODE != FT_KEY) {
        float mx[2] = {-INFINITY, -INFINITY};
        for (int g = 0; g < m / 32; ++g) {
          f32x16 U[2];
          project(g, U);
#pragma unroll
          for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int v = 0; v < 16; v += 2) mx[tt] = max3(mx[tt], U[tt][v], U[tt][v + 1]);
        }
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
          mx[tt] = fmaxf(mx[tt], __shfl_xor(mx[tt], 32, 64)) - nrm[tt];  // maximum logit of the row
          sh[tt] = mx[tt];
          if (t0 + 32 * tt + l32 < L) wmax = fmaxf(wmax, mx[tt]);
        }
        if (MODE == FT_QUERY && hf == 0) {
#pragma unroll
          for (int tt = 0; tt < 2; ++tt)
            if (stab != nullptr && t0 + 32 * tt + l32 < L) stab[(size_t)bh * L + t0 + 32 * tt + l32] = sh[tt] / kLog2e;
        }
      } else {
        sh[0] = sh[1] = cslice;
      }
      if (MODE != FT_KEY_MAX) {
        // exponentiate and store, two units (64 features = one 128-byte row piece) at a time
        const int row = lane / 8, ch = lane % 8;
        for (int gp = 0; gp < m / 64; ++gp) {
          f32x16 U[2][2];
          project(2 * gp, U[0]);
          project(2 * gp + 1, U[1]);
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) {
            const float off = -nrm[tt] - sh[tt] - half_log2_m;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                u32x2 w = {pack_bf16(fast_exp2(U[u][tt][4 * g] + off), fast_exp2(U[u][tt][4 * g + 1] + off)),
                           pack_bf16(fast_exp2(U[u][tt][4 * g + 2] + off), fast_exp2(U[u][tt][4 * g + 3] + off))};
                *reinterpret_cast<u32x2*>(stage + l32 * SM::stage_row + (32 * u + 8 * g + 4 * hf) * 2) = w;
              }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int ps = 0; ps < 4; ++ps) {
              const int tok = t0 + 32 * tt + 8 * ps + row;
              u32x4 w = *reinterpret_cast<const u32x4*>(stage + (8 * ps + row) * SM::stage_row + 16 * ch);
              if (tok < L) *reinterpret_cast<u32x4*>(phi + ((size_t)bh * L + tok) * m + 64 * gp + 8 * ch) = w;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
          }
        }
      }
    }
    if (MODE == FT_KEY_MAX) {  // one partial maximum per work item
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) wmax = fmaxf(wmax, __shfl_xor(wmax, o, 64));
      __syncthreads();
      if (lane == 0) red[wv] = wmax;
      __syncthreads();
      if (tid == 0) pmax[item] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    }
    if (MODE == FT_KEY && chunk == 0 && tid == 0 && stab != nullptr) stab[bh] = cslice / kLog2e;
  }
}

// Runs of tiles: as many workgroups as fit the chip at once (by registers sixteen waves a CU at D = 64, eight at D = 128;
// by LDS three workgroups at m = 256), every tile its own while they suffice.
struct FtPlan {
  int wgs_per_bh, tiles_per_wg;
};
FtPlan feat_plan(const Problem& pb) {
  const dark_params& p = pb.p;
  const int nw = p.m / 64;
  const int by_waves = (p.d == 64 ? 16 : 8) / nw;
  const int by_lds = (int)(160 * 1024 / (p.d == 64 ? FtSmem<64>::total(nw) : FtSmem<128>::total(nw)));
  const int per_cu = by_waves < by_lds ? by_waves : by_lds;
  const long long BH = pb.BH(), fit = 256LL * (per_cu > 0 ? per_cu : 1);
  const int nt = (p.L + 31) / 32;
  long long w = fit / (BH > 0 ? BH : 1);
  w = w < 1 ? 1 : (w > nt ? nt : w);
  FtPlan f;
  f.tiles_per_wg = (int)((nt + w - 1) / w);
  f.wgs_per_bh = (nt + f.tiles_per_wg - 1) / f.tiles_per_wg;
  return f;
}

// Which kernel (figures at k_featurize_rows): at d = 128 one wave of 64 features waits for its fragments of M' at any length, two
// waves do once the chip is full, from some 350,000 rows; three or more share the reads better than a second sweep costs.
bool feat_rows(const Problem& pb) {
  const dark_params& p = pb.p;
  return p.d == 128 && (p.m == 64 || (p.m == 128 && pb.rows() > 350000));
}
// partial maxima of the keys: one per workgroup of k_featurize, one per work item of k_featurize_rows
size_t feat_pmax(const Problem& pb) {
  return (size_t)pb.BH() * (feat_rows(pb) ? (pb.p.L + 255) / 256 : feat_plan(pb).wgs_per_bh);
}

template <int D>
dark_status launch_feat_rows(const Problem& pb, const void* X, const _Float16* Ah, const _Float16* Mh, int is_query,
                             void* phi, float* stab, float* pmax) {
  const dark_params& p = pb.p;
  const int chunks_per_bh = (p.L + 255) / 256, n_items = (int)(pb.BH() * chunks_per_bh);
  const int items_per_wg = (n_items + 511) / 512;
  const unsigned grid = (unsigned)((n_items + items_per_wg - 1) / items_per_wg);
  const size_t lds = FrSmem<D>::total(p.m);
  auto run = [&](auto kern) -> dark_status {
    DARK_TRY(allow_lds(kern, lds));
    DARK_LAUNCH(KID_FEATURIZE, pb.st, kern, dim3(grid), dim3(256), lds, (const unsigned short*)X, Ah, Mh, (unsigned short*)phi, stab,
                pmax, p.H, p.L, p.m, chunks_per_bh, n_items, items_per_wg);
    return DARK_OK;
  };
  if (is_query) return run(k_featurize_rows<D, FT_QUERY>);
  DARK_TRY(run(k_featurize_rows<D, FT_KEY_MAX>));
  return run(k_featurize_rows<D, FT_KEY>);
}

template <int D>
dark_status launch_feat(const Problem& pb, const void* X, const _Float16* Ah, const _Float16* Mh, int is_query,
                        void* phi, float* stab, float* pmax) {
  const dark_params& p = pb.p;
  const FtPlan f = feat_plan(pb);
  const int nw = p.m / 64;
  const size_t lds = FtSmem<D>::total(nw);
  // a launch holds 2^32 - 1 threads: as many batch entries at a time (all of them, but for tens of millions of short rows)
  const long long per_b = (long long)p.H * f.wgs_per_bh, most = 0xffffffffLL / (64 * nw) / per_b;
  if (most < 1) return DARK_EUNSUPPORTED;
  auto run = [&](auto kern) -> dark_status {
    DARK_TRY(allow_lds(kern, lds));
    for (long long b = 0; b < p.B; b += most) {
      const long long nb = p.B - b < most ? p.B - b : most;
      const size_t bh = (size_t)b * p.H, row = bh * p.L;
      DARK_LAUNCH(KID_FEATURIZE, pb.st, kern, dim3((unsigned)(nb * per_b)), dim3(64 * nw), lds, (const unsigned short*)X + row * D,
                  Ah, Mh, (unsigned short*)phi + row * p.m, stab == nullptr ? stab : stab + (is_query ? row : bh),
                  pmax + b * per_b, p.H, p.L, p.m, f.wgs_per_bh, f.tiles_per_wg);
    }
    return DARK_OK;
  };
  if (is_query) return run(k_featurize<D, FT_QUERY>);
  DARK_TRY(run(k_featurize<D, FT_KEY_MAX>));
  return run(k_featurize<D, FT_KEY>);
}

}  // namespace

bool fused_featurize_supported(const Problem& pb) {
  const dark_params& p = pb.p;
  if (p.io_dtype != DARK_BF16) return false;
  const bool shape64 = p.d == 64 && p.r == 64, shape128 = p.d == 128 && p.r == 128;
  if (!shape64 && !shape128) return false;
  return p.m % 64 == 0 && p.m <= (shape64 ? 896 : 384);   // a wave per 64 features
}

dark_status fused_featurize(const Problem& pb, Arena& ar, const void* X, const float* M, const float* W, int is_query,
                            void* phi, float* stab) {
  const dark_params& p = pb.p;
  _Float16* Ah = ar.take<_Float16>((size_t)p.H * p.m * p.d);
  _Float16* Mh = ar.take<_Float16>((size_t)p.H * p.r * p.d);
  float* pmax = ar.take<float>(feat_pmax(pb));
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  DARK_TRY(fused_launch_prep(pb, M, W, Ah, Mh, !feat_rows(pb)));
  if (feat_rows(pb)) return launch_feat_rows<128>(pb, X, Ah, Mh, is_query, phi, stab, pmax);
  if (p.d == 64) return launch_feat<64>(pb, X, Ah, Mh, is_query, phi, stab, pmax);
  return launch_feat<128>(pb, X, Ah, Mh, is_query, phi, stab, pmax);
}

}  // namespace dark
