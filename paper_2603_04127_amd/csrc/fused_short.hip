// Short sequences on the fused MFMA path (gfx950; bf16 inputs, fp32 accumulation): two launches instead of four.
//
// The kernels of fused.hip cut the keys of a (b,h) into slices, whose states a third kernel merges, and start from operand
// copies that a fourth one prepares.  Where a sequence has some dozens of tiles each of those launches is two or three memory
// round trips around almost no work.  Here a workgroup owns a block of features of one (b,h) and all of its keys, so that
// nothing has to be merged between workgroups, and forms its block of A' itself:
//   k_short_keys     per (b,h, block of features): S^T, z and the block's shift; A' for the readout
//   k_short_readout  per (b,h, tokens): out = phi_Q S / phi_Q z, the features divided over the waves
// Everything is in the log2 domain with A' and M' as in fused.hip (Section 4.1 feature map, Appendix B).
// 36 (b,h) of 509 tokens, d = 64, m = 256: 29.6 us in four launches, 18.7 in two (one of 1024 tokens: 25.5 and 18.2).
#include <cfloat>
#include <cmath>

#include "fused_common.h"

namespace dark {
using namespace fz;
namespace {

constexpr int kTok = 32;     // tokens per tile
constexpr int kWaves = 8;
constexpr int NT = 64 * kWaves;

__device__ __forceinline__ f32x16 mm_f16(half8 a, half8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 mm_bf16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8*>(&a), *reinterpret_cast<bf16x8*>(&b), c, 0, 0, 0);
}
__device__ __forceinline__ half8 as_half8(u32x4 v) { return *reinterpret_cast<half8*>(&v); }
// Workgroups are dealt to the eight XCDs in turn: neighbours, which share a (b,h), go to one of them (and its L2).
__device__ __forceinline__ int xcd_order(int i, int n) { return n % 8 == 0 ? (i % 8) * (n / 8) + i / 8 : i; }
// What this wave has written to LDS is there for its other lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A packed accumulator as an operand meets its partner's contraction index in this order (bits 2 and 3 exchanged): S^T is
// stored in it, so that a lane's eight features are one 16-byte read.
__device__ __forceinline__ int chain_feature(int piece) { return 16 * (piece / 2) + 4 * (piece % 2); }

// Features of a workgroup: the state of a wave, FB features by D value columns, is 64 accumulator registers either way.
template <int D>
constexpr int short_fb() { return D == 64 ? 64 : 32; }

template <int D>
struct ShortSmem {
  static constexpr int FB = short_fb<D>();
  static constexpr int AS = D + 8;                                   // halves per row of A' and M'
  static constexpr size_t a_bytes = (size_t)FB * AS * 2, m_bytes = (size_t)D * AS * 2;
  static constexpr size_t t_bytes = (size_t)kTok * AS * 2;           // a wave's tile, of K and then of V
  static constexpr size_t off_m = a_bytes, off_v = a_bytes + m_bytes;
  static constexpr int LW = D + 4;                                   // W and M as they are, before the tiles
  static constexpr size_t off_w = off_v, off_mf = off_w + (size_t)FB * LW * 4;
  static constexpr size_t part = (size_t)FB * D * 4;                 // a wave's state
  static constexpr size_t off_cz = kWaves * part;                    // [wave][shift | z][FB], then the factors [wave][FB]
  static constexpr size_t off_n = off_cz + (size_t)kWaves * 3 * FB * 4;
  static constexpr size_t total = off_n + (size_t)kWaves * kTok * 4;
  static_assert(off_v + kWaves * t_bytes <= off_n && off_mf + (size_t)D * D * 4 <= off_n && total <= 160 * 1024, "LDS map");
};
// Element (column c, feature f) of a wave's state in LDS: the 16-byte pieces of a row permuted, so that neither 32 rows of one
// piece nor one row after another meet on a bank.
template <int D>
__device__ __forceinline__ int part_at(int c, int f) {
  constexpr int FB = short_fb<D>(), N = FB / 4;
  return c * FB + 4 * ((f / 4) ^ (c % N)) + f % 4;
}

// ---------------------------------------------------------------------------
// k_short_keys: a wave takes every eighth tile of 32 keys, and the waves' states meet in LDS, in wave order.  Each tile
// costs its wave the norms (formed again for every block of features: the price of having no launch before this one),
// the projection, the exponentials and phi^T V, with no barrier; K and V pass through the wave's own LDS tile, so that
// memory sees whole lines.  Bound by vector issue (two waves a SIMD) and its three phases' latencies; at 36 (b,h) of 509
// tokens, 144 workgroups: 3.4 us until A' is there, 1.9 us a tile, 2.7 us to join the states.
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(NT, 2) void k_short_keys(const unsigned short* __restrict__ Kg,
                                                      const unsigned short* __restrict__ Vg, const float* __restrict__ M,
                                                      const float* __restrict__ W, _Float16* __restrict__ Ah,
                                                      unsigned short* __restrict__ St, float* __restrict__ zt,
                                                      float* __restrict__ cf, int H, int L, int m, int w_shared,
                                                      float alpha) {
  using SM = ShortSmem<D>;
  constexpr int FB = SM::FB, FT = FB / 32, CT = D / 32, NS = D / 16, AS = SM::AS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  _Float16* Asl = reinterpret_cast<_Float16*>(smem);
  _Float16* Msl = reinterpret_cast<_Float16*>(smem + SM::off_m);
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const int l32 = lane % 32, hf = lane / 32, l16 = lane % 16, kg = lane / 16;
  const int nblk = m / FB, wg = xcd_order(blockIdx.x, gridDim.x), bh = wg / nblk, blk = wg % nblk, f0 = FB * blk, h = bh % H;
  const int nt = (L + kTok - 1) / kTok;
  unsigned char* vt = smem + SM::off_v + wv * SM::t_bytes;
  _Float16* xs = reinterpret_cast<_Float16*>(vt);
  float* nl = reinterpret_cast<float*>(smem + SM::off_n) + kTok * wv;

  // a tile on its way: whole rows of K and V
  constexpr int VP = kTok * D / 8 / 64, CPR = D / 8;
  u32x4 kr[VP], vr[VP];
  auto fetch = [&](int t) {
#pragma unroll
    for (int u = 0; u < VP; ++u) {
      const int i = lane + 64 * u;
      const size_t at = ((size_t)bh * L + min(t * kTok + i / CPR, L - 1)) * D + 8 * (i % CPR);
      kr[u] = *reinterpret_cast<const u32x4*>(Kg + at);
      vr[u] = *reinterpret_cast<const u32x4*>(Vg + at);
    }
  };
  {
    // The block's rows of W, and M, pass through LDS (whole lines from memory: read from there as operands, 16 rows by 16 bytes an
    // instruction, they took 2 us); A' by fp32 MFMA 16x16x4, M' as fp16.
    constexpr int NB = (FB / 16) * (D / 16) / kWaves, RB = FB / 16;   // 16x16 pieces of a wave; all of one row block
    constexpr int WP = FB * D / 4 / NT, MP = D * D / 4 / NT, LW = SM::LW, QR = D / 4;
    float* Wl = reinterpret_cast<float*>(smem + SM::off_w);
    float* Ml = reinterpret_cast<float*>(smem + SM::off_mf);
    const f32x4* Mb = reinterpret_cast<const f32x4*>(M + (size_t)h * D * D);
    const f32x4* Wb = reinterpret_cast<const f32x4*>(W + ((w_shared ? 0 : (size_t)h * m) + f0) * D);
    f32x4 mv[MP], wr[WP];
#pragma unroll
    for (int u = 0; u < WP; ++u) wr[u] = Wb[tid + NT * u];
#pragma unroll
    for (int u = 0; u < MP; ++u) mv[u] = Mb[tid + NT * u];
    if (wv < nt) fetch(wv);
    __builtin_amdgcn_sched_barrier(0);   // every load is requested before the first is waited for
    const float fa = alpha * kLog2e, fm = alpha * sqrtf(0.5f * kLog2e);
#pragma unroll
    for (int u = 0; u < WP; ++u) *reinterpret_cast<f32x4*>(Wl + ((tid + NT * u) / QR) * LW + 4 * ((tid + NT * u) % QR)) = wr[u];
#pragma unroll
    for (int u = 0; u < MP; ++u) {
      typedef _Float16 h4 __attribute__((ext_vector_type(4)));
      const int i = tid + NT * u, r = i / QR, q = i % QR;
      *reinterpret_cast<f32x4*>(Ml + r * D + 4 * q) = mv[u];
      const f32x4 x = mv[u] * fm;
      *reinterpret_cast<h4*>(Msl + r * AS + 4 * q) = h4{(_Float16)x[0], (_Float16)x[1], (_Float16)x[2], (_Float16)x[3]};
    }
    __syncthreads();
    const int rb = wv % RB, cb = (wv / RB) * NB;
    const float *w = Wl + (16 * rb + l16) * LW + 4 * kg, *mc = Ml + 4 * kg * D + 16 * cb + l16;
    f32x4 acc[NB][2] = {};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(w + 16 * s);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int u = 0; u < NB; ++u)
          acc[u][j % 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], mc[(16 * s + j) * D + 16 * u], acc[u][j % 2], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        Asl[(16 * rb + 4 * kg + v) * AS + 16 * (cb + u) + l16] = (_Float16)((acc[u][0][v] + acc[u][1][v]) * fa);
  }
  __syncthreads();
  if (bh < H) {   // the first batch entry leaves the block of A' for the readout, as operand fragments
    for (int i = tid; i < FB * CPR; i += NT) {
      const int fl = i % 64, s = (i / 64) % NS, ft = i / (64 * NS);
      *reinterpret_cast<u32x4*>(Ah + ((size_t)h * m + f0) * D + 8 * i) =
          *reinterpret_cast<const u32x4*>(Asl + (32 * ft + fl % 32) * AS + 16 * s + 8 * (fl / 32));
    }
  }
  half8 af[FT][NS];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int s = 0; s < NS; ++s) af[ft][s] = *reinterpret_cast<const half8*>(Asl + (32 * ft + l32) * AS + 16 * s + 8 * hf);
  f32x16 S[FT][CT] = {};                 // registers = features, lane = value column
  float z[FT], c[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    z[ft] = 0.f;
    c[ft] = -INFINITY;                   // a wave without a tile counts for nothing
  }
  // V fragment: value column 32 ct + l32, tokens 16 hh + 4 hf + [0,4) and those + 8
  const int jj = l32 % 16, tl = 4 * hf + jj / 4, kq = 2 * (l32 / 16) + (jj % 4) / 2;
  for (int t = wv; t < nt; t += kWaves) {
    asm volatile("" ::: "memory");       // the last tile's rows and norms have been read
#pragma unroll
    for (int u = 0; u < VP; ++u) {
      const int i = lane + 64 * u, row = i / CPR, ch = i % CPR;
      *reinterpret_cast<u32x4*>(xs + row * AS + 8 * ch) = bf16x8_to_f16x8(kr[u]);
    }
    wave_sync();
    half8 xf[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) xf[s] = *reinterpret_cast<const half8*>(xs + l32 * AS + 16 * s + 8 * hf);
    asm volatile("" ::: "memory");       // (LDS operations of one wave complete in order)
#pragma unroll
    for (int u = 0; u < VP; ++u) {
      const int i = lane + 64 * u, row = i / CPR, ch = i % CPR;
      *reinterpret_cast<u32x4*>(vt + row * 2 * D + 16 * (ch ^ v_swz<2 * D>(row))) = vr[u];
    }
    if (t + kWaves < nt) fetch(t + kWaves);
    float n = 0.f;
#pragma unroll
    for (int rb = 0; rb < D / 32; ++rb) {
      f32x16 x = {};
#pragma unroll
      for (int s = 0; s < NS; ++s) x = mm_f16(*reinterpret_cast<const half8*>(Msl + (32 * rb + l32) * AS + 16 * s + 8 * hf), xf[s], x);
#pragma unroll
      for (int v = 0; v < 16; ++v) n = fmaf(x[v], x[v], n);
    }
    n += xor32(n);
    if (t * kTok + l32 >= L) n = INFINITY;   // rows past the end: features exactly zero
    if (hf == 0) nl[l32] = n;
    f32x16 U[FT] = {};
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) U[ft] = mm_f16(xf[s], af[ft][s], U[ft]);
    wave_sync();
    f32x4 n4[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) n4[a] = *reinterpret_cast<const f32x4*>(nl + 8 * a + 4 * hf);
    u32x4 pk[FT][2];
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        U[ft][v] -= n4[v / 4][v % 4];
        U[ft][v + 1] -= n4[v / 4][v % 4 + 1];
        mx = max3(mx, U[ft][v], U[ft][v + 1]);
      }
      mx = fmaxf(mx, xor32(mx));
      const bool first = t < kWaves;
      if (first || __any(mx > c[ft] + kRaise)) {   // set the wave's shifts, or raise them (rare)
        const float before = c[ft];
        if (first || mx > c[ft] + kRaise) c[ft] = fmaxf(mx, -FLT_MAX);
        if (!first) {
          const float f = fast_exp2(before - c[ft]);
          z[ft] *= f;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float fr = __shfl(f, 8 * (v / 4) + 4 * hf + (v % 4), 64);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) S[ft][ct][v] *= fr;
          }
        }
      }
      float zs = 0.f;
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float e0 = fast_exp2(U[ft][8 * hh + 2 * q] - c[ft]), e1 = fast_exp2(U[ft][8 * hh + 2 * q + 1] - c[ft]);
          zs += e0;
          zs += e1;
          pk[ft][hh][q] = pack_bf16(e0, e1);
        }
      z[ft] += zs;
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const unsigned char* r = vt + (16 * hh + tl) * 2 * D + 16 * ((kq + 4 * ct) ^ v_swz<2 * D>(tl)) + 8 * (jj % 2);
        const u32x2 lo = lds_read_tr16(reinterpret_cast<const unsigned short*>(r));
        const u32x2 hi = lds_read_tr16(reinterpret_cast<const unsigned short*>(r + 8 * 2 * D));
        const u32x4 v = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) S[ft][ct] = mm_bf16(pk[ft][hh], v, S[ft][ct]);
      }
  }
  __syncthreads();   // operands and tiles have been read: the states take their place
  float* part = reinterpret_cast<float*>(smem + wv * SM::part);
  float* cz = reinterpret_cast<float*>(smem + SM::off_cz);
  float* fac = cz + kWaves * 2 * FB;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *reinterpret_cast<f32x4*>(part + part_at<D>(32 * ct + l32, 32 * ft + 8 * a + 4 * hf)) =
            f32x4{S[ft][ct][4 * a], S[ft][ct][4 * a + 1], S[ft][ct][4 * a + 2], S[ft][ct][4 * a + 3]};
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    const float zs = z[ft] + xor32(z[ft]);
    if (hf == 0) {
      cz[(2 * wv) * FB + 32 * ft + l32] = c[ft];
      cz[(2 * wv + 1) * FB + 32 * ft + l32] = zs;
    }
  }
  __syncthreads();
  // the block's shift: the largest of all waves and features (it cancels against the same shift on the query side)
  float cs = -INFINITY;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) cs = fmaxf(cs, cz[2 * w * FB + lane % FB]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) cs = fmaxf(cs, __shfl_xor(cs, o, 64));
  if (tid < kWaves * FB) fac[tid] = fast_exp2(cz[2 * (tid / FB) * FB + tid % FB] - cs);
  __syncthreads();
  if (tid < FB) {
    float zs = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) zs = fmaf(fac[w * FB + tid], cz[(2 * w + 1) * FB + tid], zs);
    zt[(size_t)bh * m + f0 + tid] = zs;
  }
  if (tid == 0) cf[(size_t)bh * nblk + blk] = cs;
  constexpr int PR = FB / 8;   // 16-byte pieces of a row of S^T
  const int col = tid / PR, fa = chain_feature(tid % PR);
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
#pragma unroll
    for (int g = 0; g < 2; ++g)
      acc[g] += *reinterpret_cast<const f32x4*>(fac + w * FB + fa + 8 * g) *
                *reinterpret_cast<const f32x4*>(smem + w * SM::part + part_at<D>(col, fa + 8 * g) * 4);
  const u32x4 o = {pack_bf16(acc[0][0], acc[0][1]), pack_bf16(acc[0][2], acc[0][3]), pack_bf16(acc[1][0], acc[1][1]),
                   pack_bf16(acc[1][2], acc[1][3])};
  const int step = f0 / 16 + tid % PR / 2;   // operand fragments: [16 features][32 columns][lane][8]
  *reinterpret_cast<u32x4*>(St + (size_t)bh * D * m + ((step * CT + col / 32) * 64 + col % 32 + 32 * (tid % 2)) * 8) = o;
}

// ---------------------------------------------------------------------------
// k_short_readout: a wave owns FW features, whose rows of A' and columns of S^T stay in its registers, and 32 tokens a step;
// m / FW waves share the tokens.  U^T[f][tok] = A' X^T, the row shift is the wave's own largest logit, N^T[c][tok] += S^T phi^T;
// the waves' parts of numerator and denominator meet in LDS under the common shift.  Both operands come as contiguous
// kilobytes a wave instruction (read by rows, 32 of them an instruction, they took 3 to 6 us).  36 (b,h) of 509 tokens: 7.5 us
// (k_readout: 10.0), of which 1.5 to 4 are the operands on their way.
// ---------------------------------------------------------------------------
template <int D, int FW, int GW, typename OutT>   // GW: waves that share 32 tokens (m = FW GW)
__global__ __launch_bounds__(64 * GW, 2) void k_short_readout(const unsigned short* __restrict__ Qg, const _Float16* __restrict__ Ah,
                                                         const unsigned short* __restrict__ St, const float* __restrict__ zt,
                                                         const float* __restrict__ cf, OutT* __restrict__ out, int H, int L,
                                                         int steps, int wgs_per_bh) {
  constexpr int m = FW * GW, FB = short_fb<D>(), FT = FW / 32, CT = D / 32, NS = D / 16, NT = 64 * GW;
  constexpr int NCH = D / 4;   // 16-byte pieces of a row of a partial numerator
  __shared__ f32x4 ex[GW][kTok * NCH];
  __shared__ float dm[GW][2][kTok];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64, l32 = lane % 32, hf = lane / 32;
  const int f0 = FW * wv;
  const int wg = xcd_order(blockIdx.x, gridDim.x), bh = wg / wgs_per_bh, h = bh % H;
  const int t_begin = (wg % wgs_per_bh) * steps * kTok;
  const int n_steps = min(steps, (L - t_begin + kTok - 1) / kTok);
  u32x4 xr[NS];
  auto fetch = [&](int t0) {
    const int tok = min(t0 + l32, L - 1);
#pragma unroll
    for (int s = 0; s < NS; ++s) xr[s] = *reinterpret_cast<const u32x4*>(Qg + ((size_t)bh * L + tok) * D + 16 * s + 8 * hf);
  };
  fetch(t_begin);
  half8 af[FT][NS];
  u32x4 sf[FT][2][CT];
  f32x4 zq[FT][4];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      af[ft][s] = *reinterpret_cast<const half8*>(a_frag16<D>(Ah, h, m, f0 + 32 * ft, s, lane));
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        sf[ft][hh][ct] = *reinterpret_cast<const u32x4*>(St + (size_t)bh * D * m + ((((f0 + 32 * ft) / 16 + hh) * CT + ct) * 64 + lane) * 8);
#pragma unroll
    for (int a = 0; a < 4; ++a) zq[ft][a] = *reinterpret_cast<const f32x4*>(zt + (size_t)bh * m + f0 + 32 * ft + 8 * a + 4 * hf);
  }
  const float cw = cf[(size_t)bh * (m / FB) + f0 / FB];
  static_assert(FW <= FB, "one shift a wave");
  for (int i = 0; i < n_steps; ++i) {
    const int t0 = t_begin + i * kTok;
    half8 xf[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) xf[s] = as_half8(bf16x8_to_f16x8(xr[s]));
    if (i + 1 < n_steps) fetch(t0 + kTok);
    f32x16 U[FT] = {};
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int ft = 0; ft < FT; ++ft) U[ft] = mm_f16(af[ft][s], xf[s], U[ft]);
    float mu = -INFINITY;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int v = 0; v < 16; v += 2) mu = max3(mu, U[ft][v], U[ft][v + 1]);
    mu = fmaxf(mu, xor32(mu));
    float den = 0.f;
    f32x16 N[CT] = {};
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        u32x4 pk;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float e0 = fast_exp2(U[ft][8 * hh + 2 * q] - mu), e1 = fast_exp2(U[ft][8 * hh + 2 * q + 1] - mu);
          den = fmaf(e0, zq[ft][2 * hh + q / 2][2 * (q % 2)], den);
          den = fmaf(e1, zq[ft][2 * hh + q / 2][2 * (q % 2) + 1], den);
          pk[q] = pack_bf16(e0, e1);
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) N[ct] = mm_bf16(sf[ft][hh][ct], pk, N[ct]);
      }
    den += xor32(den);
    if (i > 0) __syncthreads();   // the last step's parts have been read
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        ex[wv][l32 * NCH + ((8 * ct + 2 * a + hf) ^ (l32 % NCH))] = f32x4{N[ct][4 * a], N[ct][4 * a + 1], N[ct][4 * a + 2], N[ct][4 * a + 3]};
    if (hf == 0) {
      dm[wv][0][l32] = den;
      dm[wv][1][l32] = mu + cw;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kTok * NCH / NT; ++u) {
      const int k = tid + NT * u, r = k / NCH, ch = k % NCH;
      float mw[GW], mx = -INFINITY;
#pragma unroll
      for (int w = 0; w < GW; ++w) {
        mw[w] = dm[w][1][r];
        mx = fmaxf(mx, mw[w]);
      }
      float d = 0.f;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < GW; ++w) {
        const float f = fast_exp2(mw[w] - mx);
        d = fmaf(f, dm[w][0][r], d);
        o += f * ex[w][r * NCH + (ch ^ (r % NCH))];
      }
      o *= 1.f / d;
      if (t0 + r < L) {
        OutT* dst = out + ((size_t)bh * L + t0 + r) * D + 4 * ch;
        if constexpr (sizeof(OutT) == 4) *reinterpret_cast<f32x4*>(dst) = o;
        else *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
      }
    }
  }
}

struct ShortBufs {
  _Float16* Ah;
  unsigned short* St;
  float *zt, *cf;
};

template <int D, int FW, int GW, typename OutT>
dark_status launch_readout(const Problem& pb, const ShortBufs& b, const void* Q, void* out) {
  const dark_params& p = pb.p;
  const int all = (p.L + kTok - 1) / kTok;
  const long long slots = GW == 4 ? 512 : 256;   // workgroups that the chip holds at once
  int steps = (int)((pb.BH() * all + slots - 1) / slots);
  if (steps > all) steps = all;
  const int wgs = (all + steps - 1) / steps;
  DARK_LAUNCH(KID_READOUT, pb.st, (k_short_readout<D, FW, GW, OutT>), dim3((unsigned)(pb.BH() * wgs)), dim3(64 * GW), 0,
              (const unsigned short*)Q, b.Ah, b.St, b.zt, b.cf, (OutT*)out, p.H, p.L, steps, wgs);
  return DARK_OK;
}

template <int D, typename OutT>
dark_status short_fwd(const Problem& pb, const ShortBufs& b, const void* Q, const void* K, const void* V, const float* M,
                      const float* W, void* out) {
  const dark_params& p = pb.p;
  DARK_TRY(allow_lds(k_short_keys<D>, ShortSmem<D>::total));
  DARK_LAUNCH(KID_KV_REDUCE, pb.st, k_short_keys<D>, dim3((unsigned)(pb.BH() * (p.m / short_fb<D>()))), dim3(NT), ShortSmem<D>::total,
              (const unsigned short*)K, (const unsigned short*)V, M, W, b.Ah, b.St, b.zt, b.cf, p.H, p.L, p.m, p.w_shared,
              std::sqrt(pb.scale));
  if constexpr (D == 128) return launch_readout<128, 32, 8, OutT>(pb, b, Q, out);
  else return p.m == 256 ? launch_readout<64, 64, 4, OutT>(pb, b, Q, out) : launch_readout<64, 64, 8, OutT>(pb, b, Q, out);
}

}  // namespace

// Measured against the general kernels, us general / these.  d = 64, m = 256: one round of workgroups over the CUs (64 (b,h)
// at most) 34 / 29 (L = 1024), 38 / 37.5 (1536), 45 / 49 (2048), with half of the CUs 37 / 35 (1800, 32 (b,h)), 34.8 / 35.7 (2048, 24),
// with fewer 33.5 / 27 (2048, 8); two 31 / 26 (256), 32 / 31 (384), 35 / 36 (512); three
// 29 / 29 (128), 30 / 31 (170).  m = 512: 39 / 35 (1536), three rounds 37 / 35 (160).  d = 128: 45 / 42 (1024), 48 / 50 (1280); two
// 40 / 37 (320), 46 / 51 (512); three 42 / 41 (80), 46 / 48 (140).
bool short_fwd_supported(const Problem& pb) {
  const dark_params& p = pb.p;
  if (p.sched_kv_wgs > 0 || p.sched_ro_wgs > 0) return false;   // a schedule of the general kernels is asked for
  if (pb.m_identity && p.d == 128) return false;   // the general kernels take |k|^2 itself there, not |M' k|^2 with a rounded M'
  const long long blocks = pb.BH() * (p.m / (p.d == 64 ? short_fb<64>() : short_fb<128>())), rounds = (blocks + 255) / 256;   // of k_short_keys
  if (rounds > (p.d == 64 && p.m == 256 ? 2 : 3)) return false;
  const int longest = p.d == 128 ? 1024 : blocks <= 64 ? 2048 : blocks <= 128 ? 1792 : 1536;   // in one round of workgroups
  return p.L * rounds * rounds <= longest;
}

dark_status short_attn_fwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V, const float* M,
                           const float* W, void* out) {
  const dark_params& p = pb.p;
  const size_t BH = (size_t)pb.BH();
  ShortBufs b;
  b.Ah = ar.take<_Float16>((size_t)p.H * p.m * p.d);
  b.St = ar.take<unsigned short>(BH * p.dv * p.m);
  b.zt = ar.take<float>(BH * p.m);
  b.cf = ar.take<float>(BH * (p.m / 32));
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  if (p.d == 64)
    return p.out_dtype == DARK_BF16 ? short_fwd<64, unsigned short>(pb, b, Q, K, V, M, W, out) : short_fwd<64, float>(pb, b, Q, K, V, M, W, out);
  return p.out_dtype == DARK_BF16 ? short_fwd<128, unsigned short>(pb, b, Q, K, V, M, W, out) : short_fwd<128, float>(pb, b, Q, K, V, M, W, out);
}

}  // namespace dark
