// Causal forward of short sequences on the fused MFMA path (gfx950; bf16 inputs, fp32 accumulation), by the kernel values
// themselves.
//
// out_i = sum_{l<=i} a_il v_l / sum_{l<=i} a_il with a_il = phi(q_i) . phi(k_l) (Section 2, before the sum over l is pulled out;
// feature map of Section 4.1).  The slices, prefix states and scan of fused_causal.hip make the work linear in the length, but
// a slice's state of 256 x (dv + 1) numbers is worth 256 keys, and each of the three passes over such states is a launch of 10 to
// 16 us however short the sequence.  Below some thousand positions the tiles of a_il are the smaller work:
//   k_prep        A', M' (fused.hip)
//   k_features    phi_Q, phi_K and V of a tile of 32 positions, as operand fragments in memory; a tile's key shift
//   k_kernel_attn per (b,h, two tiles of queries): a_il tile by tile of 32 keys, N += a V, D += a 1; several waves share a query's keys
// Nothing is kept between the two but bf16 features; the numerator and the denominator use the same kernel values, each two bf16.
#include <cfloat>
#include <cmath>

#include "fused_common.h"

namespace dark {
using namespace fz;
namespace {

constexpr int kTok = 32;     // positions per tile
constexpr int kWaves = 8;
constexpr int NT = 64 * kWaves;
constexpr int kM = 256;      // features: 32 a wave
constexpr int kSteps = kM / 16;
constexpr size_t kTileF = (size_t)kTok * kM;   // features of a tile: [16 features][lane][8]

__device__ __forceinline__ f32x16 mm_f16(half8 a, half8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 mm_bf16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8*>(&a), *reinterpret_cast<bf16x8*>(&b), c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// k_features: a workgroup per tile of 32 positions, 32 features a wave; every lane ends with its position's largest logit over all
// features (queries: the row's shift; keys: less the norm, for the tile's shift), so that one exchange through LDS serves
// shifts and norms.  The accumulators, packed, are the fragments that k_kernel_attn multiplies.
// Bound by the operands on their way (64 KB of A' a workgroup): 16 (b,h) of 777 positions, d = 128: 9.9 us, 4.5 with the chip empty.
// ct: per tile its key shift, and whether V has an infinity or NaN there.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool nonfinite_lo(unsigned w) { return (w & 0x7f80u) == 0x7f80u; }   // two bf16 in w
__device__ __forceinline__ bool nonfinite_hi(unsigned w) { return (w & 0x7f800000u) == 0x7f800000u; }
__device__ __forceinline__ u32x4 finite_part(u32x4 v) {   // eight bf16, those that are not finite as zero
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] &= (nonfinite_lo(v[i]) ? 0u : 0xffffu) | (nonfinite_hi(v[i]) ? 0u : 0xffff0000u);
  return v;
}

template <int D>
__global__ __launch_bounds__(NT, 4) void k_features(const unsigned short* __restrict__ Qg, const unsigned short* __restrict__ Kg,
                                                    const unsigned short* __restrict__ Vg, const _Float16* __restrict__ Ah,
                                                    const _Float16* __restrict__ Mh, unsigned short* __restrict__ Fq,
                                                    unsigned short* __restrict__ Fk, unsigned short* __restrict__ Vf,
                                                    float* __restrict__ ct, int BH, int H, int L, int nt) {
  constexpr int NS = D / 16, AS = D + 8, CPR = D / 8, NCH = kTok * CPR, CT = D / 32;
  __shared__ __attribute__((aligned(16))) _Float16 xs[2][kTok * AS];       // keys, queries
  __shared__ __attribute__((aligned(16))) unsigned short vs[kTok * D];
  __shared__ __attribute__((aligned(16))) float np[kTok][8], mx[2][kWaves][kTok];
  __shared__ int odd[kWaves];   // the wave's piece of V has an infinity or NaN
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const int l32 = lane % 32, hf = lane / 32, l16 = lane % 16, g16 = lane / 16;
  const int bh = blockIdx.x % BH, t = blockIdx.x / BH, h = bh % H, t0 = t * kTok;   // neighbours in different (b,h), as in k_kernel_attn
  u32x4 kr = {}, qr = {}, vr = {};
  if (tid < NCH) {
    const size_t at = ((size_t)bh * L + min(t0 + tid / CPR, L - 1)) * D + 8 * (tid % CPR);
    kr = *reinterpret_cast<const u32x4*>(Kg + at);
    qr = *reinterpret_cast<const u32x4*>(Qg + at);
    vr = *reinterpret_cast<const u32x4*>(Vg + at);
  }
  half8 af[NS], mf[D / 32];
#pragma unroll
  for (int s = 0; s < NS; ++s) af[s] = *reinterpret_cast<const half8*>(a_frag16<D>(Ah, h, kM, 32 * wv, s, lane));
  const bool normer = wv < D / 16;   // sixteen rows of M' each
#pragma unroll
  for (int s = 0; s < D / 32; ++s)
    mf[s] = *reinterpret_cast<const half8*>(Mh + ((size_t)h * D + 16 * (wv % (D / 16)) + l16) * D + 32 * s + 8 * g16);
  if (tid < NCH) {
    const int row = tid / CPR, ch = tid % CPR;
    *reinterpret_cast<u32x4*>(xs[0] + row * AS + 8 * ch) = bf16x8_to_f16x8(kr);
    *reinterpret_cast<u32x4*>(xs[1] + row * AS + 8 * ch) = bf16x8_to_f16x8(qr);
    *reinterpret_cast<u32x4*>(vs + row * D + 8 * (ch ^ v_swz<2 * D>(row))) = vr;
  }
  bool nf = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) nf |= nonfinite_lo(vr[i]) | nonfinite_hi(vr[i]);
  nf = __any(nf);
  if (lane == 0) odd[wv] = nf;
  __syncthreads();
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  if (normer) {
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
      f32x4 acc = zero4;   // x~[row 16 wv + 4 g16 + i][token 16 tb + l16]
#pragma unroll
      for (int s = 0; s < D / 32; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(mf[s], *reinterpret_cast<const half8*>(xs[0] + (16 * tb + l16) * AS + 32 * s + 8 * g16), acc, 0, 0, 0);
      float sq = acc[0] * acc[0];
      sq = fmaf(acc[1], acc[1], sq);
      sq = fmaf(acc[2], acc[2], sq);
      sq = fmaf(acc[3], acc[3], sq);
      sq += xor16(sq);
      sq += xor32(sq);
      if (g16 == 0) np[16 * tb + l16][wv] = sq;
    }
  }
  f32x16 U[2] = {};   // this wave's features (registers) of the tile's keys, queries (lane)
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int x = 0; x < 2; ++x) U[x] = mm_f16(af[s], *reinterpret_cast<const half8*>(xs[x] + l32 * AS + 16 * s + 8 * hf), U[x]);
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    float m0 = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; v += 2) m0 = max3(m0, U[x][v], U[x][v + 1]);
    m0 = fmaxf(m0, xor32(m0));
    if (hf == 0) mx[x][wv][l32] = m0;
  }
  __syncthreads();
  float mk = mx[0][0][l32], mq = mx[1][0][l32], n = 0.f;
#pragma unroll
  for (int w = 1; w < kWaves; ++w) {
    mk = fmaxf(mk, mx[0][w][l32]);
    mq = fmaxf(mq, mx[1][w][l32]);
  }
#pragma unroll
  for (int w = 0; w < D / 16; w += 4) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(&np[l32][w]);
    n += (a[0] + a[1]) + (a[2] + a[3]);
  }
  if (t0 + l32 >= L) n = INFINITY;   // rows past the end: features exactly zero
  float c = mk - n;                  // the tile's shift: its largest key logit over all features
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) c = fmaxf(c, __shfl_xor(c, o, 64));
  c = fmaxf(c, -FLT_MAX);
  if (tid == 0) {
    int any = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) any |= odd[w];
    *reinterpret_cast<u32x2*>(ct + 2 * ((size_t)bh * nt + t)) = u32x2{__float_as_uint(c), (unsigned)any};
  }
  unsigned short* dst[2] = {Fk, Fq};
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 pk;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float u0 = U[x][8 * hh + 2 * q], u1 = U[x][8 * hh + 2 * q + 1];
        pk[q] = x == 0 ? pack_bf16(fast_exp2((u0 - n) - c), fast_exp2((u1 - n) - c)) : pack_bf16(fast_exp2(u0 - mq), fast_exp2(u1 - mq));
      }
      *reinterpret_cast<u32x4*>(dst[x] + ((size_t)bh * nt + t) * kTileF + ((2 * wv + hh) * 64 + lane) * 8) = pk;
    }
  }
  if (wv < 2 * CT) {   // V fragment (16 positions hh, 32 columns ct): column l32, positions 4 hf + [0,4) and those + 8
    const int hh = wv / CT, cb = wv % CT, jj = l32 % 16, tl = 16 * hh + 4 * hf + jj / 4, chunk = 4 * cb + 2 * (l32 / 16) + (jj % 4) / 2;
    const unsigned short* r = vs + tl * D + 8 * (chunk ^ v_swz<2 * D>(tl)) + 4 * (jj % 2);
    const u32x2 lo = lds_read_tr16(r), hi = lds_read_tr16(r + 8 * D);
    *reinterpret_cast<u32x4*>(Vf + ((size_t)bh * nt + t) * kTok * D + (wv * 64 + lane) * 8) = u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
}

// Waves of the far tile of queries (far + 1 tiles of keys; near + 1 are the others'), so that none takes more than `steps` =
// ceil((far + near + 2) / kWaves) tiles of keys, or one more where that division does not come out.  One more is enough for steps
// <= 8 (x / (n + 1) + y / (n + 1), each rounded up, is at most 10 n / (n + 1) < 9); that it is for every number of tiles taken
// here, the one of nine steps (64 tiles) among them, the assertion below counts out.
__host__ __device__ constexpr int prompt_far_waves(int far, int near, int steps) {
  int wf = far / steps + 1;
  if (wf + near / steps + 1 > kWaves) wf = far / (steps + 1) + 1;
  return wf;
}
constexpr bool prompt_split_ok(int nt) {
  for (int i = 0; 2 * i < nt - 1; ++i) {
    const int far = nt - 1 - i, s = nt / kWaves + 1, wf = prompt_far_waves(far, i, s);
    if (wf < 1 || wf >= kWaves || far / wf > s || i / (kWaves - wf) > s) return false;   // at most s + 1 tiles a wave
  }
  return true;
}
constexpr bool prompt_splits_ok(int most) {
  for (int nt = 1; nt <= most; ++nt)
    if (!prompt_split_ok(nt)) return false;
  return true;
}
constexpr int kMaxTiles = 64;
static_assert(prompt_splits_ok(kMaxTiles), "every wave's share of the key tiles");

// ---------------------------------------------------------------------------
// k_kernel_attn: kernel values P^T[key][query] of 32 x 32 by sixteen MFMAs over the features, the wave's running scalar shift C (a tile's
// shift c enters as the factor 2^(c - C); the queries' own shifts cancel), N^T += V^T P^T, D += 1 P^T.  A workgroup takes two
// tiles of queries, which its eight waves (two a SIMD) share.
// PAIRS: a tile from the back and its counterpart from the front, nt + 1 tiles of kernel values whichever they are, the
// waves dealt to the two in proportion: no workgroup is longer than another (25 tiles: 4 steps instead of 7).  A wave's keys pass
// through its own sixteen kilobytes of LDS, the next tile's on their way while this one's products with V run; the loop has
// no barrier.  Bound by the longest wave: 16 (b,h) of 777 positions 14.6 us, with neighbours 18.3 (the whole call 28 and 31.6).
// Otherwise: neighbouring tiles, four waves each, every fourth key tile a wave.  The two waves of one kg share its key tile
// through LDS, each bringing half of it, so that the keys are read half as often: the better one where the workgroups are more
// than the chip holds and the sum of them counts.  A step of four tiles takes 1.7 us, of which the matrix pipe 0.8, the rest LDS and
// the chain from scores to products.  Measured besides: four waves of 64 queries with 512 registers (slower, and spills once the
// scores of the next tile are formed beside this one's products).
// ---------------------------------------------------------------------------
constexpr int kKW = 4;   // waves of a tile of queries (neighbours)

template <int D, bool PAIRS, typename OutT>
__global__ __launch_bounds__(NT, 2) void k_kernel_attn(const unsigned short* __restrict__ Fq, const unsigned short* __restrict__ Fk,
                                                       const unsigned short* __restrict__ Vf, const float* __restrict__ ct,
                                                       OutT* __restrict__ out, int BH, int L, int nt, int steps) {
  constexpr int CT = D / 32, NCH = D / 4;
  // key tiles [16 features][lane][8]: one of every wave, or two sets of four; after the last the waves' numerators
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float dm[kWaves][kTok], cw[kWaves];
  f32x4* ex = reinterpret_cast<f32x4*>(smem);
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64), l32 = lane % 32, hf = lane / 32;
  // Workgroups are dealt to the eight XCDs in turn.  Neighbours have different (b,h), so that of an even number of them each
  // XCD and its L2 sees a half, a quarter or an eighth.  Of an odd number it would see all, which from some ten megabytes of
  // features on are more than an L2 holds: there every XCD takes a run of workgroups, (b,h) after (b,h).  us, dealt in turn / in
  // runs: 9 (b,h) 46.8 / 38.2 (L = 1792), 33.5 / 33.7 (1200); 13 40.9 / 33.4 (1200), 30.1 / 29.7 (800); 15 40.2 / 32.4 (1050);
  // 21 37.9 / 32.3 (700); 49 39.4 / 35.9 (300); 7 43.7 / 40.3 (2016), 35.5 / 36.0 (1500), 20.4 / 19.8 (300); 5 39.1 / 39.7
  // (2048), 28.7 / 27.8 (1000); 3 36.4 / 36.3 (2048), 18.1 / 18.5 (257); 1 33.3 / 34.0 (2048), 21.6 / 21.9 (700): never more than
  // 2 % behind.  An even number, 12 of 1152, dealt in runs: 32.5 / 34.3.
  int bh = blockIdx.x % BH, wg = blockIdx.x / BH;
  if (PAIRS && BH % 2 != 0) {
    const int n = gridDim.x, x = blockIdx.x % 8, at = x * (n / 8) + min(x, n % 8) + blockIdx.x / 8, per = n / BH;
    bh = at / per;
    wg = at % per;
  }
  // waves [0, wf) take the tile of queries `far`, the others `near` (PAIRS: the middle one of an odd number is all the waves';
  // neighbours: the longest rows first, far is past the end in the last of an odd number)
  const int near = PAIRS ? wg : 2 * ((nt + 1) / 2 - 1 - wg), far = PAIRS ? nt - 1 - wg : near + 1;
  const int wf = !PAIRS ? kKW : far == near ? kWaves : prompt_far_waves(far, near, steps);
  const bool is_far = wv < wf;
  const int tq = is_far ? far : near, kg = is_far ? wv : wv - wf, stride = is_far ? wf : kWaves - wf;
  const size_t tile0 = (size_t)bh * nt;
  f32x16 N[CT] = {}, den = {};   // registers = columns (den: every register alike), lane = query
  float C = -INFINITY;           // a wave without a tile counts for nothing
  const int t_last = min(far, nt - 1), g = is_far ? 0 : 1;   // neighbours: the last key tile of the workgroup, this wave's half
  auto keys = [&](int i) { return smem + (PAIRS ? wv : (i % 2) * kKW + kg) * kSteps * 1024; };
  auto dma_k = [&](int i) {   // keys of step i
    const int t = PAIRS ? kg + stride * i : min(kKW * i + kg, t_last), s0 = PAIRS ? 0 : kSteps / 2 * g;
    const unsigned short* src = Fk + (tile0 + t) * kTileF + (s0 * 64 + lane) * 8;
    unsigned char* dst = keys(i) + s0 * 1024;
#pragma unroll
    for (int s = 0; s < (PAIRS ? kSteps : kSteps / 2); ++s) dma16_to_lds(src + 512 * s, dst + 1024 * s);
  };
  const int n_steps = PAIRS ? (kg <= tq ? (tq - kg) / stride + 1 : 0) : t_last / kKW + 1;   // PAIRS: this wave's
  if (!PAIRS) dma_k(0);
  u32x4 qf[kSteps];
  if (n_steps > 0) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s) qf[s] = *reinterpret_cast<const u32x4*>(Fq + (tile0 + min(tq, nt - 1)) * kTileF + (64 * s + lane) * 8);
    if (PAIRS) {
      __builtin_amdgcn_sched_barrier(0);
      dma_k(0);
    }
  }
  const u32x4 ones = {kOnesBf16x2, kOnesBf16x2, kOnesBf16x2, kOnesBf16x2};
  for (int i = 0; i < n_steps; ++i) {   // (wave-uniform)
    const int t = kg + stride * i, tc = min(t, t_last);
    wait_vmcnt0();
    if (PAIRS) {   // this wave's keys are there
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    } else {
      __syncthreads();   // this step's keys are there, the other set has been read
    }
    u32x4 vf[2][CT];
#pragma unroll
    for (int j = 0; j < 2 * CT; ++j) vf[j / CT][j % CT] = *reinterpret_cast<const u32x4*>(Vf + (tile0 + tc) * kTok * D + (j * 64 + lane) * 8);
    const u32x2 ctile = *reinterpret_cast<const u32x2*>(ct + 2 * (tile0 + tc));
    const float c = __uint_as_float(ctile[0]);
    if (!PAIRS) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + 1 < n_steps) dma_k(i + 1);
      if (t > tq) continue;   // wave-uniform
    }
    const u32x4* kt = reinterpret_cast<const u32x4*>(keys(i)) + lane;
    // the fragments are requested four products ahead of their use
    constexpr int PF = 4;
    u32x4 kf[PF];
#pragma unroll
    for (int s = 0; s < PF; ++s) kf[s] = kt[64 * s];
    __builtin_amdgcn_sched_barrier(0);
    f32x16 P = {};   // registers = keys, lane = query
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      P = mm_bf16(kf[s % PF], qf[s], P);
      if (s + PF < kSteps) kf[s % PF] = kt[64 * (s + PF)];
      __builtin_amdgcn_sched_barrier(0);
    }
    if (PAIRS) {
      // V is there before the next keys are requested: the counter of loads in flight is one for both
#pragma unroll
      for (int j = 0; j < 2 * CT; ++j) asm volatile("" : "+v"(vf[j / CT][j % CT]));
      if (i + 1 < n_steps) dma_k(i + 1);   // the last of these keys have entered their product
    }
    if (c > C + kRaise || i == 0) {   // wave-uniform; after the first tile rare
      const float f = i == 0 ? 0.f : fast_exp2(C - c);
      C = c;
      den *= f;
#pragma unroll
      for (int b = 0; b < CT; ++b) N[b] *= f;
    }
    P *= fast_exp2(c - C);
    if (t == tq) {
#pragma unroll
      for (int v = 0; v < 16; ++v) P[v] = 8 * (v / 4) + 4 * hf + (v % 4) <= l32 ? P[v] : 0.f;
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      // Kernel values as two bf16 each, sixteen bits: rounded to one they alone add a quarter to the result's error (2.2e-3 instead
      // of 1.7e-3; slices and scan 2.0e-3).  N and D take the same numbers, so that N / D is a convex combination of value rows.
      u32x4 p0, p1;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float a = P[8 * hh + 2 * q], b = P[8 * hh + 2 * q + 1];
        p0[q] = pack_bf16(a, b);
        p1[q] = pack_bf16(a - __uint_as_float(p0[q] << 16), b - __uint_as_float(p0[q] & 0xffff0000u));
      }
#pragma unroll
      for (int b = 0; b < CT; ++b) N[b] = mm_bf16(vf[hh][b], p0, N[b]);
      // The second number is zero or negative half of the time: an infinity of V meets the first one only, and stays one.
      if (__builtin_amdgcn_readfirstlane(ctile[1]) != 0) {   // (wave-uniform, rare)
#pragma unroll
        for (int b = 0; b < CT; ++b) vf[hh][b] = finite_part(vf[hh][b]);
      }
#pragma unroll
      for (int b = 0; b < CT; ++b) N[b] = mm_bf16(vf[hh][b], p1, N[b]);
      den = mm_bf16(ones, p1, mm_bf16(ones, p0, den));
    }
  }
  static_assert(kTok * NCH * 16 == kSteps * 1024, "PAIRS: a wave's numerator takes the place of its own keys, which it has read");
  if (!PAIRS) __syncthreads();   // the keys have been read
#pragma unroll
  for (int b = 0; b < CT; ++b)
#pragma unroll
    for (int a = 0; a < 4; ++a)
      ex[wv * kTok * NCH + l32 * NCH + ((8 * b + 2 * a + hf) ^ (l32 % NCH))] = f32x4{N[b][4 * a], N[b][4 * a + 1], N[b][4 * a + 2], N[b][4 * a + 3]};
  if (hf == 0) dm[wv][l32] = den[0];
  if (lane == 0) cw[wv] = C;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2 * kTok * NCH / NT; ++u) {
    constexpr int kHalf = kTok * NCH / NT;   // pieces of a tile a thread
    static_assert(kTok * NCH % NT == 0, "a piece of a thread is the far tile's or the near one's for all of them");
    if (PAIRS && u >= kHalf && far == near) break;
    const int k = tid + NT * (u % kHalf), r = k / NCH, ch = k % NCH;
    const int w0 = u < kHalf ? 0 : wf, w1 = u < kHalf ? wf : kWaves, tok = (u < kHalf ? far : near) * kTok + r;
    float Cm = -INFINITY;
    for (int w = w0; w < w1; ++w) Cm = fmaxf(Cm, cw[w]);
    float d = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    for (int w = w0; w < w1; ++w) {
      const float f = fast_exp2(cw[w] - Cm);
      d = fmaf(f, dm[w][r], d);
      o += f * ex[w * kTok * NCH + r * NCH + (ch ^ (r % NCH))];
    }
    o *= 1.f / d;
    if (tok < L) {
      OutT* dst = out + ((size_t)bh * L + tok) * D + 4 * ch;
      if constexpr (sizeof(OutT) == 4) *reinterpret_cast<f32x4*>(dst) = o;
      else *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
    }
  }
}
constexpr size_t kAttnLds = (size_t)kWaves * kSteps * 1024;
static_assert(kAttnLds >= (size_t)kWaves * kTok * 128 * 4, "the numerators take the keys' place");

// One round of workgroups of k_kernel_attn over the CUs.
inline bool one_round(long long BH, long long nt) { return BH * ((nt + 1) / 2) <= 256; }

struct PromptBufs {
  _Float16 *Ah, *Mh;
  unsigned short *Fq, *Fk, *Vf;
  float* ct;
  int nt;
};

template <int D, typename OutT>
dark_status prompt_fwd(const Problem& pb, const PromptBufs& b, const void* Q, const void* K, const void* V, void* out) {
  const dark_params& p = pb.p;
  DARK_LAUNCH(KID_FEATURIZE, pb.st, k_features<D>, dim3((unsigned)(pb.BH() * b.nt)), dim3(NT), 0, (const unsigned short*)Q,
              (const unsigned short*)K, (const unsigned short*)V, b.Ah, b.Mh, b.Fq, b.Fk, b.Vf, b.ct, (int)pb.BH(), p.H, p.L, b.nt);
  // Pairs of equal length where one round of workgroups over the CUs holds them all and the longest row has two steps or more, us
  // neighbours / pairs: one head 15.5 / 15.9 (L = 128), 17.7 / 17.1 (256), 25.7 / 21.7 (700), 32.6 / 26.2 (1152); 16 (b,h) 15.9 / 16.9
  // (128), 19.7 / 18.7 (257), 31.6 / 27.6 (777), in two rounds 39 / 46 (1152); 64 (b,h) in two 29 / 34 (320).
  const long long wgs = pb.BH() * ((b.nt + 1) / 2);
  const bool pairs = one_round(pb.BH(), b.nt) && b.nt >= kWaves;
  auto kern = pairs ? k_kernel_attn<D, true, OutT> : k_kernel_attn<D, false, OutT>;
  DARK_TRY(allow_lds(kern, kAttnLds));
  DARK_LAUNCH(KID_CAUSAL_SCAN, pb.st, kern, dim3((unsigned)wgs), dim3(NT), kAttnLds, b.Fq, b.Fk, b.Vf, b.ct, (OutT*)out,
              (int)pb.BH(), p.L, b.nt, b.nt / kWaves + 1);
  return DARK_OK;
}

}  // namespace

// Against the slices and the scan, us: one head 23 / 15 (L = 17), 30 / 22 (700), 34 / 26 (1152), 36 / 34 (2048); 7 (b,h) 43.5 / 42.3
// (2016), 9 (b,h) 46.8 / 41.6 (1792), 16 (b,h) 32 / 17 (128), 41 / 28 (777): one round of workgroups, any length that the split of the
// waves is for.  More workgroups than CUs: 16 (b,h) 47 / 39 (1152); 36 (b,h) 54 / 49 (864); 64 (b,h) 64 / 53 (640), 77 / 90
// (1024); 256 (b,h) 95 / 85 (320), 112 / 135 (416); 4096 (b,h) 704 / 135 (17), 788 / 238 (64): the tiles of a_il count.
bool prompt_supported(const Problem& pb) {
  const dark_params& p = pb.p;
  // d = 64 keeps the scan: its training form hands the prefix states to the backward pass and returns the same bits.  So does the
  // identity geometry, whose key norms are |k|^2 itself there, not |M' k|^2 with a rounded M'
  if (p.d != 128 || pb.m_identity || pb.small_ws || p.sched_cs_wgs > 0 || p.sched_cs_state > 0 || p.sched_kv_wgs > 0) return false;
  const long long nt = (p.L + kTok - 1) / kTok;
  if (one_round(pb.BH(), nt)) return nt <= kMaxTiles;
  return nt <= 36 && pb.BH() * nt * nt <= 28000;
}

dark_status prompt_attn_fwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V, const float* M,
                            const float* W, void* out) {
  const dark_params& p = pb.p;
  const size_t BH = (size_t)pb.BH();
  PromptBufs b;
  b.nt = (p.L + kTok - 1) / kTok;
  b.Ah = ar.take<_Float16>((size_t)p.H * p.m * p.d);
  b.Mh = ar.take<_Float16>((size_t)p.H * p.r * p.d);
  b.Fq = ar.take<unsigned short>(BH * b.nt * kTileF);
  b.Fk = ar.take<unsigned short>(BH * b.nt * kTileF);
  b.Vf = ar.take<unsigned short>(BH * b.nt * kTok * p.d);
  b.ct = ar.take<float>(BH * b.nt * 2);
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  DARK_TRY(fused_launch_prep(pb, M, W, b.Ah, b.Mh, true));
  return p.out_dtype == DARK_BF16 ? prompt_fwd<128, unsigned short>(pb, b, Q, K, V, out) : prompt_fwd<128, float>(pb, b, Q, K, V, out);
}

}  // namespace dark
