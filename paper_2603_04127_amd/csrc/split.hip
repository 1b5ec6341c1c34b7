// fp32 path for d = r = dv = 64 and m a multiple of 64: bidirectional attention that never writes a feature matrix, in
// fp32 accuracy on the bf16 matrix cores (three-plane operands, split.h).  The general fp32 kernels (generic.hip), which
// serve every other shape, write logits and features to memory and pass over them several times; at B H L = 24,576,
// m = 256 they take 165 us in thirteen launches.
//
// Per (b,h), everything in the log2 domain (alpha = sqrt(scale), Section 4.1 and Appendix B):
//   A' = alpha log2e W M,  n'(x) = |alpha sqrt(log2e / 2) M x|^2
//   phi_K,lj = exp2(k_l . A'_j - n'(k_l) - c_j),  phi_Q,ij = exp2(q_i . A'_j + c_j - mu_i)
// with a running shift per feature and slice of the keys (brought to c_j by the merge) and a running shift per query.
//
// Kernels:
//   k_sp_prep     planes of A' for every head; n' of every key
//   k_sp_states   per (b,h, slice, 256 features): S_j += phi_K,lj v_l, z_j += phi_K,lj; a wave owns 32 features
//   k_sp_merge    fixed-order merge of the slice states, planes of S^T for the readout
//   k_sp_readout  per (b,h, 128 queries): out = phi_Q S / phi_Q z; a wave owns 32 queries
// Measured (fp32 inputs, against the general kernels): B H L = 24,576, m = 256: 7 + 16 + 6 + 17 us, 45 us a call
// (165 before); B H L = 393,216: 37 + 186 + 7 + 163 us (1.72 ms before); one head, L = 256, m = 64: 23 us, the launches
// (77 before).
#include <cmath>

#include "split.h"

namespace dark {
using namespace sp;
namespace {

constexpr int kD = 64;       // d = r = dv
constexpr int kTok = 32;     // tokens per tile
constexpr int kGrp = 64;     // features per group of the readout
constexpr int LDX = 72;      // row pitch (16-bit elements) of LDS tiles with 64 columns
constexpr float kTailNorm = 1e30f;  // norm of the rows past the end: their features are exp2(-1e30) = 0
// A shift is raised once a logit exceeds it by 2^kRaise: features stay below that, sums over any length far inside
// the fp32 range, and what lies more than 2^-(126 - kRaise) below the largest key of a feature vanishes.
static_assert(kRaise <= 32.f, "sums of features must stay far from the end of the fp32 range");

// ---------------------------------------------------------------------------
// k_sp_prep: blocks [0, H nA): sixteen rows of A' of one head, fp32 sums over the rows of M in LDS, stored as planes
// [H][3][m][64].  The other blocks: a wave forms n' of tiles of 32 keys, x~^T[r][tok] = M' X^T by MFMA with M' as
// planes in registers, the sum of squares over registers.
// ---------------------------------------------------------------------------
template <int NP>
__global__ __launch_bounds__(256) void k_sp_prep(const float* __restrict__ M, const float* __restrict__ W,
                                                 us* __restrict__ Apl, const void* __restrict__ Kg,
                                                 float* __restrict__ nrm, int H, int L, int m, int w_shared,
                                                 float alpha, int n_tiles, int tiles_per_wave) {
  __shared__ __attribute__((aligned(16))) float Ws[16][kD + 4];
  __shared__ __attribute__((aligned(16))) float Mt[kD][kD];
  const int tid = threadIdx.x;
  const int nA = m / 16;
  if ((int)blockIdx.x < H * nA) {
    const int h = blockIdx.x / nA, j0 = 16 * (blockIdx.x % nA);
    const f32x4* Mp = reinterpret_cast<const f32x4*>(M + (size_t)h * kD * kD);
    const float* w = W + (w_shared ? 0 : (size_t)h * m * kD) + (size_t)j0 * kD;
    f32x4 mv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) mv[u] = Mp[tid + 256 * u];
    const f32x4 wv = reinterpret_cast<const f32x4*>(w)[tid];
#pragma unroll
    for (int u = 0; u < 4; ++u) reinterpret_cast<f32x4*>(&Mt[0][0])[tid + 256 * u] = mv[u];
    *reinterpret_cast<f32x4*>(&Ws[tid / 16][4 * (tid % 16)]) = wv;
    __syncthreads();
    const int jj = tid / 16, cq = tid % 16;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int t = 0; t < kD; ++t) {
      const float wt = Ws[jj][t];
      const f32x4 mt = *reinterpret_cast<const f32x4*>(&Mt[t][4 * cq]);
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x] = fmaf(wt, mt[x], acc[x]);
    }
    acc *= alpha * kLog2e;
    unsigned p[2][3];
    split_pair(acc[0], acc[1], p[0][0], p[0][1], p[0][2]);
    split_pair(acc[2], acc[3], p[1][0], p[1][1], p[1][2]);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl)
      *reinterpret_cast<u32x2*>(Apl + (((size_t)h * 3 + pl) * m + j0 + jj) * kD + 4 * cq) = u32x2{p[0][pl], p[1][pl]};
    return;
  }
  const int lane = tid % 64, l32 = lane % 32, hf = lane / 32;
  const int wave = ((int)blockIdx.x - H * nA) * 4 + tid / 64;
  const int nt = (L + kTok - 1) / kTok;
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float fm = alpha * sqrtf(0.5f * kLog2e);
  u32x4 mp[2][4][3];
  int cur_h = -1;
  for (int i = 0; i < tiles_per_wave; ++i) {
    const int tile = wave * tiles_per_wave + i;
    if (tile >= n_tiles) return;
    const int bh = tile / nt, tok = (tile % nt) * kTok + l32, h = bh % H;
    Raw8<NP> xr[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) xr[s].load(Kg, ((size_t)bh * L + min(tok, L - 1)) * kD + 16 * s + 8 * hf);
    if (h != cur_h) {
      cur_h = h;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const f32x4* mr = reinterpret_cast<const f32x4*>(M + ((size_t)h * kD + 32 * rb + l32) * kD + 16 * s + 8 * hf);
          split8(mr[0] * fm, mr[1] * fm, mp[rb][s]);
        }
    }
    f32x16 x[2] = {zero16, zero16};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 xf[NP];
      xr[s].planes(xf);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) x[rb] = mm_all(mp[rb][s], xf, x[rb]);
    }
    float n = 0.f;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int v = 0; v < 16; ++v) n = fmaf(x[rb][v], x[rb][v], n);
    n += xor32(n);
    if (hf == 0 && tok < L) nrm[(size_t)bh * L + tok] = n;
  }
}

// ---------------------------------------------------------------------------
// k_sp_states: the state of one slice.  NW waves of 32 features each; tiles of 32 tokens staged as planes, two
// buffers, one barrier per tile (the next tile is requested before, and stored after, the products of this one).
// U[tok][f] = X A'^T leaves a feature per lane and tokens along the registers, the contraction index of phi^T V, so
// the split features go from the accumulator straight into the second product; V fragments by transposing reads.
// Matrix-pipe bound with fp32 inputs (48 MFMAs = 1536 cycles per wave and tile against ~220 vector instructions).
// ---------------------------------------------------------------------------
template <int NP>
struct StSmem {
  static constexpr size_t x_bytes = (size_t)NP * kTok * LDX * 2;
  static constexpr size_t v_bytes = (size_t)NP * kTok * kD * 2;
  static constexpr size_t n_bytes = kTok * 4;
  static constexpr size_t buf = x_bytes + v_bytes + n_bytes;
  static constexpr size_t total = 2 * buf;
};

template <int NP, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_sp_states(const void* __restrict__ Kg, const void* __restrict__ Vg,
                                                          const us* __restrict__ Apl, const float* __restrict__ nrm,
                                                          float* __restrict__ Spart, float* __restrict__ zpart,
                                                          float* __restrict__ cpart, int H, int L, int m, int P,
                                                          int slice_len, int nfb) {
  using SM = StSmem<NP>;
  constexpr int NT = 64 * NW, NTASK = 512 / NT;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const int l32 = lane % 32, hf = lane / 32;
  const int fb = blockIdx.x % nfb, work = blockIdx.x / nfb;
  const int bh = work / P, p = work % P, h = bh % H;
  const int tok_begin = p * slice_len, tok_end = min(L, tok_begin + slice_len);
  const int ntile = (tok_end - tok_begin + kTok - 1) / kTok;
  const int f0 = fb * 256 + wv * 32;
  const bool active = f0 < m;   // the last block of features may be short

  Raw8<NP> st[NTASK];
  float nst = 0.f;
  // task i: eight elements of a row of K (i < 256) or of V
  auto fetch = [&](int t) {
#pragma unroll
    for (int u = 0; u < NTASK; ++u) {
      const int i = tid + NT * u, c = i % 256;
      const int tok = min(tok_begin + t * kTok + c / 8, tok_end - 1);
      st[u].load(i < 256 ? Kg : Vg, ((size_t)bh * L + tok) * kD + 8 * (c % 8));
    }
    if (tid < kTok) {
      const int tok = tok_begin + t * kTok + tid;
      nst = tok < tok_end ? nrm[(size_t)bh * L + tok] : kTailNorm;
    }
  };
  auto store = [&](int t) {
    unsigned char* base = smem + (t & 1) * SM::buf;
#pragma unroll
    for (int u = 0; u < NTASK; ++u) {
      const int i = tid + NT * u, c = i % 256, row = c / 8, ch = c % 8;
      u32x4 pl[NP];
      st[u].planes(pl);
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        if (i < 256) *reinterpret_cast<u32x4*>(base + (q * kTok + row) * LDX * 2 + 16 * ch) = pl[q];
        else *reinterpret_cast<u32x4*>(base + SM::x_bytes + (q * kTok + row) * 128 + 16 * (ch ^ v_swz<128>(row))) = pl[q];
      }
    }
    if (tid < kTok) reinterpret_cast<float*>(base + SM::x_bytes + SM::v_bytes)[tid] = nst;
  };

  fetch(0);
  u32x4 af[4][3];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int q = 0; q < 3; ++q)
      af[s][q] = *reinterpret_cast<const u32x4*>(Apl + (((size_t)h * 3 + q) * m + min(f0, m - 32) + l32) * kD + 16 * s + 8 * hf);
  store(0);
  __syncthreads();

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 S[2] = {zero16, zero16};
  float z = 0.f, c = 0.f;
  // V fragment: value column 32 ct + l32, tokens 16 hh + 4 hf + [0,4) and 16 hh + 8 + 4 hf + [0,4) (chain order)
  const int jj = l32 % 16, tl = 4 * hf + jj / 4, kq = 2 * (l32 / 16) + (jj % 4) / 2;
  unsigned voff[2];
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) voff[ct] = tl * 128 + 16 * ((kq + 4 * ct) ^ v_swz<128>(tl)) + 8 * (jj % 2);

  for (int t = 0; t < ntile; ++t) {
    if (t + 1 < ntile) fetch(t + 1);
    if (active) {
      const unsigned char* base = smem + (t & 1) * SM::buf;
      f32x16 U = zero16;
      {
        u32x4 xf[4][NP];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int q = 0; q < NP; ++q)
            xf[s][q] = *reinterpret_cast<const u32x4*>(base + (q * kTok + l32) * LDX * 2 + 32 * s + 16 * hf);
#pragma unroll
        for (int s = 0; s < 4; ++s) U = mm_low(xf[s], af[s], U);
#pragma unroll
        for (int s = 0; s < 4; ++s) U = mm(xf[s][0], af[s][0], U);
      }
      const float* nl = reinterpret_cast<const float*>(base + SM::x_bytes + SM::v_bytes);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 n4 = *reinterpret_cast<const f32x4*>(nl + 8 * a + 4 * hf);
#pragma unroll
        for (int j = 0; j < 4; ++j) U[4 * a + j] -= n4[j] + c;
      }
      float mx = U[0];
#pragma unroll
      for (int v = 1; v < 15; v += 2) mx = max3(mx, U[v], U[v + 1]);
      mx = fmaxf(mx, U[15]);
      mx = fmaxf(mx, xor32(mx));
      if (t == 0 || __any(mx > kRaise)) {   // set the shift, or raise it (rare)
        const float delta = (t == 0 || mx > kRaise) ? mx : 0.f;
        c += delta;
#pragma unroll
        for (int v = 0; v < 16; ++v) U[v] -= delta;
        if (t > 0) {
          const float f = fast_exp2(-delta);
          z *= f;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float fr = __shfl(f, 8 * (v / 4) + 4 * hf + (v % 4), 64);
            S[0][v] *= fr;
            S[1][v] *= fr;
          }
        }
      }
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        u32x4 pk[3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float e0 = fast_exp2(U[8 * hh + 2 * q]), e1 = fast_exp2(U[8 * hh + 2 * q + 1]);
          z += e0;
          z += e1;
          unsigned a, b, d;
          split_pair(e0, e1, a, b, d);
          pk[0][q] = a; pk[1][q] = b; pk[2][q] = d;
        }
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          u32x4 vf[NP];
#pragma unroll
          for (int q = 0; q < NP; ++q) {
            const unsigned char* vr = base + SM::x_bytes + q * kTok * 128 + hh * 16 * 128 + voff[ct];
            const u32x2 lo = lds_read_tr16(reinterpret_cast<const us*>(vr));
            const u32x2 hi = lds_read_tr16(reinterpret_cast<const us*>(vr + 8 * 128));
            vf[q] = u32x4{lo[0], lo[1], hi[0], hi[1]};
          }
          S[ct] = mm_all(pk, vf, S[ct]);
        }
      }
    }
    if (t + 1 < ntile) store(t + 1);
    __syncthreads();
  }
  if (!active) return;
  const size_t ob = ((size_t)bh * P + p) * m + f0;
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int v = 0; v < 16; ++v) Spart[(ob + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * ct + l32] = S[ct][v];
  z += xor32(z);
  if (hf == 0) {
    zpart[ob + l32] = z;
    cpart[ob + l32] = c;
  }
}

// ---------------------------------------------------------------------------
// k_sp_merge: per (b,h, 32 features): c_j = max over the slices, [S|z]_j = sum_p 2^(c_pj - c_j) [S|z]_pj with p
// ascending; S^T leaves as planes [BH][3][64][m], features in chain order (split.h).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_sp_merge(const float* __restrict__ Spart, const float* __restrict__ zpart,
                                                  const float* __restrict__ cpart, us* __restrict__ St,
                                                  float* __restrict__ zt, float* __restrict__ ct, int m, int P) {
  __shared__ __attribute__((aligned(16))) us tile[3][kD][40];
  const int nblk = m / 32;
  const int bh = blockIdx.x / nblk, blk = blockIdx.x % nblk;
  const int tid = threadIdx.x, f = tid / 8, c8 = 8 * (tid % 8);
  const size_t row0 = (size_t)bh * P * m + 32 * blk + f;
  constexpr int PB = 8;   // slices in flight
  float cs = -INFINITY;
  for (int p0 = 0; p0 < P; p0 += PB) {
    float cv[PB];
#pragma unroll
    for (int u = 0; u < PB; ++u) cv[u] = cpart[row0 + (size_t)min(p0 + u, P - 1) * m];
#pragma unroll
    for (int u = 0; u < PB; ++u) cs = fmaxf(cs, cv[u]);
  }
  f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
  float z = 0.f;
  for (int p0 = 0; p0 < P; p0 += PB) {
    f32x4 v[PB][2];
    float cv[PB], zv[PB];
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      if (p0 + u < P) {   // uniform
        const size_t r = row0 + (size_t)(p0 + u) * m;
        v[u][0] = *reinterpret_cast<const f32x4*>(Spart + r * kD + c8);
        v[u][1] = *reinterpret_cast<const f32x4*>(Spart + r * kD + c8 + 4);
        cv[u] = cpart[r];
        zv[u] = zpart[r];
      }
    }
#pragma unroll
    for (int u = 0; u < PB; ++u)
      if (p0 + u < P) {
        const float fac = fast_exp2(cv[u] - cs);
        a0 += fac * v[u][0];
        a1 += fac * v[u][1];
        z = fmaf(fac, zv[u], z);
      }
  }
  const int pos = chain_pos(f);
  u32x4 pl[3];
  split8(a0, a1, pl);
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int j = 0; j < 8; ++j) tile[q][c8 + j][pos] = (us)(j % 2 ? pl[q][j / 2] >> 16 : pl[q][j / 2] & 0xffffu);
  if (tid % 8 == 0) {
    zt[(size_t)bh * m + 32 * blk + f] = z;
    ct[(size_t)bh * m + 32 * blk + f] = cs;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int i = tid + 256 * u, q = i / 256, c = (i % 256) / 4, k = i % 4;
    *reinterpret_cast<u32x4*>(St + (((size_t)bh * 3 + q) * kD + c) * m + 32 * blk + 8 * k) =
        *reinterpret_cast<const u32x4*>(&tile[q][c][8 * k]);
  }
}

// ---------------------------------------------------------------------------
// k_sp_readout: a wave owns 32 queries (lane = query): U^T[f][tok] = A' X^T, features along the registers, so the row
// shift, the denominator and the rescaling are per-lane scalars and phi^T enters N^T[c][tok] += S^T phi^T from the
// accumulator.  The features come in groups of 64 whose operands (planes of A' and S^T, 55 KB) the workgroup stages
// in LDS; with NWF = 2 two groups are staged at a time and two waves share 32 queries, each taking every other group,
// their halves joined at the end.
// ---------------------------------------------------------------------------
struct RdSmem {
  static constexpr size_t a_bytes = (size_t)3 * kGrp * LDX * 2;   // A' [plane][f][d]
  static constexpr size_t s_bytes = (size_t)3 * kD * LDX * 2;     // S^T [plane][c][f], chain order
  static constexpr size_t cz_bytes = (size_t)2 * kGrp * 4;        // shifts, z
  static constexpr size_t slot = a_bytes + s_bytes + cz_bytes;
};

template <int NP, int NWF, typename OutT>
__global__ __launch_bounds__(256 * NWF, 2) void k_sp_readout(const void* __restrict__ Qg, const us* __restrict__ Apl,
                                                             const us* __restrict__ St, const float* __restrict__ zt,
                                                             const float* __restrict__ ct, OutT* __restrict__ out,
                                                             int H, int L, int m, int wgs_per_bh) {
  using SM = RdSmem;
  constexpr int NT = 256 * NWF;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const int l32 = lane % 32, hf = lane / 32;
  const int wf = NWF == 1 ? 0 : wv / 4, wt = wv % 4;
  const int bh = blockIdx.x / wgs_per_bh, h = bh % H;
  const int tok = (blockIdx.x % wgs_per_bh) * 4 * kTok + wt * kTok + l32;
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  Raw8<NP> xr[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) xr[s].load(Qg, ((size_t)bh * L + min(tok, L - 1)) * kD + 16 * s + 8 * hf);
  u32x4 xf[4][NP];
  f32x16 N[2] = {zero16, zero16};
  float D = 0.f, mu = -INFINITY;
  const int ngrp = m / kGrp;
  for (int g0 = 0; g0 < ngrp; g0 += NWF) {
    if (g0 > 0) __syncthreads();   // everyone is done with the previous groups' operands
    constexpr int NCH = 2 * 3 * 64 * 8;   // 16-byte pieces of a group: A' then S^T
    constexpr int PER = NCH * NWF / NT;
    u32x4 v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = tid + NT * u, slot = i / NCH, j = i % NCH, q = (j % (NCH / 2)) / 512, row = (j % 512) / 8, ch = j % 8;
      const int g = min(g0 + slot, ngrp - 1);
      const us* src = j < NCH / 2 ? Apl + (((size_t)h * 3 + q) * m + g * kGrp + row) * kD + 8 * ch
                                  : St + (((size_t)bh * 3 + q) * kD + row) * m + g * kGrp + 8 * ch;
      v[u] = *reinterpret_cast<const u32x4*>(src);
    }
    float cz = 0.f;
    if (tid < 2 * kGrp * NWF) {
      const int slot = tid / (2 * kGrp), i = tid % (2 * kGrp), g = min(g0 + slot, ngrp - 1);
      cz = (i < kGrp ? ct : zt)[(size_t)bh * m + g * kGrp + i % kGrp];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = tid + NT * u, slot = i / NCH, j = i % NCH, q = (j % (NCH / 2)) / 512, row = (j % 512) / 8, ch = j % 8;
      *reinterpret_cast<u32x4*>(smem + slot * SM::slot + (j < NCH / 2 ? 0 : SM::a_bytes) + (q * 64 + row) * LDX * 2 + 16 * ch) = v[u];
    }
    if (tid < 2 * kGrp * NWF)
      reinterpret_cast<float*>(smem + (tid / (2 * kGrp)) * SM::slot + SM::a_bytes + SM::s_bytes)[tid % (2 * kGrp)] = cz;
    if (g0 == 0) {
#pragma unroll
      for (int s = 0; s < 4; ++s) xr[s].planes(xf[s]);
    }
    __syncthreads();
    if (g0 + wf >= ngrp) continue;   // wave-uniform; the barriers are reached by every wave
    const unsigned char* sa = smem + wf * SM::slot;
    const unsigned char* ss = sa + SM::a_bytes;
    const float* cs = reinterpret_cast<const float*>(ss + SM::s_bytes);
    f32x16 U[2] = {zero16, zero16};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int fb = 0; fb < 2; ++fb) {
        u32x4 a[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
          a[q] = *reinterpret_cast<const u32x4*>(sa + (q * 64 + 32 * fb + l32) * LDX * 2 + 32 * s + 16 * hf);
        U[fb] = mm_all(a, xf[s], U[fb]);
      }
    float bm = -INFINITY;
#pragma unroll
    for (int fb = 0; fb < 2; ++fb)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 c4 = *reinterpret_cast<const f32x4*>(cs + 32 * fb + 8 * a + 4 * hf);
#pragma unroll
        for (int j = 0; j < 4; ++j) U[fb][4 * a + j] += c4[j];
        bm = max3(bm, fmaxf(U[fb][4 * a], U[fb][4 * a + 1]), fmaxf(U[fb][4 * a + 2], U[fb][4 * a + 3]));
      }
    bm = fmaxf(bm, xor32(bm));
    if (__any(bm > mu + kRaise)) {   // the first group sets the shift of the row; later ones raise it (rare)
      const float mn = bm > mu + kRaise ? bm : mu, f = fast_exp2(mu - mn);
      mu = mn;
      D *= f;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v2 = 0; v2 < 16; ++v2) N[b][v2] *= f;
    }
#pragma unroll
    for (int fb = 0; fb < 2; ++fb)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        u32x4 pk[3];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const f32x4 z4 = *reinterpret_cast<const f32x4*>(cs + kGrp + 32 * fb + 16 * hh + 8 * a + 4 * hf);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float e0 = fast_exp2(U[fb][8 * hh + 4 * a + 2 * j] - mu), e1 = fast_exp2(U[fb][8 * hh + 4 * a + 2 * j + 1] - mu);
            D = fmaf(e0, z4[2 * j], D);
            D = fmaf(e1, z4[2 * j + 1], D);
            unsigned p0, p1, p2;
            split_pair(e0, e1, p0, p1, p2);
            pk[0][2 * a + j] = p0; pk[1][2 * a + j] = p1; pk[2][2 * a + j] = p2;
          }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          u32x4 sf[3];
#pragma unroll
          for (int q = 0; q < 3; ++q)
            sf[q] = *reinterpret_cast<const u32x4*>(ss + (q * 64 + 32 * b + l32) * LDX * 2 + (32 * fb + 16 * hh) * 2 + 16 * hf);
          N[b] = mm_all(sf, pk, N[b]);
        }
      }
  }
  D += xor32(D);
  if constexpr (NWF == 2) {
    // the second wave of a pair hands its half over; lane = query in both
    __syncthreads();
    float* ex = reinterpret_cast<float*>(smem) + (size_t)wt * 64 * 34 + lane;
    if (wf == 1) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) ex[64 * (16 * b + v)] = N[b][v];
      ex[64 * 32] = D;
      ex[64 * 33] = mu;
    }
    __syncthreads();
    if (wf == 1) return;
    const float mo = ex[64 * 33], mn = fmaxf(mu, mo);   // a wave without a group has mu = -inf and zeros
    const float f0 = fast_exp2(mu - mn), f1 = fast_exp2(mo - mn);
    D = D * f0 + ex[64 * 32] * f1;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) N[b][v] = N[b][v] * f0 + ex[64 * (16 * b + v)] * f1;
  }
  if (tok >= L) return;
  const float inv = 1.f / D;
  OutT* o = out + ((size_t)bh * L + tok) * kD + 4 * hf;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 w = {N[b][4 * a] * inv, N[b][4 * a + 1] * inv, N[b][4 * a + 2] * inv, N[b][4 * a + 3] * inv};
      if constexpr (sizeof(OutT) == 4) {
        *reinterpret_cast<f32x4*>(o + 32 * b + 8 * a) = w;
      } else {
        *reinterpret_cast<u32x2*>(o + 32 * b + 8 * a) = u32x2{pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
      }
    }
}

// ------------------------------- host side ---------------------------------
// Slices of the key pass: about one workgroup per CU (eight waves; more of the smaller ones), whole tiles.
void sp_slices(const Problem& pb, int* P, int* slice_len) {
  const dark_params& p = pb.p;
  const int nfb = (p.m + 255) / 256;
  const int wgs = p.m >= 256 ? 256 : (p.m == 128 ? 512 : 1024);
  long long want = wgs / (pb.BH() * nfb > 0 ? pb.BH() * nfb : 1);
  want = want < 1 ? 1 : (want > 64 ? 64 : want);
  int sl = (int)((p.L + want - 1) / want);
  sl = (sl + kTok - 1) / kTok * kTok;
  *slice_len = sl;
  *P = (p.L + sl - 1) / sl;
}

struct SpBufs {
  us *Apl, *St;
  float *nrm, *Spart, *zpart, *cpart, *zt, *ct;
  int P, sl;
};

SpBufs take_bufs(const Problem& pb, Arena& ar) {
  const dark_params& p = pb.p;
  const size_t BH = (size_t)pb.BH();
  SpBufs b{};
  sp_slices(pb, &b.P, &b.sl);
  b.Apl = ar.take<us>((size_t)p.H * 3 * p.m * kD);
  b.nrm = ar.take<float>(BH * p.L);
  b.Spart = ar.take<float>(BH * b.P * p.m * kD);
  b.zpart = ar.take<float>(BH * b.P * p.m);
  b.cpart = ar.take<float>(BH * b.P * p.m);
  b.St = ar.take<us>(BH * 3 * kD * p.m);
  b.zt = ar.take<float>(BH * p.m);
  b.ct = ar.take<float>(BH * p.m);
  return b;
}

template <int NP>
dark_status launch_prep(const Problem& pb, const SpBufs& b, const void* K, const float* M, const float* W) {
  const dark_params& p = pb.p;
  const long long nt = pb.BH() * ((p.L + kTok - 1) / kTok);
  const int tpw = (int)((nt + 4095) / 4096);   // one tile per wave until every SIMD has four
  const long long waves = (nt + tpw - 1) / tpw;
  const unsigned grid = (unsigned)(p.H * (p.m / 16) + (waves + 3) / 4);
  DARK_LAUNCH(KID_PREP, pb.st, k_sp_prep<NP>, dim3(grid), dim3(256), 0, M, W, b.Apl, K, b.nrm, p.H, p.L, p.m, p.w_shared,
              std::sqrt(pb.scale), (int)nt, tpw);
  return DARK_OK;
}

template <int NP, int NW>
dark_status launch_states(const Problem& pb, const SpBufs& b, const void* K, const void* V) {
  const dark_params& p = pb.p;
  const int nfb = (p.m + 255) / 256;
  auto kern = k_sp_states<NP, NW>;
  DARK_TRY(allow_lds(kern, StSmem<NP>::total));
  DARK_LAUNCH(KID_KV_REDUCE, pb.st, kern, dim3((unsigned)(pb.BH() * b.P * nfb)), dim3(64 * NW), StSmem<NP>::total, K, V,
              b.Apl, b.nrm, b.Spart, b.zpart, b.cpart, p.H, p.L, p.m, b.P, b.sl, nfb);
  return DARK_OK;
}

template <int NP, int NWF, typename OutT>
dark_status launch_readout(const Problem& pb, const SpBufs& b, const void* Q, void* out) {
  const dark_params& p = pb.p;
  auto kern = k_sp_readout<NP, NWF, OutT>;
  const size_t lds = NWF * RdSmem::slot;
  DARK_TRY(allow_lds(kern, lds));
  const int per = (p.L + 4 * kTok - 1) / (4 * kTok);
  DARK_LAUNCH(KID_READOUT, pb.st, kern, dim3((unsigned)(pb.BH() * per)), dim3(256 * NWF), lds, Q, b.Apl, b.St, b.zt, b.ct,
              (OutT*)out, p.H, p.L, p.m, per);
  return DARK_OK;
}

template <int NP>
dark_status sp_forward(const Problem& pb, const SpBufs& b, const void* Q, const void* K, const void* V, const float* M,
                       const float* W, void* out) {
  const dark_params& p = pb.p;
  DARK_TRY((launch_prep<NP>(pb, b, K, M, W)));
  if (p.m == 64) DARK_TRY((launch_states<NP, 2>(pb, b, K, V)));
  else if (p.m == 128) DARK_TRY((launch_states<NP, 4>(pb, b, K, V)));
  else DARK_TRY((launch_states<NP, 8>(pb, b, K, V)));
  DARK_LAUNCH(KID_KV_MERGE, pb.st, k_sp_merge, dim3((unsigned)(pb.BH() * (p.m / 32))), dim3(256), 0, b.Spart, b.zpart,
              b.cpart, b.St, b.zt, b.ct, p.m, b.P);
  // two waves per 32 queries while that is what it takes to give every SIMD two waves
  const bool pair = p.m > kGrp && pb.BH() * ((p.L + kTok - 1) / kTok) <= 1536;
  if (p.out_dtype == DARK_BF16) {
    if (pair) return launch_readout<NP, 2, us>(pb, b, Q, out);
    return launch_readout<NP, 1, us>(pb, b, Q, out);
  }
  if (pair) return launch_readout<NP, 2, float>(pb, b, Q, out);
  return launch_readout<NP, 1, float>(pb, b, Q, out);
}

}  // namespace

bool split_supported(const Problem& pb) {
  const dark_params& p = pb.p;
  return p.d == kD && p.r == kD && p.dv == kD && p.m % kGrp == 0 && pb.BH() * (long long)(p.L + kTok) < (1LL << 31) &&
         pb.BH() * (long long)p.m < (1LL << 24);
}

dark_status split_attn_fwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V, const float* M,
                           const float* W, void* out) {
  const SpBufs b = take_bufs(pb, ar);
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  return pb.p.io_dtype == DARK_BF16 ? sp_forward<1>(pb, b, Q, K, V, M, W, out) : sp_forward<3>(pb, b, Q, K, V, M, W, out);
}

}  // namespace dark
