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
//   k_sp_keys     the first three in one, where the sequence is short
// Measured (fp32 inputs, against the general kernels): B H L = 24,576, m = 256: 5.7 + 15 + 4.5 + 17 us, 42 us a call
// (165 before); B H L = 393,216: 0.37 ms (1.60 before); one head, L = 256, m = 64: 18 us, two launches (77 before).
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "split.h"

namespace dark {
using namespace sp;
namespace {

constexpr int kD = 64;       // d = r = dv
constexpr int kTok = 32;     // tokens per tile
constexpr int kGrp = 32;     // features per group of the kernels whose waves own tokens
constexpr int LDX = 72;      // row pitch (16-bit elements) of LDS tiles with 64 columns
// Norm (or row shift) of the rows past the end: their features are exp2(-inf) = 0.  Not a large finite number: the norms of the
// rows themselves may be larger, and then the rows past the end are the ones that count.
constexpr float kTailNorm = INFINITY;
// A shift is raised once a logit exceeds it by 2^kRaise: features stay below that, sums over any length far inside
// the fp32 range, and what lies more than 2^-(126 - kRaise) below the largest key of a feature vanishes.
static_assert(kRaise <= 32.f, "sums of features must stay far from the end of the fp32 range");

// The matrices that the matrix cores meet as operands (A', S and R, and their transposes) are stored as planes of operand
// fragments: with a feature per row [m / 32][16 columns][lane][8], transposed (contraction over the features, in chain order)
// [m / 16][32 rows][lane][8].  A wave's fragment is one contiguous kilobyte.  Read as rows, 32 of them by 16 or 32 bytes an
// instruction, it takes the CU's address unit four times as long (8 heads, L = 1000, m = 128, a training step, with the chunks' rows
// split by all waves together: 122.4 -> 115.8 us; an encoder layer of 24 x 1024: 44.9 -> 43.8).  `at`: the head, or the (b,h).
__device__ __forceinline__ const us* a_frag(const us* Apl, size_t at, int m, int q, int f, int s, int lane) {   // f: first of 32 features
  return Apl + (at * 3 + q) * m * kD + ((f / 32) * 4 + s) * 512 + lane * 8;
}
__device__ __forceinline__ const us* at_frag(const us* Atp, size_t at, int m, int q, int f, int b, int lane) {   // f: first of 16 features
  return Atp + (at * 3 + q) * m * kD + ((f / 16) * 2 + b) * 512 + lane * 8;
}

// A group of 32 features of such a matrix, either way round, is 4 KB per plane: twelve fragments, which go straight from memory
// to LDS as they are (fetch_group), a group ahead of their use.  A wave reads a fragment at sixteen bytes a lane, without bank
// conflicts; no register holds them on the way.
constexpr unsigned kPlaneBytes = 4096, kOpBytes = 3 * kPlaneBytes;
// Two arrays of a float per feature (shifts, z) ride behind the operands of their group.
constexpr unsigned kCzBytes = 2 * kGrp * 4;
// As dma16_to_lds and by its rules, four bytes a lane.
__device__ __forceinline__ void word_to_lds(const float* src, void* lds) {
  const unsigned base = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)lds);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(base) : "memory", "m0");
}
// Four waves bring an operand, three fragments each; of eight waves the halves take every other one.
template <int NW, int N>
__device__ __forceinline__ void fetch_group(const us* const (&op)[N], const float* c, const float* z, int m, int g, unsigned char* dst,
                                            int wv, int lane) {
  static_assert(NW == 4 || NW == 8, "waves that fetch");
#pragma unroll
  for (int o = 0; o < N; ++o)
    if (NW == 4 || wv / 4 == o % 2) {   // wave-uniform
#pragma unroll
      for (int q = 0; q < 3; ++q)
        dma16_to_lds(op[o] + (size_t)q * m * kD + g * (kGrp * kD) + wv % 4 * 512, 16 * lane, dst + o * kOpBytes + q * kPlaneBytes + 1024 * (wv % 4));
    }
  if (c != nullptr && wv == NW - 1) word_to_lds((lane < kGrp ? c : z) + g * kGrp + lane % kGrp, dst + N * kOpBytes);
}
// Everything this wave has asked for is in LDS, and what it read from there has been read: the group may be used and the one before
// it be replaced.
__device__ __forceinline__ void group_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// Fragment i of an operand in LDS (rows: step i of 16 columns; transposed: 2 (step of 16 features) + block of 32 rows).
__device__ __forceinline__ void op_frag(u32x4 (&a)[3], const unsigned char* op, int i, int lane) {
#pragma unroll
  for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const u32x4*>(op + q * kPlaneBytes + 1024 * i + 16 * lane);
}

// ---------------------------------------------------------------------------
// k_sp_prep: blocks [0, H nA): sixteen rows of A' of one head by fp32 MFMA 16x16x4, a wave per sixteen columns, stored as planes
// (fragments, above); BWD: also A'^T, and four blocks per head for alpha^2 M^T M [H][3][64][64] (fragments as of A').  The other
// blocks: n' of the keys of one head in all batch entries, x~^T[r][tok] = M' X^T by MFMA, the sum of squares over registers; M' is
// split once a workgroup and read from LDS, and a wave's tiles of 32 keys pass through LDS, so that memory sees whole lines.
// Two memory round trips with the launch.  24 (b,h) of 1024 keys, m = 256, fp32: 7.3 us when every wave read its rows of M and K as
// fragments (24 loads of 32 rows) and summed A' by vector FMAs, now 5.7; a training step of 8 heads, L = 1000, m = 128: 115.8 -> 114.3.
// Short sequences share a workgroup: a forward of 512 x 8 of 64 tokens, m = 64, takes 182 us, with one (b,h) a workgroup 199
// (190 when every wave split M' for itself).
// ---------------------------------------------------------------------------
template <int NP>
struct PrepSmem {
  static constexpr int KROW = NP == 3 ? (kD + 4) * 4 : LDX * 2;   // bytes per row of a wave's tile of keys
  static constexpr size_t keys = (size_t)3 * kD * LDX * 2;        // behind the planes of M'
  static constexpr size_t norm = keys + (size_t)4 * kTok * KROW;
  static constexpr size_t w = (size_t)kD * kD * 4;                // A' and M^T M: W behind M, then the result's planes
  static constexpr size_t tile = w + (size_t)16 * (kD + 4) * 4;
  static constexpr size_t ops = tile + (size_t)3 * 16 * LDX * 2;
  static constexpr size_t total = norm > ops ? norm : ops;
};

template <int NP, bool BWD>
__global__ __launch_bounds__(256) void k_sp_prep(const float* __restrict__ M, const float* __restrict__ W,
                                                 us* __restrict__ Apl, us* __restrict__ Atp, us* __restrict__ G2p,
                                                 const void* __restrict__ Kg,
                                                 float* __restrict__ nrm, int H, int L, int m, int w_shared,
                                                 float alpha, int B, int wgs_per_h, int tiles_per_wave) {
  using SM = PrepSmem<NP>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const int nA = m / 16;
  const int nG = BWD ? 4 : 0;   // blocks per head for M^T M
  if ((int)blockIdx.x < H * (nA + nG)) {
    const bool isA = (int)blockIdx.x < H * nA;
    const int blk = isA ? blockIdx.x : blockIdx.x - H * nA, per = isA ? nA : nG;
    const int h = blk / per, j0 = 16 * (blk % per), l16 = lane % 16, kg = lane / 16;
    float* Mt = reinterpret_cast<float*>(smem);             // [64][64]
    float* Ws = reinterpret_cast<float*>(smem + SM::w);     // [16][68]
    us* tile = reinterpret_cast<us*>(smem + SM::tile);      // planes [3][16][LDX]
    const f32x4* Mp = reinterpret_cast<const f32x4*>(M + (size_t)h * kD * kD);
    f32x4 mv[4], wv4 = {};
#pragma unroll
    for (int u = 0; u < 4; ++u) mv[u] = Mp[tid + 256 * u];
    if (isA) wv4 = reinterpret_cast<const f32x4*>(W + ((w_shared ? 0 : (size_t)h * m) + j0) * kD)[tid];
#pragma unroll
    for (int u = 0; u < 4; ++u) reinterpret_cast<f32x4*>(Mt)[tid + 256 * u] = mv[u];
    *reinterpret_cast<f32x4*>(Ws + (tid / 16) * (kD + 4) + 4 * (tid % 16)) = wv4;
    __syncthreads();
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = 16 * s + 4 * kg + j;   // rows of W M: sum over W[row][t] M[t][col]; of M^T M: over M[t][row] M[t][col]
        const float x = isA ? Ws[l16 * (kD + 4) + t] : Mt[t * kD + j0 + l16];
        acc[j % 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, Mt[t * kD + 16 * wv + l16], acc[j % 2], 0, 0, 0);
      }
    acc[0] += acc[1];
    acc[0] *= isA ? alpha * kLog2e : alpha * alpha;
#pragma unroll
    for (int v = 0; v < 4; v += 2) {
      unsigned p[3];
      split_pair(acc[0][v], acc[0][v + 1], p[0], p[1], p[2]);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        us* d = tile + (q * 16 + 4 * kg + v) * LDX + 16 * wv + l16;
        d[0] = (us)(p[q] & 0xffffu);
        d[LDX] = (us)(p[q] >> 16);
      }
    }
    __syncthreads();
    us* dst = isA ? Apl : G2p;
    const int rows = isA ? m : kD;
    for (int i = tid; i < 3 * 128; i += 256) {
      const int q = i / 128, s = i / 32 % 4, hf = i / 16 % 2, r = i % 16;
      *reinterpret_cast<u32x4*>(const_cast<us*>(a_frag(dst, h, rows, q, j0, s, j0 % 32 + r + 32 * hf))) =
          *reinterpret_cast<const u32x4*>(tile + (q * 16 + r) * LDX + 16 * s + 8 * hf);
    }
    if (BWD && isA) {
      for (int i = tid; i < 3 * kD * 2; i += 256) {   // a column's eight features in chain order
        const int q = i / (2 * kD), k = i / kD % 2, d = i % kD;
        unsigned w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const us* c = tile + (q * 16 + 4 * k + 8 * (e / 2) + 2 * (e % 2)) * LDX + d;
          w[e] = c[0] | (unsigned)c[LDX] << 16;
        }
        *reinterpret_cast<u32x4*>(const_cast<us*>(at_frag(Atp, h, m, q, j0, d / 32, d % 32 + 32 * k))) = u32x4{w[0], w[1], w[2], w[3]};
      }
    }
    return;
  }
  const int l32 = lane % 32, hf = lane / 32;
  const int blk = blockIdx.x - H * (nA + nG), h = blk / wgs_per_h;
  const int nt = (L + kTok - 1) / kTok;   // tile t: of batch entry t / nt
  const int t_begin = (blk % wgs_per_h * 4 + __builtin_amdgcn_readfirstlane(wv)) * tiles_per_wave, t_end = min(B * nt, t_begin + tiles_per_wave);
  us* Ms = reinterpret_cast<us*>(smem);
  unsigned char* ks = smem + SM::keys + (size_t)wv * kTok * SM::KROW;
  constexpr int KP = NP == 3 ? 8 : 4, CPR = NP == 3 ? 16 : 8;   // 16-byte pieces of a tile: per lane, per row
  u32x4 kr[KP];
  auto row = [&](int t, int r) { return ((size_t)(t / nt) * H + h) * L + min(t % nt * kTok + r, L - 1); };
  auto fetch = [&](int t) {
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      const int i = lane + 64 * u;
      kr[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const unsigned char*>(Kg) + (row(t, i / CPR) * CPR + i % CPR) * 16);
    }
  };
  {
    const float fm = alpha * sqrtf(0.5f * kLog2e);
    f32x4 mv[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < 2; ++k) mv[u][k] = reinterpret_cast<const f32x4*>(M + (size_t)h * kD * kD)[2 * (tid + 256 * u) + k];
    if (t_begin < t_end) fetch(t_begin);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = tid + 256 * u;
      u32x4 p[3];
      split8(mv[u][0] * fm, mv[u][1] * fm, p);
#pragma unroll
      for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(Ms + (q * kD + i / 8) * LDX + 8 * (i % 8)) = p[q];
    }
  }
  __syncthreads();
  for (int t = t_begin; t < t_end; ++t) {
    asm volatile("" ::: "memory");   // the last tile has been read
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      const int i = lane + 64 * u;
      *reinterpret_cast<u32x4*>(ks + (i / CPR) * SM::KROW + 16 * (i % CPR)) = kr[u];
    }
    if (t + 1 < t_end) fetch(t + 1);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    Logits x[2];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      Raw8<NP> r;
      r.load(ks + l32 * SM::KROW, 16 * s + 8 * hf);
      u32x4 xf[NP];
      r.planes(xf);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        u32x4 a[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const u32x4*>(Ms + (q * kD + 32 * rb + l32) * LDX + 16 * s + 8 * hf);
        x[rb].add_ax(a, xf);
      }
    }
    float n = 0.f;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const f32x16 xs = x[rb].sum();
#pragma unroll
      for (int v = 0; v < 16; ++v) n = fmaf(xs[v], xs[v], n);
    }
    n += xor32(n);
    if (hf == 0 && t % nt * kTok + l32 < L) nrm[row(t, l32)] = n;
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
      af[s][q] = *reinterpret_cast<const u32x4*>(a_frag(Apl, h, m, q, min(f0, m - 32), s, lane));
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
      Logits lg;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 xf[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q)
          xf[q] = *reinterpret_cast<const u32x4*>(base + (q * kTok + l32) * LDX * 2 + 32 * s + 16 * hf);
        lg.add_xa(xf, af[s]);
      }
      f32x16 U = lg.sum();
      const float* nl = reinterpret_cast<const float*>(base + SM::x_bytes + SM::v_bytes);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 n4 = *reinterpret_cast<const f32x4*>(nl + 8 * a + 4 * hf);
#pragma unroll
        for (int j = 0; j < 4; ++j) U[4 * a + j] -= n4[j];
      }
      float mx = U[0];
#pragma unroll
      for (int v = 1; v < 15; v += 2) mx = max3(mx, U[v], U[v + 1]);
      mx = fmaxf(mx, U[15]);
      mx = fmaxf(mx, xor32(mx));
      // Set the shift, or raise it (rare).  The logits meet the shift only afterwards: less a shift far below them they would
      // be rounded to its last place.  Keys whose norm term overflows have logits of -inf; the shift stays finite.
      if (t == 0 || __any(mx > c + kRaise)) {
        const float before = c;
        if (t == 0 || mx > c + kRaise) c = fmaxf(mx, -FLT_MAX);
        if (t > 0) {
          const float f = fast_exp2(before - c);
          z *= f;
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float fr = __shfl(f, 8 * (v / 4) + 4 * hf + (v % 4), 64);
            S[0][v] *= fr;
            S[1][v] *= fr;
          }
        }
      }
      float zt = 0.f;   // summed by tile: a chain over the whole slice would round as often as it has keys
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        u32x4 pk[3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float e0 = fast_exp2(U[8 * hh + 2 * q] - c), e1 = fast_exp2(U[8 * hh + 2 * q + 1] - c);
          zt += e0;
          zt += e1;
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
      z += zt;
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
// ascending.  MG_FWD: S^T leaves as fragments.  MG_S: S instead (the backward's query passes).  MG_R: the partial states are the
// backward's R, which carry no shifts; R and R^T.
// ---------------------------------------------------------------------------
enum { MG_FWD = 0, MG_S = 1, MG_R = 2 };
template <int MODE>
__global__ __launch_bounds__(256) void k_sp_merge(const float* __restrict__ Spart, const float* __restrict__ zpart,
                                                  const float* __restrict__ cpart, us* __restrict__ St,
                                                  us* __restrict__ Sf, float* __restrict__ zt, float* __restrict__ ct,
                                                  int m, int P) {
  __shared__ __attribute__((aligned(16))) us tile[MODE == MG_S ? 1 : 3][kD][40];
  const int nblk = m / 32;
  const int bh = blockIdx.x / nblk, blk = blockIdx.x % nblk;
  const int tid = threadIdx.x, f = tid / 8, c8 = 8 * (tid % 8);
  const size_t row0 = (size_t)bh * P * m + 32 * blk + f;
  constexpr int PB = 8;   // slices in flight
  f32x4 v[PB][2];
  float cv[PB], zv[PB];
  auto load = [&](int p0) {
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      if (p0 + u < P) {   // uniform
        const size_t r = row0 + (size_t)(p0 + u) * m;
        v[u][0] = *reinterpret_cast<const f32x4*>(Spart + r * kD + c8);
        v[u][1] = *reinterpret_cast<const f32x4*>(Spart + r * kD + c8 + 4);
        if (MODE != MG_R) cv[u] = cpart[r];
        zv[u] = zpart[r];
      }
    }
  };
  load(0);   // the first slices' states do not wait for the shifts
  float cs = -INFINITY;
  if (MODE != MG_R) {
    for (int p0 = PB; p0 < P; p0 += PB) {
      float cx[PB];
#pragma unroll
      for (int u = 0; u < PB; ++u) cx[u] = cpart[row0 + (size_t)min(p0 + u, P - 1) * m];
#pragma unroll
      for (int u = 0; u < PB; ++u) cs = fmaxf(cs, cx[u]);
    }
#pragma unroll
    for (int u = 0; u < PB; ++u)
      if (u < P) cs = fmaxf(cs, cv[u]);
  }
  f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = a0;
  float z = 0.f;
  for (int p0 = 0; p0 < P; p0 += PB) {
    if (p0 > 0) load(p0);
#pragma unroll
    for (int u = 0; u < PB; ++u)
      if (p0 + u < P) {
        const float fac = MODE == MG_R ? 1.f : fast_exp2(cv[u] - cs);
        a0 += fac * v[u][0];
        a1 += fac * v[u][1];
        z = fmaf(fac, zv[u], z);
      }
  }
  const int pos = chain_pos(f);
  u32x4 pl[3];
  split8(a0, a1, pl);
  if (MODE != MG_S) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int j = 0; j < 8; ++j) tile[q][c8 + j][pos] = (us)(j % 2 ? pl[q][j / 2] >> 16 : pl[q][j / 2] & 0xffffu);
  }
  if (tid % 8 == 0) {
    zt[(size_t)bh * m + 32 * blk + f] = z;
    if (MODE != MG_R) ct[(size_t)bh * m + 32 * blk + f] = cs;
  }
  if (MODE != MG_FWD) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
      *reinterpret_cast<u32x4*>(const_cast<us*>(a_frag(Sf, bh, m, q, 32 * blk, c8 / 16, f + 32 * (c8 / 8 % 2)))) = pl[q];
  }
  if (MODE == MG_S) return;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int st = tid / 128, b = tid / 64 % 2, fl = tid % 64;   // plane u; step of 16 features, block of columns, lane of the fragment
    *reinterpret_cast<u32x4*>(const_cast<us*>(at_frag(St, bh, m, u, 32 * blk + 16 * st, b, fl))) =
        *reinterpret_cast<const u32x4*>(&tile[u][32 * b + fl % 32][16 * st + 8 * (fl / 32)]);
  }
}

// ---------------------------------------------------------------------------
// k_sp_keys: the merged state of all keys of a (b,h) and its operand planes in one launch, where the sequence is short: what
// k_sp_prep, k_sp_states and k_sp_merge do in three.  A workgroup owns 32 features of one (b,h) and all of its keys, a
// wave every eighth tile of them, so nothing has to pass between workgroups: the block of A' takes one 16x16 fp32 MFMA chain a
// wave, the norms are formed again for every block of features (that is the price: half of the matrix work), and the waves'
// states meet in LDS, in wave order.  W, M and the wave's tiles pass through LDS, so that memory sees whole lines.
// Matrix pipe and vector issue of one CU bound it, 5.4 us for eight tiles of fp32.  One head, L = 256, m = 64: 20.1 us in four
// launches (the host's time for them), 17.8 in two.
// ---------------------------------------------------------------------------
constexpr int kKeyWaves = 8;
template <int NP>
struct KeySmem {
  static constexpr int LDE = 72;   // floats per feature of a wave's state: both halves of a wave on banks of their own
  static constexpr size_t a_bytes = (size_t)3 * 32 * LDX * 2, m_bytes = (size_t)3 * kD * LDX * 2;
  static constexpr int KROW = PrepSmem<NP>::KROW;                // bytes per row of a tile of keys
  static constexpr size_t v_bytes = (size_t)NP * kTok * 128;     // planes of a tile of V
  static constexpr size_t t_bytes = (size_t)kTok * KROW > v_bytes ? (size_t)kTok * KROW : v_bytes;   // a wave's tile, of K and then of V
  static constexpr size_t off_t = a_bytes + m_bytes;
  static constexpr size_t off_w = off_t, off_m = off_w + (size_t)32 * (kD + 4) * 4;   // W and M as they are, before the tiles
  static constexpr size_t part = (size_t)32 * LDE * 4;
  static constexpr size_t cz = kKeyWaves * part;                 // [wave][shift | z][32]
  static constexpr size_t turn = cz + kKeyWaves * 2 * 32 * 4;    // S^T on its way out
  static constexpr size_t end_ops = off_t + kKeyWaves * t_bytes, end_m = off_m + (size_t)kD * kD * 4;
  static constexpr size_t end_part = turn + (size_t)3 * kD * 40 * 2;
  static constexpr size_t nl = end_ops > end_part ? (end_ops > end_m ? end_ops : end_m) : (end_part > end_m ? end_part : end_m);   // a wave's norms
  static constexpr size_t total = nl + kKeyWaves * 32 * 4;
  static_assert(total <= 160 * 1024, "LDS map");
};

template <int NP>
__global__ __launch_bounds__(64 * kKeyWaves, 2) void k_sp_keys(const void* __restrict__ Kg, const void* __restrict__ Vg,
                                                               const float* __restrict__ M, const float* __restrict__ W,
                                                               us* __restrict__ Apl, us* __restrict__ St,
                                                               float* __restrict__ zt, float* __restrict__ ct, int H,
                                                               int L, int m, int w_shared, float alpha) {
  using SM = KeySmem<NP>;
  constexpr int NT = 64 * kKeyWaves;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const int l32 = lane % 32, hf = lane / 32, l16 = lane % 16, kg = lane / 16;
  us* Asl = reinterpret_cast<us*>(smem);
  us* Msl = reinterpret_cast<us*>(smem + SM::a_bytes);
  // neighbouring workgroups, which share a (b,h), go to one XCD
  const int n = gridDim.x, wg = n % 8 == 0 ? (blockIdx.x % 8) * (n / 8) + blockIdx.x / 8 : blockIdx.x;
  const int nblk = m / 32, bh = wg / nblk, f0 = 32 * (wg % nblk), h = bh % H;
  const int nt = (L + kTok - 1) / kTok;
  constexpr int KP = NP == 3 ? 8 : 4, CPR = NP == 3 ? 16 : 8;   // 16-byte pieces of a tile: per lane, per row
  u32x4 kr[KP], vr[KP];
  auto fetch = [&](int t) {
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      const int i = lane + 64 * u;
      const size_t at = (((size_t)bh * L + min(t * kTok + i / CPR, L - 1)) * CPR + i % CPR) * 16;
      kr[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const unsigned char*>(Kg) + at);
      vr[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const unsigned char*>(Vg) + at);
    }
  };
  {
    float* Wl = reinterpret_cast<float*>(smem + SM::off_w);   // [32][68]
    float* Ml = reinterpret_cast<float*>(smem + SM::off_m);   // [64][64]
    const f32x4* mr = reinterpret_cast<const f32x4*>(M + (size_t)h * kD * kD);
    const f32x4 w0 = reinterpret_cast<const f32x4*>(W + ((w_shared ? 0 : (size_t)h * m) + f0) * kD)[tid];
    const f32x4 m0 = mr[2 * tid], m1 = mr[2 * tid + 1];
    if (wv < nt) fetch(wv);
    __builtin_amdgcn_sched_barrier(0);
    *reinterpret_cast<f32x4*>(Wl + (tid / 16) * (kD + 4) + 4 * (tid % 16)) = w0;
    reinterpret_cast<f32x4*>(Ml)[2 * tid] = m0;
    reinterpret_cast<f32x4*>(Ml)[2 * tid + 1] = m1;
    const float fm = alpha * sqrtf(0.5f * kLog2e);
    u32x4 mp[3];
    split8(m0 * fm, m1 * fm, mp);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(Msl + (q * kD + tid / 8) * LDX + 8 * (tid % 8)) = mp[q];
    __syncthreads();
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) {   // the order of k_sp_prep: the same bits
        const int t = 16 * s + 4 * kg + j;
        acc[j % 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(Wl[(16 * (wv / 4) + l16) * (kD + 4) + t], Ml[t * kD + 16 * (wv % 4) + l16], acc[j % 2], 0, 0, 0);
      }
    acc[0] += acc[1];
    acc[0] *= alpha * kLog2e;
#pragma unroll
    for (int v = 0; v < 4; v += 2) {
      unsigned p[3];
      split_pair(acc[0][v], acc[0][v + 1], p[0], p[1], p[2]);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        us* d = Asl + (q * 32 + 16 * (wv / 4) + 4 * kg + v) * LDX + 16 * (wv % 4) + l16;
        d[0] = (us)(p[q] & 0xffffu);
        d[LDX] = (us)(p[q] >> 16);
      }
    }
  }
  __syncthreads();
  if (bh < H) {   // the first batch entry leaves the block of A' for the readout
    for (int i = tid; i < 3 * 256; i += NT) {
      const int q = i / 256, s = i / 64 % 4, fl = i % 64;
      *reinterpret_cast<u32x4*>(const_cast<us*>(a_frag(Apl, h, m, q, f0, s, fl))) =
          *reinterpret_cast<const u32x4*>(Asl + (q * 32 + fl % 32) * LDX + 16 * s + 8 * (fl / 32));
    }
  }
  f32x16 S[2] = {};
  float z = 0.f, c = -INFINITY;   // a wave without a tile counts for nothing
  float* nl = reinterpret_cast<float*>(smem + SM::nl) + 32 * wv;
  unsigned char* ts = smem + SM::off_t + wv * SM::t_bytes;
  const us *ap = Asl + l32 * LDX + 8 * hf, *mp = Msl + l32 * LDX + 8 * hf;
  const int jj = l32 % 16, tl = 4 * hf + jj / 4, kq = 2 * (l32 / 16) + (jj % 4) / 2;
  for (int t = wv; t < nt; t += kKeyWaves) {
    asm volatile("" ::: "memory");   // the last tile's values and norms have been read
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      const int i = lane + 64 * u;
      *reinterpret_cast<u32x4*>(ts + (i / CPR) * SM::KROW + 16 * (i % CPR)) = kr[u];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    u32x4 xf[4][NP];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      Raw8<NP> r;
      r.load(ts + l32 * SM::KROW, 16 * s + 8 * hf);
      r.planes(xf[s]);
    }
    asm volatile("" ::: "memory");   // (LDS operations of one wave complete in order)
#pragma unroll
    for (int u = 0; u < KP; ++u) {
      const int i = lane + 64 * u, row = i / CPR;
      if constexpr (NP == 3) {
        unsigned p[2][3];
        split_pair(__uint_as_float(vr[u][0]), __uint_as_float(vr[u][1]), p[0][0], p[0][1], p[0][2]);
        split_pair(__uint_as_float(vr[u][2]), __uint_as_float(vr[u][3]), p[1][0], p[1][1], p[1][2]);
        const int c4 = i % CPR;
#pragma unroll
        for (int q = 0; q < 3; ++q)
          *reinterpret_cast<u32x2*>(ts + (q * kTok + row) * 128 + 16 * ((c4 / 2) ^ v_swz<128>(row)) + 8 * (c4 % 2)) = u32x2{p[0][q], p[1][q]};
      } else {
        *reinterpret_cast<u32x4*>(ts + row * 128 + 16 * ((i % CPR) ^ v_swz<128>(row))) = vr[u];
      }
    }
    if (t + kKeyWaves < nt) fetch(t + kKeyWaves);
    float nn = 0.f;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      Logits x;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 a[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const u32x4*>(mp + (q * kD + 32 * rb) * LDX + 16 * s);
        x.add_ax(a, xf[s]);
      }
      const f32x16 xs = x.sum();
#pragma unroll
      for (int v = 0; v < 16; ++v) nn = fmaf(xs[v], xs[v], nn);
    }
    nn += xor32(nn);
    if (t * kTok + l32 >= L) nn = kTailNorm;
    if (hf == 0) nl[l32] = nn;
    Logits lg;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 a[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const u32x4*>(ap + q * 32 * LDX + 16 * s);
      lg.add_xa(xf[s], a);
    }
    f32x16 U = lg.sum();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 n4 = *reinterpret_cast<const f32x4*>(nl + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) U[4 * a + j] -= n4[j];
    }
    float mx = U[0];
#pragma unroll
    for (int v = 1; v < 15; v += 2) mx = max3(mx, U[v], U[v + 1]);
    mx = fmaxf(mx, U[15]);
    mx = fmaxf(mx, xor32(mx));
    const bool first = t < kKeyWaves;
    if (first || __any(mx > c + kRaise)) {   // set the wave's shifts, or raise them (rare), as in k_sp_states
      const float before = c;
      if (first || mx > c + kRaise) c = fmaxf(mx, -FLT_MAX);
      if (!first) {
        const float f = fast_exp2(before - c);
        z *= f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float fr = __shfl(f, 8 * (v / 4) + 4 * hf + (v % 4), 64);
          S[0][v] *= fr;
          S[1][v] *= fr;
        }
      }
    }
    float zs_t = 0.f;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 pk[3];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float e0 = fast_exp2(U[8 * hh + 2 * q] - c), e1 = fast_exp2(U[8 * hh + 2 * q + 1] - c);
        zs_t += e0;
        zs_t += e1;
        unsigned a, b, d;
        split_pair(e0, e1, a, b, d);
        pk[0][q] = a; pk[1][q] = b; pk[2][q] = d;
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        u32x4 vf[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          const unsigned char* r = ts + (q * kTok + 16 * hh + tl) * 128 + 16 * ((kq + 4 * b) ^ v_swz<128>(tl)) + 8 * (jj % 2);
          const u32x2 lo = lds_read_tr16(reinterpret_cast<const us*>(r)), hi = lds_read_tr16(reinterpret_cast<const us*>(r + 8 * 128));
          vf[q] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
        S[b] = mm_all(pk, vf, S[b]);
      }
    }
    z += zs_t;
  }
  __syncthreads();   // the operands have been read
  float* part = reinterpret_cast<float*>(smem + wv * SM::part);
  float* cz = reinterpret_cast<float*>(smem + SM::cz);
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) part[(8 * (v / 4) + 4 * hf + (v % 4)) * SM::LDE + 32 * b + l32] = S[b][v];
  z += xor32(z);
  if (hf == 0) {
    cz[64 * wv + l32] = c;
    cz[64 * wv + 32 + l32] = z;
  }
  __syncthreads();
  const int f = tid / 16, c4 = 4 * (tid % 16);
  float cw[kKeyWaves], cs = -INFINITY;
#pragma unroll
  for (int w = 0; w < kKeyWaves; ++w) {
    cw[w] = cz[64 * w + f];
    cs = fmaxf(cs, cw[w]);
  }
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float zs = 0.f;
#pragma unroll
  for (int w = 0; w < kKeyWaves; ++w) {
    const float fac = fast_exp2(cw[w] - cs);
    acc += fac * *reinterpret_cast<const f32x4*>(smem + w * SM::part + (f * SM::LDE + c4) * 4);
    zs = fmaf(fac, cz[64 * w + 32 + f], zs);
  }
  unsigned p[2][3];
  split_pair(acc[0], acc[1], p[0][0], p[0][1], p[0][2]);
  split_pair(acc[2], acc[3], p[1][0], p[1][1], p[1][2]);
  us* turn = reinterpret_cast<us*>(smem + SM::turn);
  const int pos = chain_pos(f);
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) turn[(q * kD + c4 + j) * 40 + pos] = (us)(j % 2 ? p[j / 2][q] >> 16 : p[j / 2][q] & 0xffffu);
  if (tid % 16 == 0) {
    zt[(size_t)bh * m + f0 + f] = zs;
    ct[(size_t)bh * m + f0 + f] = cs;
  }
  __syncthreads();
  for (int i = tid; i < 3 * kD * 4; i += NT) {
    const int q = i / 256, st = i / 128 % 2, b = i / 64 % 2, fl = i % 64;   // as in k_sp_merge
    *reinterpret_cast<u32x4*>(const_cast<us*>(at_frag(St, bh, m, q, f0 + 16 * st, b, fl))) =
        *reinterpret_cast<const u32x4*>(turn + (q * kD + 32 * b + fl % 32) * 40 + 16 * st + 8 * (fl / 32));
  }
}

// ---------------------------------------------------------------------------
// k_sp_readout: a wave owns 32 queries (lane = query): U^T[f][tok] = A' X^T, features along the registers, so the row
// shift, the denominator and the rescaling are per-lane scalars and phi^T enters N^T[c][tok] += S^T phi^T from the
// accumulator.  The features come in groups of 32 whose operands (planes of A' and S^T, 24 KB) go straight to LDS, a step ahead;
// with NWF = 2 two groups are there at a time and two waves share 32 queries, each taking every other group, their halves
// joined at the end.
// ---------------------------------------------------------------------------
constexpr unsigned kRdSlot = 2 * kOpBytes + kCzBytes;   // A', S^T, shifts and z of a group

template <int NP, int NWF, typename OutT>
__global__ __launch_bounds__(256 * NWF, 2) void k_sp_readout(const void* __restrict__ Qg, const us* __restrict__ Apl,
                                                             const us* __restrict__ St, const float* __restrict__ zt,
                                                             const float* __restrict__ ct, OutT* __restrict__ out,
                                                             int H, int L, int m, int wgs_per_bh) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hf = lane / 32;
  const int wf = NWF == 1 ? 0 : wv / 4, wt = wv % 4;
  const int bh = blockIdx.x / wgs_per_bh, h = bh % H;
  const int tok = (blockIdx.x % wgs_per_bh) * 4 * kTok + wt * kTok + l32;
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  Raw8<NP> xr[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) xr[s].load(Qg, ((size_t)bh * L + min(tok, L - 1)) * kD + 16 * s + 8 * hf);
  const us* const ops[2] = {a_frag(Apl, h, m, 0, 0, 0, 0), at_frag(St, bh, m, 0, 0, 0, 0)};
  const float *cb = ct + (size_t)bh * m, *zb = zt + (size_t)bh * m;
  const int ngrp = m / kGrp;   // even
  auto fetch = [&](int g0) {   // the four waves that use a group fetch it
    fetch_group<4>(ops, cb, zb, m, g0 + wf, smem + ((g0 / NWF & 1) * NWF + wf) * kRdSlot, wt, lane);
  };
  fetch(0);
  u32x4 xf[4][NP];
#pragma unroll
  for (int s = 0; s < 4; ++s) xr[s].planes(xf[s]);
  f32x16 N[2] = {zero16, zero16};
  float D = 0.f, mu = -INFINITY;
  for (int g0 = 0; g0 < ngrp; g0 += NWF) {
    group_barrier();
    if (g0 + NWF < ngrp) fetch(g0 + NWF);
    const unsigned char* sa = smem + ((g0 / NWF & 1) * NWF + wf) * kRdSlot;
    const unsigned char* ss = sa + kOpBytes;
    const float* cs = reinterpret_cast<const float*>(ss + kOpBytes);
    Logits lg;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 a[3];
      op_frag(a, sa, s, lane);
      lg.add_ax(a, xf[s]);
    }
    f32x16 U = lg.sum();
    float bm = -INFINITY;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 c4 = *reinterpret_cast<const f32x4*>(cs + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) U[4 * a + j] += c4[j];
      bm = max3(bm, fmaxf(U[4 * a], U[4 * a + 1]), fmaxf(U[4 * a + 2], U[4 * a + 3]));
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
    float Dg = 0.f;   // summed by group
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 pk[3];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const f32x4 z4 = *reinterpret_cast<const f32x4*>(cs + kGrp + 16 * hh + 8 * a + 4 * hf);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float e0 = fast_exp2(U[8 * hh + 4 * a + 2 * j] - mu), e1 = fast_exp2(U[8 * hh + 4 * a + 2 * j + 1] - mu);
          Dg = fmaf(e0, z4[2 * j], Dg);
          Dg = fmaf(e1, z4[2 * j + 1], Dg);
          unsigned p0, p1, p2;
          split_pair(e0, e1, p0, p1, p2);
          pk[0][2 * a + j] = p0; pk[1][2 * a + j] = p1; pk[2][2 * a + j] = p2;
        }
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        u32x4 sf[3];
        op_frag(sf, ss, 2 * hh + b, lane);
        N[b] = mm_all(sf, pk, N[b]);
      }
    }
    D += Dg;
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

// ---------------------------------------------------------------------------
// Backward (bidirectional).  With [S|z] as above, D_i = phi_Q,i . z, G = dOut:
//   gd_i = -G_i . out_i = -sum_j phi_Q,ij (S_j . G_i) / D_i,  [R|Rd]_j = sum_i phi_Q,ij / D_i [G_i | gd_i]
//   dl_Q,ij = phi_Q,ij / D_i (S_j . G_i + z_j gd_i),   dl_K,lj = phi_K,lj (R_j . v_l + Rd_j),   dV_l = sum_j phi_K,lj R_j
// G meets S and the features as it is, so that a bf16 G is one plane (G / D would be three), and gd comes from the terms that the
// logit gradients are made of: no numerator is formed.
//   dQ = dl_Q A,   dK_l = dl_K,l A - s_l alpha^2 M^T M k_l,   s_l = sum_j dl_K,lj     (A = A' / log2e)
//   T = dl_Q^T Q + dl_K^T K,   Rm = sum_l s_l k_l k_l^T,   dM = alpha W^T T - alpha^2 M Rm
// Features are recomputed where they are needed, in the orientation in which they are needed: a contraction over
// features wants a token per lane, one over tokens a feature per lane, and neither then passes anything between waves.
//   k_sp_bwd_q    (a wave: 32 queries)    mu, 1/D, gd of every query; dQ
//   k_sp_bwd_qs   (a wave: 32 features)   [R|Rd] and the query half of T, per slice
//   k_sp_bwd_k    (a wave: 32 keys)       dV, dK, s
//   k_sp_bwd_ks   (a wave: 32 features)   the key half of T, Rm, per slice
//   k_sp_sum, k_sp_dm                     sums over slices and batch, dM
//   k_sp_bwd_qf   the first two in one, bf16 inputs and m = 256
// B H L = 49,152, m = 256, bf16 inputs: k_sp_bwd_qf 42 us, k_sp_bwd_k 36, k_sp_bwd_ks 24 (fp32 general kernels, which write
// [rows, m] matrices and read them back in sixteen GEMMs: 620 us for the whole backward).
// ---------------------------------------------------------------------------
constexpr float kLn2 = 0.6931471805599453f;
// Planes of the eight accumulator entries of step hh: an operand fragment in chain order.
__device__ __forceinline__ void split_acc(const f32x16& x, int hh, u32x4 (&p)[3]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    unsigned a, b, c;
    split_pair(x[8 * hh + 2 * q], x[8 * hh + 2 * q + 1], a, b, c);
    p[0][q] = a; p[1][q] = b; p[2][q] = c;
  }
}
__device__ __forceinline__ f32x16 zero_acc() {
  return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}

// Two buffers, each a group's A', S, shifts and z, and A'^T for the second sweep.
constexpr unsigned kQT = 2 * kOpBytes + kCzBytes, kQBuf = kQT + kOpBytes;

template <int NP, int NW>
__global__ __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) void k_sp_bwd_q(
    const void* __restrict__ Qg, const void* __restrict__ Gg, const us* __restrict__ Apl, const us* __restrict__ Atp,
    const us* __restrict__ Sf, const float* __restrict__ zt, const float* __restrict__ ct, float* __restrict__ dQ,
    float* __restrict__ mu_out, float* __restrict__ rd_out, float* __restrict__ gd_out, int H, int L, int m,
    int wgs_per_bh) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wt = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hf = lane / 32;
  const int bh = blockIdx.x / wgs_per_bh, h = bh % H;
  const int tok = (blockIdx.x % wgs_per_bh) * NW * kTok + wt * kTok + l32;
  const size_t row = (size_t)bh * L + min(tok, L - 1);
  const int ngrp = m / kGrp;
  const us* const ops[2] = {a_frag(Apl, h, m, 0, 0, 0, 0), a_frag(Sf, bh, m, 0, 0, 0, 0)};
  const us* const opt[1] = {at_frag(Atp, h, m, 0, 0, 0, 0)};
  const float *cb = ct + (size_t)bh * m, *zb = zt + (size_t)bh * m;
  auto fetch = [&](int g, unsigned char* buf) { fetch_group<NW>(ops, cb, zb, m, g, buf, wt, lane); };
  auto fetch_t = [&](int g, unsigned char* buf) { fetch_group<NW>(opt, nullptr, nullptr, m, g, buf + kQT, wt, lane); };

  u32x4 xf[4][NP], gf[4][NP];
  {
    Raw8<NP> xr[4], gr[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      xr[s].load(Qg, row * kD + 16 * s + 8 * hf);
      gr[s].load(Gg, row * kD + 16 * s + 8 * hf);
    }
    fetch(0, smem);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      xr[s].planes(xf[s]);
      gr[s].planes(gf[s]);
    }
  }
  auto project = [&](const unsigned char* buf) {
    const float* cz = reinterpret_cast<const float*>(buf + 2 * kOpBytes);
    Logits lg;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 a[3];
      op_frag(a, buf, s, lane);
      lg.add_ax(a, xf[s]);
    }
    f32x16 U = lg.sum();
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 c4 = *reinterpret_cast<const f32x4*>(cz + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) U[4 * a + j] += c4[j];
    }
    return U;
  };
  // E + S G
  auto value_grad = [&](const unsigned char* buf, f32x16 E) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 a[3];
      op_frag(a, buf + kOpBytes, s, lane);
      E = mm_all(a, gf[s], E);
    }
    return E;
  };
  // first sweep: the denominator and G . N = sum_j phi_Q,j (S G)_j
  float D = 0.f, dot = 0.f, mu = -FLT_MAX;   // finite, though all features be zero
  for (int g = 0; g < ngrp; ++g) {
    const unsigned char* buf = smem + (g & 1) * kQBuf;
    group_barrier();
    if (g + 1 < ngrp) fetch(g + 1, smem + (~g & 1) * kQBuf);
    else if (dQ != nullptr) fetch_t(g, smem + (g & 1) * kQBuf);
    const f32x16 U = project(buf), E = value_grad(buf, zero_acc());
    float bm = U[0];
#pragma unroll
    for (int v = 1; v < 15; v += 2) bm = max3(bm, U[v], U[v + 1]);
    bm = fmaxf(bm, U[15]);
    // The row shift is the largest logit so far: all that a raise rescales is two sums, and with features of up to 2^kRaise the
    // products with G, which is not divided by D, would leave the fp32 range that much earlier.
    const float mn = fmaxf(mu, fmaxf(bm, xor32(bm))), f = fast_exp2(mu - mn);
    mu = mn;
    D *= f;
    dot *= f;
    float Dg = 0.f, dg = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 z4 = *reinterpret_cast<const f32x4*>(buf + 2 * kOpBytes + (kGrp + 8 * a + 4 * hf) * 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float e = fast_exp2(U[4 * a + j] - mu);
        Dg = fmaf(e, z4[j], Dg);
        dg = fmaf(e, E[4 * a + j], dg);
      }
    }
    D += Dg;
    dot += dg;
  }
  D += xor32(D);
  dot += xor32(dot);
  const float rd = tok < L ? 1.f / D : 0.f, gd = -dot * rd;
  if (hf == 0 && tok < L) {
    mu_out[row] = mu;
    rd_out[row] = rd;
    gd_out[row] = gd;
  }
  if (dQ == nullptr) return;
  // second sweep, backwards (the last group's operands are still there): dl_Q and dQ
  f32x16 X[2] = {zero_acc(), zero_acc()};   // dQ^T
  for (int g = ngrp - 1; g >= 0; --g) {
    const unsigned char* buf = smem + (g & 1) * kQBuf;
    group_barrier();
    if (g > 0) {
      fetch(g - 1, smem + (~g & 1) * kQBuf);
      fetch_t(g - 1, smem + (~g & 1) * kQBuf);
    }
    const f32x16 U = project(buf);
    f32x16 E;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 z4 = *reinterpret_cast<const f32x4*>(buf + 2 * kOpBytes + (kGrp + 8 * a + 4 * hf) * 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) E[4 * a + j] = gd * z4[j];
    }
    E = value_grad(buf, E);
#pragma unroll
    for (int v = 0; v < 16; ++v) E[v] *= fast_exp2(U[v] - mu) * rd;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 pk[3];
      split_acc(E, hh, pk);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        u32x4 tf[3];
        op_frag(tf, buf + kQT, 2 * hh + b, lane);
        X[b] = mm_all(tf, pk, X[b]);
      }
    }
  }
  if (tok >= L) return;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 w = {X[b][4 * a] * kLn2, X[b][4 * a + 1] * kLn2, X[b][4 * a + 2] * kLn2, X[b][4 * a + 3] * kLn2};
      *reinterpret_cast<f32x4*>(dQ + row * kD + 32 * b + 8 * a + 4 * hf) = w;
    }
}

// Two buffers, each a group's A', R, R^T, A'^T, shifts and Rd; at the end alpha^2 M^T M.
constexpr unsigned kKBuf = 4 * kOpBytes + kCzBytes;

template <int NP, int NW>
__global__ __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) void k_sp_bwd_k(
    const void* __restrict__ Kg, const void* __restrict__ Vg, const us* __restrict__ Apl, const us* __restrict__ Atp,
    const us* __restrict__ G2p, const us* __restrict__ Rt, const us* __restrict__ Rf, const float* __restrict__ Rd,
    const float* __restrict__ ct, const float* __restrict__ nrm, float* __restrict__ dK, float* __restrict__ dV,
    float* __restrict__ s_out, int H, int L, int m, int wgs_per_bh) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wt = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hf = lane / 32;
  const int bh = blockIdx.x / wgs_per_bh, h = bh % H;
  const int tok = (blockIdx.x % wgs_per_bh) * NW * kTok + wt * kTok + l32;
  const size_t row = (size_t)bh * L + min(tok, L - 1);
  const int ngrp = m / kGrp;
  const us* const ops[4] = {a_frag(Apl, h, m, 0, 0, 0, 0), a_frag(Rf, bh, m, 0, 0, 0, 0), at_frag(Rt, bh, m, 0, 0, 0, 0),
                            at_frag(Atp, h, m, 0, 0, 0, 0)};
  const us* const g2[2] = {a_frag(G2p, h, kD, 0, 0, 0, 0), a_frag(G2p, h, kD, 0, kGrp, 0, 0)};
  auto fetch = [&](int g) { fetch_group<NW>(ops, ct + (size_t)bh * m, Rd + (size_t)bh * m, m, g, smem + (g & 1) * kKBuf, wt, lane); };
  u32x4 xf[4][NP], vf[4][NP];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    Raw8<NP> xr, vr;
    xr.load(Kg, row * kD + 16 * s + 8 * hf);
    vr.load(Vg, row * kD + 16 * s + 8 * hf);
    xr.planes(xf[s]);
    vr.planes(vf[s]);
  }
  const float n = nrm[row];
  fetch(0);
  f32x16 Xv[2] = {zero_acc(), zero_acc()}, Xk[2] = {zero_acc(), zero_acc()};   // dV^T, dK^T
  float s_l = 0.f;
  for (int g = 0; g < ngrp; ++g) {
    const unsigned char* buf = smem + (g & 1) * kKBuf;
    group_barrier();
    if (g + 1 < ngrp) {
      fetch(g + 1);
    } else {   // 64 rows, as two operands
      fetch_group<NW>(g2, nullptr, nullptr, kD, 0, smem + (~g & 1) * kKBuf, wt, lane);
    }
    const float* cz = reinterpret_cast<const float*>(buf + 4 * kOpBytes);
    Logits lg;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 a[3];
      op_frag(a, buf, s, lane);
      lg.add_ax(a, xf[s]);
    }
    f32x16 U = lg.sum(), E;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 c4 = *reinterpret_cast<const f32x4*>(cz + 8 * a + 4 * hf);
      const f32x4 r4 = *reinterpret_cast<const f32x4*>(cz + kGrp + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        U[4 * a + j] = fast_exp2(U[4 * a + j] - n - c4[j]);
        E[4 * a + j] = r4[j];
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 a[3];
      op_frag(a, buf + kOpBytes, s, lane);
      E = mm_all(a, vf[s], E);
    }
    float sg = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      E[v] *= U[v];
      sg += E[v];
    }
    s_l += sg;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 pk[3];
      split_acc(U, hh, pk);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        u32x4 a[3];
        op_frag(a, buf + 2 * kOpBytes, 2 * hh + b, lane);
        Xv[b] = mm_all(a, pk, Xv[b]);
      }
      split_acc(E, hh, pk);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        u32x4 a[3];
        op_frag(a, buf + 3 * kOpBytes, 2 * hh + b, lane);
        Xk[b] = mm_all(a, pk, Xk[b]);
      }
    }
  }
  s_l += xor32(s_l);
  // the norm term: - s alpha^2 M^T M k
  group_barrier();
  const unsigned char* opg = smem + (ngrp & 1) * kKBuf;
  const bool valid = tok < L;   // every lane holds rows of the operands: none may leave before the last MFMA
  if (hf == 0 && valid) s_out[row] = s_l;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    f32x16 Y = zero_acc();
    if (dK != nullptr) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 a[3];
        op_frag(a, opg + b * kOpBytes, s, lane);
        Y = mm_all(a, xf[s], Y);
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      f32x4 wk, wv;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        wk[j] = Xk[b][4 * a + j] * kLn2 - s_l * Y[4 * a + j];
        wv[j] = Xv[b][4 * a + j];
      }
      if (dK != nullptr && valid) *reinterpret_cast<f32x4*>(dK + row * kD + 32 * b + 8 * a + 4 * hf) = wk;
      if (dV != nullptr && valid) *reinterpret_cast<f32x4*>(dV + row * kD + 32 * b + 8 * a + 4 * hf) = wv;
    }
  }
}

// The passes with a feature per lane.  KEYS == false (k_sp_bwd_qs): tokens are queries, the second tensor is G;
// [R|Rd] += (phi_Q / D)^T [G|gd], T += dl_Q^T Q.  KEYS == true (k_sp_bwd_ks): tokens are keys, the
// second tensor is V;  T += dl_K^T K on top of the query half, and Rm += (s k)^T k, a 32 x 32 block in each of the first
// four 32-feature waves.  Tiles of 32 tokens as planes, rows of 128 bytes with the chunk swizzle of the transposing
// reads, under which the row reads are free of bank conflicts too; two buffers, one barrier per tile.
template <int NP, bool KEYS>
struct FsSmem {
  static constexpr int NS = KEYS ? 3 : 0;           // planes of s k
  static constexpr size_t pl = (size_t)kTok * 128;
  static constexpr size_t y = NP * pl, sx = y + NP * pl, sc = sx + NS * pl;
  static constexpr size_t buf = sc + (KEYS ? 1 : 3) * kTok * 4;
  static constexpr size_t total = 2 * buf;
};

template <int NP, int NW, bool KEYS>
__global__ __launch_bounds__(64 * NW, NW == 8 ? 2 : 1) void k_sp_bwd_fs(
    const void* __restrict__ Xg, const void* __restrict__ Yg, const us* __restrict__ Apl, const us* __restrict__ Sf,
    const float* __restrict__ zt, const float* __restrict__ ct, const float* __restrict__ row_a,
    const float* __restrict__ row_b, const float* __restrict__ row_c, float* __restrict__ Rpart,
    float* __restrict__ Rdpart, float* __restrict__ Tpart, float* __restrict__ Rmpart, int H, int L, int m, int P,
    int slice_len, int nfb) {
  // row_a: mu (queries), n' (keys);  row_b: 1/D, s;  row_c: gd, -.   Sf, zt: S, z (queries), R, Rd (keys)
  using SM = FsSmem<NP, KEYS>;
  constexpr int NT = 64 * NW, NTASK = 512 / NT;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  const int l32 = lane % 32, hf = lane / 32;
  const int fb = blockIdx.x % nfb, work = blockIdx.x / nfb;
  const int bh = work / P, p = work % P, h = bh % H;
  const int tok_begin = p * slice_len, tok_end = min(L, tok_begin + slice_len);
  const int ntile = (tok_end - tok_begin + kTok - 1) / kTok;
  const int f0 = fb * 256 + wv * 32;
  const bool active = f0 < m;
  const int fr = min(f0, m - 32) + l32;   // this lane's feature

  Raw8<NP> st[NTASK];
  float sb[NTASK];            // keys: s of the X rows
  float sa = 0.f, sr = 0.f, sc = 0.f;
  auto fetch = [&](int t) {
#pragma unroll
    for (int u = 0; u < NTASK; ++u) {
      const int i = tid + NT * u, c = i % 256, tk = tok_begin + t * kTok + c / 8;
      const size_t r = (size_t)bh * L + min(tk, tok_end - 1);
      st[u].load(i < 256 ? Xg : Yg, r * kD + 8 * (c % 8));
      sb[u] = KEYS && i < 256 && tk < tok_end ? row_b[r] : 0.f;
    }
    if (tid < kTok) {
      const int tk = tok_begin + t * kTok + tid;
      const size_t r = (size_t)bh * L + min(tk, tok_end - 1);
      sa = tk < tok_end ? row_a[r] : kTailNorm;
      if (!KEYS) {
        sr = tk < tok_end ? row_b[r] : 0.f;
        sc = tk < tok_end ? row_c[r] : 0.f;
      }
    }
  };
  auto store = [&](int t) {
    unsigned char* base = smem + (t & 1) * SM::buf;
#pragma unroll
    for (int u = 0; u < NTASK; ++u) {
      const int i = tid + NT * u, c = i % 256, row = c / 8, at = row * 128 + 16 * ((c % 8) ^ v_swz<128>(row));
      {
        u32x4 pl[NP];
        st[u].planes(pl);
#pragma unroll
        for (int q = 0; q < NP; ++q) *reinterpret_cast<u32x4*>(base + (i < 256 ? 0 : SM::y) + q * SM::pl + at) = pl[q];
      }
      if (KEYS && i < 256) {   // s k, three planes
        f32x4 lo, hi;
        if constexpr (NP == 3) {
          lo = st[u].lo;
          hi = st[u].hi;
        } else {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            lo[2 * q] = __uint_as_float(st[u].w[q] << 16);
            lo[2 * q + 1] = __uint_as_float(st[u].w[q] & 0xffff0000u);
            hi[2 * q] = __uint_as_float(st[u].w[2 + q] << 16);
            hi[2 * q + 1] = __uint_as_float(st[u].w[2 + q] & 0xffff0000u);
          }
        }
        u32x4 pl[3];
        split8(lo * sb[u], hi * sb[u], pl);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(base + SM::sx + q * SM::pl + at) = pl[q];
      }
    }
    if (tid < kTok) {
      reinterpret_cast<float*>(base + SM::sc)[tid] = sa;
      if (!KEYS) {
        reinterpret_cast<float*>(base + SM::sc)[kTok + tid] = sr;
        reinterpret_cast<float*>(base + SM::sc)[2 * kTok + tid] = sc;
      }
    }
  };

  fetch(0);
  // operands of this wave's features: A' (k = d) and S or R (k = c), one feature per lane
  u32x4 af[4][3], sf[4][3];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      af[s][q] = *reinterpret_cast<const u32x4*>(a_frag(Apl, h, m, q, min(f0, m - 32), s, lane));
      sf[s][q] = *reinterpret_cast<const u32x4*>(a_frag(Sf, bh, m, q, min(f0, m - 32), s, lane));
    }
  const float cf = ct[(size_t)bh * m + fr], zf = zt[(size_t)bh * m + fr];
  const size_t ob = ((size_t)bh * P + p) * m + f0;
  f32x16 R[2] = {zero_acc(), zero_acc()}, T[2] = {zero_acc(), zero_acc()};
  float rdsum = 0.f;
  if (KEYS && active) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) T[b][v] = Tpart[(ob + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32];
  }
  store(0);
  __syncthreads();
  const int jj = l32 % 16, tl = 4 * hf + jj / 4, kq = 2 * (l32 / 16) + (jj % 4) / 2;
  unsigned voff[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) voff[b] = tl * 128 + 16 * ((kq + 4 * b) ^ v_swz<128>(tl)) + 8 * (jj % 2);
  // the same element order (chain order of the tokens) for an operand of token columns: column 32 b + l32
  auto frag_t = [&](const unsigned char* plane, int hh, int b) {
    const unsigned char* vr = plane + hh * 16 * 128 + voff[b];
    const u32x2 lo = lds_read_tr16(reinterpret_cast<const us*>(vr));
    const u32x2 hi = lds_read_tr16(reinterpret_cast<const us*>(vr + 8 * 128));
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  };
  const unsigned roff = l32 * 128;
  const int rsw = v_swz<128>(l32);

  for (int t = 0; t < ntile; ++t) {
    if (t + 1 < ntile) fetch(t + 1);
    const unsigned char* base = smem + (t & 1) * SM::buf;
    if (active) {
      const float* scal = reinterpret_cast<const float*>(base + SM::sc);
      Logits lg;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 x[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) x[q] = *reinterpret_cast<const u32x4*>(base + q * SM::pl + roff + 16 * ((2 * s + hf) ^ rsw));
        lg.add_xa(x, af[s]);
      }
      f32x16 U = lg.sum(), E;
      float rdt = 0.f;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 a4 = *reinterpret_cast<const f32x4*>(scal + 8 * a + 4 * hf);
        f32x4 r4, d4 = {1.f, 1.f, 1.f, 1.f};
        if (!KEYS) {
          r4 = *reinterpret_cast<const f32x4*>(scal + kTok + 8 * a + 4 * hf);
          d4 = *reinterpret_cast<const f32x4*>(scal + 2 * kTok + 8 * a + 4 * hf);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          U[4 * a + j] = fast_exp2(KEYS ? U[4 * a + j] - a4[j] - cf : U[4 * a + j] + cf - a4[j]);
          if (!KEYS) U[4 * a + j] *= r4[j];
          E[4 * a + j] = d4[j] * zf;
          if (!KEYS) rdt = fmaf(U[4 * a + j], d4[j], rdt);
        }
      }
      rdsum += rdt;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        u32x4 y[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q)
          y[q] = *reinterpret_cast<const u32x4*>(base + SM::y + q * SM::pl + roff + 16 * ((2 * s + hf) ^ rsw));
        E = mm_all(y, sf[s], E);
      }
      E *= U;
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        u32x4 pk[3];
        if constexpr (!KEYS) {
          split_acc(U, hh, pk);
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            u32x4 y[NP];
#pragma unroll
            for (int q = 0; q < NP; ++q) y[q] = frag_t(base + SM::y + q * SM::pl, hh, b);
            R[b] = mm_all(pk, y, R[b]);
          }
        }
        split_acc(E, hh, pk);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          u32x4 x[NP];
#pragma unroll
          for (int q = 0; q < NP; ++q) x[q] = frag_t(base + q * SM::pl, hh, b);
          T[b] = mm_all(pk, x, T[b]);
        }
      }
    }
    if (KEYS && fb == 0) {
      // Rm block (e, b) of wave 2 e + b (of waves 0 and 1 alone when the workgroup has only two)
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          if (NW >= 4 ? wv == 2 * e + b : wv == b) {
            f32x16& acc = R[NW >= 4 ? 0 : e];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
              u32x4 sx[3], x[NP];
#pragma unroll
              for (int q = 0; q < 3; ++q) sx[q] = frag_t(base + SM::sx + q * SM::pl, hh, e);
#pragma unroll
              for (int q = 0; q < NP; ++q) x[q] = frag_t(base + q * SM::pl, hh, b);
              acc = mm_all(sx, x, acc);
            }
          }
    }
    if (t + 1 < ntile) store(t + 1);
    __syncthreads();
  }
  if (active) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const size_t o = (ob + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32;
        Tpart[o] = T[b][v];
        if (!KEYS) Rpart[o] = R[b][v];
      }
    if (!KEYS) {
      rdsum += xor32(rdsum);
      if (hf == 0) Rdpart[ob + l32] = rdsum;
    }
  }
  if (KEYS && fb == 0) {
    float* rm = Rmpart + ((size_t)bh * P + p) * kD * kD;
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        if (NW >= 4 ? wv == 2 * e + b : wv == b) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            rm[(32 * e + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32] = R[NW >= 4 ? 0 : e][v];
        }
  }
}

// A wave's 32 x 32 block (lane = token, registers = features) turned in its own LDS patch: planes [32 tokens][32 features],
// read back with the feature per lane and the tokens of step hh in chain order.
constexpr int kPatchRow = 32 + 4;   // 16-bit elements
constexpr size_t kPatchPlane = (size_t)32 * kPatchRow * 2;
__device__ __forceinline__ void patch_write(unsigned char* patch, const f32x16& x, int lane) {
  const int l32 = lane % 32, hf = lane / 32;
  asm volatile("" ::: "memory");   // what the patch held has been read
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    unsigned p0[3], p1[3];
    split_pair(x[4 * a], x[4 * a + 1], p0[0], p0[1], p0[2]);
    split_pair(x[4 * a + 2], x[4 * a + 3], p1[0], p1[1], p1[2]);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      *reinterpret_cast<u32x2*>(patch + q * kPatchPlane + (l32 * kPatchRow + 8 * a + 4 * hf) * 2) = u32x2{p0[q], p1[q]};
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ void patch_read(u32x4 (&p)[3], const unsigned char* patch, int hh, int lane) {
  const int l32 = lane % 32, hf = lane / 32, jj = l32 % 16;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const us* r = reinterpret_cast<const us*>(patch + q * kPatchPlane) + (16 * hh + 4 * hf + jj / 4) * kPatchRow +
                  16 * (l32 / 16) + 4 * (jj % 4);
    const u32x2 lo = lds_read_tr16(r), hi = lds_read_tr16(r + 8 * kPatchRow);
    p[q] = u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
}

// k_sp_bwd_qf: what k_sp_bwd_q and k_sp_bwd_qs do, in one pass over the features, for bf16 inputs and m = 256: eight waves hold
// all features of a (b,h), 32 each, and walk a slice of tokens in tiles of 32 (lane = token).
//   first half   logits, e = 2^(u - mu) under the wave's own row shift, S G; the wave's parts of D and of G . N
//   second half  D, gd from the eight parts; phi / D and dl_Q;  dl_Q (registers) times A'^T gives the wave's part of dQ; both are
//                turned in the wave's own LDS slot for [R|Rd] and T, which stay in registers; the part of dQ takes the slot
// and the parts of dQ are added in the first half of the next tile, one 16-byte piece a thread, in wave order.  Two barriers a tile.
// A' is needed both ways round: two planes as rows in LDS (read straight and transposed), the third in registers, as is S.
// Against the two passes: 72 instead of 96 products a wave and tile, and half of the exponentials and splits.  24 x 2048 tokens:
// 35 + 27 -> 42 us (one head of 65, the whole step: 109 -> 73).  A tile takes some 11,000 cycles, for 4,600 of matrix pipe and 4,900 of
// vector issue: bound by issue and by the chain of a tile with all of a SIMD's two waves in the same half of it.  The third planes
// and the order of the second half are what fits 256 registers; with spills the kernel took 60 us, since a reload waits for the
// next tile's rows.
// PAST: dK, dV, dM or dW is wanted too.  dQ alone needs neither R nor T (48 products) and no slices to sum over, so that few heads of
// a long sequence still fill the chip; the bits of dQ are the same.  dQ alone, us, two passes (as they are now) / with R and T /
// without: one head of 65,536 tokens 105 / 207 / 98, of 2048 48 / 33 / 29; 24 x 2048 62 / 68 / 56.  All gradients, two passes / fused:
// one head of 2048 113 / 90, 16,384 153 / 144, 32,768 197 / 204, 131,072 545 / 604 (64 slices on 256 CUs; 649 before the fused pass);
// two heads of 65,536 398 / 374, six 868 / 797.
struct QfSmem {
  static constexpr size_t pl = (size_t)256 * 128;                   // a plane of A'
  static constexpr size_t slot = (size_t)kTok * kD * 4;             // part of dQ of a wave; before that its turned blocks
  static constexpr size_t tile = (size_t)kTok * 128, buf = 2 * tile;   // Q, G
  static constexpr size_t x = 2 * pl, t = x + 8 * slot, part = t + 2 * buf, cz = part + 3 * kTok * 8 * 4;
  static constexpr size_t total = cz + 2 * 256 * 4;
};
constexpr int kTurnRow = 36;   // floats
__device__ __forceinline__ void stage() { __builtin_amdgcn_sched_barrier(0); }   // keeps the scheduler from mixing what would not fit the registers
static_assert((size_t)kTok * kTurnRow * 4 <= QfSmem::slot && 3 * 32 * (32 + 4) * 2 <= QfSmem::slot, "turned blocks fit a slot");
static_assert(QfSmem::total <= 160 * 1024, "LDS of a CU");

template <bool PAST>
__global__ __launch_bounds__(512, 2) void k_sp_bwd_qf(
    const us* __restrict__ Qg, const us* __restrict__ Gg, const us* __restrict__ Apl, const us* __restrict__ Atp,
    const us* __restrict__ Sf, const float* __restrict__ zt, const float* __restrict__ ct, float* __restrict__ dQ,
    float* __restrict__ Rpart, float* __restrict__ Rdpart, float* __restrict__ Tpart, int H, int L, int P, int slice_len) {
  using SM = QfSmem;
  constexpr int m = 256;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hf = lane / 32;
  const int bh = blockIdx.x / P, p = blockIdx.x % P, h = bh % H;
  const int tok_begin = p * slice_len, tok_end = min(L, tok_begin + slice_len);
  const int ntile = (tok_end - tok_begin + kTok - 1) / kTok;
  const int f0 = 32 * wv;
  float* part = reinterpret_cast<float*>(smem + SM::part);
  const float* cz = reinterpret_cast<const float*>(smem + SM::cz);
  unsigned char* slot = smem + SM::x + wv * SM::slot;

  // staging: four waves bring the rows of Q, four those of G; lane i of a wave fills position i % 8 of row i / 8 of its eight
  const int srow = 8 * (wv % 4) + lane / 8;
  const us* src = (wv < 4 ? Qg : Gg) + (size_t)bh * L * kD + 8 * (lane % 8 ^ v_swz<128>(srow));
  auto fetch = [&](int t) {
    dma16_to_lds(src + (size_t)min(tok_begin + t * kTok + srow, tok_end - 1) * kD, smem + SM::t + (t & 1) * SM::buf + wv * 1024);
  };
  fetch(0);
  {
    float* w = reinterpret_cast<float*>(smem + SM::cz);
    w[tid] = tid < m ? ct[(size_t)bh * m + tid] : zt[(size_t)bh * m + tid - m];
  }
  u32x4 sf[4][2], sf2[4], ar2[4];
  // the third planes, anew for every tile: to hold them takes registers that the second half needs
  auto third = [&]() {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      sf2[s] = *reinterpret_cast<const u32x4*>(a_frag(Sf, bh, m, 2, f0, s, lane));
      ar2[s] = *reinterpret_cast<const u32x4*>(a_frag(Apl, h, m, 2, f0, s, lane));
    }
  };
  const int rsw = v_swz<128>(l32);
  const unsigned roff = l32 * 128;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int q = 0; q < 2; ++q) sf[s][q] = *reinterpret_cast<const u32x4*>(a_frag(Sf, bh, m, q, f0, s, lane));
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<u32x4*>(smem + q * SM::pl + f0 * 128 + roff + 16 * ((2 * s + hf) ^ rsw)) =
          *reinterpret_cast<const u32x4*>(a_frag(Apl, h, m, q, f0, s, lane));
  }
  wait_vmcnt0();
  third();
  lds_barrier();

  // The lane's parts of the LDS offsets: rows (16-byte chunk hf; chunk 2 s + hf by exclusive or), transposed, and the lane's piece of
  // a part of dQ.  Renewed every tile: otherwise the compiler carries every sum of them across the loop and spills.
  const int jj = l32 % 16, tl = 4 * hf + jj / 4, kq = 2 * (l32 / 16) + (jj % 4) / 2;
  unsigned dir = roff + 16 * (hf ^ rsw), tr = tl * 128 + 16 * (kq ^ v_swz<128>(tl)) + 8 * (jj % 2);
  unsigned own = (unsigned)SM::x + wv * (unsigned)SM::slot + l32 * 256 + 16 * (hf ^ (l32 & 15));
  unsigned turn = (unsigned)SM::x + wv * (unsigned)SM::slot + (4 * hf * kTurnRow + l32) * 4;   // a feature's column of the turned block
  auto ld128 = [&](unsigned at) { return *reinterpret_cast<const u32x4*>(smem + at); };
  auto frag_t = [&](unsigned plane, int hh, int b) {   // column 32 b + l32, rows of step hh in chain order
    const us* vr = reinterpret_cast<const us*>(smem + ((tr ^ (64 * b)) + plane + hh * 16 * 128));
    const u32x2 lo = lds_read_tr16(vr), hi = lds_read_tr16(vr + 8 * 64);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  };
  // the parts of dQ of tile t: thread i adds columns 4 (i % 16) + [0,4) of token i / 16
  auto reduce_dq = [&](int t) {
    const int tk = tid / 16, c = tid % 16, at = tk * 256 + 16 * (c ^ (tk & 15));
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 8; ++w) a += *reinterpret_cast<const f32x4*>(smem + SM::x + w * SM::slot + at);
    const int tok = tok_begin + t * kTok + tk;
    if (tok < tok_end) *reinterpret_cast<f32x4*>(dQ + ((size_t)bh * L + tok) * kD + 4 * c) = a * kLn2;
  };

  // LDS operations of one wave complete in order: between what the wave writes to its slot and what it reads back
  auto turned = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  f32x16 R[2] = {zero_acc(), zero_acc()}, T[2] = {zero_acc(), zero_acc()};
  float rdsum = 0.f;
  for (int t = 0; t < ntile; ++t) {
    const unsigned base = (unsigned)SM::t + (t & 1) * (unsigned)SM::buf, ap = f0 * 128;
    asm volatile("" : "+v"(dir), "+v"(tr), "+v"(own), "+v"(turn));
    // ---- first half ----
    f32x16 U, E = zero_acc();
    {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const u32x4 y[1] = {ld128((dir ^ (32 * s)) + base + (unsigned)SM::tile)};
        const u32x4 a[3] = {sf[s][0], sf[s][1], sf2[s]};
        E = mm_all(a, y, E);
      }
      Logits lg;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const unsigned at = dir ^ (32 * s);
        const u32x4 x[1] = {ld128(at + base)};
        const u32x4 a[3] = {ld128(at + ap), ld128(at + ap + (unsigned)SM::pl), ar2[s]};
        lg.add_ax(a, x);
      }
      U = lg.sum();
    }
    stage();
    if (t + 1 < ntile) fetch(t + 1);
    if (dQ != nullptr && t > 0) reduce_dq(t - 1);
    stage();
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 c4 = *reinterpret_cast<const f32x4*>(cz + f0 + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) U[4 * a + j] += c4[j];
    }
    float mu = U[0];
#pragma unroll
    for (int v = 1; v < 15; v += 2) mu = max3(mu, U[v], U[v + 1]);
    mu = fmaxf(mu, U[15]);
    mu = fmaxf(fmaxf(mu, xor32(mu)), -FLT_MAX);   // finite, though all features of the wave be zero
    float den = 0.f, dot = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 z4 = *reinterpret_cast<const f32x4*>(cz + m + f0 + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float e = fast_exp2(U[4 * a + j] - mu);
        U[4 * a + j] = e;
        den = fmaf(e, z4[j], den);
        dot = fmaf(e, E[4 * a + j], dot);
      }
    }
    den += xor32(den);
    dot += xor32(dot);
    if (hf == 0) {
      part[l32 * 8 + wv] = mu;
      part[(kTok + l32) * 8 + wv] = den;
      part[(2 * kTok + l32) * 8 + wv] = dot;
    }
    lds_barrier();
    // ---- second half ----
    float mx = -INFINITY, D = 0.f, N = 0.f;
    {
      f32x4 m4[2], d4[2], o4[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        m4[k] = *reinterpret_cast<const f32x4*>(part + l32 * 8 + 4 * k);
        d4[k] = *reinterpret_cast<const f32x4*>(part + (kTok + l32) * 8 + 4 * k);
        o4[k] = *reinterpret_cast<const f32x4*>(part + (2 * kTok + l32) * 8 + 4 * k);
        mx = max3(mx, fmaxf(m4[k][0], m4[k][1]), fmaxf(m4[k][2], m4[k][3]));
      }
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const float f = fast_exp2(m4[w / 4][w % 4] - mx);
        D = fmaf(f, d4[w / 4][w % 4], D);
        N = fmaf(f, o4[w / 4][w % 4], N);
      }
    }
    const float rd = tok_begin + t * kTok + l32 < tok_end ? 1.f / D : 0.f, gd = -N * rd, rw = rd * fast_exp2(mu - mx);
    u32x4 at2[4];   // the third plane of A'^T, on its way while phi is turned
    if (dQ != nullptr) {
#pragma unroll
      for (int i = 0; i < 4; ++i) at2[i] = *reinterpret_cast<const u32x4*>(at_frag(Atp, h, m, 2, f0 + 16 * (i / 2), i % 2, lane));
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 z4 = *reinterpret_cast<const f32x4*>(cz + m + f0 + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        U[4 * a + j] *= rw;
        E[4 * a + j] = U[4 * a + j] * fmaf(gd, z4[j], E[4 * a + j]);
      }
      if (PAST) *reinterpret_cast<f32x4*>(slot + (l32 * kTurnRow + 8 * a + 4 * hf) * 4) = f32x4{U[4 * a], U[4 * a + 1], U[4 * a + 2], U[4 * a + 3]};
    }
    if (PAST && hf == 0) reinterpret_cast<float*>(slot + kTok * kTurnRow * 4)[l32] = gd;   // of the tile's tokens
    turned();
    stage();
    f32x16 X[2] = {zero_acc(), zero_acc()};   // this wave's part of dQ^T
    {
      u32x4 pk[2][3];   // dl_Q
      f32x16 Ft;        // phi / D, feature per lane
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) split_acc(E, hh, pk[hh]);
      float rdt = 0.f;
      if (PAST) {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const f32x4 g4 = *reinterpret_cast<const f32x4*>(slot + kTok * kTurnRow * 4 + (8 * a + 4 * hf) * 4);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            Ft[4 * a + j] = *reinterpret_cast<const float*>(smem + turn + (8 * a + j) * kTurnRow * 4);
            rdt = fmaf(Ft[4 * a + j], g4[j], rdt);
          }
        }
        rdsum += rdt;
        turned();
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int q = 0; q < 3; ++q)
            *reinterpret_cast<u32x2*>(slot + q * kPatchPlane + (l32 * kPatchRow + 8 * a + 4 * hf) * 2) =
                u32x2{pk[a / 2][q][2 * (a % 2)], pk[a / 2][q][2 * (a % 2) + 1]};
        turned();
      }
      if (dQ != nullptr) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const u32x4 a[3] = {frag_t(ap, hh, b), frag_t(ap + (unsigned)SM::pl, hh, b), at2[2 * hh + b]};
            X[b] = mm_all(a, pk[hh], X[b]);
          }
      }
      // [R|Rd] += (phi / D)^T [G|gd]
      if (PAST) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          u32x4 pf[3];
          split_acc(Ft, hh, pf);
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const u32x4 y[1] = {frag_t(base + (unsigned)SM::tile, hh, b)};
            R[b] = mm_all(pf, y, R[b]);
          }
        }
      }
    }
    stage();
    if (PAST) {
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        u32x4 pk[3];
        patch_read(pk, slot, hh, lane);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const u32x4 x[1] = {frag_t(base, hh, b)};
          T[b] = mm_all(pk, x, T[b]);
        }
      }
    }
    turned();
    if (dQ != nullptr) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 4; ++a)
          *reinterpret_cast<f32x4*>(smem + (own ^ (128 * b + 32 * a))) = f32x4{X[b][4 * a], X[b][4 * a + 1], X[b][4 * a + 2], X[b][4 * a + 3]};
    }
    wait_vmcnt0();   // the next tile
    third();
    lds_barrier();
  }
  if (dQ != nullptr) reduce_dq(ntile - 1);
  if (!PAST) return;
  const size_t ob = ((size_t)bh * P + p) * m + f0;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const size_t o = (ob + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32;
      Tpart[o] = T[b][v];
      Rpart[o] = R[b][v];
    }
  rdsum += xor32(rdsum);
  if (hf == 0) Rdpart[ob + l32] = rdsum;
}

// Per head: Tsum = sum over batch entries and slices of T, Rmsum likewise, in ascending order; sixteen slices requested
// together (memory round trips are all there is).
__global__ __launch_bounds__(256) void k_sp_sum(const float* __restrict__ T, const float* __restrict__ Rm,
                                                float* __restrict__ Tsum, float* __restrict__ Rmsum, int B, int H, int m,
                                                int P) {
  const long long per4 = ((long long)m + kD) * kD / 4;
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= H * per4) return;
  const int h = (int)(idx / per4);
  const long long e = 4 * (idx % per4), te = (long long)m * kD;
  const bool ist = e < te;
  const size_t pitch = ist ? (size_t)te : (size_t)kD * kD;
  const float* src = ist ? T + e : Rm + (e - te);
  f32x4 run = {0.f, 0.f, 0.f, 0.f};
  const int n = B * P;
  auto add = [&](auto batch, int s0) {
    constexpr int NB = decltype(batch)::value;
    f32x4 v[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int i = min(s0 + u, n - 1);
      v[u] = *reinterpret_cast<const f32x4*>(src + (((size_t)(i / P) * H + h) * P + i % P) * pitch);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NB; ++u)
      if (s0 + u < n) run += v[u];
  };
  int s0 = 0;
  for (; s0 + 8 < n; s0 += 16) add(std::integral_constant<int, 16>{}, s0);
  if (s0 < n) add(std::integral_constant<int, 8>{}, s0);
  *reinterpret_cast<f32x4*>(ist ? Tsum + (size_t)h * te + e : Rmsum + (size_t)h * kD * kD + (e - te)) = run;
}

// dM[h][r][d] = alpha sum_j W[h][j][r] Tsum[h][j][d] - alpha^2 sum_e M[h][r][e] Rmsum[h][e][d]: one block per (h, 16 rows, 32
// columns), a quarter of j and of e per wave by fp32 MFMAs 16x16x4 with operands straight from memory (m / 16 steps, sixteen in
// flight), the four parts joined in LDS.  A thread per element with its chain of 16 loads after 16 loads: 8.8 us at 12 heads,
// m = 256, now 5.0 us.
__global__ __launch_bounds__(256) void k_sp_dm(const float* __restrict__ Tsum, const float* __restrict__ Rmsum,
                                               const float* __restrict__ M, const float* __restrict__ W,
                                               float* __restrict__ dM, int m, int w_shared, float alpha) {
  __shared__ float part[4][16][32 + 1];
  const int h = blockIdx.x / 8, r0 = 16 * (blockIdx.x % 4), d0 = 32 * (blockIdx.x / 4 % 2);
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64, l16 = lane % 16, kg = lane / 16;
  const int ns = m / 16, j0 = wv * (m / 4) + kg;
  const float* wp = W + (w_shared ? 0 : (size_t)h * m * kD) + (size_t)j0 * kD + r0 + l16;
  const float* tp = Tsum + ((size_t)h * m + j0) * kD + d0 + l16;
  const f32x4 mr = *reinterpret_cast<const f32x4*>(M + ((size_t)h * kD + r0 + l16) * kD + 16 * wv + 4 * kg) * -alpha;
  const float* rp = Rmsum + ((size_t)h * kD + 16 * wv + 4 * kg) * kD + d0 + l16;
  float rm[4][2];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int t = 0; t < 2; ++t) rm[j][t] = rp[j * kD + 16 * t];
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  for (int s0 = 0; s0 < ns; s0 += 16) {
    float a[16], b[16][2];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int at = 4 * min(s0 + u, ns - 1) * kD;
      a[u] = wp[at];
#pragma unroll
      for (int t = 0; t < 2; ++t) b[u][t] = tp[at + 16 * t];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (s0 + u < ns) {   // uniform
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], b[u][t], acc[t], 0, 0, 0);
      }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(mr[j], rm[j][t], acc[t], 0, 0, 0);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wv][4 * kg + v][16 * t + l16] = acc[t][v];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int r = tid / 32 + 8 * u, c = tid % 32;
    dM[((size_t)h * kD + r0 + r) * kD + d0 + c] = alpha * ((part[0][r][c] + part[1][r][c]) + (part[2][r][c] + part[3][r][c]));
  }
}

// ---------------------------------------------------------------------------
// Causal form (m <= 256).  The sequence is cut into chunks of 32 positions; the state of every chunk comes from
// k_sp_states (slices of one tile), and
//   k_sp_scan    exclusive prefix states, in the running maximum c_j of the chunks' shifts (a key is never stored under
//                a shift set by a later chunk), as operand planes of every chunk
//   k_sp_causal  a workgroup per chunk, a wave per 32 features: N = phi_Q S_before + A V, D = phi_Q z_before + A 1 with
//                the masked tile A_il = phi_Q,i . phi_K,l; the waves' halves of N, D, A meet in LDS once.
// Nothing but the tensors, the prefix states and the results is in memory, and a problem of a few thousand positions
// still has a wave for every SIMD; what bounds it are the memory round trips and chains of dependent products of one
// wave, not a pipe.  fp32 training step, 8 heads, L = 1000, m = 128: 103 us in twelve launches (two passes of 18 and 17 us,
// scans of 8 to 11); the general kernels take 383 us in fifty.
//
// Backward (notation of the bidirectional one; [S|z] before the chunk plus the tile, [R|Rd] after it plus the tile; l <= i in a tile):
//   gd_i = -(sum_j phi_Q,ij (S_j . G_i) + sum_l A_il (G_i . v_l)) / D_i,   E_il = G_i . v_l + gd_i
//   dl_Q,ij = phi_Q,ij / D_i (S_j . G_i + z_j gd_i + sum_l E_il phi_K,lj)
//   dl_K,lj = phi_K,lj (R_j . v_l + Rd_j + sum_i phi_Q,ij E_il / D_i),     dV_l = sum_j phi_K,lj R_j + sum_i A_il G_i / D_i
//   k_sp_causal_q     dQ, the chunk's [R|Rd] and query half of T; leaves mu, 1/D and the tiles A, E / D
//   k_sp_scan (reverse)  exclusive suffix sums of [R|Rd], brought to each chunk's shifts
//   k_sp_causal_k     dV, dK, the key half of T, Rm
// ---------------------------------------------------------------------------

// Operand fragments of a chunk's 64 x m state whose contraction index is the feature: [step of 16 features][32 columns]
// [plane][lane][8], so that a wave's fragment is one contiguous kilobyte.
__device__ __forceinline__ size_t frag_at(int step, int cb, int pl) { return (size_t)((step * 2 + cb) * 3 + pl) * 512; }

// k_sp_scan: exclusive running sums of the chunk states of one (b,h), eight features a workgroup, 32 chunks a pass.
// REV: from the last chunk to the first.  St: fragments over features (above).  The factors between the chunks' shifts
// depend on feature and chunk only and are formed once, by scans over the lanes of a wave per feature, and left in LDS.  Thread = one
// column, eight features and a segment of four chunks, whose states it holds in registers: the eight segments are walked at
// the same time, once for their sums, which meet in LDS, and once for the results.  Every store of a wave is a whole kilobyte (with
// four features a thread two waves wrote half lines each).  8 heads, 32 chunks, m = 128: 9.5 -> 8.4 us; with the factors by one thread
// per feature, entry after entry, 9.5 -> 9.2 us.
template <bool REV>
__global__ __launch_bounds__(512) void k_sp_scan(const float* __restrict__ Spart, const float* __restrict__ zpart,
                                                 const float* __restrict__ cpart, us* __restrict__ St,
                                                 float* __restrict__ zpre, float* __restrict__ cpre, int m, int nc) {
  constexpr int SEG = 8, LEN = 4, NK = SEG * LEN;
  __shared__ __attribute__((aligned(16))) float sh[NK][8], down[NK][8], up[NK][8], zs[NK][8];
  __shared__ f32x4 sums[SEG][2][64];
  __shared__ f32x4 sdown[SEG][2];   // a segment's whole factor
  const int tid = threadIdx.x, nblk = m / 8, bh = blockIdx.x / nblk, blk = blockIdx.x % nblk;
  const int c = tid % 64, seg = tid / 64;
  // feature q of the workgroup (q = 4 quad + j): a fragment's eight are [0,4) and [8,12) from fb
  const int fb = 16 * (blk / 2) + 4 * (blk % 2);
  const size_t frag = frag_at(fb / 16, c / 32, 0) + ((c % 32) + 32 * (blk % 2)) * 8;
  const int kq = tid / 8, q8 = tid % 8, fq = fb + 8 * (q8 / 4) + q8 % 4;   // chunk and feature of the factor phase
  auto chunk_at = [&](int k) { return (size_t)bh * nc + (REV ? nc - 1 - k : k); };
  f32x4 run[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};   // the sum of all chunks before the pass, under the shift of the last of them
  float zrun = 0.f, carry_c = REV ? 0.f : -INFINITY;   // feature of this wave (factor phase): likewise for z; that shift
  for (int k0 = 0; k0 < nc; k0 += NK) {
    const int np = min(NK, nc - k0), kb = seg * LEN;
    f32x4 v[LEN][2];
#pragma unroll
    for (int u = 0; u < LEN; ++u) {
      const size_t r = chunk_at(k0 + min(kb + u, np - 1)) * m + fb;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[u][j / 4][j % 4] = Spart[(r + 8 * (j / 4) + j % 4) * kD + c];
    }
    if (tid < NK * 8) {
      const size_t r = chunk_at(k0 + min(kq, np - 1)) * m + fq;
      sh[kq][q8] = cpart[r];
      zs[kq][q8] = zpart[r];
    }
    __syncthreads();
    {
      // wave w: feature w of the workgroup, lane k: chunk k0 + k.  Running shifts, factors, and z by scans over the lanes (z is a
      // chain of affine maps r -> down r + up z); lanes past the last chunk repeat its shift with factor one and nothing added
      const int w = tid / 64, k = min(tid % 64, np - 1);
      const bool in = tid % 64 < np;
      const int fw = fb + 8 * (w / 4) + w % 4;
      const float ck = sh[k][w], zk = zs[k][w];
      float to = REV ? ck : fmaxf(ck, carry_c);
      if (!REV)
#pragma unroll
        for (int o = 1; o < NK; o <<= 1) {
          const float x = __shfl_up(to, o, 64);
          if (tid % 64 >= o) to = fmaxf(to, x);
        }
      float prev = __shfl_up(to, 1, 64);
      if (tid % 64 == 0) prev = carry_c;
      const float dn = !in ? 1.f : k0 + k > 0 ? fast_exp2(REV ? to - prev : prev - to) : 0.f;
      const float u = !in ? 0.f : REV ? 1.f : fast_exp2(ck - to);
      float D = dn, U = u * zk;
#pragma unroll
      for (int o = 1; o < NK; o <<= 1) {
        const float xD = __shfl_up(D, o, 64), xU = __shfl_up(U, o, 64);
        if (tid % 64 >= o) {
          U = fmaf(xU, D, U);
          D *= xD;
        }
      }
      const float r = fmaf(zrun, D, U);
      float rb = __shfl_up(r, 1, 64);
      if (tid % 64 == 0) rb = zrun;
      if (in) {
        down[k][w] = dn;
        up[k][w] = u;
        const size_t at = chunk_at(k0 + k) * m + fw;
        if (!REV) cpre[at] = to;
        zpre[at] = rb * dn;
      }
      carry_c = __shfl(to, NK - 1, 64);
      zrun = __shfl(r, NK - 1, 64);
    }
    __syncthreads();
    // the segment's own sum under its last shift
    f32x4 sr[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, sd[2] = {{1.f, 1.f, 1.f, 1.f}, {1.f, 1.f, 1.f, 1.f}};
#pragma unroll
    for (int u = 0; u < LEN; ++u)
      if (kb + u < np) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const f32x4 d = *reinterpret_cast<const f32x4*>(&down[kb + u][4 * g]), f = *reinterpret_cast<const f32x4*>(&up[kb + u][4 * g]);
          sr[g] = sr[g] * d + f * v[u][g];
          sd[g] *= d;
        }
      }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      sums[seg][g][c] = sr[g];
      if (c == 0) sdown[seg][g] = sd[g];
    }
    __syncthreads();
    f32x4 br[2] = {run[0], run[1]};
    for (int q = 0; q < SEG; ++q)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        if (q == seg) br[g] = run[g];
        run[g] = run[g] * sdown[q][g] + sums[q][g][c];   // an empty segment has factor one and sum zero
      }
#pragma unroll
    for (int u = 0; u < LEN; ++u)
      if (kb + u < np) {
        us* st = St + chunk_at(k0 + kb + u) * 3 * kD * m + frag;
#pragma unroll
        for (int g = 0; g < 2; ++g) br[g] *= *reinterpret_cast<const f32x4*>(&down[kb + u][4 * g]);
        u32x4 pl[3];
        split8(br[0], br[1], pl);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x4*>(st + q * 512) = pl[q];
#pragma unroll
        for (int g = 0; g < 2; ++g) br[g] += *reinterpret_cast<const f32x4*>(&up[kb + u][4 * g]) * v[u][g];
      }
    __syncthreads();
  }
}

// Operand fragments read straight from memory.
__device__ __forceinline__ void a_frags(u32x4 (&a)[3], const us* Apl, int h, int m, int f, int s, int lane) {
#pragma unroll
  for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const u32x4*>(a_frag(Apl, h, m, q, f, s, lane));
}
__device__ __forceinline__ void at_frags(u32x4 (&a)[3], const us* Atp, int h, int m, int f, int b, int lane) {
#pragma unroll
  for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const u32x4*>(at_frag(Atp, h, m, q, f, b, lane));
}
// The planes of a chunk's queries and keys in LDS, [queries, keys][plane][32][LDX], split by all waves together from whole
// lines (a wave that fetches and splits its own fragments repeats the other waves' work).
template <int NP>
struct RowStage {
  static constexpr size_t bytes = (size_t)2 * NP * kTok * LDX * 2;
  Raw8<NP> r[4];   // two waves have four pieces of eight elements each
  __device__ __forceinline__ void load(const void* Qg, const void* Kg, size_t row0, int nvalid, int tid, int nt) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = tid + nt * u, c = i % 256;
      if (i < 512) r[u].load(i < 256 ? Qg : Kg, (row0 + min(c / 8, nvalid - 1)) * kD + 8 * (c % 8));   // wave-uniform
    }
  }
  __device__ __forceinline__ void store(unsigned char* dst, int tid, int nt) const {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = tid + nt * u, c = i % 256;
      if (i < 512) {
        u32x4 p[NP];
        r[u].planes(p);
#pragma unroll
        for (int q = 0; q < NP; ++q)
          *reinterpret_cast<u32x4*>(dst + (((i / 256) * NP + q) * kTok + c / 8) * LDX * 2 + 16 * (c % 8)) = p[q];
      }
    }
  }
  static __device__ __forceinline__ void frag(u32x4 (&p)[NP], const unsigned char* src, int which, int s, int lane) {
#pragma unroll
    for (int q = 0; q < NP; ++q)
      p[q] = *reinterpret_cast<const u32x4*>(src + ((which * NP + q) * kTok + lane % 32) * LDX * 2 + 32 * s + 16 * (lane / 32));
  }
};
__device__ __forceinline__ void chunk_frag(u32x4 (&a)[3], const us* st, int step, int cb, int lane) {
#pragma unroll
  for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const u32x4*>(st + frag_at(step, cb, q) + lane * 8);
}
// Columns of a [tokens][64] tensor as operand rows: column 32 b + lane % 32, tokens of step hh in chain order.  Rows past the end are
// zero.
template <int NP>
__device__ __forceinline__ void col_values(float (&x)[8], const void* base, size_t row0, int nvalid, int hh, int b, int lane) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int t = 16 * hh + 8 * (e / 4) + 4 * (lane / 32) + e % 4;
    const size_t at = (row0 + min(t, nvalid - 1)) * kD + 32 * b + lane % 32;
    float v;
    if constexpr (NP == 3) v = reinterpret_cast<const float*>(base)[at];
    else v = __uint_as_float((unsigned)reinterpret_cast<const us*>(base)[at] << 16);
    x[e] = t < nvalid ? v : 0.f;
  }
}
__device__ __forceinline__ void split_values(const float (&x)[8], u32x4 (&p)[3]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    unsigned a, b, c;
    split_pair(x[2 * q], x[2 * q + 1], a, b, c);
    p[0][q] = a; p[1][q] = b; p[2][q] = c;
  }
}
template <int NP>
__device__ __forceinline__ void col_planes(const float (&x)[8], u32x4 (&p)[NP]) {
  if constexpr (NP == 3) {
    split_values(x, p);
  } else {   // bf16 values: their upper halves are the numbers
#pragma unroll
    for (int q = 0; q < 4; ++q) p[0][q] = __builtin_amdgcn_perm(__float_as_uint(x[2 * q + 1]), __float_as_uint(x[2 * q]), 0x07060302u);
  }
}
// per-token factors of step hh in chain order, from LDS
__device__ __forceinline__ void chain_scalars(float (&f)[8], const float* lds, int hh, int hf) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(lds + 16 * hh + 4 * hf), b = *reinterpret_cast<const f32x4*>(lds + 16 * hh + 8 + 4 * hf);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[e] = a[e];
    f[4 + e] = b[e];
  }
}
// A wave's 32 features of a chunk state, turned: from the fragments over features (St above) into the wave's LDS area
// [plane][64 columns][32 features], to be read with a feature per lane and the columns as the contraction index.
constexpr size_t kTurnPlane = (size_t)64 * kPatchRow * 2;
typedef u32x4 StateFrags[2][2][3];
__device__ __forceinline__ void load_state(StateFrags& s, const us* st, int step0, int lane) {
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int b = 0; b < 2; ++b) chunk_frag(s[hh][b], st, step0 + hh, b, lane);
}
__device__ __forceinline__ void turn_state(unsigned char* area, const StateFrags& s, int lane) {
  asm volatile("" ::: "memory");   // what the area held has been read
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 3; ++q) {   // a lane's eight: features 16 hh + 4 hf + [0,4) and 16 hh + 8 + 4 hf + [0,4) of its column
        us* d = reinterpret_cast<us*>(area + q * kTurnPlane) + (32 * b + lane % 32) * kPatchRow + 16 * hh + 4 * (lane / 32);
        *reinterpret_cast<u32x2*>(d) = u32x2{s[hh][b][q][0], s[hh][b][q][1]};
        *reinterpret_cast<u32x2*>(d + 8) = u32x2{s[hh][b][q][2], s[hh][b][q][3]};
      }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// columns 16 s + 8 hf + [0,8)
__device__ __forceinline__ void turned_frag(u32x4 (&p)[3], const unsigned char* area, int s, int lane) {
  const int l32 = lane % 32, hf = lane / 32, jj = l32 % 16;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const us* r = reinterpret_cast<const us*>(area + q * kTurnPlane) + (16 * s + 8 * hf + jj / 4) * kPatchRow +
                  16 * (l32 / 16) + 4 * (jj % 4);
    const u32x2 lo = lds_read_tr16(r), hi = lds_read_tr16(r + 4 * kPatchRow);
    p[q] = u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
}

struct CausalSmem {
  static constexpr size_t scal = 3 * 32 * 4;                 // per-token scalars
  static constexpr size_t spart = scal, ynorm = spart + 8 * 32 * 4;   // key pass: a wave's part of s; the norm term [2][32][32]
  static constexpr size_t ex = ynorm + 2 * 32 * 32 * 4;
  // A wave's area.  In turn: the rows of all waves; the turned state (14 KB, backward); what the waves exchange (forward: N, A, D, mu,
  // 13 KB; query side of the backward: A, mu, D, G.N, 5 KB); the patch, in the upper half; the wave's part of dQ in the lower half, or
  // its parts of dV and dK (8 KB each).
  static constexpr size_t ex_wave = (size_t)64 * 64 * 4, patch = 8192;
  __host__ __device__ static constexpr size_t total(int nw) { return ex + nw * ex_wave; }
};
static_assert(CausalSmem::patch + 3 * kPatchPlane <= CausalSmem::ex_wave && 3 * kTurnPlane <= CausalSmem::ex_wave &&
                  CausalSmem::total(8) <= 160 * 1024 && RowStage<3>::bytes <= 2 * CausalSmem::ex_wave, "LDS map");

template <int NP, typename OutT>
__global__ __launch_bounds__(512, 2) void k_sp_causal(
    const void* __restrict__ Qg, const void* __restrict__ Kg, const void* __restrict__ Vg, const us* __restrict__ Apl,
    const us* __restrict__ St, const float* __restrict__ zpre, const float* __restrict__ cpre, const float* __restrict__ nrm,
    OutT* __restrict__ out, int H, int L, int m, int nc) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64, nw = blockDim.x / 64;
  const int l32 = lane % 32, hf = lane / 32;
  const size_t chunk = blockIdx.x;
  const int bh = blockIdx.x / nc, h = bh % H;
  const int t0 = (blockIdx.x % nc) * kTok, nvalid = min(kTok, L - t0);
  const size_t row0 = (size_t)bh * L + t0, row = row0 + min(l32, nvalid - 1);
  const int f0 = 32 * wv;
  unsigned char* ex = smem + CausalSmem::ex;

  RowStage<NP> rows;
  rows.load(Qg, Kg, row0, nvalid, tid, blockDim.x);
  u32x4 af[4][3];
#pragma unroll
  for (int s = 0; s < 4; ++s) a_frags(af[s], Apl, h, m, f0, s, lane);
  StateFrags sf;
  load_state(sf, St + chunk * 3 * kD * m, f0 / 16, lane);
  const float n = l32 < nvalid ? nrm[row] : kTailNorm;
  f32x4 c4[4], z4[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    c4[a] = *reinterpret_cast<const f32x4*>(cpre + chunk * m + f0 + 8 * a + 4 * hf);
    z4[a] = *reinterpret_cast<const f32x4*>(zpre + chunk * m + f0 + 8 * a + 4 * hf);
  }
  rows.store(ex, tid, blockDim.x);
  lds_barrier();
  Logits lq, lk;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    u32x4 xq[NP], xk[NP];
    RowStage<NP>::frag(xq, ex, 0, s, lane);
    RowStage<NP>::frag(xk, ex, 1, s, lane);
    lq.add_ax(af[s], xq);
    lk.add_ax(af[s], xk);
  }
  f32x16 U = lq.sum(), Fk = lk.sum();   // query logits, key features; a token per lane, features along the registers
  float mu = -INFINITY, D = 0.f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      U[4 * a + j] += c4[a][j];
      Fk[4 * a + j] = fast_exp2(Fk[4 * a + j] - n - c4[a][j]);
      mu = fmaxf(mu, U[4 * a + j]);
    }
  }
  mu = fmaxf(mu, xor32(mu));
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      U[4 * a + j] = fast_exp2(U[4 * a + j] - mu);
      D = fmaf(U[4 * a + j], z4[a][j], D);
    }
  D += xor32(D);
  f32x16 N[2] = {zero_acc(), zero_acc()}, At = zero_acc();   // At: registers = keys l, lane = query i
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pq[3], pk[3];
    split_acc(U, hh, pq);
    split_acc(Fk, hh, pk);
    At = mm_all(pk, pq, At);
#pragma unroll
    for (int b = 0; b < 2; ++b) N[b] = mm_all(sf[hh][b], pq, N[b]);
  }
  float vc[2][8];   // columns of V, of the first two waves
  if (wv < 2) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) col_values<NP>(vc[hh], Vg, row0, nvalid, hh, wv, lane);
  }
  // the waves' parts meet
  lds_barrier();   // the rows have been read
  {
    float* o = reinterpret_cast<float*>(ex + (size_t)wv * CausalSmem::ex_wave) + 4 * lane;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      *reinterpret_cast<f32x4*>(o + 256 * a) = f32x4{N[0][4 * a], N[0][4 * a + 1], N[0][4 * a + 2], N[0][4 * a + 3]};
      *reinterpret_cast<f32x4*>(o + 256 * (4 + a)) = f32x4{N[1][4 * a], N[1][4 * a + 1], N[1][4 * a + 2], N[1][4 * a + 3]};
      *reinterpret_cast<f32x4*>(o + 256 * (8 + a)) = f32x4{At[4 * a], At[4 * a + 1], At[4 * a + 2], At[4 * a + 3]};
    }
    *reinterpret_cast<f32x4*>(o + 256 * 12) = f32x4{D, mu, 0.f, 0.f};
  }
  lds_barrier();
  if (wv >= 2) return;   // two waves finish
  for (int w = 0; w < nw; ++w) mu = fmaxf(mu, reinterpret_cast<const float*>(ex + (size_t)w * CausalSmem::ex_wave)[4 * lane + 256 * 12 + 1]);
  N[0] = N[1] = At = zero_acc();
  D = 0.f;
  for (int w = 0; w < nw; ++w) {
    const float* o = reinterpret_cast<const float*>(ex + (size_t)w * CausalSmem::ex_wave) + 4 * lane;
    const f32x4 dm = *reinterpret_cast<const f32x4*>(o + 256 * 12);
    const float f = fast_exp2(dm[1] - mu);
    D = fmaf(f, dm[0], D);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(o + 256 * a), y = *reinterpret_cast<const f32x4*>(o + 256 * (4 + a)),
                  z = *reinterpret_cast<const f32x4*>(o + 256 * (8 + a));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        N[0][4 * a + j] = fmaf(f, x[j], N[0][4 * a + j]);
        N[1][4 * a + j] = fmaf(f, y[j], N[1][4 * a + j]);
        At[4 * a + j] = fmaf(f, z[j], At[4 * a + j]);
      }
    }
  }
  float ad = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    if (8 * (v / 4) + 4 * hf + (v % 4) > l32) At[v] = 0.f;
    ad += At[v];
  }
  D += ad + xor32(ad);
  // N^T[c][i] += sum_l v_l[c] A_il (half of the columns in each of the first two waves)
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pa[3];
    split_acc(At, hh, pa);
    u32x4 v[NP];
    col_planes<NP>(vc[hh], v);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (b != wv) continue;
      N[b] = mm_all(v, pa, N[b]);
    }
  }
  if (l32 >= nvalid) return;
  const float inv = 1.f / D;
  OutT* o = out + row * kD + 4 * hf;
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    if (b != wv) continue;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 w = {N[b][4 * a] * inv, N[b][4 * a + 1] * inv, N[b][4 * a + 2] * inv, N[b][4 * a + 3] * inv};
      if constexpr (sizeof(OutT) == 4) *reinterpret_cast<f32x4*>(o + 32 * b + 8 * a) = w;
      else *reinterpret_cast<u32x2*>(o + 32 * b + 8 * a) = u32x2{pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
    }
  }
}

// The query side of the backward, a wave per 32 features.  As in the bidirectional passes G meets the states and the values as it is
// and G.N is summed from the terms of the logit gradients, sum_f phi_f (S G)_f + sum_l a_il G.v_l: no numerator is formed, and what the
// waves exchange is their parts of the kernel values, of D and of that sum (5 KB a wave; with N, 13).  Up to m = 128 a wave has its
// SIMD to itself and nothing but its own instructions to hide a round trip behind: the states, V, and the columns of G and Q are asked
// for a phase or more before their use, barriers wait for LDS only, and the stores of R and T come last.  8 heads, L = 1000, m = 128:
// 26 -> 18.3 us (26 still without the requests ahead: of 41,000 cycles some 20,000 were waits).
template <int NP>
__global__ __launch_bounds__(512, 2) void k_sp_causal_q(
    const void* __restrict__ Qg, const void* __restrict__ Kg, const void* __restrict__ Vg, const void* __restrict__ Gg,
    const us* __restrict__ Apl, const us* __restrict__ Atp, const us* __restrict__ St,
    const float* __restrict__ zpre, const float* __restrict__ cpre, const float* __restrict__ nrm, float* __restrict__ dQ,
    float* __restrict__ mu_out, float* __restrict__ rd_out, float* __restrict__ Atile, float* __restrict__ Etile,
    float* __restrict__ Rpart, float* __restrict__ Rdpart, float* __restrict__ Tpart, int H, int L, int m, int nc) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64, nw = blockDim.x / 64;
  const int l32 = lane % 32, hf = lane / 32;
  const size_t chunk = blockIdx.x;
  const int bh = blockIdx.x / nc, h = bh % H;
  const int t0 = (blockIdx.x % nc) * kTok, nvalid = min(kTok, L - t0);
  const size_t row0 = (size_t)bh * L + t0, row = row0 + min(l32, nvalid - 1);
  const int f0 = 32 * wv;
  float* scal = reinterpret_cast<float*>(smem);   // gd of the tile's queries
  unsigned char* ex = smem + CausalSmem::ex;
  unsigned char* area = ex + (size_t)wv * CausalSmem::ex_wave;
  unsigned char* patch = area + CausalSmem::patch;

  RowStage<NP> rows;
  rows.load(Qg, Kg, row0, nvalid, tid, blockDim.x);
  u32x4 af[4][3];
#pragma unroll
  for (int s = 0; s < 4; ++s) a_frags(af[s], Apl, h, m, f0, s, lane);
  StateFrags sf;
  load_state(sf, St + chunk * 3 * kD * m, f0 / 16, lane);
  Raw8<NP> gr[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) gr[s].load(Gg, row * kD + 16 * s + 8 * hf);
  const float n = l32 < nvalid ? nrm[row] : kTailNorm;
  rows.store(ex, tid, blockDim.x);
  lds_barrier();
  f32x16 U, Fk;   // query logits, key features; a token per lane, features along the registers
  {
    Logits lq, lk;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 xq[NP], xk[NP];
      RowStage<NP>::frag(xq, ex, 0, s, lane);
      RowStage<NP>::frag(xk, ex, 1, s, lane);
      lq.add_ax(af[s], xq);
      lk.add_ax(af[s], xk);
    }
    U = lq.sum();
    Fk = lk.sum();
  }
  Raw8<NP> vr[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) vr[s].load(Vg, row * kD + 16 * s + 8 * hf);
  f32x4 c4[4], z4[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    c4[a] = *reinterpret_cast<const f32x4*>(cpre + chunk * m + f0 + 8 * a + 4 * hf);
    z4[a] = *reinterpret_cast<const f32x4*>(zpre + chunk * m + f0 + 8 * a + 4 * hf);
  }
  lds_barrier();   // the rows have been read
  turn_state(area, sf, lane);
  u32x4 gf[4][NP];
#pragma unroll
  for (int s = 0; s < 4; ++s) gr[s].planes(gf[s]);
  // S G (registers = features) and G.v_l (registers = keys), lane = query
  f32x16 P = zero_acc(), E = zero_acc(), At = zero_acc();
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    u32x4 v[NP], a[3];
    turned_frag(a, area, s, lane);
    P = mm_all(a, gf[s], P);
    vr[s].planes(v);
    E = mm_all(v, gf[s], E);
  }
  float mu = -INFINITY, D = 0.f, dot = 0.f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      U[4 * a + j] += c4[a][j];
      Fk[4 * a + j] = fast_exp2(Fk[4 * a + j] - n - c4[a][j]);
      mu = fmaxf(mu, U[4 * a + j]);
    }
  }
  mu = fmaxf(mu, xor32(mu));
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      U[4 * a + j] = fast_exp2(U[4 * a + j] - mu);
      D = fmaf(U[4 * a + j], z4[a][j], D);
      dot = fmaf(U[4 * a + j], P[4 * a + j], dot);
    }
  D += xor32(D);
  dot += xor32(dot);
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {   // At: registers = keys l, lane = query i
    u32x4 pq[3], pk[3];
    split_acc(U, hh, pq);
    split_acc(Fk, hh, pk);
    At = mm_all(pk, pq, At);
  }
  // the waves' parts meet: every wave reads them all.  They lie below the patches, and what takes their place is written two barriers on
  asm volatile("" ::: "memory");   // the turned state has been read
  {
    float* o = reinterpret_cast<float*>(area) + 4 * lane;
#pragma unroll
    for (int a = 0; a < 4; ++a)
      *reinterpret_cast<f32x4*>(o + 256 * a) = f32x4{At[4 * a], At[4 * a + 1], At[4 * a + 2], At[4 * a + 3]};
    *reinterpret_cast<f32x4*>(o + 256 * 4) = f32x4{mu, D, dot, 0.f};
  }
  patch_write(patch, Fk, lane);
  float gc[2][2][8], qc[2][2][8];   // columns of G and Q, for R and T
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      col_values<NP>(gc[hh][b], Gg, row0, nvalid, hh, b, lane);
      col_values<NP>(qc[hh][b], Qg, row0, nvalid, hh, b, lane);
    }
  lds_barrier();
  const float mu_own = mu;
  for (int w = 0; w < nw; ++w) mu = fmaxf(mu, reinterpret_cast<const float*>(ex + (size_t)w * CausalSmem::ex_wave)[4 * lane + 256 * 4]);
  At = zero_acc();
  D = dot = 0.f;
  for (int w = 0; w < nw; ++w) {
    const float* o = reinterpret_cast<const float*>(ex + (size_t)w * CausalSmem::ex_wave) + 4 * lane;
    const f32x4 md = *reinterpret_cast<const f32x4*>(o + 256 * 4);
    const float f = fast_exp2(md[0] - mu);
    D = fmaf(f, md[1], D);
    dot = fmaf(f, md[2], dot);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(o + 256 * a);
#pragma unroll
      for (int j = 0; j < 4; ++j) At[4 * a + j] = fmaf(f, x[j], At[4 * a + j]);
    }
  }
  float ad = 0.f, ed = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    if (8 * (v / 4) + 4 * hf + (v % 4) > l32) At[v] = E[v] = 0.f;
    ad += At[v];
    ed = fmaf(At[v], E[v], ed);
  }
  D += ad + xor32(ad);
  dot += ed + xor32(ed);
  const float rd = l32 < nvalid ? 1.f / D : 0.f, gd = -dot * rd;
  U *= fast_exp2(mu_own - mu) * rd;   // phi_Q / D
#pragma unroll
  for (int v = 0; v < 16; ++v) E[v] = 8 * (v / 4) + 4 * hf + (v % 4) > l32 ? 0.f : E[v] + gd;
  if (wv == 0 && hf == 0) {
    scal[l32] = gd;
    if (l32 < nvalid) {
      mu_out[row] = mu;
      rd_out[row] = rd;
    }
  }
  if (wv < 2) {   // the tiles, rows = keys; E for features that are not divided by D (infinite 1/D: not beyond the mask)
    float* dst = (wv == 0 ? Atile : Etile) + chunk * kTok * kTok + l32;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int l = 8 * (v / 4) + 4 * hf + (v % 4);
      dst[l * kTok] = wv == 0 ? At[v] : l > l32 ? 0.f : E[v] * rd;
    }
  }
  // dl_Q = phi_Q / D (S G + gd z + sum_l phi_K,l (G.v_l + gd)): registers = features, lane = query
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int j = 0; j < 4; ++j) P[4 * a + j] = fmaf(gd, z4[a][j], P[4 * a + j]);
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pe[3], pk[3];
    split_acc(E, hh, pe);
    patch_read(pk, patch, hh, lane);
    P = mm_all(pk, pe, P);
  }
  P *= U;
  f32x16 X[2] = {zero_acc(), zero_acc()};   // this wave's part of dQ^T
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pl[3];
    split_acc(P, hh, pl);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      u32x4 t[3];
      at_frags(t, Atp, h, m, f0 + 16 * hh, b, lane);
      X[b] = mm_all(t, pl, X[b]);
    }
  }
  lds_barrier();   // gd is there; every wave has read the parts
  float* part = reinterpret_cast<float*>(area);   // [32 queries][64]
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int a = 0; a < 4; ++a)
      *reinterpret_cast<f32x4*>(part + (l32 * 16 + ((8 * b + 2 * a + hf) ^ (l32 % 16))) * 4) =
          f32x4{X[b][4 * a], X[b][4 * a + 1], X[b][4 * a + 2], X[b][4 * a + 3]};
  // R and T of the chunk: a feature per lane row, tokens contracted
  f32x16 R[2] = {zero_acc(), zero_acc()}, T[2] = {zero_acc(), zero_acc()};
  float rdsum = 0.f;
  const size_t ob = chunk * m + f0;
  patch_write(patch, U, lane);
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pq[3];
    patch_read(pq, patch, hh, lane);
    float fd[8];
    chain_scalars(fd, scal, hh, hf);
#pragma unroll
    for (int e = 0; e < 4; ++e) {   // Rd: the features of this lane's half of the tokens, put together again
      rdsum += ((__uint_as_float(pq[0][e] << 16) + __uint_as_float(pq[1][e] << 16)) + __uint_as_float(pq[2][e] << 16)) * fd[2 * e];
      rdsum += ((__uint_as_float(pq[0][e] & 0xffff0000u) + __uint_as_float(pq[1][e] & 0xffff0000u)) +
                __uint_as_float(pq[2][e] & 0xffff0000u)) * fd[2 * e + 1];
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      u32x4 y[NP];
      col_planes<NP>(gc[hh][b], y);
      R[b] = mm_all(pq, y, R[b]);
    }
  }
  rdsum += xor32(rdsum);
  patch_write(patch, P, lane);
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pl[3];
    patch_read(pl, patch, hh, lane);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      u32x4 x[NP];
      col_planes<NP>(qc[hh][b], x);
      T[b] = mm_all(pl, x, T[b]);
    }
  }
  lds_barrier();
  if (dQ != nullptr) {
    for (int i = tid; i < kTok * 16; i += blockDim.x) {
      const int r = i / 16, c = i % 16;
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
      for (int w = 0; w < nw; ++w)
        s += *reinterpret_cast<const f32x4*>(ex + (size_t)w * CausalSmem::ex_wave + (r * 16 + (c ^ (r % 16))) * 16);
      if (r < nvalid) *reinterpret_cast<f32x4*>(dQ + (row0 + r) * kD + 4 * c) = s * kLn2;
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const size_t o = (ob + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32;
      Rpart[o] = R[b][v];
      Tpart[o] = T[b][v];
    }
  if (hf == 0) Rdpart[ob + l32] = rdsum;
}

// The key side of a chunk: a wave per 32 features, requests ahead as above (18.0 -> 17.0 us, though six registers spill; the forward
// 10.4 -> 9.5).  Where several waves share a SIMD and the states still lie in the caches the forward can lose by them: fp32, m = 256,
// the whole call, 24 heads of 1024 85.7 -> 87.8 us, 64 heads of 512 117 -> 120, but 24 heads of 3000 251 -> 243.
template <int NP>
__global__ __launch_bounds__(512, 2) void k_sp_causal_k(
    const void* __restrict__ Qg, const void* __restrict__ Kg, const void* __restrict__ Vg, const void* __restrict__ Gg,
    const us* __restrict__ Apl, const us* __restrict__ Atp, const us* __restrict__ G2p, const us* __restrict__ Rt,
    const float* __restrict__ Rd, const float* __restrict__ cpre,
    const float* __restrict__ nrm, const float* __restrict__ mu_in, const float* __restrict__ rd_in,
    const float* __restrict__ Atile, const float* __restrict__ Etile, float* __restrict__ dK, float* __restrict__ dV,
    float* __restrict__ Tpart, float* __restrict__ Rmpart, int H, int L, int m, int nc) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64, nw = blockDim.x / 64;
  const int l32 = lane % 32, hf = lane / 32;
  const size_t chunk = blockIdx.x;
  const int bh = blockIdx.x / nc, h = bh % H;
  const int t0 = (blockIdx.x % nc) * kTok, nvalid = min(kTok, L - t0);
  const size_t row0 = (size_t)bh * L + t0, row = row0 + min(l32, nvalid - 1);
  const int f0 = 32 * wv;
  float* scal = reinterpret_cast<float*>(smem);   // mu, 1/D of the tile's queries, s of its keys
  float* spart = reinterpret_cast<float*>(smem + CausalSmem::spart);
  unsigned char* ex = smem + CausalSmem::ex;
  unsigned char* patch = ex + (size_t)wv * CausalSmem::ex_wave + CausalSmem::patch;

  // what a phase needs from memory is asked for a phase or more before: a lone wave on its SIMD has nothing else to hide it behind
  const us* rt = Rt + chunk * 3 * kD * m;
  StateFrags sf;
  Raw8<NP> vr[4];
  f32x16 Fq, Fk;   // query features (lane = feature, registers = queries), key features (lane = key)
  {
    RowStage<NP> rows;
    rows.load(Qg, Kg, row0, nvalid, tid, blockDim.x);
    u32x4 af[4][3];
#pragma unroll
    for (int s = 0; s < 4; ++s) a_frags(af[s], Apl, h, m, f0, s, lane);
    float mu_t = kTailNorm, rd_t = 0.f;
    if (tid < nvalid) {
      mu_t = mu_in[row0 + tid];
      rd_t = rd_in[row0 + tid];
    }
    rows.store(ex, tid, blockDim.x);
    load_state(sf, rt, f0 / 16, lane);
    if (tid < kTok) {
      scal[tid] = mu_t;
      scal[32 + tid] = rd_t;
    }
    lds_barrier();
    Logits lq, lk;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 xq[NP], xk[NP];
      RowStage<NP>::frag(xq, ex, 0, s, lane);
      RowStage<NP>::frag(xk, ex, 1, s, lane);
      lq.add_xa(xq, af[s]);
      lk.add_ax(af[s], xk);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) vr[s].load(Vg, row * kD + 16 * s + 8 * hf);
    lds_barrier();   // the rows have been read
    Fq = lq.sum();
    Fk = lk.sum();
  }
  const float n = l32 < nvalid ? nrm[row] : kTailNorm;
  const float cf = cpre[chunk * m + f0 + l32];
  f32x16 P;   // dphi_K, then dl_K: registers = features, lane = key
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const f32x4 c4 = *reinterpret_cast<const f32x4*>(cpre + chunk * m + f0 + 8 * a + 4 * hf);
    const f32x4 r4 = *reinterpret_cast<const f32x4*>(Rd + chunk * m + f0 + 8 * a + 4 * hf);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Fk[4 * a + j] = fast_exp2(Fk[4 * a + j] - n - c4[j]);
      P[4 * a + j] = r4[j];
    }
  }
  // tiles: rows = keys, a lane's key row in chain order of the queries
  f32x4 te[2][2], ta[2][2];
  auto tile_row = [&](f32x4(&x)[2][2], const float* tile) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int q = 0; q < 2; ++q) x[hh][q] = *reinterpret_cast<const f32x4*>(tile + chunk * kTok * kTok + l32 * kTok + 16 * hh + 4 * hf + 8 * q);
  };
  tile_row(te, Etile);
  {
    unsigned char* area = ex + (size_t)wv * CausalSmem::ex_wave;
    turn_state(area, sf, lane);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 v[NP], a[3];
      vr[s].planes(v);
      turned_frag(a, area, s, lane);
      P = mm_all(a, v, P);
    }
  }
  u32x4 tf[2][2][3];
  float gc[2][8];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int b = 0; b < 2; ++b) at_frags(tf[hh][b], Atp, h, m, f0 + 16 * hh, b, lane);
  if (wv < 2) {
    tile_row(ta, Atile);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) col_values<NP>(gc[hh], Gg, row0, nvalid, hh, wv, lane);
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const f32x4 m4 = *reinterpret_cast<const f32x4*>(scal + 8 * a + 4 * hf);
#pragma unroll
    for (int j = 0; j < 4; ++j) Fq[4 * a + j] = fast_exp2(Fq[4 * a + j] + cf - m4[j]);
  }
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pq[3], pe[3];
    split_acc(Fq, hh, pq);
    split8(te[hh][0], te[hh][1], pe);
    P = mm_all(pq, pe, P);
  }
  float s_l = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    P[v] *= Fk[v];
    s_l += P[v];
  }
  s_l += xor32(s_l);
  f32x16 Xv[2] = {zero_acc(), zero_acc()}, Xk[2] = {zero_acc(), zero_acc()};   // this wave's parts of dV^T, dK^T
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    u32x4 pk[3], pl[3];
    split_acc(Fk, hh, pk);
    split_acc(P, hh, pl);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      Xv[b] = mm_all(sf[hh][b], pk, Xv[b]);
      Xk[b] = mm_all(tf[hh][b], pl, Xk[b]);
    }
    if (wv < 2) {   // the tile's part of dV: a half of the columns in each of two waves
      u32x4 pa[3], y[3];
      split8(ta[hh][0], ta[hh][1], pa);
      float fr[8];
      chain_scalars(fr, scal + 32, hh, hf);
#pragma unroll
      for (int e = 0; e < 8; ++e) gc[hh][e] *= fr[e];
      split_values(gc[hh], y);
#pragma unroll
      for (int b = 0; b < 2; ++b)
        if (b == wv) Xv[b] = mm_all(y, pa, Xv[b]);
    }
  }
  // T: the query half is in Tpart
  float kc[2][2][8];   // columns of K, for T and Rm
  {
    f32x16 T[2] = {zero_acc(), zero_acc()}, Tq[2];
    const size_t ob = chunk * m + f0;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int b = 0; b < 2; ++b) col_values<NP>(kc[hh][b], Kg, row0, nvalid, hh, b, lane);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) Tq[b][v] = Tpart[(ob + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32];
    patch_write(patch, P, lane);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 pl[3];
      patch_read(pl, patch, hh, lane);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        u32x4 x[NP];
        col_planes<NP>(kc[hh][b], x);
        T[b] = mm_all(pl, x, T[b]);
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) Tpart[(ob + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32] = Tq[b][v] + T[b][v];
  }
  Raw8<NP> kr[4];   // keys and M^T M, for the norm term
  u32x4 gm[4][3];
  if (wv < 2) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      kr[s].load(Kg, row * kD + 16 * s + 8 * hf);
      a_frags(gm[s], G2p, h, kD, 32 * wv, s, lane);
    }
  }
  if (hf == 0) spart[32 * wv + l32] = s_l;
  asm volatile("" ::: "memory");   // the patch has been read: dK takes its place
  {
    float* part = reinterpret_cast<float*>(ex + (size_t)wv * CausalSmem::ex_wave);   // dV, dK: [32 keys][64] each
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int at = (l32 * 16 + ((8 * b + 2 * a + hf) ^ (l32 % 16))) * 4;
        *reinterpret_cast<f32x4*>(part + at) = f32x4{Xv[b][4 * a], Xv[b][4 * a + 1], Xv[b][4 * a + 2], Xv[b][4 * a + 3]};
        *reinterpret_cast<f32x4*>(part + 2048 + at) = f32x4{Xk[b][4 * a], Xk[b][4 * a + 1], Xk[b][4 * a + 2], Xk[b][4 * a + 3]};
      }
  }
  lds_barrier();
  // s of every key, and the norm term s alpha^2 M^T M k (columns 32 wv + [0,32) by the first two waves)
  float s_tot = 0.f;
  for (int w = 0; w < nw; ++w) s_tot += spart[32 * w + l32];
  if (wv == 0 && hf == 0) scal[64 + l32] = s_tot;
  float* ynorm = reinterpret_cast<float*>(smem + CausalSmem::ynorm);   // [column half][32 keys][32]
  if (wv < 2) {
    f32x16 Y = zero_acc();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 x[NP];
      kr[s].planes(x);
      Y = mm_all(gm[s], x, Y);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
      *reinterpret_cast<f32x4*>(ynorm + 1024 * wv + (l32 * 8 + ((2 * a + hf) ^ (l32 % 8))) * 4) =
          f32x4{Y[4 * a] * s_tot, Y[4 * a + 1] * s_tot, Y[4 * a + 2] * s_tot, Y[4 * a + 3] * s_tot};
  }
  lds_barrier();
  for (int i = tid; i < kTok * 16; i += blockDim.x) {
    const int r = i / 16, c = i % 16;
    f32x4 sv = {0.f, 0.f, 0.f, 0.f}, sk = sv;
    for (int w = 0; w < nw; ++w) {
      const unsigned char* part = ex + (size_t)w * CausalSmem::ex_wave + (r * 16 + (c ^ (r % 16))) * 16;
      sv += *reinterpret_cast<const f32x4*>(part);
      sk += *reinterpret_cast<const f32x4*>(part + 2048 * 4);
    }
    sk = sk * kLn2 - *reinterpret_cast<const f32x4*>(ynorm + 1024 * (c / 8) + (r * 8 + ((c % 8) ^ (r % 8))) * 4);
    if (r < nvalid) {
      if (dV != nullptr) *reinterpret_cast<f32x4*>(dV + (row0 + r) * kD + 4 * c) = sv;
      if (dK != nullptr) *reinterpret_cast<f32x4*>(dK + (row0 + r) * kD + 4 * c) = sk;
    }
  }
  // Rm of the chunk: rows e = 32 (wv / 2) + ., columns 32 (wv % 2) + . (both row blocks in turn when there are two waves)
  for (int blk = wv; blk < 4; blk += nw) {
    const int e = blk / 2, b = blk % 2;
    f32x16 acc = zero_acc();
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      float x[8], y[8], fs[8];
      chain_scalars(fs, scal + 64, hh, hf);
#pragma unroll
      for (int q = 0; q < 8; ++q) {   // wave-uniform
        x[q] = (e ? kc[hh][1][q] : kc[hh][0][q]) * fs[q];
        y[q] = b ? kc[hh][1][q] : kc[hh][0][q];
      }
      u32x4 sx[3], kx[NP];
      split_values(x, sx);
      col_planes<NP>(y, kx);
      acc = mm_all(sx, kx, acc);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
      Rmpart[chunk * kD * kD + (size_t)(32 * e + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * b + l32] = acc[v];
  }
}

// ------------------------------- host side ---------------------------------
// Slices of the key pass: about one workgroup per CU (eight waves; more of the smaller ones), whole tiles, and never
// more than 4096 keys, so that the rounding of the running fp32 sums does not grow with L (the general kernels' bound).  At most
// `most` per (b,h): each is a state that is written and summed.
void sp_slices(const Problem& pb, int* P, int* slice_len, int most = 64) {
  const dark_params& p = pb.p;
  const int nfb = (p.m + 255) / 256;
  const int wgs = p.m >= 256 ? 256 : (p.m == 128 ? 512 : 1024);
  long long want = wgs / (pb.BH() * nfb > 0 ? pb.BH() * nfb : 1);
  want = want < 1 ? 1 : (want > most ? most : want);
  int sl = (int)((p.L + want - 1) / want);
  sl = (sl + kTok - 1) / kTok * kTok;
  if (sl > 4096) sl = 4096;
  *slice_len = sl;
  *P = (p.L + sl - 1) / sl;
}

struct SpBufs {
  us *Apl, *Atp, *G2p, *St, *Sf;   // Atp, G2p, Sf: backward only
  float *nrm, *Spart, *zpart, *cpart, *zt, *ct;
  int P, sl;
};

SpBufs take_bufs(const Problem& pb, Arena& ar, bool bwd) {
  const dark_params& p = pb.p;
  const size_t BH = (size_t)pb.BH();
  SpBufs b{};
  sp_slices(pb, &b.P, &b.sl);
  b.Apl = ar.take<us>((size_t)p.H * 3 * p.m * kD);
  b.nrm = ar.take<float>(BH * p.L);
  b.Spart = ar.take<float>(BH * b.P * p.m * kD);
  b.zpart = ar.take<float>(BH * b.P * p.m);
  b.cpart = ar.take<float>(BH * b.P * p.m);
  if (!bwd) b.St = ar.take<us>(BH * 3 * kD * p.m);
  b.zt = ar.take<float>(BH * p.m);
  b.ct = ar.take<float>(BH * p.m);
  if (bwd) {
    b.Atp = ar.take<us>((size_t)p.H * 3 * p.m * kD);
    b.G2p = ar.take<us>((size_t)p.H * 3 * kD * kD);
    b.Sf = ar.take<us>(BH * 3 * kD * p.m);
  }
  return b;
}

template <int NP, bool BWD>
dark_status launch_prep(const Problem& pb, const SpBufs& b, const void* K, const float* M, const float* W) {
  const dark_params& p = pb.p;
  const int nt = (p.L + kTok - 1) / kTok;
  const int tiles = p.B * nt;   // of a head
  const int tpw = std::min((int)((pb.BH() * nt + 4095) / 4096), (tiles + 3) / 4);   // one tile per wave until every SIMD has four
  const int wgs = (tiles + 4 * tpw - 1) / (4 * tpw);
  const unsigned grid = (unsigned)(p.H * (p.m / 16 + (BWD ? 4 : 0) + wgs));
  auto kern = k_sp_prep<NP, BWD>;
  DARK_TRY(allow_lds(kern, PrepSmem<NP>::total));
  DARK_LAUNCH(KID_PREP, pb.st, kern, dim3(grid), dim3(256), PrepSmem<NP>::total, M, W, b.Apl, b.Atp, b.G2p, K, b.nrm, p.H, p.L, p.m,
              p.w_shared, std::sqrt(pb.scale), p.B, wgs, tpw);
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

template <int NP>
dark_status launch_states(const Problem& pb, const SpBufs& b, const void* K, const void* V) {
  if (pb.p.m == 64) return launch_states<NP, 2>(pb, b, K, V);
  if (pb.p.m == 128) return launch_states<NP, 4>(pb, b, K, V);
  return launch_states<NP, 8>(pb, b, K, V);
}

template <int NP, int NWF, typename OutT>
dark_status launch_readout(const Problem& pb, const SpBufs& b, const void* Q, void* out) {
  const dark_params& p = pb.p;
  auto kern = k_sp_readout<NP, NWF, OutT>;
  const size_t lds = 2 * NWF * kRdSlot;
  DARK_TRY(allow_lds(kern, lds));
  const int per = (p.L + 4 * kTok - 1) / (4 * kTok);
  DARK_LAUNCH(KID_READOUT, pb.st, kern, dim3((unsigned)(pb.BH() * per)), dim3(256 * NWF), lds, Q, b.Apl, b.St, b.zt, b.ct,
              (OutT*)out, p.H, p.L, p.m, per);
  return DARK_OK;
}

// A', n' and the merged state of all keys: what the forward and the backward pass start from.
template <int NP, bool BWD>
dark_status sp_key_state(const Problem& pb, const SpBufs& b, const void* K, const void* V, const float* M, const float* W) {
  const dark_params& p = pb.p;
  DARK_TRY((launch_prep<NP, BWD>(pb, b, K, M, W)));
  DARK_TRY((launch_states<NP>(pb, b, K, V)));
  DARK_LAUNCH(KID_KV_MERGE, pb.st, k_sp_merge<BWD ? MG_S : MG_FWD>, dim3((unsigned)(pb.BH() * (p.m / 32))), dim3(256), 0,
              b.Spart, b.zpart, b.cpart, b.St, b.Sf, b.zt, b.ct, p.m, b.P);
  return DARK_OK;
}

// Where one workgroup takes all keys of 32 features (k_sp_keys): one round of workgroups over the CUs, and few enough tiles a wave
// that the norms formed again by every block cost less than the launches.  The line lies where one head, whose launches are the
// shortest, gains nothing any more (+0.6 us at worst, m = 128); more heads would gain beyond it.  us, three kernels / this one, one
// head: m = 64 18.7 / 14.9 (L = 33), 19.1 / 17.8 (256), 19.7 / 19.8 (288), 19.9 / 22.8 (416); m = 128 21.4 / 20.5 (256),
// 22.2 / 22.8 (320), 22.7 / 25.3 (416); m = 256 27.7 / 25.5 (256), 28.9 / 28.1 (384), 28.9 / 30.2 (416).  24 (b,h): m = 64
// 22.1 / 20.7 (288), 25.1 / 24.4 (512); m = 128 27.3 / 24.0 (320), 29.6 / 27.3 (512); m = 256 36.8 / 30.9 (384), 36.0 / 33.8 (512),
// 43.6 / 46.4 (1024).  Two rounds (64 (b,h), m = 256): 39 / 42 (256).
bool keys_in_one(const Problem& pb) {
  const int m = pb.p.m;
  return pb.BH() * (m / 32) <= 256 && pb.p.L <= 256 + (m < 256 ? m : 256) / 2;
}

template <int NP>
dark_status sp_forward(const Problem& pb, const SpBufs& b, const void* Q, const void* K, const void* V, const float* M,
                       const float* W, void* out) {
  const dark_params& p = pb.p;
  if (keys_in_one(pb)) {
    auto kern = k_sp_keys<NP>;
    DARK_TRY(allow_lds(kern, KeySmem<NP>::total));
    DARK_LAUNCH(KID_KV_REDUCE, pb.st, kern, dim3((unsigned)(pb.BH() * (p.m / 32))), dim3(64 * kKeyWaves), KeySmem<NP>::total, K, V, M, W,
                b.Apl, b.St, b.zt, b.ct, p.H, p.L, p.m, p.w_shared, std::sqrt(pb.scale));
  } else {
    DARK_TRY((sp_key_state<NP, false>(pb, b, K, V, M, W)));
  }
  // two waves per 32 queries while that is what it takes to give every SIMD two waves
  const bool pair = p.m > 64 && pb.BH() * ((p.L + kTok - 1) / kTok) <= 1536;
  if (p.out_dtype == DARK_BF16) {
    if (pair) return launch_readout<NP, 2, us>(pb, b, Q, out);
    return launch_readout<NP, 1, us>(pb, b, Q, out);
  }
  if (pair) return launch_readout<NP, 2, float>(pb, b, Q, out);
  return launch_readout<NP, 1, float>(pb, b, Q, out);
}

struct SpGrads {
  const void* dOut;
  float *dQ, *dK, *dV, *dM, *dW;
};
struct SpBwdBufs {   // mu, rd, gd: where the query side goes in two passes
  float *mu, *rd, *gd, *s, *Rpart, *Rdpart, *Tpart, *Rmpart, *Rd, *Tsum, *Rmsum;
  us *Rt, *Rf;
};

bool query_side_fused(const dark_params& p) { return p.io_dtype == DARK_BF16 && p.m == 256; }

template <int NP, int NW>
dark_status launch_bwd_tokens(const Problem& pb, const SpBufs& b, const SpBwdBufs& w, const void* X, const void* Y,
                              const SpGrads& g, bool keys) {
  const dark_params& p = pb.p;
  const int per = (p.L + NW * kTok - 1) / (NW * kTok);
  const dim3 grid((unsigned)(pb.BH() * per));
  if (keys) {
    auto kern = k_sp_bwd_k<NP, NW>;
    const size_t lds = 2 * kKBuf;
    DARK_TRY(allow_lds(kern, lds));
    DARK_LAUNCH(KID_BWD_REV, pb.st, kern, grid, dim3(64 * NW), lds, X, Y, b.Apl, b.Atp, b.G2p, w.Rt, w.Rf, w.Rd, b.ct, b.nrm,
                g.dK, g.dV, w.s, p.H, p.L, p.m, per);
  } else {
    auto kern = k_sp_bwd_q<NP, NW>;
    const size_t lds = 2 * kQBuf;
    DARK_TRY(allow_lds(kern, lds));
    DARK_LAUNCH(KID_BWD_FWD, pb.st, kern, grid, dim3(64 * NW), lds, X, Y, b.Apl, b.Atp, b.Sf, b.zt, b.ct, g.dQ, w.mu,
                w.rd, w.gd, p.H, p.L, p.m, per);
  }
  return DARK_OK;
}

template <int NP, int NW, bool KEYS>
dark_status launch_bwd_fs(const Problem& pb, const SpBufs& b, const SpBwdBufs& w, const void* X, const void* Y) {
  const dark_params& p = pb.p;
  const int nfb = (p.m + 255) / 256;
  auto kern = k_sp_bwd_fs<NP, NW, KEYS>;
  DARK_TRY(allow_lds(kern, FsSmem<NP, KEYS>::total));
  DARK_LAUNCH(KEYS ? KID_BWD_REV : KID_BWD_FWD, pb.st, kern, dim3((unsigned)(pb.BH() * b.P * nfb)), dim3(64 * NW),
              (FsSmem<NP, KEYS>::total), X, Y, b.Apl, KEYS ? w.Rf : b.Sf, KEYS ? w.Rd : b.zt, b.ct, KEYS ? b.nrm : w.mu,
              KEYS ? w.s : w.rd, w.gd, w.Rpart, w.Rdpart, w.Tpart, w.Rmpart, p.H, p.L, p.m, b.P, b.sl, nfb);
  return DARK_OK;
}
template <int NP, bool KEYS>
dark_status launch_bwd_fs(const Problem& pb, const SpBufs& b, const SpBwdBufs& w, const void* X, const void* Y) {
  if (pb.p.m == 64) return launch_bwd_fs<NP, 2, KEYS>(pb, b, w, X, Y);
  if (pb.p.m == 128) return launch_bwd_fs<NP, 4, KEYS>(pb, b, w, X, Y);
  return launch_bwd_fs<NP, 8, KEYS>(pb, b, w, X, Y);
}

// dM and dW from the P pieces per (b,h) of T and Rm.
template <int NP>
dark_status sp_backward(const Problem& pb, const SpBufs& b, const SpBwdBufs& w, const void* Q, const void* K,
                        const void* V, const float* M, const float* W, const SpGrads& g) {
  const dark_params& p = pb.p;
  DARK_TRY((sp_key_state<NP, true>(pb, b, K, V, M, W)));
  // eight waves share an operand group unless the smaller workgroups still find a CU each
  const bool four = pb.BH() * ((p.L + 4 * kTok - 1) / (4 * kTok)) <= 256;
  const bool geometry = g.dM != nullptr || g.dW != nullptr, past = geometry || g.dK != nullptr || g.dV != nullptr;
  if (query_side_fused(p)) {
    auto kern = past ? k_sp_bwd_qf<true> : k_sp_bwd_qf<false>;
    int P = b.P, sl = b.sl;
    if (!past) sp_slices(pb, &P, &sl, 256);
    DARK_TRY(allow_lds(kern, QfSmem::total));
    DARK_LAUNCH(KID_BWD_FWD, pb.st, kern, dim3((unsigned)(pb.BH() * P)), dim3(512), QfSmem::total, (const us*)Q,
                (const us*)g.dOut, b.Apl, b.Atp, b.Sf, b.zt, b.ct, g.dQ, w.Rpart, w.Rdpart, w.Tpart, p.H, p.L, P, sl);
  } else {
    DARK_TRY((four ? launch_bwd_tokens<NP, 4>(pb, b, w, Q, g.dOut, g, false)
                   : launch_bwd_tokens<NP, 8>(pb, b, w, Q, g.dOut, g, false)));
    if (past) DARK_TRY((launch_bwd_fs<NP, false>(pb, b, w, Q, g.dOut)));
  }
  if (!past) return DARK_OK;
  DARK_LAUNCH(KID_BWD_SUFFIX, pb.st, k_sp_merge<MG_R>, dim3((unsigned)(pb.BH() * (p.m / 32))), dim3(256), 0, w.Rpart, w.Rdpart,
              (const float*)nullptr, w.Rt, w.Rf, w.Rd, (float*)nullptr, p.m, b.P);
  DARK_TRY((four ? launch_bwd_tokens<NP, 4>(pb, b, w, K, V, g, true) : launch_bwd_tokens<NP, 8>(pb, b, w, K, V, g, true)));
  if (!geometry) return DARK_OK;
  DARK_TRY((launch_bwd_fs<NP, true>(pb, b, w, K, V)));
  return launch_geometry(pb, w.Tpart, w.Rmpart, b.P, w.Tsum, w.Rmsum, M, W, g.dM, g.dW);
}

// ---- causal ----
struct ScBufs {
  us *Apl, *Atp, *G2p, *St;
  float *nrm, *Spart, *zpart, *cpart, *zpre, *cpre;
  int nc;
};

ScBufs take_causal(const Problem& pb, Arena& ar, bool bwd) {
  const dark_params& p = pb.p;
  ScBufs b{};
  b.nc = (p.L + kTok - 1) / kTok;
  const size_t n = (size_t)pb.BH() * b.nc * p.m;
  b.Apl = ar.take<us>((size_t)p.H * 3 * p.m * kD);
  b.nrm = ar.take<float>((size_t)pb.BH() * p.L);
  b.Spart = ar.take<float>(n * kD);
  b.zpart = ar.take<float>(n);
  b.cpart = ar.take<float>(n);
  b.St = ar.take<us>(n * 3 * kD);
  b.zpre = ar.take<float>(n);
  b.cpre = ar.take<float>(n);
  if (bwd) {
    b.Atp = ar.take<us>((size_t)p.H * 3 * p.m * kD);
    b.G2p = ar.take<us>((size_t)p.H * 3 * kD * kD);
  }
  return b;
}

template <int NP, bool BWD>
dark_status sc_prefix(const Problem& pb, const ScBufs& b, const void* K, const void* V, const float* M, const float* W) {
  SpBufs s{};
  s.Apl = b.Apl; s.Atp = b.Atp; s.G2p = b.G2p; s.nrm = b.nrm;
  s.Spart = b.Spart; s.zpart = b.zpart; s.cpart = b.cpart;
  s.P = b.nc;
  s.sl = kTok;
  DARK_TRY((launch_prep<NP, BWD>(pb, s, K, M, W)));
  DARK_TRY((launch_states<NP>(pb, s, K, V)));
  DARK_LAUNCH(KID_CAUSAL_PREFIX, pb.st, k_sp_scan<false>, dim3((unsigned)(pb.BH() * (pb.p.m / 8))), dim3(512), 0, b.Spart,
              b.zpart, b.cpart, b.St, b.zpre, b.cpre, pb.p.m, b.nc);
  return DARK_OK;
}

template <int NP, typename OutT>
dark_status sc_forward(const Problem& pb, const ScBufs& b, const void* Q, const void* K, const void* V, const float* M,
                       const float* W, void* out) {
  const dark_params& p = pb.p;
  DARK_TRY((sc_prefix<NP, false>(pb, b, K, V, M, W)));
  auto kern = k_sp_causal<NP, OutT>;
  const size_t lds = CausalSmem::total(p.m / 32);
  DARK_TRY(allow_lds(kern, lds));
  DARK_LAUNCH(KID_CAUSAL_SCAN, pb.st, kern, dim3((unsigned)(pb.BH() * b.nc)), dim3(2 * p.m), lds, Q, K, V, b.Apl, b.St, b.zpre,
              b.cpre, b.nrm, (OutT*)out, p.H, p.L, p.m, b.nc);
  return DARK_OK;
}

struct ScBwdBufs {
  float *mu, *rd, *At, *Et, *Tpart, *Rmpart, *Tsum, *Rmsum;
};

template <int NP>
dark_status sc_backward(const Problem& pb, const ScBufs& b, const ScBwdBufs& w, const void* Q, const void* K,
                        const void* V, const float* M, const float* W, const SpGrads& g) {
  const dark_params& p = pb.p;
  DARK_TRY((sc_prefix<NP, true>(pb, b, K, V, M, W)));
  const size_t lds = CausalSmem::total(p.m / 32);
  const dim3 grid((unsigned)(pb.BH() * b.nc)), block(2 * p.m);
  float *Rpart = b.Spart, *Rdpart = b.zpart;   // the chunk states have been summed up by then
  {
    auto kern = k_sp_causal_q<NP>;
    DARK_TRY(allow_lds(kern, lds));
    DARK_LAUNCH(KID_BWD_FWD, pb.st, kern, grid, block, lds, Q, K, V, g.dOut, b.Apl, b.Atp, b.St, b.zpre, b.cpre, b.nrm, g.dQ,
                w.mu, w.rd, w.At, w.Et, Rpart, Rdpart, w.Tpart, p.H, p.L, p.m, b.nc);
  }
  const bool geometry = g.dM != nullptr || g.dW != nullptr;
  if (!geometry && g.dK == nullptr && g.dV == nullptr) return DARK_OK;
  // the suffix states take the place of the prefix states
  DARK_LAUNCH(KID_BWD_SUFFIX, pb.st, k_sp_scan<true>, dim3((unsigned)(pb.BH() * (p.m / 8))), dim3(512), 0, Rpart, Rdpart,
              b.cpre, b.St, b.zpre, (float*)nullptr, p.m, b.nc);
  {
    auto kern = k_sp_causal_k<NP>;
    DARK_TRY(allow_lds(kern, lds));
    DARK_LAUNCH(KID_BWD_REV, pb.st, kern, grid, block, lds, Q, K, V, g.dOut, b.Apl, b.Atp, b.G2p, b.St, b.zpre, b.cpre,
                b.nrm, w.mu, w.rd, w.At, w.Et, g.dK, g.dV, w.Tpart, w.Rmpart, p.H, p.L, p.m, b.nc);
  }
  return geometry ? launch_geometry(pb, w.Tpart, w.Rmpart, b.nc, w.Tsum, w.Rmsum, M, W, g.dM, g.dW) : DARK_OK;
}

}  // namespace

dark_status launch_geometry(const Problem& pb, const float* Tpart, const float* Rmpart, int P, float* Tsum, float* Rmsum,
                            const float* M, const float* W, float* dM, float* dW) {
  const dark_params& p = pb.p;
  const long long n = (long long)p.H * (p.m + kD) * kD / 4;
  DARK_LAUNCH(KID_BWD_DM, pb.st, k_sp_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, Tpart, Rmpart, Tsum, Rmsum, p.B,
              p.H, p.m, P);
  if (dM != nullptr)
    DARK_LAUNCH(KID_BWD_DM, pb.st, k_sp_dm, dim3((unsigned)(8 * p.H)), dim3(256), 0, Tsum, Rmsum, M, W, dM, p.m, p.w_shared,
                std::sqrt(pb.scale));
  if (dW != nullptr) DARK_TRY(launch_dw(pb, Tsum, 1, M, dW));
  return DARK_OK;
}

bool split_supported(const Problem& pb) {
  const dark_params& p = pb.p;
  return p.d == kD && p.r == kD && p.dv == kD && p.m % 64 == 0 && pb.BH() * (long long)(p.L + kTok) < (1LL << 31) &&
         pb.BH() * (long long)p.m < (1LL << 24);
}

dark_status split_attn_fwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V, const float* M,
                           const float* W, void* out) {
  const SpBufs b = take_bufs(pb, ar, false);
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  return pb.p.io_dtype == DARK_BF16 ? sp_forward<1>(pb, b, Q, K, V, M, W, out) : sp_forward<3>(pb, b, Q, K, V, M, W, out);
}

dark_status split_attn_bwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V, const float* M,
                           const float* W, const void* dOut, float* dQ, float* dK, float* dV, float* dM, float* dW) {
  const dark_params& p = pb.p;
  const SpBufs b = take_bufs(pb, ar, true);
  const size_t BH = (size_t)pb.BH(), rows = BH * p.L;
  SpBwdBufs w{};
  if (!query_side_fused(p)) {
    w.mu = ar.take<float>(rows);
    w.rd = ar.take<float>(rows);
    w.gd = ar.take<float>(rows);
  }
  w.s = ar.take<float>(rows);
  w.Rpart = b.Spart;   // the slice states of the keys are merged by then
  w.Rdpart = b.zpart;
  w.Tpart = ar.take<float>(BH * b.P * p.m * kD);
  w.Rmpart = ar.take<float>(BH * b.P * kD * kD);
  w.Rd = ar.take<float>(BH * p.m);
  w.Rt = ar.take<us>(BH * 3 * kD * p.m);
  w.Rf = ar.take<us>(BH * 3 * kD * p.m);
  w.Tsum = ar.take<float>((size_t)p.H * p.m * kD);
  w.Rmsum = ar.take<float>((size_t)p.H * kD * kD);
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  const SpGrads g = {dOut, dQ, dK, dV, dM, dW};
  return p.io_dtype == DARK_BF16 ? sp_backward<1>(pb, b, w, Q, K, V, M, W, g) : sp_backward<3>(pb, b, w, Q, K, V, M, W, g);
}

// Where the per-chunk kernels are the better ones.  Their states are read and written per 32 positions (the general
// kernels': per 128) and the scan walks them 32 at a time, eight features a workgroup, so a single head of great length
// and very large problems bound them.  Measured against the general kernels, fp32: forward 89 -> 32 us (one head,
// L = 300), 313 -> 204 us (24 heads, L = 2048, m = 256), 404 -> 326 us (one head, L = 65,536, m = 128): taken up to that
// length.  Backward 237 -> 63, 767 -> 610, and 417 -> 328 us (one head, L = 16,384, m = 128), but 1289 -> 1284 us at
// 24 heads, L = 4096, m = 256 and 995 -> 1270 us at one head, L = 65,536: taken up to those sizes.
bool split_causal_supported(const Problem& pb, bool bwd) {
  // a caller's shorter chunks stand for a smaller window of key logits under one shift
  if (!split_supported(pb) || pb.p.m > 256 || pb.chunk < kTok) return false;
  const int m = pb.p.m, L = pb.p.L;
  const long long nc = (L + kTok - 1) / kTok, feats = pb.BH() * (long long)m;
  // Many heads of short sequences: up to p->chunk positions the general kernels have one state per (b,h) and no scan, these one
  // per 32 positions whether it is scanned or not.  While those states stay in the caches the fewer launches win, beyond that
  // the general kernels do.  Forward, us, general / these: fp32 m = 256 at 1024 (b,h) 365 / 446 (L = 8), 527 / 612 (64),
  // 788 / 904 (128), 1199 / 1009 (160), at 256 (b,h) 158 / 124, 210 / 153, 259 / 211; m = 192 at 2048 (b,h) 524 / 687 (8),
  // 1292 / 1430 (128); m = 128 at 4096 (b,h) 724 / 918 (8), 1207 / 1232 (64), 1608 / 1486 (96); m = 64 always these; bf16
  // inputs m = 256 at 2048 (b,h) 650 / 909 (8), 1571 / 1660 (128), m = 192 1127 / 1144 (96), m = 128 at 4096 (b,h) 736 / 895
  // (8), 925 / 919 (32).  Backward, fp32, m = 256: 1024 (b,h) 1212 / 1295 (L = 48), 1003 / 876 (32); 2048 (b,h) 1610 / 1717 (8).
  if (L <= pb.chunk) {
    const int few = pb.p.io_dtype == DARK_F32 ? 3 * m / 2 - 120 : m == 128 ? 48 : m - 100;
    if (!bwd && feats > (m >= 192 ? 120 : 176) * 1024 && L <= few) return false;
    if (bwd && m >= 192 && feats * nc > 500000) return false;
  }
  return bwd ? nc <= 512 && feats * nc <= 3072LL * 256 : nc <= 2048;
}

// Bidirectional backward: merging and splitting the states of every (b,h) costs the same however few positions there are, so
// very short sequences of many heads are the general kernels'.  us, general / these: fp32 m = 256 at 2048 (b,h) 1221 / 1345
// (L = 1), 1262 / 1363 (8), 1351 / 1379 (16), 1469 / 1376 (32), at 512 (b,h) 377 / 349 (1); m = 1024 at 1024 (b,h) 2200 / 2530
// (1), 2387 / 2568 (16), 2559 / 2577 (32); m = 128 at 4096 (b,h) 1327 / 1423 (1), 1390 / 1446 (8), 1505 / 1457 (16); m = 64 at
// 4096 (b,h) 895 / 820 (1); bf16 inputs m = 1024 at 2048 (b,h) 4273 / 4459 (1), 4445 / 4594 (8), 4663 / 4590 (16), m = 512 at
// 1024 (b,h) 1170 / 1165 (1).
bool split_bwd_supported(const Problem& pb) {
  if (!split_supported(pb)) return false;
  const long long feats = pb.BH() * (long long)pb.p.m;
  if (pb.p.io_dtype == DARK_F32) {
    if (pb.p.m < 192) return pb.p.L > 8 || pb.p.m < 128 || feats <= 256 * 1024;
    return pb.p.L > 20 || feats <= (pb.p.m > 256 ? 150 : 176) * 1024;
  }
  return pb.p.L > 8 || pb.p.m < 512 || feats <= 900 * 1024;
}

// The chunk states take 640 m bytes per 32 positions, a third more than the general kernels' matrices at m = 256 (21 GB
// instead of 15.7 at 64 x 65,536).  Nothing passes between (b,h): a large problem goes through in groups of equal size, whole batch
// entries or some heads of one, whose states use the same scratch.  The results do not depend on the grouping.  The line lies
// where a group still fills the chip: 8 heads of 65,536 positions, m = 128 (1.3 GB), in one group 1.12 ms, in two 1.40, in
// eight 2.65 (general kernels 1.89); 96 heads of 4096, m = 256 (2.0 GB), 1.62 ms in one, 1.63 in two.
constexpr size_t kGroupBytes = (size_t)2 << 30;

dark_status split_attn_causal_fwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V,
                                  const float* M, const float* W, void* out) {
  const dark_params& p = pb.p;
  const size_t one = (size_t)((p.L + kTok - 1) / kTok) * p.m * 640;
  const long long fit = one < kGroupBytes ? (long long)(kGroupBytes / one) : 1;
  auto share = [](long long n, long long most) { return most >= n ? n : (n + (n + most - 1) / most - 1) / ((n + most - 1) / most); };
  const int nb = fit < p.H ? 1 : (int)share(p.B, fit / p.H), nh = (int)share(p.H, fit);
  Problem part = pb;
  part.p.B = nb;
  part.p.H = nh;
  const ScBufs b = take_causal(part, ar, false);
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  const bool in16 = p.io_dtype == DARK_BF16, out16 = p.out_dtype == DARK_BF16;
  for (int b0 = 0; b0 < p.B; b0 += nb)
    for (int h0 = 0; h0 < p.H; h0 += nh) {
      part.p.B = p.B - b0 < nb ? p.B - b0 : nb;
      part.p.H = p.H - h0 < nh ? p.H - h0 : nh;
      const size_t at = ((size_t)b0 * p.H + h0) * p.L * kD;
      auto in = [&](const void* x) { return static_cast<const void*>(static_cast<const char*>(x) + at * (in16 ? 2 : 4)); };
      void* o = static_cast<char*>(out) + at * (out16 ? 2 : 4);
      const float *Mp = M + (size_t)h0 * kD * kD, *Wp = W + (p.w_shared ? 0 : (size_t)h0 * p.m * kD);
      if (in16)
        DARK_TRY((out16 ? sc_forward<1, us>(part, b, in(Q), in(K), in(V), Mp, Wp, o)
                        : sc_forward<1, float>(part, b, in(Q), in(K), in(V), Mp, Wp, o)));
      else
        DARK_TRY((out16 ? sc_forward<3, us>(part, b, in(Q), in(K), in(V), Mp, Wp, o)
                        : sc_forward<3, float>(part, b, in(Q), in(K), in(V), Mp, Wp, o)));
    }
  return DARK_OK;
}

dark_status split_attn_causal_bwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V,
                                  const float* M, const float* W, const void* dOut, float* dQ, float* dK, float* dV,
                                  float* dM, float* dW) {
  const dark_params& p = pb.p;
  const ScBufs b = take_causal(pb, ar, true);
  const size_t rows = (size_t)pb.BH() * p.L, chunks = (size_t)pb.BH() * b.nc;
  ScBwdBufs w{};
  w.mu = ar.take<float>(rows);
  w.rd = ar.take<float>(rows);
  w.At = ar.take<float>(chunks * kTok * kTok);
  w.Et = ar.take<float>(chunks * kTok * kTok);
  w.Tpart = ar.take<float>(chunks * p.m * kD);
  w.Rmpart = ar.take<float>(chunks * kD * kD);
  w.Tsum = ar.take<float>((size_t)p.H * p.m * kD);
  w.Rmsum = ar.take<float>((size_t)p.H * kD * kD);
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow) return DARK_EWORKSPACE;
  const SpGrads g = {dOut, dQ, dK, dV, dM, dW};
  return p.io_dtype == DARK_BF16 ? sc_backward<1>(pb, b, w, Q, K, V, M, W, g) : sc_backward<3>(pb, b, w, Q, K, V, M, W, g);
}

}  // namespace dark
