// Fused MFMA backward of the causal DARK attention (gfx950): bf16 inputs, fp32 accumulation, fp32 gradients.
// d = r = dv = 64, m = 256.  No [rows, m] matrix is ever written to memory: features, their gradients and
// the 32 x 32 tiles of kernel values live in LDS and registers of the workgroup that walks a slice.
//
// Notation (per (b,h); the paper makes M learnable, Section 4, and fixes the feature map in Section 4.1;
// the gradients are the chain rule through that definition and the causal prefix form of Section 2's
// factorisation).  With a_il = phi(q_i).phi(k_l) for l <= i, D_i = sum_l a_il, out_i = sum_l a_il v_l / D_i
// and G = dOut:
//   da_il = (G_i.v_l + gd_i) / D_i,  gd_i = -G_i.out_i
//   phihat_Q,i = phi_Q,i / D_i                      (so phihat_Q,i . phi_K,l = a_il / D_i)
//   dlogit_Q,ij = phihat_Q,ij [ (S_<=i G_i)_j + gd_i z_<=i,j ],   S_<=i = sum_{l<=i} phi_K,l v_l^T, z likewise
//   dlogit_K,lj = phi_K,lj   [ (Rn_>=l v_l)_j + Rd_>=l,j ],       Rn_>=l = sum_{i>=l} phihat_Q,i G_i^T,
//                                                                 Rd_>=l = sum_{i>=l} phihat_Q,i gd_i
//   dV_l = Rn_>=l^T phi_K,l
//   dQ_i = alpha A^T dlogit_Q,i;   dK_l = alpha A^T dlogit_K,l - s_l alpha^2 M^T M k_l,  s_l = sum_j dlogit_K,lj
//   dM   = alpha W^T T - alpha^2 M Rm,  T = sum_tokens dlogit x^T (queries and keys),  Rm = sum_l s_l k_l k_l^T
// (the derivative through a query's norm term vanishes identically: scaling all features of a query leaves
// out_i unchanged).  Sums over l <= i split into the keys before the tile (running state, forward order) and
// the keys of the tile (masked 32 x 32 blocks); sums over i >= l likewise in reverse order.
//
// Kernels, after the key norms, the slice states and their exclusive prefix of the causal forward path:
//   k_bwd_fwd     per (b,h, slice), tiles in forward order: D_i, out_i, dQ, the query half of T, the slice's
//                 contribution to Rn, Rd; leaves lambda_i = log2 of the denominator (with the row shift) and
//                 gd_i per token for the reverse pass
//   k_bwd_suffix  exclusive suffix sums of the slices' Rn, Rd contributions
//   k_bwd_rev     per (b,h, slice), tiles in reverse order: dV, dK, the key half of T, Rm
//   then the sums over slices and batch in fixed order and dM per head (launch_geometry)
// Everything is in the log2 domain with the fp16 operands A' = alpha log2e W M and M' of the forward path.
// Key shifts: one scalar per slice, the forward path's running shift c*_p (the largest shift of slices 0..p),
// under which the slice's prefix state is stored and its keys are featurised in both tile kernels; the
// suffix sums bring the later slices' contributions down to it.  So the key logits may rise or fall along a
// sequence without limit; what has to fit the fp32 exponent range (about 2^100 between the smallest useful
// and the largest feature) is their spread inside one slice.
#include <cmath>

#include "fused_common.h"

namespace dark {
using namespace fz;
namespace {

constexpr int kT = 32;        // tokens per tile
constexpr int kF = 256;       // features
constexpr int kD = 64;        // d = r = dv
constexpr int kNW = 8;        // waves of a workgroup
constexpr int kNT = 64 * kNW;
constexpr int LDE = 68;       // fp32 pitch of the partial dV tiles
constexpr float kBigShift = 3.0e4f;  // a shift that sends exp2 to zero

typedef unsigned short us;

__device__ __forceinline__ f32x16 mm_bf16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<bf16x8*>(&a), *reinterpret_cast<bf16x8*>(&b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mm_f16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<half8*>(&a), *reinterpret_cast<half8*>(&b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mm16_f16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<half8*>(&a), *reinterpret_cast<half8*>(&b), c, 0, 0, 0);
}
// Tiles in LDS, rows of 64, 256 or 32 elements without padding, their 16-byte chunks permuted within the row: element
// (row, col) sits at index<COLS>(row, col).  A read of one chunk from each of 16 consecutive rows and a transposing read of 64
// bytes from each of four rows (aligned to four) both cover the banks once.  (With rows of 72 and 264 elements, which
// serve the former, the transposing reads met two to four deep: they were what bound both kernels.  The counters still show a
// quarter of the LDS cycles as conflicts; these reads having none, they are those of the stores and exchanges.)
template <int COLS>
__device__ __forceinline__ int index(int row, int col) {
  static_assert(COLS == 32 || COLS == 64 || COLS == 256, "row lengths of the tiles");
  const int q = (row >> 2) & 3;
  const int swz = COLS == 32 ? q : COLS == 64 ? (2 * (row & 2)) ^ q : (4 * (row & 3)) | q;
  return row * COLS + 8 * ((col / 8) ^ swz) + col % 8;
}
// Operand fragments of a 32x32x16 MFMA.  From a tile stored [row][k] with k contiguous lane (l32, hf) takes the eight elements
// k0 + 8 hf + [0,8) of row r0 + l32 (the A operand: row = output row, and the B operand: row = output column, alike); from a
// tile stored [k][n] with n contiguous two transposing reads: within a group of 16 lanes, lane i points at row i / 4, columns
// 4 (i % 4) .. + 3 of a 4 x 16 patch and lane l receives column l of the four rows.  CHAIN: in the order in which a packed
// accumulator holds its rows (slots 0..3: rows 4 hf + [0,4), slots 4..7: those + 8), for the operand that meets one.
// The lane's part of the byte offsets is kept in registers (Lanes); what is added to it is known to the compiler and goes
// into the instruction.  (Left to itself it keeps some ninety sums of both across the loop, and spills.)
__device__ __forceinline__ u32x4 ld128(const unsigned char* smem, unsigned off) {
  return *reinterpret_cast<const u32x4*>(smem + off);
}
__device__ __forceinline__ u32x4 ld_tr(const unsigned char* smem, const unsigned (&off)[2], unsigned add) {
  const u32x2 lo = lds_read_tr16(reinterpret_cast<const us*>(smem + (off[0] + add)));
  const u32x2 hi = lds_read_tr16(reinterpret_cast<const us*>(smem + (off[1] + add)));
  return u32x4{lo[0], lo[1], hi[0], hi[1]};
}
template <int COLS, bool CHAIN>
__device__ __forceinline__ void tr_offsets(unsigned (&off)[2], unsigned base, int n0, int lane) {
  const int l16 = lane % 16, grp = lane / 16;
  const int row = (CHAIN ? 4 : 8) * (grp / 2) + l16 / 4, col = n0 + 16 * (grp % 2) + 4 * (l16 % 4);
  off[0] = base + 2 * index<COLS>(row, col);
  off[1] = base + 2 * index<COLS>(row + (CHAIN ? 8 : 4), col);
}
__device__ __forceinline__ unsigned pack_f16(float a, float b) {
  fp16x2 h;
  h[0] = (__fp16)a;
  h[1] = (__fp16)b;
  return *reinterpret_cast<unsigned*>(&h);
}
__device__ __forceinline__ float bf_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(unsigned w) { return __uint_as_float(w & 0xffff0000u); }

// Byte offsets in LDS: what both tile kernels have, then the forward-order (F) and the reverse-order kernel's (R) own.
constexpr size_t kTileBytes = (size_t)kT * kD * 2;
constexpr size_t kBufBytes = 4 * kTileBytes;   // tiles of Q and K (fp16), V and dOut (bf16; zero past the end)
struct BwdSmem {
  static constexpr size_t al = 0;                              // A' fp16 [256][64]
  static constexpr size_t x = al + (size_t)kF * kD * 2;        // two tile buffers
  static constexpr size_t ph = x + 2 * kBufBytes;              // features bf16 [32][256] on their way to the transposing reads
  // F: logit gradients fp16 [32][256] (R: they replace phihat_Q); copy of the states, S^T bf16 [64][256]
  static constexpr size_t dl = ph + (size_t)kT * kF * 2, st = dl + (size_t)kT * kF * 2;
  static constexpr size_t f_vec = st + (size_t)kD * kF * 2;    // z fp32 [256]
  static constexpr size_t f_tok = f_vec + (size_t)kF * 4;      // norms of the keys of the two tiles [2][32]
  static constexpr size_t f_part = f_tok + (size_t)2 * kT * 4; // partial results of the waves [3][32][8]
  static constexpr size_t f_gd = f_part + (size_t)kNW * 3 * kT * 4;  // gd, a copy per wave [8][32]
  static constexpr size_t fwd_total = f_gd + (size_t)kNW * kT * 4;
  static constexpr size_t r_vec = dl;                          // Rd fp32 [256]
  static constexpr size_t r_tok = r_vec + (size_t)kF * 4;      // per-token inputs of the two tiles: [2][norm | lambda | gd][32]
  static constexpr size_t r_part = r_tok + (size_t)2 * 3 * kT * 4;   // partial sums of the waves [32][8]
  static constexpr size_t r_sl = r_part + (size_t)kNW * kT * 4;      // s, a copy per wave [8][32]
  // R: a region per wave, first for the copy of its state, Rn^T bf16 [64][32], then for its part of dV, fp32 [32][LDE];
  // at the start M' fp16 [64][64]
  static constexpr size_t r_g2 = r_sl + (size_t)kNW * kT * 4;         // M'^T M' fp16 [64][64]
  static constexpr size_t r_ex = r_g2 + (size_t)kD * kD * 2;
  static constexpr size_t rev_total = r_ex + (size_t)kNW * kT * LDE * 4;
};
static_assert(BwdSmem::fwd_total <= 160 * 1024 && BwdSmem::rev_total <= 160 * 1024, "backward tiles must fit the LDS of one CU");
static_assert((size_t)kD * 32 * 2 <= (size_t)kT * LDE * 4, "a wave's state copy must fit its region");

// Steps along a row are an exclusive or, steps over 16 or more rows a sum.
struct Lanes {
  unsigned dir;      // tile of 64 columns, row l32; k-step s: ^ 32 s
  unsigned trc[2];   // ... contraction over the rows, chain order; columns 32 ..: ^ 64, k-step s: + 16 rows
  unsigned ft[2];    // features of this wave in a [token][256] tile, contraction over tokens, chain order
  unsigned put;      // ... where the accumulator rows 8 a + 4 hf + [0,4) of token l32 go: ^ 16 a
  unsigned back[2], row;   // back_project: A' (k-step s: + 32 rows); logit gradients of its token (k-step s < 4: ^ 64 s)
  __device__ __forceinline__ void init(int wv, int lane) {
    const int l32 = lane % 32, hf = lane / 32, l16 = lane % 16, kg = lane / 16;
    dir = 2 * index<kD>(l32, 8 * hf);
    put = BwdSmem::ph + 2 * index<kF>(l32, 32 * wv + 4 * hf);
    row = 2 * index<kF>(16 * (wv / 4) + l16, 8 * kg);
    tr_offsets<kD, true>(trc, 0, 0, lane);
    tr_offsets<kF, true>(ft, BwdSmem::ph, 32 * wv, lane);
#pragma unroll
    for (int u = 0; u < 2; ++u) back[u] = 2 * index<kD>(8 * kg + 4 * u + l16 / 4, 16 * (wv % 4) + 4 * (l16 % 4));
  }
  __device__ __forceinline__ void renew() {   // keeps the compiler from carrying derived offsets from tile to tile
    asm volatile("" : "+v"(dir), "+v"(put), "+v"(row), "+v"(trc[0]), "+v"(trc[1]), "+v"(ft[0]), "+v"(ft[1]), "+v"(back[0]), "+v"(back[1]));
  }
};
constexpr unsigned kRow64 = kD * 2, kRow256 = kF * 2;   // bytes per tile row
constexpr unsigned kXq = BwdSmem::x, kXk = kXq + kTileBytes, kVt = kXk + kTileBytes, kGt = kVt + kTileBytes;

// The 32-token tiles of Q, K, V and dOut: fetched into registers a tile ahead (tile_fetch), written to the buffer of
// their parity while the other one is in use (tile_commit).  Threads 0..255 carry Q and V pieces, the others K and dOut: xb
// and yb are the first rows of this wave's two.
struct TileRegs {
  u32x4 x, y;
};
__device__ __forceinline__ TileRegs tile_fetch(const us* xb, const us* yb, int tok0, int L, int tid) {
  const int c = tid % 256;
  const unsigned off = (unsigned)min(c / 8, L - 1 - tok0) * kD + 8 * (c % 8);
  const u32x4 zero = {0u, 0u, 0u, 0u};
  TileRegs t;
  t.x = *reinterpret_cast<const u32x4*>(xb + (size_t)tok0 * kD + off);
  t.y = tok0 + c / 8 < L ? *reinterpret_cast<const u32x4*>(yb + (size_t)tok0 * kD + off) : zero;
  return t;
}
__device__ __forceinline__ void tile_commit(unsigned char* buf, const TileRegs& t, int tid) {
  const int c = tid % 256;
  unsigned char* at = buf + (tid / 256) * kTileBytes + 2 * index<kD>(c / 8, 8 * (c % 8));
  *reinterpret_cast<u32x4*>(at) = bf16x8_to_f16x8(t.x);
  *reinterpret_cast<u32x4*>(at + 2 * kTileBytes) = t.y;
}

// A' of head h into LDS.
__device__ __forceinline__ void load_a(us* Al, const _Float16* Ah, int h, int tid) {
  const us* src = reinterpret_cast<const us*>(Ah) + (size_t)h * kF * kD;
  constexpr int NU = kF * kD / 8 / kNT;
  u32x4 v[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) v[u] = *reinterpret_cast<const u32x4*>(src + 8 * (size_t)(tid + kNT * u));
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int i = tid + kNT * u;
    *reinterpret_cast<u32x4*>(Al + index<kD>(i / 8, 8 * (i % 8))) = v[u];
  }
}

// Packed features of one 32-feature block, token per lane: element v of the accumulator is half v % 2 of word v / 2.
__device__ __forceinline__ float feat(const u32x4 (&p)[2], int v) {
  const unsigned w = p[v / 8][(v % 8) / 2];
  return v % 2 ? bf_hi(w) : bf_lo(w);
}
__device__ __forceinline__ void pack_acc(const f32x16& x, u32x4 (&p)[2]) {
#pragma unroll
  for (int q = 0; q < 8; ++q) p[q / 4][q % 4] = pack_bf16(x[2 * q], x[2 * q + 1]);
}
// A block's packed values (rows 8 a + 4 hf + [0,4), lane = row of the tile) to their places.
__device__ __forceinline__ void put_rows(unsigned char* smem, unsigned put, unsigned add, const u32x4 (&p)[2]) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
    *reinterpret_cast<u32x2*>(smem + ((put ^ (16 * a)) + add)) = u32x2{p[a / 2][2 * (a % 2)], p[a / 2][2 * (a % 2) + 1]};
}
// Orders a wave's own LDS accesses for the compiler; the hardware completes them in order.
__device__ __forceinline__ void own_lds_order() { asm volatile("" ::: "memory"); }
// Ends a stage for the instruction scheduler, which otherwise requests the operands of all stages at once and spills.
__device__ __forceinline__ void stage() { __builtin_amdgcn_sched_barrier(0); }

// This wave's 16 x 16 block of dlogit A': token 16 (wv / 4) + lane % 16, columns 16 (wv % 4) + 4 (lane / 16) + [0,4).
__device__ __forceinline__ f32x4 back_project(const unsigned char* smem, const Lanes& ln, unsigned dl) {
  f32x4 o[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int s = 0; s < 8; ++s)
    o[s % 2] = mm16_f16(ld_tr(smem, ln.back, BwdSmem::al + 32 * s * kRow64), ld128(smem, (ln.row ^ (64 * (s % 4))) + dl + 256 * (s / 4)), o[s % 2]);
  return o[0] + o[1];
}

// ---------------------------------------------------------------------------
// k_bwd_fwd, k_bwd_rev: eight waves of 32 features each.  A wave keeps the states of its features in accumulators and forms
// every contraction over features from its own registers, where a packed accumulator is an operand; what remains to be
// joined between waves are three numbers per token (F) or the value gradients and one number per token (R), so a tile
// takes two barriers.  The first version gave each product of a tile to one or two of the eight waves and passed features,
// E and N through LDS, nine barriers a tile: 15,000 cycles per 32 tokens where the matrix products take 2,300.  Now 9,000,
// bound by vector issue (some 1,100 instructions per SIMD and tile).  98,304 rows: 110 -> 73 us and 97 -> 74 us.  Four waves
// of 64 features with 512 registers each: 88 and 90 us, nothing hides a wave's waits.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kNT, 1) void k_bwd_fwd(const us* __restrict__ Qg, const us* __restrict__ Kg,
                                                   const us* __restrict__ Vg, const us* __restrict__ Gg,
                                                   const _Float16* __restrict__ Ah, const float* __restrict__ nrm,
                                                   const float* __restrict__ Spre, const float* __restrict__ zpre,
                                                   const float* __restrict__ cpre, float* __restrict__ dQ,
                                                   float* __restrict__ lam, float* __restrict__ gdv,
                                                   float* __restrict__ dRn, float* __restrict__ dRd,
                                                   float* __restrict__ TQ, int H, int L, int P, int slice_len,
                                                   float inv_log2e) {
  using SM = BwdSmem;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  us* Al = reinterpret_cast<us*>(smem + SM::al);
  float* zs = reinterpret_cast<float*>(smem + SM::f_vec);
  float* tk = reinterpret_cast<float*>(smem + SM::f_tok);
  float* part = reinterpret_cast<float*>(smem + SM::f_part);
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hf = lane / 32;
  float* gdw = reinterpret_cast<float*>(smem + SM::f_gd) + wv * kT;
  const int bh = blockIdx.x / P, p = blockIdx.x % P;
  const int h = bh % H;
  const int tok_begin = p * slice_len;
  const int tok_end = min(L, tok_begin + slice_len);
  if (tok_begin >= tok_end) return;
  const int ntile = (tok_end - tok_begin + kT - 1) / kT;
  const size_t row0 = (size_t)bh * L;
  const us* xb = (wv < 4 ? Qg : Kg) + row0 * kD;
  const us* yb = (wv < 4 ? Vg : Gg) + row0 * kD;
  const float* nb = nrm + row0;
  const float c_ref = cpre[(size_t)bh * P + p];  // the running shift of this slice: its prefix state is expressed in it
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const size_t sb = ((size_t)bh * P + p) * kF;
  // an accumulator's element in a [feature][column] state in memory
  auto st_at = [&](int db, int v) { return (unsigned)(4 * hf * kD + l32 + (8 * (v / 4) + (v % 4)) * kD + 32 * db); };

  TileRegs nxt = tile_fetch(xb, yb, tok_begin, L, tid);
  float nk_nxt = (tid < kT && tok_begin + tid < L) ? nb[tok_begin + tid] : kBigShift;
  // state before the tile of this wave's features: S (rows features, lane = value column), z (lane = feature);
  // the slice's contributions to Rn, Rd, T_Q
  f32x16 S[2], Rn[2], Tq[2];
  const int f0 = 32 * wv;
  const unsigned a_rows = BwdSmem::al + f0 * kRow64;   // this wave's rows of A'
  float z = zpre[sb + f0 + l32], rd = 0.f;
#pragma unroll
  for (int db = 0; db < 2; ++db) {
    Rn[db] = Tq[db] = zero16;
#pragma unroll
    for (int v = 0; v < 16; ++v) S[db][v] = (Spre + (sb + f0) * kD)[st_at(db, v)];
  }
  load_a(Al, Ah, h, tid);
  Lanes ln;
  ln.init(wv, lane);
  unsigned st_tr[2];   // S^T, contraction over value columns
  tr_offsets<kF, false>(st_tr, SM::st, f0, lane);
  auto publish = [&]() {
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      u32x4 sp[2];
      pack_acc(S[db], sp);
      put_rows(smem, ln.put, SM::st - SM::ph + 32 * db * kRow256, sp);
    }
    if (hf == 0) zs[f0 + l32] = z;
  };
  publish();
  tile_commit(smem + SM::x, nxt, tid);
  if (tid < kT) tk[tid] = nk_nxt;
  lds_barrier();

  auto store_dq = [&](int tok0) {
    const f32x4 o = back_project(smem, ln, SM::dl);
    const unsigned i = 16 * (wv / 4) + lane % 16;
    if (tok0 + (int)i < L) *reinterpret_cast<f32x4*>(dQ + (row0 + tok0) * kD + (i * kD + 16 * (wv % 4) + 4 * (lane / 16))) = o * inv_log2e;
  };

  for (int t = 0; t < ntile; ++t) {
    const int tok0 = tok_begin + t * kT;
    ln.renew();
    const unsigned par = (t & 1) * kBufBytes;   // this tile's buffer
    const unsigned dir = ln.dir + par;
    const unsigned trc[2][2] = {{ln.trc[0] + par, ln.trc[1] + par}, {(ln.trc[0] ^ 64) + par, (ln.trc[1] ^ 64) + par}};
    // ---- first half: everything that does not need the denominators ---------------------------------
    if (t + 1 < ntile) {
      nxt = tile_fetch(xb, yb, tok0 + kT, L, tid);
      nk_nxt = (tid < kT && tok0 + kT + tid < L) ? nb[tok0 + kT + tid] : kBigShift;
    }
    u32x4 pq[2], pk[2];   // phi_Q, phi_K, token per lane
    float mu = -INFINITY, den = 0.f, dot = 0.f;
    f32x16 uq = zero16;         // at the end phi_Q before it is rounded
    {
      f32x16 uk = zero16;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const u32x4 xq = ld128(smem, (dir ^ (32 * s)) + kXq), xk = ld128(smem, (dir ^ (32 * s)) + kXk);
        const u32x4 af = ld128(smem, (ln.dir ^ (32 * s)) + a_rows);
        uk = mm_f16(af, xk, uk);
        uq = mm_f16(af, xq, uq);
      }
      const float sub = tk[(t & 1) * kT + l32] + c_ref;
#pragma unroll
      for (int v = 0; v < 16; ++v) uk[v] = fast_exp2(uk[v] - sub);
      pack_acc(uk, pk);
      put_rows(smem, ln.put, 0, pk);
#pragma unroll
      for (int v = 0; v < 16; v += 2) mu = max3(mu, uq[v], uq[v + 1]);
      mu = fmaxf(mu, xor32(mu));
#pragma unroll
      for (int v = 0; v < 16; ++v) uq[v] = fast_exp2(uq[v] - mu);
      pack_acc(uq, pq);
    }
    stage();
    // (S G_i)_f and G_i . v_l (rows features / keys, lane = query)
    f32x16 sg = zero16, ge = zero16, at = zero16;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x4 gf = ld128(smem, (dir ^ (32 * s)) + kGt);
      sg = mm_bf16(ld_tr(smem, st_tr, 16 * s * kRow256), gf, sg);
      ge = mm_bf16(ld128(smem, (dir ^ (32 * s)) + kVt), gf, ge);
    }
    stage();
    // this wave's part of the kernel values phi_Q,i . phi_K,l, of the denominators, and of G_i . N_i = sum_f phi_Q,if (S G_i)_f
    // + sum_l a_il G_i . v_l: with the very terms that enter the logit gradients, G_i . (v_l - out_i) cancels there as it
    // does in exact arithmetic
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) at = mm_bf16(pk[hh], pq[hh], at);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 z4 = *reinterpret_cast<const f32x4*>(zs + f0 + 8 * a + 4 * hf);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float f = feat(pq, 4 * a + j);
        den = fmaf(f, z4[j], den);
        dot = fmaf(f, sg[4 * a + j], dot);
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float a = 8 * (v / 4) + 4 * hf + (v % 4) <= l32 ? at[v] : 0.f;
      den += a;
      dot = fmaf(a, ge[v], dot);
    }
    den += xor32(den);
    dot += xor32(dot);
    if (hf == 0) {
      part[l32 * kNW + wv] = mu;
      part[(kT + l32) * kNW + wv] = den;
      part[(2 * kT + l32) * kNW + wv] = dot;
    }
    stage();
    if (dQ != nullptr && t > 0) store_dq(tok0 - kT);   // of the previous tile
    lds_barrier();
    // ---- second half ----------------------------------------------------------------------------
    const bool valid = tok0 + l32 < L;
    float mx = -INFINITY, dsum = 0.f, dots = 0.f;
    {
      f32x4 m4[2], d4[2], o4[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        m4[k] = *reinterpret_cast<const f32x4*>(part + l32 * kNW + 4 * k);
        d4[k] = *reinterpret_cast<const f32x4*>(part + (kT + l32) * kNW + 4 * k);
        o4[k] = *reinterpret_cast<const f32x4*>(part + (2 * kT + l32) * kNW + 4 * k);
        mx = max3(mx, fmaxf(m4[k][0], m4[k][1]), fmaxf(m4[k][2], m4[k][3]));
      }
#pragma unroll
      for (int w = 0; w < kNW; ++w) {
        const float f = fast_exp2(m4[w / 4][w % 4] - mx);
        dsum = fmaf(f, d4[w / 4][w % 4], dsum);
        dots = fmaf(f, o4[w / 4][w % 4], dots);
      }
    }
    const float rho = valid ? 1.f / dsum : 0.f;
    const float gd = -rho * dots;
    const float rw = rho * fast_exp2(mu - mx);   // phi_Q of this wave times this: phi_Q / D
    if (hf == 0) gdw[l32] = gd;
    if (wv == 0 && hf == 0 && valid) {
      (lam + (row0 + tok0))[l32] = mx + __builtin_log2f(dsum);
      (gdv + (row0 + tok0))[l32] = gd;
    }
    // E_il = G_i . v_l + gd_i for l <= i
    u32x4 ep[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) ge[v] = 8 * (v / 4) + 4 * hf + (v % 4) <= l32 ? ge[v] + gd : 0.f;
    pack_acc(ge, ep);
    // features of the keys, feature per lane
    u32x4 kf[2];
    own_lds_order();
#pragma unroll
    for (int s = 0; s < 2; ++s) kf[s] = ld_tr(smem, ln.ft, 16 * s * kRow256);
    own_lds_order();
    stage();
    // dlogit_Q,if = phi_Q,if / D_i ( (S G_i)_f + gd_i z_f + sum_{l<=i} E_il phi_K,lf )
#pragma unroll
    for (int s = 0; s < 2; ++s) sg = mm_bf16(kf[s], ep[s], sg);
    u32x4 hat[2], dlp[2];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const f32x4 z4 = *reinterpret_cast<const f32x4*>(zs + f0 + 8 * a + 4 * hf);
      float e[4], d[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        e[j] = uq[4 * a + j] * rw;
        d[j] = e[j] * fmaf(z4[j], gd, sg[4 * a + j]);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        hat[a / 2][2 * (a % 2) + j] = pack_bf16(e[2 * j], e[2 * j + 1]);
        dlp[a / 2][2 * (a % 2) + j] = pack_f16(d[2 * j], d[2 * j + 1]);
      }
    }
    put_rows(smem, ln.put, 0, hat);
    put_rows(smem, ln.put, SM::dl - SM::ph, dlp);
    own_lds_order();
    stage();
    // the states take the tile
    f32x4 gk[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) gk[a] = *reinterpret_cast<const f32x4*>(gdw + 8 * a + 4 * hf);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      u32x4 vf[2], gf[2], xf[2];
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        vf[db] = ld_tr(smem, trc[db], kVt + 16 * s * kRow64);
        gf[db] = ld_tr(smem, trc[db], kGt + 16 * s * kRow64);
        xf[db] = ld_tr(smem, trc[db], kXq + 16 * s * kRow64);
      }
      const u32x4 qf = ld_tr(smem, ln.ft, 16 * s * kRow256);
      const u32x4 df = ld_tr(smem, ln.ft, SM::dl - SM::ph + 16 * s * kRow256);
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        S[db] = mm_bf16(kf[s], vf[db], S[db]);
        Rn[db] = mm_bf16(qf, gf[db], Rn[db]);
        Tq[db] = mm_f16(df, xf[db], Tq[db]);
      }
      // z_f += sum_l phi_K,lf,  Rd_f += sum_i phihat_Q,if gd_i (this half-wave's tokens)
      float za = 0.f, ra = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 g4 = gk[2 * s + q / 2];
        za += bf_lo(kf[s][q]) + bf_hi(kf[s][q]);
        ra = fmaf(bf_lo(qf[q]), g4[2 * (q % 2)], ra);
        ra = fmaf(bf_hi(qf[q]), g4[2 * (q % 2) + 1], ra);
      }
      z += za + xor32(za);
      rd += ra + xor32(ra);
    }
    publish();
    if (t + 1 < ntile) {
      tile_commit(smem + SM::x + ((t + 1) & 1) * kBufBytes, nxt, tid);
      if (tid < kT) tk[((t + 1) & 1) * kT + tid] = nk_nxt;
    }
    lds_barrier();
  }
  if (dQ != nullptr) store_dq(tok_begin + (ntile - 1) * kT);
  // ---- the slice's contributions ---------------------------------------------------------------------
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      (dRn + (sb + f0) * kD)[st_at(db, v)] = Rn[db][v];
      (TQ + (sb + f0) * kD)[st_at(db, v)] = Tq[db][v];
    }
  if (hf == 0) dRd[sb + f0 + l32] = rd;
}

// ---------------------------------------------------------------------------
// k_bwd_suffix: Rsuf_p = sum_{p' > p} 2^(c*_p - c*_p') dR_p' (p' descending: fixed order), separate output.
// The contribution of slice p' was formed with denominators in the scale of its own running shift c*_p', and
// meets key features of slice p, which are in the scale of c*_p <= c*_p': the factor (at most one) brings it
// there.  One thread per four state entries; the Rd vector rides at the end.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_bwd_suffix(const float* __restrict__ dRn, const float* __restrict__ dRd,
                                                    const float* __restrict__ cpre, float* __restrict__ Rn,
                                                    float* __restrict__ Rd, int P, long long BH) {
  // four consecutive entries per thread; per (b,h) the kF x kD entries of Rn, then the kF of Rd
  const long long per4 = ((long long)kF * kD + kF) / 4;
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= BH * per4) return;
  const long long bh = idx / per4, e = 4 * (idx % per4);
  const bool isn = e < (long long)kF * kD;
  const float* src = isn ? dRn + (size_t)bh * P * kF * kD + e : dRd + (size_t)bh * P * kF + (e - (long long)kF * kD);
  float* dst = isn ? Rn + (size_t)bh * P * kF * kD + e : Rd + (size_t)bh * P * kF + (e - (long long)kF * kD);
  const size_t pitch = isn ? (size_t)kF * kD : (size_t)kF;
  const float* cb = cpre + (size_t)bh * P;
  f32x4 run = {0.f, 0.f, 0.f, 0.f};
  float c_later = 0.f;  // shift of the slice handled last
  for (int p0 = P - 1; p0 >= 0; p0 -= 8) {   // eight slices' loads in flight, then the (ordered) running sums
    f32x4 v[8];
    float c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p0 - u >= 0) {
        v[u] = *reinterpret_cast<const f32x4*>(src + (size_t)(p0 - u) * pitch);
        c[u] = cb[p0 - u];
      }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p0 - u >= 0) {
        if (p0 - u < P - 1) run *= fast_exp2(c[u] - c_later);
        c_later = c[u];
        *reinterpret_cast<f32x4*>(dst + (size_t)(p0 - u) * pitch) = run;
        run += v[u];
      }
  }
}

// ---------------------------------------------------------------------------
// k_bwd_rev: tiles in reverse order, the running suffix states Rn, Rd in registers.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kNT, 1) void k_bwd_rev(const us* __restrict__ Qg, const us* __restrict__ Kg,
                                                   const us* __restrict__ Vg, const us* __restrict__ Gg,
                                                   const _Float16* __restrict__ Ah, const _Float16* __restrict__ Mh,
                                                   const float* __restrict__ nrm, const float* __restrict__ cpre,
                                                   const float* __restrict__ lam, const float* __restrict__ gdv,
                                                   const float* __restrict__ Rsn, const float* __restrict__ Rsd,
                                                   float* __restrict__ dK, float* __restrict__ dV,
                                                   const float* __restrict__ TQ, float* __restrict__ TK,
                                                   float* __restrict__ RM, int H, int L, int P, int slice_len,
                                                   float inv_log2e) {
  using SM = BwdSmem;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  us* Al = reinterpret_cast<us*>(smem + SM::al);
  float* rds = reinterpret_cast<float*>(smem + SM::r_vec);
  float* tk = reinterpret_cast<float*>(smem + SM::r_tok);
  float* part = reinterpret_cast<float*>(smem + SM::r_part);
  float* sl = reinterpret_cast<float*>(smem + SM::r_sl) + (threadIdx.x / 64) * kT;
  float* ex = reinterpret_cast<float*>(smem + SM::r_ex);
  const int tid = threadIdx.x, lane = tid % 64, wv = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hf = lane / 32, l16 = lane % 16, kg = lane / 16;
  const int bh = blockIdx.x / P, p = blockIdx.x % P;
  const int h = bh % H;
  const int tok_begin = p * slice_len;
  const int tok_end = min(L, tok_begin + slice_len);
  if (tok_begin >= tok_end) return;
  const int ntile = (tok_end - tok_begin + kT - 1) / kT;
  const size_t row0 = (size_t)bh * L;
  const us* xb = (wv < 4 ? Qg : Kg) + row0 * kD;
  const us* yb = (wv < 4 ? Vg : Gg) + row0 * kD;
  const float c_ref = cpre[(size_t)bh * P + p];  // keys of this slice are featurised under its own running shift
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const size_t sb = ((size_t)bh * P + p) * kF;
  // an accumulator's element in a [feature][column] state in memory
  auto st_at = [&](int db, int v) { return (unsigned)(4 * hf * kD + l32 + (8 * (v / 4) + (v % 4)) * kD + 32 * db); };

  // the first three waves carry the tokens' norm, lambda and gd
  const float* sc_src = (wv == 0 ? nrm : wv == 1 ? lam : gdv) + row0;
  auto fetch_scalar = [&](int tk0) { return wv < 3 && lane < kT && tk0 + lane < L ? (sc_src + tk0)[lane] : wv < 2 ? kBigShift : 0.f; };
  const int t_last = tok_begin + (ntile - 1) * kT;
  TileRegs nxt = tile_fetch(xb, yb, t_last, L, tid);
  float sc_nxt = fetch_scalar(t_last);
  // running suffix state of this wave's features; the slice's T: the query half comes from the forward-order pass
  f32x16 Rn[2], Tk[2], Rm = zero16;   // Rm: block (wv % 4 / 2, wv % 2), half of the tokens
  const int f0 = 32 * wv;
  const unsigned a_rows = BwdSmem::al + f0 * kRow64;   // this wave's rows of A'
  float rd = Rsd[sb + f0 + l32];
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      Rn[db][v] = (Rsn + (sb + f0) * kD)[st_at(db, v)];
      Tk[db][v] = (TQ + (sb + f0) * kD)[st_at(db, v)];
    }
  // G2 = M'^T M' (= alpha^2 log2e/2 M^T M), fp16
  {
    us* Ml = reinterpret_cast<us*>(ex);
    us* Gl = reinterpret_cast<us*>(smem + SM::r_g2);
    const us* src = reinterpret_cast<const us*>(Mh) + (size_t)h * kD * kD;
    static_assert(kD * kD / 8 == kNT, "a piece of M' per thread");
    *reinterpret_cast<u32x4*>(Ml + index<kD>(tid / 8, 8 * (tid % 8))) = *reinterpret_cast<const u32x4*>(src + 8 * (size_t)tid);
    __syncthreads();
    if (wv < 4) {
      const int eb = wv / 2, db = wv % 2;
      unsigned me[2], md[2];
      tr_offsets<kD, false>(me, SM::r_ex, 32 * eb, lane);
      tr_offsets<kD, false>(md, SM::r_ex, 32 * db, lane);
      f32x16 acc = zero16;  // rows e, columns d
#pragma unroll
      for (int s = 0; s < kD / 16; ++s)
        acc = mm_f16(ld_tr(smem, me, 16 * s * kRow64), ld_tr(smem, md, 16 * s * kRow64), acc);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        Gl[index<kD>(32 * eb + 8 * (v / 4) + 4 * hf + (v % 4), 32 * db + l32)] = (us)(pack_f16(acc[v], 0.f) & 0xffffu);
    }
  }
  load_a(Al, Ah, h, tid);
  Lanes ln;
  ln.init(wv, lane);
  // this wave's region: copy of Rn before the tile, [64 value columns][32 features]; dV takes its place
  unsigned rt_tr[2];
  const unsigned rm_a = 64 * (wv % 4 / 2), rm_b = 64 * (wv % 2);
  const unsigned own = SM::r_ex + wv * kT * LDE * 4, rt_put = own + 2 * index<32>(l32, 4 * hf);
  tr_offsets<32, false>(rt_tr, own, 0, lane);
  // key of back_project's token, its columns of G2
  const unsigned nk_row = 2 * index<kD>(16 * (wv / 4) + l16, 8 * kg), g2_row = SM::r_g2 + 2 * index<kD>(16 * (wv % 4) + l16, 8 * kg);
  if (hf == 0) rds[f0 + l32] = rd;
  tile_commit(smem + SM::x + ((ntile - 1) & 1) * kBufBytes, nxt, tid);
  if (wv < 3 && lane < kT) tk[(((ntile - 1) & 1) * 3 + wv) * kT + lane] = sc_nxt;
  lds_barrier();

  for (int t = ntile - 1; t >= 0; --t) {
    const int tok0 = tok_begin + t * kT;
    ln.renew();
    const unsigned par = (t & 1) * kBufBytes;   // this tile's buffer
    const unsigned dir = ln.dir + par;
    const unsigned trc[2][2] = {{ln.trc[0] + par, ln.trc[1] + par}, {(ln.trc[0] ^ 64) + par, (ln.trc[1] ^ 64) + par}};
    const float* tkt = tk + (t & 1) * 3 * kT;
    if (t > 0) {
      nxt = tile_fetch(xb, yb, tok0 - kT, L, tid);
      sc_nxt = fetch_scalar(tok0 - kT);
    }
    // ---- first half: features, kernel values, logit gradients, partial dV -----------------------------
    u32x4 pq[2], pk[2];   // phihat_Q = exp2(u - lambda), phi_K, token per lane
    u32x4 rp[2][2];       // Rn
    {
      f32x16 uq = zero16, uk = zero16;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const u32x4 xq = ld128(smem, (dir ^ (32 * s)) + kXq), xk = ld128(smem, (dir ^ (32 * s)) + kXk);
        const u32x4 af = ld128(smem, (ln.dir ^ (32 * s)) + a_rows);
        uq = mm_f16(af, xq, uq);
        uk = mm_f16(af, xk, uk);
      }
      const float subk = tkt[l32] + c_ref, subq = tkt[kT + l32];
#pragma unroll
      for (int v = 0; v < 16; ++v) uq[v] = fast_exp2(uq[v] - subq);
      pack_acc(uq, pq);
      put_rows(smem, ln.put, 0, pq);
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        pack_acc(Rn[db], rp[db]);
        put_rows(smem, rt_put, 32 * db * 32 * 2, rp[db]);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) uk[v] = fast_exp2(uk[v] - subk);
      pack_acc(uk, pk);
    }
    own_lds_order();
    stage();
    // a_il / D_i (this wave's part), G_i . v_l + gd_i, rows queries, lane = key, for i >= l
    u32x4 ap[2], ep[2];
    f32x16 dl;
    {
      f32x16 at = zero16, ge;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 g4 = *reinterpret_cast<const f32x4*>(tkt + 2 * kT + 8 * a + 4 * hf);   // gd
#pragma unroll
        for (int j = 0; j < 4; ++j) ge[4 * a + j] = g4[j];
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) {   // the logit gradients start from Rd
        const f32x4 r4 = *reinterpret_cast<const f32x4*>(rds + f0 + 8 * a + 4 * hf);
#pragma unroll
        for (int j = 0; j < 4; ++j) dl[4 * a + j] = r4[j];
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const u32x4 vf = ld128(smem, (dir ^ (32 * s)) + kVt);
        ge = mm_bf16(ld128(smem, (dir ^ (32 * s)) + kGt), vf, ge);
        dl = mm_bf16(ld_tr(smem, rt_tr, 16 * s * 32 * 2), vf, dl);
      }
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) at = mm_bf16(pq[hh], pk[hh], at);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const bool in = 8 * (v / 4) + 4 * hf + (v % 4) >= l32;
        at[v] = in ? at[v] : 0.f;
        ge[v] = in ? ge[v] : 0.f;
      }
      pack_acc(at, ap);
      pack_acc(ge, ep);
    }
    stage();
    u32x4 gf[2][2], qf[2];   // dOut (lane = column) and phihat_Q (lane = feature), contraction over queries
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int db = 0; db < 2; ++db) gf[db][s] = ld_tr(smem, trc[db], kGt + 16 * s * kRow64);
      qf[s] = ld_tr(smem, ln.ft, 16 * s * kRow256);
    }
    own_lds_order();
    // dV^T (rows columns of V, lane = key)
    if (dV != nullptr) {
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        f32x16 acc = zero16;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) acc = mm_bf16(rp[db][hh], pk[hh], acc);
#pragma unroll
        for (int s = 0; s < 2; ++s) acc = mm_bf16(gf[db][s], ap[s], acc);
        float* e = ex + (wv * kT + l32) * LDE + 32 * db + 4 * hf;
#pragma unroll
        for (int a = 0; a < 4; ++a) *reinterpret_cast<f32x4*>(e + 8 * a) = f32x4{acc[4 * a], acc[4 * a + 1], acc[4 * a + 2], acc[4 * a + 3]};
      }
    }
    stage();
    // dlogit_K,lf = phi_K,lf ( (Rn v_l)_f + Rd_f + sum_{i>=l} phihat_Q,if E_il )
    float ssum = 0.f;
#pragma unroll
    for (int s = 0; s < 2; ++s) dl = mm_bf16(qf[s], ep[s], dl);
    u32x4 dlp[2];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float d0 = feat(pk, 2 * q) * dl[2 * q], d1 = feat(pk, 2 * q + 1) * dl[2 * q + 1];
      ssum += d0 + d1;
      dlp[q / 4][q % 4] = pack_f16(d0, d1);
    }
    put_rows(smem, ln.put, 0, dlp);   // in the place of phihat_Q
    ssum += xor32(ssum);
    if (hf == 0) part[l32 * kNW + wv] = ssum;
    stage();
    // the suffix state takes the tile's queries
    float ra = 0.f;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int db = 0; db < 2; ++db) Rn[db] = mm_bf16(qf[s], gf[db][s], Rn[db]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 g4 = *reinterpret_cast<const f32x4*>(tkt + 2 * kT + 16 * s + 8 * (q / 2) + 4 * hf);
        ra = fmaf(bf_lo(qf[s][q]), g4[2 * (q % 2)], ra);
        ra = fmaf(bf_hi(qf[s][q]), g4[2 * (q % 2) + 1], ra);
      }
    }
    rd += ra + xor32(ra);
    stage();
    if (hf == 0) rds[f0 + l32] = rd;
    lds_barrier();
    // ---- second half: dV, dK, T_K, Rm -----------------------------------------------------------------
    {
      const f32x4 a = *reinterpret_cast<const f32x4*>(part + l32 * kNW), b = *reinterpret_cast<const f32x4*>(part + l32 * kNW + 4);
      if (hf == 0) sl[l32] = ((a[0] + a[1]) + (a[2] + a[3])) + ((b[0] + b[1]) + (b[2] + b[3]));
      own_lds_order();
    }
    if (dV != nullptr && tok0 + tid / 16 < L) {
      const float* e = ex + (tid / 16) * LDE + 4 * (tid % 16);
      f32x4 x = *reinterpret_cast<const f32x4*>(e);
#pragma unroll
      for (int w = 1; w < kNW; ++w) x += *reinterpret_cast<const f32x4*>(e + w * kT * LDE);
      *reinterpret_cast<f32x4*>(dV + (row0 + tok0) * kD + 4 * (unsigned)tid) = x;
    }
    if (dK != nullptr) {
      const int l = 16 * (wv / 4) + l16, c0 = 16 * (wv % 4) + 4 * kg;
      const f32x4 o = back_project(smem, ln, SM::ph);
      f32x4 n = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 2; ++s) n = mm16_f16(ld128(smem, (g2_row ^ (64 * s))), ld128(smem, (nk_row ^ (64 * s)) + par + kXk), n);
      const float s_l = sl[l];
      if (tok0 + l < L) *reinterpret_cast<f32x4*>(dK + (row0 + tok0) * kD + (unsigned)(l * kD + c0)) = (o - 2.f * s_l * n) * inv_log2e;
    }
    // T_K += dlogit^T K;  Rm += (s k) k^T, tokens 16 (wv / 4) + [0,16) here: slots 0..3 are 4 hf + [0,4), slots 4..7 those + 8
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const u32x4 df = ld_tr(smem, ln.ft, 16 * s * kRow256);
#pragma unroll
      for (int db = 0; db < 2; ++db) Tk[db] = mm_f16(df, ld_tr(smem, trc[db], kXk + 16 * s * kRow64), Tk[db]);
    }
    {
      const unsigned add = kXk + (wv / 4) * 16 * kRow64 + par;
      const unsigned ra[2] = {ln.trc[0] ^ rm_a, ln.trc[1] ^ rm_a}, rb[2] = {ln.trc[0] ^ rm_b, ln.trc[1] ^ rm_b};
      u32x4 xa = ld_tr(smem, ra, add);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const f32x4 s4 = *reinterpret_cast<const f32x4*>(sl + 16 * (wv / 4) + 8 * c + 4 * hf);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const unsigned wq = xa[2 * c + q];
          const fp16x2 hv2 = *reinterpret_cast<const fp16x2*>(&wq);
          xa[2 * c + q] = pack_f16((float)hv2[0] * s4[2 * q], (float)hv2[1] * s4[2 * q + 1]);
        }
      }
      Rm = mm_f16(xa, ld_tr(smem, rb, add), Rm);
    }
    if (t > 0) {
      tile_commit(smem + SM::x + ((t - 1) & 1) * kBufBytes, nxt, tid);
      if (wv < 3 && lane < kT) tk[(((t - 1) & 1) * 3 + wv) * kT + lane] = sc_nxt;
    }
    lds_barrier();
  }
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      (TK + (sb + f0) * kD)[st_at(db, v)] = Tk[db][v];
  float* half = ex + (wv % 4) * 64 * 16 + lane;   // the upper four waves hand their halves of Rm over
  if (wv >= 4)
#pragma unroll
    for (int v = 0; v < 16; ++v) half[64 * v] = Rm[v];
  lds_barrier();
  if (wv < 4) {
    const size_t rb = ((size_t)bh * P + p) * kD;
#pragma unroll
    for (int v = 0; v < 16; ++v)
      RM[(rb + 32 * (wv / 2) + 8 * (v / 4) + 4 * hf + (v % 4)) * kD + 32 * (wv % 2) + l32] = Rm[v] + half[64 * v];
  }
}

}  // namespace

bool fused_bwd_supported(const Problem& pb, bool causal) {
  const dark_params& p = pb.p;
  return causal && p.io_dtype == DARK_BF16 && p.d == 64 && p.r == 64 && p.dv == 64 && p.m == 256;
}

dark_status fused_attn_bwd(const Problem& pb, Arena& ar, const void* Q, const void* K, const void* V, const float* M,
                           const float* W, const void* dOut, float* dQ, float* dK, float* dV, float* dM, float* dW) {
  const dark_params& p = pb.p;
  const long long BH = pb.BH();
  int P, sl;
  causal_slices(pb, &P, &sl);

  const size_t nstate = (size_t)BH * P * kF;
  // operand copies, key norms and prefix states: from the forward's hand-over buffer when the caller has one
  Arena sv(pb.saved, pb.saved_bytes);
  const bool handover = pb.saved_mode == 2 && ar.base != nullptr;
  const CausalKeep kp = take_causal_keep(handover ? sv : ar, pb, P);
  _Float16 *Ah = kp.Ah, *Mh = kp.Mh;
  float *Spre = kp.Spre, *zpre = kp.zpre, *cpre = kp.cpre, *nrm = kp.nrm;
  unsigned short* Spart = ar.take<unsigned short>(nstate * kD);
  float* zpart = ar.take<float>(nstate);
  float* cpart = ar.take<float>(nstate);
  float* lam = ar.take<float>((size_t)BH * p.L);
  float* gdv = ar.take<float>((size_t)BH * p.L);
  float* dRn = ar.take<float>(nstate * kD);
  float* dRd = ar.take<float>(nstate);
  float* Rsn = ar.take<float>(nstate * kD);
  float* Rsd = ar.take<float>(nstate);
  float* TQ = ar.take<float>(nstate * kD);
  float* TK = ar.take<float>(nstate * kD);
  float* RM = ar.take<float>((size_t)BH * P * kD * kD);
  float* Tsum = ar.take<float>((size_t)p.H * kF * kD);
  float* Rmsum = ar.take<float>((size_t)p.H * kD * kD);
  if (ar.base == nullptr) return DARK_OK;
  if (ar.overflow || sv.overflow) return DARK_EWORKSPACE;

  if (!handover) {
    DARK_TRY(fused_launch_prep(pb, M, W, Ah, Mh, false));
    DARK_TRY(fused_causal_states64(pb, K, V, Ah, Mh, nrm, Spart, zpart, cpart, Spre, zpre, cpre, P, sl));
  }
  const float inv_log2e = 0.6931471805599453f;
  const unsigned grid = (unsigned)(BH * P);
  typedef const unsigned short* cus;
  DARK_TRY(allow_lds(k_bwd_fwd, BwdSmem::fwd_total));
  DARK_LAUNCH(KID_BWD_FWD, pb.st, k_bwd_fwd, dim3(grid), dim3(kNT), BwdSmem::fwd_total, (cus)Q, (cus)K, (cus)V, (cus)dOut, Ah,
              nrm, Spre, zpre, cpre, dQ, lam, gdv, dRn, dRd, TQ, p.H, p.L, P, sl, inv_log2e);
  {
    const long long n = BH * ((long long)kF * kD + kF) / 4;
    DARK_LAUNCH(KID_BWD_SUFFIX, pb.st, k_bwd_suffix, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, dRn, dRd, cpre, Rsn, Rsd, P,
                BH);
  }
  DARK_TRY(allow_lds(k_bwd_rev, BwdSmem::rev_total));
  DARK_LAUNCH(KID_BWD_REV, pb.st, k_bwd_rev, dim3(grid), dim3(kNT), BwdSmem::rev_total, (cus)Q, (cus)K, (cus)V, (cus)dOut, Ah, Mh,
              nrm, cpre, lam, gdv, Rsn, Rsd, dK, dV, TQ, TK, RM, p.H, p.L, P, sl, inv_log2e);
  if (dM != nullptr || dW != nullptr) return launch_geometry(pb, TK, RM, P, Tsum, Rmsum, M, W, dM, dW);
  return DARK_OK;
}

}  // namespace dark
