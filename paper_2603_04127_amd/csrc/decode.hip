// One step of causal random-feature attention as a recurrence: the state (S, z) of a (b,h) absorbs the new
// key/value pair and the new query reads it out (the causal form of Section 2's linear attention, one token
// at a time: out_t = phi(q_t)^T S_t / phi(q_t)^T z_t with S_t = S_{t-1} + phi(k_t) v_t^T, z_t = z_{t-1} + phi(k_t)).
// The state is kept under one scalar shift c per (b,h) (natural-log domain): it holds sum_l exp(logit_l - c) v_l^T;
// a new key whose largest logit exceeds c raises c and rescales the state.
// One workgroup per (b,h); fp32 arithmetic.  k_decode_rows serves d = r = dv = 64 or 128 with the usual feature counts,
// k_decode_step everything else.
#include <cmath>

#include "common.h"

namespace dark {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ float ld1(const T* p, size_t i);
template <>
__device__ __forceinline__ float ld1<float>(const float* p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float ld1<unsigned short>(const unsigned short* p, size_t i) {
  return __uint_as_float((unsigned)p[i] << 16);
}
__device__ __forceinline__ void st1(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st1(unsigned short* p, size_t i, float v) {
  // round to nearest even
  unsigned u = __float_as_uint(v);
  if ((u & 0x7f800000u) != 0x7f800000u) u += 0x7fffu + ((u >> 16) & 1u);
  p[i] = (unsigned short)(u >> 16);
}

__device__ __forceinline__ float block_max(float v, float* red, int tid) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  __syncthreads();
  if (tid % 64 == 0) red[tid / 64] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}
__device__ __forceinline__ float block_sum(float v, float* red, int tid) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if (tid % 64 == 0) red[tid / 64] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// LDS: xq[d], xk[d], tq[r], tk[r], eq[m], ek[m], vv[dv], num[256] (partial numerators), red[4]
template <typename T>
__global__ __launch_bounds__(256) void k_decode_step(const T* __restrict__ q, const T* __restrict__ k,
                                                     const T* __restrict__ v, const float* __restrict__ M,
                                                     const float* __restrict__ W, float* __restrict__ S,
                                                     float* __restrict__ z, float* __restrict__ c, T* __restrict__ out,
                                                     int H, int d, int r, int m, int dv, int w_shared, float alpha) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* xq = reinterpret_cast<float*>(smem);
  float* xk = xq + d;
  float* tq = xk + d;
  float* tk = tq + r;
  float* eq = tk + r;
  float* ek = eq + m;
  float* vv = reinterpret_cast<float*>(smem) + ((2 * d + 2 * r + 2 * m + 3) / 4) * 4;   // 16-byte aligned
  float* num = vv + ((dv + 3) / 4) * 4;      // [256]
  float* red = num + 256;    // [4]
  const int tid = threadIdx.x, bh = blockIdx.x, h = bh % H;
  // The state does not depend on anything computed here: when it is small enough (16 pieces of 16 bytes per
  // thread: m dv <= 16384) all of it is requested first and arrives while the logits are being formed.
  const int cg = (dv + 3) / 4;             // groups of four columns
  float* Sb = S + (size_t)bh * m * dv;
  float* zb = z + (size_t)bh * m;
  const bool vec = dv % 4 == 0 && 256 % cg == 0;
  const int col = vec ? 4 * (tid % cg) : 0, rstep = vec ? 256 / cg : 1;
  const bool early = vec && m <= 16 * rstep;
  f32x4 se[16];
  if (early) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int j = tid / cg + u * rstep;
      if (j < m) se[u] = *reinterpret_cast<const f32x4*>(Sb + (size_t)j * dv + col);
    }
  }
  for (int i = tid; i < d; i += 256) {
    xq[i] = alpha * ld1<T>(q, (size_t)bh * d + i);
    xk[i] = alpha * ld1<T>(k, (size_t)bh * d + i);
  }
  for (int i = tid; i < dv; i += 256) vv[i] = ld1<T>(v, (size_t)bh * dv + i);
  __syncthreads();
  // x~ = M x'
  const float* Mh = M != nullptr ? M + (size_t)h * r * d : nullptr;  // null: the identity (r == d)
  for (int t = tid; t < r; t += 256) {
    float a = 0.f, b = 0.f;
    if (Mh != nullptr && d % 4 == 0) {   // rows of M as 16-byte loads, eight in flight
      const f32x4* mr = reinterpret_cast<const f32x4*>(Mh + (size_t)t * d);
      for (int e0 = 0; e0 < d / 4; e0 += 8) {
        f32x4 mv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) mv[u] = mr[min(e0 + u, d / 4 - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (e0 + u < d / 4) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              a = fmaf(mv[u][x], xq[4 * (e0 + u) + x], a);
              b = fmaf(mv[u][x], xk[4 * (e0 + u) + x], b);
            }
          }
      }
    } else if (Mh != nullptr) {
      for (int e = 0; e < d; ++e) {
        const float mv = Mh[(size_t)t * d + e];
        a = fmaf(mv, xq[e], a);
        b = fmaf(mv, xk[e], b);
      }
    } else {
      a = xq[t];
      b = xk[t];
    }
    tq[t] = a;
    tk[t] = b;
  }
  __syncthreads();
  float nq = 0.f, nk = 0.f;
  for (int t = tid; t < r; t += 256) {
    nq = fmaf(tq[t], tq[t], nq);
    nk = fmaf(tk[t], tk[t], nk);
  }
  nq = 0.5f * block_sum(nq, red, tid);
  nk = 0.5f * block_sum(nk, red, tid);
  // logits
  const float* Wh = W + (w_shared ? 0 : (size_t)h * m * r);
  float mq = -INFINITY, mk = -INFINITY;
  for (int j = tid; j < m; j += 256) {
    float a = 0.f, b = 0.f;
    if (r % 4 == 0) {
      const f32x4* wr = reinterpret_cast<const f32x4*>(Wh + (size_t)j * r);
      for (int t0 = 0; t0 < r / 4; t0 += 8) {
        f32x4 wv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) wv[u] = wr[min(t0 + u, r / 4 - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (t0 + u < r / 4) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              a = fmaf(wv[u][x], tq[4 * (t0 + u) + x], a);
              b = fmaf(wv[u][x], tk[4 * (t0 + u) + x], b);
            }
          }
      }
    } else {
      for (int t = 0; t < r; ++t) {
        const float wv = Wh[(size_t)j * r + t];
        a = fmaf(wv, tq[t], a);
        b = fmaf(wv, tk[t], b);
      }
    }
    a -= nq;
    b -= nk;
    eq[j] = a;
    ek[j] = b;
    mq = fmaxf(mq, a);
    mk = fmaxf(mk, b);
  }
  mq = block_max(mq, red, tid);
  mk = block_max(mk, red, tid);
  const float c_old = c[bh];
  const float c_new = fmaxf(c_old, mk);
  const float down = expf(c_old - c_new);   // 0 for the first token (c_old = -inf)
  for (int j = tid; j < m; j += 256) {
    eq[j] = expf(eq[j] - mq);
    ek[j] = expf(ek[j] - c_new);
  }
  __syncthreads();
  // state update and read-out: thread t walks the rows j = t / cg, t / cg + 256 / cg, ... of its column group
  float den = 0.f;
  for (int j = tid; j < m; j += 256) {
    const float zn = zb[j] * down + ek[j];
    zb[j] = zn;
    den = fmaf(eq[j], zn, den);
  }
  den = block_sum(den, red, tid);
  const float inv = 1.f / den;
  if (vec) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const f32x4 v4 = *reinterpret_cast<const f32x4*>(vv + col);
    if (early) {
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int j = tid / cg + u * rstep;
        if (j < m) {
          const float e = ek[j], f = eq[j];
          f32x4 sn;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            sn[x] = fmaf(e, v4[x], se[u][x] * down);
            acc[x] = fmaf(f, sn[x], acc[x]);
          }
          *reinterpret_cast<f32x4*>(Sb + (size_t)j * dv + col) = sn;
        }
      }
    } else
    for (int j0 = tid / cg; j0 < m; j0 += 4 * rstep) {
      f32x4 sv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (j0 + u * rstep < m) sv[u] = *reinterpret_cast<const f32x4*>(Sb + (size_t)(j0 + u * rstep) * dv + col);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + u * rstep;
        if (j < m) {
          const float e = ek[j], f = eq[j];
          f32x4 sn;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            sn[x] = fmaf(e, v4[x], sv[u][x] * down);
            acc[x] = fmaf(f, sn[x], acc[x]);
          }
          *reinterpret_cast<f32x4*>(Sb + (size_t)j * dv + col) = sn;
        }
      }
    }
    // add the partial numerators of the threads that share a column group
    __syncthreads();
    for (int x = 0; x < 4; ++x) {
      num[tid] = acc[x];
      __syncthreads();
      if (tid < cg) {
        float s = 0.f;
        for (int u = tid; u < 256; u += cg) s += num[u];
        st1(out, (size_t)bh * dv + 4 * tid + x, s * inv);
      }
      __syncthreads();
    }
  } else {
    // general shapes: a thread per column
    for (int col = tid; col < dv; col += 256) {
      float acc = 0.f;
      for (int j = 0; j < m; ++j) {
        const float sn = fmaf(ek[j], vv[col], Sb[(size_t)j * dv + col] * down);
        Sb[(size_t)j * dv + col] = sn;
        acc = fmaf(eq[j], sn, acc);
      }
      st1(out, (size_t)bh * dv + col, acc * inv);
    }
  }
  if (tid == 0) c[bh] = c_new;
}

// d = r = dv = D, m = MF: sixteen waves, and every global load of the step (the rows of M and W, the state, z) is issued
// before the first wait, so the step pays one memory round trip and then four short phases with a barrier between them.
// The 16-byte pieces of a row lie in D / 4 consecutive lanes: the loads are whole lines, and the dot products with x (and
// x~) end in a sum over those lanes.  128 (b,h), D = 128, m = 256 (37 MB, 7.2 us at the rate of a copy): 10.2 us; the general
// kernel, a thread per row of M and W and four waves, takes 24.5.
template <int N>
__device__ __forceinline__ float row_ror(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float lanes16_sum(float v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  return v + row_ror<1>(v);
}
__device__ __forceinline__ float lanes16_max(float v) {
  v = fmaxf(v, row_ror<8>(v));
  v = fmaxf(v, row_ror<4>(v));
  v = fmaxf(v, row_ror<2>(v));
  return fmaxf(v, row_ror<1>(v));
}
// a summed over lanes l and l ^ 16 in the even rows of sixteen lanes, b likewise in the odd ones
__device__ __forceinline__ float join16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float wave_all_sum(float v) {
  v = lanes16_sum(v);
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float wave_all_max(float v) {
  v = lanes16_max(v);
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}

template <typename T, int D, int MF>
__global__ __launch_bounds__(1024) void k_decode_rows(const T* __restrict__ q, const T* __restrict__ k,
                                                      const T* __restrict__ v, const float* __restrict__ M,
                                                      const float* __restrict__ W, float* __restrict__ S,
                                                      float* __restrict__ z, float* __restrict__ c, T* __restrict__ out,
                                                      int H, int w_shared, float alpha) {
  constexpr int NT = 1024, PR = D / 4;                    // lanes per row
  constexpr int NM = D * PR / NT, NW = MF * PR / NT;      // pieces per thread: of M; of W and of the state
  static_assert(D == 64 || D == 128, "a row spans one or two groups of sixteen lanes");
  __shared__ __attribute__((aligned(16))) float x[2][D], xt[2][D], lg[2][MF], acc[16][D];
  __shared__ float dsum[16];
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64, bh = blockIdx.x, h = bh % H;
  const int col = tid % PR, row0 = tid / PR;
  constexpr int RS = NT / PR;                             // rows from one piece of a thread to the next
  const f32x4* Wp = reinterpret_cast<const f32x4*>(W + (w_shared ? 0 : (size_t)h * MF * D));
  f32x4* Sp = reinterpret_cast<f32x4*>(S + (size_t)bh * MF * D);
  float xin = 0.f;
  if (tid < 2 * D) xin = alpha * ld1<T>(tid < D ? q : k, (size_t)bh * D + tid % D);
  f32x4 mv[NM], wr[NW], sv[NW];
  if (M != nullptr) {
    const f32x4* Mp = reinterpret_cast<const f32x4*>(M + (size_t)h * D * D);
#pragma unroll
    for (int u = 0; u < NM; ++u) mv[u] = Mp[tid + NT * u];
  }
#pragma unroll
  for (int u = 0; u < NW; ++u) wr[u] = Wp[tid + NT * u];
  f32x4 v4;
#pragma unroll
  for (int e = 0; e < 4; ++e) v4[e] = ld1<T>(v, (size_t)bh * D + 4 * col + e);
  const float c_old = c[bh];
  float zo = 0.f;
  if (tid < MF) zo = z[(size_t)bh * MF + tid];
#pragma unroll
  for (int u = 0; u < NW; ++u) sv[u] = Sp[tid + NT * u];
  if (tid < 2 * D) x[tid / D][tid % D] = xin;
  __syncthreads();
  // x~ = M x', both tokens
  if (M != nullptr) {
    const f32x4 xq = *reinterpret_cast<const f32x4*>(&x[0][4 * col]), xk = *reinterpret_cast<const f32x4*>(&x[1][4 * col]);
#pragma unroll
    for (int u = 0; u < NM; ++u) {
      float a = mv[u][0] * xq[0], b = mv[u][0] * xk[0];
#pragma unroll
      for (int e = 1; e < 4; ++e) {
        a = fmaf(mv[u][e], xq[e], a);
        b = fmaf(mv[u][e], xk[e], b);
      }
      const int r = row0 + RS * u;
      if (D == 128) {
        const float s = lanes16_sum(join16(a, b));
        if (lane % 16 == 0) xt[(lane / 16) % 2][r] = s;
      } else {
        a = lanes16_sum(a);
        b = lanes16_sum(b);
        if (lane % 16 < 2) xt[lane % 16][r] = lane % 16 ? b : a;
      }
    }
  } else if (tid < 2 * D) {
    xt[tid / D][tid % D] = x[tid / D][tid % D];
  }
  __syncthreads();
  // logits of the thread's rows, both tokens; the norms by every wave for itself
  {
    const f32x4 tq = *reinterpret_cast<const f32x4*>(&xt[0][4 * col]), tk = *reinterpret_cast<const f32x4*>(&xt[1][4 * col]);
    float nq = 0.f, nk = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      nq = fmaf(tq[e], tq[e], nq);
      nk = fmaf(tk[e], tk[e], nk);
    }
    // a row's lanes hold all of x~
    float n;   // D = 128: the query's norm in even rows of sixteen lanes, the key's in odd ones
    if (D == 128) {
      n = 0.5f * lanes16_sum(join16(nq, nk));
    } else {
      nq = 0.5f * lanes16_sum(nq);
      nk = 0.5f * lanes16_sum(nk);
      n = lane % 16 ? nk : nq;
    }
#pragma unroll
    for (int u = 0; u < NW; ++u) {
      float a = wr[u][0] * tq[0], b = wr[u][0] * tk[0];
#pragma unroll
      for (int e = 1; e < 4; ++e) {
        a = fmaf(wr[u][e], tq[e], a);
        b = fmaf(wr[u][e], tk[e], b);
      }
      const int r = row0 + RS * u;
      if (D == 128) {
        const float s = lanes16_sum(join16(a, b));
        if (lane % 16 == 0) lg[(lane / 16) % 2][r] = s - n;
      } else {
        a = lanes16_sum(a);
        b = lanes16_sum(b);
        if (lane % 16 < 2) lg[lane % 16][r] = (lane % 16 ? b : a) - n;
      }
    }
  }
  __syncthreads();
  // the maxima, by every wave for itself
  float mq = -INFINITY, mk = -INFINITY;
#pragma unroll
  for (int u = 0; u < MF / 64; ++u) {
    mq = fmaxf(mq, lg[0][lane + 64 * u]);
    mk = fmaxf(mk, lg[1][lane + 64 * u]);
  }
  mq = wave_all_max(mq);
  mk = wave_all_max(mk);
  const float c_new = fmaxf(c_old, mk);
  const float down = expf(c_old - c_new);   // 0 for the first token (c_old = -inf)
  // features; z and the denominator
  float e0 = 0.f, e1 = 0.f;
  if (tid < MF) {
    e0 = expf(lg[0][tid] - mq);
    e1 = expf(lg[1][tid] - c_new);
  }
  __syncthreads();   // every wave has read the logits
  if (tid < MF) {
    lg[0][tid] = e0;
    lg[1][tid] = e1;
    const float zn = zo * down + e1;
    z[(size_t)bh * MF + tid] = zn;
    const float d = wave_all_sum(e0 * zn);
    if (lane == 0) dsum[wv] = d;
  }
  if (tid == 0) c[bh] = c_new;
  __syncthreads();
  f32x4 a4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < NW; ++u) {
    const float f = lg[0][row0 + RS * u], e = lg[1][row0 + RS * u];
    f32x4 sn;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sn[i] = fmaf(e, v4[i], sv[u][i] * down);
      a4[i] = fmaf(f, sn[i], a4[i]);
    }
    Sp[tid + NT * u] = sn;
  }
  // sum over the rows: lanes of equal column of the wave, then the waves
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (D == 64) a4[i] += __shfl_xor(a4[i], 16, 64);
    a4[i] += __shfl_xor(a4[i], 32, 64);
  }
  if (lane < PR) *reinterpret_cast<f32x4*>(&acc[wv][4 * col]) = a4;
  __syncthreads();
  if (tid < D) {
    float s = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) s += acc[w][tid];
#pragma unroll
    for (int w = 0; w < (MF + 63) / 64; ++w) den += dsum[w];
    st1(out, (size_t)bh * D + tid, s / den);
  }
}

template <typename T>
bool launch_rows(const Problem& pb, const T* q, const T* k, const T* v, const float* M, const float* W, float* S, float* z,
                 float* c, T* out, dark_status* st) {
  const dark_params& p = pb.p;
  if (p.r != p.d || p.dv != p.d) return false;
  if (pb.BH() > 0xffffffffLL / 1024) return false;   // a launch holds 2^32 - 1 threads
  auto go = [&](auto kern) -> dark_status {
    DARK_LAUNCH(KID_DECODE, pb.st, kern, dim3((unsigned)pb.BH()), dim3(1024), 0, q, k, v, M, W, S, z, c, out, p.H,
                p.w_shared, std::sqrt(pb.scale));
    return DARK_OK;
  };
  if (p.d == 64 && p.m == 128) *st = go(k_decode_rows<T, 64, 128>);
  else if (p.d == 64 && p.m == 256) *st = go(k_decode_rows<T, 64, 256>);
  else if (p.d == 64 && p.m == 512) *st = go(k_decode_rows<T, 64, 512>);
  else if (p.d == 128 && p.m == 128) *st = go(k_decode_rows<T, 128, 128>);
  else if (p.d == 128 && p.m == 256) *st = go(k_decode_rows<T, 128, 256>);
  else return false;
  return true;
}

}  // namespace

dark_status decode_step(const Problem& pb, const void* q, const void* k, const void* v, const float* M,
                        const float* W, float* S, float* z, float* c, void* out) {
  const dark_params& p = pb.p;
  const size_t lds = (size_t)(2 * p.d + 2 * p.r + 2 * p.m + p.dv + 8 + 256 + 4) * sizeof(float);
  if (lds > 48 * 1024) return DARK_EUNSUPPORTED;
  dark_status rows_st = DARK_OK;
  if (p.io_dtype == DARK_BF16 ? launch_rows(pb, (const unsigned short*)q, (const unsigned short*)k, (const unsigned short*)v,
                                            M, W, S, z, c, (unsigned short*)out, &rows_st)
                              : launch_rows(pb, (const float*)q, (const float*)k, (const float*)v, M, W, S, z, c, (float*)out,
                                            &rows_st))
    return rows_st;
  const unsigned grid = (unsigned)pb.BH();
  const float alpha = std::sqrt(pb.scale);
  if (p.io_dtype == DARK_BF16)
    DARK_LAUNCH(KID_DECODE, pb.st, k_decode_step<unsigned short>, dim3(grid), dim3(256), lds, (const unsigned short*)q,
                (const unsigned short*)k, (const unsigned short*)v, M, W, S, z, c, (unsigned short*)out, p.H, p.d, p.r,
                p.m, p.dv, p.w_shared, alpha);
  else
    DARK_LAUNCH(KID_DECODE, pb.st, k_decode_step<float>, dim3(grid), dim3(256), lds, (const float*)q, (const float*)k,
                (const float*)v, M, W, S, z, c, (float*)out, p.H, p.d, p.r, p.m, p.dv, p.w_shared, alpha);
  return DARK_OK;
}

}  // namespace dark
