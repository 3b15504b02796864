// Epilogues of the projection kernels (device code): bias, activation,
// residual and Euler updates, GeGLU, head scatter with RoPE, row tables; per
// element, per four aligned columns of a tile in LDS, and from the matrix
// accumulators.
#pragma once
#include "common.h"
#include "rownorm.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2v;

// s0 + v0^2 + v1^2 + v2^2 + v3^2 and s1 + v4^2 + ... + v7^2 with the bf16
// pair dot instruction (two accumulators keep the chain short)
__device__ __forceinline__ void sumsq8(const bf16x8& v, float& s0, float& s1) {
  const bf16x2v p0 = __builtin_shufflevector(v, v, 0, 1), p1 = __builtin_shufflevector(v, v, 2, 3);
  const bf16x2v p2 = __builtin_shufflevector(v, v, 4, 5), p3 = __builtin_shufflevector(v, v, 6, 7);
  s0 = __builtin_amdgcn_fdot2_f32_bf16(p0, p0, s0, false);
  s1 = __builtin_amdgcn_fdot2_f32_bf16(p2, p2, s1, false);
  s0 = __builtin_amdgcn_fdot2_f32_bf16(p1, p1, s0, false);
  s1 = __builtin_amdgcn_fdot2_f32_bf16(p3, p3, s1, false);
}
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
struct __attribute__((packed, aligned(4))) f32x4u { f32x4 v; };      // four floats at any float's address

// ---------------------------------------------------------------- epilogue
__device__ __forceinline__ float act_apply(float x, int act) {
  if (act == ACT_SILU) return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x));   // -0 once e^-x overflows
  if (act == ACT_GELU) {
    // tanh form: 0.5 x (1 + tanh u) with u = sqrt(2/pi) (x + 0.044715 x^3),
    // evaluated through the identity 0.5 (1 + tanh u) = 1 / (1 + e^(-2u)):
    // the hardware exp2 and reciprocal (about 1 ulp each) in place of the
    // library tanh; e^(-2u) = +inf for very negative x gives -0, = 0 for very
    // positive x gives x
    const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
    return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-2.8853900817779268f * u));   // 2 log2 e
  }
  return x;
}

__device__ __forceinline__ void store_elem(void* base, long idx, int type, float v) {
  if (type == ET_BF16) reinterpret_cast<bf16*>(base)[idx] = (bf16)v;
  else reinterpret_cast<float*>(base)[idx] = v;
}

// The residual update x + g * (d + b) (g = the gate, or 1) and the Euler
// update x + dt * (d + b), each one explicit fused multiply-add after the
// bias add, so that every epilogue path (per-element, vector, from
// registers, the reduce fused with a row norm) rounds alike.
__device__ __forceinline__ float upd(float x, float d, float b, float g) { return fmaf(d + b, g, x); }
__device__ __forceinline__ f32x4 upd(f32x4 x, f32x4 d, f32x4 b, f32x4 g) {
  return f32x4{upd(x[0], d[0], b[0], g[0]), upd(x[1], d[1], b[1], g[1]), upd(x[2], d[2], b[2], g[2]),
               upd(x[3], d[3], b[3], g[3])};
}

// Epilogue for output row m and the four columns n0..n0+3 (n0 % 4 == 0).
template <int MODE>
__device__ __forceinline__ void epilogue4(const GemmArgs& a, int m, int n0, float v[4]) {
  if (m >= a.M || n0 >= a.N) return;
  const int nv = min(4, a.N - n0);
  switch (MODE) {
    case EPI_STORE: {
      long row = a.row_group > 0 ? (long)(m / a.row_group) * a.row_group_stride + (long)(m % a.row_group) * a.ldo
                                 : (long)m * a.ldo;
      float r[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float x = v[j];
        if (j < nv) {
          if (a.bias) x += a.bias[n0 + j];
          if (a.tab) x += a.tab[(long)(m % a.tab_period) * a.ldtab + n0 + j];
        }
        r[j] = act_apply(x, a.act);
      }
      if (a.out_type == ET_BF16) {
        bf16* o = reinterpret_cast<bf16*>(a.out) + row + n0;
        if (nv == 4 && ((reinterpret_cast<uintptr_t>(o) & 7) == 0)) {
          bf16x4 w = {(bf16)r[0], (bf16)r[1], (bf16)r[2], (bf16)r[3]};
          *reinterpret_cast<bf16x4*>(o) = w;
        } else {
          for (int j = 0; j < nv; ++j) o[j] = (bf16)r[j];
        }
      } else {
        float* o = reinterpret_cast<float*>(a.out) + row + n0;
        if (nv == 4) {
          reinterpret_cast<f32x4u*>(o)->v = f32x4{r[0], r[1], r[2], r[3]};
        } else {
          for (int j = 0; j < nv; ++j) o[j] = r[j];
        }
        if (a.out2) {
          bf16* o2 = reinterpret_cast<bf16*>(a.out2) + (long)m * a.ldo2 + n0;
          for (int j = 0; j < nv; ++j) o2[j] = (bf16)r[j];
        }
      }
      break;
    }
    case EPI_RESID: {
      long row = a.row_group > 0 ? (long)(m / a.row_group) * a.row_group_stride + (long)(m % a.row_group) * a.ldo
                                 : (long)m * a.ldo;
      float* o = reinterpret_cast<float*>(a.out) + row + n0;
      for (int j = 0; j < nv; ++j) {
        o[j] = upd(o[j], v[j], a.bias ? a.bias[n0 + j] : 0.0f, a.gate ? a.gate[n0 + j] : 1.0f);
        if (a.out2) reinterpret_cast<bf16*>(a.out2)[(long)m * a.ldo2 + n0 + j] = (bf16)o[j];
      }
      break;
    }
    case EPI_GEGLU: {
      // weight rows interleaved: row 2f = gate f, row 2f + 1 = up f
      bf16* ob = reinterpret_cast<bf16*>(a.out);
      float* of = reinterpret_cast<float*>(a.out);
      const int f0 = n0 >> 1;
      for (int j = 0; j + 1 < nv; j += 2) {
        float g = v[j], u = v[j + 1];
        if (a.bias) { g += a.bias[n0 + j]; u += a.bias[n0 + j + 1]; }
        float r = act_apply(g, ACT_GELU) * u;
        long idx = (long)m * a.ldo + f0 + (j >> 1);
        if (a.out_type == ET_BF16) ob[idx] = (bf16)r; else of[idx] = r;
      }
      break;
    }
    case EPI_QKV: {
      const QkvEpi& q = a.qkv;
      const int c0 = q.n_off + n0;            // logical column (multiple of 4)
      const int hd = q.hd;
      const int b = m / q.seq, i = m % q.seq;
      int seg, head, j0;
      if (c0 < q.n_q * hd) { seg = 0; head = c0 / hd; j0 = c0 % hd; }
      else if (c0 < (q.n_q + q.n_kv) * hd) { seg = 1; head = (c0 - q.n_q * hd) / hd; j0 = (c0 - q.n_q * hd) % hd; }
      else { seg = 2; head = (c0 - (q.n_q + q.n_kv) * hd) / hd; j0 = (c0 - (q.n_q + q.n_kv) * hd) % hd; }
      float x[4];
      for (int j = 0; j < 4; ++j) x[j] = v[j] + ((a.bias && j < nv) ? a.bias[n0 + j] : 0.0f);
      void* dst; long idx;
      if (seg == 0) { dst = q.q; idx = (long)b * q.q_sb + (long)head * q.q_sh + (long)i * q.q_si; }
      else if (seg == 1) { dst = q.k; idx = (long)b * q.k_sb + (long)head * q.k_sh + (long)i * q.k_si; }
      else { dst = q.v; idx = (long)b * q.v_sb + (long)head * q.v_sh + (long)i * q.v_si; }
      if (seg < 2 && q.pos0 >= 0) {
        // weight rows of q and k are stored pair-interleaved per head:
        // row 2t holds dimension t and row 2t + 1 holds dimension t + hd/2,
        // so these four columns are dims (t, t+1) and (t+hd/2, t+1+hd/2)
        const int half = hd >> 1, pos = q.pos0 + i, t = j0 >> 1;
        const f32x4 cs = *reinterpret_cast<const f32x4*>(q.rope_cs + ((long)pos * half + t) * 2);  // c_t s_t c_t+1 s_t+1
        const float lo0 = x[0] * cs[0] - x[1] * cs[1], hi0 = x[1] * cs[0] + x[0] * cs[1];
        const float lo1 = x[2] * cs[2] - x[3] * cs[3], hi1 = x[3] * cs[2] + x[2] * cs[3];
        if (a.out_type == ET_BF16) {
          bf16* d = reinterpret_cast<bf16*>(dst) + idx;
          *reinterpret_cast<bf16x2*>(d + t) = bf16x2{(bf16)lo0, (bf16)lo1};
          *reinterpret_cast<bf16x2*>(d + t + half) = bf16x2{(bf16)hi0, (bf16)hi1};
        } else {
          float* d = reinterpret_cast<float*>(dst) + idx;
          d[t] = lo0; d[t + 1] = lo1; d[t + half] = hi0; d[t + half + 1] = hi1;
        }
      } else if (a.out_type == ET_BF16 && nv == 4) {
        *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(dst) + idx + j0) =
            bf16x4{(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
      } else {
        for (int j = 0; j < nv; ++j) store_elem(dst, idx + j0 + j, a.out_type, x[j]);
      }
      break;
    }
    case EPI_EULER: {
      float* o = reinterpret_cast<float*>(a.out) + (long)m * a.ldo + n0;
      for (int j = 0; j < nv; ++j) o[j] = upd(o[j], v[j], a.bias ? a.bias[n0 + j] : 0.0f, a.dt);
      break;
    }
  }
}

// ---------------------------------------------------------------- tile epilogue
// Epilogue of a whole output tile staged in LDS as fp32 (ROWS rows of BN
// columns, row stride LDC floats). Thread t finishes the four columns
// nc = (t % (BN/4)) * 4 of rows t / (BN/4) + it * (NT / (BN/4)). What depends
// only on the columns (bias, gate, QKV head and destination) is read or
// computed once per thread, and every load that depends on the row (the old
// residual or Euler state, the position table, the RoPE angles) is issued for
// all of the thread's rows before the first store, so the row loads share one
// memory round trip instead of one each. Arithmetic per element is that of
// epilogue4. Valid when a.epi_vec is set (N % 4 == 0 and every vector access
// aligned; see epi_vec_ok); otherwise callers use epilogue4.
// The epilogue of NIT rows ms[] (valid where ok[]) of the four columns
// n0..n0+3 (n0 < N), in two parts: load() reads everything that does not
// depend on the product (bias, gate, row table, old residual or Euler state,
// RoPE angles) and computes the destinations, finish() applies it to the
// sums t[] and stores. Kernels whose K loop is one memory round trip call
// load() ahead of it, so that the two round trips overlap.
__device__ __forceinline__ long out_row(const GemmArgs& a, int m) {
  return a.row_group > 0 ? (long)(m / a.row_group) * a.row_group_stride + (long)(m % a.row_group) * a.ldo
                         : (long)m * a.ldo;
}

template <int MODE, int NIT>
struct EpiRows {
  f32x4 bias, gate, aux[NIT];     // aux: row table, old value, or (cos, sin) of dims t and t + 1
  long off[NIT];
  void* dst;
  int half, tt, j0;
  bool rope;

  __device__ __forceinline__ void load(const GemmArgs& a, const int (&ms)[NIT], const bool (&ok)[NIT], int n0) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    bias = a.bias ? *reinterpret_cast<const f32x4*>(a.bias + n0) : zero;
    if constexpr (MODE == EPI_STORE) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        aux[it] = (a.tab && ok[it]) ? *reinterpret_cast<const f32x4*>(a.tab + (long)(ms[it] % a.tab_period) * a.ldtab + n0)
                                    : zero;
      }
    } else if constexpr (MODE == EPI_RESID || MODE == EPI_EULER) {
      const float* out = reinterpret_cast<const float*>(a.out);
      gate = (MODE == EPI_RESID && a.gate) ? *reinterpret_cast<const f32x4*>(a.gate + n0) : f32x4{1.f, 1.f, 1.f, 1.f};
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        off[it] = (MODE == EPI_RESID ? out_row(a, ms[it]) : (long)ms[it] * a.ldo) + n0;
        aux[it] = ok[it] ? *reinterpret_cast<const f32x4*>(out + off[it]) : zero;
      }
    } else if constexpr (MODE == EPI_GEGLU) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) off[it] = (long)ms[it] * a.ldo + (n0 >> 1);
    } else if constexpr (MODE == EPI_QKV) {
      const QkvEpi& q = a.qkv;
      const int c0 = q.n_off + n0, hd = q.hd;
      int seg, head;
      if (c0 < q.n_q * hd) { seg = 0; head = c0 / hd; j0 = c0 % hd; }
      else if (c0 < (q.n_q + q.n_kv) * hd) { seg = 1; head = (c0 - q.n_q * hd) / hd; j0 = (c0 - q.n_q * hd) % hd; }
      else { seg = 2; head = (c0 - (q.n_q + q.n_kv) * hd) / hd; j0 = (c0 - (q.n_q + q.n_kv) * hd) % hd; }
      dst = seg == 0 ? q.q : seg == 1 ? q.k : q.v;
      const long sb = seg == 0 ? q.q_sb : seg == 1 ? q.k_sb : q.v_sb;
      const long sh = seg == 0 ? q.q_sh : seg == 1 ? q.k_sh : q.v_sh;
      const long si = seg == 0 ? q.q_si : seg == 1 ? q.k_si : q.v_si;
      rope = seg < 2 && q.pos0 >= 0;
      half = hd >> 1; tt = j0 >> 1;
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int b = ms[it] / q.seq, i = ms[it] % q.seq;
        off[it] = (long)b * sb + (long)head * sh + (long)i * si;
        // (cos, sin) of dims t and t + 1 at position pos0 + i
        aux[it] = (rope && ok[it]) ? *reinterpret_cast<const f32x4*>(q.rope_cs + ((long)(q.pos0 + i) * half + tt) * 2) : zero;
      }
    }
  }

  __device__ __forceinline__ void finish(const GemmArgs& a, const f32x4 (&t)[NIT], const int (&ms)[NIT],
                                         const bool (&ok)[NIT], int n0) const {
    if constexpr (MODE == EPI_STORE) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        if (!ok[it]) continue;
        f32x4 x = t[it] + bias + aux[it];
        if (a.act != ACT_NONE) {
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = act_apply(x[j], a.act);
        }
        const long o = out_row(a, ms[it]) + n0;
        if (a.out_type == ET_BF16) {
          *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(a.out) + o) = bf16x4{(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
        } else {
          *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + o) = x;
          if (a.out2)
            *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(a.out2) + (long)ms[it] * a.ldo2 + n0) =
                bf16x4{(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
        }
      }
    } else if constexpr (MODE == EPI_RESID || MODE == EPI_EULER) {
      float* out = reinterpret_cast<float*>(a.out);
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        if (!ok[it]) continue;
        f32x4 r;
        if constexpr (MODE == EPI_RESID) r = upd(aux[it], t[it], bias, gate);
        else r = upd(aux[it], t[it], bias, f32x4{a.dt, a.dt, a.dt, a.dt});
        *reinterpret_cast<f32x4*>(out + off[it]) = r;
        if (MODE == EPI_RESID && a.out2)
          *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(a.out2) + (long)ms[it] * a.ldo2 + n0) =
              bf16x4{(bf16)r[0], (bf16)r[1], (bf16)r[2], (bf16)r[3]};
      }
    } else if constexpr (MODE == EPI_GEGLU) {
      // weight rows interleaved: column 2f = gate f, 2f + 1 = up f
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        if (!ok[it]) continue;
        const f32x4 x = t[it] + bias;
        const float r0v = act_apply(x[0], ACT_GELU) * x[1], r1v = act_apply(x[2], ACT_GELU) * x[3];
        if (a.out_type == ET_BF16)
          *reinterpret_cast<bf16x2*>(reinterpret_cast<bf16*>(a.out) + off[it]) = bf16x2{(bf16)r0v, (bf16)r1v};
        else {
          float* of = reinterpret_cast<float*>(a.out) + off[it];
          of[0] = r0v;
          of[1] = r1v;
        }
      }
    } else if constexpr (MODE == EPI_QKV) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        if (!ok[it]) continue;
        const f32x4 x = t[it] + bias;
        if (rope) {
          // columns are dims (t, t+1) and (t+hd/2, t+1+hd/2): weight rows of q and
          // k are stored pair-interleaved per head
          const f32x4 c = aux[it];
          const float lo0 = x[0] * c[0] - x[1] * c[1], hi0 = x[1] * c[0] + x[0] * c[1];
          const float lo1 = x[2] * c[2] - x[3] * c[3], hi1 = x[3] * c[2] + x[2] * c[3];
          if (a.out_type == ET_BF16) {
            bf16* d = reinterpret_cast<bf16*>(dst) + off[it];
            *reinterpret_cast<bf16x2*>(d + tt) = bf16x2{(bf16)lo0, (bf16)lo1};
            *reinterpret_cast<bf16x2*>(d + tt + half) = bf16x2{(bf16)hi0, (bf16)hi1};
          } else {
            float* d = reinterpret_cast<float*>(dst) + off[it];
            d[tt] = lo0; d[tt + 1] = lo1; d[tt + half] = hi0; d[tt + half + 1] = hi1;
          }
        } else if (a.out_type == ET_BF16) {
          *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(dst) + off[it] + j0) = bf16x4{(bf16)x[0], (bf16)x[1], (bf16)x[2], (bf16)x[3]};
        } else {
          *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(dst) + off[it] + j0) = x;
        }
      }
    }
  }
};

template <int MODE, int NIT>
__device__ __forceinline__ void epi_rows(const GemmArgs& a, const f32x4 (&t)[NIT], const int (&ms)[NIT],
                                         const bool (&ok)[NIT], int n0) {
  EpiRows<MODE, NIT> e;
  e.load(a, ms, ok, n0);
  e.finish(a, t, ms, ok, n0);
}

// The folded norm's row scale as a multiply of its own, never fused with the
// bias add that follows, so that every epilogue path (LDS tile, per-element,
// from registers) rounds alike.
__device__ __forceinline__ f32x4 row_scale(f32x4 t, float s) {
#pragma clang fp contract(off)
  return t * s;
}

// Thread tid of NT finishes the tile's rows r0 + it * RS of its four columns
// (see above), GRP rows per memory round trip (GRP bounds the registers the
// row loads hold); the tile is the sum of NSUM fp32 planes in LDS (plane
// stride ROWS * LDC floats), added in plane order, times rsc[row] when rsc
// (an LDS array of per-row scales) is given.
template <int MODE, int BN, int ROWS, int NT, int LDC, int NSUM = 1, int GRP = 8>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& a, const float* Cs, int m_blk, int n_blk, int tid,
                                              const float* rsc = nullptr) {
  // GeGLU has no row loads to overlap and its activation is long: two rows at
  // a time keep its registers within the kernels' budget
  constexpr int GR = MODE == EPI_GEGLU ? 2 : GRP;
  constexpr int CPT = BN / 4, RS = NT / CPT, NIT = (ROWS + RS - 1) / RS, G = NIT < GR ? NIT : GR;
  static_assert(NT % CPT == 0, "threads must cover whole rows");
  const int nc = (tid % CPT) * 4, r0 = tid / CPT, n0 = n_blk + nc;
  if (n0 >= a.N) return;
#pragma unroll
  for (int g0 = 0; g0 < NIT; g0 += G) {
    f32x4 t[G];
    int ms[G];
    bool ok[G];
#pragma unroll
    for (int it = 0; it < G; ++it) {
      const int mr = r0 + (g0 + it) * RS;
      ms[it] = m_blk + mr;
      ok[it] = g0 + it < NIT && (ROWS % RS == 0 || mr < ROWS) && ms[it] < a.M;
      t[it] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (ok[it]) {
        t[it] = *reinterpret_cast<const f32x4*>(Cs + mr * LDC + nc);
#pragma unroll
        for (int z = 1; z < NSUM; ++z) t[it] += *reinterpret_cast<const f32x4*>(Cs + z * ROWS * LDC + mr * LDC + nc);
        if (rsc) t[it] = row_scale(t[it], rsc[mr]);
      }
    }
    epi_rows<MODE, G>(a, t, ms, ok, n0);
  }
}

// Epilogue of the split-K partial pass: the fp32 tile (the sum of NSUM
// planes, in plane order) goes to the workspace slice of K range bz (the
// reduce kernel runs the epilogue).
template <int BN, int ROWS, int NT, int LDC, int NSUM = 1>
__device__ __forceinline__ void tile_store_partial(const GemmArgs& a, const float* Cs, int m_blk, int n_blk, int bz,
                                                   int tid) {
  constexpr int CPT = BN / 4, RS = NT / CPT, NIT = (ROWS + RS - 1) / RS;
  const int ldp = (a.N + 3) & ~3;
  float* part = a.ws + (long)bz * a.M * ldp;
  const int nc = (tid % CPT) * 4, r0 = tid / CPT, n = n_blk + nc;
  if (n >= a.N) return;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int mr = r0 + it * RS, m = m_blk + mr;
    if ((ROWS % RS == 0 || mr < ROWS) && m < a.M) {
      f32x4 t = *reinterpret_cast<const f32x4*>(Cs + mr * LDC + nc);
#pragma unroll
      for (int z = 1; z < NSUM; ++z) t += *reinterpret_cast<const f32x4*>(Cs + z * ROWS * LDC + mr * LDC + nc);
      *reinterpret_cast<f32x4*>(part + (long)m * ldp + n) = t;
    }
  }
}

// ---------------------------------------------------------------- epilogue from registers
// A wave's four fragments i = 0..3 along the weight rows: lane (lr, lq) of
// fragment (i, j) holds weight columns nb + 16 i + 4 lq .. + 3 of activation
// row mb + 16 j + lr (lr = lane % 16, lq = lane / 16). A 4 x 4 transpose of
// 32-bit words over the four 16-lane rows of the wave (two 32-lane and two
// 16-lane swaps) hands lane lq the words of fragment i = lq from all four
// lanes that share its row: 16 consecutive weight columns.
__device__ __forceinline__ void xpose4x4(unsigned (&p)[4]) {
  const auto s02 = __builtin_amdgcn_permlane32_swap(p[0], p[2], false, false);   // rows 0,1 <-> 2,3
  const auto s13 = __builtin_amdgcn_permlane32_swap(p[1], p[3], false, false);
  const auto s01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);   // rows 0 <-> 1, 2 <-> 3
  const auto s23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
  p[0] = s01[0]; p[1] = s01[1]; p[2] = s23[0]; p[3] = s23[1];
}

__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
  const bf16x2 h = bf16x2{(bf16)lo, (bf16)hi};
  return *reinterpret_cast<const unsigned*>(&h);
}

// The bias of the lane's four columns of each fragment (loaded ahead of the
// K loop where registers allow, so its latency is not paid at the end).
__device__ __forceinline__ void reg_bias(const GemmArgs& a, int nb, int lane, f32x4 (&bias)[4]) {
  const int lq = lane >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n0 = nb + 16 * i + 4 * lq;
    bias[i] = (a.bias && n0 < a.N) ? *reinterpret_cast<const f32x4*>(a.bias + n0) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// The GeGLU or plain bf16-store epilogue of such a wave tile, without the LDS
// round trip: GeGLU (a fragment holds two whole gate/up pairs) leaves one
// word per fragment and the lane stores 16 bytes (output columns nb / 2 +
// 8 lq ..); a store leaves two words per fragment (both halves transposed)
// and the lane stores 32 bytes (columns nb + 16 lq ..). reg_epi_ok states
// what the caller must hold (N % 16 == 0, so a group of 16 columns is wholly
// inside or outside; aligned rows; no row table, row groups or copy).
template <int MODE, int TM>
__device__ __forceinline__ void reg_epilogue(const GemmArgs& a, const f32x4 (&acc)[4][TM], const f32x4 (&bias)[4], int nb,
                                             int mb, int lane) {
  static_assert(MODE == EPI_GEGLU || MODE == EPI_STORE, "GeGLU or plain store");
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const int lr = lane & 15, lq = lane >> 4;
  const bool col_ok = nb + 16 * lq < a.N;
  bf16* out = reinterpret_cast<bf16*>(a.out) + (MODE == EPI_GEGLU ? (nb >> 1) + 8 * lq : nb + 16 * lq);
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = mb + 16 * j + lr;
    if constexpr (MODE == EPI_GEGLU) {
      unsigned p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 x = acc[i][j] + bias[i];
        p[i] = pack_bf16x2(act_apply(x[0], ACT_GELU) * x[1], act_apply(x[2], ACT_GELU) * x[3]);
      }
      xpose4x4(p);
      if (m < a.M && col_ok) *reinterpret_cast<u32x4*>(out + (long)m * a.ldo) = u32x4{p[0], p[1], p[2], p[3]};
    } else {
      unsigned lo[4], hi[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 x = acc[i][j] + bias[i];
        if (a.act != ACT_NONE) {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = act_apply(x[e], a.act);
        }
        lo[i] = pack_bf16x2(x[0], x[1]);
        hi[i] = pack_bf16x2(x[2], x[3]);
      }
      xpose4x4(lo);
      xpose4x4(hi);
      if (m < a.M && col_ok) {
        u32x4* o = reinterpret_cast<u32x4*>(out + (long)m * a.ldo);
        o[0] = u32x4{lo[0], hi[0], lo[1], hi[1]};
        o[1] = u32x4{lo[2], hi[2], lo[3], hi[3]};
      }
    }
  }
}

// The residual update x += gate * (D + bias) of a wave tile from the
// accumulators (no LDS pass): fragment (i, j) of lane (lr, lq) covers the
// four fp32 columns nb + 16 i + 4 lq .. + 3 of row mb + 16 j + lr, one
// 16-byte read and write each (a row's four lanes cover 64 contiguous
// bytes). The old values, bias and gate are read ahead of the K loop
// (reg_resid_load): the block alone reads and writes its tile, and the
// launcher checks that the product's input does not overlap the output.
__device__ __forceinline__ long resid_row(const GemmArgs& a, int m) {
  return a.row_group > 0 ? (long)(m / a.row_group) * a.row_group_stride + (long)(m % a.row_group) * a.ldo
                         : (long)m * a.ldo;
}

template <int TN, int TM>
__device__ __forceinline__ void reg_resid_load(const GemmArgs& a, int nb, int mb, int lane, f32x4 (&old)[TN][TM],
                                               f32x4 (&bias)[TN], f32x4 (&gate)[TN]) {
  const int lr = lane & 15, lq = lane >> 4;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f}, one = {1.f, 1.f, 1.f, 1.f};
  const float* out = reinterpret_cast<const float*>(a.out);
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    const int n0 = nb + 16 * i + 4 * lq;
    bias[i] = (a.bias && n0 < a.N) ? *reinterpret_cast<const f32x4*>(a.bias + n0) : zero;
    gate[i] = (a.gate && n0 < a.N) ? *reinterpret_cast<const f32x4*>(a.gate + n0) : one;
  }
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = mb + 16 * j + lr;
    const long ro = m < a.M ? resid_row(a, m) : 0;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int n0 = nb + 16 * i + 4 * lq;
      old[i][j] = (m < a.M && n0 < a.N) ? *reinterpret_cast<const f32x4*>(out + ro + n0) : zero;
    }
  }
}

template <int TN, int TM>
__device__ __forceinline__ void reg_resid(const GemmArgs& a, const f32x4 (&acc)[TN][TM], const f32x4 (&old)[TN][TM],
                                          const f32x4 (&bias)[TN], const f32x4 (&gate)[TN], int nb, int mb, int lane) {
  const int lr = lane & 15, lq = lane >> 4;
  float* out = reinterpret_cast<float*>(a.out);
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int m = mb + 16 * j + lr;
    if (m >= a.M) continue;
    const long ro = resid_row(a, m);
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int n0 = nb + 16 * i + 4 * lq;
      if (n0 >= a.N) continue;
      const f32x4 r = upd(old[i][j], acc[i][j], bias[i], gate[i]);
      *reinterpret_cast<f32x4*>(out + ro + n0) = r;
      if (a.out2)
        *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(a.out2) + (long)m * a.ldo2 + n0) =
            bf16x4{(bf16)r[0], (bf16)r[1], (bf16)r[2], (bf16)r[3]};
    }
  }
}
