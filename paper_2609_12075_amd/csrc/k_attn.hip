// Prefix-KV attention for both VLA stages on gfx950.
//
// One kernel serves every attention of the path: bidirectional prefill over
// the image+text prefix (grouped-query heads), the ViT's per-image attention,
// the action tokens' attention over [prefix K,V of the paired LLM layer ;
// their own K,V] (two key segments, no concatenation copy), and the DiT's
// self- and cross-attention. Keys/values stream through LDS in tiles of 64;
// softmax is online in fp32 (exp2 domain); both products run on the matrix
// cores (v_mfma_f32_16x16x32_bf16).
//
// Work decomposition: rows of a block are (query head within its KV group,
// query position) pairs, so all query heads sharing a KV head read each K/V
// tile once. Block = 4 waves x 16 rows. The score tile is computed
// transposed (S^T = K Q^T) so a lane holds four keys of one query; the
// probabilities then feed P V as the B operand without leaving registers,
// with the key order inside each 32-key chunk permuted consistently on the
// V side.
#include <algorithm>
#include <type_traits>

#include "common.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

namespace {

constexpr int BQ = 64;    // rows per block
constexpr int BKV = 64;   // keys per tile

__device__ __forceinline__ const bf16* seg_row(const AttnArgs& a, int which, int b, int g, int key, bool is_v) {
  const AttnSeg& s = a.seg[which];
  const bf16* base = reinterpret_cast<const bf16*>(is_v ? s.v : s.k);
  long off = is_v ? ((long)b * s.v_sb + (long)g * s.v_sh + (long)key * s.v_si)
                  : ((long)b * s.k_sb + (long)g * s.k_sh + (long)key * s.k_si);
  return base + off;
}

template <int HDP>
__global__ void __launch_bounds__(256) attn_mfma_kernel(AttnArgs a) {
  constexpr int LDK = HDP + 8;       // K tile row stride (elements)
  constexpr int LDV = BKV + 8;       // V^T tile row stride
  constexpr int NC = HDP / 32;       // 32-wide chunks of the head dimension
  constexpr int ND = HDP / 16;       // 16-wide output subtiles
  constexpr int CH = HDP / 8;        // 8-element chunks per key row
  __shared__ __attribute__((aligned(16))) bf16 Ks[BKV][LDK];
  __shared__ __attribute__((aligned(16))) bf16 Vt[HDP][LDV];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int S = a.splits > 1 ? a.splits : 1;      // key ranges (split-KV)
  // die-aware order: the row tiles sharing one (request, KV head) K/V stream
  // are consecutive logical blocks and so share one die's L2
  int bx, by, bz;
  xcd_remap(bx, by, bz);
  const int b = bz / S, split = bz % S, g = by;
  const int G = a.Hq / a.Hkv;
  const int rows = G * a.Lq;
  const int hd = a.hd;
  const int lq = lane & 15, grp = lane >> 4;

  // this lane's query row
  const int r = bx * BQ + wave * 16 + lq;
  const bool rvalid = r < rows;
  const int jh = rvalid ? r / a.Lq : 0, qi = rvalid ? r % a.Lq : 0;
  const int h = g * G + jh;

  bf16x8 qf[NC];
  {
    const bf16* qp = reinterpret_cast<const bf16*>(a.q) + (long)b * a.q_sb + (long)h * a.q_sh + (long)qi * a.q_si;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int d = c * 32 + grp * 8;
      qf[c] = (rvalid && d < hd) ? *reinterpret_cast<const bf16x8*>(qp + d) : bf16x8{};
    }
  }

  f32x4 o[ND];
#pragma unroll
  for (int t = 0; t < ND; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float sl2 = a.scale * 1.4426950408889634f;   // scale * log2(e)

  const int len0 = a.seg[0].len;
  const int kbeg = S > 1 ? split * a.kchunk : 0;
  const int kend = S > 1 ? min(len0 + a.seg[1].len, kbeg + a.kchunk) : len0 + a.seg[1].len;
  // K/V tile chunks (8 elements) handled by this thread; with PREFETCH the
  // next tile's chunks are loaded into registers while the current tile is
  // consumed, hiding the global-load latency behind the matrix work.
  constexpr int PER = BKV * CH / 256;
  constexpr bool PREFETCH = HDP <= 128;
  // Chunk j of this thread: key row kr, dims d8..d8+7. When the chunk count
  // divides by 4, a thread owns R = CH/4 consecutive keys of one 8-dim chunk,
  // so its V^T values for one dim are R consecutive bf16 (one vector store).
  constexpr bool GROUPED = CH % 4 == 0 && 256 % CH == 0;
  constexpr int R = GROUPED ? CH / 4 : 1;
  auto chunk_of = [&](int j, int& kr, int& d8) {
    if constexpr (GROUPED) {
      d8 = (tid % CH) * 8;
      kr = (tid / CH) * R + j;
    } else {
      const int c = tid + 256 * j;
      kr = c / CH;
      d8 = (c % CH) * 8;
    }
  };
  auto load_chunk = [&](int k0, int kr, int d8, bool is_v) {
    const int kg = k0 + kr;
    if (kg < kend && d8 < hd) {
      const int which = kg < len0 ? 0 : 1;
      const int key = which ? kg - len0 : kg;
      return *reinterpret_cast<const bf16x8*>(seg_row(a, which, b, g, key, is_v) + d8);
    }
    return bf16x8{};
  };
  // V^T store of this thread's PER chunks (R keys per dim when grouped)
  auto store_vt = [&](const bf16x8 (&vr)[PER]) {
    int kr, d8;
    if constexpr (GROUPED) {
      chunk_of(0, kr, d8);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (R == 1) {
          Vt[d8 + e][kr] = vr[0][e];
        } else if constexpr (R == 2) {
          typedef __attribute__((ext_vector_type(2))) __bf16 v2;
          *reinterpret_cast<v2*>(&Vt[d8 + e][kr]) = v2{vr[0][e], vr[1][e]};
        } else {
          static_assert(R == 8, "grouped staging supports 1, 2 or 8 keys per thread");
          *reinterpret_cast<bf16x8*>(&Vt[d8 + e][kr]) =
              bf16x8{vr[0][e], vr[1][e], vr[2][e], vr[3][e], vr[4][e], vr[5][e], vr[6][e], vr[7][e]};
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        chunk_of(j, kr, d8);
#pragma unroll
        for (int e = 0; e < 8; ++e) Vt[d8 + e][kr] = vr[j][e];
      }
    }
  };
  bf16x8 kreg[PER], vreg[PER];
  auto load_regs = [&](int k0) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      int kr, d8;
      chunk_of(j, kr, d8);
      kreg[j] = load_chunk(k0, kr, d8, false);
      vreg[j] = load_chunk(k0, kr, d8, true);
    }
  };
  if constexpr (PREFETCH) load_regs(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += BKV) {
    // ---- stage K (row-major) and V (transposed) tiles into LDS
    if constexpr (PREFETCH) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        int kr, d8;
        chunk_of(j, kr, d8);
        *reinterpret_cast<bf16x8*>(&Ks[kr][d8]) = kreg[j];
      }
      store_vt(vreg);
    } else {
      // K then V, PER chunks each in flight at once
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        int kr, d8;
        chunk_of(j, kr, d8);
        kreg[j] = load_chunk(k0, kr, d8, false);
      }
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        int kr, d8;
        chunk_of(j, kr, d8);
        *reinterpret_cast<bf16x8*>(&Ks[kr][d8]) = kreg[j];
      }
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        int kr, d8;
        chunk_of(j, kr, d8);
        vreg[j] = load_chunk(k0, kr, d8, true);
      }
      store_vt(vreg);
    }
    __syncthreads();
    if constexpr (PREFETCH) {
      if (k0 + BKV < kend) load_regs(k0 + BKV);
    }

    // ---- S^T = K Q^T for 4 subtiles of 16 keys
    f32x4 s[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      s[st] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Ks[st * 16 + lq][c * 32 + grp * 8]);
        s[st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[c], s[st], 0, 0, 0);
      }
    }
    // lane holds scores of query lq for keys st*16 + 4*grp + i
    float mx = -INFINITY;
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int kg = k0 + st * 16 + grp * 4 + i;
        float v = kg < kend ? s[st][i] * sl2 : -INFINITY;
        s[st][i] = v;
        mx = fmaxf(mx, v);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);
    const float alpha = exp2f(m_run - m_new);
    float psum = 0.f;
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float p = exp2f(s[st][i] - m_new);
        s[st][i] = p;
        psum += p;
      }
    psum += __shfl_xor(psum, 16);
    psum += __shfl_xor(psum, 32);
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int t = 0; t < ND; ++t) o[t] *= alpha;

    // ---- O^T += V^T P^T over two 32-key chunks. K-slot jj of lane group grp
    // is key 4*grp + jj (jj < 4) or 16 + 4*grp + jj - 4 (jj >= 4) of the chunk.
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      bf16x8 pf = {(bf16)s[2 * kc][0], (bf16)s[2 * kc][1], (bf16)s[2 * kc][2], (bf16)s[2 * kc][3],
                   (bf16)s[2 * kc + 1][0], (bf16)s[2 * kc + 1][1], (bf16)s[2 * kc + 1][2], (bf16)s[2 * kc + 1][3]};
#pragma unroll
      for (int t = 0; t < ND; ++t) {
        const bf16* vr = &Vt[t * 16 + lq][kc * 32 + grp * 4];
        bf16x4 lo = *reinterpret_cast<const bf16x4*>(vr);
        bf16x4 hi = *reinterpret_cast<const bf16x4*>(vr + 16);
        bf16x8 vf = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[t], 0, 0, 0);
      }
    }
    __syncthreads();
  }

  if (!rvalid) return;
  if (S > 1) {
    // split-KV: unnormalised output and (max, sum) of this key range, fp32
    const long row = ((long)b * a.Hq + h) * a.Lq + qi;
    float* po = a.ws + (row * S + split) * hd;
#pragma unroll
    for (int t = 0; t < ND; ++t) {
      const int d = t * 16 + grp * 4;
      if (d < hd) *reinterpret_cast<f32x4*>(po + d) = o[t];
    }
    if (grp == 0) {
      float* st = a.ws + (long)a.B * a.Hq * a.Lq * S * hd + (row * S + split) * 2;
      st[0] = m_run;
      st[1] = l_run;
    }
    return;
  }
  const float inv = 1.0f / l_run;
  bf16* op = reinterpret_cast<bf16*>(a.o) + (long)b * a.o_sb + (long)h * a.o_sh + (long)qi * a.o_si;
#pragma unroll
  for (int t = 0; t < ND; ++t) {
    const int d = t * 16 + grp * 4;
    if (d < hd) {
      bf16x4 w = {(bf16)(o[t][0] * inv), (bf16)(o[t][1] * inv), (bf16)(o[t][2] * inv), (bf16)(o[t][3] * inv)};
      *reinterpret_cast<bf16x4*>(op + d) = w;
    }
  }
}

// Split-KV merge: LPR lanes per query row (the fewest of 16, 32, 64 whose
// four dims each cover the head dim, so 64 / LPR rows share a wavefront)
// combine the key ranges in order: m = max m_s, l = sum l_s 2^(m_s - m),
// o = sum o_s 2^(m_s - m) / l. Each lane owns four consecutive dims; its
// range statistics and all (<= 16) partial loads are issued together before
// any is used (one memory round trip instead of two: 7.6 -> 6.4 us for the
// pi0-shaped action attention at batch 8, four ranges).
constexpr int MAX_SPLITS = 16;
template <int LPR>
__global__ void __launch_bounds__(256) attn_combine_kernel(AttnArgs a) {
  constexpr int RPW = 64 / LPR;
  const int lane = threadIdx.x & 63, sub = lane % LPR;
  const long row = (blockIdx.x * 4L + (threadIdx.x >> 6)) * RPW + lane / LPR;
  if (row >= (long)a.B * a.Hq * a.Lq) return;
  const int S = a.splits, hd = a.hd, d = sub * 4;
  const bool dok = d < hd;
  const float* st = a.ws + (long)a.B * a.Hq * a.Lq * S * hd + row * S * 2;
  const float* po = a.ws + row * S * hd + (dok ? d : 0);
  float ms[MAX_SPLITS], ls[MAX_SPLITS], w[MAX_SPLITS];
  f32x4 part[MAX_SPLITS];
#pragma unroll
  for (int q = 0; q < MAX_SPLITS; ++q) {
    ms[q] = q < S ? st[2 * q] : -INFINITY;
    ls[q] = q < S ? st[2 * q + 1] : 0.f;
    part[q] = (q < S && dok) ? *reinterpret_cast<const f32x4*>(po + (long)q * hd) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float m = -INFINITY;
#pragma unroll
  for (int q = 0; q < MAX_SPLITS; ++q) m = fmaxf(m, ms[q]);
  float l = 0.f;
#pragma unroll
  for (int q = 0; q < MAX_SPLITS; ++q) {
    w[q] = q < S ? exp2f(ms[q] - m) : 0.f;
    l += q < S ? ls[q] * w[q] : 0.f;
  }
  const float inv = 1.0f / l;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < MAX_SPLITS; ++q) acc += part[q] * w[q];
  if (!dok) return;
  const int qi = (int)(row % a.Lq), h = (int)((row / a.Lq) % a.Hq), b = (int)(row / ((long)a.Lq * a.Hq));
  bf16* op = reinterpret_cast<bf16*>(a.o) + (long)b * a.o_sb + (long)h * a.o_sh + (long)qi * a.o_si;
  *reinterpret_cast<bf16x4*>(op + d) =
      bf16x4{(bf16)(acc[0] * inv), (bf16)(acc[1] * inv), (bf16)(acc[2] * inv), (bf16)(acc[3] * inv)};
}

// fp32 attention: the same row decomposition (query head within its KV group,
// query position) in tiles of 16 rows, both products on the fp32 matrix
// instructions, operands straight from global memory into registers. A
// block's NW waves split the keys (16 keys at a time, tile t to wave t % NW)
// and merge their (max, sum, output) through LDS in wave order. The score
// tile is computed transposed (S^T = K Q^T), so a lane holds four keys of one
// query, and those are the P operand of the second product as they are. What
// bounds it is latency: a wave of the small model's attention (90-180 keys)
// has one or two key tiles, whose loads are all issued before the first use.
template <int HDP>
__global__ void __launch_bounds__(512) attn_f32_kernel(AttnArgs a) {
  constexpr int NW = 8, NC = HDP / 16;               // 16-wide chunks of the head dimension
  // values requested after the scores: keys and values at once spilled 78
  // registers a lane (8 heads of 256, 50 tokens, 866 keys, batch 2 84.5 -> 66.6
  // us; 300 tokens and keys 79 -> 59; 31 rows of 136, one key 13.6 -> 9.9)
  constexpr bool LATE = HDP > 128;
  constexpr int REC = HDP / 4 + 4;                   // merge record of a lane: output, max, sum, pad
  __shared__ __attribute__((aligned(16))) float mg[NW / 2][64 * REC];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int g = blockIdx.y, b = blockIdx.z, G = a.Hq / a.Hkv, hd = a.hd;
  const int r = blockIdx.x * 16 + lr;
  const bool rvalid = r < G * a.Lq;
  const int jh = rvalid ? r / a.Lq : 0, qi = rvalid ? r % a.Lq : 0, h = g * G + jh;
  const float* qp = reinterpret_cast<const float*>(a.q) + (long)b * a.q_sb + (long)h * a.q_sh + (long)qi * a.q_si;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 qf[NC], o[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int d = c * 16 + lk * 4;
    qf[c] = d < hd ? *reinterpret_cast<const f32x4*>(qp + d) : zero;
    o[c] = zero;
  }
  const int len0 = a.seg[0].len, total = len0 + a.seg[1].len, nt = (total + 15) / 16;
  float m_run = -INFINITY, l_run = 0.f;
  auto row = [&](int key, bool is_v) -> const float* {
    const int which = key < len0 ? 0 : 1, kk = which ? key - len0 : key;
    const AttnSeg& s = a.seg[which];
    return is_v ? reinterpret_cast<const float*>(s.v) + (long)b * s.v_sb + (long)g * s.v_sh + (long)kk * s.v_si
                : reinterpret_cast<const float*>(s.k) + (long)b * s.k_sb + (long)g * s.k_sh + (long)kk * s.k_si;
  };
  for (int t = wave; t < nt; t += NW) {
    // keys past the end read the last key's rows; their scores become -inf and
    // their values zeros
    const float* kp = row(min(t * 16 + lr, total - 1), false);
    f32x4 kf[NC], vf[NC];                            // vf[c][e]: V[key 4 lk + e][16 c + lr]
#pragma unroll
    for (int c = 0; c < NC; ++c) kf[c] = c * 16 + lk * 4 < hd ? *reinterpret_cast<const f32x4*>(kp + c * 16 + lk * 4) : zero;
    auto load_v = [&]() {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* vp = row(min(t * 16 + lk * 4 + e, total - 1), true);
#pragma unroll
        for (int c = 0; c < NC; ++c) vf[c][e] = c * 16 + lr < hd ? vp[c * 16 + lr] : 0.f;
      }
    };
    // values past the end: probability 0 times an infinity would be a NaN
    auto clear_v = [&]() {
      if (t * 16 + 16 > total) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < NC; ++c)
            if (t * 16 + lk * 4 + e >= total) vf[c][e] = 0.f;
      }
    };
    if constexpr (!LATE) load_v();
    if constexpr (HDP == 128) clear_v();     // (350 keys 18.7 us here, 19.3 below; at 64 it is the other way round)
    f32x4 sc = zero;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[c][e], sc, 0, 0, 0);
    if constexpr (LATE) load_v();
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[e] = t * 16 + lk * 4 + e < total ? sc[e] * a.scale : -INFINITY;
      mx = fmaxf(mx, sc[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx), alpha = __expf(m_run - m_new);
    float ps = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[e] = __expf(sc[e] - m_new);
      ps += sc[e];
    }
    ps += __shfl_xor(ps, 16);
    ps += __shfl_xor(ps, 32);
    l_run = l_run * alpha + ps;
    m_run = m_new;
    if constexpr (HDP != 128) clear_v();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      o[c] *= alpha;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][e], sc[e], o[c], 0, 0, 0);
    }
  }
  // merge the waves, the upper half into the lower until wave 0 holds all (a
  // wave without keys has max -inf and sum 0, and weighs nothing)
  for (int n = NW / 2; n > 0; n /= 2) {
    if (wave >= n && wave < 2 * n) {
      float* dst = mg[wave - n] + lane * REC;
#pragma unroll
      for (int c = 0; c < NC; ++c) *reinterpret_cast<f32x4*>(dst + 4 * c) = o[c];
      dst[HDP / 4] = m_run;
      dst[HDP / 4 + 1] = l_run;
    }
    __syncthreads();
    if (wave < n) {
      const float* src = mg[wave] + lane * REC;
      const float m2 = src[HDP / 4], l2 = src[HDP / 4 + 1], m = fmaxf(m_run, m2);
      const float w1 = m_run == m ? 1.f : __expf(m_run - m), w2 = m2 == m ? 1.f : __expf(m2 - m);
#pragma unroll
      for (int c = 0; c < NC; ++c) o[c] = o[c] * w1 + *reinterpret_cast<const f32x4*>(src + 4 * c) * w2;
      l_run = l_run * w1 + l2 * w2;
      m_run = m;
    }
    __syncthreads();
  }
  if (wave != 0 || !rvalid) return;
  float* op = reinterpret_cast<float*>(a.o) + (long)b * a.o_sb + (long)h * a.o_sh + (long)qi * a.o_si;
  const float inv = 1.0f / l_run;
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c * 16 + lk * 4 < hd) *reinterpret_cast<f32x4*>(op + c * 16 + lk * 4) = o[c] * inv;
}


// ---------------------------------------------------------------- v2 kernel
// Same row decomposition, softmax and products as attn_mfma_kernel, with the
// K/V staging of the multi-stage projection kernel: tiles move global -> LDS
// with the CDNA4 direct loads (global_load_lds_dwordx4, lane l's 16 bytes at
// LDS base + 16 l) through a ring of NS tiles, so the next round of tiles
// loads while this one is consumed, without registers. Rows are unpadded and
// key-major for both K and V; the 16-byte chunk c of row r sits in slot
// c ^ swz(r), which makes the 16-row fragment reads conflict-free. The P V
// product needs V^T fragments (one dimension, 8 keys per lane); they come
// from the transposing LDS read (ds_read_b64_tr_b16): within each 16-lane
// group, source lane s points at 4 dimensions of one key row (row
// 4-block + s / 4, dims 4 (s % 4) ..), and lane i receives dimension i of the
// group's 4 keys. Chunks past hd and keys past the range read zeros.
//
// KS > 1 splits the block's key range over KS groups of 4 waves (tile t goes
// to group t % KS), so short decode ranges run KS tiles at a time with KS
// waves per SIMD; the groups' (max, sum, output) are merged through LDS at
// the end in group order (as the split-KV combine does across blocks).
typedef short v4s __attribute__((ext_vector_type(4)));

// A row statistic combined with the value of lane l ^ 16 (l ^ 32): one CDNA4
// permlane swap of a value with itself exchanges the 16-lane rows (32-lane
// halves), and its two results hold the lane's own value and its partner's.
// The maximum that passes a NaN on (a row with a NaN score is NaN in either
// case): gfx950 has it as one instruction of two or three operands, where
// fmaxf first has to quiet each operand by an instruction of its own.
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float max_x16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return vmax(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_x32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return vmax(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int N>
__device__ __forceinline__ float max_of(const f32x4 (&s)[N]) {
  float m = s[0][0];
#pragma unroll
  for (int i = 1; i < 4 * N; i += 2) m = i + 1 < 4 * N ? vmax(vmax(m, s[i / 4][i % 4]), s[(i + 1) / 4][(i + 1) % 4]) : vmax(m, s[i / 4][i % 4]);
  return m;
}
__device__ __forceinline__ float sum_x16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_x32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int HDP>
struct V2 {
  static constexpr int BKV = HDP >= 256 ? 32 : 64;          // keys per tile
  static constexpr int CR = HDP / 8;                          // 16-byte chunks per row
  static constexpr int ROWB = HDP * 2;
  static constexpr int TILE = BKV * ROWB;                     // bytes of a K (or V) tile
  // ring depth in tiles (KS = 1). Two tiles of 16 KiB at head dim 64: four
  // blocks a CU instead of the two that a ring of four leaves; the tile loop
  // is a chain of LDS reads, exponentials and products, which more waves hide
  // better than deeper loads (12 heads, 1024 keys: 9 images 84.7 -> 68.7 us,
  // 3 images 39.8 -> 33.9; 15 heads, 240 keys, batch 16 18.7 -> 16.5)
  static constexpr int NS = 2 * TILE <= 8192 ? 4 : 2;
  static constexpr int RP = CR >= 16 ? 1 : 16 / CR;           // rows per 256 bytes (one bank cycle)
  static constexpr int SWM = (CR >= 16 ? 16 : CR) - 1;
  __device__ static constexpr int swz(int r) { return (r / RP) & SWM; }
};

// (two waves a SIMD at least: with the register file of one the compiler
// keeps the products' results in the accumulation registers and copies them)
// HDU: the head dims (of HDP in a row) whose fragments are read and multiplied;
// a head dim of 72 in rows of 128 skips the subtiles past 80 (24 images, 256
// keys, 16 heads 30.6 -> 27.6 us).
template <int HDP, int KS, int HDU = HDP>
__global__ void __launch_bounds__(256 * KS, 2) attn_v2_kernel(AttnArgs a) {
  using C = V2<HDP>;
  constexpr int BKV = C::BKV, ROWB = C::ROWB, TILE = C::TILE, CR = C::CR;
  constexpr int NW = 4 * KS;                       // waves per block
  constexpr int IW = TILE / 1024 / NW;             // 1 KiB direct loads per wave per tile (K or V)
  static_assert(IW >= 1 && IW * NW * 1024 == TILE, "tile loads must spread evenly over the waves");
  constexpr int NR = KS == 1 ? C::NS : 2;          // ring depth in rounds of KS tiles
  constexpr int NC = (HDU + 31) / 32, ND = HDU / 16;
  static_assert(HDU % 16 == 0 && HDU <= HDP, "whole subtiles");
  constexpr int RING = NR * KS * 2 * TILE;
  constexpr int MST = ND * 4 + 4;                   // merge record: o, m, l, pad (16-byte aligned)
  constexpr int MERGE = KS > 1 ? (KS - 1) * 256 * MST * 4 : 0;
  __shared__ __attribute__((aligned(1024))) char smem[RING > MERGE ? RING : MERGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave >> 2, wrow = wave & 3;       // key group, row group
  const int S = a.splits > 1 ? a.splits : 1;
  int bx, by, bz;
  xcd_remap(bx, by, bz);
  const int b = bz / S, split = bz % S, g = by;
  const int G = a.Hq / a.Hkv;
  const int rows = G * a.Lq;
  const int hd = a.hd;
  const int lq = lane & 15, grp = lane >> 4;

  const int r = bx * BQ + wrow * 16 + lq;
  const bool rvalid = r < rows;
  const int jh = rvalid ? r / a.Lq : 0, qi = rvalid ? r % a.Lq : 0;
  const int h = g * G + jh;

  bf16x8 qf[NC];
  {
    const bf16* qp = reinterpret_cast<const bf16*>(a.q) + (long)b * a.q_sb + (long)h * a.q_sh + (long)qi * a.q_si;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int d = c * 32 + grp * 8;
      qf[c] = (rvalid && d < hd) ? *reinterpret_cast<const bf16x8*>(qp + d) : bf16x8{};
    }
  }

  const int len0 = a.seg[0].len;
  const int kbeg = S > 1 ? split * a.kchunk : 0;
  const int kend = S > 1 ? min(len0 + a.seg[1].len, kbeg + a.kchunk) : len0 + a.seg[1].len;
  const int nt = kend > kbeg ? (kend - kbeg + BKV - 1) / BKV : 0;
  const int nrounds = (nt + KS - 1) / KS;
  const bf16* Z = reinterpret_cast<const bf16*>(a.zeros);

  // Loop-invariant addressing: the (request, KV head) base of each segment's
  // K and V rows in bytes and, per lane and load, the byte offset of its row
  // and chunk; per tile only the segment bases move (scalar work) and each
  // lane picks its row's segment.
  const long kbase0 = (long)a.seg[0].k + ((long)b * a.seg[0].k_sb + (long)g * a.seg[0].k_sh) * 2;
  const long kbase1 = (long)a.seg[1].k + ((long)b * a.seg[1].k_sb + (long)g * a.seg[1].k_sh) * 2;
  const long vbase0 = (long)a.seg[0].v + ((long)b * a.seg[0].v_sb + (long)g * a.seg[0].v_sh) * 2;
  const long vbase1 = (long)a.seg[1].v + ((long)b * a.seg[1].v_sb + (long)g * a.seg[1].v_sh) * 2;
  const long kst0 = a.seg[0].k_si * 2, kst1 = a.seg[1].k_si * 2, vst0 = a.seg[0].v_si * 2, vst1 = a.seg[1].v_si * 2;
  // (head dim 256 with one key group keeps the per-tile computation: the
  // hoisted offsets would cost it half its occupancy)
  constexpr bool HOIST = !(HDP >= 256 && KS == 1);
  constexpr int IWH = HOIST ? IW : 1;
  int lrow[IWH], lok[IWH];
  unsigned rk0[IWH], rk1[IWH], rv0[IWH], rv1[IWH];  // < 2^32 (checked by the launcher)
#pragma unroll
  for (int i = 0; i < IWH; ++i) {
    const int u = (i * NW + wave) * 64 + lane, row = u / CR, c = (u % CR) ^ C::swz(row), d8 = c * 8;
    lrow[i] = row;
    lok[i] = d8 < hd;
    rk0[i] = (unsigned)(row * kst0 + d8 * 2); rk1[i] = (unsigned)(row * kst1 + d8 * 2);
    rv0[i] = (unsigned)(row * vst0 + d8 * 2); rv1[i] = (unsigned)(row * vst1 + d8 * 2);
  }

  // round p holds tiles p KS .. p KS + KS - 1 in ring slot p % NR; each tile
  // is its K tile then its V tile. 16-byte unit u of a tile is (row u / CR,
  // slot u % CR); wave w loads units [(i NW + w) 64, + 64) for i < IW.
  auto issue = [&](int p) {
    char* base = smem + (p % NR) * KS * 2 * TILE;
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const int t = p * KS + q;
      char* kt = base + q * 2 * TILE;
      const int k0 = kbeg + t * BKV;
      // row k0 + r of segment 1 is its row k0 - len0 + r (used only for rows >= len0)
      const long tk0 = kbase0 + k0 * kst0, tk1 = kbase1 + (long)(k0 - len0) * kst1;
      const long tv0 = vbase0 + k0 * vst0, tv1 = vbase1 + (long)(k0 - len0) * vst1;
#pragma unroll
      for (int i = 0; i < IW; ++i) {
        const bf16 *ks = Z, *vs = Z;
        if constexpr (HOIST) {
          const int kk = k0 + lrow[i];
          if (t < nt && kk < kend && lok[i]) {
            const bool s1 = kk >= len0;
            ks = reinterpret_cast<const bf16*>(s1 ? tk1 + rk1[i] : tk0 + rk0[i]);
            vs = reinterpret_cast<const bf16*>(s1 ? tv1 + rv1[i] : tv0 + rv0[i]);
          }
        } else {
          const int u = (i * NW + wave) * 64 + lane, row = u / CR, c = (u % CR) ^ C::swz(row), d8 = c * 8;
          const int kk = k0 + row;
          if (t < nt && kk < kend && d8 < hd) {
            const int which = kk < len0 ? 0 : 1;
            const int key = which ? kk - len0 : kk;
            ks = seg_row(a, which, b, g, key, false) + d8;
            vs = seg_row(a, which, b, g, key, true) + d8;
          }
        }
        __builtin_amdgcn_global_load_lds(ks, kt + (i * NW + wave) * 1024, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(vs, kt + TILE + (i * NW + wave) * 1024, 16, 0, 0);
      }
    }
  };

  f32x4 o[ND];
#pragma unroll
  for (int u = 0; u < ND; ++u) o[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const float sl2 = a.scale * 1.4426950408889634f;   // scale * log2(e)
  constexpr int PER_ROUND = KS * 2 * IW;             // direct loads per wave per round

#pragma unroll
  for (int p = 0; p < NR - 1; ++p)
    if (p < nrounds) issue(p);
  for (int p = 0; p < nrounds; ++p) {
    // round p has landed once at most the NR - 2 later rounds' loads are
    // pending; the barrier (no fence) then also guarantees every wave is done
    // with round p - 1, whose slot the next issue overwrites
    if (p + NR - 2 < nrounds) {
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"((NR - 2) * PER_ROUND) : "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    if (p + NR - 1 < nrounds) issue(p + NR - 1);
    const int t = p * KS + kg;
    if (t >= nt) continue;
    const char* Kt = smem + (p % NR) * KS * 2 * TILE + kg * 2 * TILE;
    const char* Vt = Kt + TILE;
    const int k0 = kbeg + t * BKV;

    // ---- S^T = K Q^T over BKV / 16 subtiles of 16 keys
    constexpr int NST = BKV / 16;
    f32x4 sc[NST];
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      sc[st] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int row = st * 16 + lq;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int cc = c * 4 + grp;
        bf16x8 kf = *reinterpret_cast<const bf16x8*>(Kt + row * ROWB + ((cc ^ C::swz(row)) << 4));
        sc[st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[c], sc[st], 0, 0, 0);
      }
    }
    // keys past the range exist only in a range's last tile (a block-uniform
    // test): they get score -inf. The running max is kept in log2 units
    // (scores times scale log2 e, positive), so each probability is one fused
    // multiply-add and the hardware exp2, whose argument is <= 0 or -inf.
    if (k0 + BKV > kend) {
#pragma unroll
      for (int st = 0; st < NST; ++st)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k0 + st * 16 + grp * 4 + i >= kend) sc[st][i] = -INFINITY;
    }
    const float m_new = vmax(m_run, max_x32(max_x16(max_of(sc))) * sl2);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[st][i], sl2, -m_new));
        sc[st][i] = pv;
        ps[i] += pv;
      }
    // (this lane's keys; the lanes of a row are added after the last tile)
    l_run = l_run * alpha + ((ps[0] + ps[1]) + (ps[2] + ps[3]));
    m_run = m_new;
#pragma unroll
    for (int u = 0; u < ND; ++u) o[u] *= alpha;

    // ---- O^T += V^T P^T per 32-key chunk; K-slot jj of lane group grp is key
    // 4 grp + jj (jj < 4) or 16 + 4 grp + jj - 4 (jj >= 4) of the chunk
    const int s4 = lane & 15;
#pragma unroll
    for (int kc = 0; kc < BKV / 32; ++kc) {
      bf16x8 pf = {(bf16)sc[2 * kc][0], (bf16)sc[2 * kc][1], (bf16)sc[2 * kc][2], (bf16)sc[2 * kc][3],
                   (bf16)sc[2 * kc + 1][0], (bf16)sc[2 * kc + 1][1], (bf16)sc[2 * kc + 1][2], (bf16)sc[2 * kc + 1][3]};
      const int r_lo = kc * 32 + 4 * grp + (s4 >> 2), r_hi = r_lo + 16;
#pragma unroll
      for (int u = 0; u < ND; ++u) {
        const int cc = 2 * u + ((s4 & 3) >> 1), off = (s4 & 1) << 3;
        const char* plo = Vt + r_lo * ROWB + ((cc ^ C::swz(r_lo)) << 4) + off;
        const char* phi = Vt + r_hi * ROWB + ((cc ^ C::swz(r_hi)) << 4) + off;
        const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(plo));
        const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(phi));
        const bf16x4 l4 = __builtin_bit_cast(bf16x4, lo), h4 = __builtin_bit_cast(bf16x4, hi);
        const bf16x8 vf = {l4[0], l4[1], l4[2], l4[3], h4[0], h4[1], h4[2], h4[3]};
        o[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, o[u], 0, 0, 0);
      }
    }
  }

  l_run = sum_x32(sum_x16(l_run));

  if constexpr (KS > 1) {
    // merge the key groups into group 0, in group order: m = max m_q,
    // l = sum l_q 2^(m_q - m), o = sum o_q 2^(m_q - m)
    __syncthreads();                               // the ring is free from here on
    float* mg = reinterpret_cast<float*>(smem);
    const int slot = wrow * 64 + lane;             // lane of a row group
    if (kg > 0) {
      float* dst = mg + ((kg - 1) * 256 + slot) * MST;
#pragma unroll
      for (int u = 0; u < ND; ++u) *reinterpret_cast<f32x4*>(dst + 4 * u) = o[u];
      dst[ND * 4] = m_run;
      dst[ND * 4 + 1] = l_run;
    }
    __syncthreads();
    if (kg > 0) return;
    float mq[KS], lq_[KS];
    mq[0] = m_run; lq_[0] = l_run;
#pragma unroll
    for (int q = 1; q < KS; ++q) {
      const float* src = mg + ((q - 1) * 256 + slot) * MST;
      mq[q] = src[ND * 4]; lq_[q] = src[ND * 4 + 1];
    }
    float m = mq[0];
#pragma unroll
    for (int q = 1; q < KS; ++q) m = fmaxf(m, mq[q]);
    float l = 0.f, w[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      w[q] = __builtin_amdgcn_exp2f(mq[q] - m);
      l += lq_[q] * w[q];
    }
#pragma unroll
    for (int u = 0; u < ND; ++u) {
      f32x4 acc = o[u] * w[0];
#pragma unroll
      for (int q = 1; q < KS; ++q)
        acc += *reinterpret_cast<const f32x4*>(mg + ((q - 1) * 256 + slot) * MST + 4 * u) * w[q];
      o[u] = acc;
    }
    m_run = m;
    l_run = l;
  }

  if (!rvalid) return;
  if (S > 1) {
    const long row = ((long)b * a.Hq + h) * a.Lq + qi;
    float* po = a.ws + (row * S + split) * hd;
#pragma unroll
    for (int u = 0; u < ND; ++u) {
      const int d = u * 16 + grp * 4;
      if (d < hd) *reinterpret_cast<f32x4*>(po + d) = o[u];
    }
    if (grp == 0) {
      float* st = a.ws + (long)a.B * a.Hq * a.Lq * S * hd + (row * S + split) * 2;
      st[0] = m_run;
      st[1] = l_run;
    }
    return;
  }
  const float inv = 1.0f / l_run;
  bf16* op = reinterpret_cast<bf16*>(a.o) + (long)b * a.o_sb + (long)h * a.o_sh + (long)qi * a.o_si;
#pragma unroll
  for (int u = 0; u < ND; ++u) {
    const int d = u * 16 + grp * 4;
    if (d < hd) {
      bf16x4 wv = {(bf16)(o[u][0] * inv), (bf16)(o[u][1] * inv), (bf16)(o[u][2] * inv), (bf16)(o[u][3] * inv)};
      *reinterpret_cast<bf16x4*>(op + d) = wv;
    }
  }
}

// ---------------------------------------------------------------- waves split the keys
// The same attention where the row tiles are few (the action stage, prefills
// of one request): a block owns 16 rows and VD dims of the output, each of
// its NW waves takes every NW-th tile of KT keys, and the waves' (max, sum,
// output) are merged in LDS in wave order. A wave moves its tiles global ->
// LDS with the direct loads into a K and a V slot of its own and waits for
// its own loads only, so there is no barrier between the queries' and the
// merge's, and each slot is loaded again as soon as its fragments are in
// registers. VD < HDP: the blocks of a row tile share its output dims, each
// forms all scores and reads its dims of V only (a block is bound by the
// ~54 bytes a clock that a CU loads, so four blocks a row tile, K whole and a
// quarter of V each, take 62 % of the time of one).
// These launches take a few microseconds, of which instruction fetch is a
// part (the code is cold in each): ragged tiles are loaded by a rolled loop,
// and block and row indices come from multiplications with host-made
// reciprocals.
// V^T fragments of NU consecutive 16-dim subtiles of one 32-key chunk: rows
// 4 grp + .. and 16 rows further, whose swizzle is the same, so the two reads
// of a subtile differ by an immediate offset only. Written out with their
// wait, because the compiler puts a wait for ALL pending global loads, the
// direct loads of the next keys among them, before each use of the builtin.
// (attn_v2_kernel keeps the builtin: its loads have landed by then, and with
// waits of its own its matrix instructions overlap the reads less, 120 -> 131
// us for the pi0-shaped prefill at batch 8.)
template <int NU, int OFF, int HI>
__device__ __forceinline__ void read_vt(bf16x8* vf, const unsigned* ad) {
  static_assert(NU == 2 || NU == 4, "two or four subtiles");
  bf16x4 l[4], h[4];
  if constexpr (NU == 4) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%12\n\tds_read_b64_tr_b16 %1, %8 offset:%13\n\t"
        "ds_read_b64_tr_b16 %2, %9 offset:%12\n\tds_read_b64_tr_b16 %3, %9 offset:%13\n\t"
        "ds_read_b64_tr_b16 %4, %10 offset:%12\n\tds_read_b64_tr_b16 %5, %10 offset:%13\n\t"
        "ds_read_b64_tr_b16 %6, %11 offset:%12\n\tds_read_b64_tr_b16 %7, %11 offset:%13\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(l[0]), "=&v"(h[0]), "=&v"(l[1]), "=&v"(h[1]), "=&v"(l[2]), "=&v"(h[2]), "=&v"(l[3]), "=&v"(h[3])
        : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3]), "n"(OFF), "n"(OFF + HI)
        : "memory");
  } else {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %4 offset:%6\n\tds_read_b64_tr_b16 %1, %4 offset:%7\n\t"
        "ds_read_b64_tr_b16 %2, %5 offset:%6\n\tds_read_b64_tr_b16 %3, %5 offset:%7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(l[0]), "=&v"(h[0]), "=&v"(l[1]), "=&v"(h[1])
        : "v"(ad[0]), "v"(ad[1]), "n"(OFF), "n"(OFF + HI)
        : "memory");
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) vf[u] = __builtin_shufflevector(l[u], h[u], 0, 1, 2, 3, 4, 5, 6, 7);
}

// The same of a 16-key tile: one read a subtile, four subtiles.
template <int NU, int OFF>
__device__ __forceinline__ void read_vt16(bf16x4* vf, const unsigned* ad) {
  static_assert(NU == 4, "four subtiles");
  bf16x4 l[4];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4 offset:%8\n\tds_read_b64_tr_b16 %1, %5 offset:%8\n\t"
      "ds_read_b64_tr_b16 %2, %6 offset:%8\n\tds_read_b64_tr_b16 %3, %7 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(l[0]), "=&v"(l[1]), "=&v"(l[2]), "=&v"(l[3])
      : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3]), "n"(OFF)
      : "memory");
#pragma unroll
  for (int u = 0; u < 4; ++u) vf[u] = l[u];
}

// The lane's byte offsets within a V tile for read_vt: subtile u reads from
// of[u % 8] + (u / 8) 256 (the swizzle touches the low 16 chunks of a row).
template <int HDP>
__device__ __forceinline__ void vt_offsets(unsigned* of) {
  using C = V2<HDP>;
  const int lane = threadIdx.x & 63, lq = lane & 15, r = 4 * (lane >> 4) + (lq >> 2);
#pragma unroll
  for (int u = 0; u < (HDP / 16 < 8 ? HDP / 16 : 8); ++u)
    of[u] = r * C::ROWB + (((2 * u + ((lq & 3) >> 1)) ^ C::swz(r)) << 4) + ((lq & 1) << 3);
}

// o += V^T P^T over the 32 or 16 keys of two fragments
__device__ __forceinline__ f32x4 pv_mma(bf16x8 v, bf16x8 p, f32x4 o) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, p, o, 0, 0, 0);
}
__device__ __forceinline__ f32x4 pv_mma(bf16x4 v, bf16x4 p, f32x4 o) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4s, v), __builtin_bit_cast(v4s, p), o, 0, 0, 0);
}

__device__ __forceinline__ unsigned lds_addr(const char* p) {
  return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) char*)(p);
}

__device__ __forceinline__ unsigned fast_div(unsigned n, unsigned mul) { return mul ? __umulhi(n, mul) : n; }

// Rows [0, n) of a tile of KT rows of HDP elements (row stride st bytes from
// base) into LDS at dst; rows from n on and 16-byte chunks from byte `end` of
// a row on are read from the zero buffer.
template <int HDP, int KT>
__device__ __forceinline__ void issue_tile(const char* base, long st, int n, int end, const char* Z, char* dst) {
  using C = V2<HDP>;
  constexpr int L = KT * C::ROWB / 1024, RPL = 64 / C::CR;   // direct loads, rows per load
  const int lane = threadIdx.x & 63, lrow = lane / C::CR;
  const unsigned lof = (unsigned)(lrow * st);
  const long step = RPL * st;
  auto chunk = [&](int i) { return (unsigned)((lane % C::CR) ^ C::swz(i * RPL + lrow)) * 16; };
  if (n >= KT && end >= C::ROWB) {
#pragma unroll
    for (int i = 0; i < L; ++i, base += step) {
      const void* p = base + (lof + chunk(i));
      __builtin_amdgcn_global_load_lds(p, dst + i * 1024, 16, 0, 0);
    }
  } else {
#pragma unroll 1
    for (int i = 0; i < L; ++i, base += step) {
      const int c = (int)chunk(i);
      const void* p = i * RPL + lrow < n && c < end ? base + (lof + c) : Z;
      __builtin_amdgcn_global_load_lds(p, dst + i * 1024, 16, 0, 0);
    }
  }
}

template <int HDP, int VD, int NW, int KT>
__global__ void __launch_bounds__(64 * NW) attn_wave_kernel(AttnArgs a) {
  using C = V2<HDP>;
  using CV = V2<VD>;
  constexpr int DS = HDP / VD;                     // blocks that share a row tile's output dims
  constexpr int KB = KT * C::ROWB, VB = KT * CV::ROWB, QB = 16 * C::ROWB;
  constexpr int LK = KB / 1024, LV = VB / 1024, LQ = QB / 1024;
  constexpr int NST = KT / 16, NC = HDP / 32, ND = VD / 16;
  static_assert(LQ <= NW && LV >= 1, "one query load a wave; a V tile fills a load");
  constexpr int RING = QB + NW * (KB + VB), MERGE = NW * (ND * 1024 + 128);
  __shared__ __attribute__((aligned(1024))) char smem[RING > MERGE ? RING : MERGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // die-aware order (xcd_remap): the row tiles of one (request, KV head) are
  // consecutive logical blocks
  const unsigned gx = gridDim.x, T = gx * gridDim.y * gridDim.z;
  const unsigned Lb = blockIdx.x + gx * (blockIdx.y + gridDim.y * blockIdx.z);
  const unsigned xr = T % 8, x = Lb % 8, ub = x * (T / 8) + (x < xr ? x : xr) + Lb / 8;
  const unsigned vb = fast_div(ub, a.mul_x), b = fast_div(vb, a.mul_y);
  const int bx = (int)(ub - vb * gx), g = (int)(vb - b * gridDim.y);
  const int tile = bx / DS, d0 = bx % DS * VD;
  const int rows = a.G * a.Lq, hd = a.hd;
  const int lq = lane & 15, grp = lane >> 4;
  const int len0 = a.seg[0].len, len1 = a.seg[1].len, nt0 = (len0 + KT - 1) / KT, nt = nt0 + (len1 + KT - 1) / KT;
  const char* Z = reinterpret_cast<const char*>(a.zeros);
  char* slot_q = smem + wave * 1024;
  char* slot_k = smem + QB + wave * (KB + VB);
  char* slot_v = slot_k + KB;

  // a tile belongs to one segment
  auto issue = [&](int t, auto is_v) {
    const int which = t >= nt0;
    const AttnSeg& sg = a.seg[which];
    const int k0 = (which ? t - nt0 : t) * KT, n = (which ? len1 : len0) - k0;
    if constexpr (decltype(is_v)::value) {
      const char* base = reinterpret_cast<const char*>(sg.v) + (sg.v_sb * b + sg.v_sh * g + sg.v_si * k0 + d0) * 2;
      issue_tile<VD, KT>(base, sg.v_si * 2, n, (hd - d0) * 2, Z, slot_v);
    } else {
      const char* base = reinterpret_cast<const char*>(sg.k) + (sg.k_sb * b + sg.k_sh * g + sg.k_si * k0) * 2;
      issue_tile<HDP, KT>(base, sg.k_si * 2, n, hd * 2, Z, slot_k);
    }
  };
  constexpr std::false_type is_k{};
  constexpr std::true_type is_v{};
  // row r of the block's tile: query head g G + r / Lq, query r % Lq
  auto row_of = [&](int r, int& head, int& qi) {
    const int jh = (int)fast_div((unsigned)r, a.mul_q);
    head = g * a.G + jh;
    qi = r - jh * a.Lq;
  };

  // the queries, 1 KiB a wave, in the layout of a K tile
  if (wave < LQ) {
    const int lr = wave * (64 / C::CR) + lane / C::CR, r = tile * 16 + lr, c = ((lane % C::CR) ^ C::swz(lr)) * 8;
    int head, qi;
    row_of(r, head, qi);
    const void* p = r < rows && c < hd ? reinterpret_cast<const bf16*>(a.q) + (a.q_sb * b + a.q_sh * head + a.q_si * qi + c)
                                       : reinterpret_cast<const bf16*>(Z);
    __builtin_amdgcn_global_load_lds(p, slot_q, 16, 0, 0);
  }
  int t = wave;
  if (t < nt) {
    issue(t, is_k);
    issue(t, is_v);
    // (this wave's queries have landed once only its first tile is pending)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LK + LV) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  asm volatile("s_barrier" ::: "memory");
  bf16x8 qf[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    qf[c] = *reinterpret_cast<const bf16x8*>(smem + lq * C::ROWB + (((c * 4 + grp) ^ C::swz(lq)) << 4));

  f32x4 o[ND];
  float m_run = -INFINITY, l_run = 0.f;            // l_run: this lane's keys
#pragma unroll
  for (int u = 0; u < ND; ++u) o[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float sl2 = a.scale * 1.4426950408889634f;
  constexpr int NU = ND < 4 ? ND : 4, NV8 = ND < 8 ? ND : 8;
  unsigned ad[NV8];
  vt_offsets<VD>(ad);
#pragma unroll
  for (int u = 0; u < NV8; ++u) ad[u] += lds_addr(slot_v);
#pragma unroll 1
  for (; t < nt; t += NW) {
    const bool next = t + NW < nt;
    const int n = t >= nt0 ? len1 - (t - nt0) * KT : len0 - t * KT;
    // this tile's keys have landed once only its values' loads are pending
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LV) : "memory");
    bf16x8 kf[NST][NC];
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      const int row = st * 16 + lq;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        kf[st][c] = *reinterpret_cast<const bf16x8*>(slot_k + row * C::ROWB + (((c * 4 + grp) ^ C::swz(row)) << 4));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (next) issue(t + NW, is_k);
    f32x4 sc[NST];
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      f32x4 s2 = {0.f, 0.f, 0.f, 0.f};             // two chains
      sc[st] = s2;
#pragma unroll
      for (int c = 0; c < NC; c += 2) {
        sc[st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st][c], qf[c], sc[st], 0, 0, 0);
        if (c + 1 < NC) s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st][c + 1], qf[c + 1], s2, 0, 0, 0);
      }
      sc[st] += s2;
    }
    if (n < KT) {
#pragma unroll
      for (int st = 0; st < NST; ++st)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (st * 16 + grp * 4 + e >= n) sc[st][e] = -INFINITY;
    }
    const float m_new = vmax(m_run, max_x32(max_x16(max_of(sc))) * sl2), alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
    typedef __attribute__((ext_vector_type(KT / 4))) __bf16 frag;   // 4 or 8 keys of a lane
    frag pf;
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[st][e], sl2, -m_new));
        pf[4 * st + e] = (bf16)pv;
        l_run += pv;
      }
#pragma unroll
    for (int u = 0; u < ND; ++u) o[u] *= alpha;
    // the values have landed once only the next keys' loads are pending
    if (next) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LK) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // key slot jj of the second product's lane group grp is key 4 grp + jj
    // (jj < 4) or 16 + 4 grp + jj - 4
    frag vf[ND];
    auto part = [&](auto h_) {
      constexpr int u0 = decltype(h_)::value * NU;
      if constexpr (u0 >= ND) return;
      else if constexpr (KT == 16) read_vt16<NU, u0 / 8 * 256>(vf + u0, ad + u0 % 8);
      else read_vt<NU, u0 / 8 * 256, 16 * CV::ROWB>(vf + u0, ad + u0 % 8);
    };
    part(std::integral_constant<int, 0>{});
    part(std::integral_constant<int, 1>{});
    part(std::integral_constant<int, 2>{});
    part(std::integral_constant<int, 3>{});
    if (next) issue(t + NW, is_v);
#pragma unroll
    for (int u = 0; u < ND; ++u) o[u] = pv_mma(vf[u], pf, o[u]);
  }

  // merge: the waves store their outputs and statistics (one without keys a
  // maximum of -inf and zeros), then each wave adds a share of the 16-dim
  // subtiles in wave order
  l_run = sum_x32(sum_x16(l_run));
  __syncthreads();                                 // every wave is done with its slots
  float* mo = reinterpret_cast<float*>(smem);
  float* mst = mo + NW * ND * 256;                 // [wave][16][2]
#pragma unroll
  for (int u = 0; u < ND; ++u) *reinterpret_cast<f32x4*>(mo + (wave * ND + u) * 256 + lane * 4) = o[u];
  if (grp == 0) *reinterpret_cast<f32x2*>(mst + (wave * 16 + lq) * 2) = f32x2{m_run, l_run};
  __syncthreads();
  if (wave >= ND) return;
  const int r = tile * 16 + lq;
  int head, qi;
  row_of(r, head, qi);
  f32x2 ml[NW];
  float w[NW], mm = -INFINITY, l = 0.f;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    ml[q] = *reinterpret_cast<const f32x2*>(mst + (q * 16 + lq) * 2);
    mm = fmaxf(mm, ml[q][0]);
  }
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    w[q] = __builtin_amdgcn_exp2f(ml[q][0] - mm);
    l += ml[q][1] * w[q];
  }
  const float inv = 1.0f / l;
  bf16* op = reinterpret_cast<bf16*>(a.o) + (a.o_sb * b + a.o_sh * head + a.o_si * qi);
#pragma unroll
  for (int u = wave; u < ND; u += NW) {
    const int d = d0 + u * 16 + grp * 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NW; ++q) acc += *reinterpret_cast<const f32x4*>(mo + (q * ND + u) * 256 + lane * 4) * w[q];
    if (r < rows && d < hd)
      *reinterpret_cast<bf16x4*>(op + d) =
          bf16x4{(bf16)(acc[0] * inv), (bf16)(acc[1] * inv), (bf16)(acc[2] * inv), (bf16)(acc[3] * inv)};
  }
}

}  // namespace

// Key groups and ranges of the kernels with blocks of 64 rows. Direct-load kernel: key groups inside a
// block (KS = 2) whenever the grid leaves CUs without a second block (short
// decode and small prefill grids), and key ranges over blocks (split-KV,
// merged by attn_combine_kernel) only when the rounds of tiles they save
// outweigh the merge: the count S minimises rounds x tile time + merge time
// (measured on MI355X: a round of 64 keys ~0.8 us at head dim 32, ~1.4 us
// at 64, of 32 keys ~2.1 us at 256; the merge ~3.5 us), at most one block
// per CU.
// Register-staged kernel (head dim 72): split when fewer than 128 blocks.
static void plan_ranges(const AttnArgs& a, int& splits, int& kchunk, int& ks) {
  const int rows = (a.Hq / a.Hkv) * a.Lq;
  const long blocks = (long)((rows + BQ - 1) / BQ) * a.Hkv * a.B;
  const int total = a.seg[0].len + a.seg[1].len, ntiles = (total + BKV - 1) / BKV;
  const bool v2 = a.zeros != nullptr;
  // two key groups per block when the grid leaves CUs free, and always at
  // head dim 256, where the second group of waves hides the per-tile latency
  // of the large output accumulators (bidirectional pi0-shaped prefill over
  // 816 keys: 155 -> 115 us at batch 8)
  ks = (v2 && a.hd > 32 && (blocks < 256 || a.hd > 128)) ? 2 : 1;
  splits = 1;
  kchunk = ntiles * BKV;
  if (!a.ws || ntiles < 2) return;
  int best = 1;
  if (v2) {
    const int tile = a.hd >= 256 ? 32 : 64;                      // keys per kernel tile
    const double t_tile = a.hd <= 32 ? 0.8 : (a.hd <= 64 ? 1.4 : (a.hd <= 128 ? 1.7 : 2.1)), t_merge = 3.5;
    const int smax = (int)std::min<long>(16, std::max<long>(1, 256 / blocks));
    double best_t = 1e30;
    for (int sp = 1; sp <= std::min(smax, ntiles); ++sp) {
      const int per = (ntiles + sp - 1) / sp;                   // 64-key units per range
      const int rounds = ((per * BKV + tile - 1) / tile + ks - 1) / ks;
      const double t = rounds * t_tile + (sp > 1 ? t_merge : 0.0);
      if (t < best_t - 1e-9) { best_t = t; best = sp; }
    }
  } else if (blocks < 128) {
    best = (int)std::min<long>({(256 + blocks - 1) / blocks, (long)ntiles, 16L});
  }
  while (best > 1 && (long)a.B * a.Hq * a.Lq * best * (a.hd + 2) > a.ws_floats) --best;
  const int per = (ntiles + best - 1) / best;
  kchunk = per * BKV;
  splits = (ntiles + per - 1) / per;              // every range holds keys
}

// The kernel whose waves split the keys, where its blocks of 16 rows are few
// and the keys at most 1024 (longer ranges: split-KV over blocks). At head dim
// 256, two or four blocks share a row tile where that leaves every CU at most
// one. Measured (us, the other kernel with its merge launch / this one):
// - head dims 33 to 128, at most one block a CU: 290 keys, 5 KV heads of 64,
//   50 tokens: batch 1 and 4 8.2 / 5.5; batch 16, 800 blocks, 8.8 / 10.7; 256
//   keys of 72 8.8 / 6.5, batch 3, 768 blocks, 9.2 / 15.
// - over 128, at most one a CU: 866 keys, 1 KV head of 256, 400 rows a
//   request: batch 1 16.7 / 10.0, 2 19.1 / 10.6, 4 21.0 / 13.4, 8 25.5 / 16.0;
//   one request's prefill, 296 keys of 256 20.0 / 9.5.
// - 256, up to two a CU (one after the other), where the other kernel's blocks
//   of 64 rows are well filled and its keys enough: 512 blocks of 128 rows a KV
//   head, 160 keys 12.7 / 13.2, 200 keys (split there) 25.4 / 15.2, 800 keys
//   31.7 / 26.3; 500 blocks of 400 rows, past the sizes it splits, 300 keys
//   16.6 / 16.7, 800 29.2 / 24.8; 512 of 32 rows, 800 keys, 36.4 / 36.7. Head
//   dims below 256 pay for the chunks past their end: 136, 400 blocks, 200
//   keys 12.5 / 15.8.
// - to 32, eight blocks a CU: by two lines (us) fitted to sweeps of 16-128
//   rows a KV head, 32-1000 keys and 256-2048 blocks, within 10 %: this kernel
//   by blocks a CU and keys (more than three blocks of eight waves start one
//   after the other), the other by its blocks a CU and tiles of 64 keys. 1024
//   blocks of 64 rows a KV head: 100 keys 5.2 / 6.3, 520 keys 10.5 / 9.7; of 17
//   rows: 150 keys 7.0 / 6.8; 2048 of 16: 300 keys 24.0 / 16.1; of 64: 1000
//   keys 21.7 / 22.9.
static long row_blocks(const AttnArgs& a, int height) {
  return ((long)(a.Hq / a.Hkv) * a.Lq + height - 1) / height * a.Hkv * a.B;
}

static bool wave_faster(const AttnArgs& a) {
  const int keys = a.seg[0].len + a.seg[1].len;
  const long blocks = row_blocks(a, 16), tall = row_blocks(a, BQ);    // of this kernel, of the other
  if (!a.zeros || keys > 1024) return false;
  if (a.hd > 32) {
    if (blocks <= 256) return true;
    return a.hd == 256 && blocks <= 512 && 3 * tall <= blocks && keys > (tall <= 128 ? 160 : 320);
  }
  if (blocks > 2048) return false;
  const double w = std::max(1.0, blocks / 256.0), t = (double)((tall + 255) / 256);
  const double t_wave = std::max(3.7 + 0.33 * w, 2.8 + 0.74 * w) + keys * (0.0012 + 0.0016 * w);
  const double t_tall = 3.2 + 0.35 * t + (keys + BKV - 1) / BKV * (0.45 + 0.31 * t);
  return t_wave <= t_tall;
}

AttnPlan attn_plan(const AttnArgs& a) {
  AttnPlan p{};
  p.splits = p.groups = 1;
  if (a.et == ET_F32) {
    p.kernel = ATTN_F32;
    p.hdp = p.dims = a.hd <= 64 ? 64 : a.hd <= 128 ? 128 : 256;
    return p;
  }
  if (wave_faster(a)) {
    const long blocks = row_blocks(a, 16);
    p.kernel = ATTN_WAVE;
    p.hdp = a.hd <= 32 ? 32 : a.hd <= 64 ? 64 : a.hd <= 128 ? 128 : 256;
    p.dims = p.hdp / (a.hd <= 128 || blocks * 2 > 256 ? 1 : blocks * 4 > 256 ? 2 : 4);
    return p;
  }
  plan_ranges(a, p.splits, p.kchunk, p.groups);
  // the direct-load kernel serves every head dim (a multiple of 8) with a
  // zero buffer, padded to the next of 32, 64, 128, 256 (chunks past hd load
  // zeros and are not stored): the ViT's 72 runs on the 128-wide variant
  // (54.8 -> 33.4 us per pi0-shaped layer at batch 8 against the
  // register-staged kernel padded to 96); callers without a zero buffer use
  // the register-staged one
  p.kernel = a.zeros ? ATTN_DIRECT : ATTN_STAGED;
  if (a.zeros) {
    p.hdp = a.hd <= 32 ? 32 : a.hd <= 64 ? 64 : a.hd <= 128 ? 128 : 256;
    p.dims = p.hdp == 128 && a.hd <= 80 && p.groups == 1 ? 80 : p.hdp;
  } else {
    p.hdp = p.dims = a.hd <= 32 ? 32 : a.hd <= 64 ? 64 : a.hd <= 96 ? 96 : 256;
  }
  return p;
}

static void launch_wave(const AttnArgs& a, const AttnPlan& p, hipStream_t s) {
  const int G = a.Hq / a.Hkv;
  AttnArgs b = a;
  b.splits = 1;
  b.G = G;
  const dim3 grid((unsigned)((G * a.Lq + 15) / 16) * (p.hdp / p.dims), a.Hkv, a.B);
  // n / d = n mul >> 32 holds while n d < 2^32: at most 2048 blocks, of 16 rows
  auto mul = [](unsigned d) { return d == 1 ? 0u : (unsigned)(((1ull << 32) + d - 1) / d); };
  b.mul_x = mul(grid.x); b.mul_y = mul(grid.y); b.mul_q = mul(a.Lq);
  // (a quarter of V each: LDS for twelve waves, 866 keys 10.9 us by eight and
  // 9.7 by twelve, 450 keys 8.1 and 7.6, 250 keys 6.5 and 6.8)
#define GO(H, V, N, K) hipLaunchKernelGGL((attn_wave_kernel<H, V, N, K>), grid, dim3(64 * N), 0, s, b)
  if (p.hdp == 32) GO(32, 32, 8, 32);
  else if (p.hdp == 64) GO(64, 64, 8, 32);
  else if (p.hdp == 128) GO(128, 128, 8, 32);
  else if (p.dims == 256) GO(256, 256, 8, 16);
  else if (p.dims == 128) GO(256, 128, 8, 16);
  else GO(256, 64, 12, 16);
#undef GO
}

template <int HDP, int KS, int HDU = HDP>
static void launch_direct(const AttnArgs& b, hipStream_t s) {
  const dim3 grid(((b.Hq / b.Hkv) * b.Lq + BQ - 1) / BQ, b.Hkv, b.B * b.splits);
  hipLaunchKernelGGL((attn_v2_kernel<HDP, KS, HDU>), grid, dim3(256 * KS), 0, s, b);
}

template <int HDP>
static void launch_reg_staged(const AttnArgs& b, hipStream_t s) {
  const dim3 grid(((b.Hq / b.Hkv) * b.Lq + BQ - 1) / BQ, b.Hkv, b.B * b.splits);
  hipLaunchKernelGGL(attn_mfma_kernel<HDP>, grid, dim3(256), 0, s, b);
}

void launch_attention(const AttnArgs& a, hipStream_t s) {
  if (a.B <= 0 || a.Lq <= 0) return;
  const AttnPlan p = attn_plan(a);
  if (p.kernel == ATTN_F32) {
    const dim3 grid(((a.Hq / a.Hkv) * a.Lq + 15) / 16, a.Hkv, a.B);
    if (p.hdp == 64) hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(512), 0, s, a);
    else if (p.hdp == 128) hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(512), 0, s, a);
    else hipLaunchKernelGGL(attn_f32_kernel<256>, grid, dim3(512), 0, s, a);
    return;
  }
  // the direct-load kernel keeps scores in log2 units scaled by a positive
  // factor and 32-bit offsets of a tile's rows within a segment
  VLA_REQUIRE(a.scale > 0.f, "attention scale must be positive");
  for (const AttnSeg& sg : a.seg)
    VLA_REQUIRE(64L * 2 * std::max(std::labs(sg.k_si), std::labs(sg.v_si)) + 2L * a.hd < (1L << 32),
                "attention key row stride too large");
  if (p.kernel == ATTN_WAVE) {
    launch_wave(a, p, s);
    return;
  }
  AttnArgs b = a;
  b.splits = p.splits;
  b.kchunk = p.kchunk;
  if (p.kernel == ATTN_DIRECT) {
    if (p.hdp == 32) launch_direct<32, 1>(b, s);
    else if (p.hdp == 64) p.groups == 2 ? launch_direct<64, 2>(b, s) : launch_direct<64, 1>(b, s);
    else if (p.dims == 80) launch_direct<128, 1, 80>(b, s);
    else if (p.hdp == 128) p.groups == 2 ? launch_direct<128, 2>(b, s) : launch_direct<128, 1>(b, s);
    else p.groups == 2 ? launch_direct<256, 2>(b, s) : launch_direct<256, 1>(b, s);
  } else {
    if (p.hdp == 32) launch_reg_staged<32>(b, s);
    else if (p.hdp == 64) launch_reg_staged<64>(b, s);
    else if (p.hdp == 96) launch_reg_staged<96>(b, s);
    else launch_reg_staged<256>(b, s);
  }
  if (b.splits > 1) {
    // 256-thread blocks of 4 wavefronts x 64 / LPR rows
    const long nrows = (long)a.B * a.Hq * a.Lq;
    auto blocks = [&](int lpr) { const long rpb = 4L * (64 / lpr); return dim3((unsigned)((nrows + rpb - 1) / rpb)); };
    if (a.hd <= 64) hipLaunchKernelGGL(attn_combine_kernel<16>, blocks(16), dim3(256), 0, s, b);
    else if (a.hd <= 128) hipLaunchKernelGGL(attn_combine_kernel<32>, blocks(32), dim3(256), 0, s, b);
    else hipLaunchKernelGGL(attn_combine_kernel<64>, blocks(64), dim3(256), 0, s, b);
  }
}
