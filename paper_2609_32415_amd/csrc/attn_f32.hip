// Joint attention over [reference; target] keys in fp32 on the matrix cores (gfx950).
//
// For fp32 workloads whose output must match an fp64 evaluation to ~1e-5: products and sums
// are fp32 throughout (v_mfma_f32_16x16x4_f32). One workgroup = QW query subtiles of 16 rows x
// KW key groups, one wavefront each. A key group takes a contiguous range of the key tiles (TK
// keys) and streams it through its own K and V tiles in LDS, which its QW wavefronts share; the
// next tiles' rows travel through registers while a tile is computed.
//
// Scores are computed transposed, S^T = K Q^T (keys on M, the wavefront's 16 queries on N):
// register r of lane group g = lane / 16 holds key 4 g + r of a 16-key block for query
// lane % 16, which is the K index the B operand of O^T += V^T P^T wants from that lane, so the
// probabilities go from the first product into the second without leaving their registers.
// The K order of the first product and the M order of the second are free: an operand
// register set is one 16-byte LDS read (head dims 16 i + 4 g .. + 3 of a key row; output dims
// 64 hh + 4 m .. + 3 of a value row), and the output rows of a lane are 16-byte stores.
//
// Iteration j issues the products of S_{j+1} with the softmax of S_j between them, then those of
// O += V_j^T P_j^T. The online softmax keeps the split (reference, target) statistics of the
// bf16 kernel. With KW > 1 the groups' statistics and outputs are combined in group order through
// LDS, the same reduction the online softmax performs across key tiles; no workspace is needed.
//
// Bound: the fp32 matrix rate, 32 cycles per product and SIMD (256 FLOP/clk/CU; 153 TFLOP/s on a
// large library product). Measured at 24 heads of 128, 1101 + 1024 keys: all queries 0.60 ms (93
// TFLOP/s), target queries 0.27 ms (98 TFLOP/s); 8 heads of 128, 2048 + 2048 keys, all queries
// 0.56 ms (124 TFLOP/s). One row per lane on the vector ALU, as this path was written before,
// took 7.8 ms for the first. What is left: the last, partly filled round of workgroups, and the
// vector instructions, which do not overlap the products (later stores or earlier loads gave
// nothing). Two per score keep the type's range: a square that keeps subnormal probabilities, and
// the difference to the unscaled max instead of one FMA. The max moves with every larger score, so
// no probability exceeds one and O overflows only where its sum does. Without the three, and
// with a max that lagged by up to 2^8, the times above were 0.59, 0.27 and 0.54 ms.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "internal.h"
#include "plan.h"

namespace refadapt {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// The running max before any key: the lowest finite value, so that keys that score -inf (a product
// that overflows, a masked key) add nothing wherever they stand, in a tile, a key group or a row;
// against -inf their difference would be NaN.
constexpr float LOWEST = -__FLT_MAX__;

// 2^(2 x): the bare exponential returns zero below 2^-126, its square keeps the subnormal
// probabilities, which a value near the largest fp32 still carries into the output.
__device__ __forceinline__ float exp2_twice(float x) {
  const float h = __builtin_amdgcn_exp2f(x);
  return h * h;
}

// x / sum for inv = 1 / sum <= 1: the product, corrected by its remainder to the rounded quotient
// (Markstein); an infinite or NaN x has no remainder.
__device__ __forceinline__ float divide(float x, float sum, float inv) {
  const float q = x * inv, r = fmaf(-q, sum, x);
  return fabsf(r) <= __FLT_MAX__ ? fmaf(r, inv, q) : q;
}

// Largest of the four values of each of one or two accumulators (NaNs ignored, as fmaxf does):
// fmaxf would first canonicalise every operand. The compiler does not place the wait states that
// an instruction in asm needs after a matrix instruction wrote its operand (11 for these) and
// before a lane swap reads its result, so the block holds them.
__device__ __forceinline__ float max_of(const f32x4 (&v)[1]) {
  float r;
  asm("s_nop 15\n\tv_max3_f32 %0, %1, %2, %3\n\tv_max_f32 %0, %0, %4\n\ts_nop 1"
      : "=&v"(r)
      : "v"(v[0][0]), "v"(v[0][1]), "v"(v[0][2]), "v"(v[0][3]));
  return r;
}
__device__ __forceinline__ float max_of(const f32x4 (&v)[2]) {
  float r;
  asm("s_nop 15\n\tv_max3_f32 %0, %1, %2, %3\n\tv_max3_f32 %0, %0, %4, %5\n\tv_max3_f32 %0, %0, %6, %7\n\t"
      "v_max_f32 %0, %0, %8\n\ts_nop 1"
      : "=&v"(r)
      : "v"(v[0][0]), "v"(v[0][1]), "v"(v[0][2]), "v"(v[0][3]), "v"(v[1][0]), "v"(v[1][1]), "v"(v[1][2]), "v"(v[1][3]));
  return r;
}

// A value combined over the query's four lane groups (lanes l, l ^ 16, l ^ 32, l ^ 48).
__device__ __forceinline__ float quad_max(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float quad_add(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Instruction order of the block that holds N score products, the softmax and LDSR operand
// reads of the first products after it: operand reads run two steps ahead, and vector
// instructions go between the products (a product occupies the matrix core for 32 cycles, an
// issue slot of the wavefront for 4).
template <int N, int MB, int LDSR>
__device__ __forceinline__ void interleave() {
  __builtin_amdgcn_sched_group_barrier(0x100, 2 * MB, 0);  // LDS reads
  __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
#pragma unroll
  for (int i = 0; i < N / 4; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x100, LDSR, 0);
}

// Key tiles per LDS buffer set: a key group of one wavefront reads only what it wrote itself,
// in order, so one K and one V tile serve; a group of several wavefronts keeps two of each and
// meets at one barrier per tile.
template <int D, int NW, int QW, int TK>
struct F32Shape {
  static constexpr int KW = NW / QW;
  static constexpr int KSTR = D + 4;                    // K row stride: 16 rows hit 16 bank groups
  static constexpr int NBUF = QW == 1 ? 1 : 2;
  static constexpr int GROUP = NBUF * TK * (KSTR + D);  // floats of one group's K and V tiles
  static constexpr int TILES = KW * GROUP;
  static constexpr int DB = D / 16;                     // 16-row blocks of O^T
  static constexpr int OREGS = 4 * DB;                  // O registers per lane
  // combining: every group but the first stores O and (m, l, m_ref, l_ref) per lane
  static constexpr int MERGE = (NW - QW) * 64 * (OREGS + 4);
  static constexpr int FLOATS = TILES > MERGE ? TILES : MERGE;
};

template <int D, int NW, int QW, int TK>
__global__ __launch_bounds__(64 * NW, 2) void attn_f32_kernel(AttnParams p) {
  using S = F32Shape<D, NW, QW, TK>;
  constexpr int KW = S::KW, KSTR = S::KSTR, DB = S::DB;
  constexpr int MB = TK / 16;        // 16-key blocks of a tile
  constexpr int KI = D / 16;         // operand reads of a key row
  constexpr int VH = D / 64;         // operand reads of a value row
  constexpr int BQ = 16 * QW;        // query rows per workgroup
  constexpr int GT = 64 * QW;        // threads of a key group
  constexpr int NV = TK * D / 4 / GT;  // float4s of one tile each thread stages
  __shared__ __attribute__((aligned(16))) float lds[S::FLOATS];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qw = wave % QW, kg = wave / QW;
  const int gtid = threadIdx.x - kg * GT;
  const int n = lane & 15, g = lane >> 4;

  const int qt_ref = p.qt_ref > 0 ? (p.n_ref + BQ - 1) / BQ : 0;
  const int qt_tgt = (p.n_tgt + BQ - 1) / BQ;
  bool use_cache = p.kvsrc == KV_CACHE;
  int first = 0;  // a reused block skips the reference query tiles
  if (p.kvsrc == KV_DEVICE) {
    const int dec = *p.decision;
    if (dec == DEC_REUSE) first = qt_ref;
    use_cache = dec != DEC_COMPUTE;
  }
  const int per_bh = qt_ref - first + qt_tgt;
  const int total = p.B * p.H * per_bh;
  const int item = p.block0 + (int)blockIdx.x;
  if (item >= total) return;
  const int tile = xcd_remap(item, total);
  const int bh = tile / per_bh;
  int qt = tile - bh * per_bh + first;
  const int b = bh / p.H, h = bh - b * p.H;
  const bool ref_rows = qt < qt_ref;
  if (!ref_rows) qt -= qt_ref;

  const View qv = ref_rows ? (use_cache && p.q_cache.p ? p.q_cache : p.q_ref) : p.q_tgt;
  const View ov = ref_rows ? p.o_ref : p.o_tgt;
  const int n_rows = ref_rows ? p.n_ref : p.n_tgt;
  const View krv = use_cache ? p.k_cache : p.k_fresh;
  const View vrv = use_cache ? p.v_cache : p.v_fresh;
  const float* kr = static_cast<const float*>(krv.p) + b * krv.sb + h * krv.sh;
  const float* vr = static_cast<const float*>(vrv.p) + b * vrv.sb + h * vrv.sh;
  const float* ky = static_cast<const float*>(p.k_tgt.p) + b * p.k_tgt.sb + h * p.k_tgt.sh;
  const float* vy = static_cast<const float*>(p.v_tgt.p) + b * p.v_tgt.sb + h * p.v_tgt.sh;

  // this group's key tiles [j0, j1); every group takes part in `steps` barriers
  const int n_rt = (p.n_ref + TK - 1) / TK;
  const int nt = n_rt + (p.n_tgt + TK - 1) / TK;
  const int j0 = (int)((int64_t)kg * nt / KW), j1 = (int)((int64_t)(kg + 1) * nt / KW);
  const int steps = (nt + KW - 1) / KW;

  float* const kbuf = lds + kg * S::GROUP;
  float* const vbuf = kbuf + S::NBUF * TK * KSTR;
  auto publish = [&]() {
    if constexpr (QW == 1)
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    else
      __syncthreads();
  };
  // Thread gtid stages float4 column `scol` of rows srow + i * RSTEP of each tile.
  constexpr int RSTEP = GT * 4 / D;
  const int srow = gtid / (D / 4), scol = 4 * (gtid % (D / 4));
  f32x4 kst[NV] = {}, vst[NV] = {};  // tiles on their way to LDS
  // One K or V stream: the address of this thread's first float4 of the next tile, the rows of
  // the view from that tile on, the view's row stride, and the tile's number. Advancing is one
  // 64-bit add; the view changes once, where the reference keys end and the target keys begin.
  struct Cursor {
    const float* ptr;
    int64_t ss;
    int rows, t;
  };
  auto set_view = [&](Cursor& cur, const float* base, int64_t ss, int first_row, int rows) {
    cur.ss = ss;
    cur.rows = rows - first_row;
    cur.ptr = base + (first_row + srow) * ss + scol;
  };
  auto fetch = [&](f32x4(&st)[NV], Cursor& cur, const float* tgt, int64_t tgt_ss) __attribute__((always_inline)) {
    if (cur.t >= j1) return;
    if (cur.t == n_rt) set_view(cur, tgt, tgt_ss, 0, p.n_tgt);
    if (cur.rows >= TK) {
      const float* src = cur.ptr;
#pragma unroll
      for (int i = 0; i < NV; ++i, src += RSTEP * cur.ss) st[i] = *reinterpret_cast<const f32x4*>(src);
    } else {
      // Past a ragged tile's end the last valid row is read again: its scores are dropped, its
      // values stored as zeros.
#pragma unroll
      for (int i = 0; i < NV; ++i)
        st[i] = *reinterpret_cast<const f32x4*>(cur.ptr + (min(srow + i * RSTEP, cur.rows - 1) - srow) * cur.ss);
    }
    cur.ptr += TK * cur.ss;
    cur.rows -= TK;
    cur.t += 1;
  };
  Cursor kc, vc;
  kc.t = vc.t = j0;
  if (j0 < n_rt) {
    set_view(kc, kr, krv.ss, j0 * TK, p.n_ref);
    set_view(vc, vr, vrv.ss, j0 * TK, p.n_ref);
  } else {
    set_view(kc, ky, p.k_tgt.ss, (j0 - n_rt) * TK, p.n_tgt);
    set_view(vc, vy, p.v_tgt.ss, (j0 - n_rt) * TK, p.n_tgt);
  }
  auto fetch_k = [&]() __attribute__((always_inline)) { fetch(kst, kc, ky, p.k_tgt.ss); };
  auto fetch_v = [&]() __attribute__((always_inline)) { fetch(vst, vc, vy, p.v_tgt.ss); };
  auto store_k = [&](int buf) {
    float* ks = kbuf + (S::NBUF > 1 ? buf : 0) * TK * KSTR + srow * KSTR + scol;
#pragma unroll
    for (int i = 0; i < NV; ++i) *reinterpret_cast<f32x4*>(ks + i * RSTEP * KSTR) = kst[i];
  };
  auto store_v = [&](int buf) {
    float* vs = vbuf + (S::NBUF > 1 ? buf : 0) * TK * D + srow * D + scol;
    if (vc.rows < 0) {  // the fetched tile is ragged
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if (srow + i * RSTEP >= TK + vc.rows) vst[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) *reinterpret_cast<f32x4*>(vs + i * RSTEP * D) = vst[i];
  };

  fetch_k();
  const int qrow = qt * BQ + 16 * qw + n;
  const bool qvalid = qrow < n_rows;
  f32x4 q[KI];
  {
    const float* qp = static_cast<const float*>(qv.p) + b * qv.sb + h * qv.sh + (int64_t)qrow * qv.ss;
#pragma unroll
    for (int i = 0; i < KI; ++i)
      q[i] = qvalid ? *reinterpret_cast<const f32x4*>(qp + 16 * i + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 o[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // l_run and l_ref hold this lane's share of the query's keys; the four lane groups of a
  // query see the same max and are added at the end.
  // Maxima are unscaled scores: (score - max) is exact for the scores near the max, where a max
  // rounded after scaling would be off by its own rounding, 2^7 in log2 at scores of 2^32.
  float m_run = LOWEST, l_run = 0.f, m_ref = LOWEST, l_ref = 0.f;
  const float c = p.sc_log2, hc = 0.5f * c;

  // scores of the K tile in buffer `buf`
  auto scores = [&](f32x4(&sc)[MB], int buf) __attribute__((always_inline)) {
    const float* ks = kbuf + (S::NBUF > 1 ? buf : 0) * TK * KSTR + n * KSTR + 4 * g;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) sc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 a[2][MB];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) a[i][mb] = *reinterpret_cast<const f32x4*>(ks + 16 * mb * KSTR + 16 * i);
#pragma unroll
    for (int i = 0; i < KI; ++i) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          sc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i & 1][mb][t], q[i][t], sc[mb], 0, 0, 0);
      if (i + 2 < KI) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          a[i & 1][mb] = *reinterpret_cast<const f32x4*>(ks + 16 * mb * KSTR + 16 * (i + 2));
      }
    }
  };

  store_k(0);
  fetch_k();
  fetch_v();
  publish();
  f32x4 sa[MB], sb[MB];
  scores(sa, 0);
  if constexpr (QW == 1) publish();
  store_k(1);
  store_v(0);

  auto iteration = [&](int s, f32x4(&sc)[MB], f32x4(&sn)[MB]) __attribute__((always_inline)) {
    const int j = j0 + s, buf = s & 1;
    publish();  // K_{j+1} and V_j are in LDS, and every wavefront has read K_j and V_{j-1}
    if (j >= j1) return;  // whole wavefronts
    fetch_k();  // K_{j+2}
    fetch_v();  // V_{j+1}
    const int valid = j < n_rt ? p.n_ref - j * TK : p.n_tgt - (j - n_rt) * TK;
    if (valid < TK) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * mb + 4 * g + r >= valid) sc[mb][r] = -__builtin_inff();
    }
    // The products of tile j + 1 with the softmax of tile j under them.
    float alpha;
    auto softmax = [&]() __attribute__((always_inline)) {
      const float m_tile = quad_max(max_of(sc));
      const float m_new = m_tile > m_run ? m_tile : m_run;
      alpha = exp2_twice((m_run - m_new) * hc);
      float rs = 0.f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[mb][r] = exp2_twice((sc[mb][r] - m_new) * hc);
        rs += (sc[mb][0] + sc[mb][1]) + (sc[mb][2] + sc[mb][3]);
      }
      l_run = l_run * alpha + rs;
      m_run = m_new;
    };
    // V operands of step k = 4 mb + r: rows 16 mb + 4 g + r
    const float* vs = vbuf + (S::NBUF > 1 ? buf : 0) * TK * D + 4 * g * D + 4 * n;
    f32x4 va[2][VH];
    auto v_operand = [&](int k) __attribute__((always_inline)) {
#pragma unroll
      for (int hh = 0; hh < VH; ++hh)
        va[k & 1][hh] = *reinterpret_cast<const f32x4*>(vs + (16 * (k >> 2) + (k & 3)) * D + 64 * hh);
    };
    if (j + 1 < j1) {
      scores(sn, buf ^ 1);
      softmax();
      v_operand(0);
      v_operand(1);
      interleave<MB * KI * 4, MB, 2 * VH>();
      asm volatile("; fused" : "+v"(alpha), "+v"(l_run));
    } else {
      softmax();
      v_operand(0);
      v_operand(1);
      asm volatile("; last" : "+v"(alpha), "+v"(l_run));
    }
    if (__any(!(alpha == 1.f))) {
#pragma unroll
      for (int i = 0; i < DB; ++i) o[i] *= alpha;
    }
    if constexpr (QW == 1) publish();
    store_k(buf);
    if constexpr (QW > 1) store_v(buf ^ 1);
#pragma unroll
    for (int k = 0; k < 4 * MB; ++k) {
#pragma unroll
      for (int hh = 0; hh < VH; ++hh)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          o[4 * hh + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[k & 1][hh][t], sc[k >> 2][k & 3], o[4 * hh + t], 0, 0, 0);
      if (k + 2 < 4 * MB) v_operand(k + 2);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (j == n_rt - 1) {
      m_ref = m_run;
      l_ref = l_run;
      l_run = 0.f;
    }
    if constexpr (QW == 1) {
      publish();
      store_v(0);
    }
  };
  int s = 0;
  for (; s + 1 < steps; s += 2) {
    iteration(s, sa, sb);
    iteration(s + 1, sb, sa);
  }
  if (s < steps) iteration(s, sa, sb);
  if (j0 < j1 && j1 < n_rt) {  // a key range inside the reference: all of it is reference mass
    m_ref = m_run;
    l_ref = l_run;
    l_run = 0.f;
  }
  l_run = quad_add(l_run);
  l_ref = quad_add(l_ref);

  float L_R, M_R = m_ref, L_Rr = l_ref;  // L_Rr: reference sum against M_R
  if constexpr (KW > 1) {
    __syncthreads();  // the tiles have been read: their memory takes the partial results
    constexpr int REC = S::OREGS + 4;
    if (kg > 0) {
      float* r0 = lds + (int64_t)(wave - QW) * 64 * REC + lane;
#pragma unroll
      for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) r0[64 * (4 * i + r)] = o[i][r];
      r0[64 * S::OREGS] = m_run;
      r0[64 * (S::OREGS + 1)] = l_run;
      r0[64 * (S::OREGS + 2)] = m_ref;
      r0[64 * (S::OREGS + 3)] = l_ref;
    }
    __syncthreads();
    if (kg > 0) return;
    const float* rec = lds + (int64_t)qw * 64 * REC + lane;
    constexpr int STEP = QW * 64 * REC;  // from one group's record of these queries to the next's
    float M = m_run;
#pragma unroll
    for (int k = 0; k < KW - 1; ++k) {
      M = fmaxf(M, rec[k * STEP + 64 * S::OREGS]);
      M_R = fmaxf(M_R, rec[k * STEP + 64 * (S::OREGS + 2)]);
    }
    // a group without keys has sums of zero
    float w = exp2f((m_run - M) * c);
    l_run *= w;
    L_Rr = l_ref > 0.f ? l_ref * exp2f((m_ref - M_R) * c) : 0.f;
#pragma unroll
    for (int i = 0; i < DB; ++i) o[i] *= w;
#pragma unroll
    for (int k = 0; k < KW - 1; ++k) {
      const float* r0 = rec + k * STEP;
      w = exp2f((r0[64 * S::OREGS] - M) * c);
      l_run += r0[64 * (S::OREGS + 1)] * w;
      const float lr = r0[64 * (S::OREGS + 3)];
      if (lr > 0.f) L_Rr += lr * exp2f((r0[64 * (S::OREGS + 2)] - M_R) * c);
#pragma unroll
      for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[i][r] += r0[64 * (4 * i + r)] * w;
    }
    m_run = M;
  }
  if (!qvalid) return;
  L_R = L_Rr > 0.f ? L_Rr * exp2f((M_R - m_run) * c) : 0.f;
  const float sum = L_R + l_run, inv = 1.f / sum;
  float* op = static_cast<float*>(const_cast<void*>(ov.p)) + b * ov.sb + h * ov.sh + (int64_t)qrow * ov.ss;
#pragma unroll
  for (int hh = 0; hh < VH; ++hh)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<f32x4*>(op + 64 * hh + 4 * (4 * g + r)) =
          f32x4{divide(o[4 * hh][r], sum, inv), divide(o[4 * hh + 1][r], sum, inv), divide(o[4 * hh + 2][r], sum, inv),
                divide(o[4 * hh + 3][r], sum, inv)};
  if (g != 0) return;
  const int64_t row = (int64_t)bh * n_rows + qrow;
  const float mass = L_R / sum;
  if (!ref_rows) {
    if (p.mass_tgt) p.mass_tgt[row] = mass;
    if (p.lse_tgt) {
      const float ln2 = 0.69314718055994531f;
      p.lse_tgt[2 * row] = fmaf(M_R, c, log2f(L_Rr)) * ln2;
      p.lse_tgt[2 * row + 1] = fmaf(m_run, c, log2f(sum)) * ln2;
    }
  } else if (p.mass_refq) {
    p.mass_refq[row] = mass;
  }
}

template <int D, int NW, int QW, int TK>
hipError_t launch(const AttnParams& p, hipStream_t stream) {
  constexpr int BQ = 16 * QW;
  const int64_t per_bh = (p.qt_ref > 0 ? (p.n_ref + BQ - 1) / BQ : 0) + (p.n_tgt + BQ - 1) / BQ;
  const int64_t total = (int64_t)p.B * p.H * per_bh;
  if (total > 0x7fffffff) return hipErrorInvalidValue;
  // One launch holds fewer than 2^32 threads: with a few rows per (batch, head) and millions of
  // these the workgroups take several.
  constexpr int64_t per_launch = (int64_t)0xffffffff / (64 * NW) & ~7;
  AttnParams q = p;
  for (int64_t first = 0; first < total; first += per_launch) {
    q.block0 = (int32_t)first;
    const unsigned n = (unsigned)std::min(per_launch, total - first);
    const hipError_t e = launch_kernel(attn_f32_kernel<D, NW, QW, TK>, dim3(n), dim3(64 * NW), 0, stream, q);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int D>
hipError_t launch_dim(const AttnParams& p, hipStream_t stream) {
  const int dev_cus = attn_bf16_slots(D, kAttnBf16BM).cus;
  const int64_t cus = dev_cus > 0 ? dev_cus : 256;
  const F32Split sp = f32_split((int64_t)p.B * p.H, p.n_ref, p.n_tgt, cus);
  switch (sp.subtiles) {
    case 4: return launch<D, 4, 4, 32>(p, stream);
    case 2: return launch<D, 4, 2, 16>(p, stream);
    default: return sp.wavefronts == 8 ? launch<D, 8, 1, 16>(p, stream) : launch<D, 4, 1, 16>(p, stream);
  }
}

}  // namespace

hipError_t launch_attn_f32(const AttnParams& p, int head_dim, hipStream_t stream) {
  return head_dim == 128 ? launch_dim<128>(p, stream) : launch_dim<64>(p, stream);
}

}  // namespace refadapt
