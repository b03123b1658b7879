// fs_device.h - device-side building blocks of stitched kernels for gfx950 (CDNA4, wave64).
//
// A stitched kernel is a generated straight-line body that calls the pieces below.  The
// body is the paper's thread composition (Section 1, Figure 2(a)): every elementwise node of
// the fused group is evaluated in registers on the lane's slice of a row.  Nodes that need
// another parallel loop - reductions and whatever consumes them - are joined inside the same
// kernel through on-chip memory, the paper's block composition (Section 1, Figure 2(b);
// Section 5.2, Algorithm 2).  On this hardware a 64-lane wavefront exchanges values through
// DPP / lane-permute instructions without touching LDS at all, so LDS is only needed when a
// row spans several wavefronts, for column partials and for transposing stores.
//
// Work decomposition (a Row schedule with split_dim = 0 in the terms of Section 4.1): a
// workgroup of WG lanes is split into G = WG / L row-groups of L lanes.  Per loop trip a
// row-group owns one row; lane `lir` of the row-group owns the 16-byte vectors
// j*L + lir (j = 0..NVL-1) of that row, i.e. E = NVL*V elements that stay in VGPRs for the
// whole body.  Consecutive lanes touch consecutive 16-byte vectors: every wave-wide memory
// instruction is fully coalesced.
//
// This header is compiled two ways: ahead of time with hipcc (to check it and for the
// probe kernels) and at run time as the prefix of every generated kernel.
#ifndef FS_DEVICE_H_
#define FS_DEVICE_H_

#define FS_DEV __device__ __forceinline__

// dtype tags (values match the host enum fs_dtype)
#define FS_DT_F32 0
#define FS_DT_BF16 1
#define FS_DT_U8 2
// reduction kinds (values match fs_reduce_kind)
#define FS_K_SUM 0
#define FS_K_MAX 1
#define FS_K_MIN 2
#define FS_K_MEAN 3

typedef unsigned int fs_u32;
typedef unsigned short fs_u16;
typedef unsigned char fs_u8;

template <int DT> struct fs_elem;
template <> struct fs_elem<FS_DT_F32> { typedef float type; };
template <> struct fs_elem<FS_DT_BF16> { typedef fs_u16 type; };
template <> struct fs_elem<FS_DT_U8> { typedef fs_u8 type; };

template <typename T, int N> struct fs_vec { typedef T type __attribute__((ext_vector_type(N))); };
template <typename T> struct fs_vec<T, 1> { typedef T type; };
// the same vector at an address that is only aligned to its elements (global memory takes 4-, 8- and 16-byte accesses at any
// address: one instruction either way)
template <typename T, int N> struct fs_vec_ua {
  typedef typename fs_vec<T, N>::type vec;
  typedef vec type __attribute__((aligned(alignof(T))));
};

// ------------------------------------------------------------------------------------------
// scalar conversions
// ------------------------------------------------------------------------------------------
FS_DEV constexpr float fs_lit(fs_u32 bits) { return __builtin_bit_cast(float, bits); }  // exact literal
FS_DEV float fs_bf16_bits_to_f32(fs_u16 h) { return __builtin_bit_cast(float, (fs_u32)h << 16); }
// round-to-nearest-even fp32 -> bf16 (v_cvt_pk_bf16_f32 on gfx950)
FS_DEV fs_u16 fs_f32_to_bf16_bits(float f) { return __builtin_bit_cast(fs_u16, (__bf16)f); }

template <int DT> FS_DEV float fs_to_f32(typename fs_elem<DT>::type x);
template <> FS_DEV float fs_to_f32<FS_DT_F32>(float x) { return x; }
template <> FS_DEV float fs_to_f32<FS_DT_BF16>(fs_u16 x) { return fs_bf16_bits_to_f32(x); }
template <> FS_DEV float fs_to_f32<FS_DT_U8>(fs_u8 x) { return x ? 1.0f : 0.0f; }

template <int DT> FS_DEV typename fs_elem<DT>::type fs_from_f32(float x);
template <> FS_DEV float fs_from_f32<FS_DT_F32>(float x) { return x; }
template <> FS_DEV fs_u16 fs_from_f32<FS_DT_BF16>(float x) { return fs_f32_to_bf16_bits(x); }
template <> FS_DEV fs_u8 fs_from_f32<FS_DT_U8>(float x) { return x != 0.0f ? (fs_u8)1 : (fs_u8)0; }

// A node's value is rounded once to its declared dtype even when it never leaves registers.
template <int DT> FS_DEV float fs_round(float x) { return x; }
template <> FS_DEV float fs_round<FS_DT_BF16>(float x) { return fs_bf16_bits_to_f32(fs_f32_to_bf16_bits(x)); }

// ------------------------------------------------------------------------------------------
// elementwise math.  + - * / sqrt max min are the IEEE operations (the translation unit is
// compiled without contraction), so values that feed a predicate are reproducible bit for bit.
// exp/log/tanh/sigmoid/gelu/rsqrt/rcp are built on the hardware's 1-ulp transcendental
// instructions (v_exp_f32, v_log_f32, v_rcp_f32, v_rsq_f32).
// ------------------------------------------------------------------------------------------
#define FS_LOG2E 1.4426950408889634f
#define FS_LN2 0.6931471805599453f

// exp(x) = 2^(x*log2e).  The product is carried in two floats (t + r) so its rounding error
// does not grow with |x|: 2^(t+r) = 2^t * (1 + r ln2 + ...).
FS_DEV float fs_exp(float x) {
  const float t = x * FS_LOG2E;
  float r = __builtin_fmaf(x, FS_LOG2E, -t);
  r = __builtin_fmaf(x, 1.925963033500494e-8f /* log2(e) - float(log2(e)) */, r);
  const float p = __builtin_amdgcn_exp2f(t);
  return __builtin_fmaf(p, r * FS_LN2, p);
}
// -x on the bits; the empty statement keeps the compiler from making a float negation of it again
FS_DEV float fs_neg(float x) {
  fs_u32 u = __builtin_bit_cast(fs_u32, x) ^ 0x80000000u;
  asm("" : "+v"(u));
  return __builtin_bit_cast(float, u);
}
FS_DEV float fs_log(float x) { return __builtin_amdgcn_logf(x) * FS_LN2; }
FS_DEV float fs_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
FS_DEV float fs_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
FS_DEV float fs_sqrt(float x) { return __builtin_sqrtf(x); }
// (Rows divide by one value in this way, too.  Its reciprocal, a correction step and a test that both operands are in the range where
// that gives the same bits: softmax fp32 [2048,50001] 164.1 us in the place of 164.9, masked softmax bf16 [16384,577] 10.13 and 10.17.)
FS_DEV float fs_div(float a, float b) { return a / b; }
FS_DEV float fs_max(float a, float b) { return __builtin_fmaxf(a, b); }
FS_DEV float fs_min(float a, float b) { return __builtin_fminf(a, b); }

// sigmoid(x) = 1 / (1 + 2^(-x log2e)); saturates cleanly to 0 and 1.
FS_DEV float fs_sigmoid(float x) {
  const float e = __builtin_amdgcn_exp2f(x * -FS_LOG2E);
  return __builtin_amdgcn_rcpf(1.0f + e);
}

// tanh: for |x| >= 1/4, 1 - 2/(e^{2|x|}+1) (no cancellation there); below, the odd Maclaurin
// polynomial through x^9 (truncation < 1e-8 relative at 1/4).  Both sides are evaluated and
// selected, so a wave never diverges.
FS_DEV float fs_tanh(float x) {
  const float ax = __builtin_fabsf(x);
  const float e = __builtin_amdgcn_exp2f(ax * (2.0f * FS_LOG2E));
  const float big = __builtin_fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
  const float x2 = x * x;
  float p = __builtin_fmaf(x2, 0.021869488536155203f, -0.053968253968253971f);
  p = __builtin_fmaf(x2, p, 0.13333333333333333f);
  p = __builtin_fmaf(x2, p, -0.33333333333333331f);
  const float small = __builtin_fmaf(ax * x2, p, ax);
  return __builtin_copysignf(ax < 0.25f ? small : big, x);
}

// tanh-GeLU: 0.5 z (1 + tanh(u)) with u = sqrt(2/pi) (z + 0.044715 z^3).  Since
// (1 + tanh u)/2 = sigmoid(2u), it is evaluated as z / (1 + 2^(-2u log2e)): no cancellation in
// the negative tail, one exp and one rcp per element.  The constants of u and of the base-2
// exponent are folded into one odd polynomial: -2u log2e = z (c2 + c1 z^2).
FS_DEV float fs_gelu_tanh(float z) {
  constexpr float c2 = -2.0f * 0.7978845608028654f * FS_LOG2E;
  constexpr float c1 = 0.044715f * c2;
  const float t = __builtin_fmaf(c1, z * z, c2);
  const float e = __builtin_amdgcn_exp2f(z * t);
  return z * __builtin_amdgcn_rcpf(1.0f + e);
}

// ------------------------------------------------------------------------------------------
// vector memory access: V elements of dtype DT per access (16 bytes for the widest dtype of
// the group).  Invalid rows / columns load zeros and store nothing.
// ------------------------------------------------------------------------------------------
// UA: the address is aligned to the element only.
template <int DT, int V, bool NT = false, bool UA = false>
FS_DEV typename fs_vec<typename fs_elem<DT>::type, V>::type fs_load_raw(const void* base, long elem_index) {
  typedef typename fs_elem<DT>::type T;
  if constexpr (UA) {
    typedef typename fs_vec_ua<T, V>::type VT;
    const VT* p = reinterpret_cast<const VT*>(static_cast<const T*>(base) + elem_index);
    return NT ? __builtin_nontemporal_load(p) : *p;
  } else {
    typedef typename fs_vec<T, V>::type VT;
    const VT* p = reinterpret_cast<const VT*>(static_cast<const T*>(base) + elem_index);
    return NT ? __builtin_nontemporal_load(p) : *p;
  }
}
template <int DT, int V, bool NT = false, bool UA = false> FS_DEV void fs_load_vec(float* dst, const void* base, long elem_index) {
  const auto raw = fs_load_raw<DT, V, NT, UA>(base, elem_index);
  if constexpr (V == 1) {
    dst[0] = fs_to_f32<DT>(raw);
  } else {
#pragma unroll
    for (int k = 0; k < V; ++k) dst[k] = fs_to_f32<DT>(raw[k]);
  }
}

template <int DT, int V, bool NT = false, bool UA = false> FS_DEV void fs_store_vec(const float* src, void* base, long elem_index) {
  typedef typename fs_elem<DT>::type T;
  typedef typename fs_vec<T, V>::type VT;
  VT raw;
  if constexpr (V == 1) {
    raw = fs_from_f32<DT>(src[0]);
  } else {
#pragma unroll
    for (int k = 0; k < V; ++k) raw[k] = fs_from_f32<DT>(src[k]);
  }
  if constexpr (UA) {
    typedef typename fs_vec_ua<T, V>::type VU;
    VU* p = reinterpret_cast<VU*>(static_cast<T*>(base) + elem_index);
    if constexpr (NT) __builtin_nontemporal_store(raw, p);
    else *p = raw;
  } else {
    VT* p = reinterpret_cast<VT*>(static_cast<T*>(base) + elem_index);
    if constexpr (NT) __builtin_nontemporal_store(raw, p);
    else *p = raw;
  }
}

// Rows whose width is no multiple of V keep V-wide accesses: a row of C columns is NV = ceil(C / V) vectors, and the last one
// covers its LAST V columns, C-V .. C-1, so its first `skip` elements repeat columns of the vector before it.  An element of a
// lane's slice is owned when it is the one its column is counted by: reductions and column accumulators' folds take owned
// elements only; stores write the repeated ones twice, with the same bits.  The rows then start at any multiple of the element
// size, which global memory accesses allow: measured on 512 MB copies, 16-byte accesses run at 95 % of the aligned rate at
// 4-byte offsets and at 92 % at 2-byte offsets, where element-wise accesses reach 82 % (4 bytes) and 42 % (2 bytes).
// RAGGED: 0 = every vector index of the slice lies inside a row of NV whole vectors; 1 + D = indices may fall beyond the row,
// and the last vector overlaps its neighbour by D elements (C = NV*V - D).
constexpr int fs_overlap(int ragged) { return ragged > 0 ? ragged - 1 : 0; }
constexpr int fs_cols(int v, int nv, int ragged) { return (int)((long)nv * v - fs_overlap(ragged)); }
// One expression serves both the clamp of vectors beyond the row and the overlapping last vector.
// (Columns beyond the row stay below 2^31 for rows of up to 2^30; longer ones compare vector indices.)
constexpr int FS_COLS_INT = 1 << 30;
template <int V, int C> FS_DEV int fs_vec_col(int vi) {
  if constexpr (C > FS_COLS_INT) return vi < C / V ? vi * V : C - V;
  return vi * V < C - V ? vi * V : C - V;
}
template <int V, int C> FS_DEV int fs_vec_skip(int vi) {
  if constexpr (C > FS_COLS_INT) return vi < C / V ? 0 : (vi - C / V) * V + (C % V ? V - C % V : V);
  return vi * V < C - V ? 0 : vi * V - (C - V);
}
template <int C, bool BIG = (C > FS_COLS_INT)> struct fs_col_index { typedef int type; };
template <int C> struct fs_col_index<C, true> { typedef long type; };
// column of vector vi, clamped into the row
template <int V, int NV, int RAGGED> FS_DEV long fs_col_of(int vi) {
  if constexpr (fs_overlap(RAGGED) != 0) return fs_vec_col<V, fs_cols(V, NV, RAGGED)>(vi);
  if (RAGGED) vi = vi < NV ? vi : NV - 1;
  return (long)vi * V;
}
// is element k of vector vi counted by this lane?
template <int V, int NV, int RAGGED> FS_DEV bool fs_owned(int vi, int k) {
  if constexpr (RAGGED == 0) return true;
  else if constexpr (fs_overlap(RAGGED) == 0) return vi < NV;
  else return k >= fs_vec_skip<V, fs_cols(V, NV, RAGGED)>(vi);
}

// Load the lane's slice of one row tile: vectors vbase + j*L + lir, j < NVL (vbase = 0 unless a
// row is cut into several column tiles).  `row_elem0` is the element index of the first column
// of a VALID row (callers clamp the row index instead of predicating the load).  NV = vectors
// per row; RAGGED (above) says some of those vector indices can fall beyond NV: they are clamped too.
// Nothing here branches, so all loads of a body are issued back to back and waited for once;
// lanes outside the tensor hold duplicates that are never stored and never reduced.
// (the _vec forms handle vector j of the slice alone: a body that is emitted vector by vector
// keeps fewer registers live)
template <int DT, int V, int NVL, int L, int NV, int RAGGED, bool NT = false>
FS_DEV void fs_load_row_vec(float (&dst)[NVL * V], const void* base, long row_elem0, int lir, int vbase, int j) {
  fs_load_vec<DT, V, NT, fs_overlap(RAGGED) != 0>(&dst[j * V], base, row_elem0 + fs_col_of<V, NV, RAGGED>(vbase + j * L + lir));
}
template <int DT, int V, int NVL, int L, int NV, int RAGGED, bool NT = false>
FS_DEV void fs_load_row(float (&dst)[NVL * V], const void* base, long row_elem0, int lir, int vbase) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) fs_load_row_vec<DT, V, NVL, L, NV, RAGGED, NT>(dst, base, row_elem0, lir, vbase, j);
}

// The lane's slice of a row that is the concatenation of two tensors in memory.  AXIS 1 (columns): a is [R,SPLIT],
// b is [R,CB], the row is a's row followed by b's (SPLIT and CB are multiples of V: no vector straddles the seam).
// AXIS 0 (rows): rows below SPLIT come from a, the others from b, both NV*V columns wide.  The source is chosen
// by selecting the address, not by branching: every lane issues exactly one load per vector.
template <int DT, int V, int NVL, int L, int NV, int RAGGED, int AXIS, long SPLIT, long CB>
FS_DEV void fs_load_row_concat(float (&dst)[NVL * V], const void* a, const void* b, long row, int lir, int vbase) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) {
    int vi = vbase + j * L + lir;
    if (RAGGED) vi = vi < NV ? vi : NV - 1;
    const long col = (long)vi * V;
    const bool first = AXIS == 1 ? col < SPLIT : row < SPLIT;
    const long idx = AXIS == 1 ? (first ? row * SPLIT + col : row * CB + (col - SPLIT)) : (first ? row : row - SPLIT) * ((long)NV * V) + col;
    fs_load_vec<DT, V>(&dst[j * V], first ? a : b, idx);
  }
}

template <int DT, int V, int NVL, int L, int NV, int RAGGED, bool NT = false>
FS_DEV void fs_store_row_vec(const float (&src)[NVL * V], void* base, long row_elem0, int lir, int vbase, bool rok, int j) {
  const int vi = vbase + j * L + lir;
  const bool ok = rok && (!RAGGED || vi < NV);
  if (ok) fs_store_vec<DT, V, NT, fs_overlap(RAGGED) != 0>(&src[j * V], base, row_elem0 + (fs_overlap(RAGGED) != 0 ? fs_col_of<V, NV, RAGGED>(vi) : (long)vi * V));
}
template <int DT, int V, int NVL, int L, int NV, int RAGGED, bool NT = false>
FS_DEV void fs_store_row(const float (&src)[NVL * V], void* base, long row_elem0, int lir, int vbase, bool rok) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) fs_store_row_vec<DT, V, NVL, L, NV, RAGGED, NT>(src, base, row_elem0, lir, vbase, rok, j);
}

// Rows whose ends lie inside cache lines, held in pieces of whole lines: a lane's slice begins at the line in which its row begins, so
// `lead` elements (less than LEAD, a line of the narrowest tensor) before the row and some behind it belong to its neighbours.  Element i
// of the slice, counted from that line, is one of the row's C when lead <= i < lead + C: only those are reduced and stored.  What bounds such
// rows are lines moved twice, by two accesses of a wavefront and by two rows: a copy of fp32 [2048,50001] takes 156 us in vectors that begin
// with the row, 141 in whole lines.  j is a constant wherever these are called: vectors that lie inside every row cost nothing.
template <int V, int L, int C, int LEAD> FS_DEV bool fs_lead_inside(int lead, int lir, int j, int k) {
  const int i = (j * L + lir) * V + (C % V ? k : 0);  // (rows of whole vectors begin and end between two of them)
  return (j * L * V >= LEAD - 1 || i >= lead) && ((j + 1) * L * V <= C || i < lead + C);
}
// Where vector j of the lane's slice is read from.  Behind the row: its last vector again.  Behind the tensor, whose last row may end inside a
// vector: its last V elements, so fs_lead_shift takes the lane's own to their places (a load in a branch would be waited for).
template <int V, int L, int C> FS_DEV int fs_lead_at(int lead, int lir, bool last_row, int j) {
  int i = (j * L + lir) * V;
  if ((j + 1) * L * V > C) {
    const int last = (lead + C - 1) & ~(V - 1);
    i = i < last ? i : last;
    if (C % V != 0 && last_row && i > lead + C - V) i = lead + C - V;
  }
  return i;
}
template <int DT, int V, int L, int C, bool NT>
FS_DEV typename fs_vec<typename fs_elem<DT>::type, V>::type fs_lead_load_raw(const void* base, long row0, int lead, int lir, bool last_row, int j) {
  return fs_load_raw<DT, V, NT, true>(base, row0 - lead + fs_lead_at<V, L, C>(lead, lir, last_row, j));
}
template <int V, int B, int E> FS_DEV void fs_shift_down(float (&v)[E], int at, int d) {  // v[at + k] = v[at + k + d], 0 <= d < V
#pragma unroll
  for (int k = 0; k + B < V; ++k) {
    const float stays = v[at + k], comes = v[at + k + B];  // (values: a choice between elements would be one between their addresses)
    v[at + k] = d & B ? comes : stays;
  }
  if constexpr (2 * B < V) fs_shift_down<V, 2 * B>(v, at, d);
}
template <int V, int NVL, int L, int C> FS_DEV void fs_lead_shift(float (&v)[NVL * V], int lead, int lir) {
  if (C % V == 0) return;
  const int from = lead + C - V, d = ((lead + C - 1) & ~(V - 1)) - from;  // (lanes behind the row hold nothing that counts: any order will do)
#pragma unroll
  for (int j = C / (L * V); j < NVL; ++j) fs_shift_down<V, 1>(v, j * V, (j * L + lir) * V > from ? d : 0);
}
template <int DT, int V, int NVL, int L, int C, bool NT>
FS_DEV void fs_lead_load_row(float (&dst)[NVL * V], const void* base, long row0, int lead, int lir, bool last_row) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) {
    const auto raw = fs_lead_load_raw<DT, V, L, C, NT>(base, row0, lead, lir, last_row, j);
#pragma unroll
    for (int k = 0; k < V; ++k) dst[j * V + k] = fs_to_f32<DT>(raw[k]);
  }
  if (last_row) fs_lead_shift<V, NVL, L, C>(dst, lead, lir);
}
template <int DT, int V, int NVL, int L, int C, int LEAD, bool NT>
FS_DEV void fs_lead_store_row_vec(const float (&src)[NVL * V], void* base, long row0, int lead, int lir, bool rok, int j) {
  const int i = (j * L + lir) * V;
  if (!rok) return;
  if ((j * L * V >= LEAD - 1 || i >= lead) && ((j + 1) * L * V <= C || i + V <= lead + C)) {
    fs_store_vec<DT, V, NT>(&src[j * V], base, row0 - lead + i);
  } else if (C % V != 0) {
#pragma unroll
    for (int k = 0; k < V; ++k)
      if (i + k >= lead && i + k < lead + C) static_cast<typename fs_elem<DT>::type*>(base)[row0 - lead + i + k] = fs_from_f32<DT>(src[j * V + k]);
  }
}
template <int DT, int V, int NVL, int L, int C, int LEAD, bool NT>
FS_DEV void fs_lead_store_row(const float (&src)[NVL * V], void* base, long row0, int lead, int lir, bool rok) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) fs_lead_store_row_vec<DT, V, NVL, L, C, LEAD, NT>(src, base, row0, lead, lir, rok, j);
}

// One chunk of a row kept in LDS in the tensor's own dtype (a kernel that walks a row once per stage reads the
// chunk from memory in the first stage only).  The lane's vector j sits at chunk-local vector j*L + lir: consecutive
// lanes touch consecutive 16-byte pieces.  What is written is what fs_load_row delivered (fp32 values that came from
// the dtype convert back to it exactly), clamped duplicates included, so a later read sees the very same registers.
template <int DT, int V, int NVL, int L> FS_DEV void fs_stage_row_chunk(void* lds_chunk, const float (&src)[NVL * V], int lir) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) fs_store_vec<DT, V>(&src[j * V], lds_chunk, (long)(j * L + lir) * V);
}
// fs_load_row and fs_stage_row_chunk in one: the vectors go to LDS as they came from memory (when `stage`), so nothing is
// spent on converting fp32 registers back to the dtype, and what a later stage reads back is the same bytes.
template <int DT, int V, int NVL, int L, int NV, int RAGGED, bool NT = false>
FS_DEV void fs_load_row_staging(float (&dst)[NVL * V], const void* base, long row_elem0, int lir, int vbase, void* lds_chunk, bool stage) {
  typedef typename fs_elem<DT>::type T;
  typedef typename fs_vec<T, V>::type VT;
#pragma unroll
  for (int j = 0; j < NVL; ++j) {
    const VT raw = fs_load_raw<DT, V, NT, fs_overlap(RAGGED) != 0>(base, row_elem0 + fs_col_of<V, NV, RAGGED>(vbase + j * L + lir));
    if (stage) *reinterpret_cast<VT*>(static_cast<T*>(lds_chunk) + (long)(j * L + lir) * V) = raw;
    if constexpr (V == 1) {
      dst[j] = fs_to_f32<DT>(raw);
    } else {
#pragma unroll
      for (int k = 0; k < V; ++k) dst[j * V + k] = fs_to_f32<DT>(raw[k]);
    }
  }
}
template <int DT, int V, int NVL, int L> FS_DEV void fs_load_row_chunk_lds(float (&dst)[NVL * V], const void* lds_chunk, int lir) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) fs_load_vec<DT, V>(&dst[j * V], lds_chunk, (long)(j * L + lir) * V);
}

// The next rows on their way while rows are worked on: the first JL vectors of a lane go from memory to LDS without passing
// registers, the rest waits in registers of their own.  A wavefront reads back what it asked for itself, 64 lanes x 16 bytes that
// follow each other, so only its own counter of outstanding accesses orders the two; the compiler does not see that dependence, the
// waits are spelled out (fs_wait_vm).  Rows that start inside a vector (UA; whole vectors of one row to a workgroup) are asked for
// in 4-byte pieces.
#define FS_LDS_BYTES(p) ((__attribute__((address_space(3))) void*)(p))
#define FS_GLOBAL_BYTES(p) ((const __attribute__((address_space(1))) void*)(p))
template <int DT, int V, int L, int NV, int RAGGED, int WG, int JL, bool UA, bool NT> FS_DEV void fs_row_ask(fs_u8* lds, const void* base, long row_elem0, int lir, int tid) {
  typedef typename fs_elem<DT>::type T;
  static_assert(V * sizeof(T) == 16 && WG % 64 == 0 && (!UA || (sizeof(T) == 4 && L == WG)), "16 bytes to a lane");
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
  for (int j = 0; j < JL; ++j) {
    fs_u8* const to = lds + (j * (WG / 64) + wave) * 1024;
    if constexpr (UA) {
      const T* const from = static_cast<const T*>(base) + row_elem0 + (j * L + wave * 64) * V + (lir & 63);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (NT) __builtin_amdgcn_global_load_lds(FS_GLOBAL_BYTES(from + q * 64), FS_LDS_BYTES(to + q * 256), 4, 0, 2);
        else __builtin_amdgcn_global_load_lds(FS_GLOBAL_BYTES(from + q * 64), FS_LDS_BYTES(to + q * 256), 4, 0, 0);
      }
    } else {
      const T* const from = static_cast<const T*>(base) + row_elem0 + fs_col_of<V, NV, RAGGED>(j * L + lir);
      if constexpr (NT) __builtin_amdgcn_global_load_lds(FS_GLOBAL_BYTES(from), FS_LDS_BYTES(to), 16, 0, 2);
      else __builtin_amdgcn_global_load_lds(FS_GLOBAL_BYTES(from), FS_LDS_BYTES(to), 16, 0, 0);
    }
  }
}
template <int DT, int V, int NVL, int WG, int JL> FS_DEV void fs_row_take(float (&dst)[NVL * V], const fs_u8* lds, int tid) {
#pragma unroll
  for (int j = 0; j < JL; ++j) fs_load_vec<DT, V>(&dst[j * V], lds + (j * (WG / 64) + (tid >> 6)) * 1024, (long)(tid & 63) * V);
}
// waits until at most N of this wavefront's accesses to global memory are outstanding (they complete in order)
template <int N> FS_DEV void fs_wait_vm() {
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | 0xf70 | (N >> 4) << 14);
  asm volatile("" : : : "memory");
}
FS_DEV void fs_wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }
// fs_lds_barrier where a row is on its way to LDS: a fence would wait for it
FS_DEV void fs_lds_barrier_ahead() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

// Workgroups go to the 8 XCDs in turn.  Workgroup b of n takes this place among the rows, so that M neighbours run on one XCD: the lines that
// they share, at the ends of their rows or in a transposed tensor, meet in its L2.
template <int M> FS_DEV int fs_xcd_place(int b, int n) {
  const int r = b % (8 * M), first = b - r;
  return first + 8 * M <= n ? first + r % 8 * M + r / 8 : b;
}

// Transposing store of the lane's slice of row `row` of a [R,C] value into a [C,R] tensor.
template <int DT, int V, int NVL, int L, int NV, int RAGGED>
FS_DEV void fs_store_row_transposed(const float (&src)[NVL * V], void* base, long R, long row, int lir, int vbase, bool rok) {
  typedef typename fs_elem<DT>::type T;
#pragma unroll
  for (int j = 0; j < NVL; ++j) {
    const int vi = vbase + j * L + lir;
    const bool ok = rok && (!RAGGED || vi < NV);
    const int col = (int)fs_col_of<V, NV, RAGGED>(vi);
    if (ok) {
#pragma unroll
      for (int k = 0; k < V; ++k) static_cast<T*>(base)[(long)(col + k) * R + row] = fs_from_f32<DT>(src[j * V + k]);
    }
  }
}

// Per-column vectors ([1,C] operands) shared by every row of the workgroup are staged once in
// LDS as fp32: one cooperative pass of the whole workgroup instead of every wavefront pulling
// its own copy through the vector cache (which is the narrower path: 64 B/clk against 128).
// The staged copy is laid out in the order lanes read it: the 4-float chunk q of vector
// vi = j*L + lir sits at chunk index (j*(V/4) + q)*L + lir, so a 128-bit LDS read by
// consecutive lanes touches consecutive 16-byte chunks (no bank conflicts).  The staging pass
// walks the LDS positions in order (thread t writes position t, t + WG, ...), so its 128-bit
// writes are conflict-free too; what it reads from memory is then 16-byte pieces V*4 bytes
// apart, a few KB from L2 once per workgroup.  SLOT = NVL*L*V floats per vector.
template <int DT, int V, int L, int C, int WG> FS_DEV void fs_stage_rowvec(float* lds, const void* src) {
  if constexpr (V % 4 == 0) {
    constexpr int Q = V / 4, NVS = (C + V - 1) / V;  // 16-byte pieces per vector access, vectors per row
    constexpr int P = ((NVS + L - 1) / L) * Q * L;  // LDS positions (16-byte pieces) of the slot, tail included
    for (int p = (int)threadIdx.x; p < P; p += WG) {
      const int l = p % L, jq = p / L, j = jq / Q, q = jq % Q, vi = j * L + l;
      if (vi >= NVS) continue;
      float tmp[4];
      fs_load_vec<DT, 4, false, C % V != 0>(tmp, src, fs_vec_col<V, C>(vi) + q * 4);
      typedef float f4 __attribute__((ext_vector_type(4)));
      f4 t4;
#pragma unroll
      for (int k = 0; k < 4; ++k) t4[k] = tmp[k];
      *reinterpret_cast<f4*>(lds + p * 4) = t4;  // one 128-bit LDS store, consecutive threads to consecutive pieces
    }
  } else {
    for (int i = (int)threadIdx.x; i < C; i += WG) {
      float tmp[1];
      fs_load_vec<DT, 1>(tmp, src, i);
      lds[i] = tmp[0];
    }
  }
}
// The same for the sum (or difference) of two per-column vectors: +-a +- b is formed once, here,
// instead of once per element of every row.
template <int DTA, int DTB, bool NEGA, bool NEGB, int V, int L, int C, int WG> FS_DEV void fs_stage_rowvec_sum(float* lds, const void* a, const void* b) {
  if constexpr (V % 4 == 0) {
    constexpr int Q = V / 4, NVS = (C + V - 1) / V;
    constexpr int P = ((NVS + L - 1) / L) * Q * L;
    for (int p = (int)threadIdx.x; p < P; p += WG) {
      const int l = p % L, jq = p / L, j = jq / Q, q = jq % Q, vi = j * L + l;
      if (vi >= NVS) continue;
      float ta[4], tb[4];
      fs_load_vec<DTA, 4, false, C % V != 0>(ta, a, fs_vec_col<V, C>(vi) + q * 4);
      fs_load_vec<DTB, 4, false, C % V != 0>(tb, b, fs_vec_col<V, C>(vi) + q * 4);
      typedef float f4 __attribute__((ext_vector_type(4)));
      f4 t4;
#pragma unroll
      for (int k = 0; k < 4; ++k) t4[k] = (NEGA ? -ta[k] : ta[k]) + (NEGB ? -tb[k] : tb[k]);
      *reinterpret_cast<f4*>(lds + p * 4) = t4;
    }
  } else {
    for (int i = (int)threadIdx.x; i < C; i += WG) {
      float ta[1], tb[1];
      fs_load_vec<DTA, 1>(ta, a, i);
      fs_load_vec<DTB, 1>(tb, b, i);
      lds[i] = (NEGA ? -ta[0] : ta[0]) + (NEGB ? -tb[0] : tb[0]);
    }
  }
}
// The lane's slice of a staged vector (same element ownership as fs_load_row).
template <int V, int NVL, int L, int NV, int RAGGED>
FS_DEV void fs_read_staged_vec(float (&dst)[NVL * V], const float* lds, int lir, int j) {
  if constexpr (V % 4 == 0) {
    constexpr int Q = V / 4;
    typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const f4 x = *reinterpret_cast<const f4*>(lds + ((j * Q + q) * L + lir) * 4);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float xk = x[k];
        dst[j * V + q * 4 + k] = xk;
      }
    }
  } else {
    const int vi = j * L + lir;
    const int col = RAGGED ? fs_vec_col<V, fs_cols(V, NV, RAGGED)>(vi) : vi * V;
#pragma unroll
    for (int k = 0; k < V; ++k) dst[j * V + k] = lds[col + k];
  }
}
template <int V, int NVL, int L, int NV, int RAGGED>
FS_DEV void fs_read_staged(float (&dst)[NVL * V], const float* lds, int lir) {
#pragma unroll
  for (int j = 0; j < NVL; ++j) fs_read_staged_vec<V, NVL, L, NV, RAGGED>(dst, lds, lir, j);
}

template <int DT> FS_DEV void fs_store1_fwd(void* base, long i, float x) {
  static_cast<typename fs_elem<DT>::type*>(base)[i] = fs_from_f32<DT>(x);
}

// Transposing store of a G x TC tile (one row per row-group, in registers) through a padded LDS
// tile: rows tile_row0 .. tile_row0+G-1 and columns col0 .. col0+TC-1 of the [R,CTOT] value become
// G consecutive elements of each of TC rows of the [CTOT,R] output, so global stores are runs of G
// elements instead of single elements R apart.  LDS holds TC x (G+1) floats (the +1 keeps the
// column-wise writes of the row-groups of a wavefront on distinct banks).  vbase = col0 / V is the
// tile's first vector in the row.  Every lane of the workgroup must call it.
template <int DT, int V, int NVL, int L, int NV, int RAGGED, int WG, int TC, bool NT = false>
FS_DEV void fs_store_tile_transposed(const float (&src)[NVL * V], float* lds, void* base, long R, long tile_row0, int lir, int rg, int vbase) {
  constexpr int G = WG / L, P = G + 1, C = fs_cols(V, NV, RAGGED);
  __syncthreads();  // the tile may still be read by its previous use
#pragma unroll
  for (int j = 0; j < NVL; ++j) {
    const int vi = j * L + lir;
    if constexpr (fs_overlap(RAGGED) != 0) {  // (owned elements only: the repeated ones may belong to the tile before)
      const int skip = fs_vec_skip<V, C>(vbase + vi);
#pragma unroll
      for (int k = 0; k < V; ++k)
        if (k >= skip) lds[(vi * V + k - skip) * P + rg] = src[j * V + k];
    } else if (!RAGGED || vbase + vi < NV) {
#pragma unroll
      for (int k = 0; k < V; ++k) lds[(vi * V + k) * P + rg] = src[j * V + k];
    }
  }
  __syncthreads();
  // a lane stores 16 bytes of a run: 4 floats, 8 bf16, 16 bytes of u8 (fewer where G does not divide)
  constexpr int WANT = 16 / (int)sizeof(typename fs_elem<DT>::type);
  constexpr int RUN = (G % WANT == 0) ? WANT : (G % 4 == 0) ? 4 : 1;
  constexpr int RPC = G / RUN;  // runs per output row
  const typename fs_col_index<C>::type col0 = (typename fs_col_index<C>::type)vbase * V;
  for (int i = (int)threadIdx.x; i < TC * RPC; i += WG) {
    const int c = i / RPC, g0 = (i % RPC) * RUN;
    const long r = tile_row0 + g0;
    if (col0 + c >= C) continue;
    float tmp[RUN];
#pragma unroll
    for (int q = 0; q < RUN; ++q) tmp[q] = lds[c * P + g0 + q];
    const long o = (long)(col0 + c) * R + r;
    if (RUN > 1 && r + RUN - 1 < R) {  // (runs start at any multiple of the element size when R is no multiple of RUN)
      fs_store_vec<DT, RUN, NT, true>(tmp, base, o);
    } else {
#pragma unroll
      for (int q = 0; q < RUN; ++q)
        if (r + q < R) fs_store1_fwd<DT>(base, o + q, tmp[q]);
    }
  }
}

template <int DT> FS_DEV float fs_load1(const void* base, long i) {
  return fs_to_f32<DT>(static_cast<const typename fs_elem<DT>::type*>(base)[i]);
}
template <int DT> FS_DEV void fs_store1(void* base, long i, float x) {
  static_cast<typename fs_elem<DT>::type*>(base)[i] = fs_from_f32<DT>(x);
}

// ------------------------------------------------------------------------------------------
// reductions
// ------------------------------------------------------------------------------------------
template <int KIND> FS_DEV float fs_red_identity() {
  return KIND == FS_K_MAX ? -__builtin_inff() : KIND == FS_K_MIN ? __builtin_inff() : 0.0f;
}
template <int KIND> FS_DEV float fs_red_op(float a, float b) {
  return KIND == FS_K_MAX ? __builtin_fmaxf(a, b) : KIND == FS_K_MIN ? __builtin_fminf(a, b) : a + b;
}

// Serial reduction of the lane's own E elements (masked columns contribute the identity).
template <int KIND, int V, int NVL, int L, int NV, int RAGGED>
FS_DEV float fs_lane_reduce(const float (&v)[NVL * V], int lir, int vbase = 0) {
  float acc = fs_red_identity<KIND>();
#pragma unroll
  for (int j = 0; j < NVL; ++j) {
    const int vi = vbase + j * L + lir;
#pragma unroll
    for (int k = 0; k < V; ++k) acc = fs_red_op<KIND>(acc, fs_owned<V, NV, RAGGED>(vi, k) ? v[j * V + k] : fs_red_identity<KIND>());
  }
  return acc;
}

template <int KIND, int V, int NVL, int L, int C, int LEAD> FS_DEV float fs_lead_lane_reduce(const float (&v)[NVL * V], int lead, int lir) {
  float acc = fs_red_identity<KIND>();
#pragma unroll
  for (int j = 0; j < NVL; ++j) {
#pragma unroll
    for (int k = 0; k < V; ++k) acc = fs_red_op<KIND>(acc, fs_lead_inside<V, L, C, LEAD>(lead, lir, j, k) ? v[j * V + k] : fs_red_identity<KIND>());
  }
  return acc;
}

template <int CTRL> FS_DEV float fs_dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}

// DPP permute that only writes the rows of 16 lanes selected by ROW_MASK; the others receive `old`.
template <int CTRL, int ROW_MASK> FS_DEV float fs_dpp_rows(float old, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, false));
}

// All-reduce inside aligned segments of W lanes of a wavefront (W = 1,2,4,...,64).  Every
// lane of a segment ends with the same bits.  Steps 1..8 are DPP lane permutes inside a row
// of 16 lanes (quad_perm, row_half_mirror, row_mirror), fused into the arithmetic
// instruction.  Across the four rows of a whole wavefront two row broadcasts (lane 15 of a row
// into the next row, lane 31 into rows 2 and 3) leave the total in lane 63, which is read into a
// scalar register: (r3 op r2) op (r1 op r0), 6 permuting instructions and one v_readlane.  Two
// segments of 32 lanes read their row totals into scalar registers and fold them there.  No LDS
// traffic.
// FIRST = 2 or 4: every FIRST lanes hold the same value, which counts once.
template <int KIND, int W, int FIRST = 1> FS_DEV float fs_segment_allreduce(float v) {
  if constexpr (W >= 2 && FIRST < 2) v = fs_red_op<KIND>(v, fs_dpp<0xB1>(v));   // quad_perm [1,0,3,2]
  if constexpr (W >= 4 && FIRST < 4) v = fs_red_op<KIND>(v, fs_dpp<0x4E>(v));   // quad_perm [2,3,0,1]
  if constexpr (W >= 8) v = fs_red_op<KIND>(v, fs_dpp<0x141>(v));  // row_half_mirror
  if constexpr (W >= 16) v = fs_red_op<KIND>(v, fs_dpp<0x140>(v)); // row_mirror
  if constexpr (W >= 64) {
    const float idn = fs_red_identity<KIND>();                     // (what the rows left out by the mask combine with)
    v = fs_red_op<KIND>(v, fs_dpp_rows<0x142, 0xa>(idn, v));       // row_bcast:15 -> rows 1 and 3
    v = fs_red_op<KIND>(v, fs_dpp_rows<0x143, 0xc>(idn, v));       // row_bcast:31 -> rows 2 and 3
    v = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
  } else if constexpr (W >= 32) {
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    const float lo = fs_red_op<KIND>(r0, r1), hi = fs_red_op<KIND>(r2, r3);
    v = (__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) < 32u) ? lo : hi;
  }
  return v;
}

// Rows that would leave half of their lanes or more idle are spread: a lane takes V of the SP * V elements that it would take alone, and
// its SP - 1 neighbours the rest.  A row reduction gathers them again: each of the SP lanes then reduces all SP * V in their order, as the
// one lane does (the order of a sum is part of its bits).
template <int SP, int V> FS_DEV void fs_gather(float (&dst)[SP * V], const float (&v)[V]) {
  static_assert(SP == 2 || SP == 4, "lanes of a quad");
#pragma unroll
  for (int k = 0; k < V; ++k) {
    if constexpr (SP == 2) {
      dst[k] = fs_dpp<0xA0>(v[k]);      // quad_perm [0,0,2,2]
      dst[V + k] = fs_dpp<0xF5>(v[k]);  // quad_perm [1,1,3,3]
    } else {
      dst[k] = fs_dpp<0x00>(v[k]);
      dst[V + k] = fs_dpp<0x55>(v[k]);
      dst[2 * V + k] = fs_dpp<0xAA>(v[k]);
      dst[3 * V + k] = fs_dpp<0xFF>(v[k]);
    }
  }
}

// Workgroup barrier that orders LDS traffic only: outstanding global loads/stores of the
// streaming body are not waited for.
FS_DEV void fs_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Cross-wave step of a row reduction when a row spans WPR = L/64 wavefronts: wave leaders
// publish their partial in LDS, one barrier, every lane folds the WPR partials in fixed order
// (so all lanes of the row hold identical bits).  `slot` points at this row-group's WPR*K
// floats inside the current ping-pong half; K reductions of one stage share the barrier.
template <int K, int WPR> struct fs_xwave {
  float* slot;
  int wir;     // wave index inside the row
  bool leader; // lane 0 of its wavefront
  FS_DEV void put(int k, float v) const {
    if (leader) slot[wir * K + k] = v;
  }
  // (rows spread over SP times their wavefronts: what one of those would hold first, in the pairs it folds in)
  template <int KIND, int SP = 1> FS_DEV float get(int k) const {
    constexpr int S = SP < WPR ? SP : WPR;
    float acc = 0.0f;
#pragma unroll
    for (int w = 0; w < WPR; w += S) {
      float v = slot[w * K + k];
      if constexpr (S == 2) v = fs_red_op<KIND>(v, slot[(w + 1) * K + k]);
      if constexpr (S == 4) v = fs_red_op<KIND>(fs_red_op<KIND>(slot[(w + 3) * K + k], slot[(w + 2) * K + k]), fs_red_op<KIND>(slot[(w + 1) * K + k], v));
      acc = w == 0 ? v : fs_red_op<KIND>(acc, v);
    }
    return acc;
  }
};

// ------------------------------------------------------------------------------------------
// column reductions: two stages, no atomics on data, bitwise deterministic.
//   stage 1  every lane accumulates its columns over the rows its workgroup visits; the G
//            row-groups of the workgroup are folded through LDS in row-group order.
//   stage 2  the workgroup's partial goes to the workspace; a ticket per fan-in group tells
//            the last arriver to fold that group's partials in index order, and it moves up
//            one level.  The only atomic is the ticket.  The survivor of the top level holds
//            the result.
// The K column reductions of a kernel travel together as one vector of K*C floats, cut into
// chunks of FV floats (FV = 4 when C allows).  Thread t owns chunks t, t+WG, ...; chunk c
// belongs to reduction c / (C/FV) and covers columns (c % (C/FV))*FV onwards.
// ------------------------------------------------------------------------------------------
template <int K, int C, int WG, int FV> struct fs_colfold {
  static constexpr int CH = C / FV;                   // chunks per reduction
  static constexpr int NCH = K * CH;                  // chunks per workgroup partial
  static constexpr int CPT = (NCH + WG - 1) / WG;     // chunks per thread
};

// 4/8/16-byte memory access that is coherent at device scope without fences: the sc1 bit makes a
// store write through to, and a load read from, the level all 8 XCDs share.
typedef fs_u32 fs_u32x2 __attribute__((ext_vector_type(2)));
typedef fs_u32 fs_u32x4 __attribute__((ext_vector_type(4)));
#define FS_AUX_SC1 0x10
FS_DEV __amdgpu_buffer_rsrc_t fs_make_rsrc(const void* base, fs_u32 bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
template <int FV> FS_DEV void fs_load_dev(float (&dst)[FV], __amdgpu_buffer_rsrc_t r, fs_u32 byte_off) {
  if constexpr (FV == 4) {
    // (each element is copied to a scalar first: a bit_cast applied directly to a vector
    // element expression reads element 0 with this compiler)
    const fs_u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, FS_AUX_SC1);
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const fs_u32 w = u[f];
      dst[f] = __builtin_bit_cast(float, w);
    }
  } else if constexpr (FV == 2) {
    const fs_u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, FS_AUX_SC1);
    const fs_u32 w0 = u[0], w1 = u[1];
    dst[0] = __builtin_bit_cast(float, w0);
    dst[1] = __builtin_bit_cast(float, w1);
  } else {
    dst[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, FS_AUX_SC1));
  }
}
template <int FV> FS_DEV void fs_store_dev(const float (&src)[FV], __amdgpu_buffer_rsrc_t r, fs_u32 byte_off) {
  if constexpr (FV == 4) {
    fs_u32x4 u;
#pragma unroll
    for (int f = 0; f < 4; ++f) u[f] = __builtin_bit_cast(fs_u32, src[f]);
    __builtin_amdgcn_raw_buffer_store_b128(u, r, byte_off, 0, FS_AUX_SC1);
  } else if constexpr (FV == 2) {
    fs_u32x2 u;
    u[0] = __builtin_bit_cast(fs_u32, src[0]);
    u[1] = __builtin_bit_cast(fs_u32, src[1]);
    __builtin_amdgcn_raw_buffer_store_b64(u, r, byte_off, 0, FS_AUX_SC1);
  } else {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(fs_u32, src[0]), r, byte_off, 0, FS_AUX_SC1);
  }
}

// Vectors of V elements that stay in registers as they came from memory (kernels that join column reductions with what needs
// their results hold several rows of a tile in a lane): 32-bit words, read and written through a buffer descriptor whose size
// is the tensor's.  Rows beyond the tensor need no clamp and no branch: they lie beyond the descriptor, where loads give zeros
// and stores are dropped.  One 32-bit offset per lane serves all rows (pairs of 64-bit addresses of 16 rows cost 32 registers).
template <int DT, int V> struct fs_words {
  static constexpr int bytes = V * (int)sizeof(typename fs_elem<DT>::type), n = bytes >= 4 ? bytes / 4 : 1;
  typedef fs_u32 type[n];
};
#define FS_AUX_NT 0x2
template <int DT, int V, bool NT> FS_DEV void fs_load_words(typename fs_words<DT, V>::type& w, __amdgpu_buffer_rsrc_t r, fs_u32 elem) {
  constexpr int BYTES = V * (int)sizeof(typename fs_elem<DT>::type), AUX = NT ? FS_AUX_NT : 0;
  const fs_u32 off = elem * (fs_u32)sizeof(typename fs_elem<DT>::type);
  if constexpr (BYTES == 16) {
    const fs_u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX);
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = u[k];
  } else if constexpr (BYTES == 8) {
    const fs_u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
    w[0] = u[0], w[1] = u[1];
  } else if constexpr (BYTES == 4) {
    w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, AUX);
  } else if constexpr (BYTES == 2) {
    w[0] = (fs_u16)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, AUX);
  } else {
    w[0] = (fs_u8)__builtin_amdgcn_raw_buffer_load_b8(r, off, 0, AUX);
  }
}
template <int DT, int V> FS_DEV void fs_unpack_words(float (&dst)[V], const typename fs_words<DT, V>::type& w) {
#pragma unroll
  for (int k = 0; k < V; ++k) {
    if constexpr (DT == FS_DT_F32) dst[k] = __builtin_bit_cast(float, w[k]);
    else if constexpr (DT == FS_DT_BF16) dst[k] = __builtin_bit_cast(float, k % 2 ? w[k / 2] & 0xffff0000u : w[k / 2] << 16);
    else dst[k] = fs_to_f32<DT>((fs_u8)(w[k / 4] >> (8 * (k % 4))));
  }
}
template <int DT, int V, bool NT> FS_DEV void fs_store_words(const float (&src)[V], __amdgpu_buffer_rsrc_t r, fs_u32 elem) {
  constexpr int ES = (int)sizeof(typename fs_elem<DT>::type), BYTES = V * ES, AUX = NT ? FS_AUX_NT : 0;
  const fs_u32 off = elem * (fs_u32)ES;
  fs_u32 w[fs_words<DT, V>::n] = {};
#pragma unroll
  for (int k = 0; k < V; ++k) {
    if constexpr (DT == FS_DT_F32) w[k] = __builtin_bit_cast(fs_u32, src[k]);
    else w[k * ES / 4] |= (fs_u32)fs_from_f32<DT>(src[k]) << (8 * (k * ES % 4));
  }
  if constexpr (BYTES == 16) {
    fs_u32x4 u;
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = w[k];
    __builtin_amdgcn_raw_buffer_store_b128(u, r, off, 0, AUX);
  } else if constexpr (BYTES == 8) {
    fs_u32x2 u;
    u[0] = w[0], u[1] = w[1];
    __builtin_amdgcn_raw_buffer_store_b64(u, r, off, 0, AUX);
  } else if constexpr (BYTES == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(w[0], r, off, 0, AUX);
  } else if constexpr (BYTES == 2) {
    __builtin_amdgcn_raw_buffer_store_b16((fs_u16)w[0], r, off, 0, AUX);
  } else {
    __builtin_amdgcn_raw_buffer_store_b8((fs_u8)w[0], r, off, 0, AUX);
  }
}
// an index the compiler does not recognise as the one it computed before (so that a pass over the rows recomputes its offsets
// instead of keeping those of the pass before in registers)
FS_DEV fs_u32 fs_opaque(fs_u32 x) {
  asm volatile("" : "+v"(x));
  return x;
}

FS_DEV int fs_lane_id() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }
// value of lane (lane ^ mask) of the same wavefront (LDS crossbar, no LDS memory)
FS_DEV float fs_shfl_xor(float v, int mask) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((fs_lane_id() ^ mask) << 2, __builtin_bit_cast(int, v)));
}

// v[0] of N values, folded in pairs (a chain of eight large sums loses half a bit more than the pairs)
template <int N, typename OP> FS_DEV void fs_pairs(float (&v)[N], OP op) {
#pragma unroll
  for (int s = 1; s < N; s *= 2)
#pragma unroll
    for (int i = 0; i + s < N; i += 2 * s) v[i] = op(v[i], v[i + s]);
}

// The value of lane (lane ^ M) of the same wavefront for M of 1 to 8, in one or two DPP moves.
template <int M> FS_DEV float fs_lane_xor(float v) {
  static_assert(M == 1 || M == 2 || M == 4 || M == 8, "inside a row of 16 lanes");
  if constexpr (M == 1) return fs_dpp<0xB1>(v);        // quad_perm [1,0,3,2]
  else if constexpr (M == 2) return fs_dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  else if constexpr (M == 8) return fs_dpp<0x128>(v);  // row_ror:8
  else {
    const int x = __builtin_bit_cast(int, v), up = __builtin_amdgcn_update_dpp(x, x, 0x104, 0xf, 0x5, false);  // row_shl:4 into lanes 0-3 and 8-11
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(up, x, 0x114, 0xf, 0xa, false));             // row_shr:4 into the others
  }
}
// One step of fs_scatter_rows: the N values of the lanes of a wavefront that differ in bit M are folded, and each of the two keeps half
// of the results (of an odd number both keep the last).  col[i] tells which value v[i] is.
template <int KIND, int M, int N> FS_DEV void fs_scatter_step(float* v, int* col) {
  constexpr int H = N / 2;
  const bool upper = (fs_lane_id() & M) != 0;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    // (values, not elements of the array, in the conditions: those would be a choice of addresses, and the array memory)
    const float a = v[i], b = v[i + H];
    const int ca = col[i], cb = col[i + H];
    if constexpr (M >= 16) {  // gfx950 exchanges halves (rows) of two registers in one instruction
      const auto s = M == 32 ? __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(fs_u32, a), __builtin_bit_cast(fs_u32, b), false, false)
                             : __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(fs_u32, a), __builtin_bit_cast(fs_u32, b), false, false);
      const fs_u32 s0 = s[0], s1 = s[1];
      v[i] = fs_red_op<KIND>(__builtin_bit_cast(float, s0), __builtin_bit_cast(float, s1));
    } else {
      const float keep = upper ? b : a, give = upper ? a : b;
      v[i] = fs_red_op<KIND>(keep, fs_lane_xor<M>(give));
    }
    col[i] = upper ? cb : ca;
  }
  if constexpr (N % 2 != 0) {
    if constexpr (M >= 16) {
      const fs_u32 a = __builtin_bit_cast(fs_u32, v[N - 1]);
      const auto s = M == 32 ? __builtin_amdgcn_permlane32_swap(a, a, false, false) : __builtin_amdgcn_permlane16_swap(a, a, false, false);
      const fs_u32 s0 = s[0], s1 = s[1];
      v[H] = fs_red_op<KIND>(__builtin_bit_cast(float, s0), __builtin_bit_cast(float, s1));
    } else {
      v[H] = fs_red_op<KIND>(v[N - 1], fs_lane_xor<M>(v[N - 1]));
    }
    col[H] = col[N - 1];
  }
}
constexpr int fs_scatter_left(int e, int l) { return l < 64 ? fs_scatter_left((e + 1) / 2, l * 2) : e; }
// The 64 / L row-groups of a wavefront folded into one another: of the E values of a lane fs_scatter_left are left, another part in each
// row-group.  (To leave all of them in all lanes takes log2(64 / L) times as many steps, each a trip through the LDS crossbar: the fold inside
// workgroups of 8 lanes a row took 3.7 us for two sums.  LayerNorm backward fp32 [40077,112] 17.8 -> 16.4 us, [16384,256] 15.4 -> 14.3, column sums +
// row norms [65536,512] 25.7 -> 25.2, [65536,64] 12.5 -> 10.3, [5728,256] 6.8 -> 5.6, batch normalisation [352,5824] 4.8 -> 4.5.)
template <int KIND, int L, int E> FS_DEV void fs_scatter_rows(float (&v)[E], int (&col)[E]) {
#pragma unroll
  for (int e = 0; e < E; ++e) col[e] = e;
  if constexpr (L <= 32) fs_scatter_step<KIND, 32, E>(v, col);
  constexpr int E1 = (E + 1) / 2, E2 = (E1 + 1) / 2, E3 = (E2 + 1) / 2, E4 = (E3 + 1) / 2, E5 = (E4 + 1) / 2;
  if constexpr (L <= 16) fs_scatter_step<KIND, 16, E1>(v, col);
  if constexpr (L <= 8) fs_scatter_step<KIND, 8, E2>(v, col);
  if constexpr (L <= 4) fs_scatter_step<KIND, 4, E3>(v, col);
  if constexpr (L <= 2) fs_scatter_step<KIND, 2, E4>(v, col);
  if constexpr (L <= 1) fs_scatter_step<KIND, 1, E5>(v, col);
}

// Stage 1, in-workgroup fold of reduction number KIDX.  acc: the lane's per-column accumulators
// in the row layout.  Fills the chunks of `vals` that belong to reduction KIDX.  When several
// row-groups share a wavefront (L < 64) they are folded inside the wavefront first (lanes l,
// l+L, l+2L, ... own the same columns; fs_scatter_rows), so the LDS area holds one row per wavefront (GL = WG/64
// rows), not one per row-group.  The C columns go through the area PC columns at a time (PC a
// multiple of 8, or C itself): wide rows need no more LDS than narrow ones, only more barriers.
// CT columns are in the row, C in the fold (one column tile, or the row rounded up to whole 16-byte chunks: columns beyond the
// row hold repeated or unwritten values, which fold to something that is not stored).
// FEW: a loop over the LDS rows that keeps eight of them in registers at a time (kernels that hold their rows across the fold).
template <int KIND, int KIDX, int K, int V, int NVL, int L, int CT, int C, int WG, int FV, int PC, bool FEW = false, int CPT>
FS_DEV void fs_colred_fold_wg(const float (&acc_in)[NVL * V], float (&vals)[CPT][FV], float* lds /* GL*PC floats */, int lir, int rg, int vbase) {
  typedef fs_colfold<K, C, WG, FV> S;
  static_assert(CPT == S::CPT, "chunks per thread");
  static_assert(PC == C || PC % 8 == 0, "piece width");
  constexpr int GL = L < 64 ? WG / 64 : WG / L;
  constexpr int E = NVL * V, LEFT = fs_scatter_left(E, L);
  float acc[E];
  int val[E];  // which of the lane's values acc[i] is
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = acc_in[e], val[e] = e;
  if constexpr (L < 64) fs_scatter_rows<KIND, L, E>(acc, val);
  const int slot = L < 64 ? (int)threadIdx.x / 64 : rg;
  if constexpr (PC >= C) {  // the whole row at once
    __syncthreads();  // the LDS area may still be read by the previous fold
    if constexpr (L < 64) {
#pragma unroll
      for (int i = 0; i < LEFT; ++i) {
        const int vi = val[i] / V * L + lir, k = val[i] % V, skip = CT % V != 0 ? fs_vec_skip<V, CT>(vbase + vi) : 0;
        if (CT % V != 0 ? k >= skip : vi < C / V) lds[slot * C + vi * V + k - skip] = acc[i];
      }
    } else {  // (whole vectors)
#pragma unroll
      for (int j = 0; j < NVL; ++j) {
        const int vi = j * L + lir;
        if constexpr (CT % V != 0) {
          const int skip = fs_vec_skip<V, CT>(vbase + vi);
#pragma unroll
          for (int k = 0; k < V; ++k)
            if (k >= skip) lds[slot * C + vi * V + k - skip] = acc[j * V + k];
        } else if (vi < C / V) {
#pragma unroll
          for (int k = 0; k < V; ++k) lds[slot * C + vi * V + k] = acc[j * V + k];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < S::CPT; ++i) {
      const int c = (int)threadIdx.x + i * WG;
      if (c >= KIDX * S::CH && c < (KIDX + 1) * S::CH) {
        const int col0 = (c - KIDX * S::CH) * FV;
        if constexpr (FEW) {
#pragma unroll
          for (int f = 0; f < FV; ++f) {
            float a = 0.0f;
            for (int g0 = 0; g0 < GL; g0 += 8) {
              float v[8];
#pragma unroll
              for (int u = 0; u < 8; ++u) v[u] = g0 + u < GL ? lds[(g0 + u) * C + col0 + f] : fs_red_identity<KIND>();
              fs_pairs<8>(v, [](float x, float y) { return fs_red_op<KIND>(x, y); });
              a = g0 == 0 ? v[0] : fs_red_op<KIND>(a, v[0]);
            }
            vals[i][f] = a;
          }
          continue;
        }
#pragma unroll
        for (int f = 0; f < FV; ++f) {
          float a = lds[col0 + f];
          for (int g = 1; g < GL; ++g) a = fs_red_op<KIND>(a, lds[g * C + col0 + f]);
          vals[i][f] = a;
        }
      }
    }
    return;
  }
  for (int p0 = 0; p0 < C; p0 += PC) {
    __syncthreads();  // the LDS area may still be read by the previous piece or fold
    if constexpr (L < 64) {
#pragma unroll
      for (int i = 0; i < LEFT; ++i) {
        const int vi = val[i] / V * L + lir, k = val[i] % V, skip = CT % V != 0 ? fs_vec_skip<V, CT>(vbase + vi) : 0, col = vi * V + k - skip - p0;
        if ((CT % V != 0 ? k >= skip : vi < C / V) && col >= 0 && col < PC) lds[slot * PC + col] = acc[i];
      }
    } else {
#pragma unroll
      for (int j = 0; j < NVL; ++j) {
        const int vi = j * L + lir;
        if constexpr (CT % V != 0) {
          const int skip = fs_vec_skip<V, CT>(vbase + vi), col = vi * V - skip - p0;
#pragma unroll
          for (int k = 0; k < V; ++k)
            if (k >= skip && col + k >= 0 && col + k < PC) lds[slot * PC + col + k] = acc[j * V + k];
        } else {
          const int col = vi * V - p0;
          if (vi < C / V && col >= 0 && col < PC) {
#pragma unroll
            for (int k = 0; k < V; ++k) lds[slot * PC + col + k] = acc[j * V + k];
          }
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < S::CPT; ++i) {
      const int c = (int)threadIdx.x + i * WG;
      const int col0 = (c - KIDX * S::CH) * FV - p0;
      if (c >= KIDX * S::CH && c < (KIDX + 1) * S::CH && col0 >= 0 && col0 < PC) {
#pragma unroll
        for (int f = 0; f < FV; ++f) {
          float a = lds[col0 + f];
          for (int g = 1; g < GL; ++g) a = fs_red_op<KIND>(a, lds[g * PC + col0 + f]);
          vals[i][f] = a;
        }
      }
    }
  }
}

// Stage 2, grid-wide fold with fan-in F.
//   part     workspace, sum over levels of n_level*K*C floats
//   tickets  workspace, one zero-initialised u32 per fan-in group per level; left zero on exit
//   flag     one u32 of LDS
//   idx, n   this workgroup's index among the n workgroups that fold together (the whole grid,
//            or the workgroups of one column tile)
// Returns true in exactly one workgroup, whose `vals` then hold the final values.
//
// Visibility across the 8 XCDs (each has its own L2) is obtained without device-scope fences,
// which write back and invalidate a whole L2 and cost microseconds each: partials are written
// with sc1 stores, every wavefront waits for its own stores to be acknowledged before the
// workgroup barrier, lane 0 then bumps the ticket with an agent-scope atomic, and the folding
// workgroup reads the partials with sc1 loads (never served by stale lines of its own L2).
// The F loads of a chunk are independent and issued in batches, so a fold costs a few memory
// round trips, not F of them; they are combined in index order, whichever workgroup folds, or (PAIRS: 1 where all reductions fold alike, 2 where
// not) in pairs of neighbours: one after the other, 256 partials through two levels of 16 lose as much as the rows do (column sums + row norms
// [32768,100] 6.4e-8 from float64, 4.1e-8 in pairs, [65536,512] 6.8e-8 and 4.4e-8, LayerNorm backward [11403,64] 1.7e-7 and 1.1e-7).  A kind after
// the other, each by the lanes whose chunks are of it: chosen per operation, two kinds cost a kernel 2 us (a thousand instructions, run once).  Not in kernels
// that only fold, whose loads then are in flight in smaller lots (column sums bf16 [36220,447] 12.5 -> 13.2 us).
template <int K, int C, int WG, int FV, int F, int PAIRS, typename KINDS, int CPT>
FS_DEV bool fs_colred_fold_grid(float (&vals)[CPT][FV], float* part, fs_u32* tickets, fs_u32* flag, fs_u32 idx, fs_u32 n) {
  typedef fs_colfold<K, C, WG, FV> S;
  static_assert(CPT == S::CPT, "chunks per thread");
  constexpr int KC = K * C;
  constexpr int FB = 16;  // loads in flight per chunk
  const int t = (int)threadIdx.x;
  while (n > 1) {
    {
      const __amdgpu_buffer_rsrc_t mine = fs_make_rsrc(part + (long)idx * KC, KC * 4);
#pragma unroll
      for (int i = 0; i < S::CPT; ++i) {
        const int c = t + i * WG;
        if (c < S::NCH) fs_store_dev<FV>(vals[i], mine, (fs_u32)c * (FV * 4));
      }
    }
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's partial stores are acknowledged
    __syncthreads();
    const fs_u32 grp = idx / F, first = grp * F;
    const fs_u32 cnt = (n - first) < (fs_u32)F ? (n - first) : (fs_u32)F;
    if (t == 0) {
      const fs_u32 old = __hip_atomic_fetch_add(&tickets[grp], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool last = old == cnt - 1;
      if (last) __hip_atomic_store(&tickets[grp], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *flag = last ? 1u : 0u;
    }
    __syncthreads();
    if (*flag == 0u) return false;
    const __amdgpu_buffer_rsrc_t theirs = fs_make_rsrc(part + (long)first * KC, cnt * (KC * 4));
#pragma unroll
    for (int i = 0; i < S::CPT; ++i) {
      const int c = t + i * WG;
      if (c < S::NCH) {
        const int k = c / S::CH;
        float a[FV];
#pragma unroll
        for (int f = 0; f < FV; ++f) a[f] = KINDS::identity(k);
        for (fs_u32 jb = 0; jb < cnt; jb += FB) {
          float tmp[FB][FV];
#pragma unroll
          for (int u = 0; u < FB; ++u) {
            const fs_u32 j = (jb + u) < cnt ? (jb + u) : (cnt - 1);  // clamped: always a valid load
            fs_load_dev<FV>(tmp[u], theirs, j * (KC * 4) + (fs_u32)c * (FV * 4));
          }
          if constexpr (PAIRS != 0) {
#pragma unroll
            for (int kk = 0; kk < (PAIRS == 1 ? 1 : K); ++kk) {
              if (PAIRS == 2 && k != kk) continue;
#pragma unroll
              for (int f = 0; f < FV; ++f) {
                float v[FB];
#pragma unroll
                for (int u = 0; u < FB; ++u) v[u] = (jb + u) < cnt ? tmp[u][f] : KINDS::identity(kk);
                fs_pairs<FB>(v, [&](float x, float y) { return KINDS::op(kk, x, y); });
                a[f] = KINDS::op(kk, a[f], v[0]);
              }
            }
          } else {
#pragma unroll
            for (int u = 0; u < FB; ++u) {
              const bool use = (jb + u) < cnt;
#pragma unroll
              for (int f = 0; f < FV; ++f) a[f] = use ? KINDS::op(k, a[f], tmp[u][f]) : a[f];
            }
          }
        }
#pragma unroll
        for (int f = 0; f < FV; ++f) vals[i][f] = a[f];
      }
    }
    part += (long)n * KC;
    const fs_u32 groups = (n + F - 1) / F;
    tickets += groups;
    idx = grp;
    n = groups;
  }
  return true;
}

// Stage 2 where all n workgroups are running at once (one to a compute unit): in the place of a tree in which one workgroup folds the
// partials of F others and then one the rest, all of them meet and fold slices of the columns, from all partials.
//   fs_colred_meet   leaves this workgroup's partial and waits until the others have: 1 they have (fold your slices), 2 they have, and this
//                    is the last one, 0 they have not after `ticks` of the 100 MHz clock (leave: nothing waits for workgroups that the
//                    device has not started).
//   fs_colred_left   of the last one: has any left?  (Then it folds their slices.)
//   counters         [0] groups of 16 workgroups that are complete, [32 * (1 + g)] workgroups of group g that have arrived (256 on one
//                    counter take 10 us), then a door for each workgroup, opened by the last one.  Zero, and left zero: by the last
//                    workgroup of a group, the last of all, who passes a door, and, where a workgroup has left, by the last of all.
//   fs_colred_slice  slice `sl`: SC chunks of FV columns; lanes SC apart take a partial each, and fold in pairs.  The results are those of
//                    chunks sl * SC + lane in the first SC lanes.
//   fs_colred_alone  one chunk by one lane, in the same order, for the slices of those who have left: slices one after the other are a
//                    chain of round trips (LayerNorm backward fp32 [8192,4096] beside a streaming kernel of another stream 1010 us).
FS_DEV fs_u32* fs_colred_door(fs_u32* counters, fs_u32 idx, fs_u32 n) { return counters + 32 * (1 + (n + 15) / 16) + idx; }
template <int K, int C, int WG, int FV, int CPT>
FS_DEV int fs_colred_meet(const float (&vals)[CPT][FV], float* part, fs_u32* counters, fs_u32* flag /* and 8 words: who has left */, fs_u32 idx, fs_u32 n, int ticks) {
  typedef fs_colfold<K, C, WG, FV> S;
  static_assert(CPT == S::CPT, "chunks per thread");
  constexpr int KC = K * C;
  const int t = (int)threadIdx.x;
  const __amdgpu_buffer_rsrc_t mine = fs_make_rsrc(part + (long)idx * KC, KC * 4);
#pragma unroll
  for (int i = 0; i < S::CPT; ++i) {
    const int c = t + i * WG;
    if (c < S::NCH) fs_store_dev<FV>(vals[i], mine, (fs_u32)c * (FV * 4));
  }
  __builtin_amdgcn_s_waitcnt(0);  // this wavefront's partial stores are acknowledged
  __syncthreads();
  if (t == 0) {
    const fs_u32 groups = (n + 15) / 16, grp = idx / 16, cnt = n - grp * 16 < 16 ? n - grp * 16 : 16;
    fs_u32* const arrived = counters + 32 * (1 + grp);
    fs_u32 met = 0;
    if (__hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == cnt - 1) {
      __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__hip_atomic_fetch_add(counters, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == groups - 1) {
        __hip_atomic_store(counters, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        met = 2;
      }
    }
    if (met == 0) {
      fs_u32* const door = fs_colred_door(counters, idx, n);
      const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
      do {
        __builtin_amdgcn_s_sleep(1);
        met = __hip_atomic_load(door, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } while (met == 0 && (long long)(__builtin_amdgcn_s_memrealtime() - t0) < (long long)ticks);
      if (met == 0) met = __hip_atomic_exchange(door, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // (1: opened in between)
      if (met != 0) __hip_atomic_store(door, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    *flag = met;
  }
  __syncthreads();
  const int met = (int)*flag;
  if (met == 2) {
    if (t < 8) flag[1 + t] = 0;
    __syncthreads();  // (every wavefront has read the flag before one writes it again)
    for (fs_u32 i = (fs_u32)t; i < n; i += WG) {
      fs_u32* const door = fs_colred_door(counters, i, n);
      if (i != idx && __hip_atomic_exchange(door, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2u) {
        __hip_atomic_store(door, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(flag, 3u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        (void)__hip_atomic_fetch_or(&flag[1 + i / 32], 1u << (i & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }
  return met;
}
FS_DEV bool fs_colred_left(const fs_u32* flag) {
  __syncthreads();
  return *flag == 3u;
}
template <int K, int C, int WG, int FV, int SC, int N, typename KINDS>
FS_DEV void fs_colred_slice(float (&vals)[FV], const float* part, float* lds /* WG/64*SC*FV floats */, int sl) {
  typedef fs_colfold<K, C, WG, FV> S;
  constexpr int KC = K * C, H = WG / SC, PS = (N + H - 1) / H, FB = PS < 8 ? PS : 8;  // H lanes to a chunk, PS partials to each
  static_assert(SC <= 64 && (SC & (SC - 1)) == 0, "slice width");
  const int t = (int)threadIdx.x, h = t / SC, c0 = sl * SC + t % SC, c = c0 < S::NCH ? c0 : S::NCH - 1, k = c / S::CH;
  const __amdgpu_buffer_rsrc_t all = fs_make_rsrc(part, N * (KC * 4));
  float a[FV];
#pragma unroll
  for (int f = 0; f < FV; ++f) a[f] = KINDS::identity(k);
  for (int j0 = 0; j0 < PS; j0 += FB) {
    float tmp[FB][FV];
#pragma unroll
    for (int u = 0; u < FB; ++u) {
      const int j = (j0 + u) * H + h;
      fs_load_dev<FV>(tmp[u], all, (fs_u32)(j < N ? j : N - 1) * (KC * 4) + (fs_u32)c * (FV * 4));
    }
#pragma unroll
    for (int u = 0; u < FB; ++u)
#pragma unroll
      for (int f = 0; f < FV; ++f) a[f] = j0 + u < PS && (j0 + u) * H + h < N ? KINDS::op(k, a[f], tmp[u][f]) : a[f];
  }
#pragma unroll
  for (int m = SC; m < 64; m <<= 1) {
    const bool upper = (fs_lane_id() & m) != 0;
#pragma unroll
    for (int f = 0; f < FV; ++f) {
      const float other = fs_shfl_xor(a[f], m);
      a[f] = KINDS::op(k, upper ? other : a[f], upper ? a[f] : other);
    }
  }
  if constexpr (WG > 64) {
    __syncthreads();  // (the slice before this one may still be read)
    if ((t & 63) < SC) {
#pragma unroll
      for (int f = 0; f < FV; ++f) lds[(t / 64 * SC + (t & 63)) * FV + f] = a[f];
    }
    __syncthreads();
    if (t < SC) {
#pragma unroll
      for (int w = 1; w < WG / 64; ++w)
#pragma unroll
        for (int f = 0; f < FV; ++f) a[f] = KINDS::op(k, a[f], lds[(w * SC + t) * FV + f]);
    }
  }
#pragma unroll
  for (int f = 0; f < FV; ++f) vals[f] = a[f];
}

FS_DEV bool fs_colred_gone(const fs_u32* flag, int idx) { return (flag[1 + idx / 32] >> (idx & 31) & 1) != 0; }
template <int K, int C, int WG, int FV, int SC, int N, typename KINDS>
FS_DEV void fs_colred_alone(float (&vals)[FV], const float* part, int c) {
  typedef fs_colfold<K, C, WG, FV> S;
  constexpr int KC = K * C, H = WG / SC, PS = (N + H - 1) / H, Q = 64 / SC, QB = Q < 8 ? Q : 8;  // (as in fs_colred_slice; Q lanes of a wavefront to a chunk)
  const int k = c / S::CH;
  const __amdgpu_buffer_rsrc_t all = fs_make_rsrc(part, N * (KC * 4));
  for (int w = 0; w < WG / 64; ++w) {
    float wave[Q / QB][FV];
#pragma unroll
    for (int b = 0; b < Q / QB; ++b) {
      float v[FV][QB];
#pragma unroll
      for (int f = 0; f < FV; ++f)
#pragma unroll
        for (int q = 0; q < QB; ++q) v[f][q] = KINDS::identity(k);
      for (int i = 0; i < PS; ++i) {
        float tmp[QB][FV];
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          const int j = i * H + w * Q + b * QB + q;
          fs_load_dev<FV>(tmp[q], all, (fs_u32)(j < N ? j : N - 1) * (KC * 4) + (fs_u32)c * (FV * 4));
        }
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
          for (int f = 0; f < FV; ++f) v[f][q] = i * H + w * Q + b * QB + q < N ? KINDS::op(k, v[f][q], tmp[q][f]) : v[f][q];
      }
#pragma unroll
      for (int f = 0; f < FV; ++f) {
        fs_pairs<QB>(v[f], [&](float x, float y) { return KINDS::op(k, x, y); });
        wave[b][f] = v[f][0];
      }
    }
#pragma unroll
    for (int f = 0; f < FV; ++f) {
      const float x = Q / QB > 1 ? KINDS::op(k, wave[0][f], wave[Q / QB - 1][f]) : wave[0][f];
      vals[f] = w == 0 ? x : KINDS::op(k, vals[f], x);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Workgroups of one column tile that meet inside a kernel: each leaves its partial (fs_tile_put) and waits until all N are there
// (fs_tile_meet), then all of them fold the partials in the same order and go on with the result (a column statistic that every
// row needs again).  Visibility as in the grid-wide fold: sc1 stores acknowledged before the bit is set, sc1 loads after it.  (A flag per
// workgroup in a word of its own that all the others read: batch normalisation fp32 [4096,1024] 10.1 -> 10.7 us, [65536,64] 13.9 -> 14.9.)
// A kernel must not depend on workgroups that the device has not started (another stream may hold the compute units): after `ticks` of
// the 100 MHz clock a waiting workgroup claims a partial that is missing, computes it from memory and puts it in its place, and so on
// until all are there: the missing rows are read once more, shared among those who wait.  A workgroup that starts late puts the same bits
// to the same place.  Every wait ends: what is missing a running workgroup has claimed, or the next one who waits claims it; and who has
// waited for claimed ones for kTilePatience does those, too (a claim may be all there is in a workspace that was never cleared).
//   counter  workgroups whose own partial is there, and kTileLate once one has waited in vain: from then on each sets the bit of what it has put
//   bits     a bit for each partial that is there, then one for each that is claimed.  All zero before and after the kernel.  (Bits that all
//            set and read from the start, in the place of the count: [65536,99] 26.7 -> 34.4 us, [1000,1000] 7.4 -> 7.9)
//   result   -1: all are there; else the partial to compute, after which fs_tile_next tells what comes then
// ------------------------------------------------------------------------------------------
template <int K, int C, int WG, int FV, int CPT>
FS_DEV void fs_tile_put(const float (&vals)[CPT][FV], float* part, int idx) {
  typedef fs_colfold<K, C, WG, FV> S;
  static_assert(CPT == S::CPT, "chunks per thread");
  constexpr int KC = K * C;
  const __amdgpu_buffer_rsrc_t mine = fs_make_rsrc(part + (long)idx * KC, KC * 4);
#pragma unroll
  for (int i = 0; i < S::CPT; ++i) {
    const int c = (int)threadIdx.x + i * WG;
    if (c < S::NCH) fs_store_dev<FV>(vals[i], mine, (fs_u32)c * (FV * 4));
  }
  __builtin_amdgcn_s_waitcnt(0);  // this wavefront's partial stores are acknowledged
  __syncthreads();
}
constexpr fs_u32 kTileLate = 1u << 30;
constexpr unsigned long long kTilePatience = 100000;  // 1 ms
template <int N> FS_DEV fs_u32 fs_tile_missing(fs_u32* counter, fs_u32* bits, int idx) {  // (one lane; one more than the partial to compute)
  constexpr int W = (N + 31) / 32;
  (void)__hip_atomic_fetch_or(&bits[idx / 32], 1u << (idx & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
  for (;;) {
    __builtin_amdgcn_s_sleep(8);  // (those who wait for the count see that it is late, and set their bits)
    if ((__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (kTileLate - 1)) == (fs_u32)N) return 0;
    const bool patient = __builtin_amdgcn_s_memrealtime() - t0 < kTilePatience;
    bool all = true;
    for (int w = 0; w < W; ++w) {
      const fs_u32 missing = (N - w * 32 >= 32 ? ~0u : (1u << (N - w * 32)) - 1) & ~__hip_atomic_load(&bits[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (missing == 0) continue;
      all = false;
      const fs_u32 open = patient ? missing & ~__hip_atomic_load(&bits[W + w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : missing, after = open & (~0u << (idx & 31));
      const fs_u32 from = after ? after : open, bit = from & (~from + 1);  // (workgroups start at different places)
      if (bit && (!(__hip_atomic_fetch_or(&bits[W + w], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit) || !patient)) return 1 + (fs_u32)(w * 32 + __builtin_ctz(bit));
    }
    if (all) return 0;
  }
}
template <int N> FS_DEV int fs_tile_meet(fs_u32* counter, fs_u32* bits, fs_u32* flag, int idx, int ticks) {
  if (threadIdx.x == 0) {
    fs_u32 seen = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
    if (seen < (fs_u32)N) {
      const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
      do {
        __builtin_amdgcn_s_sleep(1);
        seen = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } while (seen < (fs_u32)N && (long long)(__builtin_amdgcn_s_memrealtime() - t0) < (long long)ticks);
      if (seen < (fs_u32)N) seen = __hip_atomic_fetch_or(counter, kTileLate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) | kTileLate;
    }
    *flag = seen > (fs_u32)N ? fs_tile_missing<N>(counter, bits, idx) : 0;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane((int)*flag) - 1;
}
template <int N> FS_DEV int fs_tile_next(fs_u32* counter, fs_u32* bits, fs_u32* flag, int idx) {
  if (threadIdx.x == 0) *flag = fs_tile_missing<N>(counter, bits, idx);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane((int)*flag) - 1;
}
// ... the fold of the N partials, once they are there.  Where the chunks leave lanes of the workgroup idle, H slices of
// PS partials are folded side by side and then, through LDS (WG floats), each other: one round of loads instead of one for every
// sixteen partials.
template <int K, int C, int WG, int N> struct fs_tile_slices {
  static constexpr int NCH = K * C, H0 = NCH < WG ? WG / NCH : 1, H = H0 < N ? H0 : N;
  static constexpr int PS = (N + H - 1) / H;
};
template <int K, int C, int WG, int N, typename KINDS, int CPT>
FS_DEV void fs_tile_fold(float (&vals)[CPT][1], const float* part, float* lds) {
  typedef fs_colfold<K, C, WG, 1> S;
  typedef fs_tile_slices<K, C, WG, N> Q;
  constexpr int KC = K * C, FB = Q::PS < 16 ? Q::PS : 16;  // loads in flight per chunk
  const __amdgpu_buffer_rsrc_t all = fs_make_rsrc(part, N * (KC * 4));
#pragma unroll
  for (int i = 0; i < S::CPT; ++i) {
    const int t = (int)threadIdx.x + i * WG, c = Q::H > 1 ? t % KC : t, h = Q::H > 1 ? t / KC : 0;
    if (c < S::NCH && h < Q::H) {
      const int k = c / S::CH;
      float a = KINDS::identity(k);
      for (int j0 = 0; j0 < Q::PS; j0 += FB) {
        float tmp[FB][1];
#pragma unroll
        for (int u = 0; u < FB; ++u) {
          const int j = h * Q::PS + j0 + u;
          fs_load_dev<1>(tmp[u], all, (fs_u32)(j < N ? j : N - 1) * (KC * 4) + (fs_u32)c * 4);
        }
        float v[FB];
#pragma unroll
        for (int u = 0; u < FB; ++u) v[u] = j0 + u < Q::PS && h * Q::PS + j0 + u < N ? tmp[u][0] : KINDS::identity(k);
        fs_pairs<FB>(v, [&](float x, float y) { return KINDS::op(k, x, y); });
        a = j0 == 0 ? v[0] : KINDS::op(k, a, v[0]);
      }
      if constexpr (Q::H > 1) lds[h * KC + c] = a;
      else vals[i][0] = a;
    }
  }
  if constexpr (Q::H > 1) {
    __syncthreads();
    const int c = (int)threadIdx.x;
    if (c < KC) {
      float a = KINDS::identity(c / S::CH);
      for (int h0 = 0; h0 < Q::H; h0 += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = h0 + u < Q::H ? lds[(h0 + u) * KC + c] : KINDS::identity(c / S::CH);
        fs_pairs<8>(v, [&](float x, float y) { return KINDS::op(c / S::CH, x, y); });
        a = h0 == 0 ? v[0] : KINDS::op(c / S::CH, a, v[0]);
      }
      vals[0][0] = a;
    }
  }
}
// A workgroup that has met its tile's others for the last time says so in the last of the tile's `count` counters, and the last one to say
// it leaves all of them, and the bits, zero.  (In two halves: the answer of the first is on its way while the results leave.)
FS_DEV fs_u32 fs_tile_leave(fs_u32* counters, int count) {
  return threadIdx.x == 0 ? __hip_atomic_fetch_add(&counters[count - 1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
}
FS_DEV void fs_tile_clear(fs_u32 before, fs_u32* counters, int count, fs_u32* bits, int words, fs_u32 n) {
  if (threadIdx.x == 0 && before == n - 1) {
    for (int i = 0; i < count; ++i) __hip_atomic_store(&counters[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int i = 0; i < words; ++i) __hip_atomic_store(&bits[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

#endif  // FS_DEVICE_H_
