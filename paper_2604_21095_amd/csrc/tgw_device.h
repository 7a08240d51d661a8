// Device code shared by the kernels' translation units: operand layouts and
// number formats, the p-value table lookup, the reduced outputs, the tile
// order and the fused epilogue of a staged block of accumulators.
#pragma once

#include "tgw_internal.h"

#include <math.h>

#include <type_traits>

namespace tgw {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ inline uint32_t bf16_bits_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ inline float bf16_to_float(uint32_t b) { return __uint_as_float(b << 16); }

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  return bf16_bits_rne(lo) | (bf16_bits_rne(hi) << 16);
}

template <int NT>
__device__ inline double block_max(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double m = 0.0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) m = fmax(m, sh[i]);
  return m;
}

template <int NT>
__device__ inline double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) s += sh[i];
  return s;
}

// reduce NV values at once; sh holds (NT/64) * NV doubles
template <int NT, int NV>
__device__ inline void block_sum_vec(double* v, double* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k)
    for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o);
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) sh[w * NV + k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    double s = 0.0;
    for (int i = 0; i < NT / 64; ++i) s += sh[i * NV + k];
    v[k] = s;
  }
}

// ---------------------------------------------------------------------------
// operand layout (must match the matrix-core fragment reads in gemm_kernel)
//
// BF16 split: block (cb, ch) holds 4096 bf16: [hl][j][lane][e], hl = 0 for
// hi, 1 for lo; j = K16 step; lane = 32 h + column; e = element.  The sample
// fed at (j, h, e) is 64 ch + 32 h + 16 (j >> 1) + 4 (j & 1) + (e >> 1) +
// 8 (e & 1), which is the order in which gemm_kernel decodes packed codes.
// FP32: block (cb, ch) holds 2048 floats: [j >> 2][lane][j & 3], j = K2 step,
// sample 64 ch + 32 h + j.
// ---------------------------------------------------------------------------
// stride: 16-bit elements per block (4096 for the 16-bit splits; 3072 for
// FP16 hi + FP8 lo, whose block keeps only the hi half in this layout)
__device__ inline int64_t operand_index_split(int64_t col, int64_t i, int n_chunks, int hl,
                                              int64_t stride = 4096) {
  const int64_t cb = col >> 5;
  const int c = (int)(col & 31);
  const int64_t ch = i >> 6;
  const int s = (int)(i & 63);
  const int h = s >> 5;
  const int rem = s & 31;
  const int jhi = rem >> 4;
  const int b = (rem >> 3) & 1;
  const int jlo = (rem >> 2) & 1;
  const int d = rem & 3;
  const int j = 2 * jhi + jlo;
  const int e = 2 * d + b;
  const int lane = 32 * h + c;
  return (cb * n_chunks + ch) * stride + hl * 2048 + j * 512 + lane * 8 + e;
}

__device__ inline int64_t operand_index_fp32(int64_t col, int64_t i, int n_chunks) {
  const int64_t cb = col >> 5;
  const int c = (int)(col & 31);
  const int64_t ch = i >> 6;
  const int s = (int)(i & 63);
  const int h = s >> 5;
  const int j = s & 31;
  const int lane = 32 * h + c;
  return (cb * n_chunks + ch) * 2048 + (j >> 2) * 256 + lane * 4 + (j & 3);
}

// FP16 hi + FP8 lo: block (cb, ch) = 6 KiB.  Bytes [0, 4096) hold the FP16
// hi terms in the split layout's hi half; bytes [4096, 6144) the e4m3 lo
// terms as [part][lane][16 bytes].  A lane (32 h + column) holds 32 bytes,
// dword D = 4 part + t, byte k; it feeds sample 64 ch + 32 h + 16 part +
// 4 k + t, the order in which the genotype FP8 decode emits them.
__device__ inline int64_t operand_index_lo8(int64_t col, int64_t i, int n_chunks) {
  const int64_t cb = col >> 5;
  const int c = (int)(col & 31);
  const int64_t ch = i >> 6;
  const int s = (int)(i & 63);
  const int h = s >> 5;
  const int part = (s >> 4) & 1;
  const int k = (s >> 2) & 3;
  const int t = s & 3;
  const int lane = 32 * h + c;
  return (cb * n_chunks + ch) * kBlockBytes8 + 4096 + part * 1024 + lane * 16 + 4 * t + k;
}

__device__ inline uint32_t f16_bits_rn(float f) {
  const _Float16 h = (_Float16)f;  // round to nearest even
  return (uint32_t)__builtin_bit_cast(uint16_t, h);
}
__device__ inline float f16_to_float(uint32_t b) { return (float)__builtin_bit_cast(_Float16, (uint16_t)b); }

// OCP FP8 E4M3 (bias 7, no infinities, largest finite 448, subnormals
// m * 2^-9), round to nearest even.  |x| must not exceed 448.
__device__ inline uint32_t e4m3_bits_rne(double x) {
  const uint32_t sign = x < 0.0 ? 0x80u : 0u;
  const double a = fabs(x);
  if (a < 0x1p-6) {
    const double m = rint(a * 0x1p9);  // subnormal step 2^-9; m = 8 is the smallest normal
    return sign | (uint32_t)m;
  }
  int e = ilogb(a);
  double q = rint(ldexp(a, 3 - e)) - 8.0;  // 3 fraction bits
  if (q >= 8.0) {
    q = 0.0;
    ++e;
  }
  return sign | (uint32_t)((e + 7) << 3) | (uint32_t)q;
}
__device__ inline double e4m3_value(uint32_t b) {
  const int e = (b >> 3) & 15, m = b & 7;
  const double v = e == 0 ? ldexp((double)m, -9) : ldexp(1.0 + m / 8.0, e - 7);
  return (b & 0x80u) ? -v : v;
}

// power-of-two shift that brings a column's largest FP8 lo term near the top
// of the e4m3 range (0 for a column without lo terms)
__device__ inline int lo_shift(double maxlo) {
  if (!(maxlo > 0.0)) return 0;
  int s = ilogb(448.0 / maxlo);
  return s < -100 ? -100 : (s > 100 ? 100 : s);
}

// lsh: the column's FP8 lo shift (FP16 hi + FP8 lo form only)
// the hi and lo parts of a value in the BF16 split, or of 2^12 times it in
// the FP16 split (round to nearest even, then the rounded remainder)
__device__ inline void split_parts(int prec, double v, uint32_t* hb, uint32_t* lb) {
  if (prec == kSplit16) {
    const double vs = v * (double)kF16Scale;
    *hb = f16_bits_rn((float)vs);
    *lb = f16_bits_rn((float)(vs - (double)f16_to_float(*hb)));
  } else {
    *hb = bf16_bits_rne((float)v);
    *lb = bf16_bits_rne((float)(v - (double)bf16_to_float(*hb)));
  }
}

// stored: the value the operand now holds (in 2^12 units for the FP16
// forms); lo: its FP8 lo term alone (FP16 + FP8 form; 0 otherwise)
__device__ inline void store_operand(void* op, int prec, int64_t col, int64_t i, int n_chunks, double v,
                                     double* stored, int lsh = 0, double* lo = nullptr) {
  if (lo) *lo = 0.0;
  if (prec == kSplit8) {
    const double vs = v * (double)kF16Scale;
    const uint32_t hb = f16_bits_rn((float)vs);
    const double hi = (double)f16_to_float(hb);
    const uint32_t qb = e4m3_bits_rne(ldexp(vs - hi, lsh));
    ((uint16_t*)op)[operand_index_split(col, i, n_chunks, 0, kBlockBytes8 / 2)] = (uint16_t)hb;
    ((uint8_t*)op)[operand_index_lo8(col, i, n_chunks)] = (uint8_t)qb;
    const double lv = ldexp(e4m3_value(qb), -lsh);
    *stored = hi + lv;
    if (lo) *lo = lv;
  } else if (prec == kSplit16 || prec == kSplit) {
    uint32_t hb, lb;
    split_parts(prec, v, &hb, &lb);
    uint16_t* p = (uint16_t*)op;
    p[operand_index_split(col, i, n_chunks, 0)] = (uint16_t)hb;
    p[operand_index_split(col, i, n_chunks, 1)] = (uint16_t)lb;
    *stored = prec == kSplit16 ? (double)f16_to_float(hb) + (double)f16_to_float(lb)
                               : (double)bf16_to_float(hb) + (double)bf16_to_float(lb);
  } else {
    const float f = (float)v;
    ((float*)op)[operand_index_fp32(col, i, n_chunks)] = f;
    *stored = (double)f;
  }
}

// interval coefficients as a plain vector type (HIP's float4 class has no
// copy from an LDS reference); the wide kernel's epilogue reads a copy of the
// table in LDS
typedef float tab4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(3))) tab4* LdsTable;

// cubic Hermite interpolation of -log10 p at |t| <= kTMax (TabPtr: the global
// table or its LDS copy)
template <class TabPtr>
__device__ inline float table_nlog10p(TabPtr tab, float at) {
  const float x = at * (float)kTabPerUnit;
  int k = (int)x;
  k = k > kTabIntervals - 1 ? kTabIntervals - 1 : k;
  const float s = x - (float)k;
  const tab4 c = tab[k];
  return fmaf(fmaf(fmaf(c.w, s, c.z), s, c.y), s, c.x);
}

// 0xff in every byte of d that is 0xff (the 8-bit dosage missing code), 0
// elsewhere: bit 7 of ((d & 0x7f) + 1) & d is set exactly for 0xff bytes
// (no carry leaves a byte); 2t - (t >> 7) spreads each marked bit over its byte
__device__ __forceinline__ uint32_t ff_bytes(uint32_t d) {
  const uint32_t t = ((d & 0x7f7f7f7fu) + 0x01010101u) & d & 0x80808080u;
  return (t << 1) - (t >> 7);
}

// The slots and the contraction are in operand units (gs per genotype unit),
// so r takes 1 / (gs ||g_res||) and beta, SE take 1 / ||g_res||.  Markers
// whose ||g_res||^2 here is below kRedoTol ||g_c||^2 get NaN (the main
// kernel then writes NaN rows and no reduced outputs) and go to the FP64
// list of their panel.
// ws: the marker's slots (in place), j: the panel, m: the marker's row, -1 for
// none (nothing is listed).
__device__ inline float2 finalize_row(const MarkerStat& st, float* ws, float wscale, int lo_slot, const RedoDev& redo,
                                      int j, int32_t m) {
  const double igs = 1.0 / (double)st.gscale;  // exact: gs is K / 128 or 1
  double h2 = st.gc2;
  for (int k = 1; k < kSlots; ++k) {
    const float wf = ws[k] * wscale;  // undo the operand scale of the Q columns
    ws[k] = wf;
    const double w = (double)wf * igs;
    h2 -= w * w;
  }
  const bool ok = st.flags == 0 && h2 > kRedoTol * st.gc2;
  if (st.flags == 0 && !ok && m >= 0) {
    const uint32_t k = atomicAdd(redo.count + j, 1u);
    redo.entries[j * redo.stride + k] = m;  // at most one entry per (marker, panel): never full
  }
  const double ih = 1.0 / sqrt(h2);
  ws[0] = st.dmu;
  if (lo_slot) ws[kLoSlot] = st.dlo;  // the slot's Q^T g is 0 (q <= 31 in every panel of the plan)
  return ok ? make_float2((float)(ih * igs), (float)ih) : make_float2(__builtin_nanf(""), __builtin_nanf(""));
}

// per-column best test: max -log10 p in the high word, the complement of
// the marker index in the low word (so equal maxima keep the first marker)
__device__ inline unsigned long long best_pack(float nl, int64_t marker) {
  return ((unsigned long long)__float_as_uint(nl > 0.f ? nl : 0.f) << 32) |
         (unsigned long long)(0xffffffffu - (uint32_t)marker);
}

// per-column top-k lists: words (bits of |t|) << 32 | (0xffffffff - marker),
// kept in decreasing order; 0 is an empty slot
__device__ inline unsigned long long topk_pack(float at, int64_t marker) {
  return ((unsigned long long)__float_as_uint(at) << 32) | (unsigned long long)(0xffffffffu - (uint32_t)marker);
}

// Inserts w into the decreasing list s[0..k) that other lanes and workgroups
// update at the same time.  Every slot only grows (atomicMax), and a value
// reaches slot i + 1 only by being pushed out of slot i or by starting there
// after slot i was seen >= it, so s[i] >= s[i + 1] holds at every moment.
// The search for the first slot below w on plain (possibly stale) reads is
// therefore safe: every slot it skips is >= w for good.  From there each
// atomicMax keeps the larger of (slot, w) and w carries the smaller one on,
// until it lands in an empty slot or drops off the end, below the k-th value.
__device__ inline void topk_insert(unsigned long long* s, int k, unsigned long long w) {
  int lo = 0, hi = k;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (__atomic_load_n(s + mid, __ATOMIC_RELAXED) >= w)
      lo = mid + 1;
    else
      hi = mid;
  }
  for (int i = lo; i < k && w != 0ull; ++i) {
    const unsigned long long old = atomicMax(s + i, w);
    w = old < w ? old : w;
  }
}

__device__ inline void append_hit(const HitDev& hits, int64_t marker, int j, int64_t p, float nl, float r) {
  const unsigned long long idx = atomicAdd(hits.count, 1ull);
  if (idx < (unsigned long long)hits.capacity) {
    Hit h;
    h.marker = marker;
    h.panel = j;
    h.pheno = (int32_t)p;
    h.nl = nl;
    h.r = r;
    hits.entries[idx] = h;
  }
}

// Tile order of the persistent kernels: super-tiles of kGroupM marker tiles
// x kGroupC column tiles, walked column group by column group, marker group
// by marker group; within a super-tile, column tile fastest.  The 32
// workgroups an XCD runs at once (wide kernel) then work on about one
// super-tile, so a genotype chunk is fetched once for kGroupC workgroups and
// an operand chunk once for kGroupM (column-tile-major order fetches the
// genotypes once per column tile).  w in [0, n_mtiles * n_ctiles) maps one
// to one; edge groups are ragged.
constexpr int kGroupM = 8, kGroupC = 4;
__device__ __forceinline__ void grouped_tile(int64_t w, int nm, int nc, int& mtile, int& ctile) {
  const int64_t full = (int64_t)nm * kGroupC;  // tiles of a full column group
  const int cg = (int)(w / full);
  const int64_t u = w - (int64_t)cg * full;
  const int c = nc - cg * kGroupC < kGroupC ? nc - cg * kGroupC : kGroupC;
  const int64_t sg = (int64_t)kGroupM * c;  // tiles of a full marker group in this column group
  const int mg = (int)(u / sg);
  const int r = (int)(u - (int64_t)mg * sg);
  const int mi = r / c;
  mtile = mg * kGroupM + mi;
  ctile = cg * kGroupC + (r - mi * c);
}

template <int NW>
struct GWords {
  typedef uint32_t type __attribute__((ext_vector_type(NW)));
};
template <>
struct GWords<1> {
  typedef uint32_t type;
};
// load through a global-address-space pointer (global_load_*, not flat_load_*)
template <class T>
__device__ __forceinline__ T gload(const void* p) {
  static_assert(sizeof(T) % 4 == 0, "gload of whole words only");
  typedef typename GWords<sizeof(T) / 4>::type V;
  const V v = *(const __attribute__((address_space(1))) V*)p;
  return __builtin_bit_cast(T, v);
}
template <class T>
__device__ __forceinline__ void gstore(void* p, T v) {
  *(__attribute__((address_space(1))) T*)p = v;
}
// a store no kernel of the scan reads back (the dense outputs): marked
// non-temporal, so the written lines do not displace operand and genotype
// lines that later tiles fetch through L2
template <class T>
__device__ __forceinline__ void gstore_nt(void* p, T v) {
  __builtin_nontemporal_store(v, (__attribute__((address_space(1))) T*)p);
}

// one 32x32x16 matrix-core step on 16-bit operands given as raw bits
template <int PREC>
__device__ __forceinline__ f32x16 mfma16(const u32x4& a, const u32x4& b, const f32x16& c) {
  if constexpr (f16_scaled(PREC)) {
    typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                  0, 0, 0);
  }
}

// the rare part of a test's epilogue: |t| > 40 goes to the FP64 tail list
// (its -log10 p written as +inf until the tail kernel replaces it; with the
// list full, the table's value at 40 stands as a lower bound and the call
// reports the overflow), and a test at or above the hit threshold is
// appended to the hit list (for tail entries the tail kernel decides).
template <class TabPtr>
__device__ __forceinline__ void epilogue_rare(bool to_tail, float nl, float at, float r, TabPtr tab, float* nl_out,
                                           int64_t row, int j, int64_t p, const TailDev& tail, const HitDev& hits,
                                           int64_t marker) {
  if (to_tail) {
    const unsigned long long idx = atomicAdd(tail.count, 1ull);
    if (idx < (unsigned long long)tail.capacity) {
      TailEntry e;
      e.row = row;
      e.panel = j;
      e.col = (int32_t)p;
      e.r = r;
      e.pad = 0;
      tail.entries[idx] = e;
      if (nl_out) gstore(nl_out, INFINITY);
      return;
    }
    nl = table_nlog10p(tab, kTMax);
    if (nl_out) gstore(nl_out, nl);
  }
  if (hits.entries && at >= hits.t_floor && nl >= hits.threshold) append_hit(hits, marker, j, p, nl, r);
}

// finish one 32-column block of a wave's staged accumulators (stage holds
// rows 0 .. 32*WMF-1 of the wave's fragments, 32 columns each): lanes run
// along columns, two rows at a time; the per-column best over the rows is
// reduced in registers and merged with one atomic per column.
// invny and sp are this lane's column values (sp already per genotype unit).
// IhPtr: GlobalRows reads each row's 1/||g_res|| from global memory; an LDS
// pointer gives the wave's rows, copied there ahead of the output stores
// (on this chip a load issued after stores waits for them to complete, so
// loads inside the row loop would serialise behind the previous row's stores).
struct GlobalRows {};
__device__ __forceinline__ float* at_byte(float* base, uint32_t ob) { return (float*)((char*)base + ob); }
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(3))) f32x2* LdsRows;

template <int WMF, class TabPtr, class IhPtr>
__device__ __forceinline__ void finish_block(const float* stage, const GemmArgs& a, const ColBlock& blk,
                                             int64_t rowbase, int h, int r32, TabPtr tab, IhPtr ih, float invny,
                                             float sp) {
  if constexpr (!std::is_same<IhPtr, GlobalRows>::value) {
    // the lane's place from a fresh v_mbcnt: a lane index kept in a register
    // across the whole kernel gets spilled, and its reload just before the row
    // loop makes the compiler wait in every iteration for the earlier stores
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    h = lane >> 5;
    r32 = lane & 31;
  }
  static_assert(WMF <= 4, "rows of a block within 32-bit store offsets");
  const int j = blk.panel;
  const PanelDev pd = a.panels[j];
  const OutDev od = a.outs[j];
  const int64_t p = blk.col0 + r32;
  const bool colok = r32 < blk.ncol;
  // dense outputs rebased at (first row, first column) of the block: with
  // ld <= 2^22 and at most 128 rows every store is within 2^31 bytes of it
  // (held in scalar registers, so that a store is scalar base + vector offset)
  OutDev odb = od;
  {
    const int64_t base = (a.out_row0 + rowbase) * od.ld + blk.col0;
    auto rebase = [base](float* q) {
      const uint64_t v = q ? (uint64_t)(q + base) : 0;
      const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
      const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
      return (float*)(((uint64_t)hi << 32) | lo);
    };
    odb.r = rebase(od.r);
    odb.beta = rebase(od.beta);
    odb.se = rebase(od.se);
    odb.t = rebase(od.t);
    odb.nl = rebase(od.nl);
  }
  // top-k of this lane's column: the list and its current last word (rows
  // whose word is not above it cannot enter)
  const bool tk_on = od.topk != nullptr;  // uniform: one panel per column block
  unsigned long long* tkp = (tk_on && colok) ? od.topk + p * od.topk_k : nullptr;
  unsigned long long tk_last = tkp ? __atomic_load_n(tkp + od.topk_k - 1, __ATOMIC_RELAXED) : ~0ull;
  if constexpr (!std::is_same<IhPtr, GlobalRows>::value) {
    // the loads above (vector loads: the kernel writes global memory, so
    // they cannot go through the scalar cache) are waited for once here;
    // waited for at their first use they would put a full wait for the
    // previous rows' stores into every iteration
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); expcnt and lgkmcnt unconstrained
  }
  float bv = -1.0f;  // largest |t| of this lane's rows (-log10 p is increasing in |t| at fixed df)
  int64_t bm = 0;
  // -log10 p is needed for the dense output, for hit candidates, and (in
  // FP64, from the tail kernel) for |t| > 40 whenever any reduced output or
  // the dense output asks for it
  const bool need_p = od.nl || od.best || a.hits.entries;
  const bool need_tab = od.nl || a.hits.entries;
  const float hit_floor = a.hits.entries ? a.hits.t_floor : __builtin_nanf("");  // NaN: no |t| reaches it
  const float sqrt_df = pd.sqrt_df, inv_sqrt_df = pd.inv_sqrt_df;
  // R rows at a time: their LDS reads and table reads are in flight together
  constexpr int R = 4;
  static_assert((WMF * 16) % R == 0, "row groups");
  for (int g = 0; g < WMF * 16; g += R) {
    float Sv[R];
    f32x2 ihv[R];  // 1 / (gs ||g_res||) for r, 1 / ||g_res|| for beta and SE
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int rr = h + 2 * (g + i);
      Sv[i] = stage[rr * 32 + r32];
      if constexpr (std::is_same<IhPtr, GlobalRows>::value) {
        int64_t mr = rowbase + rr;
        mr = mr < a.nm ? mr : a.nm - 1;
        const float2 v = gload<float2>(a.invh + mr * a.n_panels + j);
        ihv[i] = f32x2{v.x, v.y};
      } else {
        ihv[i] = ih[rr];
      }
    }
    float rv[R], atv[R];
    bool okv[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int rr = h + 2 * (g + i);
      okv[i] = colok && rowbase + rr < a.nm;
      const float invh = ihv[i].y;
      float r = Sv[i] * ihv[i].x * invny;
      if (r > 1.0f) r = 1.0f;
      if (r < -1.0f) r = -1.0f;
      // 1 - r^2 is 0 or at least about 2^-24, never subnormal: the hardware
      // square root and reciprocal square root (1 ulp) serve as they are
      const float omr2 = (1.0f - r) * (1.0f + r);
      const float t = r * sqrt_df * __builtin_amdgcn_rsqf(omr2);
      const uint32_t ob = ((uint32_t)rr * (uint32_t)od.ld + (uint32_t)r32) * 4u;
      if (okv[i]) {
        if (odb.r) gstore_nt(at_byte(odb.r, ob), r);
        if (odb.beta) gstore_nt(at_byte(odb.beta, ob), r * sp * invh);
        if (odb.se) gstore_nt(at_byte(odb.se, ob), sp * invh * __builtin_amdgcn_sqrtf(omr2) * inv_sqrt_df);
        if (odb.t) gstore_nt(at_byte(odb.t, ob), t);
      }
      rv[i] = r;
      atv[i] = fabsf(t);
      if (okv[i] && atv[i] > bv) {  // NaN never enters
        bv = atv[i];
        bm = a.m_begin + a.out_row0 + rowbase + rr;
      }
    }
    if (need_p) {
      float nlv[R];
      if (need_tab) {  // the table at min(|t|, 40) (NaN reads the last interval): R reads in flight together
        tab4 cv[R];
        float sv[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const float x = fminf(atv[i], kTMax) * (float)kTabPerUnit;
          int k = (int)x;
          k = k > kTabIntervals - 1 ? kTabIntervals - 1 : k;
          sv[i] = x - (float)k;
          cv[i] = tab[k];
        }
#pragma unroll
        for (int i = 0; i < R; ++i) nlv[i] = fmaf(fmaf(fmaf(cv[i].w, sv[i], cv[i].z), sv[i], cv[i].y), sv[i], cv[i].x);
      } else {
#pragma unroll
        for (int i = 0; i < R; ++i) nlv[i] = 0.0f;
      }
      uint32_t rare = 0;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const float at = atv[i];
        // |t| <= 40: the table; NaN and +inf carry over; 40 < |t| < inf: the tail
        const bool to_tail = okv[i] && at > kTMax && at != INFINITY;
        const float nl = at <= kTMax ? nlv[i] : at;
        nlv[i] = nl;
        if (okv[i] && !to_tail && odb.nl) gstore_nt(at_byte(odb.nl, ((uint32_t)(h + 2 * (g + i)) * (uint32_t)od.ld + (uint32_t)r32) * 4u), nl);
        const bool hit = okv[i] && !to_tail && at >= hit_floor && nl >= a.hits.threshold;
        rare |= (to_tail || hit) ? 1u << i : 0u;
      }
      if (__builtin_amdgcn_ballot_w64(rare != 0)) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
          if (rare & (1u << i)) {
            const int rr = h + 2 * (g + i);
            const int64_t row = a.out_row0 + rowbase + rr;
            const uint32_t ob = ((uint32_t)rr * (uint32_t)od.ld + (uint32_t)r32) * 4u;
            const float at = atv[i];
            epilogue_rare(at > kTMax && at != INFINITY, nlv[i], at, rv[i], tab,
                          odb.nl ? at_byte(odb.nl, ob) : (float*)nullptr, row, j, p, a.tail, a.hits, a.m_begin + row);
          }
        }
      }
    }
    if (tk_on) {
      unsigned long long tw[R];
      uint32_t tkm = 0;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        tw[i] = topk_pack(atv[i], a.m_begin + a.out_row0 + rowbase + h + 2 * (g + i));
        tkm |= (okv[i] && atv[i] == atv[i] && tw[i] > tk_last) ? 1u << i : 0u;
      }
      if (__builtin_amdgcn_ballot_w64(tkm != 0)) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
          if (tkm & (1u << i)) {
            topk_insert(tkp, od.topk_k, tw[i]);
            tk_last = __atomic_load_n(tkp + od.topk_k - 1, __ATOMIC_RELAXED);
          }
        }
      }
    }
  }
  if (od.best) {  // uniform: one panel per column block
    const float ov = __shfl_xor(bv, 32);
    const int64_t om = __shfl_xor(bm, 32);
    if (ov > bv || (ov == bv && om < bm)) {
      bv = ov;
      bm = om;
    }
    if (h == 0 && colok && bv >= 0.0f) {
      // beyond |t| = 40 the table's value at 40 is a lower bound that the
      // FP64 tail kernel replaces
      const float nl = bv == INFINITY ? INFINITY : table_nlog10p(tab, bv <= kTMax ? bv : kTMax);
      atomicMax(od.best + p, best_pack(nl, bm));
    }
  }
}

// Two FP16 values (the halves of v) to OCP e4m3, round to nearest even,
// into bytes 0 and 1 (lo) or 2 and 3 (hi) of old, the other two kept.
// Written as the instruction itself: this compiler's builtin for it, given
// several calls that differ only in v, emitted the conversion of the first v
// for all of them.
__device__ __forceinline__ uint32_t cvt_pk_e4m3_lo(uint32_t old, uint32_t v) {
  asm("v_cvt_scalef32_pk_fp8_f16 %0, %1, 1.0" : "+v"(old) : "v"(v));
  return old;
}
__device__ __forceinline__ uint32_t cvt_pk_e4m3_hi(uint32_t old, uint32_t v) {
  asm("v_cvt_scalef32_pk_fp8_f16 %0, %1, 1.0 op_sel:[0,0,1]" : "+v"(old) : "v"(v));
  return old;
}

}  // namespace tgw
