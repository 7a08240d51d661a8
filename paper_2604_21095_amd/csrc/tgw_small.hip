// The contraction on small tiles: scans whose 512 x 128 tiles would leave
// most of the GPU idle (few markers, or a panel of a few columns), and the
// Q^T g contraction of the split forms.
#include "tgw_device.h"

#include <algorithm>
#include <cmath>

namespace tgw {

typedef int i32x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------
// One workgroup per tile: 4 waves of WMF 32-row fragments across WN column
// blocks of phenotypes and NQB packed hi|lo blocks of covariates.
//   MODE kTest,  NQB = 0: the scan's tests, Q^T g from a.wws / a.invh
//   MODE kTest,  NQB > 0: one panel whose columns fit in one tile: Q^T g, the
//                         markers' ||g_res|| and the tests in one pass
//   MODE kRawHL, WN = 0:  Q^T g alone (slots to a.raw_out)
// Every accumulator takes the same matrix-core steps in the same order as in
// the wide kernel (chunk by chunk; within a chunk the four K16 steps, the FP8
// lo step at the place the wide tile a.lo_tile gives it), so a test's bits do
// not depend on the tile that computed it.
//
// Rows: a lane pair (h = 0, 1) of a fragment row reads eight chunks (one
// 128-byte run of the row) at a time, 64 bytes per lane, and swaps halves
// with v_permlane32_swap, so that each lane ends up with its half of every
// chunk; the next eight chunks are requested a whole group ahead.  (8-bit
// dosages: a lane reads its own 32 bytes of a chunk, two chunks at a time.)
// Operand: staged through LDS, CS chunks per stage, two stages, the stage
// after the next one in registers; one barrier per stage.  Chunks past the
// last one are staged as zeros, which leave the accumulators as they are.
// The decode (56 VALU instructions per fragment and chunk in the FP16 + FP8
// form, about the issue time of the matrix-core steps against one column
// block) runs a step ahead of the matrix-core instructions it feeds.
//
// PHASE (cohorts of more than kSegMin chunks, whose accumulators are the sums
// of segments, added in order): 1 leaves the accumulators of one segment of a
// tile in a.part, 2 adds a tile's segments and finishes it, 0 does all of a
// shorter cohort at once.  A cohort of 500,001 samples has 8 segments: with
// 4,096 markers and 8 phenotypes, 256 workgroups instead of 32 (scan 3.92 ->
// 0.65 ms; r's error against FP64 1.5e-5 -> 1.6e-6 of its size).
// ---------------------------------------------------------------------------
template <int PREC, int MODE, int WMF, int WN, int NQB, bool G8, int PHASE>
__global__ __launch_bounds__(256, 2) void gemm_small_kernel(GemmArgs a) {
  constexpr int NW = 4, NT = NW * 64, TM = NW * WMF * 32;
  constexpr bool HL = MODE == kRawHL;
  constexpr bool F8 = PREC == kSplit8;
  constexpr bool LO16 = !F8;
  constexpr bool FUSED = MODE == kTest && NQB > 0;
  static_assert(PREC != kFP32 && MODE != kRaw && (HL ? (WN == 0 && NQB == 1) : WN >= 1), "split forms");
  static_assert(!G8 || PREC != kSplit, "8-bit dosages run the FP16 forms");
  constexpr int SB = block_bytes(PREC);      // bytes of a phenotype block's chunk
  constexpr int QB = kBlockBytes / 2;        // used bytes of a packed covariate block's chunk
  constexpr int CHB = WN * SB + NQB * QB;    // staged bytes per chunk
  constexpr int CS = 8 * CHB <= 80 * 1024 ? 4 : 4 * CHB <= 80 * 1024 ? 2 : 1;
  constexpr int STG = CS * CHB;
  constexpr int NQ = STG / (NT * 16);
  constexpr int PPF = CS * SB / 1024, PPC = SB / 1024;  // 1 KiB pieces per phenotype block and stage, per chunk
  constexpr int QPF = CS * QB / 1024, QPC = QB / 1024;
  constexpr int GCH = 8;                     // chunks per unrolled group
  static_assert(STG % (NT * 16) == 0 && GCH % (2 * CS) == 0, "stage shape");
  constexpr int QOFF = WN * CS * SB;         // covariate blocks within a stage
  // epilogue: one fragment of accumulators per wave, the rows' 1/||g_res||,
  // the p-value table, and (fused) the rows' slots
  constexpr int WSP = kSlots + 4;            // padded slots of a row
  constexpr int STAGE_BYTES = MODE == kTest ? NW * 32 * 32 * 4 : 0;
  constexpr int IH_BYTES = MODE == kTest ? TM * 8 : 0;
  constexpr int TAB_BYTES = MODE == kTest ? kTabIntervals * 16 : 0;
  constexpr int WS_BYTES = FUSED ? TM * WSP * 4 : 0;
  constexpr int EPI_BYTES = PHASE == 1 ? 0 : STAGE_BYTES + IH_BYTES + TAB_BYTES + WS_BYTES;
  constexpr int LOOP_BYTES = PHASE == 2 ? 16 : 2 * STG;
  __shared__ __attribute__((aligned(16))) char smem[LOOP_BYTES > EPI_BYTES ? LOOP_BYTES : EPI_BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5;
  const int r32 = lane & 31;
  const int64_t tiles = (int64_t)a.n_mtiles * a.n_ctiles;
  // each XCD takes an eighth of the tiles; of a segmented cohort, an eighth of
  // the whole segments' tiles (segment by segment) and then of the last one's,
  // which may be nearly empty (N = 70,001: 70 chunks after 1,024, half the
  // XCDs would have had nothing else; 10,000 markers x 600 phenotypes, FP16 + FP8: 3.08
  // against 1.92 ms)
  const int xcd = blockIdx.x & 7;
  const int64_t whole = PHASE == 1 ? tiles * (a.n_segs - 1) : 0;
  const int64_t wlo = whole * xcd / 8, wcnt = whole * (xcd + 1) / 8 - wlo;
  const int64_t slot = blockIdx.x >> 3;
  int seg = 0;
  int64_t tile_w;
  if (slot < wcnt) {
    seg = (int)((wlo + slot) / tiles);
    tile_w = wlo + slot - seg * tiles;
  } else {
    if (PHASE == 1) seg = a.n_segs - 1;
    tile_w = tiles * xcd / 8 + (slot - wcnt);
    if (tile_w >= tiles * (xcd + 1) / 8) return;
  }
  int mtile, ctile;
  grouped_tile(tile_w, a.n_mtiles, a.n_ctiles, mtile, ctile);
  ctile += a.ct0;
  // the chunks [ch_lo, nch) of this workgroup
  const int ch_lo = PHASE == 1 ? seg * a.seg_len : 0;
  const int nch = PHASE == 1 && ch_lo + a.seg_len < a.n_chunks ? ch_lo + a.seg_len : a.n_chunks;

  // this wave's 1 KiB pieces of a stage: source, chunk stride and chunk of each
  const char* bsrc[NQ];
  int bch[NQ], bstr[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int piece = q * NW + wave;
    if (piece < WN * PPF) {
      const int cb = ctile * WN + piece / (WN ? PPF : 1);
      bsrc[q] = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN].op + (piece % PPC) * 1024;
      bch[q] = (piece % (WN ? PPF : 1)) / PPC;
      bstr[q] = SB;
    } else {
      const int qp = piece - WN * PPF;
      const int qb = qp / (NQB ? QPF : 1);
      const char* wop = HL ? a.cblocks[ctile].op : (const char*)a.panels[0].wop + (int64_t)qb * a.n_chunks * kBlockBytes;
      bsrc[q] = wop + (qp % QPC) * 1024;
      bch[q] = (qp % QPF) / QPC;
      bstr[q] = kBlockBytes;
    }
  }
  u32x4 breg[NQ];
  const uint32_t lane16 = lane * 16;
  auto load_stage = [&](int ch0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int ch = ch0 + bch[q] < nch ? ch0 + bch[q] : nch - 1;
      breg[q] = gload<u32x4>(bsrc[q] + (int64_t)ch * bstr[q] + lane16);
    }
  };
  auto store_stage = [&](int buf, int ch0) __attribute__((always_inline)) {
    if (ch0 + CS > nch) {  // uniform: chunks past the last one are zero
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (ch0 + bch[q] >= nch) breg[q] = u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) *(u32x4*)(smem + buf * STG + (q * NW + wave) * 1024 + lane16) = breg[q];
  };

  const int64_t rowbase = a.row0 + (int64_t)mtile * TM + wave * (WMF * 32);
  const uint8_t* ap[WMF];
  uint2 lut[WMF];
  uint32_t lut8[WMF];
#pragma unroll
  for (int fm = 0; fm < WMF; ++fm) {
    int64_t mr = rowbase + fm * 32 + r32;
    mr = mr < a.nm ? mr : a.nm - 1;
    ap[fm] = a.geno + (a.m0 + mr) * a.row_bytes + (G8 ? 32 * h : 0);
    const uint4 l4 = gload<uint4>(a.mlut + mr);
    lut[fm] = make_uint2(l4.x, l4.y);
    lut8[fm] = l4.z;
  }
  // FP8 lo step of (fragment, column block): after K16 step los[fm][fn]
  int los[WMF][WN ? WN : 1], bscale[WN ? WN : 1];
#pragma unroll
  for (int fn = 0; fn < WN; ++fn) {
    const int cb = ctile * WN + fn;
    bscale[fn] = 127;
    if constexpr (F8) {
      const ColBlock blk = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN];
      if (cb < a.n_cblocks && r32 < blk.ncol) bscale[fn] = a.panels[blk.panel].lscale[blk.col0 + r32];
    }
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
      los[fm][fn] = G8 ? 2 : a.lo_tile == 1 ? (cb & 3) : a.lo_tile == 6 ? ((cb >> 1) & 3) : ((wave * WMF + fm) & 3);
  }

  f32x16 acc[WMF][WN ? WN : 1], accq[WMF][NQB ? NQB : 1];
#pragma unroll
  for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) acc[fm][fn][i] = 0.0f;
#pragma unroll
      for (int fq = 0; fq < NQB; ++fq) accq[fm][fq][i] = 0.0f;
    }

  // 2-bit codes: raw[fm][i] of lane half h is chunk ch0 + 4h + i whole
  auto load_rows = [&](int ch0, u32x4 (*dst)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (G8) {  // 16-byte piece i & 1 of this half's bytes of chunk ch0 + (i >> 1)
          const int ch = ch0 + (i >> 1) < nch ? ch0 + (i >> 1) : nch - 1;
          dst[fm][i] = gload<u32x4>(ap[fm] + (int64_t)ch * 64 + 16 * (i & 1));
        } else {
          const int ch = ch0 + 4 * h + i < nch ? ch0 + 4 * h + i : nch - 1;
          dst[fm][i] = gload<u32x4>(ap[fm] + (int64_t)ch * 16);
        }
      }
  };
  // then dwords 0, 1 of raw[fm][i] are this half's codes of chunk ch0 + i, and
  // dwords 2, 3 those of chunk ch0 + 4 + i
  auto swap_rows = [&](u32x4 (*raw)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const auto s = __builtin_amdgcn_permlane32_swap(raw[fm][i][d], raw[fm][i][2 + d], false, false);
          raw[fm][i][d] = s[0];
          raw[fm][i][2 + d] = s[1];
        }
  };
  // raw[0]: the current eight chunks' rows, raw[1]: the next eight's (8-bit
  // dosages: pairs of chunks, alternating)
  u32x4 raw[2][WMF][4];
  // code dword k of chunk u of the group (u = 8: the next group's first chunk)
  auto src = [&](int u, int fm, int k) __attribute__((always_inline)) -> uint32_t {
    if constexpr (G8) return raw[(u >> 1) & 1][fm][2 * (u & 1) + (k >> 2)][k & 3];
    return raw[u >> 3][fm][u & 3][((u & 7) < 4 ? 0 : 2) + (k & 1)];
  };

  u32x4 A[2][WMF];                // operand of this step and the next
  uint32_t lo4[WMF][4], hi4[WMF][4];  // operand bytes of the current code dword's sixteen samples
  i32x8 A8[F8 ? WMF : 1], A8n[F8 && !G8 ? WMF : 1];
  // bytes of the samples of code dword p of chunk u: low, high and FP8 bytes
  // of samples d, d + 4, d + 8, d + 12 sit in one dword
  auto expand = [&](int u, int p) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint32_t y = (src(u, fm, p) >> (2 * d)) & 0x03030303u;
        lo4[fm][d] = __builtin_amdgcn_perm(lut[fm].x, lut[fm].x, y);
        hi4[fm][d] = __builtin_amdgcn_perm(lut[fm].y, lut[fm].y, y);
      }
  };
  auto expand8 = [&](int u, int p) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
      for (int d = 0; d < 4; ++d)
        A8n[F8 && !G8 ? fm : 0][4 * p + d] =
            (int)__builtin_amdgcn_perm(lut8[fm], lut8[fm], (src(u, fm, p) >> (2 * d)) & 0x03030303u);
  };
  // the operand of step j of chunk u
  auto operand = [&](int u, int j, u32x4* dst) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm) {
      if constexpr (!G8) {  // samples (d, d + 8) of the dword at even steps, (d + 4, d + 12) at odd ones
#pragma unroll
        for (int d = 0; d < 4; ++d)
          dst[fm][d] = __builtin_amdgcn_perm(hi4[fm][d], lo4[fm][d], (j & 1) ? 0x07030501u : 0x06020400u);
      } else {
        const int k0 = 4 * (j >> 1) + (j & 1);
        const uint32_t D0 = src(u, fm, k0), D1 = src(u, fm, k0 + 2);
        const uint32_t M0 = ff_bytes(D0), M1 = ff_bytes(D1);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t x = __builtin_amdgcn_perm(D1, D0, 0x0c000c00u | ((4u + d) << 16) | d) | 0x64006400u;
          const uint32_t v =
              __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, x) + __builtin_bit_cast(f16x2, lut[fm].x));
          const uint32_t mk = __builtin_amdgcn_perm(M1, M0, d | (d << 8) | ((4u + d) << 16) | ((4u + d) << 24));
          dst[fm][d] = (mk & lut[fm].y) | (~mk & v);
        }
        if constexpr (F8) {  // as the wide kernel's cvt8
          const int p = j >> 1;
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            uint32_t v = (j & 1) ? (uint32_t)A8[fm][4 * p + d] : 0u;
            if (j & 1) {
              v = cvt_pk_e4m3_hi(v, dst[fm][d]);
              v = __builtin_amdgcn_perm(v, v, 0x03010200u);
            } else {
              v = cvt_pk_e4m3_lo(v, dst[fm][d]);
            }
            A8[fm][4 * p + d] = (int)v;
          }
        }
      }
    }
  };
  u32x4 bh[2][WN ? WN : 1], bl[2][WN ? WN : 1], bq[2][NQB ? NQB : 1];
  auto read_b = [&](const char* stage, int c, int j, int set) __attribute__((always_inline)) {
#pragma unroll
    for (int fn = 0; fn < WN; ++fn) {
      const char* tile = stage + (fn * CS + c) * SB;
      bh[set][fn] = *(const u32x4*)(tile + j * 1024 + lane16);
      if constexpr (LO16) bl[set][fn] = *(const u32x4*)(tile + 4096 + j * 1024 + lane16);
    }
#pragma unroll
    for (int fq = 0; fq < NQB; ++fq)
      bq[set][fq] = *(const u32x4*)(stage + QOFF + (fq * CS + c) * QB + j * 1024 + lane16);
  };

  // this wave's accumulators of a segment, [fragment and block][element][lane]
  constexpr int NACC = WMF * (WN + NQB);
  auto part_at = [&](int sg) {
    return a.part + (((int64_t)sg * tiles + tile_w) * NW + wave) * (NACC * 16 * 64) + lane;
  };
  auto each_acc = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm) {
#pragma unroll
      for (int fn = 0; fn < WN; ++fn) f(acc[fm][fn], fm * (WN + NQB) + fn);
#pragma unroll
      for (int fq = 0; fq < NQB; ++fq) f(accq[fm][fq], fm * (WN + NQB) + WN + fq);
    }
  };
  if constexpr (PHASE == 2) {
    for (int sg = 0; sg < a.n_segs; ++sg) {
      const float* p = part_at(sg);
      each_acc([&](f32x16& v, int x) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float e = gload<float>(p + (x * 16 + i) * 64);
          v[i] = sg == 0 ? e : v[i] + e;
        }
      });
    }
  } else {
    load_stage(ch_lo);
    load_rows(ch_lo, raw[0]);
    if constexpr (G8) load_rows(ch_lo + 2, raw[1]);
    store_stage(0, ch_lo);
    load_stage(ch_lo + CS);
    __syncthreads();
    if constexpr (!G8) {
      swap_rows(raw[0]);
      expand(0, 0);
      if constexpr (F8) {
        expand8(0, 0);
        expand8(0, 1);
      }
    }
    operand(0, 0, A[0]);
    read_b(smem, 0, 0, 0);
    for (int ch0 = ch_lo; ch0 < nch; ch0 += GCH) {
      if constexpr (!G8) load_rows(ch0 + GCH, raw[1]);
#pragma unroll
      for (int u = 0; u < GCH; ++u) {
        const int buf = (u / CS) & 1;
        const char* stage = smem + buf * STG;
        if (!G8 && u == 7) swap_rows(raw[1]);
        i32x8 B8[F8 ? WN : 1];
        if constexpr (F8) {
#pragma unroll
          for (int fn = 0; fn < WN; ++fn) {
            const char* tile = stage + (fn * CS + u % CS) * SB + 4096;
            const u32x4 p0 = *(const u32x4*)(tile + lane16);
            const u32x4 p1 = *(const u32x4*)(tile + 1024 + lane16);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              B8[fn][t] = (int)p0[t];
              B8[fn][4 + t] = (int)p1[t];
            }
          }
          if constexpr (!G8) {
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm) A8[fm] = A8n[fm];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int cs = j & 1, ns = cs ^ 1;
          if (j < 3) read_b(stage, u % CS, j + 1, ns);
          if (j == 3) {
            if (u % CS == CS - 1) {  // this chunk's stage is read: the next one's turn
              store_stage(buf ^ 1, ch0 + u + 1);
              load_stage(ch0 + u + 1 + CS);
              __syncthreads();
              read_b(smem + (buf ^ 1) * STG, 0, 0, ns);
            } else {
              read_b(stage, u % CS + 1, 0, ns);
            }
          }
          // decode for the next step (and the next chunk's FP8 operand)
          if constexpr (!G8) {
            if (j == 1) expand(u, 1);
            if (j == 3) expand(u + 1, 0);
            if constexpr (F8) {
              if (j == 0) expand8(u + 1, 0);
              if (j == 2) expand8(u + 1, 1);
            }
            operand(j < 3 ? u : u + 1, (j + 1) & 3, A[ns]);
          } else {
            operand(j < 3 ? u : u + 1, (j + 1) & 3, A[ns]);
            if (j == 2 && (u & 1)) load_rows(ch0 + u + 3, raw[(u >> 1) & 1]);  // this pair's codes are decoded
          }
#pragma unroll
          for (int fm = 0; fm < WMF; ++fm) {
#pragma unroll
            for (int fq = 0; fq < NQB; ++fq) accq[fm][fq] = mfma16<PREC>(A[cs][fm], bq[cs][fq], accq[fm][fq]);
#pragma unroll
            for (int fn = 0; fn < WN; ++fn) acc[fm][fn] = mfma16<PREC>(A[cs][fm], bh[cs][fn], acc[fm][fn]);
          }
          if constexpr (LO16) {
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
              for (int fn = 0; fn < WN; ++fn) acc[fm][fn] = mfma16<PREC>(A[cs][fm], bl[cs][fn], acc[fm][fn]);
          }
          if constexpr (F8) {
#pragma unroll
            for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
              for (int fn = 0; fn < WN; ++fn)
                if (G8 ? j == 2 : los[fm][fn] == j)
                  acc[fm][fn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A8[fm], B8[fn], acc[fm][fn], 0, 0, 0,
                                                                                127, 0, bscale[fn]);
          }
        }
      }
      if constexpr (!G8) {
#pragma unroll
        for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
          for (int i = 0; i < 4; ++i) raw[0][fm][i] = raw[1][fm][i];
      }
    }
    __syncthreads();  // all waves are done with the stages
  }
  if constexpr (PHASE == 1) {
    float* p = part_at(seg);
    each_acc([&](f32x16& v, int x) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 16; ++i) gstore(p + (x * 16 + i) * 64, v[i]);
    });
    return;
  }

  if constexpr (HL) {
    // slot col0 + r32, r32 < 16: hi product (column r32) plus lo product
    // (column r32 + 16); a panel's only block also zeroes the 16 slots after
    const ColBlock blk = a.cblocks[ctile];
#pragma unroll
    for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float v = accq[fm][0][i];
        const float o = __shfl_xor(v, kHLSlots);
        const int64_t mr = rowbase + fm * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
        if (mr < a.nm && r32 < blk.ncol)
          gstore(a.raw_out + mr * a.raw_ld + blk.col0 + r32, r32 < kHLSlots ? v + o : 0.0f);
      }
  } else {
    float cinv[WN], csp[WN];
#pragma unroll
    for (int fn = 0; fn < WN; ++fn) {
      const int cb = ctile * WN + fn;
      const ColBlock blk = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN];
      const PanelDev& pdb = a.panels[blk.panel];
      const bool colok = cb < a.n_cblocks && r32 < blk.ncol;
      cinv[fn] = colok ? gload<float>(pdb.invny + blk.col0 + r32) : 0.f;
      csp[fn] = colok ? gload<float>(pdb.scale + blk.col0 + r32) * a.gunit : 0.f;
    }
    float* stage = (float*)smem + wave * (32 * 32);
    float2* ihl = (float2*)(smem + STAGE_BYTES) + wave * (WMF * 32);
    float* wsl = (float*)(smem + STAGE_BYTES + IH_BYTES + TAB_BYTES) + wave * (WMF * 32 * WSP);
    if constexpr (FUSED) {
      // Q^T g of this wave's rows into LDS, then one lane per row forms
      // ||g_res|| as finalize_kernel does
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm)
#pragma unroll
        for (int fq = 0; fq < 2; ++fq)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            float v = 0.0f;
            if (fq < NQB) {
              v = accq[fm][fq < NQB ? fq : 0][i];
              v += __shfl_xor(v, kHLSlots);
            }
            if (r32 < kHLSlots) wsl[(fm * 32 + 8 * (i >> 2) + 4 * h + (i & 3)) * WSP + fq * kHLSlots + r32] = v;
          }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (lane < WMF * 32) {
        const int64_t m = rowbase + lane;
        ihl[lane] = finalize_row(a.mstat[m < a.nm ? m : a.nm - 1], wsl + lane * WSP, a.wscale, a.lo_slot, a.redo, 0,
                                 m < a.nm ? (int32_t)m : -1);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // projection correction (see gemm_kernel)
#pragma unroll
    for (int fn = 0; fn < WN; ++fn) {
      const int cb = ctile * WN + fn;
      const ColBlock blk = a.cblocks[cb < a.n_cblocks ? cb : ctile * WN];
      const float* cwp = a.panels[blk.panel].cw + (int64_t)(blk.col0 + r32) * kSlots + 8 * h;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const float4 c0 = gload<float4>(cwp + 16 * ks);
        const float4 c1 = gload<float4>(cwp + 16 * ks + 4);
        const u32x4 bo = {pack_bf16x2(c0.x, c0.y), pack_bf16x2(c0.z, c0.w), pack_bf16x2(c1.x, c1.y),
                          pack_bf16x2(c1.z, c1.w)};
#pragma unroll
        for (int fm = 0; fm < WMF; ++fm) {
          tab4 w0, w1;
          if constexpr (FUSED) {
            const tab4* wp = (const tab4*)(wsl + (fm * 32 + r32) * WSP + 16 * ks + 8 * h);
            w0 = wp[0];
            w1 = wp[1];
          } else {
            int64_t mr = rowbase + fm * 32 + r32;
            mr = mr < a.nm ? mr : a.nm - 1;
            const float* wp = a.wws + (mr * a.n_panels + blk.panel) * kSlots + 16 * ks + 8 * h;
            w0 = gload<tab4>(wp);
            w1 = gload<tab4>(wp + 4);
          }
          const u32x4 ao = {pack_bf16x2(w0.x, w0.y), pack_bf16x2(w0.z, w0.w), pack_bf16x2(w1.x, w1.y),
                            pack_bf16x2(w1.z, w1.w)};
          acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ao),
                                                                __builtin_bit_cast(bf16x8, bo), acc[fm][fn], 0, 0, 0);
        }
      }
    }
    // 32 x 32 accumulators at a time through this wave's 4 KiB of LDS; the
    // rows' 1/||g_res|| and the p-value table of the block's panel in LDS too
    int panel = -1;  // whose rows and table are in LDS (uniform)
#pragma unroll
    for (int fn = 0; fn < WN; ++fn) {
      const int cb = ctile * WN + fn;
      if (cb >= a.n_cblocks) break;
      const ColBlock blk = a.cblocks[cb];
      if (blk.panel != panel) {
        panel = blk.panel;
        __syncthreads();
        if constexpr (!FUSED) {
          for (int k = lane; k < WMF * 32; k += 64) {
            int64_t mr = rowbase + k;
            mr = mr < a.nm ? mr : a.nm - 1;
            ihl[k] = gload<float2>(a.invh + mr * a.n_panels + panel);
          }
        }
        tab4* tl = (tab4*)(smem + STAGE_BYTES + IH_BYTES);
        const tab4* tg = (const tab4*)a.panels[panel].table;
        for (int k = tid; k < kTabIntervals; k += NT) tl[k] = gload<tab4>(tg + k);
        __syncthreads();
      }
#pragma unroll
      for (int fm = 0; fm < WMF; ++fm) {
#pragma unroll
        for (int i = 0; i < 16; ++i) stage[(8 * (i >> 2) + 4 * h + (i & 3)) * 32 + r32] = acc[fm][fn][i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        finish_block<1>(stage, a, blk, rowbase + fm * 32, h, r32, (LdsTable)(smem + STAGE_BYTES + IH_BYTES),
                        (LdsRows)(ihl + fm * 32), cinv[fn], csp[fn]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
  }
}

// {waves, fragments per wave, column blocks} of the compiled shapes
static const TileShape kSmall[] = {{4, 1, 1}, {4, 2, 1}, {4, 1, 2}, {4, 2, 2}, {4, 1, 4}};
constexpr int kNumSmall = sizeof(kSmall) / sizeof(kSmall[0]);
int n_small_shapes() { return kNumSmall; }
TileShape small_shape(int idx) { return kSmall[idx]; }

// What a marker block costs on a tile shape, in cycles at 2.4 GHz: per round of
// the tiles over the CUs a fixed part (prologue, epilogue) and a part per
// 64-sample chunk; `alone` with one tile per CU at the most, `shared` per tile
// with more.  Fitted to 1,987 scans per shape and form (dense outputs or the
// best test: N = 500 to 65,000, 500 to 100,000 markers, 65 to 20,480
// phenotypes), whose times it gives to 3 % (one standard deviation) from N =
// 4,000 on.  The wide tile computes a 32 x 32 block in 240 cycles (FP16 + FP8)
// against 330 to 460 here, but spends ten times as much on a tile's fixed part
// and leaves CUs idle where its tiles number less than the CUs, and in its
// last round.
namespace {
struct Cost {
  double kfixed, chunk;  // thousand cycles, cycles
};
struct TileCost {
  Cost wide, alone[kNumSmall], shared[kNumSmall];
};
const TileCost& tile_cost(int prec, bool g8) {
  static const TileCost f8 = {{165, 3730}, {{0, 680}, {8, 1170}, {11, 1030}, {32, 2010}, {26, 1740}},
                              {{2, 460}, {6, 900}, {7, 800}, {14, 1330}, {14, 1330}}};
  static const TileCost f8_g8 = {{140, 8600}, {{0, 1110}, {12, 2050}, {12, 1380}, {32, 2600}, {26, 1860}},
                                 {{2, 950}, {5, 1910}, {5, 1240}, {18, 2300}, {16, 1790}}};
  static const TileCost f16 = {{165, 5020}, {{0, 730}, {11, 1080}, {10, 1250}, {30, 1820}, {24, 2270}},
                               {{2, 570}, {4, 950}, {6, 1020}, {10, 1600}, {12, 1880}}};
  static const TileCost f16_g8 = {{220, 9240}, {{0, 1250}, {10, 2030}, {10, 1740}, {30, 2620}, {26, 2830}},
                                  {{4, 900}, {8, 1710}, {6, 1420}, {13, 2380}, {16, 2340}}};
  static const TileCost bf16 = {{165, 5010}, {{0, 740}, {8, 1100}, {9, 1260}, {29, 1840}, {24, 2270}},
                                {{2, 570}, {4, 940}, {4, 1010}, {12, 1600}, {11, 1860}}};
  static const TileCost fp32 = {{105, 43700}, {{5, 2960}, {6, 6650}, {0, 6460}, {20, 12310}, {24, 10910}},
                                {{0, 3150}, {0, 6350}, {4, 5980}, {6, 11550}, {16, 10610}}};
  static const TileCost fp32_g8 = {{110, 41200}, {{2, 2800}, {12, 6000}, {6, 6350}, {28, 11640}, {22, 10940}},
                                   {{0, 2760}, {0, 5610}, {8, 5530}, {12, 10770}, {29, 9660}}};
  if (prec == kFP32) return g8 ? fp32_g8 : fp32;
  return prec == kSplit8 ? (g8 ? f8_g8 : f8) : prec == kSplit16 ? (g8 ? f16_g8 : f16) : bf16;
}
int64_t n_tiles(int64_t nm, int n_cb, const TileShape& t) {
  return (nm + t.tm() - 1) / t.tm() * ((n_cb + t.wn_frags - 1) / t.wn_frags);
}
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
constexpr TileShape kWide{4, 4, 4};
constexpr double kSegFlush = 20e3;  // adding a segment to the sums in memory

double wide_cycles(const ScanShape& s) {
  const Cost& c = tile_cost(s.prec, s.g8).wide;
  return s.wide_rel * (double)ceil_div(n_tiles(s.nm, s.n_cb, kWide), s.n_cu) *
         (1e3 * c.kfixed + s.n_chunks * c.chunk + (s.n_segs - 1) * kSegFlush);
}
// one launch (a pair of them above one segment) of `tiles`
double launch_cycles(const ScanShape& s, int i, int64_t tiles) {
  const TileCost& c = tile_cost(s.prec, s.g8);
  const double one = 1e3 * c.alone[i].kfixed + std::min(s.seg_len, s.n_chunks) * c.alone[i].chunk;
  const int64_t wgs = tiles * s.n_segs;
  if (wgs <= s.n_cu) return one;
  double chunks = (double)ceil_div(wgs, s.n_cu) * s.n_chunks;  // of the fullest CU
  if (s.n_segs > 1) {  // the last segments fill up the CUs that have fewer whole ones
    const int64_t whole = tiles * (s.n_segs - 1);
    chunks = std::max((double)ceil_div(whole, s.n_cu) * s.seg_len, (double)tiles * s.n_chunks / s.n_cu);
  }
  return std::max(one, ceil_div(wgs, s.n_cu) * 1e3 * c.shared[i].kfixed + chunks * c.shared[i].chunk);
}
// Segmented scans take a launch for as many tiles as the buffer for the
// segments' sums holds, as launch_gemm_small cuts them.  The last one can be a
// few tiles that cost a whole round: FP16 + FP8, N = 80,000, 2,000 markers x
// 4,300 phenotypes on 256 x 64 tiles are 512 + 32 tiles and take 3.43 ms, on
// wide ones 2.82.
double small_cycles(const ScanShape& s, int i) {
  const TileShape& t = kSmall[i];
  if (s.n_segs <= 1) return launch_cycles(s, i, n_tiles(s.nm, s.n_cb, t));
  const int64_t nm = ceil_div(s.nm, t.tm()), nc = ceil_div(s.n_cb, t.wn_frags);
  const int64_t fit = s.part_bytes / ((int64_t)t.waves * t.wm_frags * t.wn_frags * 4096 * s.n_segs);
  const int64_t c = std::max<int64_t>(1, std::min(nc, fit)), m = std::max<int64_t>(1, fit / c);
  double sum = (double)(nm / m) * (nc / c) * launch_cycles(s, i, std::min(m, nm) * c);
  if (nm % m) sum += (double)(nc / c) * launch_cycles(s, i, nm % m * c);
  if (nc % c) sum += (double)nm * launch_cycles(s, i, nc % c);  // then m is 1
  return sum;
}

// Filling top-k lists: microseconds per list entry that a shape takes more (or
// less) than the wide tile.  Every wave runs the serial insertions of its own
// rows, column block by column block: few columns per wave are the faster ones
// (500 markers x 2,000 phenotypes, k = 50: 512 x 128 tiles 5.4 ms, 256 x 32
// 0.9, 128 x 32 0.7).  But each wave starts on the list as it stands, so many
// waves with few rows each insert what others displace (one phenotype, 100,000
// markers, k = 50, N = 500: 1.0 ms on wide tiles, 1.6 on 256 x 32, 2.2 on 128 x
// 32), most of all in one burst, where the contraction is short.  The
// register-staged default tiles of FP32 and of 8-bit dosages in the FP16 split
// have half the rows per wave.
// Above two column blocks the terms are a least-squares fit to 2,620 scans
// (N = 500 to 60,000, 500 to 60,000 markers, 65 to 20,480 phenotypes, k = 1,
// 10, 50), kept within the range that they were fitted to.  The shape they
// give takes 1.3 % longer than the fastest one on average (25 % at the most),
// and four of the scans are more than 5 % slower than on the wide tile (14 % at
// the most).  Without any term for the lists it is 7.6 % (94 %), and up to 1.55
// times the wide tile's time.
struct InsertFit {
  double one, m, mm, n, rounds, p, pn, p4;
};
const InsertFit* insert_fit(bool fp32) {
  static const InsertFit f16[kNumSmall] = {{-45, 21.2, -4.9, -1.1, -5.4, 15.9, -1.07, 10.5},
                                           {-43, 18.7, -3.7, -0.5, -6, 9.6, -1.37, 4.6},
                                           {-33, 22.3, -4.5, -0.7, -7.1, 16.9, -1.08, 4.1},
                                           {-34, 17.5, -2.7, -0.6, -5.7, 8.4, -0.57, 0.1},
                                           {-24, 23, -1.5, -0.9, -8.5, 14, -0.61, -0.3}};
  static const InsertFit f32[kNumSmall] = {{-27, 9.2, -3.8, 1.9, -4.4, 9.2, -1.87, 9.8},
                                           {-23, 6.4, -2.8, 2.8, -6.3, 5, -2.08, -0.5},
                                           {-17, 10.7, -3.5, 3.3, -5, 13.6, -1.28, 3},
                                           {-17, 4.9, -2.6, 2.5, -2.4, 6.2, -0.72, -2},
                                           {-10, 10.2, -0.8, 2.4, -4.6, 11.1, -0.19, -0.3}};
  return fp32 ? f32 : f16;
}
double insert_us(const ScanShape& s, int i) {
  const double m = (double)s.nm;
  const bool half = s.prec == kFP32 || (s.prec == kSplit16 && s.g8);
  if (s.n_cb <= 2) {
    double narrow;  // 256 x 32
    if (half)
      narrow = 0.0;
    else if (s.n_cb == 2)
      narrow = 1.5e-4 * m - 5.0;
    else
      narrow = 1.3e-4 * m * (n_tiles(s.nm, 1, kSmall[1]) > s.n_cu ? std::max(0.0, 1.0 - s.n_chunks / 128.0) : 1.0) +
               (m > 15000 ? 7.0 : 0.0);
    if (i == 1) return narrow;
    if (s.n_cb == 1) return narrow + std::min(5e-4 * m, 20.0) - 1.5;
    return s.prec == kFP32 ? narrow : narrow + std::min(4e-4 * m, 16.0) - 4.0;
  }
  const InsertFit& f = insert_fit(s.prec == kFP32)[i];
  const double lm = std::log(std::clamp(m, 500.0, 40000.0) / 3000.0);
  const double ln = std::log(std::clamp((double)s.n_chunks, 8.0, 1000.0) / 64.0);
  const double p = std::min(32.0 * s.n_cb, 20480.0) / 4000.0;
  const double rounds = (double)std::min<int64_t>(ceil_div(n_tiles(s.nm, s.n_cb, kWide), s.n_cu), 12);
  return f.one + f.m * lm + f.mm * lm * lm + f.n * ln + f.rounds * rounds + f.p * p + f.pn * p * ln +
         f.p4 * std::min(p, 1.0);
}
}  // namespace

// Q^T g beside the tests saves the second decode of the genotypes (a third
// of the two kernels' time) and two launches; the panel's columns then have
// to fit in one tile.  One column block and one covariate block: two
// fragments per wave halve the operand reads (1,450 cycles per tile against
// 2 x 830), but 256-row tiles leave more of the last round empty.  Of 592
// scans (dense outputs or the best test, N = 500 to 60,000, up to 100,000
// markers) all take at most 0.9 of the wide tile's time.
static int small_fused_shape(const ScanShape& s) {
  if (s.n_cb == 2) return 2;
  if (s.nqb > 1 || s.g8) return 0;
  const int64_t r0 = ceil_div(n_tiles(s.nm, 1, kSmall[0]) * s.n_segs, s.n_cu);
  const int64_t r1 = ceil_div(n_tiles(s.nm, 1, kSmall[1]) * s.n_segs, s.n_cu);
  return r1 * (r1 > 1 ? 1450 : 1720) < r0 * (r0 > 1 ? 830 : 1000) ? 1 : 0;
}

// A small tile has to be 1 % faster by the estimate (FP16 + FP8, N = 60,000,
// 10,000 markers x 1,000 phenotypes: 2.28 ms on the 128 x 64 tiles, 2.00 on the
// wide ones).  10 % above 65,536 samples, where the estimate is rougher: of 718
// such scans nine are then more than 2 % slower than on wide tiles (9 % at the
// most), twenty with 1 %.  10 % also for top-k lists of long sums in FP16 +
// FP8: half a round of its wide tiles runs at a higher clock than a full chip
// of small ones (N = 48,190, 985 markers x 8,419 phenotypes, k = 1: 1.68 ms
// against 1.85 to 2.00), and of 514 top-k scans three are then more than 5 %
// slower than on wide tiles (10 % at the most), ten (19 %) with 1 %.  For the
// other forms and for 8-bit dosages neither figure changes.
static double small_margin(const ScanShape& s) {
  return s.n_chunks > kSegMin || (s.topk_k > 0 && s.prec == kSplit8 && !s.g8 && s.n_chunks > 200) ? 0.9 : 0.99;
}
SmallChoice small_choice(const ScanShape& s) {
  const bool fusable = s.prec != kFP32 && s.nqb > 0 && s.n_cb <= 2;
  if (fusable && s.topk_k == 0) return SmallChoice{small_fused_shape(s), true};
  double wide = wide_cycles(s);
  SmallChoice best;
  double least = 0.0;
  auto offer = [&](int i, bool fused, double t) {
    if (best.shape < 0 || t < least) least = t, best = SmallChoice{i, fused};
  };
  const bool lists = s.topk_k > 0, one_block = fusable && s.n_cb == 1;
  // the separate Q^T g that a fused shape saves
  const double q = one_block ? 0.8 * s.nqb * std::min(small_cycles(s, 0), small_cycles(s, 1)) : 0.0;
  wide += q;
  for (int i = 0; i < kNumSmall; ++i) {
    if (lists && s.n_cb <= 2 && i > 1) break;
    const double t = small_cycles(s, i) + (lists ? 2400.0 * s.topk_k * insert_us(s, i) : 0.0);
    if (one_block && (i == 0 || (s.nqb == 1 && !s.g8)))
      offer(i, true, t);
    else
      offer(i, false, t + q);
  }
  return least < small_margin(s) * wide ? best : SmallChoice{};
}

// 256-row tiles once they fill the GPU (100,000 markers, N = 23,000: 0.21 ms
// against 0.25 ms on 128-row ones), else 128-row ones (4,096 markers, N =
// 500,001 in one segment: 2.0 against 3.2 ms)
int small_q_shape(int prec, int64_t nm, int n_cb, int n_segs, int n_cu) {
  return prec != kFP32 && n_tiles(nm, n_cb, kSmall[1]) * n_segs > n_cu ? 1 : 0;
}

template <int PREC, int NQB, bool G8, int PH>
static const void* small_fn(int idx) {
  switch (idx) {
    case 0: return (const void*)gemm_small_kernel<PREC, kTest, 1, 1, NQB, G8, PH>;
    case 1:
      if constexpr (NQB < 2 && !(G8 && NQB)) return (const void*)gemm_small_kernel<PREC, kTest, 2, 1, NQB, G8, PH>;
      return nullptr;
    case 2: return (const void*)gemm_small_kernel<PREC, kTest, 1, 2, NQB, G8, PH>;
    case 3:
      if constexpr (NQB == 0) return (const void*)gemm_small_kernel<PREC, kTest, 2, 2, NQB, G8, PH>;
      return nullptr;
    case 4:
      if constexpr (NQB == 0) return (const void*)gemm_small_kernel<PREC, kTest, 1, 4, NQB, G8, PH>;
      return nullptr;
  }
  return nullptr;
}

template <int PREC, bool G8, int PH>
static const void* small_fn_q(int idx, int nqb) {
  return nqb == 0   ? small_fn<PREC, 0, G8, PH>(idx)
         : nqb == 1 ? small_fn<PREC, 1, G8, PH>(idx)
                    : small_fn<PREC, 2, G8, PH>(idx);
}

template <int PREC, bool G8, int PH>
static const void* small_hl_fn(int idx) {
  return idx == 0   ? (const void*)gemm_small_kernel<PREC, kRawHL, 1, 0, 1, G8, PH>
         : idx == 1 ? (const void*)gemm_small_kernel<PREC, kRawHL, 2, 0, 1, G8, PH>
                    : nullptr;
}

template <int PH>
static const void* small_kernel(int idx, int prec, int mode, int nqb, bool g8) {
  if (mode == kRawHL) {
    if (prec == kSplit16) return g8 ? small_hl_fn<kSplit16, true, PH>(idx) : small_hl_fn<kSplit16, false, PH>(idx);
    if constexpr (PH == 0)
      if (prec == kSplit && !g8) return small_hl_fn<kSplit, false, PH>(idx);
  } else if (mode == kTest) {
    if (prec == kSplit8) return g8 ? small_fn_q<kSplit8, true, PH>(idx, nqb) : small_fn_q<kSplit8, false, PH>(idx, nqb);
    if (prec == kSplit16)
      return g8 ? small_fn_q<kSplit16, true, PH>(idx, nqb) : small_fn_q<kSplit16, false, PH>(idx, nqb);
    if constexpr (PH == 0)
      if (prec == kSplit && !g8) return small_fn_q<kSplit, false, PH>(idx, nqb);
  }
  return nullptr;
}

// whole: workgroups of the segments before the last (phase 1)
static hipError_t launch_tiles(const void* fn, const GemmArgs& a, int64_t tiles, hipStream_t s, int64_t whole = 0) {
  if (!fn) return hipErrorInvalidValue;
  const int64_t grid = (whole + 7) / 8 * 8 + (tiles + 7) / 8 * 8;  // what the fullest XCD's ranges hold, from each
  GemmArgs arg = a;
  void* params[] = {&arg};
  return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(256), params, 0, s);
}

// workgroups per launch: a grid holds less than 2^32 threads
constexpr int64_t kMaxGroups = int64_t(1) << 23;

hipError_t launch_gemm_small(int idx, int prec, int mode, int nqb, const GemmArgs& a, hipStream_t s, bool g8) {
  if (prec == kFP32)  // these walk their tiles
    return launch_tiles(gemm_small_fp32_fn(idx, mode, g8), a,
                        std::min((int64_t)a.n_mtiles * a.n_ctiles, kMaxGroups), s);
  // as many tiles at a time as a launch takes and a.part holds the segments of:
  // whole rows of column tiles where one row fits, else parts of a row
  const TileShape t = kSmall[idx];
  int64_t fit = kMaxGroups;
  if (a.n_segs > 1)
    fit = std::min(fit / a.n_segs, a.part_bytes / ((int64_t)t.waves * t.wm_frags *
                                                   (mode == kRawHL ? 1 : t.wn_frags + nqb) * 4096 * a.n_segs));
  if (fit < 1) return hipErrorInvalidValue;
  const int nc = (int)std::min<int64_t>(a.n_ctiles, fit);
  const int64_t nm = fit / nc;
  hipError_t e = hipSuccess;
  for (int64_t m0 = 0; e == hipSuccess && m0 < a.n_mtiles; m0 += nm)
    for (int c0 = 0; e == hipSuccess && c0 < a.n_ctiles; c0 += nc) {
      GemmArgs b = a;
      b.row0 = m0 * t.tm();
      b.ct0 = c0;
      b.n_mtiles = (int)std::min<int64_t>(nm, a.n_mtiles - m0);
      b.n_ctiles = std::min(nc, a.n_ctiles - c0);
      const int64_t n = (int64_t)b.n_mtiles * b.n_ctiles;
      if (a.n_segs <= 1) {
        e = launch_tiles(small_kernel<0>(idx, prec, mode, nqb, g8), b, n, s);
        continue;
      }
      e = launch_tiles(small_kernel<1>(idx, prec, mode, nqb, g8), b, n, s, n * (a.n_segs - 1));
      if (e == hipSuccess) e = launch_tiles(small_kernel<2>(idx, prec, mode, nqb, g8), b, n, s);
    }
  return e;
}

}  // namespace tgw
