// Wide-tile protected GEMM for gfx950 (bf16 operands): the layer's unbatched
// products, with the same checksum algebra as gemm_abft.hip (the column
// checksums A^c of the tile's row blocks as extra MFMA rows, the row checksums
// B^r as extra MFMA columns, both from their bf16 hi/lo images).
//
// What bounds these products is the data each MFMA needs. A 128 x 128 tile
// asks L2 for one byte per 64 flop, which at the matrix cores' rate is all it
// has, and waves of 128 x 32 ask the LDS for 320 cycles of reads per 256
// cycles of MFMA; a 256 x 256 tile of eight 128 x 64 waves halves the first
// and brings the second to 192. Two waves per SIMD; each 64-deep step has one
// barrier, in its middle: before it a wave reads the step's second half of
// fragments while it multiplies the first half, after it the next step's
// first half while it multiplies the second, so no wave waits for LDS, and
// the stage all waves have finished reading is refilled at once (a whole step
// ahead of its use). At 8192 x 12288 x 4096 with checks 1002 -> 714 us (1.15
// PFLOP/s; the vendor library without checks 641), dX with dWqkv of that layer
// 1891 -> 1392, at 8192 x 2304 x 768 (128 x 128 tiles, this pipeline) 57 -> 47.
#include <algorithm>

#include "abft_internal.hpp"
#include "abft_device.hpp"
#include "direct_lds.hpp"
#include "wide_copy.hpp"

namespace abft {
namespace {

typedef short short8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ const GemmDesc& wide_desc(int slot) {
#if defined(__HIP_DEVICE_COMPILE__)
  auto gp = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(gp));
  return *((const GemmDesc*)gp + slot);
#else
  return *static_cast<const GemmDesc*>(nullptr);  // the host pass emits no device code
#endif
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

__device__ __forceinline__ void wg_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One operand of a workgroup: its runs (WideRuns) shared among the NW waves.
// In both images the lanes an LDS read serves together hit different banks.
template <bool KMAJ, int ROWS, int NW>
struct Opnd : WideRuns<KMAJ> {
  static constexpr int BYTES = ROWS * 128;
  static constexpr int PER = ROWS / 8 / NW;  // runs per wave
  static_assert(ROWS % (8 * NW) == 0, "whole runs per wave");
};

// K-major fragment (MFMA 16x16x32 operand): row lane % 16 of the 16 at
// `off`, k = 32 kk + 8 (lane / 16) + 0..7
__device__ __forceinline__ int kfrag_off(int lane, int kk) {
  const int r = lane & 15, g = lane >> 4;
  return r * 128 + (((4 * kk + g) ^ (r & 7)) << 4);
}
// MN-major: the two transposing reads of the same fragment (rows rb..rb+15)
__device__ __forceinline__ int tfrag_off(int lane, int rb) {
  const int s = lane & 15, g = lane >> 4, t = (s >> 2) & 3;
  const int b = (rb >> 4) & 3, e = (s & 3) >> 1;
  return (rb >> 6) * 8192 + (8 * g + (s >> 2)) * 128 + ((2 * (b ^ t) + e) << 4) + (s & 1) * 8;
}
__device__ __forceinline__ bf16x8 lds_k(const char* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ bf16x8 lds_t(const char* p) {
  const short4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p);
  const short4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p + 4 * 128));
  const short8_t v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, v);
}
__device__ __forceinline__ floatx4 mma(const bf16x8& a, const bf16x8& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// sum over the four 16-lane groups (the lanes sharing lane % 16)
__device__ __forceinline__ float groups_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  x += __shfl_xor(x, 32, 64);
  return x;
}

struct WideCoord {
  int op, b, h, row, col;
};
__device__ __forceinline__ WideCoord wide_coord(const CoordMap& mp, int m, int n) {
  WideCoord c;
  c.op = mp.op_base + n / mp.op_span;
  const int nn = n % mp.op_span;
  c.b = mp.rows_per_b ? m / mp.rows_per_b : 0;
  c.row = mp.rows_per_b ? m % mp.rows_per_b : m;
  c.h = mp.head_cols ? nn / mp.head_cols : 0;
  c.col = mp.head_cols ? nn % mp.head_cols : nn;
  return c;
}
__device__ __forceinline__ bool wide_fault(const CoordMap& mp, int N, const abft_fault& f, int* m,
                                           int* n) {
  const int nops = (N + mp.op_span - 1) / mp.op_span;
  if (f.op < mp.op_base || f.op >= mp.op_base + nops) return false;
  *m = mp.rows_per_b ? f.b * mp.rows_per_b + f.row : f.row;
  *n = (f.op - mp.op_base) * mp.op_span + (mp.head_cols ? f.h * mp.head_cols : 0) + f.col;
  return true;
}

// TC: output type (bf16, or fp32 for the weight gradients); WGM x WGN waves
// of 128 x 16 JN outputs; two LDS stages of 64 k each.
template <class TC, bool AK, bool BKM, int WGM, int WGN, int JN, bool PROT>
struct Wide {
  static constexpr int NST = 2;
  static constexpr int IM = 8, WM = 128, WN = 16 * JN;
  static constexpr int BM = WM * WGM, BN = WN * WGN, NW = WGM * WGN, NTH = 64 * NW;
  using OA = Opnd<AK, BM, NW>;
  using OB = Opnd<BKM, BN, NW>;
  // strips: the column strip holds 4 rows per checksum block of 32 rows or
  // more, the row strip 4 per block of 64 columns or more
  static constexpr int CS_ROWS = 16, RS_ROWS = 16;
  static constexpr int OFF_B = OA::BYTES, OFF_C = OFF_B + OB::BYTES;
  static constexpr int OFF_R = OFF_C + (PROT ? CS_ROWS * 128 : 0);
  static constexpr bool HAS_RS = PROT && sizeof(TC) == 2 && AK && !BKM;  // the QKV product
  static constexpr int STAGE = OFF_R + (HAS_RS ? RS_ROWS * 128 : 0);
  static constexpr int NPER = OA::PER + OB::PER;
  // epilogue: the rounded tile (bf16 outputs), the propagated checksums
  static constexpr int LDT = BN + 8;
  static constexpr int TILE = sizeof(TC) == 2 ? BM * LDT * 2 : 0;
  static constexpr int CCV = PROT ? 4 * BN * 8 : 0;
  static constexpr int LDS = std::max(NST * STAGE, TILE + CCV);
  static_assert(LDS <= 160 * 1024, "fits the LDS");
  // the waves sharing a column range split its strip columns
  static constexpr int JS = (JN + WGM - 1) / WGM, IS = IM / WGN;

  struct Frags {
    bf16x8 a[IM], b[JN];
  };

  __device__ static __forceinline__ void run(const GemmDesc& g, char* smem, int lin, int total,
                                             int slot) {
    // tile: one contiguous range per XCD, walked in bands of 1024 rows
    const int ntm = (g.M + BM - 1) / BM, ntn = (g.N + BN - 1) / BN;
    const int q = total / 8, rem = total % 8, x = lin % 8, jx = lin / 8;
    const int v = x * q + min(x, rem) + jx, per = ntm * ntn;
    const int kslice = v / per, r = v % per;
    constexpr int GM = 1024 / BM;
    const int band = r / (GM * ntn), idx = r % (GM * ntn);
    const int rows_in_band = min(GM, ntm - band * GM);
    const int m0 = (band * GM + idx % rows_in_band) * BM, n0 = (idx / rows_in_band) * BN;
    if constexpr (HAS_RS) {
      if (g.Br != nullptr && n0 >= g.cr_n_begin) {
        body<true>(g, smem, m0, n0, kslice, slot);
        return;
      }
    }
    body<false>(g, smem, m0, n0, kslice, slot);
  }

  // ROWSTRIP: the tile carries the row strip (V tiles of the QKV product)
  template <bool ROWSTRIP>
  __device__ static __forceinline__ void body(const GemmDesc& g, char* smem, int m0, int n0,
                                              int kslice, int slot) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6), wm = wave / WGN, wn = wave % WGN;
    const int M = g.M, N = g.N, K = g.K;
    const bool split = sizeof(TC) == 4 && g.splitk > 1;
    int k_lo = 0, k_hi = K;
    if (split) {
      const int kc = ((K + g.splitk - 1) / g.splitk + 63) / 64 * 64;
      k_lo = min(K, kslice * kc);
      k_hi = min(K, k_lo + kc);
    }
    const int nk = (k_hi - k_lo + 63) / 64;

    const int lg_rm = __builtin_ctz(g.Rm), lg_rn = __builtin_ctz(g.Rn);
    // copies: operand runs, then the strips' runs (waves 0.. the column
    // strip's, the next waves the row strip's)
    const uint32_t lda = uint32_t(g.lda) * 2, ldb = uint32_t(g.ldb) * 2;
    const u32x4 ra = rsrc_of(g.A, uint32_t(AK ? M : K) * lda);
    const u32x4 rb = rsrc_of(g.B, uint32_t(BKM ? N : K) * ldb);
    const uint32_t va = OA::lane_part(lda, lane), vb = OB::lane_part(ldb, lane);
    const uint32_t lds0 = lds_addr(smem);
    int srun = -1;            // this wave's strip run
    bool srow = false;        // of the row strip
    u32x4 rs = ra;
    uint32_t vs = 0;
    if (PROT) {
      const int wc = ((4 * BM >> lg_rm) + 7) / 8;
      const int wr = ROWSTRIP ? ((4 * BN >> lg_rn) + 7) / 8 : 0;
      if (wave < wc) {
        srun = wave;
        const uint32_t ld = uint32_t(g.ldaci) * 2;
        rs = rsrc_of(g.Aci, uint32_t(4 * (M >> lg_rm)) * ld);
        vs = wide_strip_part(ld, 4 * (m0 >> lg_rm) + 8 * srun, 4 * (M >> lg_rm), lane);
      } else if (wave < wc + wr) {
        srun = wave - wc;
        srow = true;
        const uint32_t ld = uint32_t(g.ldbri) * 2;
        const int rows = 4 * ((N - g.cr_n_begin) >> lg_rn);
        rs = rsrc_of(g.Bri, uint32_t(rows) * ld);
        vs = wide_strip_part(ld, 4 * ((n0 - g.cr_n_begin) >> lg_rn) + 8 * srun, rows, lane);
      }
    }
    const bool sx = PROT && srun >= 0;
    const uint32_t lds_s = uni(lds0 + (srow ? OFF_R : OFF_C) + srun * 1024);
    uint32_t sa[OA::PER], sb[OB::PER];
#pragma unroll
    for (int j = 0; j < OA::PER; ++j)
      sa[j] = OA::run_part(lda, m0, M, wave * OA::PER + j) + uint32_t(k_lo) * OA::k_part(lda);
#pragma unroll
    for (int j = 0; j < OB::PER; ++j)
      sb[j] = OB::run_part(ldb, n0, N, wave * OB::PER + j) + uint32_t(k_lo) * OB::k_part(ldb);
    const uint32_t ss = uint32_t(k_lo) * 2;
    const uint32_t ka = 64 * OA::k_part(lda), kb = 64 * OB::k_part(ldb);
    const uint32_t la0 = lds0 + wave * (OA::PER * 1024);
    const uint32_t lb0 = lds0 + OFF_B + wave * (OB::PER * 1024);
    auto issue = [&](int kt) {
      const uint32_t st = uint32_t(kt % NST) * STAGE;
#pragma unroll
      for (int j = 0; j < OA::PER; ++j)
        dma16(ra, la0 + st + j * 1024, va, sa[j] + uint32_t(kt) * ka);
#pragma unroll
      for (int j = 0; j < OB::PER; ++j)
        dma16(rb, lb0 + st + j * 1024, vb, sb[j] + uint32_t(kt) * kb);
      if (sx) dma16(rs, lds_s + st, vs, ss + uint32_t(kt) * 128);
    };
    floatx4 acc[IM][JN], accs[JS], accr[IS];
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < JS; ++j) accs[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < IS; ++i) accr[i] = floatx4{0.f, 0.f, 0.f, 0.f};

    // fragment offsets within a stage (kk = 0; kk = 1 flips the K-major
    // chunk's bit 2, moves MN-major rows 32 down)
    const int ak0 = AK ? wm * (WM * 128) + kfrag_off(lane, 0) : 0;
    const int ak1 = AK ? wm * (WM * 128) + kfrag_off(lane, 1) : 0;
    int at[4], bt[JN];
    if constexpr (!AK) {
#pragma unroll
      for (int b = 0; b < 4; ++b) at[b] = tfrag_off(lane, wm * WM + 16 * b);
    }
    const int bk0 = OFF_B + wn * (WN * 128) + kfrag_off(lane, 0);
    const int bk1 = OFF_B + wn * (WN * 128) + kfrag_off(lane, 1);
    if constexpr (!BKM) {
#pragma unroll
      for (int j = 0; j < JN; ++j) bt[j] = OFF_B + tfrag_off(lane, wn * WN + 16 * j);
    }
    const int cs0 = OFF_C + kfrag_off(lane, 0), cs1 = OFF_C + kfrag_off(lane, 1);
    const int rs0 = OFF_R + kfrag_off(lane, 0), rs1 = OFF_R + kfrag_off(lane, 1);

    auto read_a = [&](const char* st, int i, int kk) {
      if constexpr (AK) return lds_k(st + (kk ? ak1 : ak0) + i * 2048);
      else return lds_t(st + at[i & 3] + (i >> 2) * 8192 + kk * 4096);
    };
    auto read_b = [&](const char* st, int j, int kk) {
      if constexpr (BKM) return lds_k(st + (kk ? bk1 : bk0) + j * 2048);
      else return lds_t(st + bt[j] + kk * 4096);
    };
    // MFMAs of one 32-deep step from `c` while the fragments of another
    // step (stage st, half kk) are read into `n`, spread over the groups of
    // MFMAs so that few registers beyond one step's are live. The strips'
    // fragments have one set of registers: used, then read again.
    bf16x8 fcs, frs;
    auto phase = [&](Frags& c, Frags& n, const char* st, int kk) {
#pragma unroll
      for (int i = 0; i < IM; ++i) {
        // reads done before group i: 2 at first, all JN + IM before the last
        constexpr int TOT = JN + IM;
#pragma unroll
        for (int q = i == 0 ? 0 : 2 + (i - 1) * (TOT - 2) / (IM - 1); q < 2 + i * (TOT - 2) / (IM - 1); ++q) {
          if (q < JN) n.b[q < JN ? q : 0] = read_b(st, q < JN ? q : 0, kk);
          else n.a[q < JN ? 0 : q - JN] = read_a(st, q < JN ? 0 : q - JN, kk);
        }
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[i][j] = mma(c.a[i], c.b[j], acc[i][j]);
        if (ROWSTRIP && i % IS == IS - 1) {
          if (wn == i / IS) {
#pragma unroll
            for (int e = 0; e < IS; ++e) accr[e] = mma(frs, c.a[i - IS + 1 + e], accr[e]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (PROT) {
        if (WGM == 1 || wm == 0) {
#pragma unroll
          for (int j = 0; j < JS; ++j) accs[j] = mma(fcs, c.b[j], accs[j]);
        } else {
#pragma unroll
          for (int j = JS; j < JN; ++j) accs[j - JS] = mma(fcs, c.b[j], accs[j - JS]);
        }
        fcs = lds_k(st + (kk ? cs1 : cs0));
      }
      if (ROWSTRIP) frs = lds_k(st + (kk ? rs1 : rs0));
    };

    for (int s = 0; s < NST && s < nk; ++s) issue(s);
    if (nk > 0) {
      Frags f0, f1;
      // stage 0 has landed; stage 1's copies of this wave are in flight
      if (nk == 1) wait_vm<0>();
      else if (sx) wait_vm<NPER + 1>();
      else wait_vm<NPER>();
      wg_barrier();
      {
        const char* st = smem;
#pragma unroll
        for (int j = 0; j < JN; ++j) f0.b[j] = read_b(st, j, 0);
#pragma unroll
        for (int i = 0; i < IM; ++i) f0.a[i] = read_a(st, i, 0);
        if (PROT) fcs = lds_k(st + cs0);
        if (ROWSTRIP) frs = lds_k(st + rs0);
      }
      int cur = 0;
      for (int kt = 0; kt < nk; ++kt) {
        phase(f0, f1, smem + cur * STAGE, 1);
        // every read of stage kt is complete; stage kt + 1 has landed
        wait_vm<0>();
        wg_barrier();
        if (kt + NST < nk) issue(kt + NST);
        cur = cur + 1 == NST ? 0 : cur + 1;
        phase(f1, f0, smem + cur * STAGE, 0);
      }
    }
    wg_barrier();  // the epilogue reuses the stages

    epilogue<ROWSTRIP>(smem, acc, accs, accr, m0, n0, k_lo, k_hi, kslice, split, tid, wm, wn, slot);
  }

  template <bool ROWSTRIP>
  __device__ static __forceinline__ void epilogue(char* smem, floatx4 (&acc)[IM][JN],
                                                  floatx4 (&accs)[JS], floatx4 (&accr)[IS], int m0,
                                                  int n0, int k_lo, int k_hi, int kslice,
                                                  bool split, int tid, int wm, int wn, int slot) {
    const GemmDesc& g = wide_desc(slot);
    const int lane = tid & 63, fr = lane & 15, g4 = lane >> 4;
    const int M = g.M, N = g.N;
    const int lg_rm = __builtin_ctz(g.Rm), lg_rn = __builtin_ctz(g.Rn);
    TC* C = static_cast<TC*>(g.C) + int64_t(kslice) * g.sCk;
    float2* ccv = reinterpret_cast<float2*>(smem + TILE);  // [row blocks of the tile][BN]
    // the strip results meet in LDS: rows 4 b .. 4 b + 3 (lane group b) are the
    // hi/lo pair of row block b's sum and of its weighted sum
    if (PROT) {
      const int jlo = wm * JS;
      if (g4 < BM >> lg_rm) {
#pragma unroll
        for (int j = 0; j < JS; ++j)
          if (jlo + j < JN)
            ccv[g4 * BN + wn * WN + (jlo + j) * 16 + fr] =
                float2{accs[j][0] + accs[j][1], accs[j][2] + accs[j][3]};
      }
      wg_barrier();
    }
    // this lane's checksum block: local block g4 of the wave's 128 rows
    const int nbw = WM >> lg_rm;
    const int blk = wm * nbw + g4;  // block of the tile
    const bool own = PROT && g4 < nbw && m0 + (blk << lg_rm) < M;
    if (own && g.Cc != nullptr) {
      float* Cc = g.Cc + int64_t(kslice) * g.sCck + int64_t(2 * ((m0 >> lg_rm) + blk)) * g.ldcc;
#pragma unroll
      for (int j = 0; j < JN; ++j) {
        const int n = n0 + wn * WN + j * 16 + fr;
        if (n < N) {
          const float2 c = ccv[blk * BN + wn * WN + j * 16 + fr];
          Cc[n] = c.x;
          Cc[g.ldcc + n] = c.y;
        }
      }
    }
    if (ROWSTRIP && g.Cr != nullptr) {
      const int nrb = BN >> lg_rn, qc0 = 2 * ((n0 - g.cr_n_begin) >> lg_rn);
      if (g4 < nrb && n0 + (g4 << lg_rn) < N) {
#pragma unroll
        for (int i = 0; i < IS; ++i) {
          const int m = m0 + wm * WM + (IS * wn + i) * 16 + fr;
          if (m < M)
            *reinterpret_cast<float2*>(g.Cr + int64_t(m) * g.ldcr + qc0 + 2 * g4) =
                float2{accr[i][0] + accr[i][1], accr[i][2] + accr[i][3]};
        }
      }
    }
    const int verify = PROT && !split ? g.verify : 0;
    // whether an injected fault (test-only) lands in this tile
    bool wf = false;
    if (!split)
      for (int f = 0; f < g.n_faults; ++f) {
        int fm, fn;
        wf |= wide_fault(g.map, N, g.faults[f], &fm, &fn) && fm >= m0 && fm < m0 + BM &&
              fn >= n0 && fn < n0 + BN;
      }

    uint32_t flags = 0;  // per j: this lane's vector (own block, column j * 16 + fr) is flagged
    if constexpr (sizeof(TC) == 2) {
      bf16_t* tile = reinterpret_cast<bf16_t*>(smem) + wm * (WM * LDT) + wn * WN;
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            tile[(16 * i + 4 * g4 + r) * LDT + 16 * j + fr] = f2bf(acc[i][j][r]);
      wave_fence();
      if (wf) {
        for (int f = 0; f < g.n_faults; ++f) {
          const abft_fault ft = g.faults[f];
          int fm, fn;
          if (!wide_fault(g.map, N, ft, &fm, &fn)) continue;
          fm -= m0 + wm * WM;
          fn -= n0 + wn * WN;
          if (fm < 0 || fm >= WM || fn < 0 || fn >= WN) continue;
          if (lane == 0) {
            bf16_t* p = tile + fm * LDT + fn;
            *p = ft.mode == ABFT_FAULT_FLIP ? flip_exponent_msb(*p) : f2bf(ft.value);
          }
          wave_fence();
        }
      }
      // detection: ones-operand MFMAs over the packed stored values (8
      // values of one column per lane for i = 2 s, 2 s + 1: together the 32
      // rows of segment s, whatever their order)
      if (verify >= 1) {
        const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          float r1 = 0.f, sa = 0.f;
#pragma unroll
          for (int s = 0; s < IM / 2; ++s) {
            uint32_t w[4];
            if (wf) {  // as stored, with the injected values
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const bf16_t* p = tile + (32 * s + 16 * (q >> 1) + 4 * g4 + 2 * (q & 1)) * LDT + 16 * j + fr;
                w[q] = uint32_t(p[0]) | (uint32_t(p[LDT]) << 16);
              }
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const floatx4& a = acc[2 * s + (q >> 1)][j];
                w[q] = uint32_t(f2bf(a[2 * (q & 1)])) | (uint32_t(f2bf(a[2 * (q & 1) + 1])) << 16);
              }
            }
            const u32x4 u = {w[0], w[1], w[2], w[3]};
            const u32x4 ua = u & 0x7fff7fffu;
            const floatx4 sm = mma(ones, __builtin_bit_cast(bf16x8, u), zero);
            const floatx4 mg = mma(ones, __builtin_bit_cast(bf16x8, ua), zero);
            if (((s * 32) >> lg_rm) == g4) {
              r1 += sm[0];
              sa += mg[0];
            }
          }
          const int n = n0 + wn * WN + 16 * j + fr;
          if (own && n < N && n >= g.verify_n_lo && n < g.verify_n_hi &&
              flagged(ccv[blk * BN + wn * WN + 16 * j + fr].x - r1, sa, g.e_rel))
            flags |= 1u << j;
        }
      }
      // 16-byte stores, WN / 8 lanes per row piece
      constexpr int CPW = WN / 8;
      static_assert((WM * CPW) % 64 == 0, "whole wave passes");
#pragma unroll
      for (int q = 0; q < WM * CPW / 64; ++q) {
        const int c = lane + q * 64, row = c / CPW, col = (c % CPW) * 8;
        const int m = m0 + wm * WM + row, n = n0 + wn * WN + col;
        if (m < M && n < N)  // (N % 8 == 0)
          *reinterpret_cast<uint4*>(C + int64_t(m) * g.ldc + n) =
              *reinterpret_cast<const uint4*>(tile + row * LDT + col);
      }
      if (PROT && __ballot(flags != 0))
        fix(g, flags, tile, C, ccv + wm * nbw * BN + wn * WN, m0 + wm * WM, n0 + wn * WN, k_lo, k_hi,
            lane);
    } else {
      if (wf) {
        for (int f = 0; f < g.n_faults; ++f) {
          const abft_fault ft = g.faults[f];
          int fm, fn;
          if (!wide_fault(g.map, N, ft, &fm, &fn)) continue;
          fm -= m0 + wm * WM;
          fn -= n0 + wn * WN;
#pragma unroll
          for (int i = 0; i < IM; ++i)
#pragma unroll
            for (int j = 0; j < JN; ++j)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (fm == 16 * i + 4 * g4 + r && fn == 16 * j + fr)
                  acc[i][j][r] = ft.mode == ABFT_FAULT_FLIP ? flip_exponent_msb(acc[i][j][r]) : ft.value;
        }
      }
      if (verify >= 1) {
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          float r1 = 0.f, sa = 0.f;
#pragma unroll
          for (int s = 0; s < IM / 2; ++s) {
            float t1 = 0.f, ta = 0.f;
#pragma unroll
            for (int i = 2 * s; i < 2 * s + 2; ++i)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                t1 += acc[i][j][r];
                ta += fabsf(acc[i][j][r]);
              }
            t1 = groups_sum(t1);
            ta = groups_sum(ta);
            if (((s * 32) >> lg_rm) == g4) {
              r1 += t1;
              sa += ta;
            }
          }
          const int n = n0 + wn * WN + 16 * j + fr;
          if (own && n < N && n >= g.verify_n_lo && n < g.verify_n_hi &&
              flagged(ccv[blk * BN + wn * WN + 16 * j + fr].x - r1, sa, g.e_rel))
            flags |= 1u << j;
        }
      }
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = m0 + wm * WM + 16 * i + 4 * g4 + r, n = n0 + wn * WN + 16 * j + fr;
            if (m < M && n < N) C[int64_t(m) * g.ldc + n] = acc[i][j][r];
          }
      if (PROT && __ballot(flags != 0)) {
        __threadfence();  // the wave reads its own stores back
        fix(g, flags, static_cast<bf16_t*>(nullptr), C, ccv + wm * nbw * BN + wn * WN, m0 + wm * WM,
            n0 + wn * WN, k_lo, k_hi, lane);
      }
    }
  }

  __device__ static __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // Flagged column vectors of a wave (Sec. 4.2), each by the whole wave:
  // located by EEC, recomputed from A and B (or fixed from the checksums),
  // checked again. The vectors lie in the wave's part of the rounded tile
  // (bf16) or of the stored output (fp32).
  __device__ static __noinline__ void fix(const GemmDesc& g, uint32_t flags, bf16_t* tile, TC* C,
                                          const float2* ccv, int mw, int nw, int k_lo, int k_hi,
                                          int lane) {
    const int R = g.Rm;
    for (int j = 0; j < JN; ++j) {
      uint64_t mask = __ballot((flags >> j) & 1u);
      while (mask) {
        const int L = __builtin_ctzll(mask);
        mask &= mask - 1;
        const int lb = L >> 4, col = 16 * j + (L & 15);
        const float2 c = ccv[lb * BN + col];
        const int row0 = lb * R;
        float x[2];
        bool in[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          in[h] = lane + 64 * h < R;
          const int row = row0 + (in[h] ? lane + 64 * h : 0);
          float v;
          if constexpr (sizeof(TC) == 2) v = bf2f(tile[row * LDT + col]);
          else
            v = __hip_atomic_load(C + int64_t(mw + row) * g.ldc + nw + col, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
          x[h] = in[h] ? v : 0.f;
        }
        const float r1 = group_sum<64>(x[0] + x[1]);
        const float r2 = group_sum<64>(fmaf(float(lane + 1), x[0], in[1] ? float(lane + 65) * x[1] : 0.f));
        const float sa = group_sum<64>((is_finite(x[0]) ? fabsf(x[0]) : 0.f) +
                                       (is_finite(x[1]) ? fabsf(x[1]) : 0.f));
        const float d1 = c.x - r1, d2 = c.y - r2;
        int idx = -1;
        if (flagged(d1, sa, g.e_rel)) {
          const bool any_inf = is_inf(d1), any_nonfin = is_nan(d1);
          uint64_t cand[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const bool fin = is_finite(x[h]);
            cand[h] = __ballot(in[h] && ((fin && fabsf(x[h]) >= g.tn) || (any_inf && is_inf(x[h])) ||
                                         (any_nonfin && !fin)));
          }
          const int cnt = __popcll(cand[0]) + __popcll(cand[1]);
          const int last = cand[1] ? 127 - __clzll(cand[1]) : (cand[0] ? 63 - __clzll(cand[0]) : -1);
          if (cnt == 1) {
            idx = last;
            if (is_finite(d1) && is_finite(d2) && !(fabsf(d2 / d1 - float(last + 1)) < 0.25f)) idx = -1;
          } else if (cnt == 0 && is_finite(d1) && is_finite(d2)) {
            const float q = d2 / d1, qi = rintf(q);
            if (q >= 0.5f && q < float(R) + 0.5f && fabsf(q - qi) < 0.25f) idx = int(qi) - 1;
          }
        }
        if (idx >= 0) {
          const int m = mw + row0 + idx, n = nw + col;
          const float old = __shfl(idx < 64 ? x[0] : x[1], idx & 63, 64);
          float val;
          int action = ABFT_ACT_RECOMPUTE;
          if (g.recompute) {
            const bf16_t* A = static_cast<const bf16_t*>(g.A);
            const bf16_t* B = static_cast<const bf16_t*>(g.B);
            float part = 0.f;
            for (int k = k_lo + lane; k < k_hi; k += 64)
              part = fmaf(bf2f(A[AK ? int64_t(m) * g.lda + k : int64_t(k) * g.lda + m]),
                          bf2f(B[BKM ? int64_t(n) * g.ldb + k : int64_t(k) * g.ldb + n]), part);
            val = group_sum<64>(part);
          } else if (is_finite(d1) && fabsf(d1) <= g.tc) {
            action = ABFT_ACT_DELTA;
            val = old + d1;
          } else {
            action = ABFT_ACT_RECONSTRUCT;
            val = c.x - group_sum<64>((lane == idx ? 0.f : x[0]) + (lane + 64 == idx ? 0.f : x[1]));
          }
          val = Storage<TC>::round(val);
          if (lane == idx) x[0] = val;
          if (lane + 64 == idx) x[1] = val;
          if (lane == 0) {
            if constexpr (sizeof(TC) == 2) tile[(row0 + idx) * LDT + col] = f2bf(val);
            C[int64_t(m) * g.ldc + n] = Storage<TC>::store(val);
            const WideCoord e = wide_coord(g.map, m, n);
            record_event(g.report, e.op, e.b, e.h, e.row, e.col, classify(old, g.tn), action, old);
          }
        }
        // anything still inconsistent is uncorrectable
        const float s1 = group_sum<64>(x[0] + x[1]);
        const float m1 = group_sum<64>(fabsf(x[0]) + fabsf(x[1]));
        if (lane == 0 && flagged(c.x - s1, m1, g.e_rel)) {
          const WideCoord e = wide_coord(g.map, mw + row0, nw + col);
          record_event(g.report, e.op, e.b, e.h, e.row, e.col, ABFT_KIND_NONE,
                       ABFT_ACT_UNCORRECTABLE, 0.f);
        }
      }
    }
  }
};

// Waves per SIMD: two workgroups share a CU where the LDS allows.
template <class W>
constexpr int wide_waves() {
  return W::LDS <= 80 * 1024 ? 2 * W::NW / 4 : W::NW / 4;
}

template <class W>
__global__ __launch_bounds__(W::NTH) __attribute__((amdgpu_waves_per_eu(wide_waves<W>())))
void wide_kernel(GemmDesc g) {
  extern __shared__ __align__(1024) char smem[];
  W::run(g, smem, blockIdx.x, gridDim.x, 0);
}

// Two independent GEMMs of the layer's backward in one launch: a weight
// gradient (WT, descriptor 0) and a projection (WP, descriptor 1), so that
// each fills the CUs the other leaves idle in its last round. Workgroups
// [0, n1) run the one with the longer K range (`first`), the rest the other;
// n1 is rounded up to a multiple of 8 so that both keep the dealing to the
// XCDs (the spare workgroups return).
template <class WT, class WP>
__global__ __launch_bounds__(WT::NTH) __attribute__((amdgpu_waves_per_eu(wide_waves<WT>())))
void wide_pair_kernel(GemmDesc gw, GemmDesc gp, int first, int t1, int n1, int t2) {
  extern __shared__ __align__(1024) char smem[];
  const bool head = int(blockIdx.x) < n1;
  const int lin = head ? int(blockIdx.x) : int(blockIdx.x) - n1, total = head ? t1 : t2;
  if (lin >= total) return;
  if (head == (first == 0)) WT::run(gw, smem, lin, total, 0);
  else WP::run(gp, smem, lin, total, 1);
}

template <class W>
int64_t wide_tiles(const GemmDesc& g) {
  return int64_t((g.M + W::BM - 1) / W::BM) * ((g.N + W::BN - 1) / W::BN) *
         (g.splitk > 1 ? g.splitk : 1);
}

template <class W>
hipError_t launch_w(const GemmDesc& g, hipStream_t s) {
  constexpr auto k = wide_kernel<W>;
  const hipError_t e = lds_limit<k>(W::LDS);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(unsigned(wide_tiles<W>(g))), dim3(W::NTH), W::LDS, s, g);
  return hipGetLastError();
}

// The tiles. Measured with checks (us a CU spends on one 64-deep step of a
// tile with all CUs busy, and per tile besides): 256 x 256 1.75 and 7, one
// workgroup per CU; 256 x 192 1.4 and 8; 128 x 128 0.58 and 2.3, two
// workgroups per CU (the 0.58 is per workgroup). Larger tiles ask L2 and LDS
// for less per flop (26.7, 28.5, 35.4 ps per output and step); smaller ones
// leave fewer CUs idle in the last round. Tiles with one wave per SIMD
// (128 x 256 or 128 x 192, four waves, three stages) measured half as fast.
enum { W256 = 0, W192 = 1, W128 = 2, NWIDE = 3 };
struct WideCost {
  int bm, bn;
  double step, fix;
};
constexpr WideCost COST[NWIDE] = {{256, 256, 1.75, 7.0}, {256, 192, 1.4, 8.0}, {128, 128, 0.58, 2.3}};
constexpr int CUS = 256;

template <class TC, bool AK, bool BKM, bool PROT> struct Shape256 {
  using T = Wide<TC, AK, BKM, 2, 4, 4, PROT>;
};
template <class TC, bool AK, bool BKM, bool PROT> struct Shape192 {
  using T = Wide<TC, AK, BKM, 2, 4, 3, PROT>;
};
template <class TC, bool AK, bool BKM, bool PROT> struct Shape128 {
  using T = Wide<TC, AK, BKM, 1, 4, 2, PROT>;
};

bool has_checks(const GemmDesc& g) { return g.Ac != nullptr || g.Br != nullptr || g.verify != 0; }

// Whether tile w takes g (already wide_operands_ok).
bool tile_ok(const GemmDesc& g, int w) {
  const int bm = COST[w].bm, bn = COST[w].bn;
  if (g.Ac != nullptr && 4 * bm / g.Rm > 16) return false;  // one 16-row strip
  // the row strip: whole column tiles of whole blocks, one 16-row strip
  if (g.Br != nullptr && (g.cr_n_begin % bn != 0 || bn % g.Rn != 0 || 4 * bn / g.Rn > 16)) return false;
  return true;
}
double tile_cost(const GemmDesc& g, int w) {
  const int ks = g.splitk > 1 ? g.splitk : 1;
  return COST[w].fix + COST[w].step * ((g.K / 64 + ks - 1) / ks);
}
int64_t tile_count(const GemmDesc& g, int w) {
  return int64_t((g.M + COST[w].bm - 1) / COST[w].bm) * ((g.N + COST[w].bn - 1) / COST[w].bn) *
         (g.splitk > 1 ? g.splitk : 1);
}
int pick(const GemmDesc& g) {
  int best = -1;
  double t = 0;
  for (int w = 0; w < NWIDE; ++w) {
    if (!tile_ok(g, w)) continue;
    const double c = double((tile_count(g, w) + CUS - 1) / CUS) * tile_cost(g, w);
    if (best < 0 || c < t) { best = w; t = c; }
  }
  return best;
}

bool wide_operands_ok(const GemmDesc& g, bool c_fp32, bool ak, bool bk) {
  if (c_fp32 ? (ak || bk) : !ak) return false;
  if (g.nb0 * g.nb1 != 1 || g.causal != 0 || g.verify > 1 || g.K % 64 != 0) return false;
  if (g.M < 1 || g.N < 1 || g.K < 64) return false;
  auto al = [](const void* p, int64_t ld) {
    return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 8 == 0;
  };
  if (!al(g.A, g.lda) || !al(g.B, g.ldb) || !al(g.C, g.ldc) || g.N % 8 != 0) return false;
  if (!wide_rows_ok(ak, g.M) || !wide_rows_ok(bk, g.N)) return false;
  const int64_t lim = int64_t(1) << 31;  // 32-bit buffer offsets
  if (((ak ? g.M : g.K) + 256) * g.lda * 2 >= lim || ((bk ? g.N : g.K) + 256) * g.ldb * 2 >= lim)
    return false;
  if (has_checks(g)) {  // the strips come from the checksums' bf16 images
    if (g.Ac == nullptr || g.Aci == nullptr || !al(g.Aci, g.ldaci) || g.Rm > 128) return false;
    if (g.Br != nullptr && (g.Bri == nullptr || !al(g.Bri, g.ldbri) || !ak || bk || c_fp32))
      return false;
  }
  if (g.splitk > 1 && !c_fp32) return false;
  // the kernel shifts by the block sizes and writes no images of its output's
  // checksums
  auto pow2 = [](int x) { return x > 0 && (x & (x - 1)) == 0; };
  return pow2(g.Rm) && pow2(g.Rn) && g.Cci == nullptr && g.Cri == nullptr;
}

template <template <class, bool, bool, bool> class S>
hipError_t launch_tile_w(const GemmDesc& g, bool c_fp32, bool bk, hipStream_t s) {
  const bool prot = has_checks(g);
  if (c_fp32)
    return prot ? launch_w<typename S<float, false, false, true>::T>(g, s)
                : launch_w<typename S<float, false, false, false>::T>(g, s);
  if (bk)
    return prot ? launch_w<typename S<bf16_t, true, true, true>::T>(g, s)
                : launch_w<typename S<bf16_t, true, true, false>::T>(g, s);
  return prot ? launch_w<typename S<bf16_t, true, false, true>::T>(g, s)
              : launch_w<typename S<bf16_t, true, false, false>::T>(g, s);
}

template <template <class, bool, bool, bool> class S, bool PROT>
hipError_t launch_pair_w(const GemmDesc& w, const GemmDesc& p, int first, hipStream_t s) {
  using WT = typename S<float, false, false, PROT>::T;
  using WP = typename S<bf16_t, true, true, PROT>::T;
  static_assert(WT::NTH == WP::NTH, "one workgroup size");
  constexpr auto k = wide_pair_kernel<WT, WP>;
  constexpr size_t lds = std::max(WT::LDS, WP::LDS);
  const hipError_t e = lds_limit<k>(lds);
  if (e != hipSuccess) return e;
  const int64_t tw = wide_tiles<WT>(w), tp = wide_tiles<WP>(p);
  const int64_t t1 = first == 0 ? tw : tp, t2 = first == 0 ? tp : tw, n1 = (t1 + 7) / 8 * 8;
  hipLaunchKernelGGL(k, dim3(unsigned(n1 + t2)), dim3(WT::NTH), lds, s, w, p, first, int(t1),
                     int(n1), int(t2));
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_wide(const GemmDesc& g, bool c_fp32, Layout la, Layout lb,
                            hipStream_t stream) {
  const bool bk = lb == Layout::KMajor;
  if (!wide_operands_ok(g, c_fp32, la == Layout::KMajor, bk)) return hipErrorNotSupported;
  switch (pick(g)) {
    case W256: return launch_tile_w<Shape256>(g, c_fp32, bk, stream);
    case W192: return launch_tile_w<Shape192>(g, c_fp32, bk, stream);
    case W128: return launch_tile_w<Shape128>(g, c_fp32, bk, stream);
  }
  return hipErrorNotSupported;
}

hipError_t launch_gemm_pair(const GemmDesc& w, const GemmDesc& p, int dtype, hipStream_t stream) {
  if (dtype != ABFT_BF16 || has_checks(w) != has_checks(p)) return hipErrorNotSupported;
  if (!wide_operands_ok(w, true, false, false) || !wide_operands_ok(p, false, true, true) ||
      p.Br != nullptr)
    return hipErrorNotSupported;
  const bool prot = has_checks(w);
  // the tile for the two together: their work over the CUs, and half of the
  // longer workgroup for the uneven end (256 x 192 measured slower for every
  // pair: dX with dWqkv at B4 S2048 H4096 1446 -> 1691 us, at B8 S1024 H768 94
  // -> 116)
  int best = -1;
  double t = 0;
  for (int c : {int(W256), int(W128)}) {
    if (!tile_ok(w, c) || !tile_ok(p, c)) continue;
    const double a = tile_cost(w, c), b = tile_cost(p, c);
    const double sum = (tile_count(w, c) * a + tile_count(p, c) * b) / CUS + std::max(a, b) / 2;
    if (best < 0 || sum < t) { best = c; t = sum; }
  }
  if (best < 0) return hipErrorNotSupported;
  const int first = tile_cost(w, best) >= tile_cost(p, best) ? 0 : 1;
  if (best == W256)
    return prot ? launch_pair_w<Shape256, true>(w, p, first, stream)
                : launch_pair_w<Shape256, false>(w, p, first, stream);
  return prot ? launch_pair_w<Shape128, true>(w, p, first, stream)
              : launch_pair_w<Shape128, false>(w, p, first, stream);
}

}  // namespace abft
