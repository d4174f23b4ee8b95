// verify_tile.hip -- tree-masked factorised verification (SpecLA §4.2) with
// the delayed state update of §5.2 fused in front of it.
//
// Unrolling the gated delta rule along a root path gives, for every node j
// (gamma_j = product of alpha over P(j); for a in P(j), D_ja = product of
// alpha over the nodes of P(j) strictly below a, which equals gamma_j /
// gamma_a but is formed as a product, so no reciprocal of a decay product
// is ever taken and strong decays underflow harmlessly to zero):
//     H_j = gamma_j H0 + sum_{a in P(j)} D_ja k_a u_a^T
//     (I + Lk) U = R,   R_j = beta_j (v_j - gamma_j H0^T k_j),
//                       Lk_ja = beta_j D_ja (k_j . k_a)   for a in P(j), a != j
//     O = Gamma Q H0 + Attn U,   Attn_ja = D_ja (q_j . k_a)   for a in P(j)
// which is the tree-masked UT form: T = (I + Lk)^-1 is the paper's
// T_tree = solve_tril(I - A_tree), and O = Q^ S0^T - Attn W S0^T + Attn U.
// Both per-column products run on the matrix cores:
//     U = T R,      O = Gamma P_q + Attn U,
// the first as a substitution over 16-row blocks (only the diagonal blocks
// of T are formed), and the only sequential work is the small per-unit
// inverse of those blocks.  Only the committed state is read.
//
// One workgroup = one (batch b, head h) unit's V-tile of CW x 16 columns
// (CW = 3, 4 or 8), or TPW = 2 consecutive such tiles, with CW + 1 wavefronts
// (CW = 3 or 4) or CW (CW = 8, where column wave 0 also takes the setup work):
//   waves 0 .. CW-1 own 16 state columns each.  They bring [Q; K] (a share
//              each, through registers into LDS), then, held back briefly, the
//              state tile (in the B-fragment order of
//              v_mfma_f32_16x16x32_bf16: 8 consecutive rows of one column per
//              32-row K-step) and the values.  The state reads and the
//              committed-row writes keep the default cache policy: a wave
//              covers only half of each 128-byte line, and with a streaming
//              hint the L2 lets the line go before the neighbouring wave
//              reads or writes the other half (measured: about 15% more HBM
//              reads, 8% more writes).  Per tile: pending path applied,
//              committed rows written back, fp32 split into bf16 hi + lo,
//              P = [Q; K] H0 accumulated on the matrix cores K-step by
//              K-step.  Then R = beta (v - gamma P_k), U = T R and
//              O = Gamma P_q + Attn U on v_mfma_f32_16x16x16bf16_1k (whose B
//              fragment is exactly the accumulator layout holding R, then U),
//              and the outputs.  With two tiles, the second tile's reads go
//              out once the first tile's registers are free.
//   wave CW    (the setup wave; wave 0 at CW = 8) owns no state of its own.
//              It takes every read that depends on another read: parent row
//              and gates -> topology and decays; the pending path with the
//              previous round's parent row and gates -> validation and, at
//              once, the factor records the path names (registers, then LDS
//              while the Grams run; a second stage for a second tile); and,
//              for two 16-node tiles with scalar gates, the second tile's
//              first d_k/2 state rows straight into LDS, which would otherwise
//              queue behind the first tile's work (measured at batch 64, 16
//              heads, d_v 128: 37.8 -> 36.9 us per launch).  After the Grams
//              it inverts the diagonal blocks of T.
// The tree-masked Grams ([Q; K] K^T tiles that hold ancestor pairs, exact
// bf16 products) run on the column waves; they and T are done while the
// first tile's state is still in flight.  Strided global accesses go through
// buffer descriptors (one VGPR offset per lane).  With fp32 activations the
// same structure runs every contraction on the fp32 matrix cores (Layout).
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace sla {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kWaveCols = 16;                    // state columns per column wave
constexpr int kPMax = 8;                          // pending steps staged in LDS
constexpr int kBP = 20;                           // fp32 row pitch of a 16x16 block

// Layer families by the form of their step (template parameter KIND):
//   kKindDelta  scalar gates: GDN, DeltaNet (alpha = 1) and the scalar decay
//               without the delta rule (beta = 0, so Lk = 0 and T = I, with
//               R = V in place of beta (v - gamma P_k): a run-time choice,
//               so that all three share one register allocation);
//   kKindGates  GLA: one gate per key dimension, no delta rule.  The decay
//               ratios become per-dimension, D_ja[i] (the product of the
//               i-th gates of P(j) strictly below a), so the scores
//               Attn_ja = sum_i q_j[i] D_ja[i] k_a[i] are formed on the
//               vector ALUs by walking each root path, and
//               O = Q~ H0 + Attn V with Q~_j = Gamma_j * q_j (fp32, split
//               into bf16 hi + lo).
constexpr int kKindDelta = 0, kKindGates = 1;

// Launches by their rounds of workgroups (resident workgroups per CU from the
// occupancy of the kernel instantiation):
//   kModePart   less than one round, or rows that are not whole 128-byte
//               lines: the state reads go out before the first barrier, so
//               that they overlap the setup wave's dependent reads, and
//               committed rows are written back;
//   kModeRound  one to kLateRounds rounds: committed rows are written through
//               (64 16-node trees, 16 heads, over 24 rotating layers: 36.7 us,
//               38.7 us written back; with d_v 144, whose rows split lines,
//               writing back is better: 23 nodes, 12 heads, batch 40, per-key
//               gates 37.7 us, 39.7 us through);
//   kModeLate   kLateRounds rounds or more: the state reads go out after the
//               first barrier (64-node trees at batch 256, eight rounds: 419 us,
//               432 us with the reads first).
// Template parameters: a run-time choice of the store policy or of the place
// of the state reads costs most of what it gains.
constexpr int kModePart = 0, kModeRound = 1, kModeLate = 2;
// fp32 activations with per-key gates take the late place in every mode for 32
// node rows and at d_k 256: the staged rows and gates then leave their registers
// before the state needs any (138 -> 228 VGPRs with the reads first at d_k 256,
// 32 nodes), and the scores hide the reads (reads first and late: 24 sequences,
// 8 heads, d_v 128, d_k 256, 16 nodes 29.3 and 25.4 us; d_k 128, 32 nodes 24.9
// and 20.0; batch 1, 12 heads, d_v 144, 23 nodes 10.7 and 10.6).  Not where it
// gains nothing on the whole: 64 node rows, 16 at d_k 64 and 128; nor with
// eight column waves, which read the state behind the scores there (d_k = d_v =
// 256, 32 nodes 43.1 and 45.7).
template <int DK, int NP, int CW, int KIND, bool F32>
constexpr bool kLateAlways = KIND == kKindGates && F32 && CW < 8 && NP <= 32 && (NP == 32 || DK == 256);

// F32: fp32 activations.  q, k, v and the pending keys are staged and read
// as fp32, and every contraction runs on v_mfma_f32_16x16x4_f32 with exact
// fp32 products (no hi/lo splits); else bf16 activations (16x16x32 bf16 for
// the Grams and P, hi/lo-split 16x16x16 bf16 for T R and Attn U).
template <int DK, int NP, int CW, int TPW, int KIND, bool F32>
struct Layout {
  static constexpr int kTileCols = CW * kWaveCols;
  static constexpr int ES = F32 ? 4 : 2;            // bytes per activation
  static constexpr int NT = NP / 16, KS = DK / 32, CH = DK * ES / 16, MT = 2 * NT;
  static constexpr int NB = NT * (NT + 1) / 2;      // lower-triangular 16x16 blocks
  static constexpr bool kDelta = KIND == kKindDelta, kGates = KIND == kKindGates;
  static constexpr int kX = 2 * NP * CH * 16;       // [Q; K], 16-byte chunks, xor-swizzled
  static constexpr int kBlk = 16 * kBP * 4;
  static constexpr int kT = kDelta ? NB * kBlk : 0;   // -Lk blocks, the diagonal ones inverted in place
  static constexpr int kAt = NB * kBlk;             // Attn blocks
  static constexpr int kPk = kPMax * DK * ES;       // pending keys (activation dtype)
  static constexpr int kPuPitch = kTileCols < kWave ? kWave : kTileCols;  // a direct load fills whole waves
  static constexpr int kPu = TPW * kPMax * kPuPitch * 4;  // pending corrected values, one stage per tile
  static constexpr int kXL = (kGates && !F32) ? kX / 2 : 0;  // low halves of Q~, same chunk layout
  static constexpr int kG = kGates ? NP * DK * 4 : 0;      // the draft's per-key gates
  static constexpr int kPg = kGates ? kPMax * DK * 4 : 0;  // pending per-key gates
  // small trees, two 64-column tiles: the second tile's first DK/2 state rows
  // are staged in LDS ahead of time (16-byte chunks, swizzled: see kernel).
  // Not for GLA: its gate stages already take 37 KB at d_k 128, and 16 KB
  // more would leave three resident workgroups per CU instead of four
  // (measured 40.1 -> 43.4 us per launch at batch 64, 16 heads).
  static constexpr bool kPrefetch = TPW == 2 && NP == 16 && CW == 4 && kDelta;
  static constexpr int kPreInstr = kPrefetch ? (DK / 2) * (kTileCols / 4) / kWave : 0;  // 16-byte loads per lane
  static constexpr int kPre = kPreInstr * kWave * 16;
  static constexpr int kTopo = NP * 8 + NP * 2 * 4 + kPMax * 4 + 16;
  static constexpr int oT = kX, oAt = oT + kT, oPk = oAt + kAt, oPu = oPk + kPk;
  static constexpr int oXL = oPu + kPu, oG = oXL + kXL, oPg = oG + kG, oPre = oPg + kPg, oTopo = oPre + kPre;
  static constexpr int kBytes = oTopo + kTopo;
};

// [Q; K] chunk (row, c) lives at row * CH + (c ^ (row & 7)): the 16 rows a
// fragment read touches fall on distinct bank groups.
template <int CH>
__device__ __forceinline__ int xchunk(int row, int c) {
  return row * CH + (c ^ (row & 7));
}

// s_waitcnt immediate that waits until at most `n` vector memory operations
// of this wave are outstanding (export and LDS counters unconstrained).
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// element (row j, column a), a <= j, of a lower-triangular 16x16-blocked matrix
[[maybe_unused]] __device__ __forceinline__ int blk(int j, int a) {
  const int bj = j >> 4;
  return ((bj * (bj + 1)) / 2 + (a >> 4)) * (16 * kBP) + (j & 15) * kBP + (a & 15);
}

[[maybe_unused]] __device__ __forceinline__ void split8(const float (&x)[8], bf16x8 &hi, bf16x8 &lo) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 h = static_cast<__bf16>(x[e]);
    hi[e] = h;
    lo[e] = static_cast<__bf16>(x[e] - static_cast<float>(h));
  }
}

[[maybe_unused]] __device__ __forceinline__ void split4(f32x4 x, s16x4 &hi, s16x4 &lo) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const __bf16 h = static_cast<__bf16>(x[e]);
    hi[e] = __builtin_bit_cast(short, h);
    lo[e] = __builtin_bit_cast(short, static_cast<__bf16>(x[e] - static_cast<float>(h)));
  }
}

[[maybe_unused]] __device__ __forceinline__ f32x4 mfma16(s16x4 a, s16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// acc += A B with A and B fp32 given as hi + lo (the lo * lo term is below
// fp32 resolution and dropped).
[[maybe_unused]] __device__ __forceinline__ f32x4 mfma16_split(s16x4 ah, s16x4 al, s16x4 bh, s16x4 bl, f32x4 acc) {
  acc = mfma16(ah, bh, acc);
  acc = mfma16(ah, bl, acc);
  return mfma16(al, bh, acc);
}

// Waves per SIMD the register allocation is held to: 6 (80 VGPRs) where the
// tile state, accumulators and LDS allow a fourth resident workgroup per CU;
// 4 (128 VGPRs) for the eight-wave form where its LDS lets two workgroups fit
// a CU; 5 (96) for 64 node rows in fp32 at d_k 64 (116 otherwise: 16 heads, batch
// 64, d_v 128, 48 nodes 67 us, 58 held); else whatever the allocation needs.
constexpr size_t kMaxLds = 160 * 1024;
constexpr size_t kDefaultLds = 64 * 1024;
template <int DK, int NP, int CW, int TPW, int KIND, bool F32>
constexpr int kMinWaves =
    F32 ? (KIND == kKindDelta && DK == 64 && NP == 64 && CW == 4 ? 5 : 1)
        : ((DK <= 128 && NP <= 16) ? 6 : (CW == 8 && 2 * Layout<DK, NP, CW, TPW, KIND, F32>::kBytes <= kMaxLds ? 4 : 1));

// KIND: the family's form (see Layout).  Without the delta rule Lk = 0, so
// T = I and U = R = V: no P_k, no Lk, no T.
// Eight column waves: column wave 0 also does the setup work, so that the
// workgroup is eight waves and two fit a CU at 124 VGPRs (a ninth wave keeps
// it to one: measured on 64-node trees at batch 256, d_v 256, 459 -> 448 us per
// launch; its state reads then go out after its record reads).
template <int CW>
constexpr int kWaves = CW == 8 ? CW : CW + 1;

// MODE: how a launch's rounds of workgroups order the state reads (kMode*).
template <int DK, int NP, int CW, int TPW, int KIND, bool F32, int MODE>
__global__ __launch_bounds__(kWaves<CW> * kWave) __attribute__((amdgpu_waves_per_eu(kMinWaves<DK, NP, CW, TPW, KIND, F32>)))
void verify_tile_kernel(VerifyArgs a) {
  using L = Layout<DK, NP, CW, TPW, KIND, F32>;
  using AT = std::conditional_t<F32, float, bf16>;  // activation element
  using VT = std::conditional_t<F32, uint32_t, uint16_t>;  // its bit pattern
  constexpr int ES = L::ES;
  constexpr int EC = 16 / ES;  // activations per 16-byte chunk
  constexpr bool DELTA = KIND == kKindDelta;
  constexpr bool GV = KIND == kKindGates;
  const bool nodelta = !DELTA || a.family == SLA_FAMILY_DECAY;  // R = V
  constexpr bool kLate = MODE == kModeLate || kLateAlways<DK, NP, CW, KIND, F32>;
  constexpr bool WT = MODE == kModeRound;       // committed rows written through at device scope
  constexpr int kColWaves = CW;                 // waves 0 .. CW-1 own state columns
  constexpr int kSetup = kWaves<CW> == CW ? 0 : CW;  // the setup wave
  constexpr int kTileCols = L::kTileCols;       // state columns per workgroup
  constexpr int KS = L::KS, NT = L::NT, MT = L::MT, CH = L::CH;
  constexpr bool kUnitT = F32 && NT == 1;                   // T with its diagonal (see U = T R)
  constexpr int NGT = NT * (NT + 1);                        // Gram tiles (both halves)
  constexpr int GT = (NGT + kColWaves - 1) / kColWaves;     // Gram tiles per column wave

  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  uint4 *xs = reinterpret_cast<uint4 *>(lds);                 // [Q; K] (GLA: high halves of Q~ in place of Q)
  float *tb = reinterpret_cast<float *>(lds + L::oT);         // -Lk blocks; diagonal ones become N = T - I
  float *ab = reinterpret_cast<float *>(lds + L::oAt);        // Attn blocks
  AT *s_pk = reinterpret_cast<AT *>(lds + L::oPk);            // [kPMax][DK]
  float *s_pu = reinterpret_cast<float *>(lds + L::oPu);      // [TPW][kPMax][kPuPitch]
  uint4 *xl = reinterpret_cast<uint4 *>(lds + L::oXL);        // GLA: low halves of Q~
  float *s_g = reinterpret_cast<float *>(lds + L::oG);        // GLA: [NP][DK] gates
  float *s_pg = reinterpret_cast<float *>(lds + L::oPg);      // GLA: [kPMax][DK] pending gates
  float *s_pre = reinterpret_cast<float *>(lds + L::oPre);    // second tile's first DK/2 state rows
  unsigned char *tp = lds + L::oTopo;
  uint64_t *s_anc = reinterpret_cast<uint64_t *>(tp);      // [NP]
  float *s_gamma = reinterpret_cast<float *>(tp + 8 * NP);  // [NP]
  float *s_be = s_gamma + NP;                               // [NP]
  float *s_palpha = s_be + NP;                              // [kPMax]
  int *s_misc = reinterpret_cast<int *>(s_palpha + kPMax);  // err, path len

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int l = tid % kWave;
  const int lc = l & 15;  // column within a wave's 16 / row within a 16-row tile
  const int lg = l >> 4;  // row group
  const int H = a.H, dv = a.dv, n = a.n;
  // this workgroup: unit (b, h), V-tiles t0 .. t0 + cnt - 1
  const int ntiles = (dv + kTileCols - 1) / kTileCols;
  const int ngroups = (ntiles + TPW - 1) / TPW;
  int wid = blockIdx.x;
  const int t0 = (wid % ngroups) * TPW;
  wid /= ngroups;
  const int cnt = TPW;  // TPW divides the tile count (the launcher checks)
  const int h = wid % H;
  const int b = wid / H;
  const int ucol = w * kWaveCols + lc;  // column within a tile
  const size_t unit = (size_t)b * H + h;
  const size_t nbase = (size_t)b * n;
  const rsrc_t sr = make_rsrc(a.state + unit * DK * dv, (uint32_t)DK * dv * 4);
  const uint32_t nstride = (uint32_t)H * dv;  // elements between consecutive nodes of a unit
  const rsrc_t vr = make_rsrc(static_cast<const AT *>(a.v) + (nbase * H + h) * dv,
                              ((uint32_t)(n - 1) * nstride + dv) * ES);
  // wave-uniform: this wave owns columns of tile t
  auto live = [&](int t) { return w < kColWaves && t * kTileCols + w * kWaveCols < dv; };
  // a wave past the last column reads outside the descriptors (zeros, no
  // traffic) instead of branching round its reads: the compiler then counts
  // the reads in flight exactly
  auto outside = [&](int t) { return live(t) ? 0u : 0x80000000u; };
  // state rows 8 lg + e + 32 ks of column t * kTileCols + ucol, in B-fragment order
  auto load_state = [&](int t, float (&hf)[KS][8], int ks0 = 0) {
    const uint32_t sv = (uint32_t)(8 * lg * dv + t * kTileCols + ucol) * 4 | outside(t);
#pragma unroll
    for (int ks = ks0; ks < KS; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) hf[ks][e] = buf_load_f32<kPolicyDefault>(sr, sv, (uint32_t)(ks * 32 + e) * dv * 4);
  };
  // values of node j = 16 mt + 4 lg + q; rows past the last node fall
  // outside the descriptor and read zero
  auto load_values = [&](int t, VT (&vraw)[NT][4]) {
    const uint32_t vv = (4 * lg * nstride + t * kTileCols + ucol) * ES;
    const uint32_t ov = outside(t);
#pragma unroll
    for (int mt = 0; mt < NT; ++mt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t o = (vv + (uint32_t)(mt * 16 + q) * nstride * ES) | ov;
        if constexpr (F32)
          vraw[mt][q] = __builtin_amdgcn_raw_buffer_load_b32(vr, o, 0, kPolicyDefault);
        else
          vraw[mt][q] = __builtin_amdgcn_raw_buffer_load_b16(vr, o, 0, kPolicyDefault);
      }
  };

  // fp32 activations: the eight values k = 32 ks + 8 lg + e (e = 0..7) of
  // stage row `row`, the A operand of v_mfma_f32_16x16x4_f32 number e of
  // K-step ks, whose K index lg then pairs with state row 32 ks + 8 lg + e
  // (exactly what a column wave's state registers hold as B operands)
  auto frag8 = [&](int row, int ks, float (&x)[8]) {
    const float4 u0 = *reinterpret_cast<const float4 *>(xs + xchunk<CH>(row, 8 * ks + 2 * lg));
    const float4 u1 = *reinterpret_cast<const float4 *>(xs + xchunk<CH>(row, 8 * ks + 2 * lg + 1));
    x[0] = u0.x, x[1] = u0.y, x[2] = u0.z, x[3] = u0.w, x[4] = u1.x, x[5] = u1.y, x[6] = u1.z, x[7] = u1.w;
  };

  // ---- setup wave: the small reads, ahead of everything else: parent row,
  //      gates, and the pending accepted path with the previous round's parent
  //      row and gates read whole, so that validating the path waits on no
  //      further read
  int p = -1;       // lane j: parent of node j
  float al = 1.f;   // lane j: alpha_j
  float be = 0.f;   // lane j: beta_j
  int plen = 0;     // accepted length
  int nodec = -1;   // lane t: node of pending step t (later clamped into the store)
  int prow_parent = -2;
  float pal = 0.f;  // lane t: gate of pending record t (later of step t's record)
  const int pn = a.has_pending ? a.pend.n : 1;
  const size_t prow = (size_t)b * pn;
  const int ln = l < n ? l : n - 1, lp = l < pn ? l : pn - 1;  // lanes past the last node re-read it
  if (w == kSetup) {
    p = a.parent[nbase + ln];
    // DeltaNet: no decay; GLA: the per-key gates enter through Q~ and Attn
    if (!GV && a.family != SLA_FAMILY_DELTANET) al = a.alpha[(nbase + ln) * H + h];
    if (DELTA && a.family != SLA_FAMILY_DECAY) be = a.beta[(nbase + ln) * H + h];
    if (a.has_pending) {
      plen = a.pend.len[b];
      nodec = a.pend.path[prow + lp];
      prow_parent = a.pend.parent[prow + lp];
      if (!GV) pal = a.pend.alpha[(prow + lp) * H + h];
    }
  }

  // ---- column waves: [Q; K] (and GLA's gates) on their way to LDS through
  //      registers, a share per wave (rows 0..NP-1: q_j, NP..2NP-1: k_j; rows
  //      past the last node fall outside the descriptors and read zero), then
  //      the first tile's state and values.  The stores to LDS wait for their
  //      own reads only, not for the state behind them.  (The setup wave used
  //      to bring [Q; K] by itself, straight into LDS, and every LDS operation
  //      behind it waited.)
  constexpr int kLanes = kColWaves * kWave;
  constexpr int kQK = 2 * NP * CH;                   // 16-byte chunks of [Q; K]
  constexpr int NQ = (kQK + kLanes - 1) / kLanes;    // and per lane
  constexpr int GC = DK / 4;                         // 16-byte chunks per gate row
  constexpr int NG = GV ? (NP * GC + kLanes - 1) / kLanes : 0;
  float hfa[KS][8], hfb[KS][8];  // hfb: the next tile's state (prefetching form only)
  VT vraw[NT][4];  // activation bit patterns, widened where they are used
  auto column_reads = [&]() {
    const uint32_t rowb = (uint32_t)H * DK;  // elements between consecutive nodes of a unit
    const uint32_t qkb = ((uint32_t)(n - 1) * rowb + DK) * ES;
    const rsrc_t qr = make_rsrc(static_cast<const AT *>(a.q) + (nbase * H + h) * DK, qkb);
    const rsrc_t kr = make_rsrc(static_cast<const AT *>(a.k) + (nbase * H + h) * DK, qkb);
    u32x4 qk[NQ], gq[NG > 0 ? NG : 1];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      if (i * kLanes + w * kWave >= kQK) continue;  // wave-uniform (three column waves)
      const int P = i * kLanes + w * kWave + l;
      const int row = P / CH, c = (P % CH) ^ (row & 7);
      const bool isq = i * kLanes + w * kWave < NP * CH;  // wave-uniform: a wave's rows lie in one half
      qk[i] = __builtin_amdgcn_raw_buffer_load_b128(isq ? qr : kr, ((uint32_t)(row % NP) * rowb + c * EC) * ES, 0,
                                                    kPolicyDefault);
    }
    if constexpr (GV) {
      const rsrc_t gr = make_rsrc(a.alpha + (nbase * H + h) * DK, ((uint32_t)(n - 1) * rowb + DK) * 4);
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        if (i * kLanes + w * kWave >= NP * GC) continue;
        const int P = i * kLanes + w * kWave + l;
        gq[i] = __builtin_amdgcn_raw_buffer_load_b128(gr, ((uint32_t)(P / GC) * rowb + (P % GC) * 4) * 4, 0, kPolicyDefault);
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // none of these moves behind the state reads
    // hold the state reads back about 0.8 us (30 x 64 cycles), so that the
    // setup reads and [Q; K] enter the memory queue ahead of the state
    // (measured per launch with no hold and with 20, 30, 45: batch 1, 8 nodes
    // 7.19, 7.28, 6.90, 7.04 us; batch 16, 16 nodes 12.05, 11.42, 11.58,
    // 11.22 us); a full round of workgroups a little longer (64 16-node trees
    // over 24 rotating layers with 30, 50, 80, 127: 36.9, 36.7, 36.9, 38.0 us)
    if (!kLate && w != kSetup) __builtin_amdgcn_s_sleep(MODE == kModeRound ? 50 : 30);
    if constexpr (!kLate && kSetup != 0) load_state(t0, hfa);
    load_values(t0, vraw);
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (i * kLanes + w * kWave < kQK) reinterpret_cast<u32x4 *>(xs)[i * kLanes + w * kWave + l] = qk[i];
    if constexpr (GV) {
#pragma unroll
      for (int i = 0; i < NG; ++i)
        if (i * kLanes + w * kWave < NP * GC) reinterpret_cast<u32x4 *>(s_g)[i * kLanes + w * kWave + l] = gq[i];
    }
  };

  // ---- setup wave: the records of kPMax steps of the accepted path, from
  //      step c0 on, for the columns of TPW tiles or of one: read into
  //      registers (node indices are clamped into the store), then put into
  //      the LDS stage
  constexpr int KI = kPMax * CH / kWave;            // 16-byte key chunks per lane
  constexpr int GI = GV ? kPMax * GC / kWave : 0;   // 16-byte gate chunks per lane
  constexpr int UC = L::kPuPitch / kWave;           // corrected values per lane, step and tile
  struct Records {
    u32x4 k[KI];
    float u[TPW][kPMax * UC];
  };
  // (32-bit offsets from the unit's first record: one sequence's rows of one
  // tensor stay below 2^31 bytes)
  const AT *const pk0 = static_cast<const AT *>(a.pend.k) + (prow * H + h) * DK;
  const float *const pg0 = a.pend.alpha + (prow * H + h) * DK;
  const float *const pu0 = a.pend.u + (prow * H + h) * dv;
  const uint32_t krow = (uint32_t)H * DK;
  auto key_at = [&](int c0, int i) {  // this lane's i-th 16-byte key chunk of the stage
    return __umul24(__shfl(nodec, c0 + (i * kWave + l) / CH), krow) + ((i * kWave + l) % CH) * EC;
  };
  auto gate_at = [&](int c0, int i) {
    return __umul24(__shfl(nodec, c0 + (i * kWave + l) / GC), krow) + ((i * kWave + l) % GC) * 4;
  };
  auto u_row = [&](int c0, int st) { return (uint32_t)__builtin_amdgcn_readlane(nodec, c0 + st) * nstride; };
  auto u_col = [&](int i, int u) {  // tile t0 + i, column block u; columns past d_v re-read the last
    const int cg = (t0 + i) * kTileCols + u * kWave + l;
    return (uint32_t)(cg < dv ? cg : dv - 1);
  };
  auto gather_gates = [&](int c0) {
    uint32_t gp[GI > 0 ? GI : 1];
#pragma unroll
    for (int x = 0; x < GI; ++x) gp[x] = gate_at(c0, x);
    __builtin_amdgcn_sched_barrier(0);  // an LDS operation after a direct load waits for it
#pragma unroll
    for (int x = 0; x < GI; ++x) load_lds16(pg0 + gp[x], s_pg + x * kWave * 4);
  };
  // the first steps' records, every tile's values: through registers (GLA's
  // gate rows straight into LDS)
  auto read_records = [&](Records &r) {
    const rsrc_t kr = make_rsrc(pk0, ((uint32_t)(pn - 1) * krow + DK) * ES);
    const rsrc_t ur = make_rsrc(pu0, ((uint32_t)(pn - 1) * nstride + dv) * 4);
#pragma unroll
    for (int i = 0; i < KI; ++i) r.k[i] = __builtin_amdgcn_raw_buffer_load_b128(kr, key_at(0, i) * ES, 0, kPolicyDefault);
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
      for (int st = 0; st < kPMax; ++st)
#pragma unroll
        for (int u = 0; u < UC; ++u) r.u[i][st * UC + u] = buf_load_f32<kPolicyDefault>(ur, u_col(i, u) * 4, u_row(0, st) * 4);
  };
  auto stage_records = [&](const Records &r) {
#pragma unroll
    for (int i = 0; i < KI; ++i) reinterpret_cast<u32x4 *>(s_pk)[i * kWave + l] = r.k[i];
    if (l < kPMax) s_palpha[l] = pal;
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
      for (int st = 0; st < kPMax; ++st)
#pragma unroll
        for (int u = 0; u < UC; ++u) s_pu[(i * kPMax + st) * L::kPuPitch + u * kWave + l] = r.u[i][st * UC + u];
    gather_gates(0);
  };
  // the records of steps c0 .. c0 + kPMax - 1 for tile t0 + i, straight into
  // LDS (no registers: the column waves' state is in theirs)
  auto restage_records = [&](int c0, int i) {
    if (l >= c0 && l < c0 + kPMax) s_palpha[l - c0] = pal;
    uint32_t kp[KI];
#pragma unroll
    for (int x = 0; x < KI; ++x) kp[x] = key_at(c0, x);
    __builtin_amdgcn_sched_barrier(0);  // an LDS operation after a direct load waits for it
#pragma unroll
    for (int x = 0; x < KI; ++x) load_lds16(pk0 + kp[x], s_pk + x * kWave * EC);
#pragma unroll
    for (int st = 0; st < kPMax; ++st)
#pragma unroll
      for (int u = 0; u < UC; ++u) load_lds4(pu0 + u_row(c0, st) + u_col(i, u), s_pu + (i * kPMax + st) * L::kPuPitch + u * kWave);
    gather_gates(c0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  };

  // ---- setup wave: path check, topology
  int maxd = 0;    // the deepest root path (wave-uniform)
  auto setup = [&](Records &rec) {
    const bool live = l < n;
    if (!live) p = -1;
    auto up = [](int x, int v) { return __shfl(v, x >= 0 ? x : 0); };
    auto upf = [](int x, float v) { return __shfl(v, x >= 0 ? x : 0); };
    // The path: step t is node path[t], whose parent must be path[t - 1] (-1
    // for t = 0).  Root paths: p_s is a node's s-th ancestor (-1 past the
    // root) and g_s the product of the gates of its first s path nodes, itself
    // included: D_jx = g_s for the ancestor x = p_s.  (An LDS round trip per
    // line of lane reads: independent ones share a line.)
    const int node = a.has_pending && l < pn ? nodec : -1;
    const bool inrange = node >= 0 && node < pn;
    nodec = inrange ? node : 0;
    const int prev = __builtin_amdgcn_update_dpp(-1, node, 0x138, 0xf, 0xf, false);  // wave_shr:1, -1 into lane 0
    int xw[4];
    float gw[4];
    const int ppar = __shfl(prow_parent, nodec), pa = up(p, p);
    const float pgate = __shfl(pal, nodec), ga = upf(p, al);
    pal = pgate;
    const bool pbad = a.has_pending && wave_any((plen < 0 || plen > pn) || (l < plen && (!inrange || ppar != prev)));
    if (a.has_pending) read_records(rec);  // at once, ahead of the topology
    xw[0] = p;
    gw[0] = al;
    xw[1] = p >= 0 ? pa : -1;
    gw[1] = p >= 0 ? al * ga : al;
    const int pb = up(xw[1], p), pc = up(xw[1], xw[1]);
    const float gb = upf(xw[1], al), gc = upf(xw[1], gw[1]);
    for (int c = l; c < (L::kT + L::kAt) / 16; c += kWave) reinterpret_cast<uint4 *>(tb)[c] = make_uint4(0, 0, 0, 0);
    xw[2] = xw[1] >= 0 ? pb : -1;
    gw[2] = xw[1] >= 0 ? gw[1] * gb : gw[1];
    xw[3] = xw[1] >= 0 ? pc : -1;
    gw[3] = xw[1] >= 0 ? gw[1] * gc : gw[1];
    const int p4 = xw[3];
    const float g4 = gw[3];

    // topology and decays; lane j owns node j
    bool bad = live && (p < -1 || p >= l);
    if (a.chain) bad = bad || (live && p != l - 1);
    int err = wave_any(bad) ? SLA_ERR_TOPOLOGY : SLA_OK;
    if (err == SLA_OK) {
      // Four walkers per lane start at ancestors 1 to 4 and hop four at a time;
      // the scalar families park each D_jx at (j, x) of the Attn and the Lk
      // blocks for the Grams.  Products of gates only: they may underflow,
      // never overflow (no reciprocal of a decay product anywhere).  One hop
      // per ancestor took 10 us of a 48-node chain's launch.
      uint64_t m = live ? (1ull << l) : 0ull;
      // block entry (l, x) is at row0 + x + 304 (x / 16) floats
      const int row0 = ((l >> 4) * ((l >> 4) + 1) / 2) * (16 * kBP) + (l & 15) * kBP;
      static_assert(16 * kBP - 16 == 304, "block pitch");
      if (DELTA && live) ab[row0 + (l >> 4) * 304 + l] = 1.f;
      while (wave_any(xw[0] >= 0)) {
        int px[4];
        float gx[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          px[r] = up(xw[r], p4);
          gx[r] = upf(xw[r], g4);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int x = xw[r];
          if (x >= 0) {
            if constexpr (DELTA) {
              const int at = row0 + (x >> 4) * 304 + x;
              ab[at] = gw[r];
              tb[at] = gw[r];
            }
            m |= 1ull << x;
            gw[r] *= gx[r];  // walker 0, once past the root: the gates of the whole path
            xw[r] = px[r];
          }
        }
      }
      const int d = __popcll(m);
      if constexpr (GV) {  // the deepest root path
        maxd = d;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) maxd = max(maxd, __shfl_xor(maxd, o));
      }
      if (live) {
        s_anc[l] = m;
        s_gamma[l] = gw[0];
        s_be[l] = be;
      }
    }
    if (err == SLA_OK && pbad) err = SLA_ERR_PATH;
    if (l == 0) {
      s_misc[0] = err;
      s_misc[1] = plen;
      s_misc[2] = maxd;
    }
    if (t0 == 0 && h == 0 && l == 0 && a.status) a.status[b] = err;
  };
  // ---- setup wave: the second tile's first DK/2 state rows into LDS, queued
  //      behind the records.  Chunk c holds row r = c / 16, column
  //      chunk (c % 16) ^ 4 ((r / 8) % 4), so that the 16 column-wave lanes of
  //      a row group and the four row groups fall on distinct banks.  Columns
  //      past d_v (a ragged last tile) re-read column 0 and are never used.
  auto stage_second_tile = [&]() {
    if constexpr (L::kPrefetch) {
      const int cb = (t0 + 1) * kTileCols;
#pragma unroll
      for (int m = 0; m < L::kPreInstr; ++m) {
        const int c = m * kWave + l;
        const int r = c >> 4;
        const int col = cb + 4 * ((c & 15) ^ (((r >> 3) & 3) << 2));
        load_lds16(a.state + (unit * DK + r) * dv + (col < dv ? col : 0), s_pre + m * kWave * 4);
      }
    }
  };

  // ---- GLA: the tree-masked scores with per-key decay ratios,
  //          Attn_ja = sum_i q_j[i] D_ja[i] k_a[i],  D_ja = product of the
  //          gates of P(j) strictly below a (j included), per key dimension,
  //      on the vector ALUs: 16 lanes per node j, each holding d_k / 16 key
  //      dimensions of qc = D_ja * q_j.  Walking up P(j) from j, every step
  //      sums qc . k_a over the 16 lanes (DPP) and then multiplies in a's
  //      gates, so qc ends as Gamma_j * q_j = Q~_j, split into bf16 hi (in
  //      place of q_j) + lo for P_q = Q~ H0.  Gate products only: they may
  //      underflow, never overflow.  The records (the key as given, the
  //      gates) are written from here.
  auto gate_scores = [&]() {
    if constexpr (GV) {
      constexpr int E = DK / 16;  // key dimensions per lane
      const int maxd = s_misc[2];
      unsigned char *xb = reinterpret_cast<unsigned char *>(xs);
      unsigned char *xlb = reinterpret_cast<unsigned char *>(xl);
      // byte offset of the 4 (E = 4) or 8 key dimensions d0 .. of stage row r
      auto xoff = [&](int r, int d0) {
        if constexpr (F32) return xchunk<CH>(r, d0 >> 2) * 16;  // four fp32 per chunk; d0 % 4 == 0
        return xchunk<CH>(r, d0 >> 3) * 16 + ((d0 >> 2) & 1) * 8;
      };
      auto load_row = [&](int r, int d0, float (&x)[E]) {
        if constexpr (F32) {
#pragma unroll
          for (int c = 0; c < E; c += 4) {
            const float4 u = *reinterpret_cast<const float4 *>(xb + xoff(r, d0 + c));
            x[c] = u.x, x[c + 1] = u.y, x[c + 2] = u.z, x[c + 3] = u.w;
          }
          return;
        }
#pragma unroll
        for (int c = 0; c < E; c += 8 < E ? 8 : E) {
          uint32_t wv[4];
          if constexpr (E >= 8) {
            const uint4 u = *reinterpret_cast<const uint4 *>(xb + xoff(r, d0 + c));
            wv[0] = u.x, wv[1] = u.y, wv[2] = u.z, wv[3] = u.w;
          } else {
            const uint2 u = *reinterpret_cast<const uint2 *>(xb + xoff(r, d0 + c));
            wv[0] = u.x, wv[1] = u.y;
          }
#pragma unroll
          for (int e = 0; e < (E >= 8 ? 8 : E); e += 2) {
            x[c + e] = __uint_as_float(wv[e / 2] << 16);
            x[c + e + 1] = __uint_as_float(wv[e / 2] & 0xffff0000u);
          }
        }
      };
      // the sum over the 16 lanes of a DPP row, in every lane
      auto row_sum = [](float v) {
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, false));  // row_half_mirror
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, false));  // row_mirror
        return v;
      };
#pragma unroll 1
      for (int it0 = w * kWave; it0 < NP * 16; it0 += kColWaves * kWave) {  // wave-uniform
        const int j = (it0 + l) >> 4, d0 = ((it0 + l) & 15) * E;
        const bool first = (l & 15) == 0;
        float qc[E];
        load_row(j, d0, qc);  // padding rows are zero
        uint64_t rest = j < n ? s_anc[j] : 0ull;
        // every lane takes all maxd steps, so the DPP rows stay whole
#pragma unroll 1
        for (int st = 0; st < maxd; ++st) {
          const bool act = rest != 0ull;
          const int an = act ? 63 - __builtin_clzll(rest) : 0;  // deepest ancestor left: j, then up
          rest &= ~(1ull << an);
          float ka[E];
          load_row(NP + an, d0, ka);
          float sdot = 0.f;
#pragma unroll
          for (int e = 0; e < E; ++e) sdot = __builtin_fmaf(qc[e], ka[e], sdot);
          sdot = row_sum(sdot);
          if (act && first) ab[blk(j, an)] = sdot;
          if (act) {
#pragma unroll
            for (int e = 0; e < E; e += 4) {
              const float4 gx = *reinterpret_cast<const float4 *>(s_g + an * DK + d0 + e);
              qc[e] *= gx.x;
              qc[e + 1] *= gx.y;
              qc[e + 2] *= gx.z;
              qc[e + 3] *= gx.w;
            }
          }
        }
        if (j >= n) {  // padding rows: zero low halves (their products are dropped)
          if constexpr (!F32) {
#pragma unroll
            for (int c = 0; c < E; c += 4) *reinterpret_cast<uint2 *>(xlb + xoff(j, d0 + c)) = make_uint2(0, 0);
          }
          continue;
        }
        if constexpr (F32) {  // Q~ in fp32 in place of q_j; the records: the key as given, the gates
#pragma unroll
          for (int c = 0; c < E; c += 4) {
            *reinterpret_cast<float4 *>(xb + xoff(j, d0 + c)) = make_float4(qc[c], qc[c + 1], qc[c + 2], qc[c + 3]);
            if (t0 == 0) {
              const size_t r = ((nbase + j) * H + h) * DK + d0 + c;
              *reinterpret_cast<float4 *>(static_cast<float *>(a.fk) + r) =
                  *reinterpret_cast<const float4 *>(xb + xoff(NP + j, d0 + c));
              *reinterpret_cast<float4 *>(a.falpha + r) = *reinterpret_cast<const float4 *>(s_g + j * DK + d0 + c);
            }
          }
          continue;
        }
#pragma unroll
        for (int c = 0; c < E; c += 4) {
          uint32_t hw[2], lw[2];
#pragma unroll
          for (int e2 = 0; e2 < 2; ++e2) {
            uint32_t hv = 0, lv = 0;
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
              const float x = qc[c + 2 * e2 + s2];
              const __bf16 xh = static_cast<__bf16>(x);
              const __bf16 xl2 = static_cast<__bf16>(x - static_cast<float>(xh));
              hv |= (uint32_t)__builtin_bit_cast(uint16_t, xh) << (16 * s2);
              lv |= (uint32_t)__builtin_bit_cast(uint16_t, xl2) << (16 * s2);
            }
            hw[e2] = hv;
            lw[e2] = lv;
          }
          *reinterpret_cast<uint2 *>(xb + xoff(j, d0 + c)) = make_uint2(hw[0], hw[1]);
          *reinterpret_cast<uint2 *>(xlb + xoff(j, d0 + c)) = make_uint2(lw[0], lw[1]);
          if (t0 == 0) {
            const size_t r = ((nbase + j) * H + h) * DK + d0 + c;
            *reinterpret_cast<uint2 *>(static_cast<bf16 *>(a.fk) + r) =
                *reinterpret_cast<const uint2 *>(xb + xoff(NP + j, d0 + c));
            *reinterpret_cast<float4 *>(a.falpha + r) = *reinterpret_cast<const float4 *>(s_g + j * DK + d0 + c);
          }
        }
      }
    }
  };

  // ---- tree-masked Grams over the column waves (scalar gates; GLA's scores
  //      were formed above): tile (mr, na) of [Q; K] K^T holds rows of node
  //      tile mr % NT against ancestor candidates of node tile na <= mr % NT;
  //      ancestor entries go to Attn blocks and Lk lists
  auto grams = [&]() {
    if constexpr (!GV) {
      f32x4 gacc[GT];
      int tc = 0;
#pragma unroll
      for (int mr = 0; mr < MT; ++mr)
#pragma unroll
        for (int na = 0; na <= mr % NT; ++na, ++tc) {
          if (tc % kColWaves != w || (mr % NT) * 16 >= n || (!DELTA && mr >= NT)) continue;
          f32x4 g = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            if constexpr (F32) {
              float av[8], bv[8];
              frag8(mr * 16 + lc, ks, av);
              frag8(NP + na * 16 + lc, ks, bv);
#pragma unroll
              for (int e = 0; e < 8; ++e) g = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[e], g, 0, 0, 0);
            } else {
              const bf16x8 af = *reinterpret_cast<const bf16x8 *>(xs + xchunk<CH>(mr * 16 + lc, ks * 4 + lg));
              const bf16x8 bf = *reinterpret_cast<const bf16x8 *>(xs + xchunk<CH>(NP + na * 16 + lc, ks * 4 + lg));
              g = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, g, 0, 0, 0);
            }
          }
          gacc[tc / kColWaves] = g;
        }
      tc = 0;
#pragma unroll
      for (int mr = 0; mr < MT; ++mr)
#pragma unroll
        for (int na = 0; na <= mr % NT; ++na, ++tc) {
          if (tc % kColWaves != w || (mr % NT) * 16 >= n || (!DELTA && mr >= NT)) continue;
          // every LDS read of the tile's metadata is issued before its first
          // write, so they share one round trip
          const int bj = mr % NT;
          const int an = na * 16 + lc;
          const int jb = bj * 16 + 4 * lg;
          uint32_t anc[4];  // the half of row j's ancestor mask that holds column an
          float dj[4], be4[4];  // dj: decay ratio D_{j,an}, parked where the entry goes
          float *const db = (mr < NT ? ab : tb) + ((bj * (bj + 1)) / 2 + na) * (16 * kBP) + 4 * lg * kBP + lc;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            anc[q] = reinterpret_cast<const uint32_t *>(s_anc)[2 * (jb + q) + (na >> 1)];
            dj[q] = db[q * kBP];
            be4[q] = mr >= NT ? s_be[jb + q] : 0.f;
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int j = jb + q;
            // every entry is written: zero unless an is an ancestor of j (rows
            // past the last node hold stale LDS words: masked by j < n; the
            // diagonal of Lk is not read)
            const bool on = j < n && an <= j && !(mr >= NT && an == j) && ((anc[q] >> (an & 31)) & 1u);
            const float dg = dj[q] * gacc[tc / kColWaves][q];
            db[q * kBP] = on ? (mr < NT ? dg : -(be4[q] * dg)) : 0.f;
          }
        }
    }
  };

  // ---- the two kinds of waves up to the barrier behind which the Grams and
  //      the records are complete: branches of their own (the wave number is
  //      scalar), so that neither's registers are live, nor its outstanding
  //      reads waited for, in the other
  if constexpr (kSetup == 0) {
    column_reads();
    if (w == kSetup) {
      Records rec;
      setup(rec);
      if (a.has_pending) stage_records(rec);
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      if constexpr (!kLate) load_state(t0, hfa);  // its own state: after its record reads
    } else if constexpr (!kLate) {
      load_state(t0, hfa);
    }
    __syncthreads();
    if (s_misc[0] != SLA_OK) return;
    gate_scores();
    if constexpr (kLate) load_state(t0, hfa);
    grams();
  } else if (w != kSetup) {
    column_reads();
    __syncthreads();
    if (s_misc[0] != SLA_OK) return;
    // many rounds of workgroups: the state goes out only now, behind the small
    // reads the setup wave waits for
    if constexpr (kLate) load_state(t0, hfa);
    gate_scores();
    grams();
  } else {
    Records rec;
    setup(rec);
    __syncthreads();
    if (s_misc[0] != SLA_OK) return;
    if (a.has_pending) stage_records(rec);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    stage_second_tile();
  }
  __syncthreads();
  plen = s_misc[1];

  if (DELTA && w == kSetup) {
    // ---- the diagonal blocks of T = (I + Lk)^-1, less the identity (kUnitT: with it), in place
    //      (the off-diagonal blocks stay -Lk: U = T R is a substitution block
    //      row by block row).  Lane (nb, c) solves column c of block nb by
    //      forward substitution in registers; the cost does not depend on the
    //      depth of the tree (one lane per row, walking its root path, took
    //      1.6 us at depth 8, 12 us on a 16-node chain and 107 us on a 48-node
    //      chain, on the critical path of a single sequence).
    const int nb = l >> 4, c = l & 15;
    if (nb < NT) {
      float *const db = tb + ((nb * (nb + 1)) / 2 + nb) * (16 * kBP);
      float x[16];
      x[0] = c == 0 ? 1.f : 0.f;
#pragma unroll
      for (int j = 1; j < 16; ++j) {
        float sum = j == c ? 1.f : 0.f;
#pragma unroll
        for (int a0 = 0; a0 < j; a0 += 4) {
          const float4 lv = *reinterpret_cast<const float4 *>(db + j * kBP + a0);
          sum = __builtin_fmaf(lv.x, x[a0], sum);
          if (a0 + 1 < j) sum = __builtin_fmaf(lv.y, x[a0 + 1], sum);
          if (a0 + 2 < j) sum = __builtin_fmaf(lv.z, x[a0 + 2], sum);
          if (a0 + 3 < j) sum = __builtin_fmaf(lv.w, x[a0 + 3], sum);
        }
        x[j] = sum;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) db[j * kBP + c] = j == c ? (kUnitT ? 1.f : 0.f) : x[j];
    }
  }

  // ---- one V-tile: [A] delayed state update, write-back, P = [Q; K] H0
  //      (bf16: state split into hi + lo; fp32: exact) and R on the column waves; barrier (T complete);
  //      [B] U = T R, O = Gamma P_q + Attn U and the stores; then the next
  //      tile's state and values go out.
  const uint32_t obytes = ((uint32_t)(n - 1) * nstride + dv) * 4;
  const rsrc_t orr = make_rsrc(a.out + (nbase * H + h) * dv, obytes);
  const rsrc_t urr = make_rsrc(a.fu + (nbase * H + h) * dv, obytes);
  auto step = [&](int i, float (&hf)[KS][8], float (&hn)[KS][8]) {
    const int t = t0 + i;
    const bool more = i + 1 < cnt;
    const bool cols_live = live(t);
    const int col = t * kTileCols + ucol;
    const uint32_t sv = (uint32_t)(8 * lg * dv + col) * 4;
    const float *pu = s_pu + i * kPMax * L::kPuPitch;

    // accumulator layout: lane (lg, lc) holds rows 4 lg .. 4 lg + 3 of each
    // 16-row tile, column lc
    f32x4 pq[NT];  // P_q = Q H0, accumulator layout
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) pq[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 rreg[NT];
    // delayed state update, kPMax steps of the accepted path at a time; longer
    // paths restage the records between two barriers (plen is
    // workgroup-uniform).  (Each column wave used to read the steps past the
    // first eight itself, two dependent reads per step.)
    for (int c0 = 0; c0 < plen; c0 += kPMax) {
      if (c0 + (plen > kPMax ? i : 0) > 0) {
        __syncthreads();
        if (w == kSetup) restage_records(c0, i);
        __syncthreads();
      }
      const int ps = plen - c0 < kPMax ? plen - c0 : kPMax;
      if (cols_live) {
        // the whole tile has normally landed by now: step-major, one LDS
        // round trip per step
        for (int st = 0; st < ps; ++st) {
          const float al = s_palpha[st];
          const float uv = pu[st * L::kPuPitch + ucol];
          constexpr int KC = F32 || GV || KS < 4 ? 2 : 4;  // K-steps per LDS round trip
#pragma unroll
          for (int k0 = 0; k0 < KS; k0 += KC) {
            float kv[KC][8];  // the key's rows 32 (k0 + c) + 8 lg + e
            float gv[KC][8];  // GLA: the gates of the same rows
#pragma unroll
            for (int c = 0; c < KC; ++c) {
              if constexpr (F32) {
                const float4 k0v = *reinterpret_cast<const float4 *>(s_pk + st * DK + (k0 + c) * 32 + 8 * lg);
                const float4 k1v = *reinterpret_cast<const float4 *>(s_pk + st * DK + (k0 + c) * 32 + 8 * lg + 4);
                kv[c][0] = k0v.x, kv[c][1] = k0v.y, kv[c][2] = k0v.z, kv[c][3] = k0v.w;
                kv[c][4] = k1v.x, kv[c][5] = k1v.y, kv[c][6] = k1v.z, kv[c][7] = k1v.w;
              } else {
                const bf16x8 kb = *reinterpret_cast<const bf16x8 *>(s_pk + st * DK + (k0 + c) * 32 + 8 * lg);
#pragma unroll
                for (int e = 0; e < 8; ++e) kv[c][e] = static_cast<float>(kb[e]);
              }
            }
            if constexpr (GV) {
#pragma unroll
              for (int c = 0; c < KC; ++c) {
                const float4 g0 = *reinterpret_cast<const float4 *>(s_pg + st * DK + (k0 + c) * 32 + 8 * lg);
                const float4 g1 = *reinterpret_cast<const float4 *>(s_pg + st * DK + (k0 + c) * 32 + 8 * lg + 4);
                gv[c][0] = g0.x, gv[c][1] = g0.y, gv[c][2] = g0.z, gv[c][3] = g0.w;
                gv[c][4] = g1.x, gv[c][5] = g1.y, gv[c][6] = g1.z, gv[c][7] = g1.w;
              }
            }
#pragma unroll
            for (int c = 0; c < KC; ++c)
#pragma unroll
              for (int e = 0; e < 8; ++e)
                hf[k0 + c][e] = apply_factor(hf[k0 + c][e], GV ? gv[c][e] : al, kv[c][e], uv);
          }
        }
      }
    }
    if (cols_live) {
      if (a.has_pending) {
        // committed rows back.  A wave writes half of each 128-byte line and
        // the neighbouring wave the other half.  Over many rounds of
        // workgroups the default policy lets the L2 merge the halves (a plain
        // streaming hint wrote them separately: 8% more HBM writes, 4.7%
        // longer launches).  In a single round the rows are written through
        // at device scope instead: what stays dirty in the L2 is written back
        // at the end of the kernel, on its critical path (measured at batched
        // tree serving 39.2 -> 37.9 us per launch; on the 1-node decode chain,
        // eight rounds, the default policy stays 2% faster).
        // (chosen at launch: a run-time branch between the two store loops
        // cost most of the gain)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            buf_store_f32<WT ? kPolicyStreamDevice : kPolicyDefault>(hf[ks][e], sr, sv, (uint32_t)(ks * 32 + e) * dv * 4);
      }
      // P_k = K H0 first (K-step by K-step as the tile lands; bf16: the
      // state split into hi + lo, fp32: exact products), so that
      // R = beta (v - gamma P_k) takes its place before P_q is built: the two
      // halves of P are never held at once
      f32x4 pk[NT];
#pragma unroll
      for (int mt = 0; mt < NT; ++mt) pk[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      bf16x8 bhi[F32 ? 1 : KS], blo[F32 ? 1 : KS];  // the state's two bf16 parts, in place of its registers
      if constexpr (DELTA && F32) {  // exact fp32 products: the state registers are the B operands
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int mt = 0; mt < NT; ++mt) {
            float av[8];
            frag8(NP + mt * 16 + lc, ks, av);
#pragma unroll
            for (int e = 0; e < 8; ++e) pk[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], hf[ks][e], pk[mt], 0, 0, 0);
          }
      } else if constexpr (DELTA) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          split8(hf[ks], bhi[ks], blo[ks]);
#pragma unroll
          for (int mt = 0; mt < NT; ++mt) {
            const bf16x8 af = *reinterpret_cast<const bf16x8 *>(xs + xchunk<CH>(NP + mt * 16 + lc, ks * 4 + lg));
            pk[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bhi[ks], pk[mt], 0, 0, 0);
            pk[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, blo[ks], pk[mt], 0, 0, 0);
          }
        }
      }
      // R in the accumulator layout (the row base is rebuilt per tile:
      // hoisted out of the tile loop it only gets spilled)
      int rb = 4 * lg;
      __asm__("" : "+v"(rb));
#pragma unroll
      for (int mt = 0; mt < NT; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = mt * 16 + rb + q;
          uint32_t vb = vraw[mt][q];
          __asm__("" : "+v"(vb));  // keeps the widening here, not next to the load
          const float vf = __uint_as_float(F32 ? vb : vb << 16);
          const float rd = DELTA ? s_be[j] * (vf - s_gamma[j] * pk[mt][q]) : vf;
          rreg[mt][q] = j < n ? (nodelta ? vf : rd) : 0.f;
        }
      if constexpr (F32) {  // Q (GLA: Q~) H0, exact fp32 products
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int mt = 0; mt < NT; ++mt) {
            float av[8];
            frag8(mt * 16 + lc, ks, av);
#pragma unroll
            for (int e = 0; e < 8; ++e) pq[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], hf[ks][e], pq[mt], 0, 0, 0);
          }
      } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          if constexpr (!DELTA) split8(hf[ks], bhi[ks], blo[ks]);
#pragma unroll
          for (int mt = 0; mt < NT; ++mt) {
            const bf16x8 af = *reinterpret_cast<const bf16x8 *>(xs + xchunk<CH>(mt * 16 + lc, ks * 4 + lg));
            pq[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bhi[ks], pq[mt], 0, 0, 0);
            pq[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, blo[ks], pq[mt], 0, 0, 0);
            if constexpr (GV) {  // Q~ lo half
              const bf16x8 afl = *reinterpret_cast<const bf16x8 *>(xl + xchunk<CH>(mt * 16 + lc, ks * 4 + lg));
              pq[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afl, bhi[ks], pq[mt], 0, 0, 0);
            }
          }
        }
      }
    }
    // the next tile's state and values go out now, while this tile's U, O
    // and stores are computed: its state registers are free since P_q, its
    // values since R
    if (TPW > 1 && more && live(t + 1)) {
      load_state(t + 1, hn, L::kPrefetch ? KS / 2 : 0);
      load_values(t + 1, vraw);
    }
    if (L::kPrefetch && w == kSetup && i == 0) __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // staged rows landed
    __syncthreads();  // T complete
    if (L::kPrefetch && more && live(t + 1)) {
      // the staged rows of the next tile: row 32 ks + 8 lg + e, column chunk
      // ucol / 4 swizzled by lg
#pragma unroll
      for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int r = ks * 32 + 8 * lg + e;
          hn[ks][e] = s_pre[(r * 16 + ((ucol >> 2) ^ (lg << 2))) * 4 + (lc & 3)];
        }
    }
    // factor records independent of the V-tile -- k (from the staged rows),
    // alpha, parent -- while the column waves compute the first tile's
    // products (off the path to the barrier above)
    if (w == kSetup && i == 0 && t0 == 0) {
      if constexpr (!GV) {  // GLA's key and gate records went out with Q~
        AT *fk = static_cast<AT *>(a.fk);
        for (int c = l; c < n * CH; c += kWave) {
          const int j = c / CH, part = c % CH;
          *reinterpret_cast<uint4 *>(fk + ((nbase + j) * H + h) * DK + part * EC) = xs[xchunk<CH>(NP + j, part)];
        }
      }
      if (l < n) {
        if constexpr (!GV) a.falpha[(nbase + l) * H + h] = al;
        if (h == 0) a.fparent[nbase + l] = p;
      }
    }
    if (cols_live) {  // no early return: every wave takes every later barrier
      // ---- U = T R, then O = Gamma P_q + Attn U, on the matrix cores; A
      //      fragments are rows j = 16 mt + lc, columns 16 ks + 4 lg .. + 3.
      //      U by block rows: X = R - sum over the blocks to the left of
      //      Lk U, then U = X + (T - I) X with the diagonal block's T: R
      //      enters the fp32 accumulators as it is
      f32x4 uacc[NT];  // same layout as R
      s16x4 uhi[NT], ulo[NT];
      auto blockrow = [&](const float *m, int mt, int ks) {  // this lane's four A elements of block (mt, ks)
        return *reinterpret_cast<const f32x4 *>(m + ((mt * (mt + 1)) / 2 + ks) * (16 * kBP) + lc * kBP + 4 * lg);
      };
#pragma unroll
      for (int mt = 0; mt < NT; ++mt) {
        uacc[mt] = rreg[mt];
        if constexpr (DELTA && F32) {
          // the corrections are summed by themselves and R enters once, at the
          // end: in the accumulators from the start it rounds every product at
          // its own size (64-node chains, d_k 64: U's error from fp64 6.0e-8,
          // then 1.5e-7; 16-node chains 6.5e-8 and 8.3e-8).  A single block
          // takes R through the diagonal of T instead: no register holds R to
          // the end (the paired form would need 82, and a wave per SIMD less).
          // A operand i: column 16 ks + 4 lg + i of row 16 mt + lc, B operand i: U[16 ks + 4 lg + i][lc]
          f32x4 cor = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < mt; ++ks) {
            const f32x4 lv = blockrow(tb, mt, ks);
#pragma unroll
            for (int i = 0; i < 4; ++i) cor = __builtin_amdgcn_mfma_f32_16x16x4f32(lv[i], uacc[ks][i], cor, 0, 0, 0);
          }
          const f32x4 nv = blockrow(tb, mt, mt);
          f32x4 x;
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = mt == 0 ? rreg[0][i] : rreg[mt][i] + cor[i];
#pragma unroll
          for (int i = 0; i < 4; ++i) cor = __builtin_amdgcn_mfma_f32_16x16x4f32(nv[i], x[i], cor, 0, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) uacc[mt][i] = kUnitT ? cor[i] : rreg[mt][i] + cor[i];
        } else if constexpr (DELTA) {
          s16x4 ah, al2, xh, xl2;
#pragma unroll
          for (int ks = 0; ks < mt; ++ks) {
            split4(blockrow(tb, mt, ks), ah, al2);
            uacc[mt] = mfma16_split(ah, al2, uhi[ks], ulo[ks], uacc[mt]);
          }
          split4(uacc[mt], xh, xl2);
          split4(blockrow(tb, mt, mt), ah, al2);
          uacc[mt] = mfma16_split(ah, al2, xh, xl2, uacc[mt]);
        }
        if constexpr (!F32) split4(uacc[mt], uhi[mt], ulo[mt]);
      }
      // outputs and corrected values of node j at ((b n + j) H + h) dv + col;
      // rows past the last node fall outside the descriptors (the whole offset
      // is carried per lane, where the range check applies) and are dropped
      const uint32_t ov = (4 * lg * nstride + col) * 4;
#pragma unroll
      for (int mt = 0; mt < NT; ++mt) {
        f32x4 oacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks <= mt; ++ks) {
          const f32x4 av = blockrow(ab, mt, ks);
          if constexpr (F32) {
#pragma unroll
            for (int i = 0; i < 4; ++i) oacc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], uacc[ks][i], oacc, 0, 0, 0);
          } else {
            s16x4 ah, alo;
            split4(av, ah, alo);
            oacc = mfma16_split(ah, alo, uhi[ks], ulo[ks], oacc);
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = mt * 16 + 4 * lg + q;
          const uint32_t vo = ov + (uint32_t)(mt * 16 + q) * nstride * 4;
          buf_store_f32<kPolicyStream>(uacc[mt][q], urr, vo, 0);
          buf_store_f32<kPolicyStream>(__builtin_fmaf(s_gamma[j], pq[mt][q], oacc[q]), orr, vo, 0);
        }
      }
    }
  };
  // straight-line, the two state register sets trading roles (in a loop
  // the compiler loses track of which loads a register still waits for;
  // four tiles in a row spill)
  static_assert(TPW == 1 || TPW == 2, "tiles per workgroup");
  step(0, hfa, hfb);
  if constexpr (TPW == 2) step(1, hfb, hfa);
}

// Rounds of workgroups from which a launch is kModeLate.
constexpr int kLateRounds = 4;

template <int DK, int NP, int CW, int TPW, int KIND, bool F32>
hipError_t launch_np(const VerifyArgs &a, hipStream_t s) {
  using L = Layout<DK, NP, CW, TPW, KIND, F32>;
  constexpr size_t lds = L::kBytes;
  if constexpr (lds > kMaxLds) {
    return hipErrorInvalidConfiguration;
  } else {
    using Kernel = void (*)(VerifyArgs);
    const Kernel part = verify_tile_kernel<DK, NP, CW, TPW, KIND, F32, kModePart>;
    const Kernel round = verify_tile_kernel<DK, NP, CW, TPW, KIND, F32, kModeRound>;
    const Kernel late = verify_tile_kernel<DK, NP, CW, TPW, KIND, F32, kLateAlways<DK, NP, CW, KIND, F32> ? kModePart : kModeLate>;
    auto allow_lds = [](Kernel k) {
      if (lds <= kDefaultLds) return hipSuccess;
      return hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    };
    // resident workgroups per CU for this instantiation (registers, LDS, waves)
    static const int per_cu = [&] {
      int k = 0;
      if (allow_lds(round) != hipSuccess ||
          hipOccupancyMaxActiveBlocksPerMultiprocessor(&k, round, kWaves<CW> * kWave, lds) != hipSuccess || k < 1) k = 1;
      return k;
    }();
    const int ntiles = (a.dv + L::kTileCols - 1) / L::kTileCols;
    const size_t groups = (size_t)a.B * a.H * ((ntiles + TPW - 1) / TPW);
    const size_t slots = (size_t)per_cu * device_cus();
    const Kernel kern = groups >= (size_t)kLateRounds * slots ? late : (groups >= slots && a.dv % 32 == 0 ? round : part);
    const hipError_t e = allow_lds(kern);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kWaves<CW> * kWave), lds, s, a);
    return hipGetLastError();
  }
}

// One V-tile per workgroup: 48 columns instead of 64 where as many tiles then
// cover d_v with fewer waves (d_v 16 to 48, 80, 96, 144) and that lets more
// workgroups share a CU.  Geometric means of three waves against four over
// these d_v, 12 heads, batch 1 to 256:
//   scalar gates  d_k 64 0.95, 0.97, 0.95 at 8, 23 and 48 nodes, d_k 128 0.96,
//                 0.95, 0.98, d_k 256 0.93, 0.94, at most 4% longer (batch 40,
//                 d_k 256, d_v 80, 8 and 23 nodes: 36.2 -> 29.5, 46.6 -> 35.5 us);
//                 not for 33 to 64 nodes at d_k 256, where one stage fills a CU
//                 anyway (1.01, up to 1.05);
//   per-key gates the scores are spread over the column waves, so fewer waves
//                 cost where the launch does not fill the CUs: 1.02 to 1.13
//                 below two tiles per CU, 1.00 to 1.05 from two to three (d_k
//                 256, and 128 in fp32, up to 16 nodes) or to four.  Above that
//                 0.90 to 1.00 for the forms of kThreeWaves, 1.01 to 1.05 for
//                 the others (no more workgroups per CU, or registers spilled
//                 to fit them), 1.04 to 1.07 for 33 to 64 nodes.
template <int DK, int NP, int KIND, bool F32>
constexpr bool kThreeWaves =
    KIND == kKindDelta ? DK < 256 || NP < 64
                       : (NP == 16 ? DK != 128 || F32 : NP == 32 && (DK == 64 || (DK == 128 && !F32)));

template <int DK, int NP, int KIND, bool F32>
hipError_t launch_single(const VerifyArgs &a, hipStream_t s) {
  if constexpr (kThreeWaves<DK, NP, KIND, F32>) {
    const int waves = a.dv / kWaveCols, tiles = (waves + 3) / 4;
    if (waves % 4 != 0 && (waves + 2) / 3 == tiles &&
        (KIND == kKindDelta || (size_t)a.B * a.H * tiles > (size_t)(NP == 16 && DK > 64 ? 3 : 4) * device_cus()))
      return launch_np<DK, NP, 3, 1, KIND, F32>(a, s);
  }
  return launch_np<DK, NP, 4, 1, KIND, F32>(a, s);
}

// Drafts of more than 16 nodes: single 64-column tiles while they do not fill
// the CUs (one, or two where two stages fit a CU's LDS); else one workgroup
// covers more columns, so that topology, Grams and the inverse serve them all
// and, where one stage fills a CU, eight column waves instead of four share it.
// Measured, us per launch: 64 nodes, 16 heads, d_k 128, d_v 256, single tiles
// against pairs of 128 columns: batch 1 12.6 and 22.2, batch 4 16.1 and 24.3,
// batch 8 (512 tiles) 21.7 and 26.0, batch 16 45.9 and 30.9; 8 heads, d_k = d_v
// = 256, 64 nodes: batch 4 19.4 and 32.8, batch 32 80.3 and 55.5 (one tile of
// 128 columns: 57.5); 16 heads, d_k 256, d_v 128, batch 16: 42.3, and 28.4 in
// one tile of 128 columns.  Where d_v holds no whole 128-column tiles, pairs of
// 64-column ones: 12 heads, d_v 80 and 96, per-key gates, batch 12 to 256: 48
// nodes at d_k 128 0.76 of the time of single tiles, 32 nodes at d_k 256 0.81.
template <int DK, int NP, int KIND, bool F32>
hipError_t launch_large(const VerifyArgs &a, hipStream_t s) {
  constexpr size_t stage = Layout<DK, NP, 4, 1, KIND, F32>::kBytes;
  constexpr size_t fit = kMaxLds / stage < 2 ? 1 : 2;
  const size_t tiles = (size_t)a.B * a.H * ((a.dv + kWaveCols * 4 - 1) / (kWaveCols * 4));
  if ((NP > 32 || fit == 1) && tiles > fit * device_cus()) {
    if (a.dv % 256 == 0) return launch_np<DK, NP, 8, 2, KIND, F32>(a, s);
    if constexpr (fit == 1) {
      if (a.dv % 128 == 0) return launch_np<DK, NP, 8, 1, KIND, F32>(a, s);
    }
    if (((a.dv + kWaveCols * 4 - 1) / (kWaveCols * 4)) % 2 == 0) return launch_np<DK, NP, 4, 2, KIND, F32>(a, s);
  }
  return launch_single<DK, NP, KIND, F32>(a, s);
}

template <int DK, int KIND, bool F32>
hipError_t launch_dk(const VerifyArgs &a, hipStream_t s) {
  // small trees: two V-tiles of a unit per workgroup once single tiles would
  // fill every CU's four workgroup slots twice over.  The launch is then one
  // round of long-lived workgroups instead of two, and q, k, topology, Grams
  // and T serve both tiles.  Below that, single tiles keep more workgroups
  // (and CUs) busy.
  if constexpr (DK <= 128) {
    const int ntiles = (a.dv + kWaveCols * 4 - 1) / (kWaveCols * 4);
    if (a.n <= 32 && ntiles % 2 == 0 && (size_t)a.B * a.H * ntiles >= (size_t)8 * device_cus())
      return a.n <= 16 ? launch_np<DK, 16, 4, 2, KIND, F32>(a, s) : launch_np<DK, 32, 4, 2, KIND, F32>(a, s);
  }
  if (a.n <= 16) return launch_single<DK, 16, KIND, F32>(a, s);
  return a.n <= 32 ? launch_large<DK, 32, KIND, F32>(a, s) : launch_large<DK, 64, KIND, F32>(a, s);
}

}  // namespace

// One translation unit per (d_k, form of the step, activation type): the
// build compiles this file once for each, so that they compile in parallel.
template <>
hipError_t launch_tile<SLA_TILE_DK, SLA_TILE_GATES != 0, SLA_TILE_F32 != 0>(const VerifyArgs &a, hipStream_t s) {
  return launch_dk<SLA_TILE_DK, SLA_TILE_GATES ? kKindGates : kKindDelta, SLA_TILE_F32 != 0>(a, s);
}

}  // namespace sla
