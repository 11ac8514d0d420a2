// Slot-walking neighbourhood convolution for any shape (Eqs. 4-5 with the
// activation of Eq. 10), from a neighbour-row table or from coordinates:
//
//   out[i][n] = act( bias[n] + sum_kk A[i][kk] W[kk][n] ),  kk = j Cin + c,
//   A[i][j Cin + c] = S[r_ij][c], absent rows 0,
//
// the slots concatenated into one reduction axis of K Cin entries, walked in
// 64-byte k-steps (32 bf16 or 16 fp32 entries), four of them to a phase.
//
// A workgroup owns R = 16 RW active rows and BN = 16 CW NCT output columns;
// its wavefronts form an RW x CW grid of 16 rows x 16 NCT columns.  Per phase:
//   * the phase's weight rows are in one of two LDS buffers, stored by all
//     threads one phase ahead from registers loaded NWS phases before that;
//     one barrier per phase;
//   * a wavefront's own input rows come straight from memory into registers,
//     16 bytes per lane and k-step, NA - 1 phases ahead.  Raw buffer loads: an
//     absent row gets an offset past the buffer and costs no memory access.
//     Their offsets (an LDS read of the row's slot) are formed a phase
//     earlier still;
//   * the weight fragments of k-step s + 1 are read from LDS before the MFMAs
//     of k-step s; no branch inside a phase.  A wavefront none of whose rows
//     has a slot of the phase skips it.  Workgroups of 128 rows sort their
//     rows by first sparse slot first, so that wavefronts share their slots.
// The product is taken transposed (A operand: weight columns, B operand:
// rows), so a lane ends with whole 16-byte runs of columns of one row and
// stores them without an LDS pass.  Each output element is summed over the
// slots in order and within a slot over the k-steps in order, as in the other
// conv kernels: where they run the same shape the results are the same bits
// (but for the split below).
//
// fp32 in the largest workgroups takes each product as six bf16 ones (SPLIT; the
// three-term splitting is that of Henry, Tang and Heinecke, "Leveraging the
// bfloat16 artificial intelligence datatype for higher-precision
// computations", 2019): an fp32 value, times 2^24 so that no term is too small
// for bf16, is three bf16 terms h + m + l exactly (8 + 8 + 8 significand bits),
// and the products h h, h m, m h, m m, h l and l h are exact in fp32.  Left out
// are m l, l m and l l, together at most 2^-23 of a product (root mean square
// about 2^-27; the rounding of an fp32 sum is up to 2^-24 of the sum).  The h h
// products are summed in one accumulator, the others, at most 2^-7 of them, in a
// second; the two are added in fp64, scaled back, and rounded once with the bias.
// Rows whose sums are not finite (an input of 2^104 or more, an infinity, a NaN,
// a sum of 2^80) are summed again on the fp32 matrix cores, the rows beside them
// in a wavefront are not (the order of rows inside a sort bucket differs from
// launch to launch).  A 32-entry k-step rounds the large sum once, where the fp32
// matrix cores round it for each of its four-entry groups with a nonzero
// product, and the 2-norm error against 64 bits is below theirs from dense
// features to two nonzero products an output (128 -> 128, nine slots half
// present, fp32 matrix cores / split: dense 4.7e-7 / 1.5e-7, half of the features
// nonzero 3.3e-7 / 1.2e-7, a tenth 1.5e-7 / 5.8e-8, 0.4% 3.9e-8 / 2.6e-8; with
// all six products in one accumulator the split erred by 3.9e-7, 2.7e-7 and
// 8.4e-8 on the last three).  Six 16-bit MFMAs of 32 entries take 96 cycles,
// eight fp32 ones 256.  The rows' terms are formed in registers, the weights' as
// they are stored to LDS (three planes).
//
// What bounds it.  Few rows: the chain of phases, each about 0.6 us (barrier,
// LDS write to read, a dependent MFMA chain), so 16-row workgroups spread over
// the CUs (262 rows, K = 9, fp32 16 -> 64: 16.8 us before, in five workgroups
// of the weight-stationary kernel, 6.9 us here; 1,965 rows 128 -> 128 fp32:
// 96 -> 18.6 us; 1,965 rows bf16 256 -> 256: 56 -> 15.8 us).  Many rows in
// fp32: the fp32 matrix rate held it at 370 us for 499 K rows 64 -> 64 with
// 0.91 of the slots present (397 us in the tiled kernel); split, 267 to 294 us
// from card to card, bound by the VALU work of the split, the LDS reads of three
// planes and the MFMAs at about equal shares, and the index prologue of every workgroup (60% of the
// slots present, tiled kernel / split: 498,778 rows 64 -> 64 392 / 245 us, 32,000
// rows 128 -> 128 117 / 55, 26,200 rows 256 -> 256 352 / 207, 300,000 rows 96 ->
// 96 668 / 391; 498,778 rows with an infinity in 2% of them 614).
// Many rows in bf16: the weight stage per 128 rows (93 K rows, K = 5, 32 -> 80:
// 30 -> 26 us; 19 K rows, K = 7, 48 -> 80 from coordinates: 16.2 -> 11.7 us).
#include <mutex>

#include "shc_internal.h"

namespace shc {

bool conv_walk_small(const GemmArgs& a, int num_cus) {
  return ((a.n_rows + 15) / 16) * ((a.Cout + 63) / 64) <= num_cus;
}

bool conv_walk_medium(const GemmArgs& a, int num_cus, int per_cu) {
  return ((a.n_rows + 127) / 128) * ((a.Cout + 31) / 32) <= (int64_t)per_cu * num_cus;
}

namespace {

constexpr int kWalkMaxSlots = 32;
constexpr int kWalkLdsLimit = 160 * 1024;
constexpr int kWalkBufferWord3 = 0x00020000;  // raw buffer resource, 32-bit data
constexpr uint32_t kWalkOutOfRange = 0x80000000u;
constexpr int kPhaseSteps = 4;  // 64-byte k-steps per phase
#define SHC_WALK_LDS __attribute__((address_space(3)))

typedef __bf16 walk_bf16x4 __attribute__((__vector_size__(4 * sizeof(__bf16))));
typedef __bf16 walk_bf16x2 __attribute__((ext_vector_type(2)));
typedef float walk_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t walk_v4u32 __attribute__((ext_vector_type(4)));
typedef uint32_t walk_v2u32 __attribute__((ext_vector_type(2)));

// weight row in LDS: fp32 rows padded by 16 bytes (the four rows a lane group
// apart then start 16 banks apart); bf16 rows unpadded, 32-byte chunks swizzled
// (split fp32: three bf16 planes)
__host__ __device__ constexpr int walk_wrow(bool bf16, bool split, int bn) {
  return bf16 || split ? bn * 2 : bn * 4 + 16;
}
__host__ __device__ constexpr int walk_wbuf(bool bf16, bool split, int bn) {
  return (split ? 3 : 1) * kPhaseSteps * (bf16 ? 32 : 16) * walk_wrow(bf16, split, bn);
}
// index area (words): srcs [K][R]; sorted: srcs_in [K][R], perm [R], cnt [K],
// hist [K + 2]; blkmask [R / 16]
__host__ __device__ constexpr int walk_idx_bytes(int K, int R, bool sorted) {
  return 4 * (K * R + R / 16 + (sorted ? K * R + R + 2 * K + 2 : 0));
}

// A pair of fp32 values times 2^24 as three bf16 pairs, 2^24 x = h + m + l
// exactly: each term is the nearest bf16 to what is left, 8 + 8 + 8 significand
// bits.  The last bit of the smallest fp32 number is 2^-149, so scaled every
// nonzero term is a normal bf16 number.  Values of 2^104 and more, infinities
// and NaN leave a term that is not finite.
constexpr float kSplitScale = 0x1p24f;
__device__ __forceinline__ void split3(walk_v2u32 x, uint32_t* h, uint32_t* m, uint32_t* l) {
  const float x0 = __uint_as_float(x[0]) * kSplitScale, x1 = __uint_as_float(x[1]) * kSplitScale;
  const uint32_t hh = __builtin_bit_cast(
      uint32_t, __builtin_convertvector(walk_f32x2{x0, x1}, walk_bf16x2));
  const float r0 = x0 - __uint_as_float(hh << 16), r1 = x1 - __uint_as_float(hh & 0xFFFF0000u);
  const uint32_t mm = __builtin_bit_cast(
      uint32_t, __builtin_convertvector(walk_f32x2{r0, r1}, walk_bf16x2));
  const float s0 = r0 - __uint_as_float(mm << 16), s1 = r1 - __uint_as_float(mm & 0xFFFF0000u);
  *h = hh;
  *m = mm;
  *l = __builtin_bit_cast(uint32_t,
                          __builtin_convertvector(walk_f32x2{s0, s1}, walk_bf16x2));
}

// NA: register sets of input rows (NA - 1 phases in flight); NWS: register
// sets of weights; MINW: wavefronts per SIMD that the registers must allow.
template <bool BF16, int RW, int CW, int NCT, int NA, int NWS, int MINW, bool SPLIT>
__global__ __launch_bounds__(64 * RW * CW, MINW) void conv_walk_kernel(GemmArgs a) {
  constexpr int NT = 64 * RW * CW;
  constexpr int E = BF16 ? 2 : 4;
  constexpr int VE = 16 / E;                 // elements per 16 bytes
  constexpr int KSTEP = 64 / E;
  constexpr int KC = kPhaseSteps * KSTEP;    // reduction entries per phase
  constexpr int R = RW * 16;
  constexpr int BN = CW * NCT * 16;
  constexpr int WROW = walk_wrow(BF16, SPLIT, BN);
  constexpr int WBUF = walk_wbuf(BF16, SPLIT, BN);
  constexpr int WPL = KC * WROW;             // a plane of the split weights
  static_assert(!SPLIT || (!BF16 && R >= 64), "the split is of fp32, in sorted workgroups");
  constexpr int VPR = BN * E / 16;
  constexpr int NWV = KC * VPR / NT;         // weight vectors per thread and phase
  static_assert(KC * VPR % NT == 0, "whole weight vectors per thread");
  constexpr bool SORT = R >= 64;
  // fp32: P tiles interleave their columns (entry q of tile ct is column
  // P q + ct of the P tiles' 16 P), so one LDS read gives a lane its weights
  // of P tiles and it ends with 4 P consecutive columns of its row
  constexpr int P = BF16 || SPLIT ? 1 : (NCT < 4 ? NCT : 4);
  typedef float WVec __attribute__((ext_vector_type(P == 1 ? 2 : P)));  // (P = 1: scalar reads)

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int K = a.K;
  int32_t* srcs = reinterpret_cast<int32_t*>(smem + 2 * WBUF);        // [K][R] by position
  uint32_t* blkmask = reinterpret_cast<uint32_t*>(srcs + K * R);      // [R / 16]
  int32_t* srcs_in = reinterpret_cast<int32_t*>(blkmask + R / 16);    // [K][R] by row
  int32_t* perm = srcs_in + K * R;                                    // [R] position -> row
  int32_t* cnt = perm + R;                                            // [K]
  int32_t* hist = cnt + K;                                            // [K + 2]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = wave / CW;
  const int wc = wave % CW;
  const int g = lane >> 4;
  const int l16 = lane & 15;
  const int64_t n = a.n_rows;
  const int Cin = a.Cin, Cout = a.Cout;
  const int Ktot = K * Cin;
  const int nks = (Ktot + KSTEP - 1) / KSTEP;
  const int nph = (nks + kPhaseSteps - 1) / kPhaseSteps;
  const int n0 = blockIdx.y * BN;

  const int64_t row0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * R;
  const int nrows = (int)min((int64_t)R, n - row0);

  // ---- weights of a phase: global -> registers -> LDS.  Rows past K Cin and
  // columns past Cout read zeros (an offset past the buffer).
  const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.W), (short)0, (int)((int64_t)Ktot * Cout * E), kWalkBufferWord3);
  auto load_w = [&](int p, i32x4 (&wv)[NWV]) {
#pragma unroll
    for (int u = 0; u < NWV; ++u) {
      const int v = u * NT + tid;
      const int k = p * KC + v / VPR;
      const int c = n0 + (v % VPR) * VE;
      const uint32_t off = (k < Ktot && c < Cout)
                               ? ((uint32_t)k * (uint32_t)Cout + (uint32_t)c) * E
                               : kWalkOutOfRange;
      wv[u] = __builtin_bit_cast(i32x4,
                                 __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off, 0, 0));
    }
  };
  // bf16: the 32-byte column chunk c of row r sits at c ^ swz_row(r), which
  // puts the rows a transposing read touches on different bank groups
  auto swz_row = [](int r) -> int {
    if constexpr (BN >= 128) return (r & 3) | (((r >> 3) & 1) << 2);
    else if constexpr (BN >= 64) return ((r >> 1) & 1) | (((r >> 3) & 1) << 1);
    else return ((r >> 1) ^ (r >> 3)) & 1;
  };
  auto store_w = [&](int buf, const i32x4 (&wv)[NWV]) {
    unsigned char* base = smem + buf * WBUF;
#pragma unroll
    for (int u = 0; u < NWV; ++u) {
      const int v = u * NT + tid;
      const int k = v / VPR;
      const int q = v % VPR;
      if constexpr (SPLIT) {
        // columns 4q .. 4q + 3 of row k, 8 bytes in each plane
        const int col = (((q >> 2) ^ swz_row(k)) << 5) + ((q & 3) << 3);
        const walk_v2u32 x = {(uint32_t)wv[u][0], (uint32_t)wv[u][1]};
        const walk_v2u32 y = {(uint32_t)wv[u][2], (uint32_t)wv[u][3]};
        uint32_t h0, m0, l0, h1, m1, l1;
        split3(x, &h0, &m0, &l0);
        split3(y, &h1, &m1, &l1);
        unsigned char* p = base + k * WROW + col;
        *reinterpret_cast<walk_v2u32*>(p) = walk_v2u32{h0, h1};
        *reinterpret_cast<walk_v2u32*>(p + WPL) = walk_v2u32{m0, m1};
        *reinterpret_cast<walk_v2u32*>(p + 2 * WPL) = walk_v2u32{l0, l1};
      } else {
        const int col = BF16 ? (((q >> 1) ^ swz_row(k)) << 5) + ((q & 1) << 4) : q * 16;
        *reinterpret_cast<i32x4*>(base + k * WROW + col) = wv[u];
      }
    }
  };
  i32x4 wreg[NWS][NWV];
#pragma unroll
  for (int s = 0; s < NWS; ++s) load_w(s, wreg[s]);

  // ---- index lists ------------------------------------------------------------
  if (tid < R / 16) blkmask[tid] = 0;
  if constexpr (SORT) {
    for (int q = tid; q < 2 * K + 2; q += NT) cnt[q] = 0;  // cnt and hist
  }
  __syncthreads();
  const int KR = K * R;
  int32_t* first = SORT ? srcs_in : srcs;
  constexpr int EB = 4;  // entries per thread in flight
  for (int e0 = 0; e0 < KR; e0 += EB * NT) {
    int32_t s[EB];
    bool in[EB];
#pragma unroll
    for (int u = 0; u < EB; ++u) in[u] = e0 + u * NT + tid < KR && (e0 + u * NT + tid) % R < nrows;
    if (a.table != nullptr) {
#pragma unroll
      for (int u = 0; u < EB; ++u) {
        const int e = in[u] ? e0 + u * NT + tid : 0;
        s[u] = a.table[(int64_t)(e / R) * n + row0 + e % R];
      }
    } else {
      int2 c[EB];
#pragma unroll
      for (int u = 0; u < EB; ++u)
        c[u] = reinterpret_cast<const int2*>(a.coords)[row0 + (in[u] ? (e0 + u * NT + tid) % R : 0)];
      int32_t nb[EB];
#pragma unroll
      for (int u = 0; u < EB; ++u) {
        in[u] = in[u] && c[u].x >= 0 && c[u].x < a.B && c[u].y >= 0 && c[u].y < a.V;
        nb[u] = a.nbr[in[u] ? (int64_t)c[u].y * K + (e0 + u * NT + tid) / R : 0];
      }
#pragma unroll
      for (int u = 0; u < EB; ++u) {
        in[u] = in[u] && nb[u] >= 0 && nb[u] < a.V;
        s[u] = a.inv[in[u] ? (int64_t)c[u].x * a.V + nb[u] : 0];
      }
    }
#pragma unroll
    for (int u = 0; u < EB; ++u) {
      const int e = e0 + u * NT + tid;
      const bool ok = in[u] && s[u] >= 0 && (int64_t)s[u] < n;
      const uint64_t bal = __ballot(ok);
      if (e < KR) {
        first[e] = ok ? s[u] : -1;
        if constexpr (SORT) {
          if (lane == 0 && bal != 0) atomicAdd(&cnt[e / R], __popcll(bal));
        } else {
          // 16 consecutive entries share a slot and a block
          if (l16 == 0 && ((bal >> (lane & 48)) & 0xFFFFu) != 0) atomicOr(&blkmask[(e % R) / 16], 1u << (e / R));
        }
      }
    }
  }
  if constexpr (SORT) {
    __syncthreads();
    // (a row's sums are its own, wherever it is placed)
    sort_by_first_slot<R, NT>(K, nrows, srcs_in, cnt, hist, srcs, perm,
                              [&](int pos, uint32_t slots) {
                                if (slots) atomicOr(&blkmask[pos >> 4], slots);
                              });
  }
  store_w(0, wreg[0]);
  load_w(NWS, wreg[0]);
  __syncthreads();

  // ---- this wavefront's blocks --------------------------------------------------
  const uint32_t all = __builtin_amdgcn_readfirstlane(blkmask[wr]);
  const __amdgpu_buffer_rsrc_t s_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.S), (short)0, (int)(n * Cin * E), kWalkBufferWord3);
  // slot of reduction entry kk by multiply-high (exact: kk Cin < 2^32)
  const uint32_t magic = a.cin_magic;
  auto slot_of = [&](int kk) -> int { return (int)__umulhi((uint32_t)kk, magic); };
  // byte offsets of this lane's vectors of phase p (LDS reads of the rows'
  // slots), and the loads themselves, a phase apart
  auto offsets = [&](int p, uint32_t (&off)[kPhaseSteps]) {
    int32_t src[kPhaseSteps];
    uint32_t c[kPhaseSteps];
    bool in[kPhaseSteps];
#pragma unroll
    for (int ks = 0; ks < kPhaseSteps; ++ks) {
      const int kk = p * KC + ks * KSTEP + g * VE;
      in[ks] = kk < Ktot;
      const int j = in[ks] ? slot_of(kk) : 0;
      c[ks] = (uint32_t)(kk - j * Cin);
      src[ks] = srcs[j * R + wr * 16 + l16];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < kPhaseSteps; ++ks)
      off[ks] = (in[ks] && src[ks] >= 0)
                    ? ((uint32_t)src[ks] * (uint32_t)Cin + c[ks]) * (uint32_t)E
                    : kWalkOutOfRange;
  };
  auto issue_a = [&](const uint32_t (&off)[kPhaseSteps], i32x4 (&dst)[kPhaseSteps]) {
#pragma unroll
    for (int ks = 0; ks < kPhaseSteps; ++ks)
      dst[ks] = __builtin_bit_cast(
          i32x4, __builtin_amdgcn_raw_buffer_load_b128(s_rsrc, off[ks], 0, 0));
  };

  // column of accumulator entry r of tile ct: a lane's entries of P tiles are
  // 4 P consecutive columns
  const int cbase = n0 + wc * NCT * 16 + 4 * P * g;
  auto col_of = [&](int ct, int r) -> int { return cbase + (ct / P) * 16 * P + P * r + ct % P; };
  // accumulators start at the bias of their columns (row l16 of a block), the
  // split's at zero: its bias joins where the two sums do
  f32x4 acc[NCT], low[SPLIT ? NCT : 1];
  auto bias_of = [&](int ct) -> f32x4 {
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (a.bias != nullptr) {
#pragma unroll
      for (int r = 0; r < 4; ++r) b[r] = col_of(ct, r) < Cout ? a.bias[col_of(ct, r)] : 0.f;
    }
    return b;
  };
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    if constexpr (SPLIT) acc[ct] = low[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    else acc[ct] = bias_of(ct);
  }

  i32x4 areg[NA][kPhaseSteps];
  uint32_t off[kPhaseSteps];  // of the phase whose loads go out next
#pragma unroll
  for (int s = 0; s < NA - 1; ++s) {
    offsets(s, off);
    issue_a(off, areg[s]);
  }
  offsets(NA - 1, off);

  // weight fragments of one k-step: bf16, two transposing reads per tile give
  // lane (g, i) entries 8g .. 8g+7 of column i; fp32, entries 4g .. 4g+3
  const int swz = swz_row(8 * g + (l16 >> 2));
  struct WFrag {
    i32x4 v[NCT];
  };
  auto read_w = [&](const unsigned char* base, int ks, WFrag& f) {
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      if constexpr (BF16) {
        const unsigned char* p0 = base + (ks * 32 + 8 * g + (l16 >> 2)) * WROW +
                                  (((wc * NCT + ct) ^ swz) << 5) + 8 * (l16 & 3);
        const walk_bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (SHC_WALK_LDS walk_bf16x4*)(const_cast<unsigned char*>(p0)));
        const walk_bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (SHC_WALK_LDS walk_bf16x4*)(const_cast<unsigned char*>(p0 + 4 * WROW)));
        const bf16x8 w = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        f.v[ct] = __builtin_bit_cast(i32x4, w);
      } else if constexpr (P == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          f.v[ct][i] = *reinterpret_cast<const int*>(base + (ks * 16 + 4 * g + i) * WROW +
                                                     ((wc * NCT + ct) * 16 + l16) * 4);
      } else if (ct % P == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const WVec w = *reinterpret_cast<const WVec*>(
              base + (ks * 16 + 4 * g + i) * WROW + ((wc * NCT + ct) * 16 + P * l16) * 4);
#pragma unroll
          for (int q = 0; q < P; ++q) f.v[ct + q][i] = __float_as_int(w[q]);
        }
      }
    }
  };
  // split weights: the three planes of column tile ct of the 32-entry k-step
  // m, entries 4g .. 4g+3 of both its halves for column i
  struct WPlanes {
    i32x4 v[3];
  };
  auto read_planes = [&](const unsigned char* base, int m, int ct, WPlanes& f) {
    const int r = 32 * m + 4 * g + (l16 >> 2);
    const int sw = swz_row(4 * g + (l16 >> 2));
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) {
      const unsigned char* p0 =
          base + pl * WPL + r * WROW + (((wc * NCT + ct) ^ sw) << 5) + 8 * (l16 & 3);
      const walk_bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (SHC_WALK_LDS walk_bf16x4*)(const_cast<unsigned char*>(p0)));
      const walk_bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (SHC_WALK_LDS walk_bf16x4*)(const_cast<unsigned char*>(p0 + 16 * WROW)));
      const bf16x8 w = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      f.v[pl] = __builtin_bit_cast(i32x4, w);
    }
  };
  auto phase = [&](int p, i32x4 (&cur)[kPhaseSteps], i32x4 (&ahead)[kPhaseSteps],
                   i32x4 (&wv)[NWV]) {
    // phase p's weights were stored before this barrier; every wavefront is
    // done with phase p - 1, whose buffer takes phase p + 1's
    __syncthreads();
    const unsigned char* base = smem + (p & 1) * WBUF;
    // the slots of the phase; a wavefront none of whose rows has one skips it
    uint32_t bits = 0;
    if (p < nph) {
      const int lo = slot_of(p * KC), hi = slot_of(min((p + 1) * KC, Ktot) - 1);
      bits = ((2u << hi) - 1u) & ~((1u << lo) - 1u);
    }
    const bool live = (all & bits) != 0u;
    WFrag wf[2];
    WPlanes wp[2];
    if (live) {
      if constexpr (SPLIT) read_planes(base, 0, 0, wp[0]);
      else read_w(base, 0, wf[0]);
    }
    issue_a(off, ahead);
    store_w((p + 1) & 1, wv);
    load_w(p + 1 + NWS, wv);
    offsets(p + NA, off);
    if (!live) return;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SPLIT) {
      // two k-steps of 32 entries; lane group g holds entries 4g .. 4g+3 of
      // each of their two 16-entry halves
      bf16x8 at[3];
#pragma unroll
      for (int st = 0; st < 2 * NCT; ++st) {
        const int m = st / NCT, ct = st % NCT;
        if (ct == 0) {
          walk_v4u32 t[3];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const i32x4& v = cur[2 * m + q / 2];
            const walk_v2u32 x = {(uint32_t)v[2 * (q & 1)], (uint32_t)v[2 * (q & 1) + 1]};
            uint32_t h, mm, l;
            split3(x, &h, &mm, &l);
            t[0][q] = h;
            t[1][q] = mm;
            t[2][q] = l;
          }
#pragma unroll
          for (int q = 0; q < 3; ++q) at[q] = __builtin_bit_cast(bf16x8, t[q]);
        }
        if (st + 1 < 2 * NCT)
          read_planes(base, (st + 1) / NCT, (st + 1) % NCT, wp[(st + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        auto mul = [&](int pl, int q, f32x4& sum) {
          sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, wp[st & 1].v[pl]), at[q], sum, 0, 0, 0);
        };
        mul(2, 0, low[ct]);
        mul(0, 2, low[ct]);
        mul(1, 1, low[ct]);
        mul(1, 0, low[ct]);
        mul(0, 1, low[ct]);
        mul(0, 0, acc[ct]);
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
#pragma unroll
    for (int ks = 0; ks < kPhaseSteps; ++ks) {
      if (ks + 1 < kPhaseSteps) read_w(base, ks + 1, wf[(ks + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (BF16) {
        const bf16x8 af = __builtin_bit_cast(bf16x8, cur[ks]);
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
          acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, wf[ks & 1].v[ct]), af, acc[ct], 0, 0, 0);
      } else {  // MFMA i contracts entry 4g + i of every lane group
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct)
            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                __int_as_float(wf[ks & 1].v[ct][i]), __int_as_float(cur[ks][i]), acc[ct], 0, 0,
                0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // register sets: phase p multiplies rows p % NA and stores weights
  // (p + 1) % NWS; whole trips of U phases (phases past the end do nothing)
  constexpr int U = NA % NWS == 0 ? NA : (NWS % NA == 0 ? NWS : NA * NWS);
  for (int p0 = 0; p0 < nph; p0 += U) {
#pragma unroll
    for (int q = 0; q < U; ++q)
      phase(p0 + q, areg[q % NA], areg[(q + NA - 1) % NA], wreg[(q + 1) % NWS]);
  }

  // The last MFMAs may sit right behind a branch; their results are read at
  // least 32 wait states later (an fp32 16x16x4 needs 18).
  auto mfma_wait = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (SPLIT) {
    // the two sums and the bias, rounded once; sums that are not finite (values
    // past the split's range, or sums near fp32's largest number times 2^-48)
    // are the fp32 matrix cores' to form
    mfma_wait();
    bool finite = true;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const f32x4 b = bias_of(ct);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        finite = finite && fabsf(acc[ct][i]) + fabsf(low[ct][i]) < __builtin_inff();
        acc[ct][i] = (float)(((double)acc[ct][i] + (double)low[ct][i]) *
                                 (1.0 / ((double)kSplitScale * kSplitScale)) +
                             (double)b[i]);
      }
    }
    // row l16's columns are in its four lane groups: all of them or none
    int out_of_range = finite ? 0 : 1;
    out_of_range |= __shfl_xor(out_of_range, 16, 64);
    out_of_range |= __shfl_xor(out_of_range, 32, 64);
    const bool redo = out_of_range != 0;
    if (__ballot(redo) != 0) {
      // the wavefront's rows again on the fp32 matrix cores, straight from memory
      f32x4 kept[NCT];
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        kept[ct] = acc[ct];
        acc[ct] = bias_of(ct);
      }
#pragma unroll 1
      for (int s = 0; s < nks; ++s) {
        const int lo = slot_of(s * KSTEP), hi = slot_of(min((s + 1) * KSTEP, Ktot) - 1);
        if ((all & ((2u << hi) - 1u) & ~((1u << lo) - 1u)) == 0u) continue;
        const int kk = s * KSTEP + 4 * g;
        const int j = kk < Ktot ? slot_of(kk) : 0;
        const int32_t src = srcs[j * R + wr * 16 + l16];
        const uint32_t aoff = (kk < Ktot && src >= 0)
                                  ? ((uint32_t)src * (uint32_t)Cin + (uint32_t)(kk - j * Cin)) * E
                                  : kWalkOutOfRange;
        const i32x4 v = __builtin_bit_cast(
            i32x4, __builtin_amdgcn_raw_buffer_load_b128(s_rsrc, aoff, 0, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) {
            const int c = n0 + (wc * NCT + ct) * 16 + l16;
            const uint32_t woff = (kk + i < Ktot && c < Cout)
                                      ? ((uint32_t)(kk + i) * (uint32_t)Cout + (uint32_t)c) * E
                                      : kWalkOutOfRange;
            const int w = __builtin_amdgcn_raw_buffer_load_b32(w_rsrc, woff, 0, 0);
            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(w),
                                                           __int_as_float(v[i]), acc[ct], 0, 0, 0);
          }
        }
      }
      mfma_wait();
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[ct][i] = redo ? acc[ct][i] : kept[ct][i];
    }
  }

  // ---- epilogue: activation, rounding, four columns of a row per store ---------
  mfma_wait();
  const bool relu = a.relu != 0;
  const __amdgpu_buffer_rsrc_t o_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      a.out, (short)0, (int)(n * Cout * E), kWalkBufferWord3);
  const int pos = wr * 16 + l16;
  const int r = SORT ? perm[pos] : pos;
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    // vector ct % P of the 4 P columns of tiles ct / P * P ..: entries
    // 4 (ct % P) + i of them
    const int c0 = ct / P * P;
    const int col = col_of(c0, 0) + 4 * (ct % P);
    const uint32_t off = (r < nrows && col < Cout)
                             ? ((uint32_t)(row0 + r) * (uint32_t)Cout + (uint32_t)col) * E
                             : kWalkOutOfRange;
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = 4 * (ct % P) + i;
      const float x = acc[c0 + q % P][q / P];
      const float rx = x > 0.f ? x : 0.f;
      v[i] = relu ? rx : x;
    }
    if constexpr (BF16) {  // round to nearest even
      const walk_bf16x2 h0 = __builtin_convertvector(walk_f32x2{v[0], v[1]}, walk_bf16x2);
      const walk_bf16x2 h1 = __builtin_convertvector(walk_f32x2{v[2], v[3]}, walk_bf16x2);
      const walk_v2u32 o = {__builtin_bit_cast(uint32_t, h0), __builtin_bit_cast(uint32_t, h1)};
      __builtin_amdgcn_raw_buffer_store_b64(o, o_rsrc, off, 0, 0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(walk_v4u32, v), o_rsrc, off, 0,
                                             0);
    }
  }
}

template <bool BF16, int RW, int CW, int NCT, int NA, int NWS, int MINW, bool SPLIT = false>
hipError_t launch_walk(const GemmArgs& a, hipStream_t stream) {
  constexpr int R = RW * 16, BN = CW * NCT * 16;
  auto kern = conv_walk_kernel<BF16, RW, CW, NCT, NA, NWS, MINW, SPLIT>;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, kWalkLdsLimit);
  });
  if (attr_err != hipSuccess) return attr_err;
  const size_t lds =
      2 * walk_wbuf(BF16, SPLIT, BN) + walk_idx_bytes(a.K, R, R >= 64);
  const dim3 grid((unsigned)((a.n_rows + R - 1) / R), (unsigned)((a.Cout + BN - 1) / BN));
  hipLaunchKernelGGL(kern, grid, dim3(64 * RW * CW), lds, stream, a);
  return hipGetLastError();
}

// Workgroups of 16 rows x 64 columns while the chip holds them at once, else
// 128 x 32 while two to a CU hold them, else 128 x 64: fp32 64 -> 64 at 3,930
// rows 12.4 / 16.3 / 23.9 us, at 7,926 rows 17.4 / 17.0 / 24.2; 128 -> 128 at
// 15,851 rows (992 workgroups of 128 x 32) 96 / 41.6 / 42.1, at 32,000 rows
// 183 / 90 / 80; bf16 256 -> 256 at 7,926 rows 71 / 24.8 / 20.5.
// The split's 128-row workgroups run two to a CU; 256 rows in 16 wavefronts
// stage the weights half as often and win while one round of them covers the
// rows (128 -> 128 at 32,000 rows 53 against 59 us; at 67,040 sparse rows 117
// against 105 the other way).
template <bool BF16>
hipError_t launch_walk_rows(const GemmArgs& a, bool split, int num_cus, hipStream_t stream) {
  if (conv_walk_small(a, num_cus))
    return launch_walk<BF16, 1, 4, 1, 4, 4, 1>(a, stream);
  if (conv_walk_medium(a, num_cus, 2)) return launch_walk<BF16, 8, 1, 2, 2, 2, 4>(a, stream);
  if constexpr (!BF16) {
    if (split && ((a.n_rows + 255) / 256) * ((a.Cout + 63) / 64) <= num_cus)
      return launch_walk<false, 16, 1, 4, 2, 1, 4, true>(a, stream);
    if (split) return launch_walk<false, 8, 1, 4, 2, 1, 4, true>(a, stream);
  }
  return launch_walk<BF16, 8, 1, 4, 2, 1, 4>(a, stream);
}

}  // namespace

bool conv_walk_supported(const GemmArgs& a, bool bf16) {
  const int e = bf16 ? 2 : 4;
  if (a.plan != nullptr || a.plan_out != nullptr) return false;
  if (a.K < 1 || a.K > kWalkMaxSlots) return false;
  // 32-bit buffer offsets
  return a.n_rows * a.Cin * e <= 0x7FFF0000LL && a.n_rows * a.Cout * e <= 0x7FFF0000LL &&
         (int64_t)a.K * a.Cin * a.Cout * e <= 0x7FFF0000LL;
}

hipError_t launch_conv_walk(const GemmArgs& a_in, bool bf16, bool split, int num_cus,
                            hipStream_t stream) {
  GemmArgs a = a_in;
  a.cin_magic = (uint32_t)(((1ull << 32) + (uint64_t)a.Cin - 1) / (uint64_t)a.Cin);
  return bf16 ? launch_walk_rows<true>(a, split, num_cus, stream)
              : launch_walk_rows<false>(a, split, num_cus, stream);
}

}  // namespace shc
