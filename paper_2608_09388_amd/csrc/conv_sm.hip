// Sparse neighbourhood convolution from a neighbour-row table (Eqs. 4-5,
// with the activation of Eq. 10), bf16, slot-major:
//
//   out[i] = act( bias + sum_{j<K} S[table[j][i]] W[j] ),  absent entries add 0.
//
// A workgroup owns 128, 192 or 320 consecutive active rows and every output
// column.  It walks the slots in order: the weights of slot j (Cin x Cout)
// sit in LDS while every wavefront multiplies its rows' slot-j neighbour rows
// by them, and slot j + 1's weights are loaded beside that work into the
// other of two buffers; the neighbour rows of slot j + 1 are in flight in
// registers meanwhile.  Each gathered row therefore feeds all Cout columns at
// once.  Rows are sorted by their first sparse slot, and a (16-row block,
// slot) pair with no present row is skipped.  Accumulation is in fp32, per
// output element in slot order and within a slot in k order.
//
// What bounds it: a slot's weight reads from LDS and its MFMAs take about as
// long each, and the table reads, the sort and the output around the slots
// would stand beside neither.  So a workgroup takes half a CU's LDS or less
// (the output staged where the weights were) and two or more share a CU, one's
// slots under another's ends; with one of 256 rows a CU those ends were 59 of
// 273 us (670,464 rows at half density, 128 -> 128 channels, nine slots; 257
// us with two of 128 rows, 220 with two of 192).  At 600,000 rows, half dense:
// 64 -> 128 149 -> 130 us, 128 -> 64 170 -> 136; seven slots 128 -> 128 278 ->
// 179.  On sparse masks the weights of every slot, loaded per workgroup, are
// the larger part (launch_sm_rows).  Each XCD takes a contiguous run of rows:
// 281 against 275 us.  A read of the weights half a k-step ahead of the MFMAs,
// or two slots of rows in flight instead of one, is slower (262 and 264
// against 257 us, 128 rows).
#include <hip/hip_runtime.h>

#include <mutex>

#include "shc_internal.h"

namespace shc {
namespace {

constexpr int kSmMaxSlots = 32;
constexpr int kSmLdsLimit = 160 * 1024;
constexpr int kSmBufferWord3 = 0x00020000;  // raw buffer resource, 32-bit data
constexpr uint32_t kSmOutOfRange = 0x80000000u;
#define SHC_SM_LDS __attribute__((address_space(3)))

typedef __bf16 sm_bf16x4 __attribute__((__vector_size__(4 * sizeof(__bf16))));
typedef __bf16 sm_bf16x2 __attribute__((ext_vector_type(2)));
typedef float sm_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t sm_v4u32 __attribute__((ext_vector_type(4)));

// LDS: two weight buffers [Cin][Cout] bf16 (32-byte column chunks XOR-
// swizzled by row), which the epilogue's staging tiles [16][Cout + 8] bf16,
// one per wavefront, replace after the last slot; srcs [K][R] int32 and
// presence bytes [K][R/16].
__host__ __device__ constexpr int sm_wbuf_bytes(int cin, int cout) { return cin * cout * 2; }
__host__ __device__ constexpr int sm_stage_row(int cout) { return cout * 2 + 16; }
// srcs [K][R] in row order, then sorted; perm [R]; per-slot counts and the
// sort's buckets [K + 2]; presence bytes [K][R / 16]
__host__ __device__ inline int sm_idx_bytes(int K, int R) {
  return 4 * (2 * K * R + R + K + K + 2) + ((K * (R / 16) + 15) & ~15) + 16;
}
__host__ __device__ constexpr int sm_work_bytes(int cin, int cout, int nw) {
  return 2 * sm_wbuf_bytes(cin, cout) > nw * 16 * sm_stage_row(cout)
             ? 2 * sm_wbuf_bytes(cin, cout)
             : nw * 16 * sm_stage_row(cout);
}
__host__ __device__ inline int sm_lds_bytes(int cin, int cout, int K, int R, int nw) {
  return sm_work_bytes(cin, cout, nw) + ((sm_idx_bytes(K, R) + 15) & ~15);
}
// Two workgroups of R rows (whichever wavefronts) to a CU
inline bool sm_two_per_cu(int cin, int cout, int K, int R) {
  return sm_lds_bytes(cin, cout, K, R, R / 16) <= kSmLdsLimit / 2;
}

struct SmArgs {
  const void* S;          // [n_rows][Cin] bf16
  const int32_t* table;   // [K][n_rows]
  const void* W;          // [K][Cin][Cout] bf16
  const float* bias;      // [Cout] or null
  void* out;              // [n_rows][Cout] bf16
  int64_t n_rows;
  int32_t K;
  int32_t relu;
};

// KS: 32-wide k-steps (Cin / 32); NCT: 16-column tiles (Cout / 16); NW:
// wavefronts per workgroup; BPW: 16-row blocks per wavefront (R = 16 NW BPW
// rows per workgroup); KF: K fixed at compile time (the slots fully
// unrolled), or 0 for any K (a loop over the slots, whose back edge makes the
// compiler wait for every load in flight); MINW: wavefronts per SIMD the
// registers leave room for; ASETS: register sets of neighbour rows (two: slot
// j + 1's go out ahead of slot j's MFMAs; one: each k-step's registers take
// slot j + 1's as soon as slot j's MFMAs have read them).
template <int KS, int NCT, int NW, int BPW, int KF, int MINW, int ASETS>
__global__ __launch_bounds__(64 * NW, MINW) void conv_sm_kernel(const SmArgs a) {
  constexpr int NT = 64 * NW;
  constexpr int Cin = KS * 32;
  constexpr int Cout = NCT * 16;
  constexpr int R = BPW * 16 * NW;
  constexpr int WROW = Cout * 2;           // weight row bytes in LDS
  constexpr int VPR = WROW / 16;           // 16-byte vectors per weight row
  constexpr int WVEC = Cin * VPR;          // vectors per slot's weights
  constexpr int NWV = WVEC / NT;           // per thread
  static_assert(WVEC % NT == 0, "whole weight vectors per thread");
  static_assert(R % 64 == 0, "a wavefront's 64 consecutive rows share a slot");
  constexpr int SROW = sm_stage_row(Cout);

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int K = KF > 0 ? KF : a.K;
  unsigned char* wbuf = smem;                                             // [2][Cin][WROW]
  int32_t* srcs_in = reinterpret_cast<int32_t*>(smem + sm_work_bytes(Cin, Cout, NW));  // [K][R]
  int32_t* srcs = srcs_in + K * R;        // [K][R], sorted positions
  int32_t* perm = srcs + K * R;           // [R] sorted position -> row
  int32_t* cnt = perm + R;                // [K] rows present per slot
  int32_t* hist = cnt + K;                // [K + 2] bucket counts, then cursors
  uint8_t* pres = reinterpret_cast<uint8_t*>(hist + K + 2);  // [K][R/16]
  unsigned char* stage = smem;             // in place of wbuf, after the last slot

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int g = lane >> 4;
  const int l16 = lane & 15;
  const int64_t n = a.n_rows;
  const int64_t row0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * R;
  const int nrows = (int)min((int64_t)R, n - row0);

  // ---- weights of a slot: global -> registers -> LDS.  The 32-byte column
  // chunk c of weight row r sits at chunk position c ^ swz_row(r): a
  // transposing B read touches rows 8g + i (+4), g < 4, i < 4, and with
  // 256-byte rows (64 banks: every row starts on bank 0) the XOR puts the
  // eight rows of g & 1 and i at eight different banks groups; with 128-byte
  // rows (two rows per bank cycle) two bits of the row do it.
  auto swz_row = [](int r) -> int {
    if constexpr (NCT >= 8) return (r & 3) | (((r >> 3) & 1) << 2);
    else return ((r >> 1) & 1) | (((r >> 3) & 1) << 1);
  };
  const unsigned char* W = static_cast<const unsigned char*>(a.W);
  // slot m's weights are loaded two slots ahead of use and stored one slot
  // ahead (buffer m & 1)
  i32x4 wreg[NWV];
  auto load_w = [&](int j) {
#pragma unroll
    for (int u = 0; u < NWV; ++u) {
      const int v = u * NT + tid;
      wreg[u] = *reinterpret_cast<const i32x4*>(W + ((int64_t)j * Cin * Cout) * 2 + v * 16);
    }
  };
  auto store_w = [&](int buf) {
    unsigned char* base = wbuf + buf * sm_wbuf_bytes(Cin, Cout);
#pragma unroll
    for (int u = 0; u < NWV; ++u) {
      const int v = u * NT + tid;
      const int k = v / VPR;
      const int q = v - k * VPR;
      const int col = (((q >> 1) ^ swz_row(k)) << 5) + ((q & 1) << 4);
      *reinterpret_cast<i32x4*>(base + k * WROW + col) = wreg[u];
    }
  };
  // B fragments of one k-step (rows 32 ks .. 32 ks + 31) from a buffer: two
  // transposing reads per 16 columns give lane (g, i) rows 8g .. 8g+7 of
  // column i; the lane's rows 32 ks + 8g + (i >> 2) and 4 more share one
  // swizzle, a per-lane constant
  const int swz = swz_row(8 * g + (l16 >> 2));
  auto read_b = [&](int buf, int ks, bf16x8* out) {
    const unsigned char* base = wbuf + buf * sm_wbuf_bytes(Cin, Cout) + ks * 32 * WROW;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const unsigned char* p0 =
          base + (8 * g + (l16 >> 2)) * WROW + (((ct ^ swz) << 5) + 8 * (l16 & 3));
      const sm_bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (SHC_SM_LDS sm_bf16x4*)(const_cast<unsigned char*>(p0)));
      const sm_bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (SHC_SM_LDS sm_bf16x4*)(const_cast<unsigned char*>(p0 + 4 * WROW)));
      out[ct] = bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    }
  };

  // ---- prologue: slot 0's weights on their way, then the table entries
  load_w(0);
  for (int q = tid; q < 2 * K + 2; q += NT) cnt[q] = 0;  // cnt and hist
  __syncthreads();
  // entries (j, t) = (e / R, e % R): a wavefront reads 64 consecutive rows of
  // one slot, coalesced, eight entries per thread in flight
  const int KR = K * R;
  for (int e0 = 0; e0 < KR; e0 += 8 * NT) {
    int32_t s[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + u * NT + tid;
      const int j = e / R, t = e - (e / R) * R;
      s[u] = (e < KR && t < nrows) ? a.table[(int64_t)j * n + row0 + t] : -1;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + u * NT + tid;
      const bool ok = (uint32_t)s[u] < (uint32_t)n;  // 0 <= s < n
      const int c = __popcll(__ballot(ok));
      if (e < KR) {
        srcs_in[e] = ok ? s[u] : -1;
        if (lane == 0 && c > 0) atomicAdd(&cnt[e / R], c);
      }
    }
  }
  __syncthreads();
  // (every row's sum runs over its own slots in order, wherever it is placed)
  sort_by_first_slot<R, NT>(K, nrows, srcs_in, cnt, hist, srcs, perm, [](int, uint32_t) {});
  __syncthreads();
  // presence of each (slot, sorted 16-row block)
  for (int e = tid; e < KR; e += NT) {
    const uint64_t bal = __ballot(srcs[e] >= 0);
    if (l16 == 0) pres[(e / R) * (R / 16) + (e % R) / 16] = ((bal >> (lane & 48)) & 0xFFFFu) != 0;
  }
  store_w(0);
  __syncthreads();

  // ---- neighbour rows of a slot for this wavefront's blocks: raw buffer
  // loads, an absent row reading zeros without touching memory
  const __amdgpu_buffer_rsrc_t s_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.S), (short)0, (int)(n * Cin * 2), kSmBufferWord3);
  i32x4 areg[ASETS][BPW][KS];
  auto offsets = [&](int j, uint32_t (&off)[BPW]) {
#pragma unroll
    for (int u = 0; u < BPW; ++u) {
      const int32_t src = j < K ? srcs[j * R + (wave * BPW + u) * 16 + l16] : -1;
      off[u] = src >= 0 ? (uint32_t)src * (uint32_t)(Cin * 2) + (uint32_t)g * 16u : kSmOutOfRange;
    }
  };
  auto load_a = [&](uint32_t off, int ks) -> i32x4 {
    return __builtin_bit_cast(
        i32x4, __builtin_amdgcn_raw_buffer_load_b128(
                   s_rsrc, off != kSmOutOfRange ? off + (uint32_t)ks * 64u : kSmOutOfRange, 0, 0));
  };
  auto issue_a = [&](int j, i32x4 (&dst)[BPW][KS]) {
    uint32_t off[BPW];
    offsets(j, off);
#pragma unroll
    for (int u = 0; u < BPW; ++u)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) dst[u][ks] = load_a(off[u], ks);
  };

  // accumulators start at the bias of their column
  f32x4 acc[BPW][NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    const float b = a.bias != nullptr ? a.bias[ct * 16 + l16] : 0.f;
#pragma unroll
    for (int u = 0; u < BPW; ++u) acc[u][ct] = f32x4{b, b, b, b};
  }

  // loads go out in the loop's own order (weights of slot m + 2 beside the
  // rows of slot m + 1), so that every slot's waits count the same loads
  issue_a(0, areg[0]);
  load_w(K > 1 ? 1 : K - 1);

  // ---- the slots, in order; register set j % ASETS, weight buffer j % 2
  auto slot = [&](int j, i32x4 (&cur)[BPW][KS], i32x4 (&ahead)[BPW][KS]) {
    // slot j's weights were stored before this barrier; every wavefront is
    // done with slot j - 1, so its buffer takes slot j + 1's, and their
    // registers slot j + 2's.  Past the last slot the weights of slot K - 1
    // are loaded and stored again, into a buffer no slot reads any more, so
    // that every slot issues the same loads.
    __syncthreads();
    store_w((j + 1) & 1);
    load_w(j + 2 < K ? j + 2 : K - 1);
    uint32_t off[BPW];
    if constexpr (ASETS == 2) issue_a(j + 1, ahead);
    else offsets(j + 1, off);
    bool live[BPW];
    bool any = false;
#pragma unroll
    for (int u = 0; u < BPW; ++u) {
      live[u] = pres[j * (R / 16) + wave * BPW + u] != 0;
      any = any || live[u];
    }
    // a wavefront none of whose rows has slot j reads no weights either
    if (ASETS == 2 && !any) return;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (any) {
        bf16x8 bfr[NCT];
        read_b(j & 1, ks, bfr);
#pragma unroll
        for (int u = 0; u < BPW; ++u) {
          if (!live[u]) continue;
          const bf16x8 af = __builtin_bit_cast(bf16x8, cur[u][ks]);
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct)
            acc[u][ct] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bfr[ct], acc[u][ct], 0, 0, 0);
        }
      }
      if constexpr (ASETS == 1)
#pragma unroll
        for (int u = 0; u < BPW; ++u) cur[u][ks] = load_a(off[u], ks);
    }
  };
  if constexpr (KF > 0) {
#pragma unroll
    for (int j = 0; j < KF; ++j) slot(j, areg[j % ASETS], areg[(j + 1) % ASETS]);
  } else {
    for (int j0 = 0; j0 < K; j0 += 2) {
      slot(j0, areg[0], areg[1 % ASETS]);
      if (j0 + 1 < K) slot(j0 + 1, areg[1 % ASETS], areg[0]);
    }
  }
  __syncthreads();  // the staging tiles take the weights' place

  // ---- epilogue: act, bf16 (round to nearest even), staged per wavefront
  // so that every lane stores 16 contiguous bytes of a row
  __builtin_amdgcn_sched_barrier(0);
  const bool relu = a.relu != 0;
  unsigned char* my_stage = stage + wave * 16 * SROW;
  const __amdgpu_buffer_rsrc_t o_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      a.out, (short)0, (int)(n * Cout * 2), kSmBufferWord3);
#pragma unroll
  for (int u = 0; u < BPW; ++u) {
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float x = acc[u][ct][r];
        const float rx = x > 0.f ? x : 0.f;
        v[r] = relu ? rx : x;
      }
      unsigned char* pp = my_stage + (g * 4) * SROW + (ct * 16 + l16) * 2;
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const sm_bf16x2 h = __builtin_convertvector(sm_f32x2{v[r], v[r + 1]}, sm_bf16x2);
        *reinterpret_cast<__bf16*>(pp + r * SROW) = h[0];
        *reinterpret_cast<__bf16*>(pp + (r + 1) * SROW) = h[1];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    constexpr int NST = 16 * VPR / 64;  // 16-byte stores per lane for the block
    i32x4 sv[NST];
#pragma unroll
    for (int t = 0; t < NST; ++t) {
      const int idx = t * 64 + lane;
      sv[t] = *reinterpret_cast<const i32x4*>(my_stage + (idx / VPR) * SROW + (idx % VPR) * 16);
    }
    int prow[NST];
#pragma unroll
    for (int t = 0; t < NST; ++t) prow[t] = perm[(wave * BPW + u) * 16 + (t * 64 + lane) / VPR];
#pragma unroll
    for (int t = 0; t < NST; ++t) {
      const int idx = t * 64 + lane;
      const int r = prow[t];
      const uint32_t off = r < nrows
                               ? ((uint32_t)(row0 + r) * (uint32_t)Cout + (uint32_t)(idx % VPR) * 8u) * 2u
                               : kSmOutOfRange;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(sm_v4u32, sv[t]), o_rsrc, off, 0,
                                             0);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

template <int KS, int NCT, int NW, int BPW, int KF, int MINW = 2, int ASETS = 2>
hipError_t launch_sm(const SmArgs& a, hipStream_t stream) {
  constexpr int R = BPW * 16 * NW;
  auto kern = conv_sm_kernel<KS, NCT, NW, BPW, KF, MINW, ASETS>;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, kSmLdsLimit);
  });
  if (attr_err != hipSuccess) return attr_err;
  const size_t lds = (size_t)sm_lds_bytes(KS * 32, NCT * 16, a.K, R, NW);
  const unsigned grid = (unsigned)((a.n_rows + R - 1) / R);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * NW), lds, stream, a);
  return hipGetLastError();
}

template <int KS, int NCT, int NW, int BPW, int ASETS = 2>
hipError_t launch_sm_k(const SmArgs& a, hipStream_t stream) {
  // nine slots unrolled: 4 to 10% (236 against 247 us at 600,000 half-dense
  // rows, 128 -> 128)
  return a.K == 9 ? launch_sm<KS, NCT, NW, BPW, 9, 2, ASETS>(a, stream)
                  : launch_sm<KS, NCT, NW, BPW, 0, 2, ASETS>(a, stream);
}

// Two workgroups to a CU's LDS, of 128 rows: eight wavefronts of one block for
// 64 input channels, four of two blocks (a weight fragment read feeds both)
// for 128 -> 64 (64 -> 128: 24 to 30 us with eight at 100,000 rows against 27
// to 31), and for 64 -> 64 past the rows the chip holds at once (300,000 rows,
// seven slots: 37 against 40 us, at 80,000 13 against 14 the other way).
// 128 -> 128 takes 192 rows, four wavefronts of three blocks with one register
// set of rows, up to ten slots, where two fit, and from 500 rows per CU (nine
// slots, 131,000 rows at 5% 45.9 against 43.5 us; ten slots 51.3 against 50.7,
// 100,000 rows 47.2 against 51.2): a third fewer weight bytes from
// L2 (each workgroup reads all of them, 32 KB a slot), which bound its sparse
// masks (nine slots, 258,048 rows at 5% 84.2 us with 128 rows, 75.1 with 192,
// 80.5 with one workgroup of 256 a CU; 600,000 at 50% 232, 197 and 255).  Eleven
// to fourteen slots take 128 rows (192 leave one workgroup a CU: 100,000 rows,
// eleven slots, 50 against 76 us), 15 and more 320 rows: one wavefront per SIMD
// holding five blocks.
template <int KS, int NCT>
hipError_t launch_sm_rows(const SmArgs& a, int num_cus, hipStream_t stream) {
  if constexpr (KS == 4) {
    if constexpr (NCT == 8) {
      if (sm_two_per_cu(KS * 32, NCT * 16, a.K, 192) && a.n_rows >= 500LL * num_cus)
        return launch_sm_k<KS, NCT, 4, 3, 1>(a, stream);
      if (!sm_two_per_cu(KS * 32, NCT * 16, a.K, 128))
        return launch_sm<KS, NCT, 4, 5, 0, 1>(a, stream);
    }
    return launch_sm_k<KS, NCT, 4, 2>(a, stream);
  } else {
    if constexpr (NCT == 4)
      if (a.n_rows > 256LL * num_cus) return launch_sm_k<KS, NCT, 4, 2>(a, stream);
    return launch_sm_k<KS, NCT, 8, 1>(a, stream);
  }
}

}  // namespace

bool conv_sm_supported(const GemmArgs& a, bool bf16) {
  if (!bf16 || a.table == nullptr || a.plan != nullptr || a.plan_out != nullptr || a.gather)
    return false;
  if (a.K < 1 || a.K > kSmMaxSlots) return false;
  if (!((a.Cin == 64 || a.Cin == 128) && (a.Cout == 64 || a.Cout == 128))) return false;
  // 32-bit buffer offsets
  if (a.n_rows * a.Cin * 2 > 0x7FFF0000LL || a.n_rows * a.Cout * 2 > 0x7FFF0000LL) return false;
  return sm_two_per_cu(a.Cin, a.Cout, a.K, 128) ||
         sm_lds_bytes(a.Cin, a.Cout, a.K, 320, 4) <= kSmLdsLimit;
}

bool conv_sm_two(const GemmArgs& a) { return sm_two_per_cu(a.Cin, a.Cout, a.K, 128); }

hipError_t launch_conv_sm(const GemmArgs& g, int num_cus, hipStream_t stream) {
  SmArgs a;
  a.S = g.S;
  a.table = g.table;
  a.W = g.W;
  a.bias = g.bias;
  a.out = g.out;
  a.n_rows = g.n_rows;
  a.K = g.K;
  a.relu = g.relu;
  if (a.n_rows == 0) return hipSuccess;
  if (g.Cin == 128 && g.Cout == 128) return launch_sm_rows<4, 8>(a, num_cus, stream);
  if (g.Cin == 128 && g.Cout == 64) return launch_sm_rows<4, 4>(a, num_cus, stream);
  if (g.Cin == 64 && g.Cout == 128) return launch_sm_rows<2, 8>(a, num_cus, stream);
  if (g.Cin == 64 && g.Cout == 64) return launch_sm_rows<2, 4>(a, num_cus, stream);
  return hipErrorInvalidValue;
}

}  // namespace shc
