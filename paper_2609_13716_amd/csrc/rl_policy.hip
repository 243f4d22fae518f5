// Standalone policy forward (obs -> logits on the MFMA MLP), standalone
// Gumbel-max sampling from given logits, and the sampler's noise function.
#include <type_traits>

#include "rl_internal.h"
#include "rl_regmlp.h"
#include "rl_sample.h"

namespace rl {

struct PolicyLayout {
  int BM;              // rows per workgroup
  int ldx, ld1, ld2;
  size_t off_x, off_h1, off_h2, off_logit, total;
};

static PolicyLayout make_policy_layout(const PolicyArgs& pol, int BM) {
  PolicyLayout L;
  const size_t es = pol.dt == DT_F32 ? 4 : 2;
  L.BM = BM;
  L.ldx = pol.dt == DT_F32 ? lds_ld<DT_F32>(pol.D) : lds_ld<DT_BF16>(pol.D);
  L.ld1 = pol.dt == DT_F32 ? lds_ld<DT_F32>(pol.H1) : lds_ld<DT_BF16>(pol.H1);
  L.ld2 = pol.dt == DT_F32 ? lds_ld<DT_F32>(pol.H2) : lds_ld<DT_BF16>(pol.H2);
  size_t o = 0;
  L.off_x = o;     o += (size_t)BM * L.ldx * es;  o = (o + 15) & ~(size_t)15;
  L.off_h1 = o;    o += (size_t)BM * L.ld1 * es;  o = (o + 15) & ~(size_t)15;
  L.off_h2 = o;    o += (size_t)BM * L.ld2 * es;  o = (o + 15) & ~(size_t)15;
  L.off_logit = o; o += (size_t)BM * MAX_NA * 4;
  L.total = o;
  return L;
}

static PolicyLayout pick_policy_layout(const PolicyArgs& pol) {
  for (int bm = 64; bm >= 16; bm >>= 1) {
    const PolicyLayout L = make_policy_layout(pol, bm);
    if (L.total <= MAX_LDS_BYTES) return L;
  }
  return make_policy_layout(pol, 16);
}

size_t policy_lds_bytes(const PolicyArgs& pol) { return pick_policy_layout(pol).total; }

template <int DT>
__global__ __launch_bounds__(NTHREADS) void policy_forward_kernel(PolicyArgs pol, PolicyLayout PL,
                                                                  const void* __restrict__ obs_v,
                                                                  const uint8_t* __restrict__ legal, int64_t rows,
                                                                  float* __restrict__ logits) {
  using T = typename DType<DT>::T;
  extern __shared__ __align__(16) uint8_t smem[];
  T* xs = reinterpret_cast<T*>(smem + PL.off_x);
  T* h1 = reinterpret_cast<T*>(smem + PL.off_h1);
  T* h2 = reinterpret_cast<T*>(smem + PL.off_h2);
  float* lg = reinterpret_cast<float*>(smem + PL.off_logit);
  const T* obs = static_cast<const T*>(obs_v);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int BM = PL.BM, D = pol.D, NA = pol.NA;
  const int64_t row0 = (int64_t)blockIdx.x * BM;
  const int nrow = (int)min((int64_t)BM, rows - row0);

  // stage the observation tile, zero-padded to ldx columns and BM rows
  for (int idx = tid; idx < BM * PL.ldx; idx += NTHREADS) {
    const int r = idx / PL.ldx, k = idx - r * PL.ldx;
    xs[idx] = (r < nrow && k < D) ? obs[(size_t)(row0 + r) * D + k] : (T)0;
  }
  // zero the K padding of the hidden tiles
  for (int idx = tid; idx < BM * PL.ld1; idx += NTHREADS) h1[idx] = (T)0;
  for (int idx = tid; idx < BM * PL.ld2; idx += NTHREADS) h2[idx] = (T)0;
  __syncthreads();
  mlp_input_layer<DT>(xs, PL.ldx, nullptr, BM, D, static_cast<const T*>(pol.W[0]), static_cast<const T*>(pol.b[0]), pol.H1, h1,
                 PL.ld1, wave, NTHREADS / 64, lane);
  __syncthreads();
  mlp_hidden<DT>(h1, PL.ld1, BM, pol.H1, static_cast<const T*>(pol.W[1]), static_cast<const T*>(pol.b[1]), pol.H2,
                 h2, PL.ld2, wave, NTHREADS / 64, lane);
  __syncthreads();
  mlp_logits<DT>(h2, PL.ld2, BM, pol.H2, static_cast<const T*>(pol.W[2]), static_cast<const T*>(pol.b[2]), NA, lg,
                 MAX_NA, wave, NTHREADS / 64, lane);
  __syncthreads();
  for (int idx = tid; idx < nrow * NA; idx += NTHREADS) {
    const int r = idx / NA, a = idx - r * NA;
    const size_t gi = (size_t)row0 * NA + idx;
    const bool ok = legal == nullptr || legal[gi] != 0;
    logits[gi] = ok ? lg[r * MAX_NA + a] : -INFINITY;
  }
}

// Persistent policy forward for compile-time sizes: each workgroup keeps the
// layer-1/2 weights in registers and layer 3 in LDS, and loops over tiles of
// MT * 16 rows (stage the observation tile with 16-byte loads, three MFMA
// layers computed transposed, masked logits out).  MINB workgroups share a
// CU so that one's loads overlap another's matrix work.
template <int DT, int D, int H1, int H2, int NA, int NW, int MT, int MINB>
__global__ __launch_bounds__(NW * 64, MINB) void policy_fwd_reg_kernel(PolicyArgs pol, const void* __restrict__ obs_v,
                                                                       const uint8_t* __restrict__ legal,
                                                                       int64_t rows, float* __restrict__ logits) {
  using T = typename DType<DT>::T;
  using B = typename BOperand<DT>::type;
  constexpr int NT = NW * 64, BM = MT * 16;
  constexpr int LDX = lds_ld<DT>(D), LD1 = lds_ld<DT>(H1), LD2 = lds_ld<DT>(H2);
  constexpr int K3 = round_up(H2, DType<DT>::KS) / DType<DT>::KS;
  constexpr int VE = 16 / sizeof(T);
  static_assert(D % VE == 0, "observation rows are whole 16-byte vectors");
  static_assert(NA <= 16, "one transposed M tile of actions");
  static_assert(MT <= NW, "one layer-3 M tile per wave");
  __shared__ __align__(16) T xs[BM * LDX];
  __shared__ __align__(16) T h1s[BM * LD1];
  __shared__ __align__(16) T h2s[BM * LD2];
  __shared__ __align__(16) B w3s[K3 * 64];
  const T* obs = static_cast<const T*>(obs_v);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  RegLayer<DT, D, H1, NW> L1;
  RegLayer<DT, H1, H2, NW> L2;
  L1.load(static_cast<const T*>(pol.W[0]), static_cast<const T*>(pol.b[0]), wave, lane);
  L2.load(static_cast<const T*>(pol.W[1]), static_cast<const T*>(pol.b[1]), wave, lane);
  if (tid < 64) {
    const int n = lane & 15;
    const T* row = static_cast<const T*>(pol.W[2]) + (size_t)(n < NA ? n : 0) * H2;
#pragma unroll
    for (int ks = 0; ks < K3; ++ks) w3s[ks * 64 + lane] = load_operand_global<DT, H2>(row, H2, ks, lane, n < NA);
  }
  float b3r[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int a = 4 * (lane >> 4) + r;
    b3r[r] = a < NA ? DType<DT>::to_f32(static_cast<const T*>(pol.b[2])[a]) : 0.f;
  }
  for (int i = tid; i < BM * LDX; i += NT) xs[i] = (T)0;
  for (int i = tid; i < BM * LD1; i += NT) h1s[i] = (T)0;
  for (int i = tid; i < BM * LD2; i += NT) h2s[i] = (T)0;
  __syncthreads();

  // Software pipeline over this workgroup's tiles: the observation tile of
  // the next iteration is loaded into registers while the current one is
  // computed, and a tile's logits are stored at the start of the next
  // iteration, after that prefetch is issued, so that waiting for the
  // prefetch never waits for just-issued stores.
  const int64_t ntiles = (rows + BM - 1) / BM;
  constexpr int VPR = D / VE, NV = BM * VPR, IT = (NV + NT - 1) / NT;
  u32x4 v[IT];
  auto prefetch = [&](int64_t tile) {
    const int64_t row0 = tile * BM;
    const int nrow = tile < ntiles ? (int)min((int64_t)BM, rows - row0) : 0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = tid + it * NT;
      const int r = i / VPR, c = (i - r * VPR) * VE;
      v[it] = (i < NV && r < nrow) ? *reinterpret_cast<const u32x4*>(obs + (size_t)(row0 + r) * D + c)
                                    : u32x4{0u, 0u, 0u, 0u};
    }
  };
  float lg[4] = {0.f, 0.f, 0.f, 0.f};
  int64_t lg_row = -1;  // global row of the pending logits (-1: none)
  auto store_logits = [&]() {
    if (lg_row >= 0) {
      const size_t gr = (size_t)lg_row * NA;
      const int g = lane >> 4;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 4 * g + r;
        if (a < NA) {
          const bool ok = legal == nullptr || legal[gr + a] != 0;
          logits[gr + a] = ok ? lg[r] : -INFINITY;
        }
      }
    }
  };
  prefetch(blockIdx.x);
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t row0 = tile * BM;
    const int nrow = (int)min((int64_t)BM, rows - row0);
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = tid + it * NT;
      const int r = i / VPR, c = (i - r * VPR) * VE;
      if (i < NV) *reinterpret_cast<u32x4*>(xs + r * LDX + c) = v[it];
    }
    __syncthreads();
    if (tile + gridDim.x < ntiles) prefetch(tile + gridDim.x);
    store_logits();
    lg_row = -1;
    {
      f32x4 acc[MT][RegLayer<DT, D, H1, NW>::OWN];
      L1.template run<MT>(xs, LDX, acc, wave, lane);
      L1.template store_tanh<MT>(acc, h1s, LD1, wave, lane);
    }
    __syncthreads();
    {
      f32x4 acc[MT][RegLayer<DT, H1, H2, NW>::OWN];
      L2.template run<MT>(h1s, LD1, acc, wave, lane);
      L2.template store_tanh<MT>(acc, h2s, LD2, wave, lane);
    }
    __syncthreads();
    if (wave < MT) {
      const int row = wave * 16 + (lane & 15);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < K3; ++ks)
        acc = mfma16<DT>(w3s[ks * 64 + lane], load_operand_lds<DT>(h2s, LD2, row, ks, lane), acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) lg[r] = acc[r] + b3r[r];
      lg_row = row < nrow ? row0 + row : -1;
    }
  }
  store_logits();
}

// Software-pipelined variant for the narrow bf16 policies (one workgroup of
// 4 waves per CU).  In a 128-wide layer the tanh epilogue (two
// transcendental instructions per value) takes longer than the layer's
// MFMAs, so each wave overlaps one tile's epilogue with the next tile's
// matrix products: iteration j of a workgroup runs
//   phase A: layer 3 of tile j-2 (logits out), layer-1 MFMAs of tile j+1
//            interleaved with the layer-1 epilogue of tile j;
//   phase B: the observation tile of j+2 staged from registers, the load of
//            tile j+3 issued, layer-2 MFMAs of tile j interleaved with the
//            layer-2 epilogue of tile j-1;
// with one barrier after each phase.  The observation tile is double
// buffered; h1 and h2 have one buffer each (every write of one is separated
// from the reads of its previous contents by a barrier).  Tiles past this
// workgroup's last are computed from zeros and never stored.  Every output
// is the same MFMA chain and epilogue as policy_fwd_reg_kernel and the
// rollout kernels, so the logits are bit-identical to theirs.
template <int D, int H1, int H2, int NA, int MT, int MINB>
__global__ __launch_bounds__(256, MINB) void policy_fwd_pipe_kernel(PolicyArgs pol, const void* __restrict__ obs_v,
                                                                  const uint8_t* __restrict__ legal, int64_t rows,
                                                                  float* __restrict__ logits) {
  constexpr int DT = DT_BF16, NW = 4, NT = NW * 64, BM = MT * 16;
  using T = typename DType<DT>::T;
  using B = typename BOperand<DT>::type;
  constexpr int LDX = lds_ld<DT>(D), LD1 = lds_ld<DT>(H1), LD2 = lds_ld<DT>(H2);
  constexpr int K3 = round_up(H2, DType<DT>::KS) / DType<DT>::KS;
  constexpr int VE = 16 / sizeof(T);
  // rows of D elements: whole 16-byte vectors, or (FLAT) a tile read as one
  // flat block of BM * D elements (16-byte aligned when BM * D is a multiple
  // of 8) and scattered into the LDS rows element by element
  constexpr bool FLAT = D % VE != 0;
  static_assert(!FLAT || (BM * D) % VE == 0, "flat observation tiles start on 16-byte boundaries");
  static_assert(NA <= 16, "one transposed M tile of actions");
  static_assert(MT <= NW, "one layer-3 M tile per wave");
  __shared__ __align__(16) T xs[2][BM * LDX];
  __shared__ __align__(16) T h1s[BM * LD1];
  __shared__ __align__(16) T h2s[BM * LD2];
  __shared__ __align__(16) B w3s[K3 * 64];
  const T* obs = static_cast<const T*>(obs_v);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  RegLayer<DT, D, H1, NW> L1;
  RegLayer<DT, H1, H2, NW> L2;
  L1.load(static_cast<const T*>(pol.W[0]), static_cast<const T*>(pol.b[0]), wave, lane);
  L2.load(static_cast<const T*>(pol.W[1]), static_cast<const T*>(pol.b[1]), wave, lane);
  if (tid < 64) {
    const int n = lane & 15;
    const T* row = static_cast<const T*>(pol.W[2]) + (size_t)(n < NA ? n : 0) * H2;
#pragma unroll
    for (int ks = 0; ks < K3; ++ks) w3s[ks * 64 + lane] = load_operand_global<DT, H2>(row, H2, ks, lane, n < NA);
  }
  float b3r[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int a = 4 * (lane >> 4) + r;
    b3r[r] = a < NA ? DType<DT>::to_f32(static_cast<const T*>(pol.b[2])[a]) : 0.f;
  }
  for (int i = tid; i < 2 * BM * LDX; i += NT) (&xs[0][0])[i] = (T)0;
  for (int i = tid; i < BM * LD1; i += NT) h1s[i] = (T)0;
  for (int i = tid; i < BM * LD2; i += NT) h2s[i] = (T)0;

  const int64_t ntiles = (rows + BM - 1) / BM;
  const int nt = (int64_t)blockIdx.x < ntiles ? (int)((ntiles - 1 - blockIdx.x) / gridDim.x) + 1 : 0;
  auto tile_of = [&](int j) { return (int64_t)blockIdx.x + (int64_t)j * gridDim.x; };
  constexpr int VPR = D / VE, NV = FLAT ? BM * D / VE : BM * VPR, IT = (NV + NT - 1) / NT;
  u32x4 v[IT];
  auto prefetch = [&](int j) {  // tile j of this workgroup into registers (zeros past the last)
    const int64_t row0 = tile_of(j) * BM;
    const int nrow = j < nt ? (int)min((int64_t)BM, rows - row0) : 0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = tid + it * NT;
      if constexpr (FLAT) {
        // flat element i * VE of the tile; the vector that holds the tile's
        // last element is read element by element (nothing past the batch)
        const int nel = nrow * D, e0 = i * VE;
        const T* src = obs + (size_t)row0 * D + e0;
        if (i < NV && e0 + VE <= nel) {
          v[it] = *reinterpret_cast<const u32x4*>(src);
        } else {
          uint32_t h[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t lo = (i < NV && e0 + 2 * q < nel) ? (uint32_t)src[2 * q] : 0u;
            const uint32_t hi = (i < NV && e0 + 2 * q + 1 < nel) ? (uint32_t)src[2 * q + 1] : 0u;
            h[q] = lo | (hi << 16);
          }
          v[it] = u32x4{h[0], h[1], h[2], h[3]};
        }
      } else {
        const int r = i / VPR, c = (i - r * VPR) * VE;
        v[it] = (i < NV && r < nrow) ? *reinterpret_cast<const u32x4*>(obs + (size_t)(row0 + r) * D + c)
                                      : u32x4{0u, 0u, 0u, 0u};
      }
    }
  };
  auto stage = [&](T* dst) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = tid + it * NT;
      if (i >= NV) continue;
      if constexpr (FLAT) {
#pragma unroll
        for (int q = 0; q < VE; ++q) {
          const int el = i * VE + q, r = el / D, c = el - r * D;
          dst[r * LDX + c] = (T)((v[it][q >> 1] >> (16 * (q & 1))) & 0xffffu);
        }
      } else {
        const int r = i / VPR, c = (i - r * VPR) * VE;
        *reinterpret_cast<u32x4*>(dst + r * LDX + c) = v[it];
      }
    }
  };

  __syncthreads();  // zero fill done before the staging writes
  prefetch(0);
  stage(xs[0]);
  prefetch(1);
  stage(xs[1]);
  prefetch(2);
  __syncthreads();
  f32x4 acc1[MT][RegLayer<DT, D, H1, NW>::OWN];
  f32x4 acc2[MT][RegLayer<DT, H1, H2, NW>::OWN];
  L1.template run<MT>(xs[0], LDX, acc1, wave, lane);
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int o = 0; o < RegLayer<DT, H1, H2, NW>::OWN; ++o) acc2[m][o] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int j = 0;; ++j) {
    // phase A
    if (j >= 2 && wave < MT) {
      const int row = wave * 16 + (lane & 15);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < K3; ++ks)
        acc = mfma16<DT>(w3s[ks * 64 + lane], load_operand_lds<DT>(h2s, LD2, row, ks, lane), acc);
      const int64_t row0 = tile_of(j - 2) * BM;
      if (row0 + row < rows) {
        const size_t gr = (size_t)(row0 + row) * NA;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 4 * (lane >> 4) + r;
          if (a < NA) {
            const bool ok = legal == nullptr || legal[gr + a] != 0;
            logits[gr + a] = ok ? acc[r] + b3r[r] : -INFINITY;
          }
        }
      }
    }
    if (j == nt + 1) break;
    L1.template run_overlapped<MT>(xs[(j + 1) & 1], LDX, acc1, h1s, LD1, wave, lane);
    __syncthreads();
    // phase B
    stage(xs[j & 1]);
    prefetch(j + 3);
    L2.template run_overlapped<MT>(h1s, LD1, acc2, h2s, LD2, wave, lane);
    __syncthreads();
  }
}

template <int D, int H1, int H2, int NA, int MT, int MINB>
static hipError_t launch_policy_pipe(const PolicyArgs& pol, const void* obs, const uint8_t* legal, int64_t rows,
                                     float* logits, hipStream_t s) {
  constexpr int BM = MT * 16;
  const int64_t ntiles = (rows + BM - 1) / BM;
  const unsigned grid = (unsigned)(ntiles < (int64_t)256 * MINB ? ntiles : (int64_t)256 * MINB);
  policy_fwd_pipe_kernel<D, H1, H2, NA, MT, MINB><<<dim3(grid), 256, 0, s>>>(pol, obs, legal, rows, logits);
  return hipGetLastError();
}

template <int DT, int D, int H1, int H2, int NA, int NW, int MT, int MINB>
static hipError_t launch_policy_reg(const PolicyArgs& pol, const void* obs, const uint8_t* legal, int64_t rows,
                                    float* logits, hipStream_t s) {
  constexpr int BM = MT * 16;
  const int64_t ntiles = (rows + BM - 1) / BM;
  const unsigned grid = (unsigned)(ntiles < (int64_t)256 * MINB ? ntiles : (int64_t)256 * MINB);
  policy_fwd_reg_kernel<DT, D, H1, H2, NA, NW, MT, MINB><<<dim3(grid), NW * 64, 0, s>>>(pol, obs, legal, rows, logits);
  return hipGetLastError();
}

static bool try_launch_policy_reg(const PolicyArgs& pol, const void* obs, const uint8_t* legal, int64_t rows,
                                  float* logits, hipStream_t s, hipError_t* err) {
#define RL_PF_CASE(DTV, DV, H1V, H2V, NAV, NWV, MTV, MINBV)                                              \
  if (pol.dt == DTV && pol.D == DV && pol.H1 == H1V && pol.H2 == H2V && pol.NA == NAV) {                   \
    *err = launch_policy_reg<DTV, DV, H1V, H2V, NAV, NWV, MTV, MINBV>(pol, obs, legal, rows, logits, s); \
    return true;                                                                                         \
  }
  // (dtype, D, H1, H2, nA, waves, 16-row M tiles per workgroup tile, workgroups per CU)
  if (pol.dt == DT_BF16 && pol.D == 192 && pol.H1 == 128 && pol.H2 == 128 && pol.NA == 6) {
    *err = launch_policy_pipe<192, 128, 128, 6, 2, 2>(pol, obs, legal, rows, logits, s);
    return true;
  }
  if (pol.dt == DT_BF16 && pol.D == 147 && pol.H1 == 128 && pol.H2 == 128 && pol.NA == 6) {  // 7 x 7 LBF
    *err = launch_policy_pipe<147, 128, 128, 6, 2, 2>(pol, obs, legal, rows, logits, s);
    return true;
  }
  RL_PF_CASE(DT_F32, 192, 128, 128, 6, 4, 4, 1)
  RL_PF_CASE(DT_BF16, 192, 64, 64, 6, 4, 4, 2)
  RL_PF_CASE(DT_F32, 192, 64, 64, 6, 4, 4, 2)
#undef RL_PF_CASE
  return false;
}

// ------------------------------------------------ tiled policy forward ----
//
// bf16 policy forward for wide layers (the 12x12 LBF, kitchen and Hanabi
// policies): three chained GEMMs per tile of BM = 16 MT rows, H / 64 waves.
//   * Wave w computes hidden units 64 w .. 64 w + 63 of every row of the tile
//     (4 x MT accumulator tiles), so each weight byte is read by one wave
//     only: weights go from L2 straight into the MFMA operand registers (the
//     fragment-major copy: 1 KB contiguous per load), two K steps ahead, and
//     never through LDS.
//   * Observation rows are staged through LDS in stages of 64 features (128
//     contiguous bytes per row, 16-byte chunks XOR-swizzled by row), loaded
//     one stage ahead into registers.
//   * h1 stays in LDS (over the staging buffers); h2 overwrites it once every
//     wave has read h1; layer 3 is computed transposed (actions x rows).
// Every output is one MFMA chain over K in increasing order, bias added
// after, so the logits are bit-identical to the other policy paths.
//
// What bounds it: at MT 8 a K step is 32 MFMAs per wave (512 cycles on its
// SIMD) against 16 KB (256 units) of weights and 8 KB of rows into the CU and
// 32 KB of LDS reads (256 cycles); under this load the clock falls to about
// 1.9 GHz, and a layer's tanh epilogue (128 values per lane at about 34 cycles) is
// hidden only as far as the two workgroups of a CU drift apart.  Tiles of 64 rows
// with the weights staged through LDS moved 60 KB of LDS per 64-row K step
// (480 cycles against 256 of MFMA): 1170-256-256-6 over 262144 rows 360 -> 223 us,
// 658-512-512-20 over 100003 rows with legality masks 328 -> 166 us, 432-256-256-6
// over 262144 rows 159 -> 102 us.  Loading the rows two stages ahead, or as single
// words, changed nothing.
// HBM reads over 262144 rows: at a row pitch that is no multiple of 128 bytes a stage
// ends inside a line, and 5-17% of the lines are read twice (1170-256-256-6 708 MB for
// 613 MB of rows; 1152 features, whole lines, 635 for 604); and each XCD reads the
// weights anew for about every round of workgroups (640-512-512-20, whole lines: 413 MB
// for 335 MB of rows, 66 times its 1.2 MB of weights).
constexpr int PT_SK = 64;  // features per staged slice: two MFMA K steps

template <int H, int MT>
struct PtLayout {
  static constexpr int BM = 16 * MT;
  static constexpr int LDH = H + 8;  // pitch of the resident activation tile
  static constexpr size_t H_BYTES = (size_t)BM * LDH * 2;
  static constexpr size_t X_BYTES = (size_t)BM * PT_SK * 2;  // one staged slice
  static constexpr size_t OFF_B = H_BYTES;                   // fp32 biases of layers 1 and 2
  static constexpr size_t TOTAL = OFF_B + 2 * H * 4;
  static_assert(2 * X_BYTES <= H_BYTES, "both staging buffers lie in the activation tile");
};

// Buffer resource over `bytes` bytes at p (raw: loads past the end read 0).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pt_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Zero the elements of an 8-element bf16 vector at or beyond `left` (the
// number of the vector's elements that lie inside the row).
__device__ __forceinline__ u32x4 pt_mask8(u32x4 v, int left) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t m = 2 * d + 1 < left ? 0xffffffffu : 2 * d < left ? 0x0000ffffu : 0u;
    v[d] &= m;
  }
  return v;
}

template <int H, int MT, bool PK>
__global__ __launch_bounds__(H, H == 256 ? 2 : 1) void policy_fwd_tiled_kernel(PolicyArgs pol,
                                                                               const uint16_t* __restrict__ obs,
                                                                               const uint8_t* __restrict__ legal,
                                                                               int64_t rows, float* __restrict__ logits) {
  using L = PtLayout<H, MT>;
  constexpr int NT = H, NW = H / 64, BM = L::BM;
  constexpr int UT = 4;  // unit tiles of a wave
  constexpr int XV = (BM * 8 + NT - 1) / NT;  // staged 16-byte vectors per thread
  constexpr bool XALL = BM * 8 % NT == 0;
  extern __shared__ __align__(16) uint8_t smem[];
  uint16_t* hs = reinterpret_cast<uint16_t*>(smem);
  uint16_t* xst = hs;  // the two staging buffers, until layer 1's outputs are stored
  float* bias_s = reinterpret_cast<float*>(smem + L::OFF_B);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int D = pol.D, NA = pol.NA;
  const int64_t row0 = (int64_t)blockIdx.x * BM;
  const int nrow = (int)min((int64_t)BM, rows - row0);

  for (int i = tid; i < 2 * H; i += NT)
    bias_s[i] = bf16_to_f32(i < H ? static_cast<const uint16_t*>(pol.b[0])[i]
                                  : static_cast<const uint16_t*>(pol.b[1])[i - H]);

  // Weight operands of a layer: unit tile 4 wave + u, K step st.  An unpacked tile is
  // loaded with four consecutive lanes on the 64 bytes of a row and moved to the
  // operand's lanes when it is used (a lane per row and 16 bytes, as the MFMA takes it,
  // touches 16 lines every 16 lanes, about 20 bytes per clock: 64-256-256-6 at 32768
  // rows 16.2 against 13.4 us, 2048-512-512-6 at 1024 rows 76.5 against 38.6).
  auto w_rsrc = [&](int l, int K) {
    const int S = (K + 31) / 32;
    return PK ? pt_rsrc(pol.Wp[l], (uint32_t)(H / 16) * S * 1024) : pt_rsrc(pol.W[l], (uint32_t)H * K * 2);
  };
  auto w_offs = [&](int K, int (&wo)[UT]) {
    const int S = (K + 31) / 32;
#pragma unroll
    for (int u = 0; u < UT; ++u)
      wo[u] = PK ? ((4 * wave + u) * S * 64 + lane) * 16 : ((64 * wave + 16 * u + (lane >> 2)) * K + 8 * (lane & 3)) * 2;
  };
  auto w_operand = [&](u32x4 v) -> u32x4 {
    if constexpr (PK) return v;
    u32x4 o;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      o[d] = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (4 * (lane & 15) + (lane >> 4)), (int)v[d]);
    return o;
  };
  auto w_load = [&](__amdgpu_buffer_rsrc_t r, int off, int st) -> u32x4 {
    return __builtin_amdgcn_raw_buffer_load_b128(r, off, st * (PK ? 1024 : 64), 0);
  };

  f32x4 acc[UT][MT];
  auto clear = [&]() {
#pragma unroll
    for (int u = 0; u < UT; ++u)
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[u][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // tanh(acc + bias) to the activation tile: four consecutive units of one row per lane
  auto epilogue = [&](const float* bias) {
#pragma unroll
    for (int u = 0; u < UT; ++u) {
      const int u0 = 64 * wave + 16 * u + 4 * (lane >> 4);
      const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + u0);
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = fast_tanh(acc[u][m][q] + b4[q]);
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<u32x2*>(hs + (16 * m + (lane & 15)) * L::LDH + u0) =
            u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      }
    }
  };

  u32x4 wr[2][UT];  // weight operands of K steps st, st + 1 (slot = st % 2), each refilled in place for st + 2
  // ---- layer 1 ----
  {
    const int S = (D + 31) / 32, NS = (D + PT_SK - 1) / PT_SK;
    const __amdgpu_buffer_rsrc_t wres = w_rsrc(0, D);
    const __amdgpu_buffer_rsrc_t xres = pt_rsrc(obs + (size_t)row0 * D, (uint32_t)nrow * D * 2);
    int wo[UT], xgo[XV], xlo[XV];
    w_offs(D, wo);
#pragma unroll
    for (int j = 0; j < XV; ++j) {
      const int v = tid + j * NT, r = v >> 3, c = v & 7;
      xgo[j] = (r * D + 8 * c) * 2;  // rows past nrow lie past the resource: read as 0
      xlo[j] = r * PT_SK + 8 * (c ^ (r & 7));
    }
    u32x4 xv[XV];
    auto fetch_x = [&](int s) {
#pragma unroll
      for (int j = 0; j < XV; ++j)
        if (XALL || tid + j * NT < BM * 8) xv[j] = __builtin_amdgcn_raw_buffer_load_b128(xres, xgo[j], s * PT_SK * 2, 0);
    };
    auto store_x = [&](int s) {
      uint16_t* xb = xst + (s & 1) * (BM * PT_SK);
#pragma unroll
      for (int j = 0; j < XV; ++j)
        if (XALL || tid + j * NT < BM * 8) *reinterpret_cast<u32x4*>(xb + xlo[j]) = xv[j];
    };
    const int brow = (lane & 15) * PT_SK;
    // K step st = 2 s + KK of staged slice s
    auto step = [&](auto kk_c, int s) {
      constexpr int KK = decltype(kk_c)::value;
      const int st = 2 * s + KK;
      const uint16_t* xb = xst + (s & 1) * (BM * PT_SK) + brow + 8 * ((4 * KK + (lane >> 4)) ^ (lane & 7));
      u32x4 b[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) b[m] = *reinterpret_cast<const u32x4*>(xb + m * 16 * PT_SK);
      if (st * 32 + 32 > D) {  // the partial last K step: nothing past the row takes part (uniform branch)
        const int left = D - st * 32 - 8 * (lane >> 4);
#pragma unroll
        for (int m = 0; m < MT; ++m) b[m] = pt_mask8(b[m], left);
      }
#pragma unroll
      for (int u = 0; u < UT; ++u) {
        u32x4 a = w_operand(wr[KK][u]);
        if (!PK && st * 32 + 32 > D) a = pt_mask8(a, D - st * 32 - 8 * (lane >> 4));
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[u][m] = mfma16<DT_BF16>(a, b[m], acc[u][m]);
        wr[KK][u] = w_load(wres, wo[u], st + 2);  // (past the last step: unused)
      }
    };
    fetch_x(0);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int u = 0; u < UT; ++u) wr[kk][u] = w_load(wres, wo[u], kk);
    clear();
    store_x(0);
    if (NS > 1) fetch_x(1);
    __syncthreads();
    for (int s = 0; s < NS; ++s) {
      step(std::integral_constant<int, 0>{}, s);
      if (2 * s + 1 < S) step(std::integral_constant<int, 1>{}, s);
      if (s + 1 < NS) store_x(s + 1);  // (its buffer was last read in stage s - 1)
      if (s + 2 < NS) fetch_x(s + 2);
      __syncthreads();
    }
  }
  // ---- layer 2: its first weights are on their way during layer 1's epilogue ----
  {
    const __amdgpu_buffer_rsrc_t wres = w_rsrc(1, H);
    int wo[UT];
    w_offs(H, wo);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int u = 0; u < UT; ++u) wr[kk][u] = w_load(wres, wo[u], kk);
    epilogue(bias_s);
    clear();
    __syncthreads();
    const uint16_t* hb = hs + (lane & 15) * L::LDH + 8 * (lane >> 4);
#pragma unroll 2
    for (int st = 0; st < H / 32; st += 2) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        u32x4 b[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) b[m] = *reinterpret_cast<const u32x4*>(hb + m * 16 * L::LDH + (st + kk) * 32);
#pragma unroll
        for (int u = 0; u < UT; ++u) {
          const u32x4 a = w_operand(wr[kk][u]);
#pragma unroll
          for (int m = 0; m < MT; ++m) acc[u][m] = mfma16<DT_BF16>(a, b[m], acc[u][m]);
          wr[kk][u] = w_load(wres, wo[u], st + kk + 2);
        }
      }
    }
  }
  __syncthreads();  // every wave is past its last read of h1
  epilogue(bias_s + H);
  __syncthreads();

  // ---- layer 3, transposed: logits^T = W3 h2^T, wave w takes row tiles w, w + NW, ... ----
  constexpr int K3 = H / 32;
  const int nat = (NA + 15) >> 4;
  for (int mt = 0; mt < nat; ++mt) {
    const int a_row = mt * 16 + (lane & 15);
    const uint16_t* w3r = static_cast<const uint16_t*>(pol.W[2]) + (size_t)(a_row < NA ? a_row : 0) * H + 8 * (lane >> 4);
    for (int rt = wave; rt < MT; rt += NW) {
      const int r = rt * 16 + (lane & 15);
      u32x4 a3[K3];
#pragma unroll
      for (int ks = 0; ks < K3; ++ks)
        a3[ks] = a_row < NA ? *reinterpret_cast<const u32x4*>(w3r + ks * 32) : u32x4{0u, 0u, 0u, 0u};
      f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < K3; ++ks)
        c = mfma16<DT_BF16>(a3[ks], *reinterpret_cast<const u32x4*>(hs + r * L::LDH + ks * 32 + 8 * (lane >> 4)), c);
      if (r < nrow) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int act = mt * 16 + 4 * (lane >> 4) + q;
          if (act < NA) {
            const size_t gi = (size_t)(row0 + r) * NA + act;
            const float lg = c[q] + bf16_to_f32(static_cast<const uint16_t*>(pol.b[2])[act]);
            logits[gi] = (legal == nullptr || legal[gi] != 0) ? lg : -INFINITY;
          }
        }
      }
    }
  }
}

template <int H, int MT, bool PK>
static hipError_t launch_policy_tiled_mt(const PolicyArgs& pol, const void* obs, const uint8_t* legal, int64_t rows,
                                         float* logits, hipStream_t s) {
  using L = PtLayout<H, MT>;
  static_assert(L::TOTAL <= MAX_LDS_BYTES, "tile fits in LDS");
  static bool attr = false;
  if (!attr) {
    const hipError_t e = hipFuncSetAttribute((const void*)policy_fwd_tiled_kernel<H, MT, PK>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)L::TOTAL);
    if (e != hipSuccess) return e;
    attr = true;
  }
  const unsigned grid = (unsigned)((rows + L::BM - 1) / L::BM);
  policy_fwd_tiled_kernel<H, MT, PK><<<dim3(grid), H, L::TOTAL, s>>>(pol, static_cast<const uint16_t*>(obs), legal,
                                                                     rows, logits);
  return hipGetLastError();
}

// Row tiles of a workgroup.  A CU works through ceil(workgroups / 256)
// workgroups, and a workgroup of MT row tiles costs about k + MT: the weights
// it reads and its prologue are the constant part (k = 3 at 256 units, two workgroups
// sharing the CU; 2 at 512).  The least product is taken, the larger tile on
// ties.  Packed weights, measured over MT 1, 2, 4, 5, 6, 7, 8 (us; chosen one starred):
// 1170-256-256-6 at 262144 rows 648, 415, 269, 264, 250, 243, 224*; at 16384
// rows 35, 22.7, 23.3*, 26, 27, 31, 33; at 4096 rows 13.0*, 13.0, 17, 21, 23, 27, 28;
// 658-512-512-20 at 100003 rows 317, 189, 169, 159*, 175, 156, 173; at 98304
// rows 345, 188, 154, 159, 145, 156, 135*.
//
// The product counts two workgroups on a CU as twice the time of one.  At 256 units
// with packed weights two of MT 4 take 1.2 to 1.4 times the time of one, so that MT 4
// is the best tile as long as all its workgroups are resident and fewer, larger
// tiles would leave a CU one workgroup: 20481 to 32768 rows (32768 rows of 34, 432
// and 1170 features, MT 4 against the 8 of the product: 11.4 and 14.6, 16.3 and 20.2,
// 28.8 and 33.3 us; 22000 rows, against 6: 11.0 and 12.1, 14.7 and 15.8, 27.2 and
// 27.2; up to 20480 rows MT 5 is as good or up to 5% better).  With unpacked weights
// that holds for narrow rows only (32768 rows of 64, 192, 432, 658 features: 13.3 and
// 15.8, 15.8 and 17.8, 23.9 and 24.1, 32.9 and 30.2; 24576 rows, against 6: 13.3 and
// 13.4, 15.6 and 15.2, 21.2 and 19.6).  Unpacked forwards over 1 to 131072 rows of 16
// to 2048 features then take 0.34 to 1.05 of their time in 64-row tiles with the weights
// staged through LDS (192-256-256-6 at 30000 rows 16.2 staged, 15.7 here;
// 658-512-512-6 at 100003 rows 335 and 200 us); the 1.05 is 0.6 us at 16 features
// and 20481 rows.
constexpr int PT_CUS = 256;
static int pt_pick_mt(int H, int D, bool packed, int64_t rows) {
  if (H == 256 && (packed || D <= 192) && rows > 16 * 5 * PT_CUS && rows <= 16 * 4 * 2 * PT_CUS) return 4;
  const int k = H == 256 ? 3 : 2;
  int best = 8;
  int64_t best_cost = INT64_MAX;
  for (int mt : {8, 7, 6, 5, 4, 2, 1}) {
    const int64_t wgs = (rows + 16 * mt - 1) / (16 * mt), cost = (wgs + PT_CUS - 1) / PT_CUS * (k + mt);
    if (cost < best_cost) {
      best_cost = cost;
      best = mt;
    }
  }
  return best;
}

template <int H, bool PK>
static hipError_t launch_policy_tiled(const PolicyArgs& pol, const void* obs, const uint8_t* legal, int64_t rows,
                                      float* logits, hipStream_t s) {
  switch (pt_pick_mt(H, pol.D, PK, rows)) {
    case 1: return launch_policy_tiled_mt<H, 1, PK>(pol, obs, legal, rows, logits, s);
    case 2: return launch_policy_tiled_mt<H, 2, PK>(pol, obs, legal, rows, logits, s);
    case 4: return launch_policy_tiled_mt<H, 4, PK>(pol, obs, legal, rows, logits, s);
    case 5: return launch_policy_tiled_mt<H, 5, PK>(pol, obs, legal, rows, logits, s);
    case 6: return launch_policy_tiled_mt<H, 6, PK>(pol, obs, legal, rows, logits, s);
    case 7: return launch_policy_tiled_mt<H, 7, PK>(pol, obs, legal, rows, logits, s);
    default: return launch_policy_tiled_mt<H, 8, PK>(pol, obs, legal, rows, logits, s);
  }
}

// Shapes the tiled kernel serves: bf16, two hidden layers of 256 or of 512
// units, an even input width.
static bool try_launch_policy_tiled(const PolicyArgs& pol, const void* obs, const uint8_t* legal, int64_t rows,
                                    float* logits, hipStream_t s, hipError_t* err) {
  if (pol.dt != DT_BF16 || pol.D % 2 != 0 || pol.H1 != pol.H2 || pol.NA > MAX_NA) return false;
  const bool pk = pol.Wp[0] != nullptr;
  if (pol.H1 == 256)
    *err = pk ? launch_policy_tiled<256, true>(pol, obs, legal, rows, logits, s)
              : launch_policy_tiled<256, false>(pol, obs, legal, rows, logits, s);
  else if (pol.H1 == 512)
    *err = pk ? launch_policy_tiled<512, true>(pol, obs, legal, rows, logits, s)
              : launch_policy_tiled<512, false>(pol, obs, legal, rows, logits, s);
  else
    return false;
  return true;
}

// ---------------------------------------------------- packed weights ----
//
// Writes the fragment-major copy of one bf16 layer W [N x K] (layout in
// packed_layer_offset): one thread per 16-byte operand block, zero outside W.
__global__ void policy_pack_kernel(const uint16_t* __restrict__ W, int N, int K, uint16_t* __restrict__ out,
                                   int64_t nvec) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nvec) return;
  const int S = (K + 31) / 32;
  const int lane = (int)(v & 63);
  const int64_t ts = v >> 6;
  const int s = (int)(ts % S), t = (int)(ts / S);
  const int n = 16 * t + (lane & 15), k0 = 32 * s + 8 * (lane >> 4);
  uint32_t h[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = (n < N && k0 + 2 * q < K) ? W[(size_t)n * K + k0 + 2 * q] : 0u;
    const uint32_t hi = (n < N && k0 + 2 * q + 1 < K) ? W[(size_t)n * K + k0 + 2 * q + 1] : 0u;
    h[q] = lo | (hi << 16);
  }
  *reinterpret_cast<u32x4*>(out + v * 8) = u32x4{h[0], h[1], h[2], h[3]};
}

hipError_t launch_policy_pack(const PolicyArgs& pol, void* packed, hipStream_t s) {
  const int dims[4] = {pol.D, pol.H1, pol.H2, pol.NA};
  for (int l = 0; l < 3; ++l) {
    const int64_t nvec = (int64_t)(packed_layer_bytes(dims[l + 1], dims[l]) / 16);
    uint16_t* out = reinterpret_cast<uint16_t*>(static_cast<uint8_t*>(packed) + packed_layer_offset(dims, l));
    policy_pack_kernel<<<dim3((unsigned)((nvec + 255) / 256)), 256, 0, s>>>(static_cast<const uint16_t*>(pol.W[l]),
                                                                          dims[l + 1], dims[l], out, nvec);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_policy_forward(const PolicyArgs& pol, const void* obs, const uint8_t* legal, int64_t rows,
                                 float* logits, hipStream_t s) {
  hipError_t err;
  if (try_launch_policy_reg(pol, obs, legal, rows, logits, s, &err)) return err;
  if (try_launch_policy_tiled(pol, obs, legal, rows, logits, s, &err)) return err;
  const PolicyLayout PL = pick_policy_layout(pol);
  const dim3 grid((unsigned)((rows + PL.BM - 1) / PL.BM));
  if (pol.dt == DT_F32) {
    static bool attr = false;
    if (!attr) {
      hipError_t e = hipFuncSetAttribute((const void*)policy_forward_kernel<DT_F32>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)MAX_LDS_BYTES);
      if (e != hipSuccess) return e;
      attr = true;
    }
    policy_forward_kernel<DT_F32><<<grid, NTHREADS, PL.total, s>>>(pol, PL, obs, legal, rows, logits);
  } else {
    static bool attr = false;
    if (!attr) {
      hipError_t e = hipFuncSetAttribute((const void*)policy_forward_kernel<DT_BF16>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)MAX_LDS_BYTES);
      if (e != hipSuccess) return e;
      attr = true;
    }
    policy_forward_kernel<DT_BF16><<<grid, NTHREADS, PL.total, s>>>(pol, PL, obs, legal, rows, logits);
  }
  return hipGetLastError();
}

// One thread per (env, agent) row: noise, scores, first argmax.
__global__ __launch_bounds__(NTHREADS) void sample_kernel(uint64_t seed, int64_t env_base, int E, int A, int NA,
                                                          uint64_t t, const float* __restrict__ logits,
                                                          const uint8_t* __restrict__ legal,
                                                          int32_t* __restrict__ actions) {
  const int64_t row = (int64_t)blockIdx.x * NTHREADS + threadIdx.x;
  if (row >= (int64_t)E * A) return;
  const int e = (int)(row / A), ag = (int)(row - (int64_t)e * A);
  int best = 0;
  float bs = -INFINITY;
  for (int a = 0; a < NA; ++a) {
    const size_t i = (size_t)row * NA + a;
    const float g = action_noise(seed, (uint64_t)(env_base + e), t, ag, a);
    const float v = action_score(logits[i], g, legal == nullptr || legal[i] != 0);
    if (v > bs) {
      bs = v;
      best = a;
    }
  }
  actions[row] = best;
}

hipError_t launch_sample(uint64_t seed, int64_t env_base, int E, int A, int NA, uint64_t t, const float* logits,
                         const uint8_t* legal, int32_t* actions, hipStream_t s) {
  const int64_t rows = (int64_t)E * A;
  sample_kernel<<<dim3((unsigned)((rows + NTHREADS - 1) / NTHREADS)), NTHREADS, 0, s>>>(seed, env_base, E, A, NA, t,
                                                                                       logits, legal, actions);
  return hipGetLastError();
}

__global__ __launch_bounds__(NTHREADS) void gumbel_kernel(const uint32_t* __restrict__ u, int64_t n,
                                                          float* __restrict__ g) {
  const int64_t i = (int64_t)blockIdx.x * NTHREADS + threadIdx.x;
  if (i < n) g[i] = gumbel24(u[i] & 0xffffffu);
}

hipError_t launch_gumbel(const uint32_t* u, int64_t n, float* g, hipStream_t s) {
  gumbel_kernel<<<dim3((unsigned)((n + NTHREADS - 1) / NTHREADS)), NTHREADS, 0, s>>>(u, n, g);
  return hipGetLastError();
}

}  // namespace rl
