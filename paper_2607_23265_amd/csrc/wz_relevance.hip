// Stage 1, streaming part: the similarity-branch Cross-Modal Scorer (Sec.
// 3.2.1) and the pooled features of the Visual Change Estimator (Sec. 3.2.2,
// Eq. (8)) in ONE kernel that reads the frames once.  Per token it needs
//     x . q_j  (all j),  |x|^2,  |q_j|^2,
// and per frame the channel sums p_t = sum_n x_{t,n} (the mean's cosine is the
// sum's) and sigma_j = sum_n x_{t,n} . q_j = p_t . q_j.  It writes them per
// work unit (and a_{t,n}, final where a workgroup has every channel); the
// per-frame kernel adds the units' partials in a fixed order and forms r_t and
// delta_t.
//
// Four decompositions, the first three with every channel in a workgroup:
//  * token tiles (fp32 inputs; bf16, Q <= 64 and some of 128 < Q <= 256): a
//    workgroup owns up to 64 tokens of a frame, its waves split the channels;
//  * shared token tiles (bf16, 64 < Q <= 128, and 32 < Q <= 64 where a CU would
//    take turns of the former): the waves share each chunk of
//    the tile and of the query in LDS and split S;
//  * wide queries (bf16, Q > 128): the waves split the query's columns, each
//    staging its own in LDS, and share the tile in LDS;
//  * channel slices (some of bf16, Q > 256): a workgroup owns up to 256 tokens
//    and a slice of channels.
#include <type_traits>

#include "wz_device.h"

namespace wz {
namespace {

constexpr int kKStep = 32;   // channels per MFMA K step (16x16x32)
constexpr int kQMax = 1024;  // validated bound on query tokens

// Per-unit outputs of the streaming pass (layouts in the workspace carve-up).
struct StreamArgs {
  const void* X;      // [T][H][W][C]
  const void* query;  // [Q][C]
  float* qg_part;
  float* sig_part;
  float* pool_part;
  float* tok_score;
  int T, N, C, Q, tiles;
  // several queries in one pass (token-tiled path): `query` holds groups x qg
  // rows (Q = groups * qg); query g's scores, column sums and norms go to the
  // buffers above advanced by g * gws bytes, its channel sums are query 0's
  int groups = 1, qg = 0;
  long long gws = 0;
};
// Channel slices (arguments that every launch would carry cost it about 0.2 us);
// with several, tok_score is left to the per-frame kernel.
struct SliceArgs : StreamArgs {
  float* s_part;
  float* g_part;
  int QP, slices;
};
static_assert(sizeof(VideoArgs<SliceArgs>) <= 4096, "per-video arguments exceed the kernel argument limit");

// bf16 dot2 helpers of the token-tiled path
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}
// Selector pairs for channel sums: dot2(x, (1, 0)) picks the low bf16 of x,
// dot2(x, (0, 1)) the high one.  They must reach the instruction in VGPRs:
// this compiler encodes the pair (1, 0) as the inline constant 1.0, which the
// hardware reads as (0, 1) for a packed bf16 operand.
constexpr uint32_t kBf16OneLo = 0x00003F80u;  // bf16 pair (1, 0)
constexpr uint32_t kBf16OneHi = 0x3F800000u;  // bf16 pair (0, 1)
// acc plus the square of a dword's channels (two bf16 or one fp32)
template <typename In>
__device__ __forceinline__ float norm_add(uint32_t v, float acc) {
  if constexpr (sizeof(In) == 2) return dot2(v, v, acc);
  else return fmaf(__uint_as_float(v), __uint_as_float(v), acc);
}
// The waves' partial sums get(0 .. WV - 1) in a fixed order: in turn, for fp32
// inputs in pairs (fewer roundings of the large sums).
template <typename In, int WV, typename Get>
__device__ __forceinline__ float wave_add(Get get) {
  float v[WV];
#pragma unroll
  for (int w = 0; w < WV; ++w) v[w] = get(w);
  if constexpr (sizeof(In) == 2) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < WV; ++w) s += v[w];
    return s;
  } else {
#pragma unroll
    for (int d = 1; d < WV; d *= 2)
#pragma unroll
      for (int w = 0; w < WV; w += 2 * d) v[w] += v[w + d];
    return v[0];
  }
}
// acc[i][n] += the 16-row tiles A[i] times the 16-column tiles B[n] over the
// 16-byte units that lane (row or column lane % 16, K group lane / 16) holds:
// bf16, one MFMA over 32 channels; fp32, four over four channels each, MFMA e
// taking element e of every lane's unit (the same channels of both operands),
// so fp32 products are exact to fp32 rounding as on the vector ALU.
template <typename In, int MT, int NT>
__device__ __forceinline__ void mfma_units(const u32x4 (&A)[MT], const u32x4 (&B)[NT], f32x4 (&acc)[MT][NT]) {
  if constexpr (sizeof(In) == 2) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int i = 0; i < MT; ++i)
        acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[i]),
                                                            __builtin_bit_cast(bf16x8, B[n]), acc[i][n], 0, 0, 0);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int i = 0; i < MT; ++i)
          acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(A[i][e]), __uint_as_float(B[n][e]),
                                                           acc[i][n], 0, 0, 0);
  }
}

// ---------------------------------------------------------------------------
// Channel slices (bf16, Q > 256 where wide_takes_slices says)
// ---------------------------------------------------------------------------
// A workgroup owns up to 256 tokens of a frame (whole frames up to H*W = 256,
// so the query is read about once per frame) and a slice of at most 1024
// channels, so that a few frames with long rows fill the chip; each wave holds
// two 16-row tiles, loads X straight into the MFMA A layout and runs, per
// 32-channel step, S += X Q^T (the query slice staged in LDS, 16 NTG columns a
// pass), G += X X^T (diagonal: |x|^2) and P = X I (identity columns: the
// step's channel sums).  One wave a step adds the query's Gram matrix (diagonal:
// |q_j|^2).  With one slice the workgroup finishes its tokens' a_{t,n}; with
// several it writes the partial x . q_j and |x|^2, which the per-frame kernel
// adds in slice order.
// NTG: 16-column query tiles per pass over the slice (queries of more tokens
// take several passes); R: depth of the X prefetch ring in 32-channel steps.
template <int NTG, int R>
__global__ __launch_bounds__(kMaxWaves / kTilesPerWave * 64) void k_relevance_slices(
    int tile_tokens, int kc, const VideoArgs<SliceArgs> va) {
  const SliceArgs f = va.v[blockIdx.y];
  const uint16_t* __restrict__ X = static_cast<const uint16_t*>(f.X);
  const uint16_t* __restrict__ query = static_cast<const uint16_t*>(f.query);
  constexpr int MTW = kTilesPerWave;
  constexpr int MAXW = kMaxWaves / MTW;
  constexpr int QB = 8;                          // query units staged per thread per batch
  __shared__ u32x4 s_q[kSliceSteps][NTG][kWave];  // the group's query slice, MFMA B layout
  __shared__ float s_poolw[MAXW][kSliceSteps * kKStep];  // per-wave channel sums of the slice
  __shared__ float s_colw[MAXW][NTG * 16];       // per-wave column sums of S
  __shared__ float s_qgw[MAXW][NTG * 16];        // per-wave |q_j|^2 partials
  __shared__ float s_xt[kMaxWaves * 16];         // |x| of the tile's tokens (one slice)
  __shared__ float s_rq[kQMax];                 // 1/|q_j| (one slice)

  int t, tile, sl;
  slice_of_block(blockIdx.x, f.tiles, f.slices, t, tile, sl);
  if (t >= f.T) return;
  const int N = f.N, C = f.C, Q = f.Q, QP = f.QP, S = f.slices;
  const int tok0 = tile * tile_tokens;
  const int TM = min(tile_tokens, N - tok0);
  const int tid = threadIdx.x, nthreads = blockDim.x;
  // wave index in a scalar register: branches on it must be scalar branches,
  // since an MFMA under an exec mask still updates every lane
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nthreads >> 6;
  const int row = lane & 15, grp = lane >> 4;
  const int c_lo = sl * kc, c_hi = min(C, c_lo + kc);
  const int kper = (c_hi - c_lo + kKStep - 1) / kKStep;  // <= kSliceSteps

  const __amdgpu_buffer_rsrc_t xres = make_rsrc(X + (size_t(t) * N + tok0) * C, uint32_t(TM) * C * 2);
  const __amdgpu_buffer_rsrc_t qres = make_rsrc(query, uint32_t(Q) * C * 2);
  int xoff[MTW];  // byte offsets of this lane's token rows (A operands) in the tile
#pragma unroll
  for (int i = 0; i < MTW; ++i) {
    const int r = (wave * MTW + i) * 16 + row;
    xoff[i] = r < TM ? r * C * 2 : kOOB;
  }

  // identity operands: slot e of the lane with column `row`, K group `grp`
  // holds channel 8*grp + e of the step; I_s selects channel 16*s + column
  bf16x8 I0, I1;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    I0[e] = (__bf16)((8 * grp + e == row) ? 1.0f : 0.0f);
    I1[e] = (__bf16)((8 * grp + e == 16 + row) ? 1.0f : 0.0f);
  }

  f32x4 G[MTW];
  float best[MTW][4];  // rows 16*(wave*MTW+i) + 4*grp + e (one slice only)
#pragma unroll
  for (int i = 0; i < MTW; ++i) {
    G[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) best[i][e] = -INFINITY;
  }
  const int groups = (Q + NTG * 16 - 1) / (NTG * 16);

  bf16x8 a[R][MTW];  // X prefetch ring: slot r holds the steps ks = r (mod R)
  auto issue = [&](int ks, bf16x8 (&dst)[MTW]) {
    const int c = c_lo + ks * kKStep + grp * 8;
    const bool ok = ks < kper && c < c_hi;
#pragma unroll
    for (int i = 0; i < MTW; ++i) dst[i] = buf_load_bf16x8(xres, ok ? xoff[i] + c * 2 : kOOB);
  };

  for (int g = 0; g < groups; ++g) {
    const int qg0 = g * NTG * 16;
    f32x4 Sacc[MTW][NTG], QG[NTG];
#pragma unroll
    for (int n = 0; n < NTG; ++n) {
      QG[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < MTW; ++i) Sacc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // X ring first, then the query slice of the group into LDS: unit
    // u -> step u / (64 NTG), tile (u / 64) % NTG, lane u % 64
#pragma unroll
    for (int r = 0; r < R; ++r) issue(r, a[r]);
    const int qunits = kper * NTG * kWave;
    for (int u0 = 0; u0 < qunits; u0 += QB * nthreads) {
      u32x4 qv[QB];
#pragma unroll
      for (int k = 0; k < QB; ++k) {
        const int u = u0 + tid + k * nthreads;
        const int l = u & 63, n = (u >> 6) % NTG, ks = u / (NTG * kWave);
        const int j = qg0 + n * 16 + (l & 15);
        const int c = c_lo + ks * kKStep + (l >> 4) * 8;
        const bool ok = u < qunits && j < Q && c < c_hi;
        qv[k] = buf_load_u32x4(qres, ok ? (j * C + c) * 2 : kOOB);
      }
#pragma unroll
      for (int k = 0; k < QB; ++k) {
        const int u = u0 + tid + k * nthreads;
        if (u < qunits) s_q[u / (NTG * kWave)][(u >> 6) % NTG][u & 63] = qv[k];
      }
    }
    __syncthreads();

    auto compute = [&](int ks, const bf16x8 (&x)[MTW], auto pool) {
      bf16x8 b[NTG];
#pragma unroll
      for (int n = 0; n < NTG; ++n) b[n] = __builtin_bit_cast(bf16x8, s_q[ks][n][lane]);
#pragma unroll
      for (int n = 0; n < NTG; ++n)
#pragma unroll
        for (int i = 0; i < MTW; ++i)
          Sacc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i], b[n], Sacc[i][n], 0, 0, 0);
      if (ks % nw == wave) {
        // query Gram matrix of the step (diagonal: |q_j|^2), spread over the waves
#pragma unroll
        for (int n = 0; n < NTG; ++n) QG[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[n], b[n], QG[n], 0, 0, 0);
      }
      if constexpr (decltype(pool)::value) {
        f32x4 P0 = {0.f, 0.f, 0.f, 0.f}, P1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < MTW; ++i) {
          G[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i], x[i], G[i], 0, 0, 0);
          P0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i], I0, P0, 0, 0, 0);
          P1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i], I1, P1, 0, 0, 0);
        }
        float v0 = (P0[0] + P0[1]) + (P0[2] + P0[3]);
        float v1 = (P1[0] + P1[1]) + (P1[2] + P1[3]);
        v0 = row_sum4(v0);
        v1 = row_sum4(v1);
        // lanes 0-15: channels 32ks+0..15 of the slice, lanes 16-31: 32ks+16..31
        if (lane < 32) s_poolw[wave][ks * kKStep + lane] = lane < 16 ? v0 : v1;
      }
    };
    // Steps 2s and 2s+1 read the two 64-byte halves of the same 128-byte
    // line of each row, so they are consumed and re-issued as a pair: the
    // second request of a line then finds the first one's miss in flight
    // instead of a line the cache may have evicted meanwhile.
    static_assert(R % 2 == 0, "the ring advances in pairs of steps");
    auto run = [&](auto pool) {
      for (int ks0 = 0; ks0 < kper; ks0 += R) {
#pragma unroll
        for (int r = 0; r < R; r += 2) {
          const int ks = ks0 + r;
          if (ks < kper) compute(ks, a[r], pool);
          if (ks + 1 < kper) compute(ks + 1, a[r + 1], pool);
          issue(ks + R, a[r]);
          issue(ks + 1 + R, a[r + 1]);
        }
      }
    };
    if (g == 0) run(std::true_type{});
    else run(std::false_type{});
    __syncthreads();

    // ---- group epilogue ----
    const bool diag = (row >> 2) == grp;  // lane holds element (row, row) of a 16x16 tile
    if (diag) {
#pragma unroll
      for (int n = 0; n < NTG; ++n) s_qgw[wave][n * 16 + row] = QG[n][row & 3];
    }
#pragma unroll
    for (int n = 0; n < NTG; ++n) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < MTW; ++i) v += (Sacc[i][n][0] + Sacc[i][n][1]) + (Sacc[i][n][2] + Sacc[i][n][3]);
      v = row_sum4(v);
      if (lane < 16) s_colw[wave][n * 16 + lane] = v;
    }
    if (g == 0) {
      const __amdgpu_buffer_rsrc_t gres = make_rsrc(f.g_part + (size_t(t) * S + sl) * N, S > 1 ? uint32_t(N) * 4 : 0u);
      if (diag) {
#pragma unroll
        for (int i = 0; i < MTW; ++i) {
          const int r = (wave * MTW + i) * 16 + row;
          const float gg = G[i][row & 3];
          if (S == 1) s_xt[r] = sqrtf(gg);
          else buf_store_f32(gg, gres, r < TM ? (tok0 + r) * 4 : kOOB);
        }
      }
      // the slice's channel sums, waves added in order
      const __amdgpu_buffer_rsrc_t pres =
          make_rsrc(f.pool_part + (size_t(t) * f.tiles + tile) * C, uint32_t(C) * 4);
      for (int c = tid; c < kper * kKStep; c += nthreads) {
        float s = 0.f;
        for (int w = 0; w < nw; ++w) s += s_poolw[w][c];
        buf_store_f32(s, pres, c_lo + c < c_hi ? (c_lo + c) * 4 : kOOB);
      }
    }
    __syncthreads();
    if (tid < NTG * 16) {
      const int j = qg0 + tid;
      float qq = 0.f, sg = 0.f;
      for (int w = 0; w < nw; ++w) {
        qq += s_qgw[w][tid];
        sg += s_colw[w][tid];
      }
      if (j < Q) {
        if (S == 1) s_rq[j] = qq > 0.f ? 1.0f / sqrtf(qq) : 0.f;
        if (tile == 0) f.qg_part[(size_t(t) * S + sl) * Q + j] = qq;
        f.sig_part[((size_t(t) * f.tiles + tile) * S + sl) * Q + j] = sg;
      }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t sres =
        make_rsrc(f.s_part + (size_t(t) * S + sl) * N * QP, S > 1 ? uint32_t(N) * QP * 4 : 0u);
#pragma unroll
    for (int n = 0; n < NTG; ++n) {
      const int j = qg0 + n * 16 + row;  // this lane's column
      if (S == 1) {
        const float rq = j < Q ? s_rq[j] : 0.f;
#pragma unroll
        for (int i = 0; i < MTW; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) best[i][e] = fmaxf(best[i][e], j < Q ? Sacc[i][n][e] * rq : -INFINITY);
      } else {
#pragma unroll
        for (int i = 0; i < MTW; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = (wave * MTW + i) * 16 + 4 * grp + e;
            buf_store_f32(Sacc[i][n][e], sres, (r < TM && j < Q) ? ((tok0 + r) * QP + j) * 4 : kOOB);
          }
      }
    }
  }

  if (S == 1) {
    // max over the 16 columns held by the lanes of this K group
#pragma unroll
    for (int i = 0; i < MTW; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) best[i][e] = fmaxf(best[i][e], __shfl_xor(best[i][e], m, kWave));
    if (row == 0) {
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = (wave * MTW + i) * 16 + 4 * grp + e;
          if (r < TM) {
            const float xn = s_xt[r];
            f.tok_score[size_t(t) * N + tok0 + r] = xn > 0.f ? best[i][e] / xn : 0.f;
          }
        }
    }
  }
}

// ---------------------------------------------------------------------------
// Token-tiled path (fp32 inputs; bf16, Q <= 64 and some of 128 < Q <= 256)
// ---------------------------------------------------------------------------
// (Described for bf16 inputs; an fp32 chunk is 32 channels, the same bytes,
// and its S runs on v_mfma_f32_16x16x4_f32.  Bound for fp32: HBM up to about
// 48 query tokens, above that the fp32 MFMA rate, a sixteenth of bf16's (T =
// 64, 14x14, C = 3584, Q = 32: 49 us for 187 MB of HBM traffic, MFMA busy 47 %
// of the cycles, vector ALU 25 %, LDS 14 %).  It
// replaced one wave per token on the vector ALU, which read the whole query
// from L2 for every token: T = 64, 14x14, C = 3584, Q = 32: 824 -> 51 us; T =
// 8, 24x24, C = 2504, Q = 96: 1219 -> 56 us.)
// A workgroup owns one tile of at most 64 tokens of one frame with ALL its
// channels, so a_{t,n} is final here and no per-slice partial scores are
// written; its tokens are one contiguous stretch of X.  The W waves (eight;
// four for one pass of two query tiles with the channel sums in LDS, where
// that measured faster) split the channels into 64-channel chunks (wave w
// takes chunks w, w + W, ...) and never wait for each other until the
// epilogue.  Per chunk a wave
//   1. loads the tile's rows and the query's rows for the chunk (8 rows x 128
//      bytes per instruction, whole cache lines; the query is L2-resident);
//   2. stores both to its own LDS buffers (16-byte units XOR-swizzled by row)
//      and, from the same registers, accumulates |x|^2, |q_j|^2 and the
//      chunk's channel sums with bf16 dot2 instructions; the channel sums are
//      reduced across the wave by DPP and lane swaps and gathered in LDS;
//   3. runs two 32-channel steps of S += X Q^T (v_mfma_f32_16x16x32_bf16) on
//      the tile's one to four 16-row tiles, reading both operands from its
//      buffers;
//   4. re-issues the ring slot for the chunk after next.
// In the epilogue each wave first reduces its own accumulator rows to
// sigma_j (lane swaps); then the waves' partial S, |x|^2, |q_j|^2 and sigma_j
// are added in wave order through LDS (two barriers), a_{t,n} = max_j S_nj /
// (|q_j| |x_n|) is formed, and the tile's channel sums leave in one coalesced
// store.
constexpr int kTokWaves = 8;
constexpr int kTokChunk = 64;      // channels per chunk (128 bytes of a bf16 row; 32 fp32 channels)
constexpr int kTokPoolMax = 8192;  // channels whose sums are gathered in LDS
constexpr size_t kTokLdsMax = 160 * 1024;  // LDS of a workgroup
// Rows a wave stages for tiles of up to 8 * ipc tokens: whole 16-row MFMA
// tiles (one to four).
constexpr int tok_rows(int ipc) { return (ipc + 1) / 2 * 16; }

// POOL: the tile's channel sums are gathered in LDS (C <= kTokPoolMax) and
// stored once at the end; otherwise a few lanes store them chunk by chunk.
// MODE kTokOne: one pass over the tile for every query column;
// kTokGroups: the query columns are f.groups queries of f.qg tokens each,
// a_{t,n} taken per query; kTokPasses: queries of more than NQ tokens, one
// pass over the tile per NQ query rows (its later reads mostly from cache),
// a_{t,n} the maximum over the passes, the channel sums taken in the first.
enum TokMode { kTokOne = 0, kTokGroups = 1, kTokPasses = 2 };
// WV: the workgroup's waves.
template <typename In, int NTG, int IPC, bool POOL, int MODE, int WV = kTokWaves>
__global__ __launch_bounds__(WV * 64) void k_relevance_tok(int tile_tokens, const VideoArgs<StreamArgs> va) {
  // A tile's MFMAs, operand reads and staging cover the 16-row tiles it has
  // tokens in, not the 64 rows a tile may hold, and the channel sums take the
  // LDS of the C at hand: short clips, split into tiles of 13 to 32 tokens to
  // fill the chip, did two to four times the contraction's work on rows of
  // zeros, one workgroup to a CU.  Four videos of T = 16 (14x14, C = 3584, Q =
  // 24) a call: 61.4 -> 47.5 us; T = 32, Q = 16: 25.5 -> 24.9 us.
  constexpr int RT = tok_rows(IPC) / 16;
  constexpr int kTokRows = 16 * RT;
  constexpr int kTokRowsPerThread = (kTokRows * 8 + WV * kWave - 1) / (WV * kWave);  // epilogue rows of a thread (8 threads a row)
  const StreamArgs f = va.v[blockIdx.y];
  const In* __restrict__ X = static_cast<const In*>(f.X);
  const In* __restrict__ query = static_cast<const In*>(f.query);
  constexpr bool BF = sizeof(In) == 2;
  constexpr int ES = int(sizeof(In));  // bytes of a channel
  constexpr int CH = 128 / ES;         // channels per chunk
  constexpr int CU = 16 / ES;          // channels per 16-byte unit
  constexpr int NQ = NTG * 16;  // query rows of the accumulators
  constexpr int QI = NQ / 8;    // query load instructions per chunk
  // chunks of loads in flight per wave: two (eight waves keep 16 chunks of
  // the tile in flight; deeper rings measured slower)
  constexpr int D = 2;
  // per-wave chunk buffers (16-byte units swizzled by row): the first kTokRows
  // rows of a wave's region stage its tile rows, the next NQ its query rows;
  // after the loop the region holds the wave's partial S [kTokRows][NQ] floats
  __shared__ __align__(16) u32x4 s_xq[WV][kTokRows + NQ][8];
  extern __shared__ __align__(16) float s_pool[];  // [C] (POOL)
  __shared__ float s_xx[WV][kTokRows];
  __shared__ float s_qq[WV][NQ];
  __shared__ float s_rq[NQ];
  __shared__ float s_sig[WV][NQ];  // per-wave column sums of S

  int t, tile;
  unit_of_block(blockIdx.x, f.tiles, t, tile);
  if (t >= f.T) return;
  const int N = f.N, C = f.C, Q = f.Q;
  const int tok0 = tile * tile_tokens;
  const int TM = min(tile_tokens, N - tok0);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, grp = lane >> 4;  // MFMA layout: row / column, K group
  const int lr = lane >> 3, lu = lane & 7;     // load layout: row lr of each 8-row group, 16-byte unit lu
  const int nch = (C + CH - 1) / CH;

  const __amdgpu_buffer_rsrc_t xres = make_rsrc_uniform(X + (size_t(t) * N + tok0) * C, uint32_t(TM) * C * ES);
  constexpr bool GR = MODE == kTokGroups;
  const int npass = MODE == kTokPasses ? (Q + NQ - 1) / NQ : 1;
  float best_all[kTokRowsPerThread];
#pragma unroll
  for (int k = 0; k < kTokRowsPerThread; ++k) best_all[k] = -INFINITY;
  for (int h = 0; h < npass; ++h) {
    const int qb = h * NQ, Qh = min(NQ, Q - qb);
    const bool sums = h == 0;
    const __amdgpu_buffer_rsrc_t qres = make_rsrc_uniform(query + size_t(qb) * C, uint32_t(Qh) * C * ES);

    // ring slot: the tile's rows 8k + lr and the query's rows 8k + lr, unit lu
    // of the chunk; chunks past the end, rows past the tile or the query and
    // channels past C read zeros
    struct Slot {
      u32x4 x[IPC];
      u32x4 q[QI];
    };
    // (query rows past Qh lie past the end of qres and read zeros; a per-lane
    // row test here would become a branch around the load)
    auto issue = [&](int c, Slot& d) {
      const int cc = c * CH + CU * lu;
      const bool ok = c < nch && cc < C;
#pragma unroll
      for (int k = 0; k < IPC; ++k) d.x[k] = buf_load_u32x4(xres, ok ? (8 * k + lr) * C * ES + cc * ES : kOOB);
#pragma unroll
      for (int k = 0; k < QI; ++k) d.q[k] = buf_load_u32x4(qres, ok ? (8 * k + lr) * C * ES + cc * ES : kOOB);
    };

    f32x4 Sacc[RT][NTG];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int n = 0; n < NTG; ++n) Sacc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    float xx[IPC], qq[QI];
#pragma unroll
    for (int k = 0; k < IPC; ++k) xx[k] = 0.f;
#pragma unroll
    for (int k = 0; k < QI; ++k) qq[k] = 0.f;
    uint32_t one_lo = kBf16OneLo, one_hi = kBf16OneHi;
    asm volatile("" : "+v"(one_lo), "+v"(one_hi));  // opaque: keeps them out of inline constants
    float* pool = POOL ? s_pool : f.pool_part + (size_t(t) * f.tiles + tile) * C;

    auto consume = [&](int c, const Slot& d) {
      // rows to LDS; |x|^2, |q_j|^2 and channel sums from the registers
      float cs[CU];
#pragma unroll
      for (int e = 0; e < CU; ++e) cs[e] = 0.f;
#pragma unroll
      for (int k = 0; k < IPC; ++k) {
        const int row = 8 * k + lr;
        const u32x4 v = d.x[k];
        s_xq[wave][row][lu ^ (row & 7)] = v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          xx[k] = norm_add<In>(v[e], xx[k]);
          if constexpr (BF) {
            cs[2 * e] = dot2(v[e], one_lo, cs[2 * e]);
            cs[2 * e + 1] = dot2(v[e], one_hi, cs[2 * e + 1]);
          } else {
            cs[e] += __uint_as_float(v[e]);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < QI; ++k) {
        const int row = 8 * k + lr;
        const u32x4 v = d.q[k];
        s_xq[wave][kTokRows + row][lu ^ (row & 7)] = v;
#pragma unroll
        for (int e = 0; e < 4; ++e) qq[k] = norm_add<In>(v[e], qq[k]);
      }
      // channel sums over the wave's rows (lanes lu, lu + 8, ..., lu + 56, in a
      // fixed order): lane 8 lr + lu ends with unit lu's channel lr (fp32: lr % 4)
      const float cw = lane_transpose_sum(cs);
      const int c0 = c * CH + CU * lu;
      if (sums && c0 < C && lr < CU) pool[c0 + lr] = cw;
    };
    // 16-byte unit 4 st + grp of a staged row (16-row tiles start at multiples of 8 rows)
    auto unit = [&](int row, int st) { return s_xq[wave][row][(4 * st + grp) ^ (row & 7)]; };
    auto contract = [&]() {
      if constexpr (BF) {
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          u32x4 A[RT], B[NTG];
#pragma unroll
          for (int i = 0; i < RT; ++i) A[i] = unit(16 * i + r16, st);
#pragma unroll
          for (int n = 0; n < NTG; ++n) B[n] = unit(kTokRows + 16 * n + r16, st);
          mfma_units<In, RT, NTG>(A, B, Sacc);
        }
      } else {
        // fp32 inputs: half a chunk's products are summed from zero and added
        // to the wave's sums once (chains of 16 products, then of the wave's
        // half chunks): one chain of C / 8 products would round more often
        // than the C / 64 of a lane-wise dot product.  At most two column
        // tiles at a time, so that the partial sums fit the registers.
        constexpr int NB = NTG < 2 ? NTG : 2;
#pragma unroll
        for (int n0 = 0; n0 < NTG; n0 += NB)
#pragma unroll
          for (int st = 0; st < 2; ++st) {
            u32x4 A[RT], B[NB];
            f32x4 part[RT][NB];
#pragma unroll
            for (int i = 0; i < RT; ++i) A[i] = unit(16 * i + r16, st);
#pragma unroll
            for (int n = 0; n < NB; ++n) B[n] = unit(kTokRows + 16 * (n0 + n) + r16, st);
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
              for (int n = 0; n < NB; ++n) part[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
            mfma_units<In, RT, NB>(A, B, part);
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
              for (int n = 0; n < NB; ++n) Sacc[i][n0 + n] += part[i][n];
          }
      }
    };

    // rows this wave never loads (8 * IPC .. kTokRows - 1) are zero in its buffer
    for (int u = 8 * IPC * 8 + lane; u < kTokRows * 8; u += kWave) (&s_xq[wave][0][0])[u] = u32x4{0u, 0u, 0u, 0u};

    // A ring of D slots: the wave's chunks c, c + 8, ..., c + 8 (D - 1) are in
    // flight while it works on the oldest.  The loads are issued in slot
    // order before and in the loop, and the norms' updates are pinned before
    // a slot's reload: otherwise the slot needs a second register set and a
    // copy at the end of the loop, and the compiler waits for the whole ring
    // once per iteration.
    auto pin = [&]() {
#pragma unroll
      for (int k = 0; k < IPC; ++k) asm volatile("" : "+v"(xx[k]));
#pragma unroll
      for (int k = 0; k < QI; ++k) asm volatile("" : "+v"(qq[k]));
    };
    Slot ring[D];
#pragma unroll
    for (int s = 0; s < D; ++s) {
      issue(wave + s * WV, ring[s]);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int c0 = wave; c0 < nch; c0 += D * WV) {
#pragma unroll
      for (int s = 0; s < D; ++s) {
        const int c = c0 + s * WV;
        __builtin_amdgcn_sched_barrier(0);
        if (c < nch) {
          consume(c, ring[s]);
          pin();
          contract();
        }
        issue(c + D * WV, ring[s]);
      }
    }

    // ---- epilogue: waves added in order; LDS-only barriers, so nothing waits
    // for outstanding global accesses ----
    auto row8_sum = [](float v) {  // the 8 lanes of a load-layout row
      v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0xB1, 0xF, 0xF, false));   // lane ^ 1
      v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x4E, 0xF, 0xF, false));   // lane ^ 2
      v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x141, 0xF, 0xF, false));  // 7 - i in 8
      return v;
    };
#pragma unroll
    for (int k = 0; k < IPC; ++k) {
      const float v = row8_sum(xx[k]);
      if (lu == 0) s_xx[wave][8 * k + lr] = v;
    }
    for (int r = 8 * IPC + lane; r < kTokRows; r += kWave) s_xx[wave][r] = 0.f;
#pragma unroll
    for (int k = 0; k < QI; ++k) {
      const float v = row8_sum(qq[k]);
      if (lu == 0) s_qq[wave][8 * k + lr] = v;
    }
    // sigma_j of the wave: its accumulator column j = 16 n + r16 summed over the
    // wave's rows (rows past the tile hold zeros), the four lane groups by
    // lane swaps
#pragma unroll
    for (int n = 0; n < NTG; ++n) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        if constexpr (BF) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v += Sacc[i][n][e];
        } else {
          v += (Sacc[i][n][0] + Sacc[i][n][1]) + (Sacc[i][n][2] + Sacc[i][n][3]);
        }
      }
      const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
      v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
      const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
      v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
      if (lane < 16) s_sig[wave][16 * n + r16] = v;
    }
    // wave w's partial S sits in its own region: [row][NQ] floats from &s_xq[w][0][0]
    static_assert((kTokRows + NQ) * 8 * 16 >= kTokRows * NQ * 4, "partial S fits the wave's region");
    auto s_part = [&](int w, int r, int j) -> float& { return reinterpret_cast<float*>(&s_xq[w][0][0])[r * NQ + j]; };
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int n = 0; n < NTG; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) s_part(wave, 16 * i + 4 * grp + e, 16 * n + r16) = Sacc[i][n][e];
    lds_barrier();  // every sum below reads the waves' partials in wave order
    if (tid < Qh) {
      const float v = wave_add<In, WV>([&](int w) { return s_sig[w][tid]; });
      const float qv = wave_add<In, WV>([&](int w) { return s_qq[w][tid]; });
      if constexpr (GR) {
        const int g = tid / f.qg, j = tid - g * f.qg;
        advance(f.sig_part, g * f.gws)[(size_t(t) * f.tiles + tile) * f.qg + j] = v;
        if (tile == 0) advance(f.qg_part, g * f.gws)[size_t(t) * f.qg + j] = qv;
      } else {
        f.sig_part[(size_t(t) * f.tiles + tile) * Q + qb + tid] = v;
        if (tile == 0) f.qg_part[size_t(t) * Q + qb + tid] = qv;
      }
    }
    if (tid < NQ) {
      const float qv = wave_add<In, WV>([&](int w) { return s_qq[w][tid]; });
      s_rq[tid] = qv > 0.f ? 1.0f / sqrtf(qv) : 0.f;
    }
    // thread -> rows tid / 8 + RS k (k < kTokRowsPerThread), columns CPT * (tid % 8) .. + CPT - 1;
    // every row's partials are read before the first barrier (the query maxima below reuse wave 0's region)
    constexpr int CPT = NQ / 8;
    constexpr int RS = WV * kWave / 8;  // rows the threads cover at once
    const int cg = (tid & 7) * CPT;
    float sv[kTokRowsPerThread][CPT], x2[kTokRowsPerThread];
#pragma unroll
    for (int k = 0; k < kTokRowsPerThread; ++k) {
      // (threads past the last row repeat it; their results are not written)
      const int row = min((tid >> 3) + RS * k, kTokRows - 1);
#pragma unroll
      for (int e = 0; e < CPT; ++e) {
        sv[k][e] = wave_add<In, WV>([&](int w) { return s_part(w, row, cg + e); });
      }
      x2[k] = wave_add<In, WV>([&](int w) { return s_xx[w][row]; });
    }
    lds_barrier();  // 1 / |q_j| in s_rq
    float rq[CPT];
#pragma unroll
    for (int e = 0; e < CPT; ++e) rq[e] = s_rq[cg + e];
    if constexpr (GR) {
      // the rows' S_nj / |q_j| into LDS (wave 0's region: every read of the
      // partials is behind the last barrier); thread g of a row's eight takes
      // the maximum over query g's columns
      float* s_cos = reinterpret_cast<float*>(&s_xq[0][0][0]);  // [kTokRows][NQ]
#pragma unroll
      for (int k = 0; k < kTokRowsPerThread; ++k)
        if ((tid >> 3) + RS * k < kTokRows) {
#pragma unroll
          for (int e = 0; e < CPT; ++e) s_cos[((tid >> 3) + RS * k) * NQ + cg + e] = sv[k][e] * rq[e];
        }
      lds_barrier();
      const int g = tid & 7;
#pragma unroll
      for (int k = 0; k < kTokRowsPerThread; ++k) {
        const int row = (tid >> 3) + RS * k;
        if (g < f.groups && row < TM) {
          float best = -INFINITY;
          for (int j = 0; j < f.qg; ++j) best = fmaxf(best, s_cos[row * NQ + g * f.qg + j]);
          const float xn = sqrtf(x2[k]);
          advance(f.tok_score, g * f.gws)[size_t(t) * N + tok0 + row] = xn > 0.f ? best / xn : 0.f;
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < kTokRowsPerThread; ++k) {
        const int row = (tid >> 3) + RS * k;
        float best = -INFINITY;
#pragma unroll
        for (int e = 0; e < CPT; ++e)
          if (cg + e < Qh) best = fmaxf(best, sv[k][e] * rq[e]);
        best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0xB1, 0xF, 0xF, false)));
        best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x4E, 0xF, 0xF, false)));
        best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x141, 0xF, 0xF, false)));
        best_all[k] = fmaxf(best_all[k], best);
        if (h == npass - 1 && (tid & 7) == 0 && row < TM) {
          const float xn = sqrtf(x2[k]);
          f.tok_score[size_t(t) * N + tok0 + row] = xn > 0.f ? best_all[k] / xn : 0.f;
        }
      }
    }
    if (h + 1 < npass) lds_barrier();  // the next pass rewrites every wave's region
  }

  if (POOL) {
    const __amdgpu_buffer_rsrc_t pres =
        make_rsrc_uniform(f.pool_part + (size_t(t) * f.tiles + tile) * C, uint32_t(C) * 4);
    for (int c4 = tid; c4 < C / 4; c4 += WV * kWave)
      buf_store_wt_b128(reinterpret_cast<const u32x4*>(s_pool)[c4], pres, c4 * 16);
  }
}

// ---------------------------------------------------------------------------
// Workgroup-shared token tiles (bf16, 64 < Q <= 128; 32 < Q <= 64 by relevance_kind's rule)
// ---------------------------------------------------------------------------
// With a wide query, per-wave channel stripes (above) would stage the query
// once per wave and add every wave's partial S through LDS.  Here the eight
// waves of a workgroup share each 64-channel chunk: the tile's rows (up to
// 64 * RTW tokens) and the query's 64 NTW rows are loaded once per workgroup
// (one 16-byte unit per thread and row group, whole cache lines), staged in a
// double-buffered LDS stage (16-byte units XOR-swizzled by row), and the
// waves tile S as 2 row groups x 4 column groups: wave (wr, wc) contracts
// 16-row tiles wr * 2 RTW .. wr * 2 RTW + 2 RTW - 1 against 16-column tiles
// NTW wc .. NTW wc + NTW - 1.  |x|^2, |q_j|^2 and the chunk's channel sums come
// from the load registers (bf16 dot2), the channel sums added over the waves in
// wave order through LDS.  One LDS-only barrier per chunk; D chunks of loads in
// flight in registers.  The row maxima and column sums of S are combined
// across the waves through LDS at the end, in a fixed order.  Two
// workgroups share a CU.  Bound: the barrier a chunk and the vector ALU's norms
// and channel sums (counters at T = 256, 27x27, C = 1152, Q = 128, 111.5 us: vector
// ALU 45 % of the cycles, LDS 31 %, MFMA 23 %, 446 MB of HBM traffic; T = 96, Q =
// 48, 48.4 us: 56 %, 27 %, 9 %, 168 MB).
constexpr int kWgWaves = 8;

template <int RTW, int NTW>
__global__ __launch_bounds__(kWgWaves * 64, 2) void k_relevance_wg(int tile_tokens, const VideoArgs<StreamArgs> va) {
  const StreamArgs f = va.v[blockIdx.y];
  constexpr int RT = 64 * RTW;                 // tile rows the stage holds
  constexpr int NQ = 64 * NTW;                 // query rows the stage holds
  constexpr int MTW = 2 * RTW;                 // 16-row tiles per wave
  constexpr int XR = RT / 64;                  // tile rows each thread loads per chunk
  constexpr int QR = NQ / 64;                  // query rows each thread loads per chunk
  constexpr int D = 2 + (RTW == 1);            // chunks of loads in flight
  __shared__ __align__(16) u32x4 s_x[2][RT][8];
  __shared__ __align__(16) u32x4 s_q[2][NQ][8];
  __shared__ __align__(16) float s_pp[2][kWgWaves][kTokChunk];  // per-wave channel sums of a chunk
  __shared__ float s_xx[RT];
  __shared__ float s_qq[NQ];
  __shared__ float s_sig[2][NQ];    // column sums of S per row group
  __shared__ float s_best[4][RT];   // row maxima of S_nj / |q_j| per column group

  int t, tile;
  unit_of_block(blockIdx.x, f.tiles, t, tile);
  if (t >= f.T) return;
  const uint16_t* __restrict__ X = static_cast<const uint16_t*>(f.X);
  const uint16_t* __restrict__ query = static_cast<const uint16_t*>(f.query);
  const int N = f.N, C = f.C, Q = f.Q;
  const int tok0 = tile * tile_tokens;
  const int TM = min(tile_tokens, N - tok0);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 2, wc = wave & 3;     // row group, column group
  const int r16 = lane & 15, grp = lane >> 4;  // MFMA layout: row / column, K group
  const int rb = tid >> 3, lu = tid & 7;       // load layout: rows rb + 64 k, 16-byte unit lu
  const int nch = (C + kTokChunk - 1) / kTokChunk;

  const __amdgpu_buffer_rsrc_t xres = make_rsrc_uniform(X + (size_t(t) * N + tok0) * C, uint32_t(TM) * C * 2);
  const __amdgpu_buffer_rsrc_t qres = make_rsrc_uniform(query, uint32_t(Q) * C * 2);
  const __amdgpu_buffer_rsrc_t pres =
      make_rsrc_uniform(f.pool_part + (size_t(t) * f.tiles + tile) * C, uint32_t(C) * 4);

  struct Slot {
    bf16x8 x[XR];
    bf16x8 q[QR];
  };
  // chunk c's units; chunks past the end, rows past the tile or the query
  // and channels past C read zeros (query rows past Q <= NQ lie past the end
  // of qres; a per-lane row test here would become a branch around the load)
  auto issue = [&](int c, Slot& d) {
    const int cc = c * kTokChunk + 8 * lu;
    const bool ok = c < nch && cc < C;
#pragma unroll
    for (int k = 0; k < XR; ++k) d.x[k] = buf_load_bf16x8(xres, ok ? (rb + 64 * k) * C * 2 + cc * 2 : kOOB);
#pragma unroll
    for (int k = 0; k < QR; ++k) d.q[k] = buf_load_bf16x8(qres, ok ? (rb + 64 * k) * C * 2 + cc * 2 : kOOB);
  };

  f32x4 Sacc[MTW][NTW];
#pragma unroll
  for (int i = 0; i < MTW; ++i)
#pragma unroll
    for (int n = 0; n < NTW; ++n) Sacc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float xx[XR], qq[QR];
#pragma unroll
  for (int k = 0; k < XR; ++k) xx[k] = 0.f;
#pragma unroll
  for (int k = 0; k < QR; ++k) qq[k] = 0.f;
  // with one column tile a wave, sums of products run in chains of D chunks,
  // added up in second accumulators (as short as the channel stripes' chains)
  constexpr bool CHAIN = NTW == 1;
  f32x4 Ssum[CHAIN ? MTW : 1];
  float xsum[XR], qsum[QR];
  if constexpr (CHAIN) {
#pragma unroll
    for (int i = 0; i < MTW; ++i) Ssum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < XR; ++k) xsum[k] = 0.f;
#pragma unroll
    for (int k = 0; k < QR; ++k) qsum[k] = 0.f;
  }
  uint32_t one_lo = kBf16OneLo, one_hi = kBf16OneHi;
  asm volatile("" : "+v"(one_lo), "+v"(one_hi));  // opaque: keeps them out of inline constants

  // units to the chunk's stage; norms and channel sums from the registers
  auto consume = [&](int c, const Slot& d) {
    const int b = c & 1;
    float cs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cs[e] = 0.f;
#pragma unroll
    for (int k = 0; k < XR; ++k) {
      const int row = rb + 64 * k;
      const u32x4 v = __builtin_bit_cast(u32x4, d.x[k]);
      s_x[b][row][lu ^ (row & 7)] = v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        xx[k] = dot2(v[e], v[e], xx[k]);
        cs[2 * e] = dot2(v[e], one_lo, cs[2 * e]);
        cs[2 * e + 1] = dot2(v[e], one_hi, cs[2 * e + 1]);
      }
    }
#pragma unroll
    for (int k = 0; k < QR; ++k) {
      const int row = rb + 64 * k;
      const u32x4 v = __builtin_bit_cast(u32x4, d.q[k]);
      s_q[b][row][lu ^ (row & 7)] = v;
#pragma unroll
      for (int e = 0; e < 4; ++e) qq[k] = dot2(v[e], v[e], qq[k]);
    }
    // the wave's channel sums (lanes lu, lu + 8, ..., lu + 56, in a fixed
    // order): lane 8 k + lu ends with channel 8 lu + k's
    s_pp[b][wave][8 * lu + (lane >> 3)] = lane_transpose_sum(cs);
  };
  // chunk c's channel sums, the waves' added in wave order by wave 0 (lane k:
  // channel k of the chunk).  Every lane of every wave issues the store (all
  // but wave 0's past the end of the buffer, which drops them), so the count of
  // memory operations in flight is the same on every path and the waits for
  // the ring's loads stay exact; the sums themselves sit behind a scalar branch.
  auto pool_out = [&](int c) {
    const int b = c & 1;
    float v = 0.f;
    if (wave == 0) {
#pragma unroll
      for (int w = 0; w < kWgWaves; ++w) v += s_pp[b][w][lane];
    }
    const int ch = c * kTokChunk + lane;
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), pres, (wave == 0 && ch < C) ? ch * 4 : kOOB, 0,
                                          kWriteThrough);
  };
  auto contract = [&](int c) {
    const int b = c & 1;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      bf16x8 B[NTW];
#pragma unroll
      for (int n = 0; n < NTW; ++n) {
        const int row = 16 * (NTW * wc + n) + r16;
        B[n] = __builtin_bit_cast(bf16x8, s_q[b][row][(4 * st + grp) ^ (row & 7)]);
      }
#pragma unroll
      for (int i = 0; i < MTW; ++i) {
        const int rt = MTW * wr + i;
        if (16 * rt < TM) {
          const int row = 16 * rt + r16;
          const bf16x8 A = __builtin_bit_cast(bf16x8, s_x[b][row][(4 * st + grp) ^ (row & 7)]);
#pragma unroll
          for (int n = 0; n < NTW; ++n) Sacc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B[n], Sacc[i][n], 0, 0, 0);
        }
      }
    }
  };

  // The loop runs to a multiple of D chunks: a chunk past the end reads
  // zeros, adds nothing and stores nowhere, and no branch around a load or
  // store makes the compiler wait for the whole ring.  The loads are issued
  // in slot order before and in the loop (the waits count the loads issued
  // after a slot's), and the norms' updates may not sink below a slot's
  // reload: the slot would need a second register set, and the copy back at
  // the end of the loop waits for the whole ring.
  Slot ring[D];
#pragma unroll
  for (int s = 0; s < D; ++s) {
    issue(s, ring[s]);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int c0 = 0; c0 < nch; c0 += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const int c = c0 + s;
      __builtin_amdgcn_sched_barrier(0);
      consume(c, ring[s]);
#pragma unroll
      for (int k = 0; k < XR; ++k) asm volatile("" : "+v"(xx[k]));
#pragma unroll
      for (int k = 0; k < QR; ++k) asm volatile("" : "+v"(qq[k]));
      lds_barrier();  // chunk c staged by every wave; chunk c - 2's stage no longer read
      issue(c + D, ring[s]);
      pool_out(c);
      contract(c);
    }
    if constexpr (CHAIN) {
#pragma unroll
      for (int i = 0; i < MTW; ++i) {
        Ssum[i] += Sacc[i][0];
        Sacc[i][0] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int k = 0; k < XR; ++k) xsum[k] += xx[k], xx[k] = 0.f;
#pragma unroll
      for (int k = 0; k < QR; ++k) qsum[k] += qq[k], qq[k] = 0.f;
    }
  }
  if constexpr (CHAIN) {
#pragma unroll
    for (int i = 0; i < MTW; ++i) Sacc[i][0] = Ssum[i];
#pragma unroll
    for (int k = 0; k < XR; ++k) xx[k] = xsum[k];
#pragma unroll
    for (int k = 0; k < QR; ++k) qq[k] = qsum[k];
  }

  // ---- epilogue ----
  auto row8_sum = [](float v) {  // the 8 lanes of a load-layout row
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0xB1, 0xF, 0xF, false));   // lane ^ 1
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x4E, 0xF, 0xF, false));   // lane ^ 2
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x141, 0xF, 0xF, false));  // 7 - i in 8
    return v;
  };
#pragma unroll
  for (int k = 0; k < XR; ++k) {
    const float v = row8_sum(xx[k]);
    if (lu == 0) s_xx[rb + 64 * k] = v;
  }
#pragma unroll
  for (int k = 0; k < QR; ++k) {
    const float v = row8_sum(qq[k]);
    if (lu == 0) s_qq[rb + 64 * k] = v;
  }
  // sigma_j of the wave's rows: accumulator column j = 16 n + r16, the four
  // lane groups added by lane swaps (rows past the tile hold zeros)
#pragma unroll
  for (int n = 0; n < NTW; ++n) {
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < MTW; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v += Sacc[i][n][e];
    v = row_sum4(v);
    if (lane < 16) s_sig[wr][16 * (NTW * wc + n) + r16] = v;
  }
  lds_barrier();  // s_qq, s_xx, s_sig complete
  if (tid < Q) {
    f.sig_part[(size_t(t) * f.tiles + tile) * Q + tid] = s_sig[0][tid] + s_sig[1][tid];
    if (tile == 0) f.qg_part[size_t(t) * Q + tid] = s_qq[tid];
  }
  // the wave's row maxima of S_nj / |q_j| over its columns j < Q
  float rq[NTW];
  bool live[NTW];
#pragma unroll
  for (int n = 0; n < NTW; ++n) {
    const int j = 16 * (NTW * wc + n) + r16;
    const float qv = s_qq[j];
    rq[n] = qv > 0.f ? 1.0f / sqrtf(qv) : 0.f;
    live[n] = j < Q;
  }
#pragma unroll
  for (int i = 0; i < MTW; ++i) {
    const int rt = MTW * wr + i;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float best = -INFINITY;
#pragma unroll
      for (int n = 0; n < NTW; ++n)
        if (live[n]) best = fmaxf(best, Sacc[i][n][e] * rq[n]);
      best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0xB1, 0xF, 0xF, false)));
      best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x4E, 0xF, 0xF, false)));
      best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x141, 0xF, 0xF, false)));
      best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x140, 0xF, 0xF, false)));
      if (r16 == e) s_best[wc][16 * rt + 4 * grp + e] = best;
    }
  }
  lds_barrier();  // s_best complete
  // a_{t,n} = max_j S_nj / (|q_j| |x_n|): the column groups' maxima in order
  for (int row = tid; row < TM; row += kWgWaves * 64) {
    const float best = fmaxf(fmaxf(s_best[0][row], s_best[1][row]), fmaxf(s_best[2][row], s_best[3][row]));
    const float xn = sqrtf(s_xx[row]);
    f.tok_score[size_t(t) * N + tok0 + row] = xn > 0.f ? best / xn : 0.f;
  }
}

// ---------------------------------------------------------------------------
// Wide queries (bf16, Q > 128)
// ---------------------------------------------------------------------------
// S has too many columns for one wave's accumulators or for a query stage that
// waves share, so the columns are dealt to eight waves (16-column tile n * 8 +
// wave, n < NTW: 128 NTW columns a pass, up to 384) and each stages its own
// columns' query rows, which no other wave uses, in LDS of its own (loaded
// straight into the MFMA layout, 16 rows' lines to an instruction, each load
// took four times the cycles of eight whole lines: 76 against 65 us at Q =
// 300).  The tile of X is staged for all of them; two chunks of 64 channels at
// a time, 16-byte units XOR-swizzled by row, X's stage double-buffered with one
// LDS-only barrier every two chunks.  The loads in flight are the next two
// chunks of the query and the next four of X, in that order: loads return in
// order, and a wait for the query must not drain X's, which come from farther.
// |x|^2, |q_j|^2 and the channel sums are formed from the registers.
// Sums of products run in chains of four chunks, added up in a second
// accumulator (one chain of C / 32 steps was three times as far from the 64-bit
// result).
// A workgroup owns at most `sub` stretches of 16 MTW tokens of one frame, one
// after another, with all channels, so a_{t,n} is final here; with sub > 1 (where
// the partial sums of finer tiles would not fit the scratch and it costs little)
// the channel and column sums add up over the stretches in order.  Queries of
// more than 384 tokens take passes over a stretch, channel sums in the first.
// Bound: staging, the barrier and the contraction follow one another with one
// workgroup, two waves a SIMD, to a CU; no unit is busy alone (counters at T = 64,
// 14x14, C = 3584, Q = 300, 69.7 us: vector ALU 36 % of the cycles, LDS 31 % with
// hardly a bank conflict, MFMA 21 %; a third of the waves' cycles wait for loads
// or the barrier, a third to issue).  <4, 3> takes all 256 registers and spills
// eight values that are set before the loops and read between them, none in the
// loop over chunks, whose loads are counted.  It replaced channel slices with
// partial scores through memory, dot products on the vector ALU for small frames
// (Q > 256), and passes of 32 columns over the tile (Q <= 256), but where
// wide_takes_slices and wide_takes_passes say.
// wz_relevance at T = 64, 14x14, C = 3584: Q = 130 84 -> 54 us, Q = 300 209 ->
// 75 us (error against 64 bits 1.3e-7 -> 0.95e-7), Q = 1024 603 -> 221 us; T =
// 40, 5x5, C = 1024, Q = 300: 1409 -> 23 us.  Four further waves that load X and
// form the sums leave the contracting ones no registers for the second
// accumulator (Q = 300 62 us, but three times the error).
constexpr int kWideWaves = 8;
constexpr int kWideThreads = kWideWaves * kWave;

// LONE: each channel is summed by itself.  Channel sums by dot2 multiply a channel's
// neighbour by 0, so an infinity makes its neighbour's sum NaN (and r_t = 0,
// delta_t = 1); frames of fewer than 49 tokens with more than 256 query tokens have
// always kept it to its own channel (r_t NaN, delta_t = 0).
template <int MTW, int NTW, bool LONE>
__global__ __launch_bounds__(kWideThreads, 2) void k_relevance_wide(int tile_tokens, int sub,
                                                                    const VideoArgs<StreamArgs> va) {
  const StreamArgs f = va.v[blockIdx.y];
  constexpr int ROWS = 64;                    // rows of the stage
  constexpr int NQ = kWideWaves * 16 * NTW;   // columns of a pass
  __shared__ __align__(16) u32x4 s_x[2][2][ROWS][8];               // two chunks a buffer
  __shared__ __align__(16) u32x4 s_q[kWideWaves][2][16 * NTW][8];  // each wave's query rows of two chunks
  __shared__ float s_pp[2][2][2 * MTW][kTokChunk];                 // per-wave channel sums of a chunk
  __shared__ float s_xx[ROWS];
  __shared__ float s_qq[kWideWaves][16 * NTW];
  __shared__ float s_best[kWideWaves][16 * MTW];  // row maxima of S_nj / |q_j| over a wave's columns

  int t, tile;
  unit_of_block(blockIdx.x, f.tiles, t, tile);
  if (t >= f.T) return;
  const int N = f.N, C = f.C, Q = f.Q;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, grp = lane >> 4;  // MFMA layout: row / column, K group
  const int rb = tid >> 3, lr = lane >> 3, lu = tid & 7;  // load layout: tile row rb, query rows 8 k + lr, 16-byte unit lu
  const int nch = (C + kTokChunk - 1) / kTokChunk;
  const int nloop = (nch + 3) / 4 * 4;  // chunks past the end read zeros and store nowhere
  const int npass = (Q + NQ - 1) / NQ;
  const int tile0 = tile * tile_tokens, tile1 = min(N, tile0 + tile_tokens);
  const int step = (tile_tokens + sub - 1) / sub;  // tokens of a stretch, at most 16 MTW
  const uint16_t* __restrict__ X = static_cast<const uint16_t*>(f.X) + size_t(t) * N * C;
  const size_t unit = size_t(t) * f.tiles + tile;
  const __amdgpu_buffer_rsrc_t pres = make_rsrc_uniform(f.pool_part + unit * C, uint32_t(C) * 4);
  uint32_t one_lo = kBf16OneLo, one_hi = kBf16OneHi;
  asm volatile("" : "+v"(one_lo), "+v"(one_hi));  // opaque: keeps them out of inline constants
  auto row8_sum = [](float v) {  // the 8 lanes of a load-layout row
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0xB1, 0xF, 0xF, false));   // lane ^ 1
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x4E, 0xF, 0xF, false));   // lane ^ 2
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x141, 0xF, 0xF, false));  // 7 - i in 8
    return v;
  };

  for (int tok0 = tile0; tok0 < tile1; tok0 += step) {
    const int TM = min(step, tile1 - tok0);
    const bool first = tok0 == tile0;
    const __amdgpu_buffer_rsrc_t xres = make_rsrc_uniform(X + size_t(tok0) * C, uint32_t(TM) * C * 2);
    for (int h = 0; h < npass; ++h) {
      const int qb = h * NQ;
      const __amdgpu_buffer_rsrc_t qres =
          make_rsrc_uniform(static_cast<const uint16_t*>(f.query) + size_t(qb) * C, uint32_t(min(NQ, Q - qb)) * C * 2);
      // the wave's last tile has columns (uniform over the wave; the others
      // hardly ever lack them)
      const bool live = qb + 16 * (kWideWaves * (NTW - 1) + wave) < Q;
      // (rows past the stretch or the query lie past the end of their buffer and read zeros)
      const int xoff = rb * C * 2 + 16 * lu;
      const int qoff = (16 * wave + lr) * C * 2 + 16 * lu, qstep = 16 * kWideWaves * C * 2;
      auto load_x = [&](int c, u32x4& d) {
        d = buf_load_u32x4(xres, c * kTokChunk + 8 * lu < C ? xoff + c * kTokChunk * 2 : kOOB);
      };
      auto load_q = [&](int c, u32x4 (&d)[NTW][2]) {
        const int off = c * kTokChunk + 8 * lu < C ? qoff + c * kTokChunk * 2 : kOOB;
#pragma unroll
        for (int n = 0; n < NTW; ++n)
#pragma unroll
          for (int k = 0; k < 2; ++k) d[n][k] = buf_load_u32x4(qres, off + n * qstep + 8 * k * C * 2);
      };
      f32x4 Sacc[MTW][NTW];
      float qq[NTW][2], xx = 0.f;
#pragma unroll
      for (int n = 0; n < NTW; ++n) {
        qq[n][0] = qq[n][1] = 0.f;
#pragma unroll
        for (int i = 0; i < MTW; ++i) Sacc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      u32x4 rx[2][2], rq[2][NTW][2];
      load_x(0, rx[0][0]);
      load_x(1, rx[0][1]);
      __builtin_amdgcn_sched_barrier(0);
      load_q(0, rq[0]);
      load_q(1, rq[1]);
      __builtin_amdgcn_sched_barrier(0);
      load_x(2, rx[1][0]);
      load_x(3, rx[1][1]);
      __builtin_amdgcn_sched_barrier(0);
      for (int c0 = 0; c0 < nloop; c0 += 4) {
        f32x4 part[MTW][NTW];
        float qp[NTW][2], xp = 0.f;
#pragma unroll
        for (int n = 0; n < NTW; ++n) {
          qp[n][0] = qp[n][1] = 0.f;
#pragma unroll
          for (int i = 0; i < MTW; ++i) part[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int c = c0 + 2 * b;
          // chunks c, c + 1: the tile's rows to the stage, |x|^2 and the channel sums
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            const u32x4 v = rx[b][m];
            s_x[b][m][rb][lu ^ (rb & 7)] = v;
            float cs[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              xp = dot2(v[e], v[e], xp);
              cs[2 * e] = LONE ? bf16_lo(v[e]) : dot2(v[e], one_lo, 0.f);
              cs[2 * e + 1] = LONE ? bf16_hi(v[e]) : dot2(v[e], one_hi, 0.f);
            }
            // lane 8 k + lu ends with channel 8 lu + k's sum over the wave's rows
            const float cw = lane_transpose_sum(cs);
            if (wave < 2 * MTW) s_pp[b][m][wave][8 * lu + lr] = cw;
          }
          asm volatile("" : "+v"(xp));  // not below the reload
          // the wave's query rows (its reads of the last two chunks are behind it), |q_j|^2
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < NTW; ++n)
#pragma unroll
              for (int k = 0; k < 2; ++k) {
                const u32x4 v = rq[m][n][k];
                s_q[wave][m][16 * n + 8 * k + lr][lu ^ lr] = v;
#pragma unroll
                for (int e = 0; e < 4; ++e) qp[n][k] = dot2(v[e], v[e], qp[n][k]);
                asm volatile("" : "+v"(qp[n][k]));
              }
          __builtin_amdgcn_sched_barrier(0);
          load_q(c + 2, rq[0]);
          load_q(c + 3, rq[1]);
          __builtin_amdgcn_sched_barrier(0);
          load_x(c + 4, rx[b][0]);
          load_x(c + 5, rx[b][1]);
          __builtin_amdgcn_sched_barrier(0);
          lds_barrier();  // the two chunks of X staged; the two before them no longer read
          // their channel sums, the waves' added in wave order by waves 0 and 1
          // (every lane stores, most past the end: the count of memory
          // operations in flight stays the same on every path)
          float v = 0.f;
          const int ch = (c + wave) * kTokChunk + lane;
          const int off = (h == 0 && wave < 2 && ch < C) ? ch * 4 : kOOB;
          if (wave < 2) {
#pragma unroll
            for (int w = 0; w < 2 * MTW; ++w) v += s_pp[b][wave][w][lane];
            if (!first) v = buf_load_f32(pres, off) + v;
          }
          buf_store_f32(v, pres, off);
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int st = 0; st < 2; ++st) {
              const int u = (4 * st + grp) ^ (r16 & 7);  // unit 4 st + grp of a row of either stage
              u32x4 A[MTW];
#pragma unroll
              for (int i = 0; i < MTW; ++i) A[i] = s_x[b][m][16 * i + r16][u];
#pragma unroll
              for (int n = 0; n < NTW; ++n) {
                if (n < NTW - 1 || live) {
                  const bf16x8 B = __builtin_bit_cast(bf16x8, s_q[wave][m][16 * n + r16][u]);
#pragma unroll
                  for (int i = 0; i < MTW; ++i)
                    part[i][n] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, A[i]), B, part[i][n], 0, 0, 0);
                }
              }
            }
        }
        xx += xp;
#pragma unroll
        for (int n = 0; n < NTW; ++n) {
          qq[n][0] += qp[n][0];
          qq[n][1] += qp[n][1];
#pragma unroll
          for (int i = 0; i < MTW; ++i) Sacc[i][n] += part[i][n];
        }
      }
      if (h == 0) {
        const float v = row8_sum(xx);
        if (lu == 0) s_xx[rb] = v;
      }
#pragma unroll
      for (int n = 0; n < NTW; ++n)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float v = row8_sum(qq[n][k]);
          if (lu == 0) s_qq[wave][16 * n + 8 * k + lr] = v;
        }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // (one wave's own LDS, in program order)
      __builtin_amdgcn_wave_barrier();
      // the wave's columns: sigma_j (rows past the stretch hold zeros), |q_j|^2
      // and its row maxima of S_nj / |q_j|
      float rqn[NTW];
#pragma unroll
      for (int n = 0; n < NTW; ++n) {
        const int j = qb + 16 * (kWideWaves * n + wave) + r16;
        float v = 0.f;
#pragma unroll
        for (int i = 0; i < MTW; ++i) v += (Sacc[i][n][0] + Sacc[i][n][1]) + (Sacc[i][n][2] + Sacc[i][n][3]);
        v = row_sum4(v);
        const float qv = s_qq[wave][16 * n + r16];
        rqn[n] = qv > 0.f ? 1.0f / sqrtf(qv) : 0.f;
        if (j < Q && lane < 16) {
          float* sig = f.sig_part + unit * Q + j;
          *sig = first ? v : *sig + v;
          if (tile == 0 && first) f.qg_part[size_t(t) * Q + j] = qv;
        }
      }
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float best = -INFINITY;
#pragma unroll
          for (int n = 0; n < NTW; ++n)
            if (qb + 16 * (kWideWaves * n + wave) + r16 < Q) best = fmaxf(best, Sacc[i][n][e] * rqn[n]);
          best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0xB1, 0xF, 0xF, false)));
          best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x4E, 0xF, 0xF, false)));
          best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x141, 0xF, 0xF, false)));
          best = fmaxf(best, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(best), 0x140, 0xF, 0xF, false)));
          if (r16 == e) {
            float& out = s_best[wave][16 * i + 4 * grp + e];
            out = h == 0 ? best : fmaxf(out, best);
          }
        }
    }
    lds_barrier();  // s_best and s_xx complete (rewritten behind at least one more barrier)
    // a_{t,n} = max_j S_nj / (|q_j| |x_n|), the waves' maxima in order
    if (tid < TM) {
      float best = s_best[0][tid];
#pragma unroll
      for (int w = 1; w < kWideWaves; ++w) best = fmaxf(best, s_best[w][tid]);
      const float xn = sqrtf(s_xx[tid]);
      f.tok_score[size_t(t) * N + tok0 + tid] = xn > 0.f ? best / xn : 0.f;
    }
  }
}

template <int MTW, bool LONE>
void launch_wide_cols(const RelPlan& pl, const VideoArgs<StreamArgs>& va, int V, hipStream_t s) {
  const dim3 grid(pl.grid, V), block(kWideThreads);
  if (pl.ntw == 2) hipLaunchKernelGGL((k_relevance_wide<MTW, 2, LONE>), grid, block, 0, s, pl.tile_tokens, pl.sub, va);
  else hipLaunchKernelGGL((k_relevance_wide<MTW, 3, LONE>), grid, block, 0, s, pl.tile_tokens, pl.sub, va);
}
template <int MTW>
void launch_wide_rows(const RelPlan& pl, const VideoArgs<StreamArgs>& va, int V, hipStream_t s) {
  if constexpr (MTW <= 3)  // fewer than 49 tokens
    if (va.v[0].N < 49 && va.v[0].Q > 256) return launch_wide_cols<MTW, true>(pl, va, V, s);
  launch_wide_cols<MTW, false>(pl, va, V, s);
}

// LDS of a token-tiled workgroup without the gathered channel sums.
constexpr size_t tok_lds(int ntg, int ipc, int wv) {
  const int rows = tok_rows(ipc), nq = 16 * ntg;
  return size_t(wv) * (rows + nq) * 128 + size_t(wv) * (rows + 2 * nq) * 4 + size_t(nq) * 4;
}
template <typename In, int NTG, int IPC, int MODE, int WV>
void launch_tok_waves(const RelPlan& pl, const VideoArgs<StreamArgs>& va, int V, hipStream_t s) {
  // the channel sums are gathered in LDS up to 32 query columns (with 64,
  // storing them chunk by chunk measured 1 % faster on full 64-token tiles:
  // 160.0 against 161.4 us per call at T = 96, 27x27, C = 1152, Q = 48)
  const size_t pool = size_t(va.v[0].C) * 4;
  if constexpr (NTG <= 2) {
    if (va.v[0].C <= kTokPoolMax && tok_lds(NTG, IPC, WV) + pool <= kTokLdsMax) {
      hipLaunchKernelGGL((k_relevance_tok<In, NTG, IPC, true, MODE, WV>), dim3(pl.grid, V), dim3(WV * kWave), pool, s,
                         pl.tile_tokens, va);
      return;
    }
  }
  // Tiles of 9 to 24 long rows that come from HBM (X beyond the 256 MB Infinity
  // Cache): LDS enough that one workgroup runs on a CU, not two or three whose
  // rows are so many more streams (Q <= 16, one / several: T = 270, 23x1, C = 22368
  // 89.1 / 95.1 us; T = 597, 22x1, C = 51224 455 / 477; T = 1850, 8x1, C = 19064,
  // shorter tiles, 244 / 221; T = 304, 26x1, C = 8512, 135 MB, 42.1 / 40.5).
  constexpr size_t kHalf = kTokLdsMax / 2 + 1024;
  const bool alone = sizeof(In) == 2 && NTG == 1 && (IPC == 2 || IPC == 3) && va.v[0].C > kTokPoolMax &&
                     size_t(va.v[0].T) * va.v[0].N * va.v[0].C * 2 > (size_t(256) << 20);
  const size_t lds = alone && tok_lds(NTG, IPC, WV) < kHalf ? kHalf - tok_lds(NTG, IPC, WV) : 0;
  hipLaunchKernelGGL((k_relevance_tok<In, NTG, IPC, false, MODE, WV>), dim3(pl.grid, V), dim3(WV * kWave), lds, s,
                     pl.tile_tokens, va);
}
template <typename In, int NTG, int IPC, int MODE>
void launch_tok_mode(const RelPlan& pl, const VideoArgs<StreamArgs>& va, int V, hipStream_t s) {
  const int C = va.v[0].C;
  // Four waves for a query of 17 to 32 tokens in one pass with the channel
  // sums in LDS (measured faster than eight).  A pass shared by queries of
  // that size (64 query columns) takes four waves too: a wave's chunks set
  // the order in which each query's sums are added, so that each query's
  // results are bitwise those of its own pass.
  if constexpr (sizeof(In) == 2 && ((NTG == 2 && MODE == kTokOne) || (NTG == 4 && MODE == kTokGroups))) {
    if (C <= kTokPoolMax && (MODE == kTokOne || (va.v[0].qg + 15) / 16 == 2)) {
      launch_tok_waves<In, NTG, IPC, MODE, 4>(pl, va, V, s);
      return;
    }
  }
  launch_tok_waves<In, NTG, IPC, MODE, kTokWaves>(pl, va, V, s);
}
template <typename In, int NTG, int IPC>
void launch_tok(const RelPlan& pl, const VideoArgs<StreamArgs>& va, int V, hipStream_t s) {
  if (va.v[0].groups > 1) {
    launch_tok_mode<In, NTG, IPC, kTokGroups>(pl, va, V, s);
  } else if (va.v[0].Q > 16 * NTG) {
    // the plan takes two query tiles for passes, with bf16 inputs tiles of at
    // most 32 tokens (checked by the caller)
    if constexpr (NTG == 2 && (sizeof(In) == 4 || IPC <= 4)) launch_tok_mode<In, NTG, IPC, kTokPasses>(pl, va, V, s);
  } else {
    launch_tok_mode<In, NTG, IPC, kTokOne>(pl, va, V, s);
  }
}

template <typename In, int NTG>
void launch_tok_tile(const RelPlan& pl, const VideoArgs<StreamArgs>& va, int V, hipStream_t s) {
  switch (pl.ipc) {
    case 1: launch_tok<In, NTG, 1>(pl, va, V, s); break;
    case 2: launch_tok<In, NTG, 2>(pl, va, V, s); break;
    case 3: launch_tok<In, NTG, 3>(pl, va, V, s); break;
    case 4: launch_tok<In, NTG, 4>(pl, va, V, s); break;
    case 5: launch_tok<In, NTG, 5>(pl, va, V, s); break;
    case 6: launch_tok<In, NTG, 6>(pl, va, V, s); break;
    case 7: launch_tok<In, NTG, 7>(pl, va, V, s); break;
    default: launch_tok<In, NTG, 8>(pl, va, V, s); break;
  }
}
template <typename In>
void launch_tok_shape(const RelPlan& pl, const VideoArgs<StreamArgs>& va, int V, hipStream_t s) {
  if (pl.ntg == 1) launch_tok_tile<In, 1>(pl, va, V, s);
  else if (pl.ntg == 2) launch_tok_tile<In, 2>(pl, va, V, s);
  else launch_tok_tile<In, 4>(pl, va, V, s);
}

}  // namespace

hipError_t launch_relevance_stream(const wz_config& c, const void* X, const void* query, float* tok_score,
                                   const Workspace& ws, hipStream_t s, const Videos& vs) {
  RelPlan pl = relevance_plan(c);
  VideoArgs<StreamArgs> va{};
  int V = vs.V;
  if (vs.shared_x && shared_pass(c, vs.V)) {
    // queries in groups of up to 64 columns, one pass over X per group (grid
    // y = group): the per-query plan's tiles, query tiles for a group's columns
    const int G = std::min(vs.V, queries_per_pass(c));
    const int QT = c.Q * G;
    pl.ntg = QT <= 16 ? 1 : QT <= 32 ? 2 : 4;
    V = (vs.V + G - 1) / G;
    for (int e = 0; e < V; ++e) {
      const int q0 = e * G, n = std::min(G, vs.V - q0);
      const Workspace w = advance(ws, q0 * vs.ws);
      va.v[e] = StreamArgs{X, advance(query, q0 * vs.q), w.qg_part, w.sig_part, w.pool_part,
                           advance(tok_score, q0 * vs.ws), c.T, c.H * c.W, c.C, c.Q * n, pl.tiles, n,
                           c.Q, vs.ws};
    }
  } else {
    for (int v = 0; v < vs.V; ++v) {
      const Workspace w = advance(ws, v * vs.ws);
      va.v[v] = StreamArgs{advance(X, v * vs.x), advance(query, v * vs.q), w.qg_part, w.sig_part,
                           w.pool_part, advance(tok_score, v * vs.ws), c.T, c.H * c.W, c.C, c.Q,
                           pl.tiles};
    }
  }
  if (pl.kind == kRelTok) {
    // columns beyond the query tiles are served by passes of two tiles only
    if (va.v[0].Q > 16 * pl.ntg && (pl.ntg != 2 || va.v[0].groups > 1 || (c.in_dtype == WZ_BF16 && pl.ipc > 4)))
      return hipErrorInvalidValue;
    if (c.in_dtype == WZ_BF16) launch_tok_shape<uint16_t>(pl, va, V, s);
    else launch_tok_shape<float>(pl, va, V, s);
  } else if (pl.kind == kRelWg) {
    if (va.v[0].groups > 1 || va.v[0].Q > 16 * pl.ntg) return hipErrorInvalidValue;
    const dim3 grid(pl.grid, V), block(kWgWaves * 64);
    if (pl.ntg == 4 && pl.rtw == 1) hipLaunchKernelGGL((k_relevance_wg<1, 1>), grid, block, 0, s, pl.tile_tokens, va);
    else if (pl.ntg == 4) hipLaunchKernelGGL((k_relevance_wg<2, 1>), grid, block, 0, s, pl.tile_tokens, va);
    else if (pl.rtw == 1) hipLaunchKernelGGL((k_relevance_wg<1, 2>), grid, block, 0, s, pl.tile_tokens, va);
    else hipLaunchKernelGGL((k_relevance_wg<2, 2>), grid, block, 0, s, pl.tile_tokens, va);
  } else if (pl.kind == kRelSlices) {
    if (va.v[0].groups > 1 || pl.mt > kMaxWaves || pl.kc > kSliceSteps * kKStep) return hipErrorInvalidValue;
    VideoArgs<SliceArgs> sa{};
    for (int v = 0; v < V; ++v) {
      const Workspace w = advance(ws, v * vs.ws);
      sa.v[v] = SliceArgs{va.v[v], w.s_part, w.g_part, qpad(c.Q), pl.slices};
    }
    hipLaunchKernelGGL((k_relevance_slices<2, 4>), dim3(pl.grid, V), dim3((pl.mt + 1) / 2 * kWave), 0, s, pl.tile_tokens,
                       pl.kc, sa);
  } else {
    if (va.v[0].groups > 1 || pl.mt > 4) return hipErrorInvalidValue;
    switch (pl.mt) {
      case 1: launch_wide_rows<1>(pl, va, V, s); break;
      case 2: launch_wide_rows<2>(pl, va, V, s); break;
      case 3: launch_wide_rows<3>(pl, va, V, s); break;
      default: launch_wide_rows<4>(pl, va, V, s); break;
    }
  }
  return hipGetLastError();
}

}  // namespace wz
