// Internal declarations shared by the gfx950 kernels and the C-ABI layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "wavezip.h"

namespace wz {

constexpr int kWave = 64;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// bf16 <-> fp32 (bf16 is the upper half of an fp32 bit pattern).
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;  // NaN stays NaN
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// Butterfly sum across the 64 lanes of a wave (every lane gets the total).
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
  return v;
}

// ---------------------------------------------------------------------------
// Decomposition of the relevance pass (shapes and limits; the kernels'
// comments give the details): token tiles of a frame, each with every channel
// (kRelSlices: also slices of channels).
// ---------------------------------------------------------------------------
constexpr int kXcds = 8;          // MI355X: workgroups are dealt to the 8 XCDs round robin
constexpr int kCUs = 256;
constexpr int kTokMax = 4096;     // validated bound on tokens per frame
constexpr int kMaxWaves = 16;     // kRelSlices: 16-row MFMA tiles per token tile
constexpr int kTilesPerWave = 2;  // kRelSlices: 16-row MFMA tiles per wave
constexpr int kSliceSteps = 32;   // kRelSlices: 32-channel steps per slice at most (the query slice sits in LDS)

// Scratch of the allocation-free call.
constexpr size_t kScratchBytes = size_t(32) << 20;

// Streaming kernels of the relevance pass, chosen by shape:
//   kRelTok  fp32; bf16, Q <= 64: token tiles, each wave a channel stripe with
//            its own LDS-transposed MFMA (above 64 query tokens, fp32 or where
//            wide_takes_passes says: passes of 32 columns per tile);
//   kRelWg   bf16, 64 < Q <= 128 (and 32 < Q <= 64, see relevance_kind): the
//            workgroup's waves share each channel chunk of the tile and the
//            query in LDS, each wave some 16-row tiles against every column;
//   kRelWide bf16, Q > 128 (but see wide_takes_passes, wide_takes_slices): the
//            waves split the query's columns and share each chunk of the tile
//            in LDS;
//   kRelSlices bf16, Q > 256 where wide_takes_slices says: tiles of up to 256
//            tokens, slices of channels.
enum RelKind { kRelTok = 0, kRelWg = 1, kRelWide = 2, kRelSlices = 3 };

// Query columns of the slices' partial scores, padded for 16-byte rows.
inline int qpad(int Q) { return (Q + 3) & ~3; }

// Token tiles per frame of at most `cap` tokens for `slots` workgroups running
// at once: the count (tiles of 16 tokens and up) with the fewest rows of X and
// query a slot loads over its turns, the smaller count on a tie.
inline int rel_tiles(const wz_config& c, int cap, int slots, int qrows) {
  const int N = c.H * c.W, tr = (c.T + kXcds - 1) / kXcds * kXcds;
  const int lo = (N + cap - 1) / cap, hi = std::max(lo, (N + 15) / 16);
  // fp32 inputs: tiles finer than 32 tokens (whose channel and column sums
  // the workspace holds, T * tiles * (C + Q) floats) only while those stay
  // under half of the allocation-free call's 32 MiB
  const bool f32 = c.in_dtype != WZ_BF16;
  long best = -1;
  int tiles = lo;
  for (int k = lo; k <= hi; ++k) {
    if (f32 && k > lo && k > (N + 31) / 32 && (long long)c.T * k * (c.C + c.Q) * 4 > (16LL << 20)) break;
    const long cost = long((long(tr) * k + slots - 1) / slots) * ((N + k - 1) / k + qrows);
    if (best < 0 || cost < best) best = cost, tiles = k;
  }
  return tiles;
}

// Workspace bytes at `tiles` token tiles a frame, one slice (see workspace_layout).
inline size_t workspace_bytes_at(const wz_config& c, int tiles, bool split);

// Token tiles per frame of kRelWide: of 16 to 64 tokens, or of up to 256 in
// stretches of at most 64.  Per 64 channels a stretch's MFMAs take as long as
// 16-row tiles x column tiles, its query reads from L2 as long as four 16-row
// tiles do: their sum over a CU's turns is the cost of a count.
inline long wide_cost(const wz_config& c, int tiles) {
  const int tr = (c.T + kXcds - 1) / kXcds * kXcds, tt = (c.H * c.W + tiles - 1) / tiles, sub = (tt + 63) / 64;
  const int rows = ((tt + sub - 1) / sub + 15) / 16 * 16;
  return long((long(tr) * tiles + kCUs - 1) / kCUs) * sub * (rows + 64);
}
// the cheapest count of tiles of at most 64 tokens, the smaller on a tie
inline int wide_best_tiles(const wz_config& c) {
  const int N = c.H * c.W, lo = (N + 63) / 64;
  int tiles = lo;
  long best = wide_cost(c, lo);
  for (int k = lo + 1; k <= (N + 15) / 16; ++k)
    if (const long cost = wide_cost(c, k); cost < best) best = cost, tiles = k;
  return tiles;
}
inline int wide_tiles(const wz_config& c) {
  const int N = c.H * c.W, tiles = wide_best_tiles(c);
  // The tiles' channel and column sums are the workspace's largest part.  Where
  // they do not fit the allocation-free call's scratch, the cheapest count that
  // does (with the filter-bank operator rows, else without), if its cost is not
  // too far up; otherwise the caller's workspace holds the finer tiles.  The
  // line: a quarter more up to 256 query tokens (wz_relevance, T = 260, 14x14,
  // C = 8192, Q = 130: passes of 32 columns 715 us, tiles of 256 tokens, at 1.6
  // times the cost, 809, of 98 tokens, at 1.2 times, 610; T = 4, 64x64, C =
  // 32768, Q = 300: 2305 us in tiles of 256 tokens on a quarter of the chip, of
  // 128 tokens 1346); half more above, where the scratch has always held tiles
  // of 256 tokens up to C = 1024 (at most 1.43 times the cost there).
  const long pct = c.Q <= 256 ? 125 : 150;
  const long most = wide_cost(c, tiles) * pct;
  for (const bool split : {true, false}) {
    if (workspace_bytes_at(c, tiles, split) <= kScratchBytes) break;
    int fit = 0;
    long best = most / 100 + 1;
    for (int k = (N + 255) / 256; k <= (N + 15) / 16 && workspace_bytes_at(c, k, split) <= kScratchBytes; ++k)
      if (const long cost = wide_cost(c, k); 100 * cost <= most && cost < best) best = cost, fit = k;
    if (fit) return fit;
  }
  return tiles;
}

// Time of kRelWide's pass in ns, from 1050 shapes over the whole accepted range
// (median error 6 %): a turn's latency by passes, chunks, column and row tiles,
// or the bytes that every workgroup reads of X and the query.
inline int wide_passes(const wz_config& c) { return (c.Q + 383) / 384; }  // of up to 384 columns
inline int wide_ntw(const wz_config& c) { return (c.Q + 128 * wide_passes(c) - 1) / (128 * wide_passes(c)); }
inline long wide_ns(const wz_config& c) {
  const int N = c.H * c.W, tr = (c.T + kXcds - 1) / kXcds * kXcds, kw = wide_best_tiles(c), ntw = wide_ntw(c);
  const int mt = ((N + kw - 1) / kw + 15) / 16;
  const long turns = (long(tr) * kw + kCUs - 1) / kCUs;
  return 5000 + std::max(turns * wide_passes(c) * (2800 + (c.C + 255) / 256 * (700 + 900 * ntw + 180 * mt * ntw)),
                         (long(c.T) * N * c.C * 200 + long(c.T) * kw * c.Q * c.C * 260) / 1000000);
}

// Whether 129 to 256 bf16 query tokens take passes of 32 columns (kRelTok)
// instead of kRelWide.  Up to 4096 channels they do not: kRelWide is never
// slower than passes were there, and its sums are nearer to 64 bits.  Above, a
// few tokens a CU leave its eight waves waiting for a long query in step with
// one another, where a wave of the passes waits for its own chunks alone (in
// tiles of at most 32 tokens; larger ones never gain).  The passes' time by
// passes, chunks and rows, or the bytes read (600 shapes, median error 5 %; the
// choice is within 8 % of the better one on all but one).  Passes against
// kRelWide, wz_relevance in us: T = 1, one token, C = 32768, Q = 129 232 / 302;
// T = 434, one token, C = 16384, Q = 160 255 / 310; T = 16, 15x15, C = 16384, Q
// = 129 161 / 175; T = 3, 27x27, C = 16384, Q = 200 250 / 211; T = 260, 14x14, C
// = 8192, Q = 130 715 / 610.
inline bool wide_takes_passes(const wz_config& c) {
  if (c.Q > 256 || c.C <= 4096) return false;
  const int N = c.H * c.W, tr = (c.T + kXcds - 1) / kXcds * kXcds, chunks = (c.C + 63) / 64, np = (c.Q + 31) / 32;
  const int kt = rel_tiles(c, 64, kCUs, 32), rows = ((N + kt - 1) / kt + 7) / 8 * 8;
  const long turns = (long(tr) * kt + kCUs - 1) / kCUs;
  const long passes = std::max(3100 + turns * (3850 + np * (1650 + chunks * (23 + 18 * rows / 5))),
                               (long(c.T) * N * c.C * np * 294 + long(c.T) * kt * c.Q * c.C * 146) / 1000000);
  return rows <= 32 && 100 * passes < 95 * wide_ns(c);
}

// kRelSlices: tiles of up to 256 tokens; slices of at most kSliceSteps steps,
// more while the grid is short of one workgroup per CU, keeping slices of at
// least 8 channel steps and per-slice partial scores (4*Q bytes a token) under a
// quarter of X (2*C).
struct SlicePlan {
  int tiles, steps, slices;  // token tiles per frame; 32-channel steps per slice; slices
};
inline SlicePlan slice_plan(const wz_config& c) {
  const int N = c.H * c.W, cap = 16 * kMaxWaves, ksteps = (c.C + 31) / 32;
  SlicePlan p;
  p.tiles = (N + cap - 1) / cap;
  const int smin = (ksteps + kSliceSteps - 1) / kSliceSteps;
  const int smax = std::max(smin, std::min(ksteps / 8, c.C / (8 * c.Q)));
  int S = smin;
  while (S < smax && (long long)c.T * p.tiles * S < kCUs) ++S;
  p.steps = (ksteps + S - 1) / S;
  p.slices = (ksteps + p.steps - 1) / p.steps;
  return p;
}
// Whether more than 256 bf16 query tokens take channel slices instead of
// kRelWide (frames of 49 tokens and up: at least two waves a workgroup).  Above
// 8192 channels a few frames leave kRelWide on a few CUs, each streaming the whole
// query; below 128 its fixed cost a tile counts; between, kRelWide is as fast or
// faster (8 % slower at the most seen).  The slices' time by turns, passes of 32
// columns, steps and rows, or the bytes read, and the per-frame kernel's reads of
// the partial scores (1300 shapes, median error 6 %; long rows take them where
// within a tenth, so that a call is at most 14 % slower than with slices, on all
// but two 8 %, and at most 28 % slower than with kRelWide).  Slices against it,
// wz_relevance in us: T = 3, 33x2, C = 64408, Q = 816 1280 / 3117; T = 8, 10x12, C
// = 32768, Q = 300 298 / 439; T = 705, 13x57, C = 56, Q = 817 653 / 795; T = 8,
// 14x14, C = 16384, Q = 1024 847 / 673; T = 64, 7x7, C = 16384, Q = 300 459 / 236.
inline bool wide_takes_slices(const wz_config& c) {
  const int N = c.H * c.W;
  if (c.Q <= 256 || N < 49 || (c.C >= 128 && c.C <= 8192)) return false;
  const SlicePlan p = slice_plan(c);
  const int tr = (c.T + kXcds - 1) / kXcds * kXcds, mt = ((N + p.tiles - 1) / p.tiles + 15) / 16;
  const long turns = (long(tr) * p.tiles * p.slices + kCUs - 1) / kCUs, part = long(N) * p.slices * c.Q * 4;
  const long pass = std::max(turns * ((c.Q + 31) / 32) * (2300 + p.steps * (128 + 10 * mt)),
                             (long(c.T) * N * c.C * 390 + long(c.T) * p.tiles * c.Q * c.C * 216) / 1000000);
  const long frame = p.slices > 1 ? 7000 + (c.T * part * 1030 + part * 33000) / 1000000 : 0;
  return 100 * (5800 + pass + frame) < (c.C > 8192 ? 110 : 97) * wide_ns(c);
}

inline RelKind relevance_kind(const wz_config& c) {
  if (c.in_dtype != WZ_BF16 || c.Q <= 32) return kRelTok;
  if (c.Q > 64)
    return c.Q <= 128 ? kRelWg : wide_takes_passes(c) ? kRelTok : wide_takes_slices(c) ? kRelSlices : kRelWide;
  // 33 to 64 query tokens: channel stripes leave one workgroup to a CU, whose
  // turns do not overlap; the shared tiles leave two, with a barrier a chunk.
  // The shared tiles where they take fewer turns and less time, both in ns
  // from 300 shapes with H, W up to 64, C up to 10240 (median error 4 %; the
  // choice is within 4 % of the better one on each, 1 % slower on average): a
  // turn of the stripes by its tile's rows in eighths, of the shared tiles in
  // sixteenths.  At Q = 48, channel stripes against shared tiles: T = 512,
  // 14x14, C = 768 74.2 / 44.4 us; T = 256, 27x27, C = 1152 163.1 / 121.9; T =
  // 200, 14x14, C = 2560 67.9 / 58.7; T = 512, 8x8, C = 3584 54.7 / 62.4; T =
  // 74, 14x14, C = 3168 40.4 / 49.8; T = 289, 10x2, C = 3672 36.6 / 53.0.  Finer
  // tiles than the stripes' would also take more workspace.  (The videos of a
  // batch do not count: each has the bits of its single call.)
  const int N = c.H * c.W, tr = (c.T + kXcds - 1) / kXcds * kXcds, chunks = (c.C + 63) / 64;
  const int kt = rel_tiles(c, 64, kCUs, 64), kw = rel_tiles(c, 128, 2 * kCUs, 64);
  const long turns_t = (long(tr) * kt + kCUs - 1) / kCUs, turns_w = (long(tr) * kw + 2 * kCUs - 1) / (2 * kCUs);
  const int rows_t = ((N + kt - 1) / kt + 7) / 8 * 8, rows_w = ((N + kw - 1) / kw + 15) / 16 * 16;
  const long tok = 4300 + turns_t * (4800 + chunks * (74 + 16 * rows_t / 3));
  const long wg = 5400 + turns_w * (4500 + chunks * (540 + (rows_w <= 64 ? 5 * rows_w : 37 * rows_w / 5)));
  return kw <= kt && turns_w < turns_t && 100 * wg < 96 * tok ? kRelWg : kRelTok;
}

struct RelPlan {
  RelKind kind;
  int tiles;        // token tiles per frame
  int tile_tokens;  // tokens per tile (the last tile of a frame may be shorter)
  int mt;           // kRelWide, kRelSlices: 16-row MFMA tiles per stretch or tile
  int sub;          // kRelWide: stretches of a token tile
  int ntw;          // kRelWide: 16-column tiles per wave
  int slices;       // channel slices (1 but for kRelSlices)
  int kc;           // kRelSlices: channels per slice
  int grid;         // workgroups: frames rounded up to a multiple of kXcds, x tiles x slices
  int ipc;          // kRelTok: row load instructions per chunk (tile rows / 8)
  int ntg;          // kRelTok, kRelWg: 16-column query tiles
  int rtw;          // kRelWg: 16-row tiles per wave (tiles of up to 64 * rtw tokens)
};

inline RelPlan relevance_plan(const wz_config& c) {
  const int N = c.H * c.W;
  RelPlan p{};
  p.kind = relevance_kind(c);
  p.slices = 1;
  if (p.kind == kRelTok) {
    // tiles of 16 to 64 tokens with every channel.  A workgroup fills a CU's
    // LDS, so a CU runs (workgroups / CUs rounded up) of them one after
    // another, each loading its tile's tokens and the query's 16-row tiles;
    // query tiles: 1, 2 or 4 of 16 columns; above 64 columns, passes of 32
    const int nq = c.Q <= 16 ? 16 : c.Q <= 32 ? 32 : c.Q <= 64 ? 64 : 32;
    p.tiles = rel_tiles(c, 64, kCUs, nq);
    p.tile_tokens = (N + p.tiles - 1) / p.tiles;
    p.ipc = (p.tile_tokens + 7) / 8;
    p.ntg = nq / 16;
  } else if (p.kind == kRelWg) {
    // tiles of at most 128 tokens; two workgroups share a CU.  Every workgroup
    // streams its tile's rows and the whole query through LDS
    p.ntg = c.Q <= 64 ? 4 : 8;
    p.tiles = rel_tiles(c, 128, 2 * kCUs, 16 * p.ntg);
    p.tile_tokens = (N + p.tiles - 1) / p.tiles;
    p.rtw = p.tile_tokens <= 64 ? 1 : 2;
  } else if (p.kind == kRelSlices) {
    const SlicePlan sp = slice_plan(c);
    p.tiles = sp.tiles;
    p.tile_tokens = (N + p.tiles - 1) / p.tiles;
    p.mt = (p.tile_tokens + 15) / 16;
    p.slices = sp.slices;
    p.kc = sp.steps * 32;
  } else {
    // one workgroup to a CU
    p.ntw = wide_ntw(c);
    p.tiles = wide_tiles(c);
    p.tile_tokens = (N + p.tiles - 1) / p.tiles;
    p.sub = (p.tile_tokens + 63) / 64;
    p.mt = ((p.tile_tokens + p.sub - 1) / p.sub + 15) / 16;
  }
  p.grid = (c.T + kXcds - 1) / kXcds * kXcds * p.tiles * p.slices;
  return p;
}

// Workgroup b works on frame t = (b / kXcds / tiles) * kXcds + b % kXcds,
// so every workgroup of a frame runs on the same XCD.
__device__ __forceinline__ void unit_of_block(int b, int tiles, int& t, int& tile) {
  const int xcd = b % kXcds, slot = b / kXcds;
  t = (slot / tiles) * kXcds + xcd;
  tile = slot % tiles;
}

// The same with the slices of each tile next to one another.
__device__ __forceinline__ void slice_of_block(int b, int tiles, int slices, int& t, int& tile, int& slice) {
  int u;
  unit_of_block(b, tiles * slices, t, u);
  tile = u / slices;
  slice = u % slices;
}

constexpr int kMaxFrames = 2048;
// frames up to which the budget is folded into the selection kernel (one wave
// computes it in registers, one, two or four frames per lane); above, a launch of
// its own computes it once (one wave up to 512 frames, eight per lane; 1024
// threads beyond), instead of every selection workgroup repeating it
constexpr int kFusedTMax = 256;

// Workspace carve-up (all offsets 256-byte aligned).
// Bytes of the filter-bank operator rows in the workspace (0 if unused).
size_t filter_rows_bytes(const wz_config& c);

struct Workspace {
  float* s_part;       // [T][slices][N][qpad(Q)] per-slice x . q_j (only with several slices)
  float* g_part;       // [T][slices][N]          per-slice |x|^2 (only with several slices)
  float* qg_part;      // [T][slices][Q]          per-slice |q_j|^2
  float* sig_part;     // [T][tiles][slices][Q]   per-unit sums over tokens of x . q_j
  float* pool_part;    // [T][tiles][C]           per-tile channel sums
  float* tok_score;    // [T*N]
  int32_t* rank;       // [T*N]                   selection rank of each token in its frame
  int32_t* byrank;     // [T*N]                   token of each rank
  float* gate;         // [T*N]                   saliency gate of each token's 2x2 block
  float* gate2;        // [T*N]                   level-2 gate of each token (two spatial levels)
  float* frame_rel;    // [T]
  float* frame_delta;  // [T]
  int32_t* budget;     // [T]
  int32_t* offset;     // [T+1]
  uint16_t* frows;     // [B][2][pad(H*W)]        filter-bank operator rows (bf16 inputs, filter spatial basis)
  size_t bytes;
};

inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// split: room for the filter-bank operator rows when the problem uses them
// (without it the modulator runs its fused form, which keeps them in LDS).
inline Workspace workspace_carve(const wz_config& c, size_t tiles, size_t slices, char* base, bool split) {
  const size_t T = c.T, N = size_t(c.H) * c.W, C = c.C, Q = c.Q, QP = qpad(c.Q), S = slices;
  Workspace w;
  size_t off = 0;
  auto take = [&](size_t bytes) { char* p = base ? base + off : nullptr; off += align256(bytes); return p; };
  w.s_part = reinterpret_cast<float*>(take(S > 1 ? T * S * N * QP * 4 : 0));
  w.g_part = reinterpret_cast<float*>(take(S > 1 ? T * S * N * 4 : 0));
  w.qg_part = reinterpret_cast<float*>(take(T * S * Q * 4));
  w.sig_part = reinterpret_cast<float*>(take(T * tiles * S * Q * 4));
  w.pool_part = reinterpret_cast<float*>(take(T * tiles * C * 4));
  w.tok_score = reinterpret_cast<float*>(take(T * N * 4));
  w.rank = reinterpret_cast<int32_t*>(take(T * N * 4));
  w.byrank = reinterpret_cast<int32_t*>(take(T * N * 4));
  w.gate = reinterpret_cast<float*>(take(T * N * 4));
  w.gate2 = reinterpret_cast<float*>(take(c.spatial_levels == 2 ? T * N * 4 : 0));
  w.frame_rel = reinterpret_cast<float*>(take(T * 4));
  w.frame_delta = reinterpret_cast<float*>(take(T * 4));
  w.budget = reinterpret_cast<int32_t*>(take(T * 4));
  w.offset = reinterpret_cast<int32_t*>(take((T + 1) * 4));
  const size_t frows = split ? filter_rows_bytes(c) : 0;
  w.frows = frows ? reinterpret_cast<uint16_t*>(take(frows)) : nullptr;
  w.bytes = off;
  return w;
}
inline size_t workspace_bytes_at(const wz_config& c, int tiles, bool split) {
  return workspace_carve(c, tiles, 1, nullptr, split).bytes;
}
inline Workspace workspace_layout(const wz_config& c, char* base, bool split = true) {
  const RelPlan pl = relevance_plan(c);
  return workspace_carve(c, pl.tiles, pl.slices, base, split);
}

// Several videos in one launch: video v = blockIdx.y of every kernel works
// on X + v*x, query + v*q, the workspace and every intermediate kept in it
// + v*ws, out_tokens + v*out, out_index + v*idx, budget + v*bud and
// offset + v*off (byte strides).  Each kernel receives one argument set per
// video, so its body sees a single video.
constexpr int kMaxVideos = 8;
struct Videos {
  int V = 1;
  long long x = 0, q = 0, ws = 0, out = 0, idx = 0, bud = 0, off = 0;
  // the V problems are V queries over one video (x = 0): when shared_pass
  // holds they share one pass over X, and problem v > 0 reads the channel
  // sums of problem 0's workspace
  bool shared_x = false;
};
// queries of one video that one token-tiled pass serves together (its 64
// query columns at most); passes over X share them when this is 2 or more
inline int queries_per_pass(const wz_config& c) { return relevance_kind(c) == kRelTok ? 64 / c.Q : 1; }
inline bool shared_pass(const wz_config& c, int V) { return V > 1 && queries_per_pass(c) >= 2; }
template <typename A>
struct VideoArgs {
  A v[kMaxVideos];
};
template <typename P>
__host__ __device__ inline P* advance(P* p, long long bytes) {
  return p ? reinterpret_cast<P*>(reinterpret_cast<uintptr_t>(p) + bytes) : p;
}
inline Workspace advance(const Workspace& w, long long bytes) {
  Workspace o = w;
  o.s_part = advance(w.s_part, bytes);
  o.g_part = advance(w.g_part, bytes);
  o.qg_part = advance(w.qg_part, bytes);
  o.sig_part = advance(w.sig_part, bytes);
  o.pool_part = advance(w.pool_part, bytes);
  o.tok_score = advance(w.tok_score, bytes);
  o.rank = advance(w.rank, bytes);
  o.byrank = advance(w.byrank, bytes);
  o.gate = advance(w.gate, bytes);
  o.gate2 = advance(w.gate2, bytes);
  o.frame_rel = advance(w.frame_rel, bytes);
  o.frame_delta = advance(w.frame_delta, bytes);
  o.budget = advance(w.budget, bytes);
  o.offset = advance(w.offset, bytes);
  o.frows = advance(w.frows, bytes);
  return o;
}

// Kernel launchers (each returns hipGetLastError() of its launches; `vs`
// batches videos, one by default).
// Streaming pass of stage 1: per-unit partials into ws (and a_{t,n} into
// tok_score unless there are several channel slices).
hipError_t launch_relevance_stream(const wz_config& c, const void* X, const void* query, float* tok_score,
                                   const Workspace& ws, hipStream_t s, const Videos& vs = Videos{});
// Per-frame finish of stage 1: a_{t,n} (several slices), r_t and delta_t;
// with `order` also every frame's selection ranks and block gates (into
// ws.rank, ws.byrank, ws.gate) for launch_assign_gather.
hipError_t launch_frame(const wz_config& c, const Workspace& ws, float* tok_score, float* frame_rel,
                        float* frame_delta, bool order, hipStream_t s, const Videos& vs = Videos{});
// Budgets alone, in one workgroup (wz_temporal_budget, and wz_condense when
// T > kFusedTMax).
hipError_t launch_budget(const wz_config& c, const float* frame_rel, const float* frame_delta, int32_t* budget,
                         int32_t* offset, float* rel_rect, hipStream_t s, const Videos& vs = Videos{});
// Selection, spatial modulation and compaction.  With offset_in the frames'
// row offsets are given; without it (T <= kFusedTMax) every workgroup computes
// the budgets from frame_rel and frame_delta itself and workgroup 0 writes
// them to budget_out / offset_out when those are not null.  With ws the
// frames' ranks and gates come from launch_frame; without it each workgroup
// forms its frame's from tok_score.
hipError_t launch_assign_gather(const wz_config& c, const void* X, const float* tok_score, const float* frame_rel,
                                const float* frame_delta, const int32_t* offset_in, const Workspace* ws,
                                int32_t* budget_out, int32_t* offset_out, void* out_tokens, int32_t* out_index,
                                hipStream_t s, const Videos& vs = Videos{});
// Workgroups per frame of launch_assign_gather for V videos at once.
int assign_groups_per_frame(const wz_config& c, int V = 1);
// Selection, spatial modulation with the db4 / bior4.4 filter bank of
// c.spatial_basis, and compaction, from the scores and the frames' row
// offsets (each workgroup ranks its frame itself).  Needs
// filter_assign_supported(c).
bool filter_assign_supported(const wz_config& c);
// With rank (the per-frame kernel's selection ranks, [T][H*W]) each workgroup
// reads its frame's ranks instead of forming them.  With rows (bf16 inputs; at
// least filter_rows_bytes(c) bytes, 16-byte aligned) the split form runs: a
// row kernel forms each kept token's operator row once per frame into rows,
// then a contraction kernel applies them to the frame's channels; without it
// one fused kernel per (frame, channel slice) forms the rows it uses.
// Whether the filter-bank modulator computes the budgets itself (T <= 64,
// Haar temporal basis, and LDS for them without fewer rows per chunk).
bool filter_budget_folds(const wz_config& c);
// With fb.rel set (filter_budget_folds(c), rank given; offset unused)
// the kernel computes the budgets itself from fb.rel and fb.delta ([T] r_t
// and delta_t) and writes them to fb.budget ([T], may be null) and the row
// offsets to fb.offset ([T+1]).
struct FoldedBudget {
  const float* rel = nullptr;
  const float* delta = nullptr;
  int32_t* budget = nullptr;
  int32_t* offset = nullptr;
};
hipError_t launch_filter_assign(const wz_config& c, const void* X, const float* tok_score, const int32_t* offset,
                                const int32_t* rank, uint16_t* rows, void* out_tokens, int32_t* out_index,
                                hipStream_t s, const Videos& vs = Videos{}, const FoldedBudget& fb = FoldedBudget{});

}  // namespace wz
