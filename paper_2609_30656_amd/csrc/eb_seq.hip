// libeb — un-pooled (sequence) lookup.
//
// Sequence recommenders (the paper's Introduction names HSTU among the
// architectures its profiling targets) consume the embedding of every
// position of a jagged feature instead of a pooled sum.  For table t and
// every position i in [start_t, end_t) = [offsets[t*B], offsets[(t+1)*B]):
//
//   out[base_t + (i - start_t) * D_t + d] = x(t, idx[i], d),   base_t = sum_{s<t} N_s D_s
//
// so table t's positions form a [N_t, D_t] block and the blocks follow in
// table order ([N, D] when all tables share D).  x is the fp32 element value
// of the pooled lookup: each is one exact conversion (or one rounding for
// int8 row-wise rows), so the output matches its definition bit for bit.
//
// Work map: a wavefront takes a span of 64*k consecutive positions (k = 1, or
// 2 for the largest calls, unless EB_BAGS_PER_WAVE says otherwise).  It finds
// the table of its first position once (the lanes test 64 tables' start
// offsets at a time and sum the earlier tables' output sizes), then walks the
// span as a stream of chunks of up to 64 positions inside one table, loading
// the next chunk's indices before the current chunk's rows are gathered.
// Rows are gathered as in the pooled lookup (LPR lanes per row, RPL rows per
// wave-wide load, addresses worked out once per chunk), converted, and stored
// with non-temporal 16-byte stores that fill whole lines (see Piece), through a
// buffer resource over the chunk's part of the output, whose range check keeps
// every store inside it.  The bag offsets inside a table are not read: only the T+1 table
// starts offsets[t*B] matter here.

#include "eb_device.h"

namespace eb {
namespace {

constexpr int64_t kTwoChunksMin = (int64_t)1 << 20;  // chunks of a call from which a wavefront takes two

struct SeqArgs {
  const TableMeta *meta;
  GatherCtx ctx;
  const void *indices;
  const void *offsets;
  float *out;
  int64_t num_indices;
  int64_t out_numel;
  int64_t num_waves;
  int32_t batch;
  int32_t num_tables;
  int32_t idx64;
  int32_t span;  // positions per wavefront, a multiple of 64
};

// offsets[t*B] clamped into [0, N]; *bad is set if it was outside
__device__ __forceinline__ int64_t table_start(const SeqArgs &a, int32_t t, bool *bad) {
  const int64_t g = (int64_t)t * a.batch;
  const int64_t v = a.idx64 ? static_cast<const int64_t *>(a.offsets)[g]
                            : (int64_t) static_cast<const int32_t *>(a.offsets)[g];
  if (v < 0 || v > a.num_indices) {
    *bad = true;
    return v < 0 ? 0 : a.num_indices;
  }
  return v;
}

__device__ __forceinline__ int64_t wave_sum64(int64_t v) {
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// A lane's share of a row in a column window (16 bytes) is read as P pieces
// of PB bytes, piece j of lane slot s at byte col + PB*(s + LPR*j), each
// converted to four fp32 values, so store j of the LPR lanes of a row writes
// one contiguous run.  The stores bound the kernel, and a store instruction
// that covers only half of each 32 bytes costs more than the loads that smaller
// pieces add: with 16-byte pieces of fp16 rows (and 8-byte ones of int8 rows)
// 8 fp16 tables of 128 values at batch 16 384 took 663 us against 396, 26 of
// 64 at batch 2048 126 us against 60, and 26 int8 tables of 128 240 us against
// 146.  Non-temporal stores are 3-30% faster than ordinary ones (428, 82, 151).
template <int DT>
struct Piece {
  static constexpr int bytes = 4 * Vals<DT>::esize;
  static constexpr int count = 16 / bytes;
};

// Lanes that hold a row of LPR 16-byte slices: where a row has fewer than 8
// of them, its pieces go to more lanes instead of following each other in one,
// so that a store still fills whole lines (26 int8 tables of 32, 2 M positions:
// 194 us, now 82; 26 fp16 tables of 32 95, now 77; 2 int8 tables of 16, 0.3 M
// positions 14.5, now 9.1.  Ordinary stores of the partial lines: 131, 103
// and 14.8).
template <int DT, int LPR>
struct RowLanes {
  static constexpr int spread = LPR >= 8 ? 1 : (8 / LPR < Piece<DT>::count ? 8 / LPR : Piece<DT>::count);
  static constexpr int lanes = LPR * spread;
  static constexpr int pieces = Piece<DT>::count / spread;
};

constexpr int kSeqStorePolicy = 2;  // non-temporal

// A chunk's rows go to consecutive rows of the output, so its stores run
// through a buffer resource over just those bytes: a lane's place is a fixed
// offset plus the step's, and a store past the chunk's rows, or past the
// output, is dropped by the range check.
struct ChunkOut {
  __amdgpu_buffer_rsrc_t rows;
};

__device__ __forceinline__ void store4(const ChunkOut &o, uint32_t at, float a, float b, float c, float d) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{a, b, c, d}), o.rows, at, 0, kSeqStorePolicy);
}

// One piece of a row (column byte b of it, or past its end: not stored).
template <int DT, bool BIG>
__device__ __forceinline__ void load_piece(const RowSource<DT, BIG> &src, decltype(RowAddr<BIG>::row) at, int b,
                                           uint32_t (&v)[Piece<DT>::bytes / 4]) {
  constexpr int W = Piece<DT>::bytes / 4;
  if constexpr (W == 4) {
    const u32x4 x = src.load_row(at, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = x[i];
  } else if constexpr (W == 2) {
    const u32x2 x = src.load_row8(at, b);
    v[0] = x[0];
    v[1] = x[1];
  } else {
    v[0] = src.load_row4(at, b);
  }
}

// Write the converted rows of steps [s0, s0 + N) of a chunk, P pieces in each
// of a row's LPR lanes; col is the window's first column byte.
template <int DT, int LPR, int P, int N, bool BIG>
__device__ __forceinline__ void copy_steps(const TableMeta &m, const RowSource<DT, BIG> &src, const RowAddr<BIG> &at,
                                           const ChunkOut &o, int s0, int col) {
  constexpr int RPL = kWave / LPR;
  constexpr int PB = Piece<DT>::bytes;
  constexpr int W = PB / 4;  // dwords per piece
  const int lane = threadIdx.x & (kWave - 1);
  const int grp = lane / LPR;
  const int slot = lane % LPR;
  uint32_t place[P];  // of the lane's pieces in the output rows of step 0
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int b = col + PB * (slot + LPR * j);
    place[j] = b < m.code_bytes ? (uint32_t)(grp * m.dim + b / Vals<DT>::esize) * 4u : kNoOffset;
  }
  uint32_t v[N][P][W];
  uint32_t sb[N];
  decltype(at.row) ar[N], as[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int r = (s0 + u) * RPL + grp;
    ar[u] = RPL == 1 ? from_lane_uniform(at.row, s0 + u) : from_lane(at.row, r);
    if constexpr (DT == kU8) as[u] = RPL == 1 ? from_lane_uniform(at.sb, s0 + u) : from_lane(at.sb, r);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int b = col + PB * (slot + LPR * j);
      load_piece<DT, BIG>(src, ar[u], b < m.code_bytes ? b : 0, v[u][j]);
    }
    sb[u] = 0u;
    if constexpr (DT == kU8) sb[u] = src.load_word(as[u]);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      float x[4];
      if constexpr (DT == kF32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(v[u][j][i]);
      } else if constexpr (DT == kF16) {
#pragma unroll
        for (int i = 0; i < W; ++i) {
          x[2 * i] = half_lo(v[u][j][i]);
          x[2 * i + 1] = half_hi(v[u][j][i]);
        }
      } else {
        // fp32(s*q + c), rounded once, as the dequantisation is defined
        const float sc = half_lo(sb[u]), c = half_hi(sb[u]);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = fmaf(sc, (float)((v[u][j][0] >> (8 * i)) & 0xFFu), c);
      }
      const uint32_t step = (uint32_t)((s0 + u) * RPL * m.dim) * 4u;  // wave-uniform
      store4(o, __builtin_elementwise_add_sat(place[j], step), x[0], x[1], x[2], x[3]);
    }
  }
}

// All rows of one chunk (positions [c, c + k.n) of a table whose block starts
// at output element rowbase for position c), in straight-line batches of up to
// U steps.
template <int DT, int LPR, bool BIG>
__device__ __forceinline__ void copy_chunk(const SeqArgs &a, const TableMeta &m, const Chunk &k, int64_t rowbase) {
  constexpr int LQ = RowLanes<DT, LPR>::lanes, P = RowLanes<DT, LPR>::pieces;
  constexpr int RPL = kWave / LQ;
  constexpr int U = Unroll<DT, RPL, false>::u;
  const int lane = threadIdx.x & (kWave - 1);
  if (__ballot(lane < k.n && k.row == kBadRow)) {
    if (lane == 0) atomicOr(a.ctx.err, kErrIndex);
  }
  const int64_t want = (int64_t)k.n * m.dim, left = a.out_numel - rowbase;
  if (want > left && lane == 0) atomicOr(a.ctx.err, kErrOutSize);
  // the rows that fit (whole pieces of 4 values: every dim is a multiple of 4)
  const int64_t fits = want < left ? want : (left > 0 ? left / 4 * 4 : 0);
  ChunkOut o;
  o.rows = __builtin_amdgcn_make_buffer_rsrc(a.out + uniform64(fits > 0 ? rowbase : 0), 0,
                                             (int)__builtin_amdgcn_readfirstlane((uint32_t)fits * 4u), kBufferFlags);
  const RowSource<DT, BIG> src(m, a.ctx);
  const RowAddr<BIG> at = src.locate(k.row);
  const int steps = (k.n + RPL - 1) / RPL;
  for (int p = 0; p < m.passes; ++p) {
    const int col = p * kPassBytes;
    int s = 0;
    for (; steps - s > U / 2; s += U) copy_steps<DT, LQ, P, U, BIG>(m, src, at, o, s, col);
    const int rem = steps - s;
    if constexpr (U >= 8) {
      if (rem > 2) {
        copy_steps<DT, LQ, P, 4, BIG>(m, src, at, o, s, col);
        continue;
      }
    }
    if constexpr (U >= 4) {
      if (rem > 1) {
        copy_steps<DT, LQ, P, 2, BIG>(m, src, at, o, s, col);
        continue;
      }
    }
    if (rem > 0) copy_steps<DT, LQ, P, 1, BIG>(m, src, at, o, s, col);
  }
}

#define EB_SEQ_LPR(LOG2)                                  \
  case LOG2:                                              \
    copy_chunk<DT, (1 << (LOG2)), BIG>(a, m, ck, rowbase); \
    break;

// DT: the storage type this launch serves (chunks of other tables are
// walked past).  LOG2 >= 0 fixes the lanes per row; LOG2 < 0 switches on each
// table's.
template <int DT, int LOG2, bool BIG>
__global__ __launch_bounds__(kBlock) void eb_seq_kernel(SeqArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t wid = (int64_t)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (wid >= a.num_waves) return;
  const int64_t p0 = wid * a.span;
  const int64_t p1 = (p0 + a.span) < a.num_indices ? (p0 + a.span) : a.num_indices;

  // the table holding p0, its position range, and the first output element of
  // its block (the sizes of the blocks of the tables before it)
  bool bad = false;
  int32_t t = -1;
  int64_t st = 0, en = 0, base = 0;
  for (int32_t g = 0; g < a.num_tables && t < 0; g += kWave) {
    const int32_t l = g + lane;
    int64_t s0 = 0, s1 = 0, before = 0;
    bool mine = false;
    if (l < a.num_tables) {
      s0 = table_start(a, l, &bad);
      s1 = table_start(a, l + 1, &bad);
      if (s1 < s0) {
        bad = true;
        s1 = s0;
      }
      mine = s0 <= p0 && p0 < s1;
      if (s1 <= p0) before = (s1 - s0) * a.meta[l].dim;
    }
    base += wave_sum64(before);
    const uint64_t hit = __ballot(mine);
    if (hit) {
      const int j = __builtin_ctzll(hit);
      t = g + j;
      st = readlane64(s0, j);
      en = readlane64(s1, j);
    }
  }
  if (__ballot(bad) && lane == 0) atomicOr(a.ctx.err, kErrOffsets);
  if (t < 0) {
    if (lane == 0) atomicOr(a.ctx.err, kErrOffsets);  // offsets do not cover this position
    return;
  }

  t = __builtin_amdgcn_readfirstlane(t);
  base = uniform64(base);
  int64_t c = p0;
  int64_t hi = en < p1 ? en : p1;
  hi = (c + kWave) < hi ? (c + kWave) : hi;
  RawChunk cur = load_chunk<false>(a.indices, nullptr, a.idx64, c, hi);
  while (true) {
    // the next chunk: the rest of this table's part of the span, or the next
    // non-empty table's first positions
    int64_t cn = hi;
    int32_t tn = t;
    int64_t stn = st, enn = en, basen = base;
    bool more = cn < p1;
    if (more && cn >= en) {
      bool badn = false;
      while (cn >= enn && tn + 1 < a.num_tables) {
        basen += (enn - stn) * table_meta(a.meta, tn).dim;
        ++tn;
        stn = enn;
        const int64_t e2 = uniform64(table_start(a, tn + 1, &badn));
        enn = e2 < stn ? stn : e2;
        if (e2 < stn) badn = true;
      }
      if (badn && lane == 0) atomicOr(a.ctx.err, kErrOffsets);
      if (cn >= enn || cn != stn) {  // positions past the last table, or a gap
        if (lane == 0) atomicOr(a.ctx.err, kErrOffsets);
        more = false;
      }
    }
    int64_t hin = 0;
    RawChunk nxt;
    if (more) {
      hin = enn < p1 ? enn : p1;
      hin = (cn + kWave) < hin ? (cn + kWave) : hin;
      nxt = load_chunk<false>(a.indices, nullptr, a.idx64, cn, hin);
    }

    const TableMeta m = table_meta(a.meta, t);
    if (m.kind / 8 == DT) {
      const int64_t rowbase = uniform64(base + (c - st) * m.dim);
      const Chunk ck = resolve(cur, m.num_rows, a.idx64);
      if constexpr (LOG2 >= 0) {
        copy_chunk<DT, (1 << (LOG2 >= 0 ? LOG2 : 0)), BIG>(a, m, ck, rowbase);
      } else {
        switch (m.kind % 8) {
          EB_SEQ_LPR(0) EB_SEQ_LPR(1) EB_SEQ_LPR(2) EB_SEQ_LPR(3) EB_SEQ_LPR(4) EB_SEQ_LPR(5) EB_SEQ_LPR(6)
          default:
            break;
        }
      }
    }
    if (!more) break;
    t = tn;
    st = stn;
    en = enn;
    base = basen;
    c = cn;
    hi = hin;
    cur = nxt;
  }
}

#undef EB_SEQ_LPR

typedef void (*SeqKernelFn)(SeqArgs);

template <int DT, bool BIG>
SeqKernelFn pick_seq(int log2) {
  switch (log2) {
    case 0: return eb_seq_kernel<DT, 0, BIG>;
    case 1: return eb_seq_kernel<DT, 1, BIG>;
    case 2: return eb_seq_kernel<DT, 2, BIG>;
    case 3: return eb_seq_kernel<DT, 3, BIG>;
    case 4: return eb_seq_kernel<DT, 4, BIG>;
    case 5: return eb_seq_kernel<DT, 5, BIG>;
    case 6: return eb_seq_kernel<DT, 6, BIG>;
    default: return eb_seq_kernel<DT, -1, BIG>;
  }
}

SeqKernelFn pick_seq(int dt, int log2, bool big) {
  if (dt == kF32) return big ? pick_seq<kF32, true>(log2) : pick_seq<kF32, false>(log2);
  if (dt == kF16) return big ? pick_seq<kF16, true>(log2) : pick_seq<kF16, false>(log2);
  return big ? pick_seq<kU8, true>(log2) : pick_seq<kU8, false>(log2);
}

}  // namespace
}  // namespace eb

using namespace eb;

extern "C" eb_status eb_forward_seq(const eb_tables *h, eb_tensor indices, eb_tensor offsets, eb_tensor out) {
  if (!h) return EB_ERR_INVALID_ARG;
  if (indices.elem_type != EB_I32 && indices.elem_type != EB_I64) return EB_ERR_DTYPE;
  if (offsets.elem_type != indices.elem_type) return EB_ERR_DTYPE;
  if (out.elem_type != EB_T_F32) return EB_ERR_DTYPE;
  if (!offsets.data) return EB_ERR_INVALID_ARG;
  if (indices.numel < 0 || (indices.numel > 0 && !indices.data)) return EB_ERR_INVALID_ARG;
  if (out.numel < 0 || (out.numel > 0 && !out.data)) return EB_ERR_INVALID_ARG;
  if (offsets.numel < 2 || (offsets.numel - 1) % h->num_tables != 0) return EB_ERR_SHAPE;
  const int64_t batch = (offsets.numel - 1) / h->num_tables;
  if (offsets.numel - 1 > INT32_MAX) return EB_ERR_SHAPE;
  const int64_t n = indices.numel;
  // each position writes one row of its table's width
  int32_t min_dim = h->max_dim;
  for (int32_t t = 0; t < h->num_tables; ++t)
    if (h->h_meta[t].dim < min_dim) min_dim = h->h_meta[t].dim;
  if (h->uniform_dim ? out.numel != n * h->uniform_dim : (out.numel < n * min_dim || out.numel > n * h->max_dim))
    return EB_ERR_SHAPE;
  const size_t isz = indices.elem_type == EB_I64 ? 8 : 4;
  if (reinterpret_cast<uintptr_t>(out.data) % 16 != 0 || reinterpret_cast<uintptr_t>(offsets.data) % isz != 0 ||
      reinterpret_cast<uintptr_t>(indices.data) % isz != 0)
    return EB_ERR_UNSUPPORTED;
  if (n == 0) return EB_OK;

  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess) return EB_ERR_HIP;
  if (cur != h->device && hipSetDevice(h->device) != hipSuccess) return EB_ERR_HIP;

  SeqArgs a;
  a.meta = h->d_meta;
  a.ctx.err = h->d_err;
  a.ctx.zero = h->d_zero;
  a.ctx.one = 1.0f;
  a.indices = indices.data;
  a.offsets = offsets.data;
  a.out = static_cast<float *>(const_cast<void *>(out.data));
  a.num_indices = n;
  a.out_numel = out.numel;
  a.batch = (int32_t)batch;
  a.num_tables = h->num_tables;
  a.idx64 = indices.elem_type == EB_I64;
  // One chunk of 64 positions per wavefront (EB_BAGS_PER_WAVE asks for more):
  // wavefronts that end soon keep the writes of neighbouring rows close in
  // time.  About sqrt(chunks / resident wavefronts) chunks, the rule before,
  // were 1-10% slower (8 fp16 tables of 128 at batch 16 384: 415 us against
  // 396; 16 int8 tables of 128, 8.7 M positions: 1 259 against 1 145).  From
  // about a million chunks on, the wavefronts' own set-up costs more than the
  // distance of the writes and two chunks are as fast or faster (one, two,
  // four chunks, ms: 140 M positions in 64 int8 tables of 128 20.3, 19.8, 20.1;
  // in 32 fp32 tables of 64 10.37, 10.17, 10.24; in 32 fp16 tables of 64 9.20,
  // 9.06, 9.29; 72 M in 64 int8 tables 10.74, 10.65, 10.87, in 32 fp16 tables of
  // 128 9.93, 9.95, 10.03; 36 M in 64 int8 tables 5.32, 5.39, 5.51).
  const int64_t chunks = (n + kWave - 1) / kWave;
  const int64_t k = h->bags_per_wave > 0 ? h->bags_per_wave : (chunks >= kTwoChunksMin ? 2 : 1);
  a.span = (int32_t)(k * kWave);
  a.num_waves = (n + a.span - 1) / a.span;

  hipError_t e = begin_checked(h);
  const unsigned grid = (unsigned)((a.num_waves + kWavesPerBlock - 1) / kWavesPerBlock);
  for (int dt = 0; dt < 3 && e == hipSuccess; ++dt) {
    if (!(h->dtype_mask & (1 << dt))) continue;
    hipLaunchKernelGGL(pick_seq(dt, h->single_log2, h->big_tables != 0), dim3(grid), dim3(kBlock), 0, h->stream, a);
    e = hipGetLastError();
  }
  const eb_status st = end_checked(h, e);
  if (cur != h->device) (void)hipSetDevice(cur);
  return st;
}
