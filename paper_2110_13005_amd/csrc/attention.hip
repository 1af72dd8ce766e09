// Fused causal self-attention for gfx950: forward (online softmax, never materialises the
// s x s matrix in HBM) and backward (probabilities recomputed from the stored log-sum-exp).
//
// All contractions run on v_mfma_f32_32x32x16_bf16.  The kernels are arranged so that the
// score tile comes out of the MFMA with the index that is contracted NEXT held in registers
// and the other index on lanes; the rounded tile is then fed straight back as an MFMA operand
// from registers (no LDS round trip):
//   forward, dQ kernel : S^T[key][query] -> lane = query, so max / sum / lse / delta are
//                        per-lane scalars; next contraction is over keys (P V, dS K).
//   dK/dV kernel       : S[query][key]   -> lane = key; next contraction is over queries
//                        (P^T dO, dS^T Q).
// Operands whose contracted index is not contiguous in the [row][d] tiles (V, and Q / dO / K
// in the backward kernels) are fetched with the transposing LDS read.
#include "common.h"
#include "host_logic.h"

#include <type_traits>

namespace axonn {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max(v of this lane, v of lane ^ 32) with v_permlane32_swap: given the same register twice it leaves the lower half-wave's
// values in both halves of one result and the upper half-wave's in both halves of the other.  Unlike a shuffle it does
// not go through the LDS queue, whose results return in order: a shuffle behind a batch of fragment reads waits for all
// of them.
__device__ __forceinline__ float max_with_other_half(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The kernels are compiled for tiles of D = 64, 128 and 192 columns; a head of any dimension d that is a multiple of 4 runs
// in the next of them, from the tile's first column on: which columns a product takes together, and so its rounding, does not
// depend on where in the matrix the head lies.  Chunks behind the head's last column read as zeros; where d is an odd multiple of
// 4, the last chunk is half the next head's (or the end of the matrix), and that half is cleared in LDS.  Zero columns add
// nothing to a product over columns, and result columns outside the head are never stored.
// Every other head then starts between two 16-byte boundaries, which costs the copies little (they take any address): 8 x 24 heads
// of 188 x 512 forward 54.7 us, dQ 69.1, dK / dV 79.5 where the same kernels with tiles that start at the boundary in front of such
// a head took 55.6, 69.6 and 79.8.
struct HeadColumns {
  int d;
  __device__ __forceinline__ int chunks() const { return (d + 7) >> 3; }
  __device__ __forceinline__ bool split() const { return d & 4; }
  // byte within a row of the half chunk behind the head
  __device__ __forceinline__ int foreign() const { return 2 * d; }
  __device__ __forceinline__ bool has4(int col) const { return col + 4 <= d; }
};

// LDS tile of R rows x D columns: D / 64 blocks of 64 columns, each R rows of 128 bytes, no padding.  Row r holds its 16-byte
// chunk c in place c ^ swizzle(r).  Both ways of reading are free of bank conflicts: 128-bit reads of 16 rows at one chunk
// find 16 different places of the 256 bytes that two rows span, and the transposing 64-bit reads, which take 64 bytes from
// each of 4 consecutive rows per half wave, find 4 different 64-byte quarters of it.  Clocks per wave instruction: 4.0 and
// 2.3; with padded rows (76 words, the best stride for both) 4.0 and 4.0.  A tile is filled by the memory pipeline,
// 1 KB (8 rows of one block) per instruction.
struct LdsBytes {                     // a place in LDS, without the checks of a generic pointer's conversions
  AXONN_LDS char* p;
  __device__ __forceinline__ explicit LdsBytes(char* shared) : p((AXONN_LDS char*)shared) {}
  __device__ __forceinline__ LdsBytes operator+(uint32_t bytes) const { LdsBytes r = *this; r.p += bytes; return r; }
};
__device__ __forceinline__ int tile_swizzle(int row) { return ((row & 2) << 1) | ((row >> 2) & 3); }
template <int R, int D>
struct Tile {
  static constexpr int BYTES = R * D * 2, BLOCK = R * 128;
  static __device__ __forceinline__ int chunk_at(int row, int ch) { return (ch >> 3) * BLOCK + row * 128 + (((ch & 7) ^ tile_swizzle(row)) << 4); }
};
// What a lane adds to a tile's address for its fragments: k-contiguous ones (MFMA operand rows = tile rows, contracted
// over columns) by the fragment's columns modulo 64, k-strided ones (operand rows = tile columns, contracted over tile
// rows, in the order in which an MFMA result tile keeps its m index in registers) by the fragment's columns modulo 64
// and the half of its 16 tile rows.
struct FragLanes {
  uint32_t kc[4], tr[2][2];
  __device__ __forceinline__ FragLanes(int lane) {
    const int g = lane >> 5, row = lane & 31;
#pragma unroll
    for (int j = 0; j < 4; ++j) kc[j] = row * 128 + (((2 * j + g) ^ tile_swizzle(row)) << 4);
    const int t = lane & 15, half = (lane >> 4) & 1;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int hi = 0; hi < 2; ++hi) {
        const int r = 8 * hi + 4 * g + (t >> 2), ch = 4 * b + 2 * half + ((t & 3) >> 1);
        tr[b][hi] = r * 128 + ((ch ^ tile_swizzle(r)) << 4) + ((t & 1) << 3);
      }
  }
};
// rows 32 r32 .., columns 16 kk ..
template <int R, int D>
__device__ __forceinline__ elemx8 frag_rows(LdsBytes tile, const FragLanes& f, int r32, int kk) {
  return *(const AXONN_LDS elemx8*)(tile.p + ((kk >> 2) * Tile<R, D>::BLOCK + r32 * (32 * 128)) + f.kc[kk & 3]);
}
// columns 32 dt .., rows 16 r16 ..
template <int R, int D>
__device__ __forceinline__ elemx8 frag_cols(LdsBytes tile, const FragLanes& f, int r16, int dt) {
  AXONN_LDS char* p = tile.p + ((dt >> 1) * Tile<R, D>::BLOCK + r16 * (16 * 128));
  union { elemx8 v; short4v h[2]; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((AXONN_LDS short4v*)(p + f.tr[dt & 1][0]));
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((AXONN_LDS short4v*)(p + f.tr[dt & 1][1]));
  return u.v;
}

// Fills tiles with rows of one head of a [rows][ld] matrix; rows beyond the last one read as zeros.  The descriptor starts at
// the tile's first row, so that offsets stay small for any sequence length.
template <int D, bool FITS>
struct TileSource {
  const elem_t* base;                  // row 0, the head's first column
  uint32_t row_bytes, row_end;         // row_end: bytes of a row up to the head's last column
  int rows;
  uint32_t v, v_last;                  // lane offset of its chunk of block 0, and of the last block (or out of range)
  uint32_t clear;                      // LDS place in a tile's first rows that this lane clears of what lies behind the head
  HeadColumns cols;
  int lane, wave;
  __device__ __forceinline__ TileSource(const elem_t* head, int64_t ld, int rows, HeadColumns cols, int tid)
      : base(head), row_bytes((uint32_t)ld * 2u), row_end((uint32_t)cols.d * 2u), rows(rows), cols(cols),
        lane(tid & 63), wave(__builtin_amdgcn_readfirstlane(tid >> 6)) {
    // wave w fills row blocks w, w + 4, ...: their swizzle is the same
    const int r = 8 * wave + (lane >> 3), ch = (lane & 7) ^ tile_swizzle(r);
    v = (uint32_t)r * row_bytes + (uint32_t)ch * 16u;
    v_last = 8 * (D / 64 - 1) + ch < cols.chunks() ? v + (D / 64 - 1) * 128u : kOutOfRange;
    const int cr = 8 * wave + (lane & 7), at = cols.foreign();
    clear = (uint32_t)cr * 128u + ((((at >> 4) & 7) ^ tile_swizzle(cr)) << 4) + (at & 8);
  }
  // the R rows from row0 on
  template <int R>
  __device__ __forceinline__ void fill(LdsBytes tile, int row0) const {
    if (!FITS) { fill_long<R>(tile, row0); return; }
    const Copies<R> c = copies<R>(tile, row0);
#pragma unroll
    for (int i = 0; i < Copies<R>::N; ++i) c.one(i, *this);
  }
  // The same one instruction at a time.
  template <int R>
  struct Copies {
    static constexpr int N = R / 32 * (D / 64);
    u32x4 rsrc;
    uint32_t lds;
    __device__ __forceinline__ void one(int i, const TileSource& s) const {
      const int block = i % (D / 64), r32 = i / (D / 64);
      const uint32_t v = block == D / 64 - 1 ? s.v_last : s.v + block * 128u;
      dma_chunk16(rsrc, v + (uint32_t)(32 * r32) * s.row_bytes, 0, lds + block * Tile<R, D>::BLOCK + r32 * (32 * 128));
    }
  };
  template <int R>
  __device__ __forceinline__ Copies<R> copies(LdsBytes tile, int row0) const {
    Copies<R> c;
    const int left = min(rows - row0, R);
    c.rsrc = rsrc_words(base + (int64_t)row0 * (row_bytes >> 1), left > 0 ? (uint32_t)(left - 1) * row_bytes + row_end : 0u);
    c.lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)tile.p) + (uint32_t)wave * 1024u;
    return c;
  }
  // Rows too long for 32-bit offsets: through registers.
  template <int R>
  __device__ __forceinline__ void fill_long(LdsBytes tile, int row0) const {
#pragma unroll 1
    for (int i = 64 * wave + lane; i < R * (D / 8); i += 256) {
      const int r = i / (D / 8), ch = i % (D / 8), row = row0 + r;
      const elem_t* p = base + (int64_t)row * (row_bytes >> 1) + ch * 8;
      uint2 lo = make_uint2(0, 0), hi = make_uint2(0, 0);
      if (row < rows && cols.has4(8 * ch)) lo = *reinterpret_cast<const uint2*>(p);
      if (row < rows && cols.has4(8 * ch + 4)) hi = *reinterpret_cast<const uint2*>(p + 4);
      *(AXONN_LDS u32x4*)(tile.p + Tile<R, D>::chunk_at(r, ch)) = u32x4{lo.x, lo.y, hi.x, hi.y};
    }
  }
  // Behind the wait for this wave's copies and in front of the barrier: clears what they brought from behind the head.
  template <int R>
  __device__ __forceinline__ void clear_foreign(LdsBytes tile) const {
    if (!cols.split()) return;
    AXONN_LDS char* p = tile.p + (cols.foreign() >> 7) * Tile<R, D>::BLOCK + clear;
#pragma unroll
    for (int r32 = 0; r32 < R / 32; ++r32)
      if (lane < 8) *(AXONN_LDS u32x2*)(p + r32 * (32 * 128)) = u32x2{0, 0};
  }
};

__device__ __forceinline__ elemx8 pack8(const floatx16& t, int first) {
  elemx8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (elem_t)t[first + e];
  return o;
}

// Work assignment of the attention kernels: block id of a 1-D grid of n_tiles * n_bh blocks -> (rank of
// the tile, batch*head index).  Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its
// own, so XCD x gets ids x, x+8, ...: those are mapped to a contiguous range of (batch, head) pairs, so
// that the K/V (or Q/dO) rows of a head are fetched into one L2 instead of all eight; inside the range
// the tiles of rank 0 (the longest-running ones under causal masking) of every head come first.
// The divisions are by numbers whose reciprocals come with the arguments: of the instructions in front of the first copy, which
// the smallest launches feel, they were half.  2 x 4 heads of 64 x 128 forward 5.20 -> 5.12 us, of 64 x 64 4.34 -> 4.14.
struct AttnWalk { uint32_t xcds, block, heads; };   // blocks are dealt by XCD (1) or not (0); reciprocals of a block row's length and of a
__device__ __forceinline__ void attn_block(uint32_t id, uint32_t n_bh, uint32_t a, AttnWalk w, int& rank, int& bi, int& hd) {
  const uint32_t len = w.xcds ? n_bh >> 3 : n_bh, j = w.xcds ? id >> 3 : id;     // j-th block of XCD id % 8
  rank = host::recip_div(j, len, w.block);
  const uint32_t bh = j - rank * len + (w.xcds ? (id & 7) * len : 0);
  bi = host::recip_div(bh, a, w.heads);
  hd = bh - bi * a;
}

// One wave's 32 x D result (the MFMA result layout: lane = row lane % 32, registers 4q .. 4q+3 of tile dt = columns
// 32 dt + 8 q + 4 (lane / 32) ..) times `mul`, rounded, to rows of `ld` elements at `head`, through LDS: stored straight from
// the MFMA layout every lane touches a row of its own, 8 bytes at a time, a memory instruction then covers 32 different
// lines, and the last stores alone took a tenth of the dK / dV kernel's time.  `stage` is 32 x (D + 8) elements of LDS that
// only this wave touches (no barrier: a wave's LDS operations keep their order).  Rows and columns that do not exist are stored out of
// a descriptor's range instead of behind branches.
template <int D, bool FITS>
__device__ __forceinline__ void store_rows_out(char* lds, const floatx16* acc, float mul, elem_t* head, int64_t ld,
                                               int n_rows, HeadColumns cols, int lane) {
  constexpr int LDO = D + 8, DT = D / 32, CPR = D / 8;      // 16-byte chunks per row
  asm volatile("" : "+v"(lane));      // places and offsets are computed here, not in front of the loop and kept through it
  elem_t* const stage = reinterpret_cast<elem_t*>(lds);
  const int g = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      elemx4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (elem_t)(acc[dt][4 * q + e] * mul);
      *reinterpret_cast<elemx4*>(stage + (lane & 31) * LDO + dt * 32 + 8 * q + 4 * g) = v;
    }
  if (FITS) {
    const uint32_t row_bytes = (uint32_t)ld * 2u;
    const int rows = min(n_rows, 32);
    const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(head, rows > 0 ? (uint32_t)(rows - 1) * row_bytes + (uint32_t)cols.d * 2u : 0u);
#pragma unroll
    for (int j = 0; j < 32 * CPR / 64; ++j) {
      const int idx = lane + 64 * j, row = idx / CPR, ch = idx % CPR;
      const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * LDO + ch * 8);
      __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, cols.has4(8 * ch + 4) ? row * row_bytes + ch * 16 : kOutOfRange, 0, 0);
    }
    if (cols.split()) {             // the half chunk in front of another head's
      const u32x2 v = *reinterpret_cast<const u32x2*>(stage + (lane & 31) * LDO + cols.d - 4);
      __builtin_amdgcn_raw_buffer_store_b64(v, rsrc, g == 0 ? lane * row_bytes + (uint32_t)(cols.d - 4) * 2u : kOutOfRange, 0, 0);
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < 32 * CPR / 64; ++j) {
    const int idx = lane + 64 * j, row = idx / CPR, ch = idx % CPR;
    const uint4 v = *reinterpret_cast<const uint4*>(stage + row * LDO + ch * 8);
    if (row >= n_rows) continue;
    elem_t* const p = head + (int64_t)row * ld + ch * 8;
    if (cols.has4(8 * ch + 4)) *reinterpret_cast<uint4*>(p) = v;
    else if (cols.has4(8 * ch)) *reinterpret_cast<uint2*>(p) = make_uint2(v.x, v.y);
  }
}

// =============================================================================== forward
// grid: ceil(s/128) * b * a workgroups; 4 waves; wave w owns queries q0 + 32w .. +31 and walks the key tiles up to the diagonal.
//
// Two workgroups share a CU, two waves a SIMD; what bounds a wave is the chain of a tile's steps.  So the LDS reads of one step
// run beside the MFMAs of another: the V fragments of a tile beside its score MFMAs, the K fragments of the next tile
// beside the P V MFMAs, and the memory pipeline fills a tile's buffer a whole tile ahead.  K and V fragments being in
// registers when the barrier of a tile is reached, its buffer is free behind it: two buffers and one barrier per tile.
// Against tiles fetched into registers, stored between two barriers, and each tile's fragments read in one go, us: 40 heads of
// 128 x 2048 58.0 -> 52.0, 16 of 128 x 8192 311 -> 278 (990 TFLOP/s), 8 x 16 of 64 x 1024 28.4 -> 27.1, 8 x 24 of 188 x 512 (every
// lane on a row of its own, 8 bytes at a time) 76 -> 50.6, 2 x 36 of 176 x 2048 256 -> 153.
template <int D, bool FITS>
__global__ __launch_bounds__(256, D > 128 ? 1 : 2) void attn_fwd_kernel(int s, int a, int n_bh, AttnWalk walk, int d,
                                                                        const elem_t* __restrict__ qkv,
                                                                        elem_t* __restrict__ o,
                                                                        float* __restrict__ lse) {
  constexpr int BKV = 64, DT = D / 32, KK = D / 16, BUF = 2 * Tile<BKV, D>::BYTES;
  constexpr int STAGED = 128 * (D + 8) * 2;
  // K and V tile, two of each, and at the end the O rows.  The Q rows lie in the second pair's place first; at D = 64 LDS has room
  // for one of their own, and the second pair is on its way from the start (8 heads of 1016 rows 15.3 -> 15.0 us).
  constexpr bool OWN_Q = D == 64;
  constexpr int Q_AT = OWN_Q ? 2 * BUF : BUF;
  __shared__ __align__(1024) char smem[Q_AT + Tile<128, D>::BYTES];
  static_assert(Tile<128, D>::BYTES == BUF && STAGED <= Q_AT + BUF, "rows staged in the tile buffers");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  int rank, bi, hd;
  attn_block(blockIdx.x, n_bh, a, walk, rank, bi, hd);
  const int qt = (s + 127) / 128 - 1 - rank;  // longest rows first
  const int h = a * d;
  const int64_t ld = 3 * (int64_t)h;
  const elem_t* qb = qkv + (int64_t)bi * s * ld + hd * d;
  const int q0 = qt * 128, qw0 = q0 + 32 * wave, qi = qw0 + (lane & 31);
  const float scale_log2 = kLog2e * rsqrtf((float)d);
  const HeadColumns cols{d};
  const FragLanes fl(lane);
  const int kv_end = min(s, q0 + 128);         // keys behind the workgroup's last query are not fetched
  const TileSource<D, FITS> q_src(qb, ld, s, cols, tid), k_src(qb + h, ld, kv_end, cols, tid), v_src(qb + 2 * h, ld, kv_end, cols, tid);

  const LdsBytes buf0(smem);
  q_src.template fill<128>(buf0 + Q_AT, q0);
  k_src.template fill<BKV>(buf0, 0);
  v_src.template fill<BKV>(buf0 + Tile<BKV, D>::BYTES, 0);
  auto fill_second = [&]() {
    k_src.template fill<BKV>(buf0 + BUF, BKV);
    v_src.template fill<BKV>(buf0 + BUF + Tile<BKV, D>::BYTES, BKV);
  };
  if (OWN_Q) {
    fill_second();
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(FITS ? 2 * TileSource<D, FITS>::template Copies<BKV>::N : 0) : "memory");
  } else {
    dma_wait_all();
  }
  q_src.template clear_foreign<128>(buf0 + Q_AT);
  k_src.template clear_foreign<BKV>(buf0);
  __syncthreads();
  elemx8 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk] = frag_rows<128, D>(buf0 + Q_AT, fl, wave, kk);

  floatx16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  const int n_kt = (kv_end + BKV - 1) / BKV;
  // the wave's own: a last tile with every key in its future is left out (0 x Inf and 0 x NaN are not 0)
  const int n_own = min(n_kt, (qw0 + 31) / BKV + 1);
  // Fragments of a tile in the order of the MFMAs that take them: K's alternate between the tile's two 32-key halves.
  auto k_frag = [&](LdsBytes buf, int i) { return frag_rows<BKV, D>(buf, fl, i & 1, i >> 1); };
  auto v_frag = [&](LdsBytes buf, int i) { return frag_cols<BKV, D>(buf + Tile<BKV, D>::BYTES, fl, i / DT, i % DT); };
  constexpr int NF = 2 * KK;                     // fragments of a K tile, and of a V tile
  static_assert(NF == 4 * DT, "one V fragment per score MFMA and one K fragment per P V MFMA");
  constexpr int EARLY = D == 128 ? 12 : NF;      // the other V fragments find registers when the scores have left theirs
  elemx8 kfr[NF], vfr[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) kfr[i] = k_frag(buf0, i);
  if (!OWN_Q && n_kt > 1) {
    __syncthreads();                             // the Q rows have been read
    fill_second();
  }
  for (int kt = 0; kt < n_own; ++kt) {
    const int k0 = kt * BKV;
    const LdsBytes buf = buf0 + (kt & 1) * BUF, next = buf0 + (~kt & 1) * BUF;
    floatx16 sacc[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[ks][r] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      sacc[i & 1] = mfma32(kfr[i], qf[i >> 1], sacc[i & 1]);
      if (i < EARLY) vfr[i] = v_frag(buf, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    // Keys beyond the query are masked in the tiles that straddle the diagonal only: a real (wave-uniform)
    // branch, so that the other tiles do not pay for the comparisons.
    if (k0 + BKV - 1 > qw0) {
      asm volatile("" ::: "memory");            // keeps the compiler from turning the branch into selects
      const int last = qi - k0 - 4 * g;         // the lane's last key, counted from its first one
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if (32 * ks + 8 * (r >> 2) + (r & 3) > last) sacc[ks][r] = -INFINITY;
        }
    }
    // Row maximum of the raw scores; in units of the exponent (log2) it is mx * scale_log2 (the scale is positive).
    float mx = sacc[0][0];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[ks][r]);
    mx = max_with_other_half(mx) * scale_log2;
    // m_run is the reference point of the exponentials, not necessarily the running maximum: it moves (and the
    // sums so far are rescaled) only when some row's maximum has grown by more than 2^8 since it was set, so
    // most tiles skip the rescaling; p stays <= 256 and the result is the same up to rounding.
    if (__builtin_amdgcn_ballot_w64(mx > m_run + 8.0f) != 0) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
    }
    const float neg_m = -m_run;
    float psum = 0.f;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = fast_exp2(fmaf(sacc[ks][r], scale_log2, neg_m));
        sacc[ks][r] = p;
        psum += p;
      }
    l_run += psum;
    elemx8 pf[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) pf[c] = pack8(sacc[c >> 1], 8 * (c & 1));
#pragma unroll
    for (int i = EARLY; i < NF; ++i) vfr[i] = v_frag(buf, i);
    // The next tile is in LDS, and everybody has taken this one's fragments: its buffer is filled with the tile after next
    // (behind the last tile too: the copies write, and other waves may still read its V).
    if (kt + 1 < n_kt) {
      dma_wait_all();
      k_src.template clear_foreign<BKV>(next);
    }
    __syncthreads();
    if (!FITS && kt + 2 < n_kt) {
      k_src.template fill<BKV>(buf, k0 + 2 * BKV);
      v_src.template fill<BKV>(buf + Tile<BKV, D>::BYTES, k0 + 2 * BKV);
    }
    // one copy per two MFMAs: in one go in front of them they take as long as half of them
    const auto ck = k_src.template copies<BKV>(buf, k0 + 2 * BKV), cv = v_src.template copies<BKV>(buf + Tile<BKV, D>::BYTES, k0 + 2 * BKV);
    static_assert(4 * TileSource<D, FITS>::template Copies<BKV>::N == NF, "copies and MFMAs");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      oacc[i % DT] = mfma32(vfr[i], pf[i / DT], oacc[i % DT]);
      kfr[i] = k_frag(next, i);
      if (FITS && i % 4 == 0) ck.one(i / 4, k_src);
      if (FITS && i % 4 == 2) cv.one(i / 4, v_src);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (n_own < n_kt) __syncthreads();
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  dma_wait_all();                 // copies of tiles beyond the last still write (zeros) to LDS
  __syncthreads();                // the tiles in LDS are done with
  store_rows_out<D, FITS>(smem + wave * (STAGED / 4), oacc, 1.f / l_tot, o + ((int64_t)bi * s + qw0) * h + hd * d, h, s - qw0, cols, lane);
  if (g == 0 && qi < s) lse[((int64_t)bi * a + hd) * s + qi] = (m_run + __log2f(l_tot)) * kLn2;
}

// ============================================================================ backward
// delta[b][a][i] = sum_d dO[i][d] * O[i][d]
// p + the products of elements first .. first + N - 1, one after the other (PAIRS: half precision in two-element dot
// products).  Both forms are fixed here: left to contraction, which of them a sum gets depends on the kernel around it.
template <int N, bool PAIRS, class V>
__device__ __forceinline__ float delta_add(float p, V ov, V dv, int first) {
#ifdef AXONN_ELEM_FP16
  if (PAIRS) {
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int e = first; e < first + N; e += 2)
      p = __builtin_amdgcn_fdot2(halfx2{ov[e], ov[e + 1]}, halfx2{dv[e], dv[e + 1]}, p, false);
    return p;
  }
#endif
  {
#pragma clang fp contract(off)
#pragma unroll
    for (int e = first; e < first + N; ++e) p = __builtin_fmaf((float)ov[e], (float)dv[e], p);
  }
  return p;
}
// For any head dimension d that is a multiple of 4: 16 lanes per (row, head), 4 elements per lane and step.
// (Launched in front of the one-launch backward and where d is not 64 or 128; at those the dQ kernel in a launch of its own forms
// delta itself.)
__global__ __launch_bounds__(256) void attn_delta_general_kernel(int64_t n_pairs, int s, int a, int d,
                                                                 const elem_t* __restrict__ o,
                                                                 const elem_t* __restrict__ dout,
                                                                 float* __restrict__ delta) {
  const int64_t pair = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);   // (row, head)
  const int j = threadIdx.x & 15;
  float p = 0.f;
  if (pair < n_pairs) {
    const elem_t* op = o + pair * d;          // rows are a * d long: pair * d = row * a * d + head * d
    const elem_t* dp = dout + pair * d;
    for (int c = 4 * j; c < d; c += 64) {
      p = delta_add<4, true>(p, *reinterpret_cast<const elemx4*>(op + c), *reinterpret_cast<const elemx4*>(dp + c), 0);
    }
  }
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) p += __shfl_xor(p, off, 64);
  if (pair < n_pairs && j == 0) {
    const int64_t row = pair / a;
    const int hd = (int)(pair % a);
    const int64_t bi = row / s, i = row % s;
    delta[(bi * a + hd) * s + i] = p;
  }
}

// dK / dV: one workgroup per tile of 128 keys and (batch, head); wave w owns keys k0 + 32w .. +31 and walks the query tiles at or below the
// diagonal.  The Q / dO tiles alternate between two LDS buffers, which the memory pipeline fills.
//
// A wave is alone on its SIMD (accumulators and K / V fragments take most of the register file), so nothing hides the
// MFMA phases of a 32-query block behind its exponentials, or an LDS round trip behind an MFMA, unless the instruction
// stream does.  The blocks of all tiles form one pipeline.  Step k of a tile issues the score MFMAs (S and dP) of block k + 1
// and the gradient MFMAs (dV and dK) of block k; half of block k + 1's exponentials run beside the gradient MFMAs, the other
// half beside the next step's score MFMAs.  A step is a run of slots: one MFMA, the LDS read of the fragment that the MFMA
// W - 1 slots later needs (a ring of W fragments, also across tiles), and a share of the exponentials.  The MFMAs are
// volatile assembly: they keep this order, and the reads stay between them where they are written.  The tile on the diagonal
// takes the same path with the mask applied to every element (a block above the diagonal comes out as zeros; the wave with
// the lowest keys needs all blocks anyway).  Zeros times infinities are not zeros: above 128 columns the gradient MFMAs of a
// block in front of the wave's keys are jumped over, so that what it holds does not reach their gradients.
// What bounds a slot is what one wave issues: a vector instruction takes 5 clocks of its 32, an exponential 9, a conversion of
// two elements 8; and the LDS, which gives a transposed fragment in 4.6 clocks without bank conflicts and in 8 with the two-way
// ones of padded rows.  40 heads of 128 x 2048 125 -> 112 us, 16 of 128 x 8192 535 -> 477, 8 x 16 of 64 x 1024 60 -> 44 (two waves
// per SIMD here, at 256 registers), against wait states in front of every MFMA, padded rows, tiles fetched into registers and
// all of a block's exponentials beside 16 of its slots; 8 x 24 of 188 x 512 (block by block, tiles of 64) 119 -> 75.
template <int D>
struct DkdvLds {
  static constexpr int BQ = D <= 128 ? 128 : 64, TILE = Tile<BQ, D>::BYTES, BUF = 2 * TILE, KEYS = Tile<128, D>::BYTES;
  // the second buffer holds the workgroup's K and V rows first
  __align__(1024) char tiles[BUF + (2 * KEYS > BUF ? 2 * KEYS : BUF)];
  __align__(16) float lse[2][BQ];
  __align__(16) float delta[2][BQ];
};
template <int D, bool FITS>
__device__ __forceinline__ void attn_bwd_dkdv(
    DkdvLds<D>& lds, int id, int s, int a, int n_bh, AttnWalk walk, int d, const elem_t* __restrict__ qkv,
    const elem_t* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ delta,
    elem_t* __restrict__ dqkv) {
  using L = DkdvLds<D>;
  constexpr int BQ = L::BQ, DT = D / 32, KK = D / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  int rank, bi, hd;
  attn_block(id, n_bh, a, walk, rank, bi, hd);    // key tile `rank` walks n_tiles - rank query tiles: longest first
  const int h = a * d;
  const int64_t ld = 3 * (int64_t)h;
  const elem_t* qb = qkv + (int64_t)bi * s * ld + hd * d;
  const float* lse_b = lse + ((int64_t)bi * a + hd) * s;
  const float* delta_b = delta + ((int64_t)bi * a + hd) * s;
  const int k0 = rank * 128, kw0 = k0 + 32 * wave, kj = kw0 + (lane & 31);
  const float scale = rsqrtf((float)d), scale_log2 = kLog2e * scale;
  const HeadColumns cols{d};
  const FragLanes fl(lane);
  const TileSource<D, FITS> q_src(qb, ld, s, cols, tid), k_src(qb + h, ld, s, cols, tid), v_src(qb + 2 * h, ld, s, cols, tid),
      do_src(dout + (int64_t)bi * s * h + hd * d, h, s, cols, tid);
  const int qt_begin = k0 / BQ, n_qt = (s + BQ - 1) / BQ;
  const LdsBytes keys(lds.tiles + L::BUF), tile0(lds.tiles);

  float r_lse, r_delta;
  // by all threads, so that no branch stands in the stream of MFMAs: those beyond the tile's rows repeat the others' work
  auto fetch_stats = [&](int qt) {
    const int at = min(qt * BQ + (tid & (BQ - 1)), s - 1);
    r_lse = lse_b[at];
    r_delta = delta_b[at];
  };
  auto store_stats = [&](int buf, int qt) {
    const bool in = qt * BQ + (tid & (BQ - 1)) < s;
    lds.lse[buf][tid & (BQ - 1)] = in ? r_lse * kLog2e : 0.f;
    lds.delta[buf][tid & (BQ - 1)] = in ? r_delta : 0.f;
  };
  k_src.template fill<128>(keys, k0);
  v_src.template fill<128>(keys + L::KEYS, k0);
  fetch_stats(qt_begin);
  q_src.template fill<BQ>(tile0, qt_begin * BQ);
  do_src.template fill<BQ>(tile0 + L::TILE, qt_begin * BQ);
  store_stats(0, qt_begin);
  dma_wait_all();
  k_src.template clear_foreign<128>(keys);
  v_src.template clear_foreign<128>(keys + L::KEYS);
  q_src.template clear_foreign<BQ>(tile0);
  do_src.template clear_foreign<BQ>(tile0 + L::TILE);
  fetch_stats(qt_begin + 1);
  __syncthreads();
  elemx8 kf[KK], vf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    kf[kk] = frag_rows<128, D>(keys, fl, wave, kk);
    vf[kk] = frag_rows<128, D>(keys + L::KEYS, fl, wave, kk);
  }
  floatx16 dvacc[DT], dkacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) dvacc[dt][r] = dkacc[dt][r] = 0.f;
  // K fragments move to the accumulation registers, which the MFMAs below read them from; V's too where these hold both
  constexpr bool VF_ACC = D <= 128;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    asm volatile("" : "+a"(kf[kk]));
    if (VF_ACC) asm volatile("" : "+a"(vf[kk]));
  }
  // the zeros are in place here, not written in front of an accumulator's first MFMA
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) asm volatile("" : "+a"(dvacc[dt]), "+a"(dkacc[dt]));

  constexpr int NB = BQ / 32, NS = 2 * KK, NG = 4 * DT, STEP = NS + NG, NSLOT = NB * STEP, W = 8;
  static_assert(NB % 2 == 0 && NSLOT % W == 0 && NS % W == 0 && NG == NS, "block parity and ring position are the same in every tile");
  floatx16 sacc[2], pacc[2];            // scores and dP of two blocks: one being formed, one in its exponentials
  uint32_t pfw[2][8], dsw[2][8];        // P and dS of a block rounded to 16 bits, two per word: MFMA operands
  floatx4 l4[2], d4[2];                 // log-sum-exp and delta of the four queries of a group; two groups in flight
  elemx8 ring[W];
  // A block number is counted from the current tile's first block; block NB is the next tile's first one.
  auto load_stats = [&](int buf, int blk, int q4) {
    const int b = blk < NB ? buf : buf ^ 1, at = 32 * (blk % NB) + 8 * q4 + 4 * g;
    l4[q4 & 1] = *reinterpret_cast<const floatx4*>(&lds.lse[b][at]);
    d4[q4 & 1] = *reinterpret_cast<const floatx4*>(&lds.delta[b][at]);
  };
  // element r of block blk: P = exp(S - lse), dS = P (dP - delta), rounded once a pair of elements is complete.  Masked:
  // keys beyond the query get no weight; `first`: the lane's key counted from the query of the tile's first row and its half.
  auto softmax_elem = [&](int buf, int blk, int r, bool masked, int first) {
    const int hf = blk & 1, q4 = r >> 2;
    float x = fmaf(sacc[hf][r], scale_log2, -l4[q4 & 1][r & 3]);
    if (masked && first > 32 * blk + 8 * q4 + (r & 3)) x = -INFINITY;
    const float p = fast_exp2(x);
    sacc[hf][r] = p;
    pacc[hf][r] = p * (pacc[hf][r] - d4[q4 & 1][r & 3]);
    if (r & 1) {
      elemx2 pp, dd;
      pp[0] = (elem_t)sacc[hf][r - 1]; pp[1] = (elem_t)sacc[hf][r];
      dd[0] = (elem_t)pacc[hf][r - 1]; dd[1] = (elem_t)pacc[hf][r];
      pfw[hf][r >> 1] = __builtin_bit_cast(uint32_t, pp);
      dsw[hf][r >> 1] = __builtin_bit_cast(uint32_t, dd);
    }
    // the group after next into the pair just used up
    if ((r & 3) == 3) load_stats(buf, q4 + 2 < 4 ? blk : blk + 1, (q4 + 2) & 3);
  };
  auto operand = [&](const uint32_t* w, int c) {
    return __builtin_bit_cast(elemx8, make_uint4(w[4 * c], w[4 * c + 1], w[4 * c + 2], w[4 * c + 3]));
  };
  // score MFMA i of block blk, and its fragment
  auto score_frag = [&](int buf, int blk, int i) -> elemx8 {
    const int b = blk < NB ? buf : buf ^ 1;
    return frag_rows<BQ, D>(tile0 + b * L::BUF + (i & 1) * L::TILE, fl, blk % NB, i >> 1);
  };
  auto score_mfma = [&](int blk, int i, elemx8 f) {
    const int hf = blk & 1, kk = i >> 1;
    if (i & 1) {
      if (kk == 0) mfma32_vgpr_zero<VF_ACC>(pacc[hf], f, vf[kk]); else mfma32_vgpr<VF_ACC>(pacc[hf], f, vf[kk]);
    } else {
      if (kk == 0) mfma32_vgpr_zero<true>(sacc[hf], f, kf[kk]); else mfma32_vgpr<true>(sacc[hf], f, kf[kk]);
    }
  };
  // slot j of a tile: within its step k the score slots of block k + 1, then the gradient slots of block k; slots beyond
  // the last are the next tile's first ones
  auto load_frag = [&](int buf, int j) -> elemx8 {
    if (j >= NSLOT) { buf ^= 1; j -= NSLOT; }
    const int k = j / STEP, i = j % STEP;
    if (i < NS) return score_frag(buf, k + 1, i);
    const int gi = i - NS, c = gi / (2 * DT), dt = (gi % (2 * DT)) >> 1;
    return frag_cols<BQ, D>(tile0 + buf * L::BUF + (gi & 1 ? 0 : L::TILE), fl, 2 * k + c, dt);
  };
  // The next tile is copied into the other buffer during the first steps of a tile, one instruction per slot, and its first
  // block is read from slot READY on.  Rows beyond the sequence read as zeros, so a tile beyond the last one needs no case of
  // its own.
  constexpr int READY = (NB - 1) * STEP - (W - 1), NCP = TileSource<D, FITS>::template Copies<BQ>::N;
  static_assert(2 * NCP < READY, "copies are issued in front of the wait for them");
  // masked: 0 no, 1 this tile, 2 the next one too
  auto tile_stream = [&](int qt, auto masked) {
    constexpr bool MASKED = decltype(masked)::value > 0, NEXT_MASKED = decltype(masked)::value > 1;
    // the gradients of block k are formed if its last query, 32 k + 31 in this tile, is not in front of the wave's keys
    constexpr bool SKIPS = MASKED && D > 128;
    const int past = SKIPS ? __builtin_amdgcn_readfirstlane(kw0 - qt * BQ - 31) : 0;
    const int buf = (qt - qt_begin) & 1, first = kj - qt * BQ - 4 * g;
    const LdsBytes next = tile0 + (buf ^ 1) * L::BUF;
    // every wave has left the tile before, whose buffer is filled again (what a wave has read of it it has used)
    asm volatile("s_barrier" : : : "memory");
    if (!FITS) {
      q_src.template fill<BQ>(next, (qt + 1) * BQ);
      do_src.template fill<BQ>(next + L::TILE, (qt + 1) * BQ);
    }
    const auto cq = q_src.template copies<BQ>(next, (qt + 1) * BQ);
    const auto cdo = do_src.template copies<BQ>(next + L::TILE, (qt + 1) * BQ);
#pragma unroll
    for (int j = 0; j < NSLOT; ++j) {
      const int k = j / STEP, i = j % STEP, gi = i - NS;
      if (gi < 0) {
        score_mfma(k + 1, i, ring[j % W]);
      } else {
        const int c = gi / (2 * DT), dt = (gi % (2 * DT)) >> 1;
        floatx16& acc = gi & 1 ? dkacc[dt] : dvacc[dt];
        const elemx8 w = operand(gi & 1 ? dsw[k & 1] : pfw[k & 1], c);
        if (SKIPS) mfma32_agpr_from(past - 32 * k, acc, ring[j % W], w);
        else mfma32_agpr(acc, ring[j % W], w);
      }
      // The scores of block k + 1 have settled when the third MFMA behind their last one has been issued (one occupies the
      // pipe for nearly the distance asked for); nothing takes them from their registers before this statement.
      if (gi == 2) {
        if (SKIPS) mfma32_settle_vgpr(sacc[(k + 1) & 1], pacc[(k + 1) & 1]);
        else asm volatile("" : "+v"(sacc[(k + 1) & 1]), "+v"(pacc[(k + 1) & 1]));
      }
      if (j == READY) {
        store_stats(buf ^ 1, qt + 1);
        dma_wait_all();
        q_src.template clear_foreign<BQ>(next);
        do_src.template clear_foreign<BQ>(next + L::TILE);
        __syncthreads();
        fetch_stats(qt + 2);
      }
      ring[(j + W - 1) % W] = load_frag(buf, j + W - 1);        // into the fragment of the slot before
      if (FITS && j < 2 * NCP) {
        if (j < NCP) cq.one(j, q_src);
        else cdo.one(j - NCP, do_src);
      }
      // the elements of block k, second half, beside the scores of k + 1; of block k + 1, first half, beside the gradients of k
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (gi < 0 && i == e * NS / 8) softmax_elem(buf, k, 8 + e, MASKED, first);
        if (gi >= 0 && gi == 3 + e * (NG - 3) / 8) softmax_elem(buf, k + 1, e, k + 1 < NB ? MASKED : NEXT_MASKED, first);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the scores of the first block, and the first half of its exponentials
#pragma unroll
  for (int i = 0; i < W - 1; ++i) ring[i] = score_frag(0, 0, i);
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    score_mfma(0, i, ring[i % W]);
    ring[(i + W - 1) % W] = i + W - 1 < NS ? score_frag(0, 0, i + W - 1) : load_frag(0, i + W - 1 - NS);
    __builtin_amdgcn_sched_barrier(0);
  }
  load_stats(0, 0, 0);
  load_stats(0, 0, 1);
  mfma32_settle_vgpr(sacc[0], pacc[0]);
#pragma unroll
  for (int r = 0; r < 8; ++r) softmax_elem(0, 0, r, true, kj - qt_begin * BQ - 4 * g);
  __builtin_amdgcn_sched_barrier(0);
  // the tiles on the diagonal, then the others in a loop of their own (so that the accumulators keep one place in
  // the register files throughout it)
  constexpr int DIAGONAL = 128 / BQ;
  tile_stream(qt_begin, std::integral_constant<int, DIAGONAL>{});
  if (DIAGONAL > 1 && qt_begin + 1 < n_qt) tile_stream(qt_begin + 1, std::integral_constant<int, 1>{});
  for (int qt = qt_begin + DIAGONAL; qt < n_qt; ++qt) tile_stream(qt, std::integral_constant<int, 0>{});
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) mfma32_settle_agpr(dvacc[dt], dkacc[dt]);
  dma_wait_all();                 // copies of tiles beyond the last still write (zeros) to LDS
  __syncthreads();                // the tiles in LDS are done with
  constexpr int STAGED = 32 * (D + 8) * 2;
  static_assert(8 * STAGED <= sizeof(lds.tiles), "the result rows fit the tile buffers");
  elem_t* dk_rows = dqkv + ((int64_t)bi * s + kw0) * ld + h + hd * d;
  store_rows_out<D, FITS>(lds.tiles + wave * STAGED, dkacc, scale, dk_rows, ld, s - kw0, cols, lane);
  store_rows_out<D, FITS>(lds.tiles + (4 + wave) * STAGED, dvacc, 1.f, dk_rows + h, ld, s - kw0, cols, lane);
}

// dQ: wave w owns queries q0 + 32w .. +31 and walks the key tiles up to the diagonal (same traversal as the forward kernel).
// FORM_DELTA (d = D = 64 or 128): the kernel also forms delta (above) for its 128 queries, from the rows of dO and O, and
// leaves it in `delta` for the dK / dV kernel, which then has to run behind this one: no launch of its own for it.  Else
// `delta` is read and `o` ignored.  by_4: the sums in the order of the launch of its own, for sequences that take that launch
// when they do not run with others.
//
// Two workgroups share a CU.  The fragments run a few MFMAs ahead through a ring, so that a wave waits for LDS only behind the
// two barriers of a tile: one when everybody has left the tile before, whose buffer the memory pipeline then fills, one when
// that has come.  40 heads of 128 x 2048 86 -> 81 us, 16 of 128 x 8192 412 -> 372, 8 x 16 of 64 x 1024
// 39.8 -> 37.8, 8 x 24 of 188 x 512 100 -> 65.
template <int D>
struct DqLds {
  static constexpr int BKV = 64, TILE = Tile<BKV, D>::BYTES, BUF = 2 * TILE;
  // K and V tile, two of each; at the ends the staged Q, dO and dQ rows
  __align__(1024) char tiles[2 * BUF];
  float delta[128];
};
template <int D, bool FITS, bool FORM_DELTA>
__device__ __forceinline__ void attn_bwd_dq(
    DqLds<D>& lds, int id, int s, int a, int n_bh, AttnWalk walk, int d, const elem_t* __restrict__ qkv,
    const elem_t* __restrict__ o, const elem_t* __restrict__ dout, const float* __restrict__ lse, float* delta,
    elem_t* __restrict__ dqkv, int by_4) {
  using L = DqLds<D>;
  constexpr int BKV = L::BKV, DT = D / 32, KK = D / 16;
  static_assert(Tile<128, D>::BYTES == L::BUF && 128 * (D + 8) * 2 <= 2 * L::BUF, "the workgroup's 128 rows fit the tile buffers");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5;
  int rank, bi, hd;
  attn_block(id, n_bh, a, walk, rank, bi, hd);
  const int qt = (s + 127) / 128 - 1 - rank;
  const int h = a * d;
  const int64_t ld = 3 * (int64_t)h;
  const elem_t* qb = qkv + (int64_t)bi * s * ld + hd * d;
  const elem_t* dob = dout + (int64_t)bi * s * h + hd * d;
  const int q0 = qt * 128, qw0 = q0 + 32 * wave, qi = qw0 + (lane & 31);
  const float scale = rsqrtf((float)d), scale_log2 = kLog2e * scale;
  const float lse_q = (qi < s) ? lse[((int64_t)bi * a + hd) * s + qi] * kLog2e : 0.f;
  float delta_q = 0.f;
  const HeadColumns cols{d};
  const FragLanes fl(lane);
  const int kv_end = min(s, q0 + 128);         // keys behind the workgroup's last query are not fetched
  const TileSource<D, FITS> q_src(qb, ld, s, cols, tid), k_src(qb + h, ld, kv_end, cols, tid), v_src(qb + 2 * h, ld, kv_end, cols, tid),
      do_src(dob, h, s, cols, tid);
  const LdsBytes buf0(lds.tiles), buf1(lds.tiles + L::BUF);

  elemx8 qf[KK], dof[KK];
  q_src.template fill<128>(buf0, q0);
  do_src.template fill<128>(buf1, q0);
  if constexpr (FORM_DELTA) {
    // O's rows and the same ones of dO: the D / 8 lanes that hold a row's chunks add up its products
    constexpr int LPR = D / 8, RSTEP = 256 / LPR, N = 128 / RSTEP;
    const elem_t* ob = o + (int64_t)bi * s * h + hd * d;
    elemx8 ov[N], dv[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int row = min(q0 + tid / LPR + j * RSTEP, s - 1);
      const int64_t at = (int64_t)row * h + (tid % LPR) * 8;
      ov[j] = *reinterpret_cast<const elemx8*>(ob + at);
      dv[j] = *reinterpret_cast<const elemx8*>(dob + at);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float p;
      if (by_4) {
        // the launch of its own's order: 4 elements of every 64 per lane, here in pairs of such lanes; at D = 128 the lanes
        // of the upper half go on from the sums of the lower half's
        float lo = delta_add<4, true>(0.f, ov[j], dv[j], 0), hi = delta_add<4, true>(0.f, ov[j], dv[j], 4);
        if (LPR == 16) {
          const float lo0 = __shfl_xor(lo, 8, 64), hi0 = __shfl_xor(hi, 8, 64);
          lo = delta_add<4, true>(lo0, ov[j], dv[j], 0);       // of the upper half's lanes; the lower half's are not used
          hi = delta_add<4, true>(hi0, ov[j], dv[j], 4);
        }
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) { lo += __shfl_xor(lo, off, 64); hi += __shfl_xor(hi, off, 64); }
        p = lo + hi;
        if (LPR == 16) p = __shfl_xor(p, 8, 64);         // to the lane that keeps it
      } else {
        p = delta_add<8, false>(0.f, ov[j], dv[j], 0);
#pragma unroll
        for (int off = LPR / 2; off > 0; off >>= 1) p += __shfl_xor(p, off, 64);
      }
      const int row = tid / LPR + j * RSTEP;
      if (tid % LPR == 0) {
        lds.delta[row] = p;
        if (q0 + row < s) delta[((int64_t)bi * a + hd) * s + q0 + row] = p;
      }
    }
  }
  dma_wait_all();
  q_src.template clear_foreign<128>(buf0);
  do_src.template clear_foreign<128>(buf1);
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk] = frag_rows<128, D>(buf0, fl, wave, kk);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) dof[kk] = frag_rows<128, D>(buf1, fl, wave, kk);
  if constexpr (FORM_DELTA) delta_q = lds.delta[32 * wave + (lane & 31)];
  else if (qi < s) delta_q = delta[((int64_t)bi * a + hd) * s + qi];
  __syncthreads();                // the rows have been read
  k_src.template fill<BKV>(buf0, 0);
  v_src.template fill<BKV>(buf0 + L::TILE, 0);
  floatx16 dqacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) dqacc[dt][r] = 0.f;

  const int n_kt = (kv_end + BKV - 1) / BKV;
  // the wave's own: a last tile with every key in its future is left out (0 x Inf and 0 x NaN are not 0)
  const int n_own = min(n_kt, (qw0 + 31) / BKV + 1);
  // Slots of a tile: per half of 32 keys NS score MFMAs (S and dP in turn), then NG for dQ; those beyond the last are the
  // next tile's.
  constexpr int NS = 2 * KK, NG = 2 * DT, HALF = NS + NG, NSLOT = 2 * HALF, W = D == 64 ? 4 : 8;
  static_assert(NSLOT % W == 0 && NG >= W - 1, "ring position");
  auto load_frag = [&](LdsBytes tile, LdsBytes next, int j) {
    if (j >= NSLOT) { tile = next; j -= NSLOT; }
    const int ks = j / HALF, i = j % HALF;
    if (i < NS) return frag_rows<BKV, D>(i & 1 ? tile + L::TILE : tile, fl, ks, i >> 1);
    return frag_cols<BKV, D>(tile, fl, 2 * ks + (i - NS) / DT, (i - NS) % DT);
  };
  elemx8 ring[W];
  dma_wait_all();
  k_src.template clear_foreign<BKV>(buf0);
  v_src.template clear_foreign<BKV>(buf0 + L::TILE);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < W - 1; ++j) ring[j] = load_frag(buf0, buf0, j);
  for (int kt = 0; kt < n_own; ++kt) {
    const int k0 = kt * BKV;
    const LdsBytes tile = buf0 + (kt & 1) * L::BUF, next = buf0 + (~kt & 1) * L::BUF;
    // every wave has left the tile before
    asm volatile("s_barrier" : : : "memory");
    k_src.template fill<BKV>(next, k0 + BKV);
    v_src.template fill<BKV>(next + L::TILE, k0 + BKV);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      floatx16 sacc, pacc;
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[r] = pacc[r] = 0.f;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const int j = ks * HALF + i;
        if (i & 1) pacc = mfma32(ring[j % W], dof[i >> 1], pacc);
        else sacc = mfma32(ring[j % W], qf[i >> 1], sacc);
        ring[(j + W - 1) % W] = load_frag(tile, next, j + W - 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      // lane = query qi; register r = key k0 + 32ks + 8*(r/4) + 4g + r%4
      // masking in the blocks that straddle the diagonal only (a wave-uniform branch, kept as one)
      if (k0 + 32 * ks + 31 > qw0) {
        asm volatile("" ::: "memory");
        const int last = qi - k0 - 4 * g;       // the lane's last key, counted from its first one
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * ks + 8 * (r >> 2) + (r & 3) > last) sacc[r] = -INFINITY;
      }
      const float neg_lse = -lse_q;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = fast_exp2(fmaf(sacc[r], scale_log2, neg_lse));
        pacc[r] = p * (pacc[r] - delta_q);
      }
      elemx8 dsf[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) dsf[c] = pack8(pacc, 8 * c);
      if (ks == 1) {              // the next tile's first fragments are read below
        dma_wait_all();
        k_src.template clear_foreign<BKV>(next);
        v_src.template clear_foreign<BKV>(next + L::TILE);
        __syncthreads();
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        const int j = ks * HALF + NS + i;
        dqacc[i % DT] = mfma32(ring[j % W], dsf[i / DT], dqacc[i % DT]);
        ring[(j + W - 1) % W] = load_frag(tile, next, j + W - 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (n_own < n_kt) {
    asm volatile("s_barrier" : : : "memory");
    __syncthreads();
  }
  dma_wait_all();
  __syncthreads();                // the tiles in LDS are done with
  store_rows_out<D, FITS>(lds.tiles + wave * (32 * (D + 8) * 2), dqacc, scale, dqkv + ((int64_t)bi * s + qw0) * ld + hd * d, ld, s - qw0, cols, lane);
}

// ------------------------------------------------------------------- backward kernels
// At D = 64 two workgroups share a CU, with 160 ordinary and 96 accumulation registers per lane: at four more 8 x 16 heads of
// 64 x 1024 take 55 us for dK / dV instead of 44.  (A second argument to __launch_bounds__ does not keep it so: it makes the compiler
// halve the 256 between the two kinds and move accumulators about between the MFMAs, at distances that it does not know.)
template <int D, bool FITS>
__global__ __launch_bounds__(256) void attn_bwd_dkdv_kernel(
    int s, int a, int n_bh, AttnWalk walk, int d, const elem_t* __restrict__ qkv, const elem_t* __restrict__ dout,
    const float* __restrict__ lse, const float* __restrict__ delta, elem_t* __restrict__ dqkv) {
  __shared__ DkdvLds<D> lds;
  attn_bwd_dkdv<D, FITS>(lds, blockIdx.x, s, a, n_bh, walk, d, qkv, dout, lse, delta, dqkv);
}
template <int D, bool FITS, bool FORM_DELTA = false>
__global__ __launch_bounds__(256, D > 128 ? 1 : 2) void attn_bwd_dq_kernel(
    int s, int a, int n_bh, AttnWalk walk, int d, const elem_t* __restrict__ qkv, const elem_t* __restrict__ o,
    const elem_t* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ delta,
    elem_t* __restrict__ dqkv, int by_4) {
  __shared__ DqLds<D> lds;
  attn_bwd_dq<D, FITS, FORM_DELTA>(lds, blockIdx.x, s, a, n_bh, walk, d, qkv, o, dout, lse, delta, dqkv, by_4);
}
// Both at once, for problems whose tiles do not fill the chip: the first half of the workgroups forms dK and dV, the second
// dQ; delta is there already.  Each half alone is a chain of up to s / 128 (s / 64) tiles per workgroup on a part of the
// CUs; side by side they take the longer of the two times.
template <int D, bool FITS>
__global__ __launch_bounds__(256) void attn_bwd_both_kernel(
    int s, int a, int n_bh, AttnWalk walk, int d, const elem_t* __restrict__ qkv, const elem_t* __restrict__ dout,
    const float* __restrict__ lse, float* delta, elem_t* __restrict__ dqkv) {
  __shared__ union { DkdvLds<D> dkdv; DqLds<D> dq; } lds;
  const int n = gridDim.x >> 1, id = blockIdx.x;
  if (id < n) attn_bwd_dkdv<D, FITS>(lds.dkdv, id, s, a, n_bh, walk, d, qkv, dout, lse, delta, dqkv);
  else attn_bwd_dq<D, FITS, false>(lds.dq, id - n, s, a, n_bh, walk, d, qkv, nullptr, dout, lse, delta, dqkv, 0);
}

// ------------------------------------------------------------------------- launchers
// Head dimensions up to 64, 128 and 192 run in tiles of that many columns.  The copies into LDS and the stores take 32-bit byte
// offsets within 128 rows (FITS); longer rows, of 2.8 million columns and more, go through registers, a chunk after the other.
// Matrices start at any element.  16 heads of 128 x 2048 at a multiple of 16 bytes, 8 bytes behind one and 2 bytes behind one, us:
// forward 39.4, 39.6 and 52.2, dQ 54.0, 49.8 and 60.8, dK / dV 57.1, 53.7 and 65.9 (through registers 147, 158 and 120).
#define AXONN_ATTN_DISPATCH(KERNEL, ...)                                                                  \
  do {                                                                                                    \
    if (d <= 64) { if (fits) hipLaunchKernelGGL((KERNEL<64, true>), grid, dim3(256), 0, st, __VA_ARGS__);       \
                   else hipLaunchKernelGGL((KERNEL<64, false>), grid, dim3(256), 0, st, __VA_ARGS__); }           \
    else if (d <= 128) { if (fits) hipLaunchKernelGGL((KERNEL<128, true>), grid, dim3(256), 0, st, __VA_ARGS__); \
                         else hipLaunchKernelGGL((KERNEL<128, false>), grid, dim3(256), 0, st, __VA_ARGS__); }    \
    else { if (fits) hipLaunchKernelGGL((KERNEL<192, true>), grid, dim3(256), 0, st, __VA_ARGS__);              \
           else hipLaunchKernelGGL((KERNEL<192, false>), grid, dim3(256), 0, st, __VA_ARGS__); }                  \
  } while (0)
static bool offsets_fit(int64_t h) { return 128 * 3 * h * 2 < (int64_t(1) << 31); }

// dK / dV and dQ as one launch while the workgroups of both find a CU each (above 64 columns the dK / dV one leaves no room for a
// second in registers and LDS).  delta then has a launch of its own, which the dQ kernel spares at 64 and 128 columns.  Backward in
// separate launches / in one, us: 16 heads of 64 x 1024 (128 tiles) 37.2 / 26.5, of 128 x 1024 53.5 / 34.4; 16 of 188 x 512 49.2 / 27.4; 3 of
// 128 x 200, 2 sequences 22.8 / 14.0; 4 of 64 x 128, 2 sequences 12.7 / 9.0.  Beyond the line one launch is the faster one, too:
// 24 heads of 64 x 1024 (192 tiles) 37.7 / 29.2, of 128 x 1024 55.4 / 40.9, of 188 x 1024 88.3 / 57.7; 16 of 64 x 2048 (256) 64.8 / 58.8.  The line
// also says in which order delta is summed (by_4), which these shapes keep.
constexpr int kBothMaxTiles = 128;

static AttnWalk attn_walk(int n_bh, int a) {
  const bool xcds = n_bh % 8 == 0;             // and with it the number of blocks
  return {xcds ? 1u : 0u, host::recip_of(xcds ? n_bh / 8 : n_bh), host::recip_of(a)};
}
static bool head_dim_supported(int d) { return d >= 4 && d <= 192 && d % 4 == 0; }

hipError_t launch_attention_fwd(int b, int s, int a, int d, const void* qkv, void* o, float* lse,
                                hipStream_t st) {
  if (!head_dim_supported(d)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(((s + 127) / 128) * b * a));
  const bool fits = offsets_fit((int64_t)a * d);
  const AttnWalk walk = attn_walk(b * a, a);
  AXONN_ATTN_DISPATCH(attn_fwd_kernel, s, a, b * a, walk, d, (const elem_t*)qkv, (elem_t*)o, lse);
  return hipGetLastError();
}

hipError_t launch_attention_bwd(int b, int s, int a, int d, const void* qkv, const void* o,
                                const float* lse, const void* dout, void* dqkv, float* delta,
                                hipStream_t st, int rule_b) {
  if (!head_dim_supported(d)) return hipErrorInvalidValue;
  const int n_tiles = ((s + 127) / 128) * b * a;
  const bool both = n_tiles <= kBothMaxTiles;
  const bool fits = offsets_fit((int64_t)a * d);
  const AttnWalk walk = attn_walk(b * a, a);
  // for d = 64 and 128 the dQ kernel forms delta itself and runs first; sequences that run together get the sums in the order
  // that rule_b of them have
  const bool dq_forms_delta = !both && (d == 64 || d == 128);
  const int by_4 = ((s + 127) / 128) * (rule_b > 0 ? rule_b : b) * a <= kBothMaxTiles;
  hipError_t e;
  dim3 grid((unsigned)n_tiles);
  if (dq_forms_delta) {
#define AXONN_ATTN_DQ(D, FITS)                                                                                                 \
  hipLaunchKernelGGL((attn_bwd_dq_kernel<D, FITS, true>), grid, dim3(256), 0, st, s, a, b * a, walk, d, (const elem_t*)qkv,          \
                     (const elem_t*)o, (const elem_t*)dout, lse, delta, (elem_t*)dqkv, by_4)
    if (d == 64) { if (fits) AXONN_ATTN_DQ(64, true); else AXONN_ATTN_DQ(64, false); }
    else { if (fits) AXONN_ATTN_DQ(128, true); else AXONN_ATTN_DQ(128, false); }
#undef AXONN_ATTN_DQ
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    AXONN_ATTN_DISPATCH(attn_bwd_dkdv_kernel, s, a, b * a, walk, d, (const elem_t*)qkv, (const elem_t*)dout, lse, (const float*)delta, (elem_t*)dqkv);
    return hipGetLastError();
  }
  const int64_t n_pairs = (int64_t)b * s * a;
  hipLaunchKernelGGL(attn_delta_general_kernel, dim3((unsigned)((n_pairs + 15) / 16)), dim3(256), 0, st, n_pairs, s, a, d,
                     (const elem_t*)o, (const elem_t*)dout, delta);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (both) {
    grid = dim3(2u * (unsigned)n_tiles);
    AXONN_ATTN_DISPATCH(attn_bwd_both_kernel, s, a, b * a, walk, d, (const elem_t*)qkv, (const elem_t*)dout, lse, delta, (elem_t*)dqkv);
    return hipGetLastError();
  }
  AXONN_ATTN_DISPATCH(attn_bwd_dkdv_kernel, s, a, b * a, walk, d, (const elem_t*)qkv, (const elem_t*)dout, lse, (const float*)delta, (elem_t*)dqkv);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  AXONN_ATTN_DISPATCH(attn_bwd_dq_kernel, s, a, b * a, walk, d, (const elem_t*)qkv, (const elem_t*)o, (const elem_t*)dout, lse, delta, (elem_t*)dqkv, 0);
  return hipGetLastError();
}
#undef AXONN_ATTN_DISPATCH

}  // namespace axonn
