// bf16 matrix product on the matrix cores (focus_gemm):
//     C[i, n] = alpha * sum_k A[r(i), k] * B[k, n],   r(i) = a_rows ? a_rows[i] : i
// with float32 accumulation, for the projections around the attention (the
// FOCUS adapter's W_Q / W_K / W_V / W_O of eq. focus-attn, and the layer's
// Q/K/V projection).  a_rows gathers A's rows, so the summary tokens' queries
// are projected without first copying their hidden states.
//
// Three kernels: gemm_bf16_skinny for few rows (bound by reading B once),
// gemm_bf16_wide for large products, and the general one, gemm_bf16: one
// workgroup = 4 waves = a 128 x 128 tile of C; each wave owns 64 x 64 as 2 x 2
// blocks of v_mfma_f32_32x32x16_bf16.  K advances 64 at a time through four LDS
// stages, copied global -> LDS directly (global_load_lds, 16 B per lane; the A
// copy gathers rows per lane).  A is read with ds_read_b128 from 128-byte rows
// whose 16-byte chunks are XOR-swizzled by row; B (row-major [K, N]) is read
// k-major with the transposing ds_read_b64_tr_b16 from 256-byte rows whose
// 64-byte granules are XOR-swizzled, as the attention's V.  One tile per compute
// unit leaves nothing else to run there, so the reads, copies and MFMAs of a
// wave are interleaved by hand: 256 x 4096 x 4096 took 51 us with two stages and a
// full wait per step, 39 with four stages, 36 with the copies between the MFMAs,
// 30 with the LDS reads between them too, 28 with 16-byte stores of C.
#include "common.h"
#include <type_traits>

namespace {

using focus::bf16x4;
using focus::bf16x8;
using focus::copy_to_lds;
using focus::f32x16;
using focus::f32x4;
using focus::u32x4;

typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

constexpr int kBM = 128, kBN = 128, kBKk = 64;   // C tile, K step
constexpr int kThreads = 256;
constexpr int kStages = 4;                       // LDS stages (a power of two)
constexpr int kGroupM = 16;                      // A row stripes per sweep of B
constexpr int kXcdM = 8;                         // row stripes an XCD works on together
constexpr int kARow = kBKk * 2;                  // bytes per A tile row (128)
constexpr int kBRow = kBN * 2;                   // bytes per B tile row (256)
constexpr int kATile = kBM * kARow;              // 16 KB
constexpr int kBTile = kBKk * kBRow;             // 16 KB

__device__ inline int a_off(int r, int c16) { return r * kARow + ((c16 ^ (r & 7)) << 4); }
__device__ inline int b_off(int r, int byte) { return r * kBRow + (((byte >> 6) ^ (r & 3)) << 6) + (byte & 63); }

// Epilogues: col8(c) is evaluated once per eight adjacent columns a lane stores
// (the first a multiple of 8), row8 once per row of them.  kAnyOrder: results
// may depend on the order in which a kernel sums k.

// C = alpha * A B, stored as bf16 or f32.
struct PlainEpi {
  static constexpr bool kAnyOrder = true;
  void* c;
  int64_t ldc;
  int32_t c_dtype;
  float alpha;
  __device__ void one(int64_t row, int64_t col, float x) const {
    if (c_dtype == FOCUS_BF16)
      reinterpret_cast<__bf16*>(c)[row * ldc + col] = (__bf16)(x * alpha);
    else
      reinterpret_cast<float*>(c)[row * ldc + col] = x * alpha;
  }
  struct Col8 {};
  __device__ Col8 col8(int64_t) const { return {}; }
  // columns col (a multiple of 8) .. col + 7 of a row
  __device__ void row8(int64_t row, int64_t col, const float (&x)[8], const Col8&) const {
    const int64_t i = row * ldc + col;
    if (c_dtype == FOCUS_BF16) {
      __bf16* p = reinterpret_cast<__bf16*>(c) + i;
      if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
        *reinterpret_cast<uint4*>(p) = make_uint4(
            focus::pack_bf16x2(x[0] * alpha, x[1] * alpha), focus::pack_bf16x2(x[2] * alpha, x[3] * alpha),
            focus::pack_bf16x2(x[4] * alpha, x[5] * alpha), focus::pack_bf16x2(x[6] * alpha, x[7] * alpha));
        return;
      }
    } else {
      float* p = reinterpret_cast<float*>(c) + i;
      if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
        reinterpret_cast<float4*>(p)[0] = make_float4(x[0] * alpha, x[1] * alpha, x[2] * alpha, x[3] * alpha);
        reinterpret_cast<float4*>(p)[1] = make_float4(x[4] * alpha, x[5] * alpha, x[6] * alpha, x[7] * alpha);
        return;
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) one(row, col + e, x[e]);
  }
};

// The layer's Q/K/V projection: columns [Q heads | K heads | V heads]; RoPE on
// Q and K at the token's position in its augmented stream (the summary tokens
// hold real positions), interleaved pairs (2i, 2i + 1) rotated by
// pos * theta^(-2i/D).  The angle is taken in revolutions,
// pos * theta^(-2i/D) / 2 pi, whose fraction is what the hardware sine and
// cosine need: the per-pair rate is held as a 64-bit binary fraction (from its
// float64 value), so the fraction of pos * rate is the top 32 bits of a
// 32 x 64-bit integer product (two 32-bit multiplies) — exact to 2^-32 of a
// revolution for any position.  K and V rows of summary tokens also go
// straight to their cache row (the compaction pass, fused into the store).
struct QkvEpi {
  // a token's Q, K and V are the same bits whether its window is projected
  // alone or with the whole layout, so every kernel used sums k in one order
  static constexpr bool kAnyOrder = false;
  int32_t H, Hkv, D, batch;
  double log2_theta;   // <= 0: no rotation
  double rate_step;    // theta^(-2 / D): a pair's rate over the previous one's
  void* q;
  void* k;
  void* v;
  const int32_t* tok_pos;
  const uint8_t* tok_kind;
  const int32_t* tok_kmer;
  const int32_t* tok_win;
  const int32_t* win_seq;
  int64_t tok_base;
  void* cache_k;
  void* cache_v;
  int64_t cache_cap;
  int32_t* cache_len;
  int32_t* err;
  // revolutions per position of pair i of a head, and its 64-bit binary fraction
  __device__ double rate(int i) const { return exp2(-(2.0 * i / D) * log2_theta) * 0.15915494309189533577; }
  __device__ static void split(double rev, uint32_t& r_hi, uint32_t& r_lo) {
    const double hi = floor(rev * 4294967296.0);
    r_hi = (uint32_t)hi;
    r_lo = (uint32_t)((rev * 4294967296.0 - hi) * 4294967296.0);
  }
  // fraction of pos * rate, in revolutions, [0, 1]
  __device__ static float turn(uint32_t pos, uint32_t r_hi, uint32_t r_lo) {
    const uint32_t f = __umulhi(pos, r_lo) + pos * r_hi;
    return (float)f * 2.3283064365386963e-10f;  // 2^-32
  }
  // columns c .. c + 7 of a tensor row (c a multiple of 8, so one head): the
  // rates of the four pairs follow from the first by theta^(-2 / D)
  struct Col8 {
    int seg;              // 0 Q, 1 K, 2 V
    int64_t c;            // first column inside its tensor row
    bool rot;             // rotated (Q or K columns, theta given)
    uint32_t r_hi[4], r_lo[4];  // revolutions per position of each pair, as a 64-bit fraction
  };
  __device__ Col8 col8(int64_t col) const {
    const int64_t qc = (int64_t)H * D, kc = (int64_t)Hkv * D;
    Col8 r;
    r.seg = col < qc ? 0 : col < qc + kc ? 1 : 2;
    r.c = r.seg == 0 ? col : r.seg == 1 ? col - qc : col - qc - kc;
    r.rot = r.seg < 2 && log2_theta > 0.0;
    double rev = r.rot ? rate((int)(r.c % D) >> 1) : 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      split(rev, r.r_hi[i], r.r_lo[i]);
      rev *= rate_step;
    }
    return r;
  }
  __device__ void row8(int64_t row, int64_t, const float (&x)[8], const Col8& cl) const {
    const int64_t t = tok_base + row;
    const int64_t qc = (int64_t)H * D, kc = (int64_t)Hkv * D;
    float y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = x[i];
    if (cl.rot) {
      const uint32_t pos = (uint32_t)tok_pos[t];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float r = turn(pos, cl.r_hi[i], cl.r_lo[i]);
        const float sn = __builtin_amdgcn_sinf(r), cs = __builtin_amdgcn_cosf(r);
        y[2 * i] = fmaf(-x[2 * i + 1], sn, x[2 * i] * cs);
        y[2 * i + 1] = fmaf(x[2 * i], sn, x[2 * i + 1] * cs);
      }
    }
    const uint4 w = make_uint4(focus::pack_bf16x2(y[0], y[1]), focus::pack_bf16x2(y[2], y[3]),
                               focus::pack_bf16x2(y[4], y[5]), focus::pack_bf16x2(y[6], y[7]));
    put8(reinterpret_cast<__bf16*>(cl.seg == 0 ? q : cl.seg == 1 ? k : v) + row * (cl.seg == 0 ? qc : kc) + cl.c, w);
    if (cl.seg > 0 && cache_k && tok_kind[t] == FOCUS_TOK_SUMMARY) {
      const int32_t cr = tok_kmer[t];
      const int32_t b = win_seq[tok_win[t]];
      if (cr < 0 || cr >= cache_cap || b < 0 || b >= batch) {
        focus::raise_err(err, FOCUS_ERR_CAPACITY);
        return;
      }
      put8(reinterpret_cast<__bf16*>(cl.seg == 1 ? cache_k : cache_v) + ((int64_t)b * cache_cap + cr) * kc + cl.c, w);
      if (cl.seg == 1 && cl.c == 0 && cache_len) atomicMax(cache_len + b, cr + 1);
    }
  }
  // eight values to a 4-byte-aligned address, in one store where it is 16-byte aligned
  __device__ static void put8(__bf16* p, uint4 w) {
    if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
      *reinterpret_cast<uint4*>(p) = w;
    } else {
      uint32_t* d = reinterpret_cast<uint32_t*>(p);
      d[0] = w.x, d[1] = w.y, d[2] = w.z, d[3] = w.w;
    }
  }
};

// Copies and waits of both tiled kernels: K advances through four LDS stages,
// copies three steps ahead.  The copies are inline assembly (focus::copy_to_lds), so
// the compiler puts no wait of its own in front of the LDS reads; the kernel's wait
// and barrier that close each step order every read after the copies it needs.

// Stores 64 x 64 results of one wave (get(i, j) = the f32x16 of its 32 x 32
// block i, j: element v is row 8 (v / 4) + 4 g + v % 4, column l32) at C[row0 ..][col0 ..]
// through kBlockLds bytes of LDS of its own: the values are parked in rows of
// kBlockRow floats (padded so that the two half-waves write different banks),
// then eight lanes take a row, eight columns each, and store 16 bytes.
// Same-wave LDS accesses complete in order, so no barrier is needed.
constexpr int kBlockRow = 72, kBlockLds = 64 * kBlockRow * (int)sizeof(float);
template <class Epi, class Get>
__device__ __forceinline__ void store_block(float* ct, int lane, int64_t row0, int64_t col0, int64_t m, const Epi& epi,
                                            const typename Epi::Col8& cl, Get get) {
  const int l32 = lane & 31, g = lane >> 5;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x16 a = get(i, j);
#pragma unroll
      for (int v = 0; v < 16; ++v) ct[(32 * i + 8 * (v >> 2) + 4 * g + (v & 3)) * kBlockRow + 32 * j + l32] = a[v];
    }
  const int r0 = lane >> 3, c0 = 8 * (lane & 7);
#pragma unroll 4
  for (int it = 0; it < 8; ++it) {
    const int r = 8 * it + r0;
    const float4* p = reinterpret_cast<const float4*>(ct + r * kBlockRow + c0);
    const float4 lo = p[0], hi = p[1];
    const float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    if (row0 + r < m) epi.row8(row0 + r, col0 + c0, x, cl);
  }
}

// NK > 0: K = 64 NK, all of it copied at once and waited for; a unit holds two
// workgroups, so one's copies and stores overlap the other's products (with one
// to two steps the four stages would only copy the last step again).
template <class Epi, int NK = 0>
__global__ __launch_bounds__(kThreads, NK > 0 ? 2 : 1) void gemm_bf16(focus_gemm_desc d, int64_t m_tiles, Epi epi) {
  constexpr int kStage = kATile + kBTile;
  constexpr int kLds = NK == 0 ? kStages * kStage : NK * kStage > 4 * kBlockLds ? NK * kStage : 4 * kBlockLds;
  __shared__ __attribute__((aligned(1024))) char buf[kLds];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31,
            g = lane >> 5;
  // Each XCD (blocks go to them round robin) takes a contiguous run of tiles,
  // kXcdM row stripes by columns, so the workgroups running together on one
  // share A stripes and B columns through its L2.
  const int64_t n_tiles = d.n / kBN, tiles = m_tiles * n_tiles, per_xcd = (tiles + focus::kXcds - 1) / focus::kXcds;
  const int64_t lin = (blockIdx.x % focus::kXcds) * per_xcd + blockIdx.x / focus::kXcds;
  if (lin >= tiles) return;
  const int64_t per_group = (int64_t)kXcdM * n_tiles;
  const int64_t grp0 = lin / per_group, in_grp = lin % per_group;
  const int64_t gm_rows = min((int64_t)kXcdM, m_tiles - grp0 * kXcdM);
  const int64_t mt = grp0 * kXcdM + in_grp % gm_rows, nt = in_grp / gm_rows;
  const int64_t m0 = mt * kBM, n0 = nt * kBN;
  const int wm = (wave & 1) * 64, wn = (wave >> 1) * 64;   // this wave's 64 x 64 in the tile

  // Copy plan: A tile = 16 wave-loads of 1 KB (8 rows x 128 B), 4 per wave;
  // B tile = 16 wave-loads (4 rows x 256 B), 4 per wave.  Lane p of a row
  // fetches the global chunk the swizzled layout keeps at its slot.
  const char* A = reinterpret_cast<const char*>(d.a);
  const char* B = reinterpret_cast<const char*>(d.b);
  const int64_t a_ld = d.lda * 2, b_ld = d.ldb * 2;
  const char* a_src[4];
  const char* b_src[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (wave * 4 + i) * 8 + (lane >> 3), p = lane & 7;   // A tile row, 16-B slot
    const int64_t gm = min(m0 + r, d.m - 1);                         // ragged M: repeat the last row
    int64_t ar = d.a_rows ? d.a_rows[gm] : gm;
    if (ar < 0 || ar >= d.a_nrows) {
      focus::raise_err(d.err, FOCUS_ERR_BOUNDS);
      ar = 0;
    }
    a_src[i] = A + ar * a_ld + ((p ^ (r & 7)) << 4);
    const int br = (wave * 4 + i) * 4 + (lane >> 4);                 // B tile row
    const int pb = lane & 15;                                        // its 16-B slot
    b_src[i] = B + (int64_t)br * b_ld + n0 * 2 + (((pb >> 2) ^ (br & 3)) * 4 + (pb & 3)) * 16;
  }
  typedef const __attribute__((address_space(3))) char lds_char;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)&buf[0] + wave * 4 * 1024;
  // copy c (of 8: A 0 .. 3, B 4 .. 7) of this wave for the step at k0 into a stage
  auto issue = [&](int64_t k0, int stage, int c) __attribute__((always_inline)) {
    const uint32_t l = lds0 + stage * kStage;
    if (c < 4)
      copy_to_lds(a_src[c] + k0 * 2, l + c * 1024);
    else
      copy_to_lds(b_src[c - 4] + k0 * b_ld, l + kATile + (c - 4) * 1024);
  };
  constexpr int kCopies = 8;  // per wave and step

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // Operands of 16-deep k-step s: A rows wm + 32 i + l32, chunk 2 s + g; B in
  // the k order of the A operand: lane (n, g) holds B[16 s + 8 g + e][n], e = 0 .. 7.
  // Each transposing read (lane = 16 grp + 4 ri + bq) gives a lane one column of
  // the 4 rows its quad points at: rows 16 s + 8 g + ri (e < 4), then 4 further
  // down (e >= 4).
  const int grp = lane >> 4, ri = (lane >> 2) & 3, bq = lane & 3;
  struct Ops {
    bf16x8 a[2][2], b[2][2];  // two k-steps
  };
  // read pair p (of 6) of a half step: per k-step the two A operands, then B 0, B 1
  auto read_pair = [&](const char* ab, int half, int p, Ops& o) __attribute__((always_inline)) {
    const int x = p / 3, s = 2 * half + x;
    if (p % 3 == 0) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        o.a[x][i] = *reinterpret_cast<const bf16x8*>(ab + a_off(wm + 32 * i + l32, 2 * s + g));
    } else {
      const int j = p % 3 - 1, kb = 16 * s + 8 * (grp >> 1) + ri;
      const char* bb = ab + kATile;
      const int col_byte = 2 * (wn + 32 * j + 16 * (grp & 1) + 4 * bq);
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(bb + b_off(kb, col_byte)));
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(bb + b_off(kb + 4, col_byte)));
      o.b[x][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  // The 8 products of a half step from `o`, between them the reads of the next
  // half step (from the stage at ab into `n`) and then four copies of the step
  // at k_nxt (a wave that sends reads or copies at once stalls until the LDS or
  // the address unit has taken them).
  auto half_step = [&](const Ops& o, Ops& n, const char* ab, int half, int64_t k_nxt, int stage, int c0)
      __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int x = q >> 2, i = (q >> 1) & 1, j = q & 1;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.a[x][i], o.b[x][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (q < 3) {
        read_pair(ab, half, 2 * q, n);
        read_pair(ab, half, 2 * q + 1, n);
      } else if (q < 7) {
        issue(k_nxt, stage, c0 + q - 3);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  auto wait_barrier = [&](auto n) __attribute__((always_inline)) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    constexpr int kVm = decltype(n)::value;  // vmcnt(kVm) expcnt(7) lgkmcnt(0)
    __builtin_amdgcn_s_waitcnt((kVm & 15) | ((kVm >> 4) << 14) | (7 << 4) | (0 << 8));
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (NK > 0) {
#pragma unroll
    for (int t = 0; t < NK; ++t)
#pragma unroll
      for (int c = 0; c < kCopies; ++c) issue(t * kBKk, t, c);
    wait_barrier(std::integral_constant<int, 0>());
#pragma unroll
    for (int t = 0; t < 2 * NK; ++t) {
      Ops o;
#pragma unroll
      for (int p = 0; p < 6; ++p) read_pair(buf + t / 2 * kStage, t & 1, p, o);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        acc[(q >> 1) & 1][q & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.a[q >> 2][(q >> 1) & 1], o.b[q >> 2][q & 1],
                                                                          acc[(q >> 1) & 1][q & 1], 0, 0, 0);
    }
  } else {
    // Step t, whose first half's operands are in registers: multiply them while
    // the second half's are read; wait until those reads and step t + 1's copies
    // have landed (the younger ones stay in flight) and barrier; multiply the
    // second half while step t + 1's first half is read.  The copies of step t +
    // 3 (past the end, of the last step again: every step starts the same
    // number) go into the stage step t - 1 left, which every wave had read by
    // that step's barrier.  One wave per SIMD: the matrix pipe works through the
    // reads and the barrier.
    const int64_t nk = d.k / kBKk;
#pragma unroll
    for (int u = 0; u < kStages - 1; ++u)
#pragma unroll
      for (int c = 0; c < kCopies; ++c) issue(min((int64_t)u, nk - 1) * kBKk, u, c);
    wait_barrier(std::integral_constant<int, (kStages - 2) * kCopies>());
    Ops h0, h1;
#pragma unroll
    for (int p = 0; p < 6; ++p) read_pair(buf, 0, p, h0);
    int st = 0;
    for (int64_t t = 0; t < nk; ++t) {
      const int64_t k_nxt = min(t + kStages - 1, nk - 1) * kBKk;
      const int old = (st + kStages - 1) & (kStages - 1), nx = (st + 1) & (kStages - 1);
      half_step(h0, h1, buf + st * kStage, 1, k_nxt, old, 0);
      wait_barrier(std::integral_constant<int, (kStages - 3) * kCopies + kCopies / 2>());
      // (past the end: a stage that holds the last step again)
      half_step(h1, h0, buf + nx * kStage, 0, k_nxt, old, kCopies / 2);
      st = nx;
    }
  }
  // no copy into LDS outlives the block
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  __syncthreads();  // and every wave is past its reads
  const int64_t col0 = n0 + wn;
  store_block(reinterpret_cast<float*>(buf + wave * kBlockLds), lane, m0 + wm, col0, d.m, epi, epi.col8(col0 + 8 * (lane & 7)),
              [&](int i, int j) { return acc[i][j]; });
}


// Large products (N a multiple of 256): one workgroup = 4 waves = a 256 x 256
// tile of C, one wave per SIMD, each 128 x 128 as 4 x 4 blocks of
// v_mfma_f32_32x32x16_bf16 (the accumulators fill the AGPRs).  Per 16-deep
// k-step a wave reads 4 A and 4 B operands from LDS for 16 MFMAs, a third less
// per MFMA than eight waves of 128 x 64; the chip runs these products at its
// power limit, so operand bytes are what a tile's shape can save.  K advances 32
// at a time through four 32 KB LDS stages in the same pipeline as the 128 x 128
// kernel: with LDS reads and copies spread between the MFMAs and the barrier in
// the middle of a step, one wave per SIMD keeps the matrix pipe busy (reads and
// copies in bursts, as in an earlier form, made this shape 7 % slower than eight
// waves).  101 000 x 4096 x 12 288: 8.63 ms with eight waves, now 8.31; x 4096:
// 2.90, now 2.76 (torch's library product on the same device: 7.69 and 2.67).
// A rows are 64 bytes: 16-byte chunk c of row r sits at c ^ ((r / 4) mod 4), so
// the 8 rows one quarter-wave reads fall into distinct bank groups; B rows are
// 512 bytes, 64-byte granules XOR-swizzled by (row mod 4) as above.
constexpr int kBM2 = 256, kBN2 = 256, kBK2 = 32;
constexpr int kARow2 = kBK2 * 2;                 // bytes per A tile row (64)
constexpr int kBRow2 = kBN2 * 2;                 // bytes per B tile row (512)
constexpr int kATile2 = kBM2 * kARow2;           // 16 KB
constexpr int kBTile2 = kBK2 * kBRow2;           // 16 KB
constexpr int kStage2 = kATile2 + kBTile2;       // A then B

// Block -> tile.  kGroupM row stripes of A sweep the column tiles before the
// next group starts, so A is read from HBM about once and B (the weights) stays
// in the last-level cache.  With sbw (columns of a super block, even) the group
// is cut into super blocks of up to 16 x sbw tiles, one round of workgroups;
// XCD x (blocks go to them round robin) takes a 4 x sbw / 2 part of each, so the
// tiles it works on together share A stripes and B columns through its L2 while
// all XCDs share the super block's in the last-level cache (101 000 x 4096 x
// 4096: 2.83 -> 2.76 ms).  A last group whose row stripes do not divide by four
// goes without: the parts would be uneven and some XCDs without work.
__device__ inline void wide_tile(int64_t bid, int64_t m_tiles, int64_t n_tiles, int sbw, int64_t& mt, int64_t& nt) {
  const int64_t per_group = (int64_t)kGroupM * n_tiles, grp0 = bid / per_group, in_grp = bid % per_group;
  const int rows = (int)min((int64_t)kGroupM, m_tiles - grp0 * kGroupM);
  if (sbw > 0 && rows % 4 == 0) {
    const int per = rows / 4, sb = 4 * per * sbw;  // tiles of a super block
    const int r = (int)(in_grp % sb), x = r % focus::kXcds, i = r / focus::kXcds;
    const int mi = (x % 4) * per + i % per;
    mt = grp0 * kGroupM + mi;
    nt = in_grp / sb * sbw + (x / 4) * (sbw / 2) + i / per;
  } else {
    mt = grp0 * kGroupM + in_grp % rows;
    nt = in_grp / rows;
  }
}

template <class Epi>
__global__ __launch_bounds__(kThreads, 1) void gemm_bf16_wide(focus_gemm_desc d, int64_t m_tiles, int sbw, Epi epi) {
  __shared__ __attribute__((aligned(1024))) char buf[kStages][kStage2];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31,
            g = lane >> 5;
  int64_t mt, nt;
  wide_tile(blockIdx.x, m_tiles, d.n / kBN2, sbw, mt, nt);
  const int64_t m0 = mt * kBM2, n0 = nt * kBN2;
  const int wm = (wave & 1) * 128, wn = (wave >> 1) * 128;  // this wave's 128 x 128 in the tile

  // Copy plan: A tile = 16 wave-loads of 1 KB (16 rows x 64 B), 4 per wave;
  // B tile = 16 wave-loads (2 rows x 512 B), 4 per wave.  Lane p of a row
  // fetches the global chunk the swizzled layout keeps at its slot.
  const char* A = reinterpret_cast<const char*>(d.a);
  const char* B = reinterpret_cast<const char*>(d.b);
  const int64_t a_ld = d.lda * 2, b_ld = d.ldb * 2;
  const char* a_src[4];
  const char* b_src[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (wave * 4 + i) * 16 + (lane >> 2), p = lane & 3;  // A tile row, 16-B slot
    const int64_t gm = min(m0 + r, d.m - 1);                         // ragged M: repeat the last row
    int64_t ar = d.a_rows ? d.a_rows[gm] : gm;
    if (ar < 0 || ar >= d.a_nrows) {
      focus::raise_err(d.err, FOCUS_ERR_BOUNDS);
      ar = 0;
    }
    a_src[i] = A + ar * a_ld + ((p ^ ((r >> 2) & 3)) << 4);
    const int br = (wave * 4 + i) * 2 + (lane >> 5), pb = lane & 31;  // B tile row, its 16-B slot
    b_src[i] = B + (int64_t)br * b_ld + n0 * 2 + (((pb >> 2) ^ (br & 3)) * 4 + (pb & 3)) * 16;
  }
  typedef const __attribute__((address_space(3))) char lds_char;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)&buf[0][0] + wave * 4 * 1024;
  auto issue = [&](int64_t k0, int stage, int c) __attribute__((always_inline)) {
    const uint32_t l = lds0 + stage * kStage2;
    if (c < 4)
      copy_to_lds(a_src[c] + k0 * 2, l + c * 1024);
    else
      copy_to_lds(b_src[c - 4] + k0 * b_ld, l + kATile2 + (c - 4) * 1024);
  };
  constexpr int kCopies = 8;  // per wave and step

  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int grp = lane >> 4, ri = (lane >> 2) & 3, bq = lane & 3;
  struct Ops {
    bf16x8 a[4], b[4];  // one k-step
  };
  // read pair p (of 6) of k-step s: A 0 1, A 2 3, B 0 .. B 3
  auto read_pair = [&](const char* ab, int s, int p, Ops& o) __attribute__((always_inline)) {
    if (p < 2) {
      const int off = (wm + l32) * kARow2 + (((2 * s + g) ^ ((l32 >> 2) & 3)) << 4);
#pragma unroll
      for (int i = 2 * p; i < 2 * p + 2; ++i) o.a[i] = *reinterpret_cast<const bf16x8*>(ab + (off + 32 * i * kARow2));
    } else {
      const int j = p - 2;
      const char* bb = ab + kATile2 + (8 * (grp >> 1) + ri) * kBRow2 + ((((wn >> 5) + j) ^ ri) << 6) + 32 * (grp & 1) + 8 * bq;
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(bb + 16 * s * kBRow2));
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(bb + (16 * s + 4) * kBRow2));
      o.b[j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  auto half_step = [&](const Ops& o, Ops& n, const char* ab, int half, int64_t k_nxt, int stage, int c0)
      __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = q >> 2, j = q & 3;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.a[i], o.b[j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (q < 6)
        read_pair(ab, half, q, n);
      else if (q & 1)
        if (q < 14) issue(k_nxt, stage, c0 + (q - 7) / 2);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  const int64_t nk = d.k / kBK2;
  auto wait_barrier = [&](auto n) __attribute__((always_inline)) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    constexpr int kVm = decltype(n)::value;  // vmcnt(kVm) expcnt(7) lgkmcnt(0)
    __builtin_amdgcn_s_waitcnt((kVm & 15) | ((kVm >> 4) << 14) | (7 << 4) | (0 << 8));
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int u = 0; u < kStages - 1; ++u)
#pragma unroll
    for (int c = 0; c < kCopies; ++c) issue(min((int64_t)u, nk - 1) * kBK2, u, c);
  wait_barrier(std::integral_constant<int, (kStages - 2) * kCopies>());
  Ops h0, h1;
#pragma unroll
  for (int p = 0; p < 6; ++p) read_pair(buf[0], 0, p, h0);
  int st = 0;
  for (int64_t t = 0; t < nk; ++t) {
    const int64_t k_nxt = min(t + kStages - 1, nk - 1) * kBK2;
    const int old = (st + kStages - 1) & (kStages - 1), nx = (st + 1) & (kStages - 1);
    half_step(h0, h1, buf[st], 1, k_nxt, old, 0);
    wait_barrier(std::integral_constant<int, (kStages - 3) * kCopies + kCopies / 2>());
    half_step(h1, h0, buf[nx], 0, k_nxt, old, kCopies / 2);
    st = nx;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
#pragma unroll
  for (int jj = 0; jj < 2; ++jj) {
    const int64_t col0 = n0 + wn + 64 * jj;
    const typename Epi::Col8 cl = epi.col8(col0 + 8 * (lane & 7));
#pragma unroll
    for (int h = 0; h < 2; ++h)
      store_block(reinterpret_cast<float*>(buf[wave]), lane, m0 + wm + 64 * h, col0, d.m, epi, cl,
                  [&](int i, int j) { return acc[2 * h + i][2 * jj + j]; });
  }
}

// Few rows (a decode step's tokens, the summaries of a few windows): reading B
// once bounds the product, so B goes from memory straight to registers.  One
// workgroup = WAVES waves = 16 MB rows x 64 columns of C; the waves take the
// 32-deep k-steps in turn and add their sums through LDS.  A lane reads 8 rows
// of B, 4 adjacent columns (8 bytes) each: lanes 0-15 of a wave cover 128
// contiguous bytes of a row, lane group g = lane / 16 the rows 8 g .. 8 g + 7,
// which are the k indices its lanes feed to v_mfma_f32_16x16x32_bf16.  The 8 x 4
// block is transposed inside the lane (16 v_perm_b32), so column j of the block
// is the B operand of product j, whose 16 columns are 4 (lane mod 16) + j.  The
// next k-step's loads are in flight while one is computed.
constexpr int kSkN = 64, kSkK = 32;

template <int MB, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void gemm_bf16_skinny(focus_gemm_desc d, PlainEpi epi) {
  __shared__ float part[WAVES][16][kSkN];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c = lane & 15, g = lane >> 4;
  const int64_t n0 = (int64_t)blockIdx.x * kSkN, m0 = (int64_t)blockIdx.y * 16 * MB;
  const char* a_src[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const int64_t gm = min(m0 + 16 * i + c, d.m - 1);  // ragged M: repeat the last row
    int64_t ar = d.a_rows ? d.a_rows[gm] : gm;
    if (ar < 0 || ar >= d.a_nrows) {
      focus::raise_err(d.err, FOCUS_ERR_BOUNDS);
      ar = 0;
    }
    a_src[i] = reinterpret_cast<const char*>(d.a) + ar * d.lda * 2 + 16 * g;
  }
  const char* b_src = reinterpret_cast<const char*>(d.b) + 8 * g * d.ldb * 2 + (n0 + 4 * c) * 2;

  struct Step {
    uint2 b[8];
    bf16x8 a[MB];
  };
  auto load = [&](int64_t t, Step& s) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; ++i) s.b[i] = *reinterpret_cast<const uint2*>(b_src + (t * kSkK + i) * d.ldb * 2);
#pragma unroll
    for (int i = 0; i < MB; ++i) s.a[i] = *reinterpret_cast<const bf16x8*>(a_src[i] + t * kSkK * 2);
  };
  f32x4 acc[MB][4];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const Step& s) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t lo = j < 2 ? s.b[2 * e].x : s.b[2 * e].y, hi = j < 2 ? s.b[2 * e + 1].x : s.b[2 * e + 1].y;
        w[e] = __builtin_amdgcn_perm(hi, lo, (j & 1) ? 0x07060302u : 0x05040100u);
      }
      const bf16x8 bop = __builtin_bit_cast(bf16x8, w);
#pragma unroll
      for (int i = 0; i < MB; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(s.a[i], bop, acc[i][j], 0, 0, 0);
    }
  };
  const int64_t nk = d.k / kSkK;
  int64_t t = wave;
  if (t < nk) {
    Step s0, s1;
    load(t, s0);
    for (; t < nk; t += 2 * WAVES) {
      if (t + WAVES < nk) load(t + WAVES, s1);
      compute(s0);
      if (t + WAVES >= nk) break;
      if (t + 2 * WAVES < nk) load(t + 2 * WAVES, s0);
      compute(s1);
    }
  }
  // acc[i][j][r] = C[m0 + 16 i + 4 g + r][n0 + 4 c + j]; thread (wave, lane)
  // adds rows wave, wave + WAVES, ... of column lane over the waves
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    if (i > 0) __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<float4*>(&part[wave][4 * g + r][4 * c]) =
          make_float4(acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]);
    __syncthreads();
#pragma unroll
    for (int r0 = 0; r0 < 16; r0 += WAVES) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) x += part[w][r0 + wave][lane];
      const int64_t row = m0 + 16 * i + r0 + wave;
      if (row < d.m) epi.one(row, n0 + lane, x);
    }
  }
}

// Columns of a super block of the wide kernel's order: an even divisor of
// n_tiles from 8 to 16, as wide as there is; 0 (plain groups) if there is none.
int super_block(int64_t n_tiles) {
  for (int w = 16; w >= 8; w -= 2)
    if (n_tiles % w == 0) return w;
  return 0;
}

// Launch C = A B (+ epilogue).  The kernel is chosen by the rounds of
// workgroups (one per compute unit) each would take; times at K = 4096 on 256
// compute units (of 712 sizes from K = 64 to 8192, M = 1 to 5000 and N = 128 to
// 32 768 none takes over 2 % longer than with the two kernels before these):
// * few rows: one round of 64 x 64 skinny tiles (M = 256, N = 4096: 26 us, the
//   128 x 128 kernel 28; M = 128, N = 12 288, two rounds: 50 against 29), and any
//   N while one row tile of up to 32 rows holds M, where a second round still
//   only reads B (M = 16, N = 12 288: 17.5 us against 28);
// * K = 64 or 128: the 128 x 128 kernel that copies all of K at once, two
//   workgroups a unit (M = 4096, N = 6144: 17.7 us against 27.1 with the larger
//   tile at K = 64, 20.4 against 29.6 at 128; M = 1000, N = 4096: 6.6 against 7.4
//   and 7.2 against 7.8 with the four stages);
// * a full round of 256 x 256 tiles takes as long as 2.75 rounds of 128 x 128
//   (78 us against 28), so those are used unless the larger tile saves more
//   rounds than that (M = 1000: N = 4096 37 us against 79, N = 12 288 108
//   against 100; M = 4096, N = 4096: 143 against 113).
template <class Epi>
focus_status launch_gemm(const focus_gemm_desc& d, const Epi& epi, focus_stream_t stream) {
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int64_t cus = focus::device_cus();
  if constexpr (Epi::kAnyOrder) {
    const int64_t sk_n = d.n / kSkN, sk_m = focus::ceil_div(d.m, 64);
    if ((d.m <= 32 || sk_n * sk_m <= cus) && sk_n <= INT32_MAX / 1024) {
      const uint32_t bx = (uint32_t)sk_n, by = (uint32_t)sk_m;
      if (d.m <= 16)
        hipLaunchKernelGGL((gemm_bf16_skinny<1, 16>), dim3(bx), dim3(1024), 0, s, d, epi);
      else if (d.m <= 32)
        hipLaunchKernelGGL((gemm_bf16_skinny<2, 8>), dim3(bx), dim3(512), 0, s, d, epi);
      else
        hipLaunchKernelGGL((gemm_bf16_skinny<4, 8>), dim3(bx, by), dim3(512), 0, s, d, epi);
      return focus::launch_status();
    }
  }
  const int64_t m_tiles = focus::ceil_div(d.m, kBM), n_tiles = d.n / kBN;
  const int64_t m_tiles2 = focus::ceil_div(d.m, kBM2), n_tiles2 = d.n / kBN2;
  const int64_t rounds = focus::ceil_div(m_tiles * n_tiles, cus), rounds2 = focus::ceil_div(m_tiles2 * n_tiles2, cus);
  if (d.n % kBN2 == 0 && d.k > 2 * kBKk && 11 * rounds2 <= 4 * rounds) {
    const int sbw = super_block(n_tiles2);
    const int64_t blocks = m_tiles2 * n_tiles2;
    if (blocks > INT32_MAX) return FOCUS_E_SHAPE;
    hipLaunchKernelGGL(gemm_bf16_wide<Epi>, dim3((uint32_t)blocks), dim3(kThreads), 0, s, d, m_tiles2, sbw, epi);
  } else {
    const int64_t blocks = focus::ceil_div(m_tiles * n_tiles, focus::kXcds) * focus::kXcds;
    if (blocks > INT32_MAX) return FOCUS_E_SHAPE;
    const dim3 grid((uint32_t)blocks), block(kThreads);
    if (d.k == kBKk)
      hipLaunchKernelGGL((gemm_bf16<Epi, 1>), grid, block, 0, s, d, m_tiles, epi);
    else if (d.k == 2 * kBKk)
      hipLaunchKernelGGL((gemm_bf16<Epi, 2>), grid, block, 0, s, d, m_tiles, epi);
    else
      hipLaunchKernelGGL(gemm_bf16<Epi>, grid, block, 0, s, d, m_tiles, epi);
  }
  return focus::launch_status();
}
}  // namespace

extern "C" focus_status focus_gemm(const focus_gemm_desc* d, focus_stream_t stream) {
  if (!d) return FOCUS_E_NULL;
  if (d->c_dtype != FOCUS_BF16 && d->c_dtype != FOCUS_F32) return FOCUS_E_DTYPE;
  if (d->m < 0 || d->n < 0 || d->k < 0 || !(d->alpha == d->alpha)) return FOCUS_E_ARG;
  if (d->m == 0 || d->n == 0) return FOCUS_OK;
  if (d->k == 0 || d->k % kBKk || d->n % kBN) return FOCUS_E_UNSUPPORTED;
  if (!d->a || !d->b || !d->c) return FOCUS_E_NULL;
  if (d->lda < d->k || d->ldb < d->n || d->ldc < d->n || d->lda % 8 || d->ldb % 8) return FOCUS_E_ARG;
  if (d->a_nrows < (d->a_rows ? 1 : d->m)) return FOCUS_E_ARG;
  if (!focus::aligned16(d->a) || !focus::aligned16(d->b) || (reinterpret_cast<uintptr_t>(d->c) & 3u) ||
      (reinterpret_cast<uintptr_t>(d->a_rows) & 7u))
    return FOCUS_E_ARG;
  const PlainEpi epi = {d->c, d->ldc, d->c_dtype, d->alpha};
  return launch_gemm(*d, epi, stream);
}

extern "C" focus_status focus_qkv_project(const focus_qkv_desc* q, focus_stream_t stream) {
  if (!q) return FOCUS_E_NULL;
  if (q->dtype != FOCUS_BF16) return q->dtype == FOCUS_F32 ? FOCUS_E_UNSUPPORTED : FOCUS_E_DTYPE;
  if (q->n_heads <= 0 || q->n_kv_heads <= 0 || q->d_model <= 0 || q->batch < 0 || q->n_rows < 0 ||
      q->tok_base < 0 || !(q->rope_theta == q->rope_theta) || (q->rope_theta > 0.f && q->rope_theta <= 1.f))
    return FOCUS_E_ARG;
  if (q->head_dim != 64 && q->head_dim != 128) return FOCUS_E_UNSUPPORTED;
  if (q->n_heads % q->n_kv_heads) return FOCUS_E_SHAPE;
  const int64_t n = ((int64_t)q->n_heads + 2 * q->n_kv_heads) * q->head_dim;
  if (n % kBN || q->d_model % kBKk) return FOCUS_E_UNSUPPORTED;
  if (q->tok_base + q->n_rows > q->totals.n_tokens) return FOCUS_E_SHAPE;
  if (q->n_rows == 0) return FOCUS_OK;
  if (!q->hidden || !q->w_qkv || !q->q || !q->k || !q->v || !q->tok_pos) return FOCUS_E_NULL;
  if (q->cache_k && (!q->cache_v || !q->tok_kind || !q->tok_kmer || !q->tok_win || !q->win_seq))
    return FOCUS_E_NULL;
  if (q->cache_k && q->cache_cap < q->totals.max_cache_per_seq && q->tok_base == 0 && q->n_rows == q->totals.n_tokens)
    return FOCUS_E_CAPACITY;
  if (!focus::aligned16(q->hidden) || !focus::aligned16(q->w_qkv)) return FOCUS_E_ARG;
  // pairs of bf16 columns are stored as one 4-byte word
  if ((reinterpret_cast<uintptr_t>(q->q) | reinterpret_cast<uintptr_t>(q->k) | reinterpret_cast<uintptr_t>(q->v) |
       reinterpret_cast<uintptr_t>(q->cache_k) | reinterpret_cast<uintptr_t>(q->cache_v)) & 3u)
    return FOCUS_E_ARG;
  focus_gemm_desc g = {};
  g.m = q->n_rows;
  g.n = n;
  g.k = q->d_model;
  g.a = q->hidden;
  g.lda = q->d_model;
  g.a_nrows = q->n_rows;
  g.b = q->w_qkv;
  g.ldb = n;
  g.err = q->err;
  QkvEpi e;
  e.H = q->n_heads;
  e.Hkv = q->n_kv_heads;
  e.D = q->head_dim;
  e.batch = q->batch;
  e.log2_theta = q->rope_theta > 0.f ? log2((double)q->rope_theta) : 0.0;
  e.rate_step = exp2(-(2.0 / e.D) * e.log2_theta);
  e.q = q->q;
  e.k = q->k;
  e.v = q->v;
  e.tok_pos = q->tok_pos;
  e.tok_kind = q->tok_kind;
  e.tok_kmer = q->tok_kmer;
  e.tok_win = q->tok_win;
  e.win_seq = q->win_seq;
  e.tok_base = q->tok_base;
  e.cache_k = q->cache_k;
  e.cache_v = q->cache_v;
  e.cache_cap = q->cache_cap;
  e.cache_len = q->cache_len;
  e.err = q->err;
  return launch_gemm(g, e, stream);
}
