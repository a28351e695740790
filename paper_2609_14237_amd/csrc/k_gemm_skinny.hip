// bf16 MFMA GEMM for the smallest decode batches (M <= 32 rows; dense, either
// weight layout): C[m, n] = sum_k A[m, k] * B[n, k] with the same epilogues as
// the other GEMM kernels.
//
// Bound by the weight stream. At these batches the tiled kernels lose to their
// own fixed parts: 64 activation rows staged whatever M is, split-K partials
// written and summed by a second launch, and few K steps per block. Here a
// block owns 16 to 64 output columns for the whole of K, its waves take every
// W-th 64-wide K step each and meet once, in LDS, at the end: no partials, no
// reduce launch, and no barrier in the loop. Each wave streams its steps (its
// rows of B, and only the 8-row groups of A that exist) through an LDS ring of
// its own with direct-to-LDS loads, eight lanes per 128-byte row segment, so
// every request is a whole cache line; loading the fragments straight into
// registers asks for 64-byte halves and stops at 5.1 TB/s. The ring XOR-swizzles
// chunks by row as the streaming kernel does, so fragment reads are free of
// bank conflicts.
//
// Measured on the 8B-shaped layer, back to back with weights rotated (before:
// 64-row tiles with split-K and their reduce launch -> now): 13 rows, tiled
// weights: qkv with RoPE 16.3 -> 14.2 us, o_proj 13.1 -> 7.9, down 24.9 -> 21.2
// (5.6 TB/s); row-major: qkv with RoPE 16.6 -> 14.1, o_proj 14.2 -> 7.7, gate_up
// + SiLU 47.7 -> 36.7 (6.4 TB/s), down 26.9 -> 21.6. One GPU's share under 8-way
// tensor parallelism, 13 rows: the step 85.9 -> 68.3 us.
//
// Two neighbours join it where they are next to it in a call's range, since at
// these batches a launch (2 us and more back to back) costs what they do:
//  - NORM: the RMSNorm before qkv or gate_up (not the router: its logits stay
//    products of the very rows the experts read). A holds the residual;
//    each wave multiplies its fragments by the gain (kept in LDS), adds up the
//    squares on the way, and the output rows are scaled by 1 / rms in the
//    epilogue, where the waves meet anyway. The conversions cost 72 VALU
//    instructions per K step and wave for 16 rows, a fifth of the issue slots
//    the weight stream leaves. The normalised rows themselves, which later
//    operators or a caller may read, are written in slices by all blocks.
//  - EPI_ROPE: RoPE and the KV append after qkv. A block takes 16 columns of the
//    first half of a head and the 16 that pair with them in the second, rotates
//    them in the epilogue and stores k and v into their page slots; angles are
//    computed while the last K steps are in flight.
// Measured: attn_norm .. kv_append 16.7 -> 12.8 us at 13 rows of the 8B-shaped
// layer; whole steps: tiny layer (4 rows) 39.7 -> 28.3 us, 8B-shaped layer at 1
// row 108.7 -> 103.9 us and at 13 rows 119.0 -> 112.4 us.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace ods {

namespace {

constexpr int kNonTemporal = 2;  // cache-policy operand of the direct-to-LDS load: nt

constexpr int EPI_ROPE = 4;  // bf16 qkv, rotated, k and v also to the KV pool (columns in pairs of half heads)

// Neighbouring operators a launch takes in.
struct SkinnyFuse {
  const uint16_t *gain;  // NORM: A is the residual, gain its RMSNorm's, xn the normalised rows to write
  uint16_t *xn;
  float eps;
  RopeArgs rope;  // EPI_ROPE
};

// Bytes of LDS: the waves' rings, which the partial tiles and the rows' sums of
// squares reuse at the end; then the contexts (EPI_ROPE) and the gain (NORM).
template <int W, int RW, int AG, int NS, int EPI>
constexpr size_t skinny_lds() {
  constexpr int FR = EPI == EPI_SILU ? 2 * RW : RW, MT = (AG + 1) / 2;
  constexpr size_t ring = (size_t)W * NS * (2 * FR + AG) * 1024;
  constexpr size_t red = (size_t)W * 16 * MT * (16 * FR + 2) * 4;
  return (ring > red ? ring : red);
}
constexpr size_t kGainLds = (size_t)kSkinnyNormMaxK * 2;
constexpr size_t kCtxLds = 256;

// W waves per block; RW 16-column output fragments per block (SiLU: RW gate and
// RW up fragments of B rows); AG 8-row groups of A (1, 2 or 4: M <= 8, 16, 32);
// NS K steps in each wave's ring.
template <int W, int RW, int AG, int NS, int EPI, bool TILED, bool NORM>
__global__ __launch_bounds__(64 * W) void gemm_skinny_kernel(GemmArgs p, SkinnyFuse fu) {
  constexpr bool ROPE = EPI == EPI_ROPE;
  static_assert(!ROPE || RW == 2, "a RoPE block holds one fragment of each half of a head");
  constexpr bool SILU = EPI == EPI_SILU;
  constexpr int FR = SILU ? 2 * RW : RW;  // 16-row B fragments per wave (SiLU: RW gate, then RW up)
  constexpr int MT = (AG + 1) / 2;        // 16-row A fragments
  constexpr int L = 2 * FR + AG;          // loads per K step and wave
  constexpr int SLOT = L * 1024;
  constexpr int COLS = 16 * RW;           // output columns per block
  constexpr int ROWS = 16 * MT;
  constexpr int PITCH = 16 * FR + 1;      // floats per row of a wave's partial tile
  constexpr int OUT = ROPE ? ROWS * 16 : ROWS * COLS, PER = (OUT + 64 * W - 1) / (64 * W);
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, q = lane >> 4;
  // First output column; a RoPE block's second fragment is half a head further.
  int half = 0, n0 = blockIdx.x * COLS;
  if constexpr (ROPE) {
    half = fu.rope.D / 2;
    n0 = (int)(blockIdx.x * 16) / half * 2 * half + (int)(blockIdx.x * 16) % half;
  }
  const int steps = (p.K + 63) / 64;
  const int cnt = (steps - wave + W - 1) / W;  // K steps wave, wave + W, ...
  uint8_t *const ring = smem + wave * NS * SLOT;
  // Blocks of different weight tiles start at different K steps: rows and tiles
  // lie a power of two apart, and in step they would ask the same HBM channels
  // (13 rows, row-major, K 8192: o_proj 28.1 -> 22.3 us, gate_up + SiLU 171 ->
  // 147; K 4096 42.5 -> 35.8). Tiles that do not lie so stay in step (K 7168, 8
  // rows: o_proj 17.9 -> 16.8 us, norm + gate_up + SiLU 110 -> 104).
  const int rot = TILED && p.K % 2048 != 0 ? 0 : (n0 >> (SILU ? 6 : 7)) % steps;
  auto step_of = [&](int i) {  // K step of this wave's turn i < cnt
    const int s = wave + i * W + rot;
    return s >= steps ? s - steps : s;
  };

  // The residual this thread will add: loaded first, so nothing waits for it at the end.
  float old[PER];
  if (EPI == EPI_RESID) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int o = tid + i * 64 * W, m = o / COLS, n = n0 + o % COLS;
      old[i] = (o < OUT && m < p.M && n < p.N) ? bf2f(((const uint16_t *)p.C)[(int64_t)m * p.ldc + n]) : 0.f;
    }
  }

  const int chunk = (lane & 7) ^ (lane >> 3);
  const uint16_t *bp[2 * FR];
#pragma unroll
  for (int f = 0; f < 2 * FR; ++f) {
    const bool up = SILU && f >= 2 * RW;
    const int n = n0 + (ROPE ? (f >> 1) * half + (f & 1) * 8 : (f % (2 * RW)) * 8) + (lane >> 3);
    if (TILED) {
      int tile, r;
      if (SILU) {
        tile = n >> 6;
        r = (n & 63) + (up ? 64 : 0);
      } else if (p.n_up > 0) {
        const bool u = n >= p.n_up;
        const int c = min(u ? n - p.n_up : n, p.n_up - 1);
        tile = c >> 6;
        r = (c & 63) + (u ? 64 : 0);
      } else {
        tile = n >> 7;
        r = n & 127;
      }
      if (n >= p.N) tile = r = 0;
      bp[f] = p.B + ((int64_t)tile * steps * 128 + r) * 64 + (lane & 7) * 8;
    } else {
      const int nc = min(n, p.N - 1);
      bp[f] = p.B + (int64_t)(up ? p.n_up + nc : nc) * p.ldb;
    }
  }
  const uint16_t *ap[AG];
#pragma unroll
  for (int t = 0; t < AG; ++t) ap[t] = p.A + (int64_t)min(t * 8 + (lane >> 3), p.M - 1) * p.lda;

  auto issue = [&](int slot, int i) {
    const int s = step_of(i);
    const int k = min(s * 64 + chunk * 8, p.K - 8);
    uint8_t *const dst = ring + slot * SLOT;
#pragma unroll
    for (int f = 0; f < 2 * FR; ++f) {
      const uint16_t *src = TILED ? bp[f] + (int64_t)s * (128 * 64) : bp[f] + k;
      __builtin_amdgcn_global_load_lds((const void *)src, (__attribute__((address_space(3))) void *)(dst + f * 1024), 16,
                                       0, kNonTemporal);
    }
#pragma unroll
    for (int t = 0; t < AG; ++t)
      __builtin_amdgcn_global_load_lds((const void *)(ap[t] + k),
                                       (__attribute__((address_space(3))) void *)(dst + (2 * FR + t) * 1024), 16, 0, 0);
  };
  const int rd0 = j * 128 + ((q ^ (j & 7)) << 4), rd1 = j * 128 + (((4 + q) ^ (j & 7)) << 4);
  f32x4 acc[MT][FR];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int f = 0; f < FR; ++f) acc[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 a[MT][2], b[FR][2];
  auto read = [&](int slot, int i) {
    const uint8_t *src = ring + slot * SLOT;
    // with AG = 1 the upper half of the A fragment lies outside the slot: those rows re-read the lower half
    const int a0 = AG == 1 ? (rd0 & ~1024) : rd0, a1 = AG == 1 ? (rd1 & ~1024) : rd1;
#pragma unroll
    for (int f = 0; f < FR; ++f) {
      b[f][0] = *(const u32x4 *)(src + f * 2048 + rd0);
      b[f][1] = *(const u32x4 *)(src + f * 2048 + rd1);
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      a[t][0] = *(const u32x4 *)(src + (2 * FR + 2 * t) * 1024 + a0);
      a[t][1] = *(const u32x4 *)(src + (2 * FR + 2 * t) * 1024 + a1);
    }
    const int s = step_of(i);
    if (!TILED && (s + 1) * 64 > p.K) {  // the last, short K step: chunks past K hold copies
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        if (s * 64 + (ks * 4 + q) * 8 >= p.K) {
#pragma unroll
          for (int f = 0; f < FR; ++f) b[f][ks] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int t = 0; t < MT; ++t) a[t][ks] = u32x4{0u, 0u, 0u, 0u};
        }
    }
  };
  const int *const ctx_lds = (const int *)(smem + skinny_lds<W, RW, AG, NS, EPI>());
  uint8_t *const gain_lds = (uint8_t *)ctx_lds + (ROPE ? kCtxLds : 0);
  float ss[MT];  // NORM: this lane's share of each row's sum of squares
#pragma unroll
  for (int t = 0; t < MT; ++t) ss[t] = 0.f;
  auto mma = [&](int i) {
    if (NORM) {
      const int s = step_of(i);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const u32x4 g = *(const u32x4 *)(gain_lds + (s * 64 + (ks * 4 + q) * 8) * 2);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          ss[t] += sumsq8(a[t][ks]);
          a[t][ks] = norm8(a[t][ks], g, 1.f);
        }
      }
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < FR; ++f)
          acc[t][f] = mfma_16x16x32(__builtin_bit_cast(bf16x8, a[t][ks]), __builtin_bit_cast(bf16x8, b[f][ks]),
                                    acc[t][f]);
  };
  if (NORM)  // the gain, 512 values a load (past K: copies of the last, against zeroed rows)
    for (int g = wave; g * 512 < p.K; g += W)
      __builtin_amdgcn_global_load_lds((const void *)(fu.gain + min(g * 512 + lane * 8, p.K - 8)),
                                       (__attribute__((address_space(3))) void *)(gain_lds + g * 1024), 16, 0, 0);
  if (ROPE && wave == 0)
    __builtin_amdgcn_global_load_lds((const void *)(fu.rope.ctx_lens + min(lane, p.M - 1)),
                                     (__attribute__((address_space(3))) void *)ctx_lds, 4, 0, 0);
#pragma unroll
  for (int u = 0; u < NS; ++u)
    if (u < cnt) issue(u, u);
  if (NORM || ROPE) {  // loads complete in order: with only ring loads outstanding the gain and contexts are there
    if (cnt >= NS) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NS * L) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
  }
  int i = 0, slot = 0;
  for (; i + NS < cnt; ++i) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * L) : "memory");
    read(slot, i);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot is in registers before it is refilled
    __builtin_amdgcn_sched_barrier(0);
    issue(slot, i + NS);
    mma(i);
    slot = slot == NS - 1 ? 0 : slot + 1;
  }
  // While the last K steps are in flight: the positions, page slots and angles of
  // this thread's pairs (EPI_ROPE), and its slice of the rows to normalise (NORM).
  int pos[PER], page[PER];
  float cs[PER], sn[PER];
  if (ROPE) {
    const RopeArgs &r = fu.rope;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int o = tid + i * 64 * W, m = min(o / 16, p.M - 1), h = n0 / r.D;
      const int ctx = ctx_lds[m];
      pos[i] = (r.ring > 0 ? ctx : min(ctx, r.cols * kPage)) - 1;  // < 0: the row is left alone
      page[i] = -1;
      if (r.do_append && h >= r.n_q && pos[i] >= 0) {
        const int lp = pos[i] / kPage;
        page[i] = r.table[(int64_t)m * r.cols + (r.ring > 0 ? lp % r.ring : lp)];
      }
      cs[i] = 1.f;
      sn[i] = 0.f;
      if (h < r.n_q + r.n_kv && pos[i] >= 0) rope_angle(pos[i], n0 % r.D + o % 16, r.D, r.theta, cs[i], sn[i]);
    }
  }
  // Slices of 64 values of a row (whole cache lines) go round the blocks, eight threads each.
  const int slices = (p.K + 63) / 64;
  auto slice_of = [&](int it, int &m, int &k) {  // this thread's 8 values of its it-th slice; false past the last slice
    const int u = blockIdx.x + gridDim.x * ((tid >> 3) + it * 8 * W);
    m = u / slices;
    k = u % slices * 64 + (tid & 7) * 8;  // K or more: past the end of a row's last, short slice; later slices may follow
    return m < p.M;
  };
  u32x4 xs = {0u, 0u, 0u, 0u};
  int xm, xk;
  if (NORM && slice_of(0, xm, xk) && xk < p.K) xs = *(const u32x4 *)(p.A + (int64_t)xm * p.lda + xk);

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  for (; i < cnt; ++i) {
    read(slot, i);
    mma(i);
    slot = slot == NS - 1 ? 0 : slot + 1;
  }
  __syncthreads();  // every wave is done with its ring
  // Sum the waves' partial tiles through LDS.
  float *const red = (float *)smem, *const red_ss = red + W * ROWS * PITCH;  // [W][ROWS]
#pragma unroll
  for (int t = 0; t < MT; ++t) {
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(wave * ROWS + t * 16 + q * 4 + e) * PITCH + f * 16 + j] = acc[t][f][e];
    if (NORM) {
      ss[t] += __shfl_xor(ss[t], 16, kWave);
      ss[t] += __shfl_xor(ss[t], 32, kWave);
      if (q == 0) red_ss[wave * ROWS + t * 16 + j] = ss[t];
    }
  }
  __syncthreads();
  auto inv_of = [&](int m) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) t += red_ss[w * ROWS + m];
    return rsqrtf(t / (float)p.K + fu.eps);
  };
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int o = tid + i * 64 * W, m = ROPE ? o / 16 : o / COLS, col = ROPE ? o % 16 : o % COLS, n = n0 + col;
    if (o >= OUT || m >= p.M || n >= p.N) continue;
    float v = 0.f, up = 0.f;  // up: the SiLU pair's up column, or the RoPE pair's second half
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float *row = red + (w * ROWS + m) * PITCH + col;
      v += row[0];
      if (SILU) up += row[COLS];
      if (ROPE) up += row[16];
    }
    if (NORM) {
      const float inv = inv_of(m);
      v *= inv;
      up *= inv;
    }
    const int64_t dst = (int64_t)m * p.ldc + n;
    if (EPI == EPI_F32) ((float *)p.C)[dst] = v;
    else if (EPI == EPI_BF16) ((uint16_t *)p.C)[dst] = f2bf(v);
    else if (EPI == EPI_RESID) ((uint16_t *)p.C)[dst] = f2bf(old[i] + v);
    else if (SILU) ((uint16_t *)p.C)[dst] = f2bf(silu(v) * up);
    if (ROPE) {
      const RopeArgs &r = fu.rope;
      const int h = n0 / r.D, d = n % r.D;
      uint16_t lo = f2bf(v), hi = f2bf(up);
      if (h < r.n_q + r.n_kv && pos[i] >= 0) {
        const float a0 = bf2f(lo), b0 = bf2f(hi);
        lo = f2bf(a0 * cs[i] - b0 * sn[i]);
        hi = f2bf(b0 * cs[i] + a0 * sn[i]);
      }
      uint16_t *c = (uint16_t *)p.C + dst;
      c[0] = lo;
      c[half] = hi;
      if (page[i] >= 0 && page[i] < r.pool_pages) {
        const int64_t blk = (int64_t)kPage * r.D;
        const int at = pos[i] % kPage;
        uint16_t *base = r.pool + (int64_t)page[i] * 2 * r.n_kv * blk;
        if (h < r.n_q + r.n_kv) {  // k: row-major slots
          uint16_t *kd = base + (h - r.n_q) * blk + at * r.D + d;
          kd[0] = lo;
          kd[half] = hi;
        } else {  // v: dim-major
          uint16_t *vd = base + (r.n_kv + h - r.n_q - r.n_kv) * blk + d * kPage + at;
          vd[0] = lo;
          vd[half * kPage] = hi;
        }
      }
    }
  }
  if (NORM) {
    for (int it = 0; slice_of(it, xm, xk); ++it) {
      if (xk >= p.K) continue;
      if (it > 0) xs = *(const u32x4 *)(p.A + (int64_t)xm * p.lda + xk);
      const u32x4 g = *(const u32x4 *)(gain_lds + xk * 2);
      *(u32x4 *)(fu.xn + (int64_t)xm * p.K + xk) = norm8(xs, g, inv_of(xm));
    }
  }
}

template <int W, int RW, int AG, int NS, int EPI, bool TILED, bool NORM>
hipError_t launch_cfg(const GemmArgs &a, const SkinnyFuse &f, hipStream_t s) {
  auto kern = gemm_skinny_kernel<W, RW, AG, NS, EPI, TILED, NORM>;
  constexpr size_t base = skinny_lds<W, RW, AG, NS, EPI>() + (EPI == EPI_ROPE ? kCtxLds : 0);
  const size_t lds = base + (NORM ? (size_t)(a.K + 511) / 512 * 1024 : 0);
  static std::atomic<uint64_t> lds_set{0};  // devices whose limit this kernel already raised
  if (hipError_t e = ensure_lds_limit((const void *)kern, base + (NORM ? kGainLds : 0), lds_set); e != hipSuccess) return e;
  const int blocks = (a.N + 16 * RW - 1) / (16 * RW);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * W), lds, s, a, f);
  return hipGetLastError();
}

// Shapes, by the number of 16-column fragments against the 256 compute units
// (8B-shaped layer at 13 rows; the other choice in parentheses):
//  - up to 256 fragments (o_proj, down): one fragment per block on as many
//    waves as LDS holds, o_proj 8.2 us (two fragments, half the chip: 10.3);
//  - up to 512 (qkv, 384): two fragments, 10.7 us, one round of 192 blocks
//    (one fragment, 1.5 rounds: 13.5);
//  - more (an unfused gate_up): four fragments on four waves;
//  - SiLU past 256 fragments: two gate and two up fragments on four waves, two
//    blocks per CU and the whole grid resident at once, 37.4 us. One fragment
//    of each (896 blocks for 512 places) runs in 36.9 us while the process has
//    one hardware queue, but in 49-57 us once it has made a second stream: then
//    blocks that replace finished ones start late, and a grid of one round
//    does not depend on it.
//  - SiLU with its norm, past 512 fragments: four and four on four waves, one
//    block per CU (the gain's LDS would keep a second one out) and one round.
template <int AG, int EPI, bool TILED, bool NORM>
hipError_t launch_shape(const GemmArgs &a, const SkinnyFuse &f, hipStream_t s) {
  const int frags = (a.N + 15) / 16;
  if constexpr (EPI == EPI_SILU) {
    if (frags <= 256) return launch_cfg<8, 1, AG, 2, EPI, TILED, NORM>(a, f, s);
    if constexpr (NORM)
      if (frags > 512) return launch_cfg<4, 4, AG, 2, EPI, TILED, NORM>(a, f, s);
    return launch_cfg<4, 2, AG, 2, EPI, TILED, NORM>(a, f, s);
  } else if constexpr (EPI == EPI_ROPE) {
    return launch_cfg<AG == 4 ? 4 : 8, 2, AG, 3, EPI, TILED, NORM>(a, f, s);
  } else {
    if (frags <= 256 || EPI == EPI_F32)
      return launch_cfg<AG == 4 ? 8 : 16, 1, AG, AG == 4 ? 3 : 2, EPI, TILED, NORM>(a, f, s);
    if (frags <= 512 || EPI == EPI_RESID) return launch_cfg<AG == 4 ? 4 : 8, 2, AG, 3, EPI, TILED, NORM>(a, f, s);
    return launch_cfg<4, 4, AG, 2, EPI, TILED, NORM>(a, f, s);
  }
}

template <int EPI, bool TILED, bool NORM>
hipError_t launch_rows(const GemmArgs &a, const SkinnyFuse &f, hipStream_t s) {
  if (a.M <= 8) return launch_shape<1, EPI, TILED, NORM>(a, f, s);
  if (a.M <= 16) return launch_shape<2, EPI, TILED, NORM>(a, f, s);
  if constexpr (NORM) return hipErrorInvalidValue;  // gemm_norm_skinny
  else return launch_shape<4, EPI, TILED, NORM>(a, f, s);
}

template <int EPI, bool NORM>
hipError_t launch_layout(const GemmArgs &a, const SkinnyFuse &f, hipStream_t s) {
  if constexpr (EPI == EPI_F32) {  // the router, never tiled
    return a.b_tiled ? hipErrorInvalidValue : launch_rows<EPI, false, NORM>(a, f, s);
  } else {
    return a.b_tiled ? launch_rows<EPI, true, NORM>(a, f, s) : launch_rows<EPI, false, NORM>(a, f, s);
  }
}

bool fits(const GemmArgs &a) { return a.M <= kSkinnyRows && !a.group_off && !a.a_gather && a.splits == 1; }

}  // namespace

hipError_t launch_gemm_skinny(const GemmArgs &a, hipStream_t s) {
  if (!fits(a)) return hipErrorInvalidValue;
  const SkinnyFuse none{};
  switch (a.epi) {
    case EPI_BF16: return launch_layout<EPI_BF16, false>(a, none, s);
    case EPI_F32: return launch_layout<EPI_F32, false>(a, none, s);
    case EPI_RESID: return launch_layout<EPI_RESID, false>(a, none, s);
    default: return launch_layout<EPI_SILU, false>(a, none, s);
  }
}

hipError_t launch_gemm_skinny_fused(const GemmArgs &a, const uint16_t *gain, float eps, uint16_t *xn,
                                    const RopeArgs *rope, hipStream_t s) {
  if (!fits(a) || (!gain && !rope) || (gain && (a.K > kSkinnyNormMaxK || !xn))) return hipErrorInvalidValue;
  SkinnyFuse f{};
  f.gain = gain;
  f.eps = eps;
  f.xn = xn;
  if (rope) {
    f.rope = *rope;
    return gain ? launch_layout<EPI_ROPE, true>(a, f, s) : launch_layout<EPI_ROPE, false>(a, f, s);
  }
  return a.epi == EPI_SILU ? launch_layout<EPI_SILU, true>(a, f, s) : hipErrorInvalidValue;
}

}  // namespace ods
