// Decision-scale block selection (Sec. 3.2: column-sum D and TopK).
//
// pooled_scores_kernel: one workgroup per (b, h, group of query tiles of
//   scale S). For every block v of scales 1..S it recomputes the S^T = K Q^T
//   tile with MFMA and adds P = exp(scale * s - lse) over each tile's queries and
//   the block's keys. Sums run in a fixed order (lane, shuffle tree, waves in
//   order), so results are deterministic.
// topk_kernel: one workgroup per (b, h, g) row; candidate v is kept iff fewer than
//   topk candidates beat it (higher score, or equal score and lower id); kept
//   ids are written ascending.
#include <type_traits>

#include "attn_chunk.h"
#include "device_common.h"
#include "launch.h"

namespace sparvar {

struct ScoreIO {
  GeoTable G;
  const void* q;
  const void* k;
  const float* lse;
  float* scores;
  int64_t q_bh_stride, k_bh_stride;
  int32_t S, G_S, NB;
  int32_t per;  // blocks per workgroup along grid.y (bf16 scoring)
  float scale_log2;
};

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Sum over the 64 lanes, in lane 63 (lane shifts as in wave_incl_scan).
__device__ __forceinline__ float wave_sum_last(float x) {
  auto add = [](float y, int32_t moved) { return y + __int_as_float(moved); };
  x = add(x, dpp_or_zero<0x111, 0xf>(__float_as_int(x)));
  x = add(x, dpp_or_zero<0x112, 0xf>(__float_as_int(x)));
  x = add(x, dpp_or_zero<0x114, 0xf>(__float_as_int(x)));
  x = add(x, dpp_or_zero<0x118, 0xf>(__float_as_int(x)));
  x = add(x, dpp_or_zero<0x142, 0xa>(__float_as_int(x)));
  x = add(x, dpp_or_zero<0x143, 0xc>(__float_as_int(x)));
  return x;
}

// fp32 (parity-grade) scoring: K rows read straight from memory, one reduction per block.
template <typename T, int D, int NW>
__global__ __launch_bounds__(NW * 64) void pooled_scores_f32_kernel(ScoreIO io) {
  constexpr bool kBF16 = std::is_same<T, bf16_bits>::value;
  __shared__ float red[NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const int32_t row = blockIdx.x;  // (b*H + h) * G_S + g
  const int32_t bh = row / io.G_S, g = row - bh * io.G_S;
  const GeoTable& G = io.G;
  const int S = io.S;
  const int32_t tw = G.Tw[S - 1];
  const Tile qt = tile_at(G, S, g / tw, g % tw);
  const int32_t nq = qt.nr * qt.nc;

  const int32_t qslot = wave * kQPerWave + l32;
  const bool qvalid = qslot < nq;
  const int32_t qi = qvalid ? qslot : 0;
  const int32_t qrow = (qt.base - G.C[S - 1]) + (qi / qt.nc) * qt.stride + (qi % qt.nc);

  const T* qplane = static_cast<const T*>(io.q) + (int64_t)bh * io.q_bh_stride;
  const T* kplane = static_cast<const T*>(io.k) + (int64_t)bh * io.k_bh_stride;
  using QFrag = typename std::conditional<kBF16, QFragBF16<D>, QFragF32<D>>::type;
  QFrag qf;
  qf.load(qplane + (int64_t)qrow * D, half);
  const float lse2 = io.lse[(int64_t)bh * G.h[S - 1] * G.w[S - 1] + qrow] * kLog2e;

  float* out = io.scores + (int64_t)row * io.NB;
  for (int32_t v = 0; v < io.NB; ++v) {
    const Tile t = block_tile(G, v);
    const int32_t rpc = kChunk / t.nc;
    float acc = 0.f;
    for (int32_t r0 = 0; r0 < t.nr; r0 += rpc) {
      const int32_t rows = (t.nr - r0 < rpc) ? t.nr - r0 : rpc;
      const Chunk c = make_chunk(t.base + r0 * t.stride, t.nc, t.stride, rows * t.nc);
      f32x16 st[2];
      chunk_scores<D>(kplane, c, qf, l32, half, st);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool ok = qvalid && key_of(kt, r, half) < c.count;
          acc += ok ? __builtin_amdgcn_exp2f(st[kt][r] * io.scale_log2 - lse2) : 0.f;
        }
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (tid == 0) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[w];
      out[v] = s;
    }
    __syncthreads();
  }
}


// bf16 scoring: one workgroup per (b, h, group of TPW query tiles of scale S),
// WPT waves per tile. Every query of a head scores against all keys of scales
// 1..S, so the tiles of a group share each K chunk: chunks stream HBM -> LDS
// (direct 16-byte loads, swizzled rows, double buffered) once per group.
// S^T = K Q^T on MFMA; each lane accumulates exp2(scale*log2e*s - lse*log2e) over
// its keys and its query; at the end of a block the wave sum goes to LDS, and a
// tile's score is the sum over its waves in order (deterministic). Blocks of a
// row are split over grid.y.
//
// At most 128 VGPRs for the four-wave forms at d = 128, four waves per SIMD: they
// took 129 (11x11 tiles, 32 planes, 32x32: 65 -> 70 us; with 128, 67).
template <int D, int WPT, int TPW>
__global__ __launch_bounds__(WPT * TPW * 64, D == 128 && WPT * TPW == 4 ? 4 : 1) void pooled_scores_kernel(ScoreIO io) {
  constexpr int NW = WPT * TPW;
  constexpr int KC = 64, NT = NW * 64, U = D / 8, kRow = D * 2, kTile = KC * kRow;
  constexpr int kLoads = KC * U / NT;
  static_assert((KC * U) % NT == 0, "chunk must split evenly over the workgroup");
  // two K stages as separate arrays, so the compiler can tell that copies into
  // one stage never touch the stage being read
  __shared__ __attribute__((aligned(16))) char kstage0[kTile];
  __shared__ __attribute__((aligned(16))) char kstage1[kTile];
  extern __shared__ float red[];  // [NW][per] per-wave block sums

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int32_t groups = (io.G_S + TPW - 1) / TPW;
  const int32_t bh = blockIdx.x / groups;
  const int32_t g0 = (blockIdx.x - bh * groups) * TPW;
  const GeoTable& G = io.G;
  const int S = io.S;
  const int32_t tw = G.Tw[S - 1];
  const int32_t g = g0 + wave / WPT;  // this wave's query tile
  const bool gvalid = g < io.G_S;
  const Tile qt = tile_at(G, S, gvalid ? g / tw : 0, gvalid ? g % tw : 0);
  const int32_t nq = qt.nr * qt.nc;
  const int32_t qslot = (wave % WPT) * kQPerWave + l32;
  const bool qvalid = gvalid && qslot < nq;
  const int32_t qi = qvalid ? qslot : 0;
  const int32_t qrow = (qt.base - G.C[S - 1]) + (qi / qt.nc) * qt.stride + (qi % qt.nc);
  const bf16_bits* qplane = static_cast<const bf16_bits*>(io.q) + (int64_t)bh * io.q_bh_stride;
  const char* kbytes = reinterpret_cast<const char*>(static_cast<const bf16_bits*>(io.k) + (int64_t)bh * io.k_bh_stride);
  QFragBF16<D> qf;
  qf.load(qplane + (int64_t)qrow * D, half);
  float lse2 = io.lse[(int64_t)bh * G.h[S - 1] * G.w[S - 1] + qrow] * kLog2e;
  // An LSE of -inf makes every exponential inf. Kept finite here, because masked
  // scores are -inf and would give NaN with it instead of adding 0.
  if (lse2 == -INFINITY) lse2 = -3.402823466e38f;

  int ld_row[kLoads], ld_unit[kLoads];
#pragma unroll
  for (int j = 0; j < kLoads; ++j) {
    const int slot = (j * NW + wave) * 64 + lane;
    ld_row[j] = slot / U;
    ld_unit[j] = (slot % U) ^ (unit_swizzle(ld_row[j]) & (U - 1));
  }
  int k_off[2][D / 16];
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    const int r = 32 * kt + l32;
#pragma unroll
    for (int s2 = 0; s2 < D / 16; ++s2) k_off[kt][s2] = r * kRow + 16 * ((2 * s2 + half) ^ (unit_swizzle(r) & (U - 1)));
  }
  auto issue = [&](const Chunk& c, auto stage_c) {
    constexpr int SG = decltype(stage_c)::value;
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int first = (j * NW + wave_s) * 64;
      const int r = ld_row[j];
      const uint32_t off = (uint32_t)(chunk_token(c, chunk_slot(r, c.count)) * D + 8 * ld_unit[j]) * 2u;
      dma16(kbytes + off, (SG == 0 ? kstage0 : kstage1) + first * 16);
    }
  };

  // this workgroup scores blocks [v0, v1)
  const int32_t per = io.per;
  const int32_t v0 = blockIdx.y * per;
  const int32_t v1 = (v0 + per < io.NB) ? v0 + per : io.NB;
  BlockWalker<KC> walk;
  walk.start(&G, v0, v1);
  Chunk c0;
  int32_t b0 = 0;
  bool last0 = false;
  bool have = walk.next(c0, b0, last0);
  if (have) issue(c0, std::integral_constant<int, 0>{});
  float psum = 0.f, part = 0.f;

  // The products of one 32-key tile interleaved with the exponentials of the tile
  // before: a product holds the matrix unit for 32 cycles, and the two or four scores
  // between products take about as long on the vector units, which otherwise run one
  // after the other (the chunk's waves leave the barrier together). Keys past the
  // chunk's count are masked first, only in tiles that have some: a mask waits for its
  // tile's products (masking both tiles of every partial chunk, 11x11 tiles as above
  // took 67 us, 63 now).
  // 16 heads of 4096 queries, 10521 keys in 172 blocks: 256 -> 204 us (865 TFLOP/s).
  constexpr int kSteps = D / 16, kPer = 16 / kSteps;
  f32x16 sc1;  // second tile of the previous chunk: -inf (adding 0) before the first
#pragma unroll
  for (int r = 0; r < 16; ++r) sc1[r] = -INFINITY;
  int32_t count1 = KC, blk1 = v0;
  bool last1 = false;
  auto add_scores = [&](const f32x16& sc, int s2) {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      part += __builtin_amdgcn_exp2f(__builtin_fmaf(sc[s2 * kPer + i], io.scale_log2, -lse2));
  };
  // after the second tile of a chunk: its sum, and at the end of a block the wave's
  auto end_chunk = [&]() {
    psum += qvalid ? part : 0.f;
    part = 0.f;
    if (last1) {
      const float sw = wave_sum_last(psum);
      if (lane == 63) red[wave * per + (blk1 - v0)] = sw;
      psum = 0.f;
    }
  };

  auto step = [&](auto stage_c) -> bool {
    constexpr int SG = decltype(stage_c)::value;
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    const char* kst = SG == 0 ? kstage0 : kstage1;
    u32x4 kf[kSteps], kg[kSteps];
#pragma unroll
    for (int s2 = 0; s2 < kSteps; ++s2) kf[s2] = *reinterpret_cast<const u32x4*>(kst + k_off[0][s2]);
    __builtin_amdgcn_sched_barrier(0);
    Chunk cn;
    int32_t bn = 0;
    bool lastn = false;
    const bool have_n = walk.next(cn, bn, lastn);
    if (have_n) issue(cn, std::integral_constant<int, SG ^ 1>{});
    if (count1 < KC) mask_tile(sc1, count1 - 32, half);
    f32x16 sc0 = zero16();
#pragma unroll
    for (int s2 = 0; s2 < kSteps; ++s2) {
      __builtin_amdgcn_sched_barrier(0);
      add_scores(sc1, s2);
      sc0 = mfma_bf16(as_bf16x8(kf[s2]), qf.f[s2], sc0);
      kg[s2] = *reinterpret_cast<const u32x4*>(kst + k_off[1][s2]);
    }
    __builtin_amdgcn_sched_barrier(0);
    end_chunk();
    if (c0.count < 32) mask_tile(sc0, c0.count, half);
    sc1 = zero16();
#pragma unroll
    for (int s2 = 0; s2 < kSteps; ++s2) {
      __builtin_amdgcn_sched_barrier(0);
      sc1 = mfma_bf16(as_bf16x8(kg[s2]), qf.f[s2], sc1);
      add_scores(sc0, s2);
    }
    __builtin_amdgcn_sched_barrier(0);
    count1 = c0.count;
    blk1 = b0;
    last1 = last0;
    c0 = cn;
    b0 = bn;
    last0 = lastn;
    return have_n;
  };
  while (have) {
    if (!step(std::integral_constant<int, 0>{})) break;
    if (!step(std::integral_constant<int, 1>{})) break;
  }
  if (count1 < KC) mask_tile(sc1, count1 - 32, half);
#pragma unroll
  for (int s2 = 0; s2 < kSteps; ++s2) add_scores(sc1, s2);
  end_chunk();
  __syncthreads();
  const int32_t nv = v1 - v0;
  for (int32_t i = tid; i < TPW * nv; i += NT) {
    const int t = i / nv;
    const int32_t v = v0 + (i - t * nv);
    if (g0 + t >= io.G_S) continue;
    float sc = 0.f;
#pragma unroll
    for (int w = 0; w < WPT; ++w) sc += red[(t * WPT + w) * per + (v - v0)];
    io.scores[((int64_t)bh * io.G_S + g0 + t) * io.NB + v] = sc;
  }
}

// One workgroup per row, a candidate per thread: its rank is the number of
// candidates that beat it, counted over the row in LDS four scores a read (the same
// address in every lane); the place of a kept id is the count of kept ids before it.
// Latency-bound: 1024 rows of 172 candidates took 22 us with one wave per row, 8 now.
// NT threads, as many waves as the row's candidates fill, up to four: with four
// throughout, 4096 rows of 47 candidates took 7.4 us and 9216 of 97 took 25.1, with
// one and two waves 4.2 and 17.7.
template <int NT>
__global__ __launch_bounds__(NT) void topk_kernel(const float* __restrict__ scores, int32_t nb, int32_t topk,
                                                  int32_t* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) float s_sc[];  // nb scores, padded with -inf to a multiple of 4
  __shared__ int32_t wt[NT / 64];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const float* sr = scores + row * nb;
  const int32_t nb4 = (nb + 3) & ~3;
  for (int32_t i = tid; i < nb4; i += NT) s_sc[i] = i < nb ? sr[i] : -INFINITY;
  __syncthreads();
  int32_t* orow = out + row * topk;
  int32_t placed = 0;
  for (int32_t v0 = 0; v0 < nb; v0 += NT) {
    const int32_t v = v0 + tid;
    int32_t better = 0;
    if (v < nb) {
      const float x = s_sc[v];
#pragma unroll 4
      for (int32_t u = 0; u < nb4; u += 4) {
        const float4 y = *reinterpret_cast<const float4*>(s_sc + u);
        // (padding: -inf never exceeds x, and its index is past v)
        better += (y.x > x) | ((y.x == x) & (u < v));
        better += (y.y > x) | ((y.y == x) & (u + 1 < v));
        better += (y.z > x) | ((y.z == x) & (u + 2 < v));
        better += (y.w > x) | ((y.w == x) & (u + 3 < v));
      }
    }
    const bool keep = v < nb && better < topk;
    int32_t total;
    const int32_t pos = placed + block_excl_scan<NT>(keep ? 1 : 0, wt, total);
    if (keep && pos < topk) orow[pos] = v;  // a strict total order selects exactly min(topk, nb)
    placed += total;
  }
  const int32_t nsel = topk < nb ? topk : nb;
  for (int32_t p = nsel + tid; p < topk; p += NT) orow[p] = -1;
}

namespace {
template <typename T, int D>
hipError_t launch_scores_f32(const ScoreIO& io, int nw, int32_t grid, hipStream_t stream) {
  switch (nw) {
    case 1: hipLaunchKernelGGL((pooled_scores_f32_kernel<T, D, 1>), dim3(grid), dim3(64), 0, stream, io); break;
    case 2: hipLaunchKernelGGL((pooled_scores_f32_kernel<T, D, 2>), dim3(grid), dim3(128), 0, stream, io); break;
    case 4: hipLaunchKernelGGL((pooled_scores_f32_kernel<T, D, 4>), dim3(grid), dim3(256), 0, stream, io); break;
    default: hipLaunchKernelGGL((pooled_scores_f32_kernel<T, D, 8>), dim3(grid), dim3(512), 0, stream, io); break;
  }
  return hipGetLastError();
}
// Query tiles of a head are grouped (TPW per workgroup) and the blocks of a row
// split over grid.y so that about 1024 workgroups run.
template <int D, int WPT, int TPW>
hipError_t launch_scores_bf16(const ScoreIO& io, int32_t BH, hipStream_t stream) {
  const int32_t grid = BH * ((io.G_S + TPW - 1) / TPW);
  int32_t splits = (1024 + grid - 1) / grid;
  if (splits > io.NB) splits = io.NB;
  if (splits < 1) splits = 1;
  const int32_t per = (io.NB + splits - 1) / splits;
  splits = (io.NB + per - 1) / per;
  ScoreIO io2 = io;
  io2.per = per;
  const size_t red = (size_t)WPT * TPW * per * sizeof(float);
  hipLaunchKernelGGL((pooled_scores_kernel<D, WPT, TPW>), dim3(grid, splits), dim3(WPT * TPW * 64), red, stream, io2);
  return hipGetLastError();
}

template <int D>
hipError_t launch_scores_bf16_d(const ScoreIO& io, int32_t BH, int wpt, hipStream_t stream) {
  switch (wpt) {
    case 1: return launch_scores_bf16<D, 1, 4>(io, BH, stream);
    case 2: return launch_scores_bf16<D, 2, 4>(io, BH, stream);
    case 4: return launch_scores_bf16<D, 4, 1>(io, BH, stream);
    default: return launch_scores_bf16<D, 8, 1>(io, BH, stream);
  }
}
}  // namespace

hipError_t launch_pooled_scores(const ScoreArgs& a, hipStream_t stream) {
  const GeoTable& G = *a.G;
  const int S = a.S;
  ScoreIO io;
  io.G = G;
  io.q = a.q;
  io.k = a.k;
  io.lse = a.lse;
  io.scores = a.scores;
  io.q_bh_stride = a.q_bh_stride;
  io.k_bh_stride = a.k_bh_stride;
  io.S = S;
  io.G_S = tiles_of(G, S);
  io.NB = G.NB[S];
  io.per = io.NB;
  io.scale_log2 = a.softmax_scale * kLog2e;
  const int32_t tile_q = G.eh[S - 1] * G.ew[S - 1];
  const int nw = tile_q <= 32 ? 1 : tile_q <= 64 ? 2 : tile_q <= 128 ? 4 : 8;
  const int32_t grid = a.BH * io.G_S;
  if (grid == 0) return hipSuccess;
  // per-wave block sums in LDS: at most 8 waves x NB floats
  if (a.bf16 && (size_t)8 * io.NB * sizeof(float) <= 32 * 1024)
    return a.d == 64 ? launch_scores_bf16_d<64>(io, a.BH, nw, stream) : launch_scores_bf16_d<128>(io, a.BH, nw, stream);
  if (a.bf16) return a.d == 64 ? launch_scores_f32<bf16_bits, 64>(io, nw, grid, stream)
                               : launch_scores_f32<bf16_bits, 128>(io, nw, grid, stream);
  return a.d == 64 ? launch_scores_f32<float, 64>(io, nw, grid, stream) : launch_scores_f32<float, 128>(io, nw, grid, stream);
}

hipError_t launch_topk(const float* scores, int32_t rows, int32_t nb, int32_t topk, int32_t* out,
                       hipStream_t stream) {
  if (rows == 0) return hipSuccess;
  const size_t shmem = (size_t)((nb + 3) & ~3) * sizeof(float);
  if (nb <= 64) hipLaunchKernelGGL(topk_kernel<64>, dim3(rows), dim3(64), shmem, stream, scores, nb, topk, out);
  else if (nb <= 128) hipLaunchKernelGGL(topk_kernel<128>, dim3(rows), dim3(128), shmem, stream, scores, nb, topk, out);
  else if (nb <= 192) hipLaunchKernelGGL(topk_kernel<192>, dim3(rows), dim3(192), shmem, stream, scores, nb, topk, out);
  else hipLaunchKernelGGL(topk_kernel<256>, dim3(rows), dim3(256), shmem, stream, scores, nb, topk, out);
  return hipGetLastError();
}

}  // namespace sparvar
