// Large-M bf16 GEMM Y = X W^T on the gfx950 matrix cores: the projections of
// a prefill (the confidence engine's scoring pass), where M is a token count
// in the thousands and the product is compute-bound (intensity ~ M flop per
// weight byte, far above the ~315 flop/byte ridge of the chip).
//
//   * workgroup tile 256 (m) x 256 (n), 8 waves in a 2 x 4 grid, each wave a
//     128 x 64 sub-tile held as 4 x 2 accumulators of the 32x32x16 bf16 MFMA
//     (128 fp32 per lane, 184 registers in all), so two waves share each SIMD
//     and one issues MFMAs while the other waits on its LDS reads or a
//     barrier (2-3% faster than 4 waves of 128 x 128 sub-tiles, one per
//     SIMD, on every 8B-class shape at M = 16K and 40K).  Where such tiles
//     leave CUs idle, tiles of 192 x 256, 128 x 256 and 128 x 128 rows and a
//     split of K over workgroups (fp32 partials, summed in split order by the
//     consumer) take over: plan_tiles weighs them;
//   * K is consumed in stages of 32 columns (64 for the 128 x 128 tile, whose
//     stages would otherwise be mostly barrier): the X and W slices of a stage
//     go straight from global memory into LDS with the gfx950 direct-to-LDS
//     loads (16 bytes per lane, no register staging), spread evenly over the
//     waves; four LDS stages keep three stages of loads in flight under the
//     MFMAs;
//   * both operands keep the fragment-major layouts of the decode path (the
//     packed weights and the tiled activations, 1 KB per 16 x 32 fragment), so
//     every direct load is one contiguous 1 KB per wave and every LDS read of
//     a 16-lane group is 256 contiguous bytes (no bank conflicts, no swizzle);
//     a row-major X is gathered into the same LDS order by the per-lane
//     addresses of the direct loads;
//   * the tile order is XCD-aware: consecutive workgroups land on different
//     XCDs, so the linear id is remapped to give each XCD a contiguous range
//     of tiles, walked in groups of 1024 rows (4 m-tiles) so the X and W slices a group
//     streams are shared in that XCD's L2 (groups of 4 measured 1-4% faster
//     than 8 at M = 16K-40K, groups of 16 7-10% slower).
// Epilogues: fp32 store, fp32 accumulate (residual update), and SwiGLU over a
// gate/up matrix packed in 32 + 32 row superblocks (bf16 output, tiled or
// row-major).
//
// Grouped form (the mixture of experts of a prefill): the m-tiles are tiles of
// BM entries of the experts' lists (tile_off from the planner), a tile's
// weights are its expert's, and its A rows are gathered per lane: the entry's
// token row of the normed input (gate/up), or the expert's SwiGLU rows (down).
// Both are row-major: a row's 32 columns of a stage are 64 consecutive bytes
// (gathered from the tiled layout they were four 16-byte pieces of four
// lines, and 65168 entries of the 30B-A3B shape's gate/up took 1138 us
// instead of 596).  The gate/up epilogue writes SwiGLU rows at the entries' positions;
// the down epilogue scatters routing weight * product into the per-slot
// outputs [slot][token][hidden].
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace sevo {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// One direct load of a wave per stage: a 1 KB operand fragment (16 rows x 32
// columns) through a wave-uniform descriptor over the region it streams.
struct LgLoad {
  __amdgpu_buffer_rsrc_t r;
  uint32_t voff;    // this lane's byte offset
  uint32_t soff;    // byte offset of the first stage (wave-uniform)
  uint32_t step;    // bytes per stage (wave-uniform)
  uint32_t lds;     // element offset in the stage buffer
};

// f(0), f(1), ... f(H - 1), the group a compile-time constant
template <int H, int h = 0, typename F>
__device__ __forceinline__ void lg_groups(F f) {
  f(std::integral_constant<int, h>{});
  if constexpr (h + 1 < H) lg_groups<H, h + 1>(f);
}

// EPI 0: out fp32 [M][ldo] = Y;  EPI 1: out += Y;  EPI 2: SwiGLU -> out_bf16;
// EPI 3 (grouped down): out [slot][token][N] = weight * Y
// XT 1: X in the tiled activation layout, else row-major with stride ldx
// GR 1: grouped (M = the rows of X: tokens for gate/up, entries for down)
// Tile BM x BN, NW waves in a grid of NW / (BN / 64) x BN / 64; a stage is
// KSUB 32-column steps.  NS LDS stages, one multiplied and up to NS - 1 loading
// (three: two workgroups per CU).  Split K (EPI 0): blockIdx.y takes kchunk columns and
// writes the partial out[blockIdx.y][M][ldo].
template <int BM, int BN, int NW, int KSUB, int EPI, int XT, int GR, int NS = 4>
__global__ __launch_bounds__(64 * NW, (NS == 3 ? 4 : 1)) void
gemm_large_kernel(const bf16_t* __restrict__ X, int ldx, int M, const bf16_t* __restrict__ W,
                  int N, int K, int kchunk, float* __restrict__ out, int ldo,
                  bf16_t* __restrict__ out_bf16, int out_tiled, int tiles_m, int tiles_n,
                  GroupArgs g) {
  constexpr int WN = BN / 64, WM = NW / WN;     // wave grid; a wave owns 64 columns
  constexpr int MT = BM / WM / 32;              // 32-row MFMA tiles per wave
  static_assert(WN * WM == NW && MT * WM * 32 == BM, "wave grid");
  constexpr int FA = BM / 16, FS = FA + BN / 16;  // fragments of a 32-column step
  constexpr int SUB = FS * 512;                   // elements of a step
  constexpr int D = (KSUB * FS + NW - 1) / NW;    // direct loads per wave and stage
  constexpr bool kIdle = D * NW != KSUB * FS;     // some waves have one load too many
  constexpr int STAGE = KSUB * SUB + (kIdle ? NW * 512 : 0);
  __shared__ __attribute__((aligned(1024))) bf16_t smem[NS * STAGE];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // ---- tile order: XCD-contiguous ranges, groups of GM m-tiles.  Grouped: of
  // the tiles that the entry lists fill (the grid has room for a part-filled
  // tile per expert more; dividing that among the XCDs left the last ones idle)
  if constexpr (GR) tiles_m = g.tile_off[g.E] * g.sub;
  const int total = tiles_m * tiles_n;
  int t = blockIdx.x;
  if (GR && t >= total) return;  // uniform over the workgroup, before any barrier
  {
    const int per = total >> 3;  // full rounds of 8
    if (t < per * 8) t = (t & 7) * per + (t >> 3);
  }
  constexpr int GM = 1024 / BM;
  const int group = t / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsize = min(GM, tiles_m - first_m);
  const int in_group = t - group * GM * tiles_n;
  const int tm = first_m + in_group % gsize;
  const int tn = in_group / gsize;
  int m0 = tm * BM;
  const int n0 = tn * BN;
  // grouped: the expert of m-tile tm and the tile's first entry of that expert
  int rows = M;      // rows of this tile's matrix (the expert's entries)
  int ent0 = 0;      // first entry of the expert
  if constexpr (GR) {
    const int table_tile = tm / g.sub, part = tm - table_tile * g.sub;
    int lo = 0, hi = g.E;  // tile_off[lo] <= table_tile < tile_off[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (g.tile_off[mid] <= table_tile) lo = mid;
      else hi = mid;
    }
    ent0 = g.offsets[lo];
    rows = g.offsets[lo + 1] - ent0;
    m0 = ((table_tile - g.tile_off[lo]) * g.sub + part) * BM;
    if (m0 >= rows) return;  // uniform, before any barrier
    W += (size_t)lo * N * K;
  }

  const int KS = K >> 5;  // 32-column steps
  const int ks0 = EPI == 0 ? blockIdx.y * (kchunk >> 5) : 0;
  const int ks1 = EPI == 0 ? min(KS, ks0 + (kchunk >> 5)) : KS;
  const int nst = (ks1 - ks0 + KSUB - 1) / KSUB;  // stages
  const int last_blk = (M - 1) >> 4;
  const int last_sb = (N >> 6) - 1;

  // ---- this wave's direct loads: fragments wave, wave + NW, ... of a stage.
  // The loop issues full stages throughout.  The descriptors of W and of a tiled
  // X end with the split, so the stages past the last one load zeros from them
  // and touch no memory; of a row-major X they may read later columns of the
  // rows before the last.  Those stages are not multiplied.
  LgLoad ld[D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const int f = wave + NW * i;
    const int sub = f / FS, r = f % FS;
    LgLoad& l = ld[i];
    l.lds = f * 512;
    if (kIdle && f >= KSUB * FS) {
      l = LgLoad{__builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(W), 0, 0, 0x00020000), 0, 0, 0,
                 (uint32_t)(KSUB * SUB + wave * 512)};
    } else if (r < FA) {
      if constexpr (GR) {
        // one descriptor over the whole X; a row past the tile's entries gets
        // an offset past the records (the direct load then writes zeros)
        static_assert(!GR || !XT, "gathered rows are row-major");
        l.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(X), 0, (uint32_t)M * ldx * 2,
                                                0x00020000);
        const int j = m0 + 16 * r + (lane & 15);
        l.voff = 0x80000000u;
        if (j < rows) {
          const int row = EPI == 2 ? g.assign[ent0 + j] / g.k : ent0 + j;
          l.voff = (uint32_t)(((size_t)row * ldx + 8 * (lane >> 4)) * 2);
        }
        l.soff = sub * 64u;
        l.step = KSUB * 64u;
      } else {
        const int blk = min((m0 >> 4) + r, last_blk);
        if constexpr (XT) {
          l.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(X + (size_t)blk * KS * 512), 0,
                                                  ks1 * 1024, 0x00020000);
          l.voff = lane * 16;
          l.soff = (ks0 + sub) * 1024u;
          l.step = KSUB * 1024u;
        } else {
          // run p = lane of the fragment is row 16 blk + p % 16, columns
          // 8 (p / 16) .. + 8 of the step; rows past M fall outside the records,
          // which end with the last row's columns of the split (X may be a
          // column slice that ends there)
          const int nr = min(16, M - 16 * blk);
          l.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(X + (size_t)16 * blk * ldx), 0,
                                                  ((nr - 1) * ldx + ks1 * 32) * 2, 0x00020000);
          l.voff = ((lane & 15) * ldx + 8 * (lane >> 4)) * 2;
          l.soff = (ks0 + sub) * 64u;
          l.step = KSUB * 64u;
        }
      }
    } else {
      const int c = r - FA;  // 16-row weight fragment c of the tile
      const int sb = min((n0 >> 6) + (c >> 2), last_sb);
      l.r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(W + (size_t)sb * KS * 2048), 0,
                                              ks1 * 4096, 0x00020000);
      l.voff = (c & 3) * 1024 + lane * 16;
      l.soff = (ks0 + sub) * 4096u;
      l.step = KSUB * 4096u;
    }
  }
  // loads [i0, i1) of stage st
  auto issue = [&](int st, int i0, int i1) {
    bf16_t* so = smem + (st % NS) * STAGE;
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (i >= i0 && i < i1) dma16(ld[i].r, ld[i].voff + (ld[i].soff + st * ld[i].step), so + ld[i].lds);
  };

  f32x16 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // LDS read offsets (elements, within a step) of this lane's operand runs.
  // A: m-tile mt covers row blocks wm * 2 MT + 2 mt + {0, 1}; lane rows l % 32.
  // B: n-tile nt is half nt of superblock wn (the gate or up half for SwiGLU),
  // fragments 2 nt + {0, 1}.
  const int half = (lane >> 4) & 1, r16 = lane & 15, khi = lane >> 5;
  const int a_off = (wm * 2 * MT + half) * 512 + r16 * 8 + khi * 128;
  const int b_off = (FA + wn * 4 + half) * 512 + r16 * 8 + khi * 128;

  constexpr int H = 2 * KSUB;  // 16-k MFMA groups of a stage
  // TR: the weights as the MFMA's A operand, so that a lane holds four
  // consecutive columns of one row (one store of a run instead of four)
  constexpr bool TR = EPI == 2;
  struct Frags {
    bf16x8v a[MT], b[2];
  };
  // operand runs of 16-k group h of stage st
  auto read = [&](Frags& f, int st, int h) {
    const bf16_t* so = smem + (st % NS) * STAGE + (h >> 1) * SUB + (h & 1) * 256;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      f.a[mt] = *reinterpret_cast<const bf16x8v*>(so + a_off + mt * 1024);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
      f.b[nt] = *reinterpret_cast<const bf16x8v*>(so + b_off + nt * 1024);
  };
  // column by column: the weight operand stays for MT products in a row (1.3%
  // faster than row by row on the 8B-class shapes at 8192 rows)
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        acc[mt][nt] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[nt], f.a[mt], acc[mt][nt], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[mt], f.b[nt], acc[mt][nt], 0, 0, 0);
  };

  // Pipeline: up to NS - 1 stages of direct loads are in flight while one is
  // multiplied.  Group h of stage kt: the LDS reads of the next group and a
  // share of stage kt + NS - 1's direct loads (its buffer held stage kt - 1, which
  // every wave finished reading before the last barrier) are interleaved with
  // the group's MFMAs; before the last group, whose reads are of stage kt + 1,
  // that stage is waited for and the waves meet.  sched_group_barrier masks:
  // 0x8 MFMA, 0x100 LDS read, 0x10 vector memory.  Spreading the direct loads
  // this way measured faster than issuing a stage's loads in one burst.
  auto interleave = [&](auto nd_tag) {
    constexpr int nd = decltype(nd_tag)::value, nm = 2 * MT, nr = MT + 2;
#pragma unroll
    for (int i = 0; i < nm; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
      constexpr int per = (nr + nm - 1) / nm;
      const int left = nr - i * per;
      if (left >= per) __builtin_amdgcn_sched_group_barrier(0x100, per, 0);
      else if (left > 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (i < nd && i < nm - 1) __builtin_amdgcn_sched_group_barrier(0x10, 1, 0);
    }
  };
  Frags fr[2];
  for (int st = 0; st < NS - 1; ++st) issue(st, 0, D);
  wait_vmcnt<(NS - 2) * D>();  // stage 0 landed
  lds_barrier();
  read(fr[0], 0, 0);
  for (int kt = 0; kt < nst; ++kt) {
    lg_groups<H>([&](auto h_tag) {
      constexpr int h = decltype(h_tag)::value;
      constexpr int i0 = D * h / H, i1 = D * (h + 1) / H;
      if constexpr (h == H - 1) {
        // the stages from kt + 2 on and this stage's share of the last may still be loading
        // (after the last stage this reads a stale buffer that is never used:
        // keeping the step unconditional keeps the LDS reads interleaved)
        wait_vmcnt<(NS - 3) * D + i0>();
        wait_lgkm0();
        lds_barrier();
      }
      issue(kt + NS - 1, i0, i1);
      if constexpr (h == H - 1) read(fr[(h + 1) & 1], kt + 1, 0);
      else read(fr[(h + 1) & 1], kt, h + 1);
      mma(fr[h & 1]);
      interleave(std::integral_constant<int, i1 - i0>{});
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  wait_vmcnt<0>();

  // ---- epilogue.  Accumulator element e of tile (mt, nt): row
  // 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32.
  // (TR: row lane % 32, column 8 (e / 4) + 4 (lane / 32) + e % 4.)
  const int col_l = lane & 31;
  auto row_of = [&](int mt, int e) {
    return m0 + (wm * MT + mt) * 32 + 8 * (e >> 2) + 4 * khi + (e & 3);
  };
  if constexpr (EPI == 2) {
    const int F = N >> 1;
    const int sbg = (n0 >> 6) + wn;
    if (sbg <= last_sb) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int row = m0 + (wm * MT + mt) * 32 + col_l;
        if (row >= rows) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int f = sbg * 32 + 8 * q + 4 * khi;
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gt = acc[mt][0][4 * q + e], u = acc[mt][1][4 * q + e];
            v[e] = gt / (1.f + __expf(-gt)) * u;
          }
          const uint2 o = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
          const size_t off = out_tiled ? act_tile_offset(row, f, F) : (size_t)(ent0 + row) * F + f;
          *reinterpret_cast<uint2*>(out_bf16 + off) = o;
        }
      }
    }
  } else if constexpr (EPI == 3) {
    // grouped down: row = entry ent0 + row of the expert -> (token, slot).
    // The tile's BM output rows and routing weights are staged in LDS first
    // (read per row in the loop below, the dependent assign -> weight loads
    // were 128 round trips per lane); every wave's direct loads have landed
    // (wait above), so after the barrier the stage buffers are free.
    lds_barrier();
    int* t_row = reinterpret_cast<int*>(smem);
    float* t_wt = reinterpret_cast<float*>(smem) + BM;
    {
      const int row = m0 + threadIdx.x;  // the first BM threads, one tile row each
      static_assert(BM <= 64 * NW, "a thread per tile row");
      if (threadIdx.x < BM && row < rows) {
        const int asg = g.assign[ent0 + row];
        const int tok = asg / g.k, slot = asg - tok * g.k;
        t_row[threadIdx.x] = slot * g.n + tok;
        t_wt[threadIdx.x] = g.weights[asg];
      }
    }
    wait_lgkm0();
    lds_barrier();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = row_of(mt, e);
        if (row >= rows) continue;
        const int lr = row - m0;
        const float wt = t_wt[lr];
        float* dst = out + (size_t)t_row[lr] * ldo;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const int col = n0 + wn * 64 + nt * 32 + col_l;
          if (col < N) dst[col] = acc[mt][nt][e] * wt;
        }
      }
  } else {
    // a whole 32-row m-tile inside M takes the unmasked path; for the update
    // form all 32 old values of an m-tile are loaded before any store so the
    // loads overlap
    if constexpr (EPI == 0) out += (size_t)blockIdx.y * M * ldo;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const bool full = m0 + (wm * MT + mt) * 32 + 32 <= M;
      float old[2][16];
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        const int col = n0 + wn * 64 + nt * 32 + col_l;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          old[nt][e] = 0.f;
          if constexpr (EPI == 1) {
            const int row = row_of(mt, e);
            if ((full || row < M) && col < N) old[nt][e] = out[(size_t)row * ldo + col];
          }
        }
      }
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        const int col = n0 + wn * 64 + nt * 32 + col_l;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = row_of(mt, e);
          if ((full || row < M) && col < N)
            out[(size_t)row * ldo + col] = EPI == 1 ? old[nt][e] + acc[mt][nt][e] : acc[mt][nt][e];
        }
      }
    }
  }
}

namespace {

struct LgArgs {
  int m, n_out, k, ldx, splits, kchunk;
  const bf16_t* x;
  const bf16_t* w;
  void* out;
  int out_tiled;
  hipStream_t st;
};

template <int BM, int BN, int NW, int KSUB, int EPI, int XT, int GR, int NS = 4>
hipError_t run_lg(const LgArgs& a, int tiles_m, const GroupArgs& g) {
  const int tiles_n = (a.n_out + BN - 1) / BN;
  hipLaunchKernelGGL((gemm_large_kernel<BM, BN, NW, KSUB, EPI, XT, GR, NS>),
                     dim3(tiles_m * tiles_n, a.splits), dim3(64 * NW), 0, a.st, a.x, a.ldx, a.m, a.w,
                     a.n_out, a.k, a.kchunk, static_cast<float*>(a.out), a.n_out,
                     static_cast<bf16_t*>(a.out), a.out_tiled, tiles_m, tiles_n, g);
  return hipGetLastError();
}

template <int BM, int BN, int KSUB>
hipError_t run_tile(const LgArgs& a, int x_tiled, int mode) {
  const int tiles_m = (a.m + BM - 1) / BM;
  const GroupArgs none{};
  if (x_tiled) {
    if (mode == 0) return run_lg<BM, BN, 8, KSUB, 0, 1, 0>(a, tiles_m, none);
    if (mode == 1) return run_lg<BM, BN, 8, KSUB, 1, 1, 0>(a, tiles_m, none);
    return run_lg<BM, BN, 8, KSUB, 2, 1, 0>(a, tiles_m, none);
  }
  if (mode == 0) return run_lg<BM, BN, 8, KSUB, 0, 0, 0>(a, tiles_m, none);
  if (mode == 1) return run_lg<BM, BN, 8, KSUB, 1, 0, 0>(a, tiles_m, none);
  return run_lg<BM, BN, 8, KSUB, 2, 0, 0>(a, tiles_m, none);
}

// The tiles, and what one costs per 1024 columns of k on a busy chip (us,
// besides kTileFixed for its prologue and epilogue): measured over m = 128 ..
// 8192 at the 8B, 32B and 30B-A3B projections.  The larger tiles move fewer
// bytes per flop (a 128 x 128 tile of 64-column stages does half the work of
// 128 x 256 in 0.6 of its time); the smaller ones and K splits fill the chip
// when there are few tiles (512 x 4096 x 12288: 220 us in 32 tiles of 256 x 256,
// 48 us in 8 splits of them; 256 x 4096 x 4096: 77 against 16 us in 64 tiles of
// 128 x 128 in 4 splits; 2242 x 4096 x 12288: 215 us in 144 tiles, 195 us in 192
// of 192 x 256).
struct LgTile {
  int bm, bn;
  double per_1024;
};
const LgTile kTiles[] = {{256, 256, 23.5}, {192, 256, 18.5}, {128, 256, 13.0}, {128, 128, 7.8}};
constexpr int kNumTiles = 4;
constexpr double kTileFixed = 8.0;     // us per tile
constexpr double kPartialPerMB = 0.4;  // us per MB of split partials, written and read back
constexpr int kMaxTileSplits = 8, kMinSplitK = 512;

}  // namespace

LinearPlan plan_tiles(int m, int n_out, int k, int mode, int fixed_splits, int max_splits) {
  LinearPlan best;
  double best_us = 1e30;
  const int splits[] = {1, 2, 3, 4, 6, kMaxTileSplits};
  for (int i = 0; i < kNumTiles; ++i) {
    const LgTile& t = kTiles[i];
    if (t.bn == 128 && k % 64) continue;  // its stages are 64 columns
    const long tiles = (long)((m + t.bm - 1) / t.bm) * ((n_out + t.bn - 1) / t.bn);
    for (int n_splits : splits) {
      int want = n_splits;
      if (fixed_splits > 0 && mode != 2) {
        if (want != 1) break;
        want = fixed_splits;
      } else if (want > 1 && (mode == 2 || want > max_splits || k < want * kMinSplitK)) {
        break;  // (the SwiGLU epilogue needs the whole K range)
      }
      const int chunk = ((k + want - 1) / want + 63) / 64 * 64;
      const int s = (k + chunk - 1) / chunk;
      // rounds of 256 workgroups, one per CU; over many rounds the last one's
      // idle CUs weigh less
      const double r = tiles * s / 256.0;
      const double rounds = r <= 1.0 ? 1.0 : r < 4.0 ? (double)(long)(r + 0.999) : r + 0.5;
      const double us = rounds * (kTileFixed + t.per_1024 * chunk / 1024.0) +
                        (s > 1 ? kPartialPerMB * 4e-6 * s * m * n_out : 0.0);
      if (us < best_us) {
        best_us = us;
        best.tile = i + 1;
        best.k_splits = s;
        best.k_chunk = chunk;
        best.rb = t.bn / 16;
        best.mb = t.bm / 16;
      }
    }
  }
  return best;
}

hipError_t launch_gemm_large(int m, int n_out, int k, int ldx, int x_tiled, int mode,
                             const LinearPlan& plan, const bf16_t* x, const bf16_t* w, void* out,
                             int out_tiled, hipStream_t st) {
  if (m == 0) return hipSuccess;
  const LgArgs a{m, n_out, k, ldx, plan.k_splits, plan.k_chunk, x, w, out, out_tiled, st};
  switch (plan.tile) {
    case 1: return run_tile<256, 256, 1>(a, x_tiled, mode);
    case 2: return run_tile<192, 256, 1>(a, x_tiled, mode);
    case 3: return run_tile<128, 256, 1>(a, x_tiled, mode);
    case 4: return run_tile<128, 128, 2>(a, x_tiled, mode);
    default: return hipErrorInvalidValue;
  }
}

// The rows of a grouped tile from the entries per expert (30B-A3B shape, us of
// a layer's experts with tiles of 64 / 128 / 256 rows: 31 entries each 273 / 268
// / 284, 62 each 330 / 299 / 315, 125 each 462 / 404 / 372, 250 each 767 / 615 /
// 622, 509 each 1426 / 1114 / 1032): half a tile per expert is padding, but the
// larger tile does more per byte.
int moe_group_rows(long long entries, int n_experts) {
  return entries < 96ll * n_experts ? 128 : 256;
}

// The down projection of 256-entry tiles in halves of 128, two workgroups per CU
// (three LDS stages of 24 KB, 99 registers): a short K leaves it bound by its
// scattered fp32 stores, which then run under the other workgroup's products,
// and an expert's last tile pads to 128 entries.  Scoring at 30B-A3B widths, two
// layers, us with whole tiles / halves: 509 entries per expert 3558 / 3510, 250
// each 1981 / 1957, 1250 each 9460 / 9403; 125 each 1238 / 1282, so the line lies
// between.  With the gate/up product on such tiles too 509 each took 3537 against
// 3469, and below 96 entries, on 128-entry tiles, 62 each 980 against 969.
constexpr long long kHalvedMinEntries = 192;

hipError_t launch_gemm_grouped(int down, int m, int n_out, int k, const bf16_t* x,
                               const bf16_t* w, void* out, const GroupArgs& g, int tile_rows,
                               int max_tiles_m, hipStream_t st) {
  if (m == 0 || max_tiles_m == 0) return hipSuccess;
  const LgArgs a{m, n_out, k, k, 1, k, x, w, out, 0, st};
  if (tile_rows == 256 && down && (long long)m >= kHalvedMinEntries * g.E) {
    GroupArgs half = g;
    half.sub = 2;
    return run_lg<128, 256, 8, 1, 3, 0, 1, 3>(a, 2 * max_tiles_m, half);
  }
  if (tile_rows == 128)
    return down ? run_lg<128, 256, 8, 1, 3, 0, 1>(a, max_tiles_m, g)
                : run_lg<128, 256, 8, 1, 2, 0, 1>(a, max_tiles_m, g);
  return down ? run_lg<256, 256, 8, 1, 3, 0, 1>(a, max_tiles_m, g)
              : run_lg<256, 256, 8, 1, 2, 0, 1>(a, max_tiles_m, g);
}

}  // namespace sevo
