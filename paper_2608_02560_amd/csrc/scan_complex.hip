// Selective-SSM scan with the diagonal complex A of Sec. 3, A = a + i w
// (a > 0 in this sign convention, the paper's w_k = pi k being one choice):
//   h_t[n] = exp(-dt_t (a[n] + i w[n])) h_{t-1}[n] + B_t[n] x_t dt_t
//   y_t    = (sum_n C_t[n] Re h_t[n] + Dskip x_t) * silu(z_t)
// with the complex state kept as (real, imaginary) fp32 pairs in VGPRs and
// stored interleaved.
//
// Same work decomposition as the real scan (one lane per (b, d) channel, 64
// adjacent channels per wave, buffer loads, 4-token tiles, for N = 16 the
// tile's B_t / C_t through a wave-private LDS slice).  Per (t, d, n): exp2 of
// dt a' for the magnitude; the angle dt w / (2 pi) in revolutions for v_cos_f32
// / v_sin_f32; then the complex multiply-add
//   re' = c re + s im + B u,   im' = c im - s re,   (c, s) = |decay| (cos, sin).
// The two take angles of up to 256 revolutions either way and reduce them
// exactly: over 4 M angles in each of [0, 8], [0, 64] and [0, 256) and their
// negatives the results are as close to the fp64 ones as those of angles
// reduced by v_fract_f32 first (largest error 1.25e-7 both; closer for negative
// angles below one revolution, 1.2e-7 against 3.6e-7, where fract rounds).  So
// a tile whose |dt| max |w| stays below that skips the 16 reductions a token;
// other tiles reduce.
// The kernel is bound by vector issue (11 plain instructions and 3
// transcendentals per state and token with DPP coefficients and every angle
// reduced, 10 and 3 now, two of them no longer DPP forms).  8 x 3000 x 2048 bf16,
// both passes 730 -> 670 us; 64 x 1000 x 2048 1034 -> 973, fp32 972 -> 917, states
// only 894 -> 814; 256 x 200 x 2048 798 -> 743.
//
// Long sequences over few channels are cut into time chunks as in the real
// scan (two levels):
//   pass 1 (summary): each chunk but the last is scanned from a zero state;
//          its complex end state and its sum of dt go to the workspace;
//   pass 2 (carry):   per (b, d, n), H_c = exp(-S_{c-1} (a + i w)) H_{c-1}
//          + s_{c-1}, sequential over chunks: the composition of the affine
//          maps h -> r h + s that each chunk applies, whose factor is the
//          product of its tokens' decays, exp(-(a + i w) sum dt);
//   pass 3 (replay):  each chunk is rescanned from its carried-in state,
//          producing y and, for the last chunk, hT.
#include "scan_kernels.h"

namespace precog {
namespace {

constexpr float kInv2Pi = 0.15915494309189535f;

// One state's update; bu = B_t u.  REDUCE: the angle may leave the domain of
// v_cos_f32 / v_sin_f32 (256 revolutions either way) and is reduced first.
template <bool REDUCE>
__device__ __forceinline__ void cstate(float& hr, float& hi, float a2, float w1, float dtv, float bu) {
  const float mag = __builtin_amdgcn_exp2f(dtv * a2);
  const float rev = REDUCE ? __builtin_amdgcn_fractf(dtv * w1) : dtv * w1;
  const float c = mag * __builtin_amdgcn_cosf(rev);
  const float s = mag * __builtin_amdgcn_sinf(rev);
  const float re = hr;
  hr = fmaf(c, re, fmaf(s, hi, bu));
  hi = fmaf(c, hi, -(s * re));
}

template <bool REDUCE, int N, int... m>
__device__ __forceinline__ void ctoken(float (&hr)[N], float (&hi)[N], const float (&a2)[N],
                                       const float (&w1)[N], float dtv, float u, float bv,
                                       std::integer_sequence<int, m...>) {
  (cstate<REDUCE>(hr[m], hi[m], a2[m], w1[m], dtv, u * row_bcast<m>(bv)), ...);
}

template <int N, typename TSt>
__device__ __forceinline__ void load_cstate(float (&hr)[N], float (&hi)[N], const TSt* src) {
#pragma unroll
  for (int n = 0; n < N; ++n) {
    hr[n] = to_f32(src[2 * n]);
    hi[n] = to_f32(src[2 * n + 1]);
  }
}

template <int N, typename TSt>
__device__ __forceinline__ void store_cstate(TSt* dst, const float (&hr)[N], const float (&hi)[N]) {
  float v[2 * N];
#pragma unroll
  for (int n = 0; n < N; ++n) {
    v[2 * n] = hr[n];
    v[2 * n + 1] = hi[n];
  }
  store_state_vec<2 * N>(dst, v);
}

// One lane = one (b, d) channel over one time chunk.  HASZ: gate present.
//   KIND == kReadout:   y and (last chunk) hT
//   KIND == kStateOnly: hT only (y == NULL: C, z, Dskip unread)
//   KIND == kSummary:   chunk end state from zero -> carry slot c+1, sum dt
// At most 168 VGPRs, nothing in scratch: three waves per SIMD, which launches of
// many rounds need.  At two, 256 x 200 x 2048 bf16 takes 800 us, at three 743;
// states of fp32 inputs 706 -> 658; 8 x 16,384 x 2048 in 256-token chunks
// 3910 -> 3590.  Two waves per SIMD that are all resident lose up to 1% to the
// bound (8 x 3000 x 2048 666 -> 670).
template <int N, typename TIn, typename TOut, typename TSt, int KIND, bool HASZ>
__global__ __launch_bounds__(kSBlock) __attribute__((amdgpu_waves_per_eu(3))) void scan_complex_kernel(
    const TIn* __restrict__ xg, const TIn* __restrict__ dtg, const TIn* __restrict__ zg,
    const TIn* __restrict__ Bg, const TIn* __restrict__ Cg, TOut* __restrict__ yg,
    const ScanParams p) {
  constexpr int kPer = N < 16 ? N : 16;
  constexpr bool kRead = KIND == kReadout;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int dblk = lb % p.dblocks;
  const int rest = lb / p.dblocks;
  const int b = rest % static_cast<int>(p.B);
  const int c = rest / static_cast<int>(p.B);
  const int64_t D = p.D;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // its addresses then hold no VGPR
  const int64_t wave_d0 = static_cast<int64_t>(dblk) * p.threads + wave * 64;
  // progress balancing between the two waves of a SIMD (scan_kernels.h)
  const bool fair = balance_enabled(p);
  __shared__ int progress[kSWaves];
  if (fair) balance_init(progress, wave);  // uniform over the workgroup
  if (wave_d0 >= D) return;
  const int64_t dtrue = wave_d0 + lane;
  const bool live = dtrue < D;
  const int64_t d = live ? dtrue : D - 1;

  const int64_t t0 = static_cast<int64_t>(c) * p.chunk;
  const int64_t t1 = min(p.L, t0 + p.chunk);
  const int nsteps = static_cast<int>(t1 > t0 ? t1 - t0 : 0);

  float a2[N], w1[N];
  load_state<N>(a2, p.A + d * N);
  load_state<N>(w1, p.A_im + d * N);
#pragma unroll
  for (int n = 0; n < N; ++n) {
    a2[n] *= -kLog2e;
    w1[n] *= kInv2Pi;
  }
  // carry slots hold (re, im) pairs: [B, C, D, N, 2]
  const int64_t DN2 = 2 * D * N;
  float hr[N], hi[N];
  if constexpr (KIND == kSummary) {
#pragma unroll
    for (int n = 0; n < N; ++n) hr[n] = hi[n] = 0.f;
  } else if (p.nchunks > 1) {
    load_cstate<N>(hr, hi, p.carry + (static_cast<int64_t>(b) * p.nchunks + c) * DN2 + 2 * d * N);
  } else if (p.flags & kHasH0) {
    load_cstate<N>(hr, hi, static_cast<const TSt*>(p.h0) + b * p.h0_stride + 2 * d * N);
  } else {
#pragma unroll
    for (int n = 0; n < N; ++n) hr[n] = hi[n] = 0.f;
  }
  const float dsk = (kRead && (p.flags & kHasD)) ? p.Dskip[d] : 0.f;

  // descriptors over this chunk's rows of x, dt, z, y ([nsteps, D]) and B, C
  // ([nsteps, N]); lane offsets in bytes
  using SI = Stream<TIn>;
  using SO = Stream<TOut>;
  const int64_t row0 = static_cast<int64_t>(b) * p.L + t0;
  const uint32_t in_row = static_cast<uint32_t>(D * sizeof(TIn));
  const uint32_t out_row = static_cast<uint32_t>(D * sizeof(TOut));
  const uint32_t bc_row = static_cast<uint32_t>(N * sizeof(TIn));
  const uint32_t ns = static_cast<uint32_t>(nsteps > 0 ? nsteps : 1);
  const auto rx = make_rsrc(xg + row0 * D, ns * in_row);
  const auto rd = make_rsrc(dtg + row0 * D, ns * in_row);
  const auto rz = make_rsrc(zg + row0 * D, ns * in_row);
  const auto rb = make_rsrc(Bg + row0 * N, ns * bc_row);
  const auto rc = make_rsrc(Cg + row0 * N, ns * bc_row);
  const auto ry = make_rsrc(yg + row0 * D, ns * out_row);
  const uint32_t dl = static_cast<uint32_t>(d) * sizeof(TIn);
  const uint32_t dly = live ? static_cast<uint32_t>(d) * sizeof(TOut) : kDropOffset;
  const int lane16 = lane & 15;
  const uint32_t el = static_cast<uint32_t>(lane16 < N ? lane16 : N - 1) * sizeof(TIn);

  // N = 16: the B (and C) rows of a tile are 32 (16-bit inputs: in lanes l and
  // l + 32, which then do the same) or 64 consecutive dwords, dword l in lane
  // l.  They go as fp32 into a
  // wave-private LDS slice when the tile is consumed and come back as
  // same-address 16-byte reads, as in the real scan: plain operands in place
  // of 32 DPP broadcasts a token, which issue more slowly, and one load per
  // array and tile in place of four.  State-only kinds gain too (without it
  // 8 x 3000 x 2048 643 us, with it 626).  Shorter N keep the broadcasts.
  constexpr bool kLds = N == 16;
  // tokens of a tile: without a readout and LDS the registers allow 8 (N = 4
  // states, 64 x 1000 x 2048: 243 -> 237 us)
  constexpr int kPF = kLds || kRead ? kPFPlain : kPFWide;
  constexpr int kDw = kPF * N * static_cast<int>(sizeof(TIn)) / 4;
  __shared__ __attribute__((aligned(16))) float bc_lds[kLds ? kSWaves : 1][kLds ? kPF : 1][2][kLds ? N : 1];

  struct Tile {
    typename SI::raw x[kPF], dt[kPF], z[kPF], b[kPF], c[kPF];
    uint32_t bw, cw;  // kLds: this lane's dword of the tile's B / C rows
  };
  Tile t0b, t1b;
  const int last = nsteps > 0 ? nsteps - 1 : 0;
  auto fetch = [&](Tile& tb, int tile) {
    if constexpr (kLds) {
      // dwords of tokens past the chunk lie past the range and read as zero
      const uint32_t end = ns * bc_row;
      const uint32_t at = static_cast<uint32_t>(tile) * (kDw * 4u);
      const uint32_t off = 4u * static_cast<uint32_t>(lane % kDw);
      tb.bw = __builtin_amdgcn_raw_buffer_load_b32(rb, off, at < end ? at : end, 0);
      if constexpr (kRead) tb.cw = __builtin_amdgcn_raw_buffer_load_b32(rc, off, at < end ? at : end, 0);
    }
#pragma unroll
    for (int k = 0; k < kPF; ++k) {
      int st = tile * kPF + k;
      st = st < last ? st : last;
      const uint32_t so = static_cast<uint32_t>(st) * in_row;
      tb.x[k] = SI::load(rx, dl, so);
      tb.dt[k] = SI::load(rd, dl, so);
      if constexpr (HASZ) tb.z[k] = SI::load(rz, dl, so);
      if constexpr (!kLds) {
        const uint32_t sb = static_cast<uint32_t>(st) * bc_row;
        tb.b[k] = SI::load(rb, el, sb);
        if constexpr (kRead) tb.c[k] = SI::load(rc, el, sb);
      }
    }
  };
  auto put = [&](uint32_t l, int which, uint32_t w) {
    if constexpr (sizeof(TIn) == 2) {  // token l / 8, coefficients 2 (l mod 8) and the next
      float* dst = &bc_lds[wave][l >> 3][which][2 * (l & 7)];
      dst[0] = __uint_as_float(w << 16);
      dst[1] = __uint_as_float(w & 0xffff0000u);
    } else {
      bc_lds[wave][l >> 4][which][l & 15] = __uint_as_float(w);
    }
  };
  auto stage = [&](const Tile& tb) {
    if constexpr (kLds) {
      // formed anew for each tile: kept, the address is the value that goes to
      // scratch, and reloading it waits for the next tile's loads
      uint32_t l = threadIdx.x;
      asm volatile("" : "+v"(l));
      l %= kDw;
      put(l, 0, tb.bw);
      if constexpr (kRead) put(l, 1, tb.cw);
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the writes are done before any read
    }
  };

  float dtacc = 0.f;
  // Token k of the tile (its registers) and of the staged coefficients (kc),
  // token st of the chunk.
  auto step = [&](const Tile& tb, int k, int kc, int st, auto reduce) {
    constexpr bool kReduce = decltype(reduce)::value;
    const float xv = SI::f32(tb.x[k]);
    const float dtv = SI::f32(tb.dt[k]);
    const float u = dtv * xv;
    float acc = 0.f;
    if constexpr (kLds && kReduce) {
#pragma unroll
      for (int n = 0; n < N; ++n) {
        cstate<true>(hr[n], hi[n], a2[n], w1[n], dtv, u * bc_lds[wave][kc][0][n]);
        if constexpr (kRead) acc = fmaf(bc_lds[wave][kc][1][n], hr[n], acc);
        if (n % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
    } else if constexpr (kLds) {
      float bl[N], cl[N];
#pragma unroll
      for (int n = 0; n < N; ++n) {
        bl[n] = bc_lds[wave][kc][0][n];
        cl[n] = kRead ? bc_lds[wave][kc][1][n] : 0.f;
      }
#pragma unroll
      for (int n = 0; n < N; ++n) {
        cstate<kReduce>(hr[n], hi[n], a2[n], w1[n], dtv, u * bl[n]);
        if constexpr (kRead) acc = fmaf(cl[n], hr[n], acc);
      }
    } else {
      ctoken<kReduce>(hr, hi, a2, w1, dtv, u, SI::f32(tb.b[k]), std::make_integer_sequence<int, kPer>{});
      if constexpr (kRead) readout_group<N, 0>(acc, SI::f32(tb.c[k]), hr);
    }
    if constexpr (kRead) {
      float out = fmaf(dsk, xv, acc);
      if constexpr (HASZ) {
        const float zv = SI::f32(tb.z[k]);
        const float e = __builtin_amdgcn_exp2f(-kLog2e * zv);
        out *= zv * __builtin_amdgcn_rcpf(1.f + e);
      }
      SO::store(ry, dly, static_cast<uint32_t>(st) * out_row, out);
    }
    if constexpr (KIND == kSummary) dtacc += dtv;
  };
  // Largest |w / (2 pi)| of this lane's states (NaN if one is).  Rounding is
  // monotone, so |dt| w_max < 256 bounds every dt w of the tile.
  float w_max = 0.f;
#pragma unroll
  for (int n = 0; n < N; ++n) w_max = __builtin_elementwise_maximum(w_max, fabsf(w1[n]));
  auto run_tile = [&](const Tile& tb, int tile, auto guard) {
    constexpr bool kGuard = decltype(guard)::value;
    stage(tb);
    bool direct = false;
    if constexpr (kLds) {
      float m = 0.f;
#pragma unroll
      for (int k = 0; k < kPF; ++k) m = __builtin_elementwise_maximum(m, fabsf(SI::f32(tb.dt[k])));
      direct = __builtin_amdgcn_ballot_w64(!(m * w_max < 256.f)) == 0;
    }
    if (direct) {
#pragma unroll
      for (int k = 0; k < kPF; ++k) {
        if (kGuard && tile * kPF + k >= nsteps) break;
        step(tb, k, k, tile * kPF + k, std::false_type{});
      }
    } else if constexpr (kLds) {
      // one token per round, so this path needs little code and, with two states
      // at a time (step), few registers: it must not set the kernel's
#pragma unroll 1
      for (int k = 0; k < kPF; ++k) {
        if (kGuard && tile * kPF + k >= nsteps) break;
        Tile tc;
        tc.x[0] = tb.x[0];
        tc.dt[0] = tb.dt[0];
        if constexpr (HASZ) tc.z[0] = tb.z[0];
#pragma unroll
        for (int i = 1; i < kPF; ++i) {
          tc.x[0] = k == i ? tb.x[i] : tc.x[0];
          tc.dt[0] = k == i ? tb.dt[i] : tc.dt[0];
          if constexpr (HASZ) tc.z[0] = k == i ? tb.z[i] : tc.z[0];
        }
        step(tc, 0, k, tile * kPF + k, std::true_type{});
      }
    } else {
#pragma unroll
      for (int k = 0; k < kPF; ++k) {
        if (kGuard && tile * kPF + k >= nsteps) break;
        step(tb, k, k, tile * kPF + k, std::true_type{});
      }
    }
  };
  constexpr std::false_type whole{};
  constexpr std::true_type guarded{};

  if (nsteps > 0) {
    fetch(t0b, 0);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): tile 0 in before tile 1 is requested
    int tile = 0;
    for (; (tile + 2) * kPF <= nsteps; tile += 2) {
      if (fair) balance_step(progress, wave, tile);
      fetch(t1b, tile + 1);
      run_tile(t0b, tile, whole);
      fetch(t0b, tile + 2);
      run_tile(t1b, tile + 1, whole);
    }
    fetch(t1b, tile + 1);
    run_tile(t0b, tile, guarded);
    run_tile(t1b, tile + 1, guarded);
  }

  // the channel once more, so that it holds no registers through the time loop
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int64_t de = wave_d0 + (tid & 63);
  if (de >= D) return;
  if constexpr (KIND == kSummary) {
    store_cstate<N>(p.carry + (static_cast<int64_t>(b) * p.nchunks + c + 1) * DN2 + 2 * de * N, hr,
                    hi);
    p.dtsum[(static_cast<int64_t>(b) * p.nchunks + c) * D + de] = dtacc;
  } else {
    if ((p.flags & kHasHT) && c == p.nchunks - 1)
      store_cstate<N>(static_cast<TSt*>(p.hT) + b * p.hT_stride + 2 * de * N, hr, hi);
  }
}

// Pass 2: per (b, d, n) lane, fold the chunk summaries in time order.
// carry[b, 0] = h0; carry[b, c] = exp(-S_{c-1} (a + i w)) carry[b, c-1]
// + s_{c-1}, where pass 1 left s_{c-1} in carry[b, c] and S_{c-1} in
// dtsum[b, c-1].  The magnitude is exp2(a' S) as in the tokens; the angle
// S w / (2 pi) is formed and reduced to [0, 1) revolutions in fp64 (it
// reaches hundreds of revolutions over a long chunk, where fp32 would keep
// too few fraction bits), then cos / sin as in the tokens.
template <typename TSt>
__global__ __launch_bounds__(256) void complex_carry_kernel(const ScanParams p, int N) {
  const int64_t DN = p.D * N;
  const int64_t gid = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (gid >= p.B * DN) return;
  const int64_t b = gid / DN;
  const int64_t dn = gid - b * DN;
  const int64_t d = dn / N;
  const float a2 = -kLog2e * p.A[dn];
  const double w1 = static_cast<double>(p.A_im[dn]) * 0.15915494309189535;  // 1 / (2 pi)
  float Hr = 0.f, Hi = 0.f;
  if (p.flags & kHasH0) {
    const TSt* src = static_cast<const TSt*>(p.h0) + b * p.h0_stride + 2 * dn;
    Hr = to_f32(src[0]);
    Hi = to_f32(src[1]);
  }
  float* cp = p.carry + b * p.nchunks * 2 * DN + 2 * dn;
  const float* sp = p.dtsum + b * p.nchunks * p.D + d;
  cp[0] = Hr;
  cp[1] = Hi;
  constexpr int kU = 4;
  for (int c0 = 1; c0 < p.nchunks; c0 += kU) {
    float sr[kU], si[kU], Sv[kU];
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      if (c0 + k < p.nchunks) {
        sr[k] = cp[(c0 + k) * 2 * DN];
        si[k] = cp[(c0 + k) * 2 * DN + 1];
        Sv[k] = sp[(c0 + k - 1) * p.D];
      }
    }
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      if (c0 + k < p.nchunks) {
        const double turns = static_cast<double>(Sv[k]) * w1;
        const float rev = static_cast<float>(turns - floor(turns));
        const float mag = __builtin_amdgcn_exp2f(a2 * Sv[k]);
        const float cs = mag * __builtin_amdgcn_cosf(rev);
        const float sn = mag * __builtin_amdgcn_sinf(rev);
        const float re = Hr;
        Hr = fmaf(cs, re, fmaf(sn, Hi, sr[k]));
        Hi = fmaf(cs, Hi, fmaf(-sn, re, si[k]));
        cp[(c0 + k) * 2 * DN] = Hr;
        cp[(c0 + k) * 2 * DN + 1] = Hi;
      }
    }
  }
}

template <int N, typename TIn, typename TOut, typename TSt>
hipError_t launch_c(const ScanParams& p, hipStream_t s) {
  const int64_t rows_blocks = static_cast<int64_t>(p.dblocks) * p.B;
  const TIn* X = static_cast<const TIn*>(p.x);
  const TIn* DT = static_cast<const TIn*>(p.dt);
  const TIn* Z = static_cast<const TIn*>(p.z);
  const TIn* BB = static_cast<const TIn*>(p.Bm);
  const TIn* CC = static_cast<const TIn*>(p.Cm);
  if (p.nchunks > 1) {
    const dim3 g1(static_cast<unsigned>(rows_blocks * (p.nchunks - 1)));
    hipLaunchKernelGGL((scan_complex_kernel<N, TIn, float, float, kSummary, false>), g1,
                       dim3(p.threads), 0, s, X, DT, Z, BB, CC, static_cast<float*>(nullptr), p);
    const int64_t lanes = p.B * p.D * N;
    hipLaunchKernelGGL((complex_carry_kernel<TSt>), dim3(static_cast<unsigned>((lanes + 255) / 256)),
                       dim3(256), 0, s, p, N);
  }
  const dim3 grid(static_cast<unsigned>(rows_blocks * p.nchunks));
  if (p.y != nullptr && (p.flags & kHasZ))
    hipLaunchKernelGGL((scan_complex_kernel<N, TIn, TOut, TSt, kReadout, true>), grid, dim3(p.threads),
                       0, s, X, DT, Z, BB, CC, static_cast<TOut*>(p.y), p);
  else if (p.y != nullptr)
    hipLaunchKernelGGL((scan_complex_kernel<N, TIn, TOut, TSt, kReadout, false>), grid,
                       dim3(p.threads), 0, s, X, DT, Z, BB, CC, static_cast<TOut*>(p.y), p);
  else
    hipLaunchKernelGGL((scan_complex_kernel<N, TIn, float, TSt, kStateOnly, false>), grid,
                       dim3(p.threads), 0, s, X, DT, Z, BB, CC, static_cast<float*>(nullptr), p);
  return hipGetLastError();
}

template <int N, typename TIn, typename TOut>
hipError_t c_state(const ScanParams& p, int state_dtype, hipStream_t s) {
  return state_dtype == 0 ? launch_c<N, TIn, TOut, float>(p, s) : launch_c<N, TIn, TOut, f16_t>(p, s);
}

template <int N, typename TIn>
hipError_t c_out(const ScanParams& p, int out_dtype, int state_dtype, hipStream_t s) {
  return out_dtype == 0 ? c_state<N, TIn, float>(p, state_dtype, s)
                        : c_state<N, TIn, bf16_t>(p, state_dtype, s);
}

template <int N>
hipError_t c_in(const ScanParams& p, int in_dtype, int out_dtype, int state_dtype, hipStream_t s) {
  return in_dtype == 0 ? c_out<N, float>(p, out_dtype, state_dtype, s)
                       : c_out<N, bf16_t>(p, out_dtype, state_dtype, s);
}

}  // namespace

hipError_t launch_scan_complex(const ScanParams& p, int N, int in_dtype, int out_dtype,
                               int state_dtype, hipStream_t s) {
  switch (N) {
    case 1: return c_in<1>(p, in_dtype, out_dtype, state_dtype, s);
    case 2: return c_in<2>(p, in_dtype, out_dtype, state_dtype, s);
    case 4: return c_in<4>(p, in_dtype, out_dtype, state_dtype, s);
    case 8: return c_in<8>(p, in_dtype, out_dtype, state_dtype, s);
    case 16: return c_in<16>(p, in_dtype, out_dtype, state_dtype, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace precog
